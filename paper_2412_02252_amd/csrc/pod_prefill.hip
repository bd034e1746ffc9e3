// Prefill attention for PoD: causal flash attention on bf16 MFMA with two logit sources.
//
// For query i and key j <= i (Eq. 3 of the paper with the window taken at the query's own
// position): j is proximal if j < S or j > i - W and its logit is q_l[i].k_l[j]; otherwise it is
// distant and its logit is the block's lowest layer's, q_a[i].k_a[j].  One softmax over all
// j <= i (Eq. 4 / appendix), values always v_l.
//
// Because a softmax accumulates in any order, the key loop runs in two phases, each with ONE
// query operand in registers and ONE key source:
//   phase D (upper layers only): key tiles that hold a distant key for some row of the
//            workgroup, with q_a and k_a; elements that are not distant for their row are masked;
//   phase P: sink tiles and band tiles, with q_l and k_l; elements that are not proximal (or not
//            causal) are masked.
// A tile that straddles a region edge is visited by both phases with complementary masks (its V
// tile is loaded twice: ~4 of 256 tiles per row block at the paper's window sizes).  At the
// block's lowest layer there is only phase P over all tiles, with the causal mask.
//
// Tiling: a workgroup of 4 waves takes 128 query rows of one head, 32 rows per wave; key/value
// tiles of 64 tokens go through LDS (KS = 2: eight waves, two key groups that take every second key tile of the same rows and
// are merged at the end: prefill_key_groups).
//   S^T[key][row] = K[key][:] . Q[row][:]     v_mfma_f32_32x32x16_bf16, A = K fragment, B = Q
//   O^T[dim][row] = sum_key V[key][dim] P[key][row]               A = V^T fragment, B = P
// Query row = MFMA column (lane % 32) in both, so softmax state, P and the output slice of a
// row stay in the same lane, and the S^T accumulators become the P operand without moving: the
// 8 keys a lane holds for one PV k-step are the keys of its 8 consecutive accumulators (tokens
// 16 ks + 4 (lane / 32) + {0..3} and + 8 of the tile), and the V^T fragments are read for that order.
//
// Softmax: base-2 with the logit scale folded into the exponent; the reference maximum is only
// moved when a tile exceeds it by more than 2^8 (probabilities then stay below 256, harmless in
// fp32 sums and in bf16), which removes most rescaling passes over the output accumulators.
#include <stdlib.h>
#include <mutex>
#include <type_traits>
#include <utility>

#include "pod_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;

constexpr int kBN = 64;
constexpr float kNegBig = -1.0e30f;
constexpr int kPF = 2;        // LDS fragment reads in flight ahead of the MFMA that uses them (1 is slower, 3 no faster)
constexpr float kLazy = 8.0f; // how far (log2) a tile's maximum may exceed the reference before rescaling

struct prefill_params {
    int n, Hq, Hkv, rep, S, W;
    int q0; // position of the first query row: q, qs and out hold rows q0 .. n-1 (k, v, ks hold 0 .. n-1)
    const pod_bf16 *q, *k, *v, *qs, *ks; // qs/ks NULL: own q,k serve every key
    pod_bf16 *out;
    float scale_log2e;
    unsigned long long lowest_mask; // bit h: kv head h takes every logit from (q, k) even if qs/ks are given
    // TAB kernels: k, v, ks are not used.  tile_tab[(stream * Hkv + kv head) * ntiles + key tile] is the device
    // address of that tile's first row for that head, rows D * 2 bytes apart; stream 0 = k, 1 = v, 2 = ks
    const unsigned long long *tile_tab;
    int ntiles;
    // TAB kernels also finish the cache update that wrote the table: if *len still is len_old it becomes len_new,
    // else *flag is raised (the update kernel made the same test and stored nothing)
    int *len, *flag;
    int len_old, len_new;
    // workgroups fill_lo .. fill_lo + fill_n - 1 of the launch store the prompt's k and v in the cache (none: fill_n = 0)
    int fill_lo, fill_n;
    // launches of one round: from this workgroup on (counted per kv head) the query tiles come in the opposite order
    int turn, per_kvh;
    pod_fill_args fill;
};

// The key tiles that query rows i0 .. i_last walk, in order: nD tiles from tD0 (phase D), nP1 sink tiles from 0, band tiles from tB.
struct tile_list { int tD0, nD, nP1, tB, count; };
__host__ __device__ inline tile_list tiles_of_rows(int i0, int i_last, int S, int W, bool has_shared)
{
    tile_list t = {0, 0, 0, 0, 0};
    if (has_shared) {
        if (i_last - W >= S) { t.tD0 = S / kBN; t.nD = (i_last - W) / kBN - t.tD0 + 1; }
        if (S > 0) t.nP1 = ((S < i_last + 1 ? S : i_last + 1) - 1) / kBN + 1;
        const int band = i0 - W + 1 > 0 ? (i0 - W + 1) / kBN : 0;
        t.tB = t.nP1 > band ? t.nP1 : band;
    }
    const int tEnd = i_last / kBN;
    t.count = t.nD + t.nP1 + (tEnd >= t.tB ? tEnd - t.tB + 1 : 0);
    return t;
}

__device__ inline bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ inline unsigned pack_bf16(float lo, float hi)
{
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    bf16x2 t = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(unsigned, t);
}

// Exchange between the two lanes (l, l ^ 32) that share a query row: v_permlane32_swap gives
// lane l its partner's value in one of the two results.  Operands and results go through empty
// asm statements: given the same value twice the compiler otherwise folds max(r0, r1) to r0.
__device__ inline void pair_exchange(float x, float &mine_or_partner0, float &mine_or_partner1)
{
    unsigned a = __builtin_bit_cast(unsigned, x), b = a;
    asm volatile("" : "+v"(b));
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    unsigned r0 = r[0], r1 = r[1];
    asm volatile("" : "+v"(r0), "+v"(r1)); // (the two results are not interchangeable either)
    mine_or_partner0 = __builtin_bit_cast(float, r0);
    mine_or_partner1 = __builtin_bit_cast(float, r1);
}
__device__ inline float pair_max(float x)
{
    float a, b;
    pair_exchange(x, a, b);
    return fmaxf(a, b);
}
__device__ inline float pair_sum(float x)
{
    float a, b;
    pair_exchange(x, a, b);
    return a + b;
}

// ---------------------------------------------------------------------------------------------
// Order of work inside a wave (software pipeline over three tiles).
//
// Measured on gfx950: a wave issues roughly one vector instruction per 5-6 cycles, a 32x32x16
// MFMA keeps the matrix pipe busy for 32 cycles, and with two waves per SIMD the pipe only
// stays busy if each wave brings at most ~3 ordinary vector instructions, one transcendental
// and one or two LDS reads per MFMA (a synthetic loop of that mix: 17-18 ns per MFMA, 14 without any of it).  So an iteration is a sequence of MFMA slots of that shape,
// taken from three different tiles:
//   iteration t:  S(t+1) = K(t+1) Q^T        (logits of the next tile)
//                 O += V(t-1)^T P(t-1)       (output update of the previous tile)
//                 P(t) = exp2(c S(t) - m)    one pair of elements per slot or two
//                 row maximum of S(t+1); one barrier.
// No exponential waits for an MFMA of the same iteration.  Slot order: the 2:1 mix QK, QK, PV
// for the first three quarters of the slots (all of S(t+1) is then complete), PV only in the
// last quarter, where the vector work is the row maximum of S(t+1).  It is needed at the top of
// the next iteration, which moves the reference maximum if the tile exceeds it by more than 2^8
// and rescales the accumulators (rare).  Masked logits are -infinity (exponential 0 whatever the
// reference); every wave walks every tile of its workgroup.  The row sum adds the bf16-rounded
// probabilities (add_four), i.e. exactly the weights the PV product uses.
//
// Data movement uses no registers: K and V tiles go from global memory straight into LDS
// (global_load_lds_dwordx4: each wave instruction fills 1 KB of consecutive LDS, lane l its 16
// bytes; which 16 bytes of the tile a lane fetches is free to choose).
// Both slots are row-major [64 tokens][D] as in global memory, so a wave instruction fetches whole
// rows (256 consecutive bytes per row at D = 128: fully coalesced requests); only the order of the
// 16-byte pieces inside a row is permuted, differently for the two readers:
//   K slot: piece c of row r sits at piece c ^ krot(r), krot(r) = (r D / 128) mod (D / 8).  The B
//           operand of the QK product (one key row, 8 dims per lane) is one ds_read_b128; the 16 rows
//           that such a read touches at once hit 16 different 16-byte bank groups.
//   V slot: 16-byte pieces of a row XOR-permuted by
//           4 (token % 4).  The A operand of the PV product (V^T: one dim, 8 tokens per lane) comes
//           out of two ds_read_b64_tr_b16 (the LDS transpose read: inside 16 lanes, lane L receives
//           element L % 4 of the four 8-byte rows addressed by lanes L / 4 + {0, 4, 8, 12}).
// K(t+2) and V(t) are requested at the start of iteration t into the slots freed by the barrier
// before, and awaited (vmcnt) before the barrier that ends the iteration; their addresses are computed at the end of iteration t-1.
// static_for<N>(f): f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>), each call its own
// instantiation with a compile-time index (no reliance on the loop unroller for big bodies)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Every element of acc plus the lane's own four bf16 values: in v_mfma_f32_4x4x4_16b_bf16 a lane holds one column of its block's
// B operand, four values of k, and with ones for A every row of that column of the result is their sum.
// (v_dot2c_f32_bf16, which this took before, does not run beside the matrix pipe as the other vector instructions do: synthetic loops,
// two waves per SIMD, 14 ns per 32x32x16 MFMA alone and with four v_fma_f32 beside it, 22 with two dot products; the whole mix of an
// iteration 17.5 -> 17.1 ns per MFMA, against 18.4 with the pairs taken apart and added.  16384 tokens x 32/8 heads x 128 4132 -> 4000 us.)
__device__ inline f32x4 add_four(u32x2 v, f32x4 acc)
{
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, v), acc, 0, 0, 0);
}

// 16 bytes per lane from base + off (off per lane) straight into LDS: lane l's go to LDS address dst + 16 l (dst the same in every lane).
// Written as the instruction itself and waited for by hand (vmcnt), because the compiler, which cannot tell the slots apart, puts a
// wait for ALL outstanding loads into LDS in front of the next transposing LDS read: every tile then stood still for the whole
// latency of the loads it had just requested.  A load into LDS has no destination register; M0 is declared as changed, which costs nothing
// since nothing else in these kernels uses it.  Both layers of a request, before -> after (kernels alone, us): 16384 tokens x 32/8 heads x 128 4350 -> 4130,
// 3001 x 16/4 x 64 84.4 -> 80.0, 777 x 32/8 x 128 48.1 -> 46.9.
typedef const __attribute__((address_space(1))) char *gbyte_ptr;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm" // (M0 is reserved, i.e. never allocated, which is no reason not to name it here)
__device__ __forceinline__ void load_lds16(gbyte_ptr base, unsigned off, unsigned dst)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(off), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop

template <int D, bool TAB, int KS>
__global__ __launch_bounds__(256 * KS, 2) void prefill_kernel(prefill_params p)
{
    constexpr int CPR = D / 8, KST = D / 16, NDB = D / 32, NKB = kBN / 32, NPS = kBN / 16;
    constexpr int BM = 128;
    // Where a tile's requests are issued.  All at once at the top of an iteration, next to another workgroup that multiplies meanwhile; one
    // in each of the first slots where the eight waves of a CU belong to one workgroup and would all stand still for them (777 tokens x 32/8
    // heads x 128, both layers 44.6 -> 43.6 us; with one key group it is the other way round, 16384 tokens 4050 -> 4074).
    constexpr bool SPREAD = KS == 2;
    constexpr int NQK = NKB * KST;   // MFMAs of one S tile = K fragments of a tile
    constexpr int NPV = NDB * NPS;   // MFMAs of one PV tile (equal to NQK)
    static_assert(NQK == NPV, "slot schedule assumes as many QK as PV MFMAs per tile");
    typedef const __attribute__((address_space(1))) u32x4 *gvec_ptr;
    typedef __attribute__((address_space(3))) char *lbyte_ptr;
    typedef __attribute__((ext_vector_type(4))) short s16x4;
    typedef __attribute__((address_space(3))) s16x4 *ltr_ptr;
    constexpr int FRAG = 64 * 16;
    constexpr int KBUF = NQK * FRAG, VBUF = kBN * D * 2; // 16 KB each at D = 128
    extern __shared__ __attribute__((aligned(16))) char lds[];   // per key group: [K slot 0][K slot 1][V slot 0][V slot 1]

    const int nqt = (p.n + BM - 1) / BM;
    int wg = blockIdx.x;
    if (!TAB && wg >= p.fill_lo) {
        wg -= p.fill_n;
        if (wg < p.fill_lo) { // cache construction: nothing here reads what it writes
            pod_fill_rows<kFillUnroll>(p.fill, p.k, p.v, (size_t)(wg + p.fill_n - p.fill_lo) * blockDim.x + threadIdx.x, (size_t)p.fill_n * blockDim.x);
            return;
        }
    }
    const int kvh = wg % p.Hkv;
    int rest = wg / p.Hkv;
    if (rest >= p.turn) rest = p.turn + p.per_kvh - 1 - rest;
    const int head = kvh * p.rep + rest % p.rep;
    // Query tiles are handed out from the last, which has most keys, to the first; where every workgroup has its place from the
    // start, the second workgroup of a CU comes from the other end of the list: a workgroup alone on its CU takes about 1.2 us per key
    // tile, two together 1.5 to 2 each, so the longest gets the shortest beside it (8192 tokens in chunks of 2048 x 32/8 heads
    // x 128, 512 workgroups of 98 to 128 key tiles in the last chunk: 1234 -> 1211 us per request of two layers).
    const int qt = nqt - 1 - rest / p.rep;
    const int i0 = qt * BM;
    const int i_last = min(i0 + BM, p.n) - 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3; // (a scalar: what depends on the wave alone stays out of the vector pipe)
    const int grp = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8); // key group: waves 4 grp .. 4 grp + 3
    char *const ldsK = lds + grp * (2 * KBUF + 2 * VBUF), *const ldsV = ldsK + 2 * KBUF;
    const int n32 = lane & 31, jj = lane >> 5;
    const int iw0 = i0 + wave * 32;
    const int iw_last = min(iw0 + 32, p.n) - 1;
    const int irow = iw0 + n32;
    const bool has_shared = p.qs != nullptr && !((p.lowest_mask >> kvh) & 1);
    const int S = p.S, W = p.W;
    const float c = p.scale_log2e;

    const tile_list tl = tiles_of_rows(i0, i_last, S, W, has_shared);
    const int tD0 = tl.tD0, nD = tl.nD, nP1 = tl.nP1, tB = tl.tB, Tall = tl.count;
    const int T = (Tall + KS - 1) / KS; // tiles of a key group: group g walks tiles g, g + KS, ... of the list
    auto tile_of = [&](int u, int &kt, bool &phaseD) __attribute__((always_inline)) {
        const int t = KS == 1 ? u : min(u * KS + grp, Tall - 1); // (past the end: the last tile again; mask_tile leaves nothing of it)
        phaseD = t < nD;
        kt = t + (phaseD ? tD0 : (t < nD + nP1 ? -nD : tB - nD - nP1));
    };

    // ---- global -> LDS.  Wave w moves K fragments w*NQK/4 .. and the V rows w*16 .. w*16+15.
    constexpr int VRI = 64 / CPR;                // V rows per wave instruction (1 KB)
    constexpr int VPW = 16 / VRI;                // V instructions per wave and tile
    constexpr int VSWZ = 4 * ((CPR / 4 - 1) & 3); // piece-permutation mask: 12 at D = 128, 4 at D = 64
    // A request is ONE scalar base per tile plus a per-lane offset that never changes (one register per
    // request of the wave), so a tile costs neither vector nor scalar address arithmetic; only the
    // prompt's last, partly filled tile takes a separate path that clamps its rows per lane.
    const unsigned rowb = TAB ? (unsigned)(D * 2) : (unsigned)p.Hkv * D * 2; // TAB: one head's rows, back to back
    const unsigned head_col = TAB ? 0u : (unsigned)(kvh * D * 2);
    typedef const __attribute__((address_space(4))) unsigned long long *tab_ptr;  // read with scalar loads
    const tab_ptr tab_k = (tab_ptr)(p.tile_tab + (size_t)kvh * p.ntiles);
    const size_t tab_stream = (size_t)p.Hkv * p.ntiles;
    const int v_r = lane / CPR;                                         // row inside a V instruction
    // K rows: a lane of a request fetches piece (slot piece ^ krot(row)) of its row, krot(row) = row * CPR / 16 mod CPR
    // (16 consecutive rows then put the same piece into 16 different 16-byte bank groups)
    auto k_col = [&](int x) { // x-th request of the wave: LDS rows 16 wave + VRI x + v_r
        const int rot = (((VRI * x + v_r) * CPR) / 16) & (CPR - 1);
        return head_col + (unsigned)(16 * ((lane % CPR) ^ rot));
    };
    const unsigned v_col = head_col + (unsigned)(16 * ((lane % CPR) ^ ((4 * (v_r & 3)) & VSWZ)));
    unsigned k_off[VPW], v_off[VPW];
#pragma unroll
    for (int x = 0; x < VPW; ++x) {
        v_off[x] = (unsigned)(16 * wave + VRI * x + v_r) * rowb + v_col;
        k_off[x] = (unsigned)(16 * wave + VRI * x + v_r) * rowb + k_col(x);
    }
    const unsigned k_dst0 = (unsigned)(uintptr_t)(lbyte_ptr)lds + grp * (2 * KBUF + 2 * VBUF) + wave * (16 * D * 2); // this wave's part of K slot 0
    const unsigned v_dst0 = k_dst0 + 2 * KBUF;                                                                        // ... of V slot 0
    // TAB: the tile's address comes out of the table with a scalar load; the callers fetch it an iteration ahead
    auto k_tile = [&](int kt, bool phaseD) __attribute__((always_inline)) { return tab_k[(phaseD ? 2 * tab_stream : 0) + kt]; };
    auto v_tile = [&](int kt) __attribute__((always_inline)) { return tab_k[tab_stream + kt]; };
    // a tile's requests: its scalar base first, then one request after the other
    const unsigned tile_bytes = kBN * rowb;
    auto k_base = [&](int kt, bool phaseD, unsigned long long tile) __attribute__((always_inline)) {
        if constexpr (TAB) return (gbyte_ptr)tile;
        else return (gbyte_ptr)(phaseD ? p.ks : p.k) + (unsigned long long)(unsigned)kt * tile_bytes;
    };
    auto v_base = [&](int kt, unsigned long long tile) __attribute__((always_inline)) {
        if constexpr (TAB) return (gbyte_ptr)tile;
        else return (gbyte_ptr)p.v + (unsigned long long)(unsigned)kt * tile_bytes;
    };
    // (the lambdas are forced inline: one that becomes a function takes its captures through scratch memory)
    auto request_k = [&](gbyte_ptr base, int slot, int x) __attribute__((always_inline)) {
        load_lds16(base, k_off[x], k_dst0 + slot * KBUF + x * (VRI * D * 2));
    };
    auto request_v = [&](gbyte_ptr base, int slot, int x) __attribute__((always_inline)) {
        load_lds16(base, v_off[x], v_dst0 + slot * VBUF + x * (VRI * D * 2));
    };
    // the prompt's last, partly filled tile: lanes past the end fetch its last row
    auto request_k_part = [&](gbyte_ptr base, int slot, int rows) __attribute__((always_inline)) {
        asm volatile("" ::: "memory"); // (keeps this a real branch: merged, both paths would pay for the clamping)
#pragma unroll
        for (int x = 0; x < VPW; ++x)
            load_lds16(base, (unsigned)min(16 * wave + VRI * x + v_r, rows - 1) * rowb + k_col(x), k_dst0 + slot * KBUF + x * (VRI * D * 2));
    };
    auto request_v_part = [&](gbyte_ptr base, int slot, int rows) __attribute__((always_inline)) {
        asm volatile("" ::: "memory");
#pragma unroll
        for (int x = 0; x < VPW; ++x)
            load_lds16(base, (unsigned)min(16 * wave + VRI * x + v_r, rows - 1) * rowb + v_col, v_dst0 + slot * VBUF + x * (VRI * D * 2));
    };
    auto request_tile_k = [&](int kt, bool phaseD, int slot, unsigned long long tile) __attribute__((always_inline)) {
        const gbyte_ptr base = k_base(kt, phaseD, tile);
        if (__builtin_expect(kt * kBN + kBN <= p.n, 1)) {
#pragma unroll
            for (int x = 0; x < VPW; ++x) request_k(base, slot, x);
        } else request_k_part(base, slot, p.n - kt * kBN);
    };
    // read offsets: K fragment lane slot; V^T transpose-read source row/piece of this lane
    // K fragment (key block kb, k-step s): lane (row n32, jj) reads piece 2 s + jj of row 32 kb + n32, stored at
    // piece (2 s + jj) ^ krot(row) = (jj ^ krot) ^ 2 s; krot(32 kb + n32) = krot(n32)
    const int k_rot = ((n32 * CPR) / 16) & (CPR - 1);
    const int k_rd0 = n32 * (D * 2) + 16 * (jj ^ k_rot);
    const int v_s = lane & 15;
    // row 4 jj + s/4 of the 16-token k-step (+8 for the second read), dims 16 ((lane/16) & 1) + 4 (s % 4) of the
    // 32-dim block db; the piece index is XORed with 4 (row % 4) = 4 (s / 4), the dim block enters as XOR 64 db
    const int v_rd0 = (4 * jj + (v_s >> 2)) * (D * 2) + ((64 * (v_s >> 2)) & (16 * VSWZ)) + 32 * ((lane >> 4) & 1) + 8 * (v_s & 3);
    int v_rd[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db) v_rd[db] = v_rd0 ^ (64 * db);

    bf16x8 qf[KST];
    auto load_q = [&](const pod_bf16 *src) __attribute__((always_inline)) {
        int row = irow, half = jj;
        // (with two key groups the own query's address, kept from the start to the phase change, does not fit the registers: computed again.
        // 777 tokens x 32/8 heads x 128, lowest / upper layer 19.4 / 24.7 -> 18.8 / 24.1 us)
        if constexpr (KS == 2) asm volatile("" : "+v"(row), "+v"(half));
        const gvec_ptr qr = (gvec_ptr)(src + ((size_t)(max(min(row, p.n - 1), p.q0) - p.q0) * p.Hq + head) * D);
#pragma unroll
        for (int s = 0; s < KST; ++s) qf[s] = as_bf16x8(qr[2 * s + half]);
#pragma unroll
        for (int s = 0; s < KST; ++s) asm volatile("" : "+v"(qf[s])); // awaited here, not wherever the paths with and without the load meet
    };

    // Boundary tiles: -infinity on the logits that are not this phase's to count.  A lane's 32 logits of a tile are keys
    // j0 + 4 jj + {8 (b >> 2) + (b & 3)}, b = 16 kb + r, ascending in b, and what counts is an interval (or causal keys
    // without an interval), so one bit mask per tile says it all: two vector instructions per logit (bit out of the mask,
    // select by it) instead of the five to seven that comparing every key's position took (upper layers' launches at n = 777,
    // 32 heads x 128, window 256: 39.3 -> 29.9 us; n = 2048: 75.1 -> 66.4).
    auto first_bits = [&](int x) __attribute__((always_inline)) { // mask of the elements b with key offset 8 (b >> 2) + (b & 3) <= x
        const int cnt = x < 0 ? 0 : x > 63 ? 32 : 4 * (x >> 3) + min((x & 7) + 1, 4);
        return (unsigned)((1ull << cnt) - 1);
    };
    auto mask_tile = [&](int u, int kt, bool phaseD, f32x16 (&sc)[NKB]) __attribute__((always_inline)) { // u-th tile of the wave's key group
        const int j0 = kt * kBN, j1 = j0 + kBN - 1;
        bool full; // every (row, key) pair of the wave counts: no masking needed
        if (phaseD) full = j0 >= S && j1 <= iw0 - W;
        else if (has_shared) full = j1 <= iw0 && (j1 < S || j0 > iw_last - W);
        else full = j1 <= iw0;
        // A wave whose rows all lie past the prompt stores nothing, so it masks nothing either: the 32 compares and selects
        // per tile it would spend hold up the three other waves at every barrier, and that in the workgroups with most keys
        // (lowest layer, n = 3001, 16 heads x 64: 111.5 -> 54.2 us; n = 777, 32 heads x 128: 40.3 -> 27.6 us).
        if (KS > 1) full = full && u * KS + grp < Tall;
        if (full || iw0 > iw_last) return;
        const int base = j0 + 4 * jj;
        const unsigned distant = first_bits(irow - W - base) & ~first_bits(S - 1 - base);
        unsigned ok = phaseD ? distant : first_bits(irow - base) & ~(has_shared ? distant : 0u);
        if (KS > 1 && u * KS + grp >= Tall) ok = 0u;
#pragma unroll
        for (int b = 0; b < NKB * 16; ++b) {
            const int keep = __builtin_amdgcn_sbfe((int)ok, b, 1); // all ones / zeros
            const float logit = sc[b >> 4][b & 15]; // (a bit cast of the vector element itself reads element 0)
            const int x = __builtin_bit_cast(int, logit);
            sc[b >> 4][b & 15] = __builtin_bit_cast(float, (keep & x) | (~keep & (int)0xff800000));
        }
    };

    f32x16 oacc[NDB];
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
    float m_ref = kNegBig, l_run = 0.f;

    auto kfrag = [&](const char *kl, int op) __attribute__((always_inline)) { // QK MFMA number op: the two key blocks alternate
        const int s = op / NKB, kb = op % NKB;
        return *(const u32x4 *)(kl + kb * 32 * (D * 2) + (k_rd0 ^ (32 * s)));
    };
    auto vfrag = [&](const char *vl, int m) __attribute__((always_inline)) {  // PV MFMA number m = ks * NDB + db
        const int ks = m / NDB, db = m % NDB;
        const lbyte_ptr a = (lbyte_ptr)(vl + ks * 16 * (D * 2)) + v_rd[db];
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ltr_ptr)a);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((ltr_ptr)(a + 8 * (D * 2)));
        u32x4 r;
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        r.x = l2.x; r.y = l2.y; r.z = h2.x; r.w = h2.y;
        return r;
    };

    f32x16 sA[NKB], sB[NKB];
    u32x4 pA[NPS], pB[NPS];
    float mx_next; // scaled row maximum of the tile the next iteration exponentiates

    // ---- prologue: K(0), K(1) in LDS, S(0) and its row maximum computed
    // tiles t, t+1, t+2 of the current iteration (key tile index, phase); shifted along at its end
    int kt_a, kt_b, kt_c;
    bool ph_a, ph_b, ph_c;
    tile_of(0, kt_a, ph_a);
    tile_of(1, kt_b, ph_b);
    tile_of(2, kt_c, ph_c);
    unsigned long long k_next = 0, v_next = 0; // TAB: addresses of the tiles the next iteration requests
    if constexpr (TAB) {
        if (wg == 0 && threadIdx.x == 0) { // the update launch before this one left the length for here
            if (*p.len == p.len_old) *p.len = p.len_new;
            else atomicOr(p.flag, 1);
        }
        request_tile_k(kt_a, ph_a, 0, k_tile(kt_a, ph_a));
        if (T > 1) request_tile_k(kt_b, ph_b, 1, k_tile(kt_b, ph_b));
        if (T > 2) k_next = k_tile(kt_c, ph_c);
        v_next = v_tile(kt_a);
    } else {
        request_tile_k(kt_a, ph_a, 0, 0);
        if (T > 1) request_tile_k(kt_b, ph_b, 1, 0);
    }
    load_q(ph_a ? p.qs : p.q);
    gbyte_ptr kb_next = k_base(kt_c, ph_c, k_next), vb_next = v_base(kt_a, v_next); // what the next iteration requests
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) sA[kb][r] = 0.f;
#pragma unroll
        for (int op = 0; op < NQK; ++op) {
            const int s = op / NKB, kb = op % NKB;
            sA[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(kfrag(ldsK, op)), qf[s], sA[kb], 0, 0, 0);
        }
        mask_tile(0, kt_a, ph_a, sA);
        float mx = -__builtin_inff();
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sA[kb][r]);
        mx_next = pair_max(mx) * c;
    }
    __syncthreads(); // every wave is done reading K(0): iteration 0 overwrites its slot

    // one iteration: FIRST has no PV slots (there is no earlier tile)
    auto iteration = [&](auto first_tag, auto slot_tag, int t, f32x16 (&sc)[NKB], f32x16 (&sn)[NKB], u32x4 (&pprev)[NPS], u32x4 (&pcur)[NPS]) {
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr int slot = decltype(slot_tag)::value; // = t % 2: every LDS address below is a compile-time offset
        const char *kl = ldsK + (slot ^ 1) * KBUF;   // K(t+1)
        const char *vl = ldsV + (slot ^ 1) * VBUF;   // V(t-1)
        // slot list: entry >= 0 is QK MFMA number entry, entry < 0 is PV MFMA number -1 - entry
        constexpr int NS = FIRST ? NQK : NQK + NPV;
        constexpr int NMIX = FIRST ? NQK : NQK + NQK / 2; // slots of the QK, QK, PV mix
        auto slot_op = [](int i) constexpr { return FIRST ? i : (i < NMIX ? ((i % 3 == 2) ? -1 - i / 3 : i - i / 3) : -1 - (i - NQK)); };
        auto frag = [&](int i) { const int op = slot_op(i); return op >= 0 ? kfrag(kl, op) : vfrag(vl, -1 - op); };
        u32x4 fr[NS];
        float tt[16][2], ee[16][2]; // staged softmax values (each lives for one slot)
        float mxv[4] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < kPF && i < NS; ++i) fr[i] = frag(i);
        __builtin_amdgcn_sched_barrier(0);
        // K(t+2) replaces K(t) and V(t) replaces V(t-2), both last read before the previous barrier.  (The first fragments are requested
        // ahead of these, so that their way through the LDS overlaps them.)
        bool more_k = t + 2 < T, more_v = true;
        if (more_k) {
            if (__builtin_expect(kt_c * kBN + kBN > p.n, 0)) { request_k_part(kb_next, slot, p.n - kt_c * kBN); more_k = false; }
            else if constexpr (!SPREAD)
#pragma unroll
                for (int x = 0; x < VPW; ++x) request_k(kb_next, slot, x);
        }
        if (__builtin_expect(kt_a * kBN + kBN > p.n, 0)) { request_v_part(vb_next, slot, p.n - kt_a * kBN); more_v = false; }
        else if constexpr (!SPREAD)
#pragma unroll
            for (int x = 0; x < VPW; ++x) request_v(vb_next, slot, x);
        if (mx_next > m_ref + kLazy) { // (rows with nothing valid so far have mx = -inf and never trigger)
            // The reference moves before tile t is exponentiated: everything computed with the old one is brought
            // to the new one.  That is the row sum, the output accumulators (tiles <= t-2), and P(t-1), whose
            // product with V(t-1) is still to come in this iteration's PV slots.
            const float alpha = __builtin_amdgcn_exp2f(m_ref - mx_next);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
            if constexpr (!FIRST) {
#pragma unroll
                for (int ks = 0; ks < NPS; ++ks)
#pragma unroll
                    for (int w = 0; w < 4; ++w) {
                        const unsigned pk = pprev[ks][w];
                        const float lo = __builtin_bit_cast(float, pk << 16), hi = __builtin_bit_cast(float, pk & 0xffff0000u);
                        pprev[ks][w] = pack_bf16(lo * alpha, hi * alpha);
                    }
            }
            m_ref = mx_next;
        }
        if (__builtin_expect(ph_a && !ph_b, 0)) load_q(p.q); // the next tile is the first of the own-key phase
        const float mr = m_ref;
        f32x4 lsum = {0.f, 0.f, 0.f, 0.f}; // this tile's row sum, four times
        __builtin_amdgcn_sched_barrier(0);
        static_for<NS>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (!FIRST && i == NMIX) {
                mask_tile(t + 1, kt_b, ph_b, sn); // boundary tiles only; S(t+1) is complete here
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (i + kPF < NS) fr[i + kPF] = frag(i + kPF);
            if constexpr (SPREAD && i < VPW) if (more_v) request_v(vb_next, slot, i);
            if constexpr (SPREAD && i >= VPW && i < 2 * VPW) if (more_k) request_k(kb_next, slot, i - VPW);
            constexpr int op = slot_op(i);
            if constexpr (op >= 0) {
                constexpr int s = op / NKB, kb = op % NKB;
                if constexpr (s == 0) {
                    f32x16 z;
#pragma unroll
                    for (int r = 0; r < 16; ++r) z[r] = 0.f;
                    sn[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[i]), qf[s], z, 0, 0, 0);
                } else {
                    sn[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[i]), qf[s], sn[kb], 0, 0, 0);
                }
            } else {
                constexpr int m = -1 - op, ks = m / NDB, db = m % NDB;
                oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(fr[i]), as_bf16x8(pprev[ks]), oacc[db], 0, 0, 0);
            }
            if constexpr (i < NMIX) {
                // this slot's share of the 16 logit pairs of tile t.  A pair takes three steps (scale and
                // shift; exponentials; pack and row sum) in three different slots, so that no
                // instruction of a slot waits for another one of the same slot.
                constexpr int v_lo = (i * 18 + NMIX - 1) / NMIX; // first step v with v * NMIX / 18 == i, if any
                static_for<(18 + NMIX - 1) / NMIX + 1>([&](auto dvc) {
                    constexpr int v = v_lo + decltype(dvc)::value;
                    if constexpr (v < 18 && v * NMIX / 18 == i) {
                        if constexpr (v >= 2) {
                            constexpr int q = v - 2;
                            unsigned pk = pack_bf16(ee[q][0], ee[q][1]);
                            // an empty asm statement is a use the compiler cannot move: without it, work whose
                            // consumer sits in a later basic block is sunk out of the slot it was placed in
                            asm volatile("" : "+v"(pk));
                            pcur[q >> 2][q & 3] = pk;
                            if constexpr (q & 1) lsum = add_four(u32x2{pcur[q >> 2][(q & 3) - 1], pk}, lsum);
                        }
                        if constexpr (v >= 1 && v <= 16) {
                            constexpr int q = v - 1;
                            float e0 = __builtin_amdgcn_exp2f(tt[q][0]), e1 = __builtin_amdgcn_exp2f(tt[q][1]);
                            asm volatile("" : "+v"(e0), "+v"(e1));
                            ee[q][0] = e0; ee[q][1] = e1;
                        }
                        if constexpr (v <= 15) {
                            constexpr int q = v;
                            float t0 = fmaf(sc[q >> 3][(2 * q) & 15], c, -mr), t1 = fmaf(sc[q >> 3][((2 * q) & 15) + 1], c, -mr);
                            asm volatile("" : "+v"(t0), "+v"(t1));
                            tt[q][0] = t0; tt[q][1] = t1;
                        }
                    }
                });
            } else {
                // last quarter: row maximum of S(t+1)
                constexpr int NL = NS - NMIX, j = i - NMIX;
                constexpr int XPS = NKB * 16 / (NL > 0 ? NL : 1); // logits per slot (FIRST has no such slots)
                static_assert(NL == 0 || (XPS * NL == NKB * 16 && XPS % 2 == 0), "");
#pragma unroll
                for (int x = j * XPS; x < (j + 1) * XPS; x += 2) {
                    float mm = __builtin_fmaxf(__builtin_fmaxf(mxv[(x >> 1) & 3], sn[x >> 4][x & 15]), sn[x >> 4][(x & 15) + 1]);
                    asm volatile("" : "+v"(mm));
                    mxv[(x >> 1) & 3] = mm;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        if (FIRST) { // no last quarter: the same housekeeping without MFMAs in between
            mask_tile(t + 1, kt_b, ph_b, sn);
#pragma unroll
            for (int x = 0; x < NKB * 16; ++x) mxv[x & 3] = fmaxf(mxv[x & 3], sn[x >> 4][x & 15]);
        }
        mx_next = pair_max(fmaxf(fmaxf(mxv[0], mxv[1]), fmaxf(mxv[2], mxv[3]))) * c;
        l_run += lsum[0];
        kt_a = kt_b; ph_a = ph_b; kt_b = kt_c; ph_b = ph_c;
        tile_of(t + 3, kt_c, ph_c);
        if constexpr (TAB) {
            if (t + 3 < T) k_next = k_tile(kt_c, ph_c);
            if (t + 1 < T) v_next = v_tile(kt_a);
        }
        kb_next = k_base(kt_c, ph_c, k_next);
        vb_next = v_base(kt_a, v_next);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's K(t+2), V(t) pieces are in LDS
        __syncthreads();
    };


    typedef std::integral_constant<int, 0> slot0;
    typedef std::integral_constant<int, 1> slot1;
    iteration(std::true_type{}, slot0{}, 0, sA, sB, pB, pA);
    for (int t = 1; t < T; t += 2) {
        iteration(std::false_type{}, slot1{}, t, sB, sA, pA, pB);
        if (t + 1 < T) iteration(std::false_type{}, slot0{}, t + 1, sA, sB, pB, pA);
    }
    // ---- epilogue: O += V(T-1)^T P(T-1)
    {
        const char *vl = ldsV + ((T - 1) & 1) * VBUF;
        auto pv = [&](const u32x4 (&pw)[NPS]) {
#pragma unroll
            for (int m = 0; m < NPV; ++m)
                oacc[m % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vfrag(vl, m)), as_bf16x8(pw[m / NDB]), oacc[m % NDB], 0, 0, 0);
        };
        if ((T - 1) & 1) pv(pB);
        else pv(pA);
    }

    if constexpr (KS == 2) {
        // Group 1 leaves its state in LDS (register by register: a lane's counterpart in group 0 holds the same rows and dims)
        // and group 0 merges it: one reference maximum, accumulators and row sums added.
        f32x4 *const box = (f32x4 *)lds + (size_t)(wave * (4 * NDB)) * 64 + lane;
        float2 *const box_ml = (float2 *)(lds + 4 * 4 * NDB * 64 * sizeof(f32x4)) + wave * 64 + lane;
        __syncthreads(); // every wave has read its last V tile
        if (grp == 1) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    box[(4 * db + a) * 64] = f32x4{oacc[db][4 * a], oacc[db][4 * a + 1], oacc[db][4 * a + 2], oacc[db][4 * a + 3]};
            *box_ml = make_float2(m_ref, l_run);
        }
        __syncthreads();
        if (grp == 1) return;
        const float2 ml = *box_ml;
        const float M = fmaxf(m_ref, ml.x); // (a group without a valid key of the row has kNegBig, weight 0 and sum 0)
        const float f0 = __builtin_amdgcn_exp2f(m_ref - M), f1 = __builtin_amdgcn_exp2f(ml.x - M);
        l_run = l_run * f0 + ml.y * f1;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f32x4 o = box[(4 * db + a) * 64];
#pragma unroll
                for (int x = 0; x < 4; ++x) oacc[db][4 * a + x] = oacc[db][4 * a + x] * f0 + o[x] * f1;
            }
    }
    const float l = pair_sum(l_run);
    if (irow < p.n && irow >= p.q0) {
        const float inv = 1.f / l;
        pod_bf16 *orow = p.out + ((size_t)(irow - p.q0) * p.Hq + head) * D;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                u32x2 o;
                o.x = pack_bf16(oacc[db][4 * a + 0] * inv, oacc[db][4 * a + 1] * inv);
                o.y = pack_bf16(oacc[db][4 * a + 2] * inv, oacc[db][4 * a + 3] * inv);
                *(u32x2 *)(orow + 32 * db + 8 * a + 4 * jj) = o;
            }
    }
}

// A launch of one round hands the second half of its workgroups out in the opposite order (prefill_params::turn) where the first half
// ends with a whole group of kv heads.
bool turns_order(int cus, int Hkv) { return cus % Hkv == 0; }

// One or two key groups per workgroup.  With two, a workgroup's 128 query rows are walked by eight waves, each half of them
// every second key tile: half the iterations on the launch's longest path, at an iteration that takes longer (eight waves
// meet at its barrier) plus the merge.  It pays where the launch is short of workgroups or of equal ones.  Compared are, in key tiles
// of a workgroup alone on its CU (1.2 us at 32/8 heads x 128):
//   one group  : of the two workgroups of a CU the longer one's tiles plus 0.66 of the other's
//   two groups : one workgroup per CU, 0.75 of its tiles + 2.2 for the merge and the longer start; where a second one follows on the
//                CU, 0.84 of both's tiles + 9.3 (that start again; and a chip that is busy twice clocks lower)
// fitted to these times per launch, one -> two groups, us (lowest layers, window 512): 32/8 x 128 n = 200 10.9 -> 12.5, 400 13.6 -> 14.4,
// 777 20.3 -> 20.1, 1024 24.6 -> 23.1, 1500 34.9 -> 33.7, 1800 41.2 -> 42.8, 2048 46.8 -> 47.5, upper layer 52.0 -> 57.5; 16/1 x 128 2048
// 40.3 -> 35.3, 3001 57.3 -> 48.4, 4096 83.3 -> 77.4; 16/4 x 64 777 14.8 -> 13.6, 3001 42.0 -> 34.5, 4096 57.5 -> 51.4; behind other keys, 32/8
// x 128: 512 rows behind 7680 148 -> 122, 1024 behind 7168 154 -> 141, 2048 behind 2048 116 -> 124, 2048 behind 6144 233 -> 240.  More than two
// workgroups per CU: one group (5000 tokens 206 -> 226).
int prefill_key_groups(int cus, int Hq, int Hkv, int n, int q0, int S, int W, bool has_shared)
{
    const int last = (n - 1) / 128, tiles = last - q0 / 128 + 1; // query tiles, handed out from the last to the first
    if (cus < 1 || (int64_t)tiles * Hq > 2 * cus) return 1;
    const int nwg = tiles * Hq;
    auto cost = [&](int tile) { // key tiles that the workgroups of a query tile (in launch order) walk
        const int i0 = (last - tile) * 128;
        return tiles_of_rows(i0, (i0 + 128 < n ? i0 + 128 : n) - 1, S, W, has_shared).count;
    };
    const bool turned = turns_order(cus, Hkv);
    double one = cost(0), two = 0.75 * one + 2.2;
    for (int t = 0; t < tiles && t * Hq < cus; ++t) {
        const int lo = t * Hq, hi = (lo + Hq < cus ? lo + Hq : cus) - 1, own = cost(t);
        if (lo + cus < nwg) { // one group: the workgroups at places cus + w of the launch run beside w
            const int w = hi < nwg - cus ? hi : nwg - cus - 1;
            const double both = own + 0.66 * cost((turned ? nwg - 1 - w : lo + cus) / Hq);
            one = both > one ? both : one;
        }
        // two groups: workgroup 2 cus - 1 - w runs where w did; a query tile's workgroups, lo .. hi, meet those of two query tiles at most
        const int near = 2 * cus - 1 - hi, far = 2 * cus - 1 - lo < nwg ? 2 * cus - 1 - lo : nwg - 1;
        if (near < nwg) {
            const int a = cost(near / Hq), b = cost(far / Hq);
            const double both = 0.84 * (own + (a > b ? a : b)) + 9.3;
            two = both > two ? both : two;
        }
    }
    return two < one ? 2 : 1;
}

} // namespace

// dynamic LDS: per key group two K slots and two V slots of kBN tokens x D bf16 each (64 KB at D = 128).  The merge of two groups
// (128 rows x D fp32 and a (maximum, sum) per lane) takes the slots' place.
static constexpr int lds_bytes(int D, int key_groups) { return key_groups * 4 * kBN * D * 2; }
static_assert(128 * 64 * 4 + 256 * 8 <= lds_bytes(64, 2) && 128 * 128 * 4 + 256 * 8 <= lds_bytes(128, 2), "the slots hold the merge");

// tile_tab != NULL: keys and values are located through the per-tile address table (k, v, k_shared are not read)
static int launch_prefill(const pod_layout &ly, int n, int q0, const void *q, const void *k, const void *v,
                          const void *q_shared, const void *k_shared, const unsigned long long *tile_tab, int ntiles,
                          int *len, int *flag, uint64_t lowest_mask, float scale, void *out, const pod_fill_args *fill, hipStream_t st)
{
    prefill_params p;
    p.n = n; p.q0 = q0; p.Hq = ly.Hq; p.Hkv = ly.Hkv; p.rep = ly.rep; p.S = ly.S; p.W = ly.W;
    p.q = (const pod_bf16 *)q; p.k = (const pod_bf16 *)k; p.v = (const pod_bf16 *)v;
    p.qs = (const pod_bf16 *)q_shared; p.ks = (const pod_bf16 *)k_shared;
    p.out = (pod_bf16 *)out;
    p.scale_log2e = scale * 1.4426950408889634f;
    p.lowest_mask = lowest_mask;
    p.tile_tab = tile_tab; p.ntiles = ntiles;
    p.len = len; p.flag = flag; p.len_old = q0; p.len_new = n;
    if (scale <= 0.f) return pod_fail(POD_ERR_INVALID_ARG, "scale must be positive");
    if (tile_tab && ntiles < (n + kBN - 1) / kBN) return pod_fail(POD_ERR_INVALID_ARG, "tile table of %d entries for %d keys", ntiles, n);
    // query tiles of 128 positions, counted from the end: the kernel takes tile (n + 127) / 128 - 1 - blockIdx.x / Hq
    const unsigned attn = (unsigned)((n + 127) / 128 - q0 / 128) * (unsigned)ly.Hq;
    // raising the dynamic-LDS limit is needed once per device; any host thread may get here first
    static const struct { const void *fn; int lds; } variants[2][2][2] = { // [head dim 64 / 128][table][key groups - 1]
        {{{(const void *)prefill_kernel<64, false, 1>, lds_bytes(64, 1)}, {(const void *)prefill_kernel<64, false, 2>, lds_bytes(64, 2)}},
         {{(const void *)prefill_kernel<64, true, 1>, lds_bytes(64, 1)}, {(const void *)prefill_kernel<64, true, 2>, lds_bytes(64, 2)}}},
        {{{(const void *)prefill_kernel<128, false, 1>, lds_bytes(128, 1)}, {(const void *)prefill_kernel<128, false, 2>, lds_bytes(128, 2)}},
         {{(const void *)prefill_kernel<128, true, 1>, lds_bytes(128, 1)}, {(const void *)prefill_kernel<128, true, 2>, lds_bytes(128, 2)}}}};
    int dev = -1, cus = 0;
    POD_HIP_TRY(hipGetDevice(&dev));
    POD_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    {
        static std::mutex attr_mutex;
        static bool attr_done[64] = {};
        if (dev < 0 || dev >= 64) return pod_fail(POD_ERR_INVALID_ARG, "device %d outside [0, 64)", dev);
        std::lock_guard<std::mutex> lock(attr_mutex);
        if (!attr_done[dev]) {
            for (const auto &by_dim : variants)
                for (const auto &by_table : by_dim)
                    for (const auto &v : by_table) POD_HIP_TRY(hipFuncSetAttribute(v.fn, hipFuncAttributeMaxDynamicSharedMemorySize, v.lds));
            attr_done[dev] = true;
        }
    }
    const int ks = prefill_key_groups(cus, ly.Hq, ly.Hkv, n, q0, ly.S, ly.W, q_shared != nullptr);
    // The cache construction rides in the same launch.  Where every attention workgroup is resident at once its workgroups come
    // last, for the slots that are free from the start or as soon as the short query tiles are done; in launches of several
    // rounds a few come first and copy next to workgroups that are busy multiplying.  (A launch of its own: n = 777 5.0 us per
    // layer, 16384 tokens 25 us, and the gap before it.)  How few: one of them copies some 600 pieces per us beside such a neighbour, so that
    // an eighth of the CUs is enough for long prompts and few kv heads, but with many kv heads the launch ends with their copying: one
    // per 300 pieces and key tile that a CU walks, up to half of the CUs.  Both layers with cache, us, an eighth -> this (attention alone):
    // 64/64 x 128 n = 1100 127 -> 80 (71), 1500 180 -> 123 (115), 3001 398 -> 369 (342), 40/40 x 128 2200 178 -> 155 (148), 32/32 x 128 2200 137 -> 117
    // (116), 64/64 x 64 1500 90 -> 81 (74); 32/8 x 128 3001 191 with an eighth, 195 with three eighths.
    p.fill_lo = 0x7fffffff; p.fill_n = 0;
    if (fill) {
        const bool resident = ks == 2 || attn <= 2u * (unsigned)cus; // (two one-group workgroups per CU)
        const size_t pieces = (size_t)n * ly.Hkv * (ly.D / 8), per_wg = (size_t)256 * ks * (resident ? kFillUnroll : 1);
        size_t wgs = (pieces + per_wg - 1) / per_wg, most = cus;
        if (!resident) {
            const size_t tiles = (size_t)(n + 127) / 128, walked = tiles * (tiles + 1) * ly.Hq / cus; // key tiles per CU
            most = pieces / (300 * walked) / 8 * 8; // (as many on every XCD)
            if (most > (size_t)cus / 2) most = cus / 2;
            if (most < ((size_t)cus + 7) / 8) most = (cus + 7) / 8;
        }
        if (wgs > most) wgs = most;
        p.fill = *fill;
        p.fill_n = (int)wgs;
        p.fill_lo = resident ? (int)attn : 0;
    }
    p.per_kvh = (int)(attn / (unsigned)ly.Hkv);
    p.turn = ks == 1 && (int64_t)attn <= 2 * cus && turns_order(cus, ly.Hkv) ? cus / ly.Hkv : p.per_kvh;
    const dim3 grid(attn + (unsigned)p.fill_n);
    const auto &var = variants[ly.D == 128][tile_tab != nullptr][ks - 1];
    void *args[] = {&p};
    POD_HIP_TRY(hipLaunchKernel(var.fn, grid, dim3(256 * ks), args, var.lds, st));
    POD_HIP_TRY(hipGetLastError());
    return POD_OK;
}

int pod_launch_prefill(const pod_layout &ly, int layer, int n, int q0, const void *q, const void *k, const void *v,
                       const void *q_shared, const void *k_shared, uint64_t lowest_mask, float scale, void *out,
                       const pod_fill_args *fill, hipStream_t st)
{
    (void)layer;
    return launch_prefill(ly, n, q0, q, k, v, q_shared, k_shared, nullptr, 0, nullptr, nullptr, lowest_mask, scale, out, fill, st);
}

int pod_launch_prefill_tiles(const pod_layout &ly, int n, int q0, const void *q, const void *q_shared,
                             const unsigned long long *tile_tab, int ntiles, int *len, int *flag, uint64_t lowest_mask, float scale,
                             void *out, hipStream_t st)
{
    return launch_prefill(ly, n, q0, q, nullptr, nullptr, q_shared, nullptr, tile_tab, ntiles, len, flag, lowest_mask, scale, out, nullptr, st);
}
