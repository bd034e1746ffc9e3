// Token selection on the distant store: the combination of the cache with a token-selection method that the
// paper's result tables list as "PoD+SnapKV" (appendix section on SnapKV: an observation window of 64 prompt
// positions, extended to grouped-query attention).  The paper gives no rule of its own; what is computed here is
// the published selection rule on the part of the cache the combination can shrink, the distant tokens (the
// proximal ones are kept in full by definition, Section 3):
//
//   votes   vote[h][t] = sum over the last `obs` prompt positions i and over the query heads g of kv head h's group
//           of the attention weight that query (i, g) gives distant token t, in the joint softmax over the keys up
//           to position i (Eq. 4).  The call is made at a block's lowest layer, where every logit is that layer's
//           own q.k (Eq. 3) and the distant logits are the ones the whole block uses.
//   top     the votes are pooled over 2r+1 neighbours (mean with zeros outside the range, or maximum), the `keep`
//           largest per kv head are selected (of equal ones the earlier token), ascending.
//   compact per layer: the selected distant rows move to the front of the distant stores, the recent ring is
//           turned to where a sequence of S + keep + W tokens has it, and the stored length becomes that: the
//           cache is then the cache of the shorter sequence and every other call works on it unchanged.
//
// The votes are a dense contraction (obs * rep query rows x n keys x D per kv head) and run on
// v_mfma_f32_32x32x16_bf16: the query rows of a kv head (64 KB at 64 positions x 4 heads x 128) are staged in LDS,
// the keys come from global memory in fragment order (a lane's fragment is 8 consecutive bf16 of one row) once per
// workgroup, and every key fragment meets all row blocks out of LDS.  Two passes over the keys:
// the first takes each query row's maximum and sum of exponentials over all keys it sees (S^T = K Q^T: a lane
// owns a query row, so the reduction over keys is in-lane), the second recomputes the distant logits transposed
// (S = Q K^T: a lane owns a key, so the sum over query rows is in-lane) and writes one vote per key.  Every sum
// has a fixed order: the votes are reproducible bit for bit.
#include <math.h>

#include <type_traits>

#include "pod_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 sel_bf16x8;
typedef __attribute__((ext_vector_type(16))) float sel_f32x16;
typedef __attribute__((ext_vector_type(4))) unsigned sel_u32x4;

constexpr int kSelThreads = 256;        // 4 waves
constexpr int kSelKeysPerIter = 128;    // 32 keys per wave
constexpr int kTopThreads = 1024;
constexpr float kLog2e = 1.4426950408889634f;

struct select_params {
    const pod_bf16 *q_obs; // [obs][Hq][D]
    const pod_bf16 *k;     // [n][Hkv][D], or NULL: the keys are read where the cache holds them (below)
    // per kv head, in bf16 elements from the cache buffer's start: row 0 of the head's sink + ring rows and of the
    // distant-key store it reads at this layer (which is its own: the call is made at the block's lowest layer)
    const pod_bf16 *cache_base;
    unsigned long long prox0[kMaxKvHeads], dist0[kMaxKvHeads];
    int n, obs, Hq, Hkv, rep, S, W;
    int R;            // obs * rep query rows per kv head; row r = (position n - obs + r / rep, head h * rep + r % rep)
    int nrb;          // blocks of 32 rows
    int keys_per_wg;  // keys per workgroup of the first pass (a multiple of 128)
    int npieces;      // workgroups per kv head in the first pass
    float scale_log2; // logit scale times log2(e)
    uint64_t head_mask;
    float2 *part;     // [Hkv][npieces][nrb * 32]  (maximum, sum of exponentials) of a row over one piece of keys
    float *stat;      // [Hkv][nrb * 32]           maximum + log2(sum of exponentials) over all keys the row sees
    float *votes;     // [Hkv][n - S - W]
};

// fragments of one row for all k-steps: 8 consecutive bf16 per k-step, at offset 8 * (lane / 32) inside the step
template <int D>
__device__ inline void load_row_fragments(const pod_bf16 *row, int lane, sel_u32x4 (&f)[D / 16])
{
    const sel_u32x4 *p = (const sel_u32x4 *)(row + 8 * (lane >> 5));
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) f[kk] = p[2 * kk];
}

// v_exp_f32: 2^x to 1 ulp; results below the smallest normal number come out as 0, which a softmax weight may
__device__ inline float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Over the 64 lanes of a wave by DPP steps inside the rows of 16 lanes, the rows through SGPRs or row broadcasts, for whole numbers (the
// order of the sums is not __shfl_xor's).  A value through LDS (__shfl) takes a round trip each, and a reduction or a scan is a chain of
// six: the top-k kernel, nine of them one after the other at 14272 tokens and 8 kv heads, 17.5 -> 16.2 us.  Call with all lanes active.
template <int CTRL, int ROWS = 0xf>
__device__ inline unsigned dpp(unsigned v) { return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, true); }
template <class F>
__device__ inline unsigned wave_reduce(unsigned v, F &&f)
{
    v = f(v, dpp<0xB1>(v));  // quad_perm [1, 0, 3, 2]
    v = f(v, dpp<0x4E>(v));  // quad_perm [2, 3, 0, 1]
    v = f(v, dpp<0x141>(v)); // row_half_mirror
    v = f(v, dpp<0x140>(v)); // row_mirror
    const auto lane = [&](int i) { return (unsigned)__builtin_amdgcn_readlane((int)v, i); };
    return f(f(lane(0), lane(16)), f(lane(32), lane(48)));
}
__device__ inline unsigned min_of(unsigned a, unsigned b) { return a < b ? a : b; }
__device__ inline unsigned max_of(unsigned a, unsigned b) { return a > b ? a : b; }
__device__ inline unsigned sum_of(unsigned a, unsigned b) { return a + b; }
__device__ inline unsigned wave_scan(unsigned v) // sum over this lane and those below it
{
    v += dpp<0x111>(v); // row_shr:1, 2, 4, 8
    v += dpp<0x112>(v);
    v += dpp<0x114>(v);
    v += dpp<0x118>(v);
    v += dpp<0x142, 0xa>(v); // row_bcast:15 into rows 1 and 3
    v += dpp<0x143, 0xc>(v); // row_bcast:31 into rows 2 and 3
    return v;
}

// where the key of position `key` of kv head h is: in the caller's array, or in the cache (sink slot, distant row,
// or the ring slot of a recent position)
__device__ inline const pod_bf16 *key_address(const select_params &p, int h, int key, int D)
{
    if (p.k) return p.k + ((size_t)key * p.Hkv + h) * D;
    if (key < p.S) return p.cache_base + p.prox0[h] + (size_t)key * D;
    if (key < p.n - p.W) return p.cache_base + p.dist0[h] + (size_t)(key - p.S) * D;
    return p.cache_base + p.prox0[h] + (size_t)(p.S + (key - p.S) % p.W) * D;
}

// (m, l) + (m2, l2) of two disjoint key sets; an empty set is (-inf, 0)
__device__ inline void merge_stat(float &m, float &l, float m2, float l2)
{
    const float M = fmaxf(m, m2);
    const float a = m > -INFINITY ? l * exp2f(m - M) : 0.f;
    const float b = m2 > -INFINITY ? l2 * exp2f(m2 - M) : 0.f;
    m = M;
    l = a + b;
}

// Query rows in LDS: a chunk of kSelChunkRows rows (8 blocks of 32) of one kv head, row-major, rows padded by 16
// bytes so that the 16 lanes of one LDS access (rows r .. r + 15, same column) fall into different banks.  A
// workgroup stages a chunk once and every fragment it then needs comes out of LDS: the keys are read from global
// memory once per workgroup and chunk instead of once per MFMA.
constexpr int kSelChunkBlocks = 8;
constexpr int kSelChunkRows = 32 * kSelChunkBlocks;
template <int D> constexpr int kSelRowBytes = D * 2 + 16;

// A thread's pieces are all requested before the first is stored: one after the other they are a chain of as many round trips
// (one wave-wide load per round trip of an L2).
template <int D, int THREADS>
__device__ inline void stage_query_rows(const select_params &p, int h, int row0, char *lds)
{
    constexpr int cpr = D / 8; // 16-byte pieces per row
    constexpr int PER = kSelChunkRows * cpr / THREADS, RPS = THREADS / cpr; // pieces per thread; rows between two of them
    static_assert(kSelChunkRows * cpr % THREADS == 0 && THREADS % cpr == 0, "");
    const int c = threadIdx.x % cpr, first = threadIdx.x / cpr;
    // (a row's position and query head are counted on from piece to piece, without a division by rep for each)
    int pos = (row0 + first) / p.rep, qh = (row0 + first) % p.rep;
    const int dpos = RPS / p.rep, dqh = RPS % p.rep;
    sel_u32x4 val[PER];
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        val[x] = sel_u32x4{0, 0, 0, 0}; // rows past the end: zeros (their logits are never used)
        if (row0 + first + x * RPS < p.R)
            val[x] = *(const sel_u32x4 *)(p.q_obs + ((size_t)pos * p.Hq + (size_t)h * p.rep + qh) * D + c * 8);
        pos += dpos;
        qh += dqh;
        if (qh >= p.rep) { qh -= p.rep; ++pos; }
    }
#pragma unroll
    for (int x = 0; x < PER; ++x) *(sel_u32x4 *)(lds + (first + x * RPS) * kSelRowBytes<D> + c * 16) = val[x];
}

template <int D>
__device__ inline void lds_row_fragments(const char *lds, int rb, int lane, sel_u32x4 (&f)[D / 16])
{
    const char *row = lds + (rb * 32 + (lane & 31)) * kSelRowBytes<D> + (lane >> 5) * 16;
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk) f[kk] = *(const sel_u32x4 *)(row + kk * 32);
}

// First pass.  Workgroup = (piece of keys, kv head, chunk of query rows); a wave walks its key blocks of 32 and, per
// key block, the chunk's row blocks: S^T = K Q^T, a lane owns query row lane % 32 of each row block and keeps that
// row's running maximum and sum of exponentials.
template <int D>
__global__ __launch_bounds__(kSelThreads) void select_stat_kernel(select_params p)
{
    const int h = blockIdx.y;
    if (!((p.head_mask >> h) & 1)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int key_lo = blockIdx.x * p.keys_per_wg;
    const int key_hi = key_lo + p.keys_per_wg < p.n ? key_lo + p.keys_per_wg : p.n;
    const int row0 = blockIdx.z * kSelChunkRows;
    const int nblk = (p.R - row0 + 31) / 32 < kSelChunkBlocks ? (p.R - row0 + 31) / 32 : kSelChunkBlocks; // row blocks in use
    __shared__ __align__(16) char ldsq[kSelChunkRows * kSelRowBytes<D>];
    __shared__ float2 red[kSelThreads / 64][kSelChunkRows];
    sel_u32x4 kf[D / 16], kn[D / 16];
    auto key_row = [&](int key0) {
        const int key = key0 + (lane & 31) < p.n ? key0 + (lane & 31) : p.n - 1;
        return key_address(p, h, key, D);
    };
    int key0 = key_lo + wave * 32;
    if (key0 < key_hi) load_row_fragments<D>(key_row(key0), lane, kn); // (on their way while the query rows are staged)
    stage_query_rows<D, kSelThreads>(p, h, row0, ldsq);
    __syncthreads();
    float m[kSelChunkBlocks], l[kSelChunkBlocks];
    int qpos[kSelChunkBlocks]; // the row's own position: it sees keys 0 .. qpos
    int pos = (row0 + (lane & 31)) / p.rep, qh = (row0 + (lane & 31)) % p.rep;
    const int dpos = 32 / p.rep, dqh = 32 % p.rep;
#pragma unroll
    for (int rb = 0; rb < kSelChunkBlocks; ++rb) {
        m[rb] = -INFINITY;
        l[rb] = 0.f;
        qpos[rb] = p.n - p.obs + (row0 + rb * 32 + (lane & 31) < p.R ? pos : 0);
        pos += dpos;
        qh += dqh;
        if (qh >= p.rep) { qh -= p.rep; ++pos; }
    }
    for (; key0 < key_hi; key0 += kSelKeysPerIter) {
#pragma unroll
        for (int kk = 0; kk < D / 16; ++kk) kf[kk] = kn[kk];
        if (key0 + kSelKeysPerIter < key_hi) load_row_fragments<D>(key_row(key0 + kSelKeysPerIter), lane, kn); // next block's keys
        auto logits = [&](int rb) {
            sel_u32x4 qf[D / 16];
            lds_row_fragments<D>(ldsq, rb, lane, qf);
            sel_f32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < D / 16; ++kk)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sel_bf16x8, kf[kk]),
                                                               __builtin_bit_cast(sel_bf16x8, qf[kk]), acc, 0, 0, 0);
            return acc;
        };
        // accumulator e of this lane: key key0 + 8 (e / 4) + 4 (lane / 32) + e % 4, query row lane % 32 of block rb
        // (the scale is positive: it commutes with the maximum, and inside the exponent it is half of a multiply-add)
        auto add_tile = [&](int rb, const sel_f32x16 &acc) {
            float tmax = acc[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) tmax = fmaxf(tmax, acc[e]);
            if (tmax > -INFINITY) {
                const float mn = fmaxf(m[rb], tmax * p.scale_log2);
                float add[2] = {0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 16; ++e) add[e & 1] += fast_exp2(__builtin_fmaf(acc[e], p.scale_log2, -mn));
                l[rb] = l[rb] * fast_exp2(m[rb] - mn) + (add[0] + add[1]); // m = -inf: l is 0 and stays 0
                m[rb] = mn;
            }
        };
        if (nblk == kSelChunkBlocks && key0 + 31 <= p.n - p.obs) {
            // all row blocks in use, and every query of the window sees all 32 keys: the next block's products run while the
            // vector pipe works on this one's
            sel_f32x16 next = logits(0);
#pragma unroll
            for (int rb = 0; rb < kSelChunkBlocks; ++rb) {
                const sel_f32x16 acc = next;
                if (rb + 1 < kSelChunkBlocks) next = logits(rb + 1);
                add_tile(rb, acc);
            }
        } else {
#pragma unroll
            for (int rb = 0; rb < kSelChunkBlocks; ++rb) {
                if (rb >= nblk) continue; // (the same in every thread)
                sel_f32x16 acc = logits(rb);
                const int seen = qpos[rb] - key0 - 4 * (lane >> 5); // qpos < n: keys past the end drop out too
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[e] = 8 * (e >> 2) + (e & 3) <= seen ? acc[e] : -INFINITY;
                add_tile(rb, acc);
            }
        }
    }
#pragma unroll
    for (int rb = 0; rb < kSelChunkBlocks; ++rb) {
        merge_stat(m[rb], l[rb], __shfl_xor(m[rb], 32), __shfl_xor(l[rb], 32)); // the two lanes of a row hold different keys
        if (lane < 32) red[wave][rb * 32 + lane] = make_float2(m[rb], l[rb]);
    }
    __syncthreads();
    const int r = row0 + threadIdx.x; // kSelThreads == kSelChunkRows: one thread per row of the chunk
    if (r < p.nrb * 32) {
        float M = red[0][threadIdx.x].x, L = red[0][threadIdx.x].y;
        for (int w = 1; w < kSelThreads / 64; ++w) merge_stat(M, L, red[w][threadIdx.x].x, red[w][threadIdx.x].y);
        p.part[((size_t)h * p.npieces + blockIdx.x) * (p.nrb * 32) + r] = make_float2(M, L);
    }
}
static_assert(kSelThreads == kSelChunkRows, "the first pass hands one row of the chunk to every thread");

// one wave per (kv head, query row): lane c holds piece c (at most 64 pieces).  Writes what the second pass
// subtracts from a logit: maximum + log2(sum), so that exp2(logit - that) is the attention weight; +infinity for
// the rows past the end (their weight is then 0).
__global__ __launch_bounds__(kSelThreads) void select_reduce_kernel(select_params p)
{
    const int h = blockIdx.y;
    if (!((p.head_mask >> h) & 1)) return;
    const int lane = threadIdx.x & 63;
    const int r = blockIdx.x * (kSelThreads / 64) + (threadIdx.x >> 6);
    if (r >= p.nrb * 32) return;
    float m = -INFINITY, l = 0.f;
    if (lane < p.npieces) {
        const float2 t = p.part[((size_t)h * p.npieces + lane) * (p.nrb * 32) + r];
        m = t.x;
        l = t.y;
    }
    float M = m;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    float L = m > -INFINITY ? l * exp2f(m - M) : 0.f;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) L += __shfl_xor(L, o); // the same order in every lane: all lanes end with the same sum
    if (lane == 0) p.stat[(size_t)h * (p.nrb * 32) + r] = r < p.R && L > 0.f ? M + log2f(L) : INFINITY; // (every row sees key 0: L > 0)
}

// Second pass.  Workgroup = (256 distant keys, kv head); a wave takes 32 of them and every row block of every chunk: S = Q K^T,
// a lane owns key lane % 32 and adds up the weights of 16 query rows per MFMA tile.  A distant key is older than every query of the
// observation window (obs <= W): no causal test.  Eight waves share one staging of the query rows, and two such workgroups fit a CU (120
// registers, 70 KB): four waves per SIMD.  Four waves that take two key blocks each, one after the other (214 registers, two waves per SIMD),
// took 15.8 instead of 13.8 us at 14272 distant tokens, 8 kv heads and 256 rows; one block each without the shared staging 19.1.
constexpr int kVoteThreads = 512;
constexpr int kSelVoteKeys = kVoteThreads / 2;     // keys per workgroup: 32 per wave

template <int D>
__global__ __launch_bounds__(kVoteThreads, 4) void select_vote_kernel(select_params p)
{
    const int h = blockIdx.y;
    if (!((p.head_mask >> h) & 1)) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int dist_hi = p.n - p.W;                                         // distant keys: S .. n - W - 1
    const int wg_key0 = p.S + blockIdx.x * kSelVoteKeys;
    __shared__ __align__(16) char ldsq[kSelChunkRows * kSelRowBytes<D>];
    __shared__ __align__(16) float ldsb[kSelChunkRows];
    const int key0 = wg_key0 + wave * 32;
    const bool have = key0 < dist_hi; // (the same in the whole wave)
    float vote = 0.f;
    sel_u32x4 kf[D / 16];
    {   // (clamped past the end: what is loaded there is not used)
        const int key = key0 + (lane & 31) < dist_hi ? key0 + (lane & 31) : dist_hi - 1;
        load_row_fragments<D>(key_address(p, h, key, D), lane, kf);
    }
    for (int row0 = 0; row0 < p.R; row0 += kSelChunkRows) {
        if (row0) __syncthreads(); // everyone is done with the previous chunk
        stage_query_rows<D, kVoteThreads>(p, h, row0, ldsq);
        if (threadIdx.x < kSelChunkRows) {
            const int r = row0 + threadIdx.x; // one row of the chunk per thread
            ldsb[threadIdx.x] = r < p.nrb * 32 ? p.stat[(size_t)h * (p.nrb * 32) + r] : INFINITY;
        }
        __syncthreads();
        if (!have) continue;
        const int nblk = (p.R - row0 + 31) / 32 < kSelChunkBlocks ? (p.R - row0 + 31) / 32 : kSelChunkBlocks;
        auto logits = [&](int rb) {
            sel_u32x4 qf[D / 16];
            lds_row_fragments<D>(ldsq, rb, lane, qf);
            sel_f32x16 acc = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < D / 16; ++kk)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(sel_bf16x8, qf[kk]),
                                                               __builtin_bit_cast(sel_bf16x8, kf[kk]), acc, 0, 0, 0);
            return acc;
        };
        // accumulator e of this lane: query row rb * 32 + 8 (e / 4) + 4 (lane / 32) + e % 4 of the chunk, key lane % 32
        auto add_tile = [&](int rb, const sel_f32x16 &acc) {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
                typedef __attribute__((ext_vector_type(4))) float f32x4;
                const f32x4 bq = *(const f32x4 *)(ldsb + rb * 32 + 8 * e4 + 4 * (lane >> 5));
#pragma unroll
                for (int j = 0; j < 4; ++j) vote += fast_exp2(acc[4 * e4 + j] * p.scale_log2 - bq[j]);
            }
        };
        if (nblk == kSelChunkBlocks) { // (the next block's products beside this one's exponentials, as in the first pass)
            sel_f32x16 next = logits(0);
#pragma unroll
            for (int rb = 0; rb < kSelChunkBlocks; ++rb) {
                const sel_f32x16 acc = next;
                if (rb + 1 < kSelChunkBlocks) next = logits(rb + 1);
                add_tile(rb, acc);
            }
        } else {
            for (int rb = 0; rb < nblk; ++rb) add_tile(rb, logits(rb));
        }
    }
    const float v = vote + __shfl_xor(vote, 32); // the two lanes of a key hold different query rows
    if (lane < 32 && key0 + lane < dist_hi) p.votes[(size_t)h * (dist_hi - p.S) + (key0 + lane - p.S)] = v;
}

// order-preserving map of a float's bits to an unsigned (larger float = larger unsigned)
__device__ inline unsigned ordered_bits(float x)
{
    unsigned u = __builtin_bit_cast(unsigned, x);
    if (u == 0x80000000u) u = 0u; // -0 and +0 are one value
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Selection, one workgroup per kv head, over the pooled votes: find the keep-th largest ordered bit pattern by histograms of
// kTopBins equal parts of the range that still holds it - first from the smallest to the largest pattern there is, then inside
// the part that was hit, a bit pattern of 32 bits in three rounds at most, the votes of one prompt in two - and write the
// indices of the selected tokens in ascending order (everything above the threshold, and the first `need` of those equal to
// it).  What a round costs are its LDS atomics, and lanes that hit the same counter take turns: parts of the range that occurs
// keep them apart, where digits of the pattern (sign and exponent first, which all votes share) had them queue: 14272 tokens, this
// kernel alone, four rounds of 8-bit digits -> this: a prompt's own votes 25.1 -> 15.6 us, uniform ones 27.2 -> 17.4.  A thread owns a run of
// ceil(m / 1024) consecutive tokens and keeps the first kTopCache of them in registers, so the passes read
// memory only for prompts of more than 1024 * kTopCache distant tokens; token order is thread order, so one scan
// over the threads' counts gives every thread the place of its first selected token.
constexpr int kTopBins = 4096;
static_assert(kTopBins == 4 * kTopThreads, "a thread searches four counters");
constexpr int kTopCache = 32;

__device__ inline float pooled_vote(const float *__restrict__ v, int t, int m, int r, int width, int use_max)
{
    const int lo = t - r > 0 ? t - r : 0, hi = t + r + 1 < m ? t + r + 1 : m;
    if (use_max) {
        float x = v[lo];
        for (int u = lo + 1; u < hi; ++u) x = fmaxf(x, v[u]);
        return x;
    }
    float acc = 0.f;
    for (int u = lo; u < hi; ++u) acc = acc + v[u];
    return acc / (float)width;
}

// pooling: one thread per (kv head, distant token), so that the window's loads of many tokens are in flight together
// (a thread of select_top_kernel walking its own run would wait for them one after the other)
__global__ __launch_bounds__(256) void select_pool_kernel(const float *__restrict__ votes, int m, uint64_t head_mask, int width,
                                                          int use_max, float *__restrict__ pooled)
{
    const int h = blockIdx.y, t = blockIdx.x * 256 + threadIdx.x;
    if (!((head_mask >> h) & 1) || t >= m) return;
    pooled[(size_t)h * m + t] = pooled_vote(votes + (size_t)h * m, t, m, width / 2, width, use_max);
}

__global__ __launch_bounds__(kTopThreads) void select_top_kernel(const float *__restrict__ pooled, int m, uint64_t head_mask, int keep,
                                                                 int32_t *sel, int sel_stride)
{
    const int h = blockIdx.x;
    if (!((head_mask >> h) & 1)) return;
    const float *pl = pooled + (size_t)h * m;
    int32_t *out = sel + (size_t)h * sel_stride;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int span = (m + kTopThreads - 1) / kTopThreads; // tokens per thread: t0 .. t0 + span - 1 (those below m)
    const int t0 = tid * span;
    unsigned ck[kTopCache]; // ordered bit patterns of the pooled votes of tokens t0 + j
#pragma unroll
    for (int j = 0; j < kTopCache; ++j) { // (loads of clamped addresses, all in flight before the first is used)
        const int t = t0 + j < m ? t0 + j : m - 1;
        ck[j] = 0u;
        if (j < span) ck[j] = __builtin_bit_cast(unsigned, pl[t]); // (span is the same in every thread)
    }
#pragma unroll
    for (int j = 0; j < kTopCache; ++j) ck[j] = j < span && t0 + j < m ? ordered_bits(__builtin_bit_cast(float, ck[j])) : 0u;
    __shared__ __align__(16) unsigned hist[kTopBins];
    __shared__ unsigned s_lo, s_need;
    __shared__ unsigned wave_tot[2][kTopThreads / 64];
    // every token of this thread's run and its key, in order (those that are not in registers eight loads at a time)
    auto each_key = [&](auto &&f) {
#pragma unroll
        for (int j = 0; j < kTopCache; ++j)
            if (j < span && t0 + j < m) f(t0 + j, ck[j]);
        for (int j = kTopCache; j < span; j += 8) {
            float v[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) v[x] = pl[t0 + j + x < m ? t0 + j + x : m - 1];
#pragma unroll
            for (int x = 0; x < 8; ++x)
                if (j + x < span && t0 + j + x < m) f(t0 + j + x, ordered_bits(v[x]));
        }
    };
    unsigned lo = ~0u, hi = 0u; // smallest and largest key
    each_key([&](int, unsigned key) { lo = key < lo ? key : lo; hi = key > hi ? key : hi; });
    lo = wave_reduce(lo, min_of);
    hi = wave_reduce(hi, max_of);
    if (lane == 0) { wave_tot[0][wave] = lo; wave_tot[1][wave] = hi; }
    __syncthreads();
    lo = wave_reduce(wave_tot[0][lane % (kTopThreads / 64)], min_of);
    hi = wave_reduce(wave_tot[1][lane % (kTopThreads / 64)], max_of);
    unsigned need = (unsigned)keep; // the threshold is the need-th largest of the keys in [lo, hi]; the same in every thread, like lo and hi
    for (;;) {
        const unsigned range = hi - lo;
        const int shift = range < kTopBins ? 0 : 32 - 12 - __builtin_clz(range); // range >> shift < kTopBins
        __syncthreads(); // (wave_tot, hist and s_* are read before they are written again)
#pragma unroll
        for (int x = 0; x < kTopBins / kTopThreads; ++x) hist[x * kTopThreads + tid] = 0;
        __syncthreads();
        each_key([&](int, unsigned key) { if (key >= lo && key <= hi) atomicAdd(&hist[(key - lo) >> shift], 1u); });
        __syncthreads();
        // thread t takes counters 4 t .. 4 t + 3; keys from its first counter on: its own, those of the wave's higher lanes, of the higher waves
        unsigned c[4], own = 0;
#pragma unroll
        for (int x = 0; x < 4; ++x) { c[x] = hist[4 * tid + x]; own += c[x]; }
        const unsigned up_to = wave_scan(own), all = (unsigned)__builtin_amdgcn_readlane((int)up_to, 63);
        unsigned from_here = all - up_to + own;
        if (lane == 0) wave_tot[0][wave] = all;
        __syncthreads();
        // and what the waves above hold: their totals in one read
        from_here += wave_reduce(lane > wave && lane < kTopThreads / 64 ? wave_tot[0][lane] : 0u, sum_of);
        unsigned above = from_here - own;
        if (above < need && need <= from_here) { // exactly one thread: the need-th largest lies in one of its counters
#pragma unroll
            for (int x = 3; x >= 0; --x) {
                if (above < need && need <= above + c[x]) {
                    s_lo = lo + ((unsigned)(4 * tid + x) << shift);
                    s_need = need - above;
                }
                above += c[x];
            }
        }
        __syncthreads();
        const unsigned part = (1u << shift) - 1;
        lo = s_lo;
        hi = hi - lo < part ? hi : lo + part;
        need = s_need;
        if (shift == 0) break;
    }
    const unsigned thr = lo; // need >= 1 entries equal to the threshold are taken, earliest first
    // tokens above / at the threshold in this thread's run, then in all runs before it
    unsigned n_gt = 0, n_eq = 0;
    each_key([&](int, unsigned key) { n_gt += key > thr; n_eq += key == thr; });
    const unsigned inc_gt = wave_scan(n_gt), inc_eq = wave_scan(n_eq);
    if (lane == 63) { wave_tot[0][wave] = inc_gt; wave_tot[1][wave] = inc_eq; }
    __syncthreads();
    unsigned gt_before = inc_gt - n_gt, eq_before = inc_eq - n_eq;
    gt_before += wave_reduce(lane < wave ? wave_tot[0][lane] : 0u, sum_of); // (the waves below)
    eq_before += wave_reduce(lane < wave ? wave_tot[1][lane] : 0u, sum_of);
    each_key([&](int t, unsigned key) {
        const bool gt = key > thr, eq = key == thr;
        if (gt || (eq && eq_before < need)) {
            const unsigned pos = gt_before + (eq_before < need ? eq_before : need);
            if (pos < (unsigned)keep) out[pos] = t;
        }
        gt_before += gt;
        eq_before += eq;
    });
}

struct compact_params {
    char *base;
    pod_layout ly;
    pod_headmap hm;
    int layer, b, n, keep;
    int rows;                         // keep + W, or keep where the ring of the shorter sequence starts at the same slot
    const int32_t *sel_all;           // [L][Hkv][keep]
    int32_t sel_layer[kMaxKvHeads];   // the lowest layer of kv head h's block: whose selection h follows here
    uint4 *ws;                        // [2][Hkv][rows][D] bf16: rows on their way (keys, then values)
};

// Row t of the selection of head h at the layer of its block's lowest layer; not a token of the distant store: row 0, and the flag.
__device__ inline size_t selected_row(const compact_params &p, int h, int row, int n_dist)
{
    const int t = p.sel_all[((size_t)p.sel_layer[h] * p.ly.Hkv + h) * p.keep + row];
    if (t >= 0 && t < n_dist) return (size_t)t;
    atomicOr((int32_t *)(p.base + p.ly.off_flag), 1);
    return 0;
}

// Compaction in one launch and without the workspace.  A workgroup owns 64 bytes of every row of one (kv head, keys or values):
// nobody else reads or writes them, so it takes all surviving rows into its registers, waits until every wave has done so, and
// stores them where the shorter sequence keeps them - any selection, in any order - first the distant rows, then the recent window where
// that turns.  A thread has a piece of up to 16 rows in flight (by_rows: a power of two that covers the count, so that few rows are not
// fetched many times over by lanes past the last), 4096 rows per workgroup; what is larger goes through the workspace (below).  The last
// workgroup to have read the stored length changes it (the count is kept where a decode step keeps its own, zero between launches), or
// raises the flag if it was not n.  Bound by latency, four accesses one after the other (the length, the selection, the rows, the
// stores): every pass over a thread's rows is straight code, indices from clamped positions, bad entries turned into row 0 by a select.  A
// condition around each row's access instead makes the compiler wait for every index and every row before the next is requested.  Two
// workgroups whose pieces make up a 128-byte line run on one XCD (an L2 that holds a line for half of it reads and writes it for nothing).
// Fill and compaction of two layers, us, three launches per layer -> one (in brackets: with a condition around each row, heads dealt out
// in grid order), 8 kv heads x 128: 3000 tokens -> 300 selected 32.5 -> 27.6 (27.4), 16384 -> 1984 63.3 -> 59.3 (59.5), 16001 -> 1984, where a window of
// 2048 turns, 71.1 -> 68.3 (70.8), 16001 -> 900 with a window of 4096 77.4 -> 72.0 (78.8); 9 x 128, that last one, 86 -> 76 (87).
// A workgroup moves its rows at the rate of one CU: few workgroups are faster at few rows and slower at many, 32 of them (4 x 128) 300 rows 27.1 -> 24.9,
// 1984 45.4 -> 43.5, 2048 and a window of 256 37.5 -> 38.3, of 4096 and 4096 63.6 -> 71.7; 16 (4 x 64) 300 rows 26.2 -> 23.9, 2048 + 256
// 28.9 -> 31.1.  64 (8 x 128) are faster up to 6000 rows or so and level from there on (4096 alone, out of 16384, 84.4 -> 85.6; 4096 + 4096
// 101 -> 96, but 80 and 72 workgroups, 10 and 9 x 128, 122 -> 128 and 112 -> 122); 104 (13 x 128), 4096 + 4096 156 -> 150.  Hence 64 up to 6144 rows
// and 96 beyond.
constexpr int kCompactWorkgroups = 64, kCompactManyRows = 6144, kCompactManyWorkgroups = 96;
constexpr int kCompactThreads = 1024, kCompactPieces = 4, kCompactRows = kCompactThreads / kCompactPieces, kCompactMost = 16;
template <int MOST, class F>
__device__ __forceinline__ void by_rows(int count, F &&f) // f(rows a thread takes a piece of, at most)
{
    if (count <= 1 * kCompactRows) f(std::integral_constant<int, 1>{});
    else if (count <= 2 * kCompactRows) f(std::integral_constant<int, 2>{});
    else if (count <= 4 * kCompactRows) f(std::integral_constant<int, 4>{});
    else if (MOST == 8 || count <= 8 * kCompactRows) f(std::integral_constant<int, 8>{});
    else f(std::integral_constant<int, MOST>{});
}

// Row to(i) of rows = row src[i / kCompactRows], i < count, all at once.  (past the last row src is the last once more, which is not stored)
template <int PER, class To>
__device__ __forceinline__ void move_rows(pod_u32x4 *rows, int cpr, int c, const int (&src)[PER], int row0, int count, To &&to)
{
    pod_u32x4 val[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) val[u] = rows[(size_t)src[u] * cpr + c];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // (a store of another wave must not overtake these)
    __builtin_amdgcn_s_waitcnt(0x0f70);              // (vmcnt(0) again, for the compiler: else every store waits for the one before it)
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = row0 + u * kCompactRows;
        if (i < count) rows[(size_t)to(i) * cpr + c] = val[u];
    }
}

// (up to 2048 rows in a kernel of its own: two workgroups per CU instead of one, 40 kv heads x 128, 1024 rows, 126 -> 122 us)
template <int MOST>
__global__ __launch_bounds__(kCompactThreads) void compact_kernel(compact_params p)
{
    const pod_layout &ly = p.ly;
    const int line = blockIdx.z * gridDim.x + blockIdx.x; // of the 2 Hkv D / 64 columns of 128 bytes: column, then keys or values, then kv head
    if (line >= 2 * ly.Hkv * (ly.D / 64)) return;
    const int col = line / (2 * ly.Hkv), pair = line - col * (2 * ly.Hkv), is_v = pair >= ly.Hkv, h = is_v ? pair - ly.Hkv : pair;
    int32_t *const len = (int32_t *)(p.base + ly.off_lens) + (size_t)p.layer * ly.B + p.b;
    const bool ok = *len == p.n;
    if (ok) {
        const int cpr = ly.D / 8, n_dist = p.n - ly.S - ly.W;
        const int c = (2 * col + blockIdx.y) * kCompactPieces + threadIdx.x % kCompactPieces, row0 = threadIdx.x / kCompactPieces;
        const bool low = (p.hm.lowest_mask >> h) & 1;
        if (is_v || low) { // (the keys of distant tokens are kept by the lowest layer of a block only)
            const int32_t *const sel = p.sel_all + ((size_t)p.sel_layer[h] * ly.Hkv + h) * p.keep;
            pod_u32x4 *const rows = is_v ? (pod_u32x4 *)(p.base + ly.off_distV) + pod_dist_row0(ly, p.layer, p.b, h) * cpr
                                         : (pod_u32x4 *)(p.base + ly.off_distK) + pod_distk_row0(ly, p.hm, p.b, h) * cpr;
            by_rows<MOST>(p.keep, [&](auto per) __attribute__((always_inline)) {
                constexpr int PER = decltype(per)::value;
                int src[PER];
                bool bad = false;
#pragma unroll
                for (int u = 0; u < PER; ++u) src[u] = sel[min(row0 + u * kCompactRows, p.keep - 1)];
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const bool in = (unsigned)src[u] < (unsigned)n_dist;
                    bad = bad || !in;
                    src[u] = in ? src[u] : 0;
                }
                move_rows<PER>(rows, cpr, c, src, row0, p.keep, [](int i) { return i; });
                if (bad) atomicOr((int32_t *)(p.base + ly.off_flag), 1);
            });
        }
        if (p.rows > p.keep) { // (position n - W + i before, S + keep + i after)
            const int W = ly.W, from = (p.n - ly.S) % W, to = p.keep % W;
            auto ring = [W](int x) { return x >= W ? x - W : x; };
            pod_u32x4 *const rows = (pod_u32x4 *)(p.base + (is_v ? ly.off_proxV : ly.off_proxK)) + (pod_prox_row0(ly, p.layer, p.b, h) + ly.S) * cpr;
            by_rows<MOST>(W, [&](auto per) __attribute__((always_inline)) {
                constexpr int PER = decltype(per)::value;
                int src[PER];
#pragma unroll
                for (int u = 0; u < PER; ++u) src[u] = ring(from + min(row0 + u * kCompactRows, W - 1));
                move_rows<PER>(rows, cpr, c, src, row0, W, [&](int i) { return ring(to + i); });
            });
        }
    }
    __syncthreads(); // every wave has used the length it read
    if (threadIdx.x == 0) {
        int32_t *const done = (int32_t *)(p.base + ly.off_stepdone) + p.b;
        const int all = 2 * 2 * ly.Hkv * (ly.D / 64);
        if (__hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == all - 1) {
            __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (ok) *len = ly.S + p.keep + ly.W;
            else atomicOr((int32_t *)(p.base + ly.off_flag), 1);
        }
    }
}

// More than 4096 rows of a kind, or too few workgroups for one launch: stage 0 copies the surviving rows into the workspace, stage 1 copies
// them back to where the shorter sequence keeps them; both do nothing unless the stored length is n (compact_commit_kernel then raises the flag).
// Rows 0 .. keep - 1: selected distant rows; rows keep .. keep + W - 1: the recent window, oldest first.
template <int STAGE>
__global__ void compact_move_kernel(compact_params p)
{
    const pod_layout &ly = p.ly;
    const int32_t *lens = (const int32_t *)(p.base + ly.off_lens);
    if (lens[(size_t)p.layer * ly.B + p.b] != p.n) return;
    const int h = blockIdx.y, is_v = blockIdx.z;
    const int cpr = ly.D / 8, rows = p.rows, n_dist = p.n - ly.S - ly.W;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * cpr) return;
    const int row = idx / cpr, c = idx % cpr;
    const bool low = (p.hm.lowest_mask >> h) & 1;
    uint4 *wsrow = p.ws + (((size_t)is_v * ly.Hkv + h) * rows + row) * cpr + c;
    uint4 *cache_row;
    if (row < p.keep) {
        if (!is_v && !low) return; // this layer keeps no distant keys for head h
        const size_t r = STAGE == 0 ? selected_row(p, h, row, n_dist) : (size_t)row;
        cache_row = is_v ? (uint4 *)(p.base + ly.off_distV) + (pod_dist_row0(ly, p.layer, p.b, h) + r) * cpr + c
                         : (uint4 *)(p.base + ly.off_distK) + (pod_distk_row0(ly, p.hm, p.b, h) + r) * cpr + c;
    } else {
        const int i = row - p.keep; // position n - W + i before, S + keep + i after
        const int slot = ly.S + (STAGE == 0 ? (p.n - ly.S + i) % ly.W : (p.keep + i) % ly.W);
        cache_row = (uint4 *)(p.base + (is_v ? ly.off_proxV : ly.off_proxK)) + (pod_prox_row0(ly, p.layer, p.b, h) + slot) * cpr + c;
    }
    if (STAGE == 0) *wsrow = *cache_row;
    else *cache_row = *wsrow;
}

__global__ void compact_commit_kernel(char *base, pod_layout ly, int layer, int b, int n, int n_new)
{
    int32_t *len = (int32_t *)(base + ly.off_lens) + (size_t)layer * ly.B + b;
    if (*len == n) *len = n_new;
    else atomicOr((int32_t *)(base + ly.off_flag), 1);
}

inline size_t up256(size_t x) { return (x + 255) / 256 * 256; }

struct select_plan { int R, nrb, keys_per_wg, npieces; size_t off_stat, bytes; };

select_plan plan_votes(const pod_layout &ly, int64_t n, int obs)
{
    select_plan s;
    s.R = obs * ly.rep;
    s.nrb = (s.R + 31) / 32;
    int per = (int)((n + 63) / 64);
    s.keys_per_wg = (per + kSelKeysPerIter - 1) / kSelKeysPerIter * kSelKeysPerIter;
    s.npieces = (int)((n + s.keys_per_wg - 1) / s.keys_per_wg);
    s.off_stat = up256((size_t)ly.Hkv * s.npieces * s.nrb * 32 * sizeof(float2));
    s.bytes = s.off_stat + up256((size_t)ly.Hkv * s.nrb * 32 * sizeof(float2));
    return s;
}

} // namespace

size_t pod_select_votes_bytes(const pod_layout &ly, int64_t n, int obs) { return plan_votes(ly, n, obs).bytes; }
size_t pod_select_top_bytes(const pod_layout &ly, int64_t n) { return up256((size_t)ly.Hkv * (size_t)(n - ly.S - ly.W) * sizeof(float)); }
size_t pod_compact_bytes(const pod_layout &ly, int keep) { return up256((size_t)2 * ly.Hkv * ((size_t)keep + ly.W) * ly.D * 2); }

int pod_launch_select_votes(const pod_cache *c, int layer, int b, uint64_t head_mask, int n, const void *q_obs, int obs, const void *k,
                            float scale, float *votes, void *ws, hipStream_t st)
{
    const pod_layout &ly = c->ly;
    const select_plan s = plan_votes(ly, n, obs);
    select_params p;
    p.q_obs = (const pod_bf16 *)q_obs; p.k = (const pod_bf16 *)k;
    p.cache_base = (const pod_bf16 *)c->base;
    const pod_headmap hm = pod_make_headmap(c, layer);
    for (int h = 0; h < ly.Hkv; ++h) {
        p.prox0[h] = ly.off_proxK / 2 + pod_prox_row0(ly, layer, b, h) * (size_t)ly.D;
        p.dist0[h] = ly.off_distK / 2 + pod_distk_row0(ly, hm, b, h) * (size_t)ly.D;
    }
    p.n = n; p.obs = obs; p.Hq = ly.Hq; p.Hkv = ly.Hkv; p.rep = ly.rep; p.S = ly.S; p.W = ly.W;
    p.R = s.R; p.nrb = s.nrb; p.keys_per_wg = s.keys_per_wg; p.npieces = s.npieces;
    p.scale_log2 = scale * kLog2e;
    p.head_mask = head_mask;
    p.part = (float2 *)ws; p.stat = (float *)((char *)ws + s.off_stat); p.votes = votes;
    const int n_dist = n - ly.S - ly.W;
    const dim3 g1(s.npieces, ly.Hkv, (s.R + kSelChunkRows - 1) / kSelChunkRows), g2((s.nrb * 32 + kSelThreads / 64 - 1) / (kSelThreads / 64), ly.Hkv), g3((n_dist + kSelVoteKeys - 1) / kSelVoteKeys, ly.Hkv);
    if (ly.D == 128) {
        hipLaunchKernelGGL(select_stat_kernel<128>, g1, dim3(kSelThreads), 0, st, p);
        hipLaunchKernelGGL(select_reduce_kernel, g2, dim3(kSelThreads), 0, st, p);
        hipLaunchKernelGGL(select_vote_kernel<128>, g3, dim3(kVoteThreads), 0, st, p);
    } else {
        hipLaunchKernelGGL(select_stat_kernel<64>, g1, dim3(kSelThreads), 0, st, p);
        hipLaunchKernelGGL(select_reduce_kernel, g2, dim3(kSelThreads), 0, st, p);
        hipLaunchKernelGGL(select_vote_kernel<64>, g3, dim3(kVoteThreads), 0, st, p);
    }
    POD_HIP_TRY(hipGetLastError());
    return POD_OK;
}

int pod_launch_select_top(int Hkv, uint64_t head_mask, const float *votes, int m, int width, int use_max, int keep,
                          float *pooled, int32_t *sel, int sel_stride, hipStream_t st)
{
    hipLaunchKernelGGL(select_pool_kernel, dim3((m + 255) / 256, Hkv), dim3(256), 0, st, votes, m, head_mask, width, use_max, pooled);
    hipLaunchKernelGGL(select_top_kernel, dim3(Hkv), dim3(kTopThreads), 0, st, (const float *)pooled, m, head_mask, keep, sel, sel_stride);
    POD_HIP_TRY(hipGetLastError());
    return POD_OK;
}

int pod_launch_compact(const pod_cache *c, int layer, int b, int n, const int32_t *sel_all, int keep, void *ws, hipStream_t st)
{
    const pod_layout &ly = c->ly;
    compact_params p;
    p.base = c->base; p.ly = ly; p.hm = pod_make_headmap(c, layer);
    p.layer = layer; p.b = b; p.n = n; p.keep = keep; p.sel_all = sel_all; p.ws = (uint4 *)ws;
    for (int h = 0; h < ly.Hkv; ++h) p.sel_layer[h] = c->lowest[(size_t)layer * ly.Hkv + h];
    // Recent position i of the ring is at slot (n - S + i) mod W before and at (keep + i) mod W after: where W divides the number of
    // dropped tokens it is there already, which is one prompt length in W: 2048 of 4096 kept rows, per layer, 7.9 + 6.4 us at 16001 tokens,
    // 5.0 + 4.0 at 16384, where it happens to.
    p.rows = keep + ((n - ly.S - ly.W - keep) % ly.W != 0 ? ly.W : 0);
    const int most = p.rows > keep && ly.W > keep ? ly.W : keep; // rows of one kind that move
    const int xcds = c->nxcd > 0 ? c->nxcd : 1, lines = 2 * ly.Hkv * (ly.D / 64);
    if (most <= kCompactMost * kCompactRows && 2 * lines >= (p.rows <= kCompactManyRows ? kCompactWorkgroups : kCompactManyWorkgroups)) {
        const dim3 g1(xcds, 2, (lines + xcds - 1) / xcds);
        if (most <= 8 * kCompactRows) hipLaunchKernelGGL(compact_kernel<8>, g1, dim3(kCompactThreads), 0, st, p);
        else hipLaunchKernelGGL(compact_kernel<kCompactMost>, g1, dim3(kCompactThreads), 0, st, p);
        POD_HIP_TRY(hipGetLastError());
        return POD_OK;
    }
    const int items = p.rows * (ly.D / 8);
    const dim3 g((items + 255) / 256, ly.Hkv, 2);
    hipLaunchKernelGGL(compact_move_kernel<0>, g, dim3(256), 0, st, p);
    hipLaunchKernelGGL(compact_move_kernel<1>, g, dim3(256), 0, st, p);
    hipLaunchKernelGGL(compact_commit_kernel, dim3(1), dim3(1), 0, st, c->base, ly, layer, b, n, ly.S + keep + ly.W);
    POD_HIP_TRY(hipGetLastError());
    return POD_OK;
}
