// Inter-layer attention similarity for the offline layer grouping (the paper's "Attention Similarity
// Measurement"): for head h and layers a, b, the Jensen-Shannon divergence of the two layers' attention
// rows, averaged over the sampled rows; the similarity is 1 minus that average with base-2 logarithms
// (base-2 JS lies in [0, 1], so identical rows give 1 and rows with disjoint support give 0).
//
// With m = (p + q) / 2 the divergence is a difference of entropies: of one pair of elements,
//     (p log2(p / m) + q log2(q / m)) / 2 = e(p) + e(q) - m log2(m),   e(x) = x log2(x) / 2,
// so a layer's logarithms are taken once per element and a pair of layers costs one sum, one logarithm, one multiplication and
// one addition per element.  The difference is taken over two elements at a time (their e's are added up first), so
// that what is accumulated over the rows is the small difference and not the two large sums it is made of.
//
// A workgroup takes one head, one half of its rows and a block pair (A, B) of BA and BB layers, B behind A or around it: every element of
// the layers is loaded once, 16 bytes per lane and layer, ahead of its use, and the layer pairs are accumulated from registers, A's rows
// and e's held, B's streamed.  The two halves leave their sums in the two places the symmetric result has for a pair;
// similarity_finish_kernel adds them (a fixed order: same bits on every call).
// Bound by vector issue: three and a half plain instructions and a logarithm per pair and element, plus what the e's cost, nine tenths of a
// pair's for every layer of a block pair: 4 + 4 layers for 16 pairs, 4 + 8 for 32.  32 layers x 32 heads x 32 rows x 2048: 673 -> 251 (4 x 4)
// -> 217 us (4 x 8); the 673 took
// p (log p - log m) + q (log q - log m) per element, in one workgroup per head and pair of 8-layer blocks with nothing requested
// ahead.  With the pair's logarithms multiplied into e(p) + e(q) directly it takes 6 % less, but rows with the same bits then come
// out a rounding error away from 1 (one sampled row of 64 entries: every fourth).  Blocks of 8 x 8 layers leave two waves per
// SIMD: 15 % slower than 4 x 4 here, 77 instead of 33 us at 8 layers.
#include <type_traits>

#include "pod_internal.h"

namespace {

constexpr int kSimThreads = 256;
constexpr int kSimHalves = 2;
typedef __attribute__((ext_vector_type(4))) float sim_f4;

// Added to every element: nothing to a probability of 2^-95 (2.5e-29) or more, whose spacing it does not reach half of, and a zero
// becomes this, whose x log2(x) is below 1e-34 (the hardware logarithm takes subnormal numbers for 0 and never meets one).  NaNs stay NaNs.
constexpr float kSimFloor = 0x1p-120f;

struct sim_params {
    const float *att; // [L][H][R][n] probabilities (rows sum to 1)
    float *sim;       // [H][L][L]
    int L, H, nblk;
    size_t rows;      // R * n elements of one (layer, head), contiguous
    int R;            // rows per (layer, head)
    int heads_by_xcd; // 8: workgroup w takes a head that is w mod 8; 1: heads in order
    int pair0;        // the launch's first block pair
};
constexpr unsigned kSimLaunch = (1u << 24) - 1; // workgroups of one launch: a grid dimension holds less than 2^32 threads

// The pairs of blocks A (BA layers) and B (BB >= BA layers, a multiple) of a head: B behind A as a whole first (all BA x BB layer pairs), then the
// B that A lies in, at its front, in its middle or at its end, where the layers behind A's own count.
template <int BA, int BB>
__global__ __launch_bounds__(kSimThreads) void similarity_kernel(sim_params p)
{
    constexpr int PER = BB / BA;
    // The block pairs of a head, whole ones first (they have most work), and inside a kind head by head: what runs at
    // the same time on an XCD are all the block pairs of a few heads, which walk the same rows and find them in its L2.
    const int x = blockIdx.x % p.heads_by_xcd, hx = p.H / p.heads_by_xcd;
    int rest = blockIdx.x / p.heads_by_xcd;
    const int h = rest % hx * p.heads_by_xcd + x;
    rest /= hx;
    const int half = rest % kSimHalves;
    rest = p.pair0 + rest / kSimHalves;
    const int noff = PER * (p.nblk * (p.nblk - 1) / 2);
    int A, B, pos = -1; // pos: A is the pos-th block of B's own layers
    if (rest < noff) {
        B = 1;
        while (rest >= PER * B) { rest -= PER * B; ++B; }
        A = rest;
    } else {
        rest -= noff;
        pos = rest / p.nblk;
        B = rest % p.nblk;
        A = PER * B + pos;
    }
    const int nA = min(BA, p.L - A * BA), nB = min(BB, p.L - B * BB); // layers of the two blocks
    if (nA <= 0) return;
    const size_t vec = p.rows / 4; // (the entry point takes R * n in multiples of 4 only)
    const size_t v_lo = vec * half / kSimHalves, v_hi = vec * (half + 1) / kSimHalves;
    float acc[BA][BB];
#pragma unroll
    for (int i = 0; i < BA; ++i)
#pragma unroll
        for (int j = 0; j < BB; ++j) acc[i][j] = 0.f;
    const sim_f4 *ra[BA], *rb[BB]; // (layers past the last repeat it; their sums are not formed)
#pragma unroll
    for (int i = 0; i < BA; ++i) ra[i] = (const sim_f4 *)(p.att + ((size_t)(A * BA + min(i, nA - 1)) * p.H + h) * p.rows);
#pragma unroll
    for (int j = 0; j < BB; ++j) rb[j] = (const sim_f4 *)(p.att + ((size_t)(B * BB + min(j, nB - 1)) * p.H + h) * p.rows);
    // x -> x / 2; returns the sums of e(x) over the first and the last two of the four elements
    typedef __attribute__((ext_vector_type(2))) float f2;
    auto halve = [](sim_f4 &v) {
        f2 e;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float f = v[k] + kSimFloor;
            v[k] = 0.5f * f;
            const float l = __builtin_amdgcn_logf(f);
            e[k >> 1] = k & 1 ? __builtin_fmaf(v[k], l, e[k >> 1]) : v[k] * l;
        }
        return e;
    };
    // (the pair's own sum is formed in the order of halve's: of two rows with the same bits it is exactly the two layers' sums, the
    // divergence exactly 0 and the similarity exactly 1, which a threshold of 1 asks for)
    auto pair_term = [](const f2 &ea, const f2 &eb, const sim_f4 &a, const sim_f4 &b) {
#pragma clang fp contract(off)
        float t[2];
#pragma unroll
        for (int k = 0; k < 4; k += 2) {
            const float m0 = a[k] + b[k], m1 = a[k + 1] + b[k + 1];
            t[k >> 1] = (ea[k >> 1] + eb[k >> 1]) - __builtin_fmaf(m1, __builtin_amdgcn_logf(m1), m0 * __builtin_amdgcn_logf(m0));
        }
        return t[0] + t[1];
    };
    // the rows of block A are requested an iteration ahead, those of block B one layer ahead
    auto walk = [&](auto first_tag) __attribute__((always_inline)) {
        constexpr int FIRST = decltype(first_tag)::value;      // layers of B before A's own (a whole pair: -BA)
        constexpr int j0 = FIRST + BA;                          // the first layer of B behind A
        sim_f4 na[BA], nb = {};
        auto request_a = [&](size_t v) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < BA; ++i) na[i] = ra[i][v];
        };
        size_t v = v_lo + threadIdx.x;
        if (v < v_hi) {
            request_a(v);
            if constexpr (j0 < BB) nb = rb[j0][v];
        }
        for (; v < v_hi; v += kSimThreads) {
            const bool more = v + kSimThreads < v_hi;
            sim_f4 xa[BA];
            f2 ea[BA];
#pragma unroll
            for (int i = 0; i < BA; ++i) xa[i] = na[i];
            if (more) request_a(v + kSimThreads);
#pragma unroll
            for (int i = 0; i < BA; ++i) ea[i] = halve(xa[i]);
            if constexpr (FIRST >= 0) { // A's own pairs
#pragma unroll
                for (int i = 0; i < BA; ++i)
#pragma unroll
                    for (int j = i + 1; j < BA; ++j)
                        if (j < nA) acc[i][FIRST + j] += pair_term(ea[i], ea[j], xa[i], xa[j]); // (wave-uniform)
            }
#pragma unroll
            for (int j = j0; j < BB; ++j) {
                sim_f4 xb = nb;
                if (j + 1 < BB) nb = rb[j + 1 < BB ? j + 1 : 0][v];
                else if (more) nb = rb[j0 < BB ? j0 : 0][v + kSimThreads];
                if (j < nB) { // (wave-uniform)
                    const f2 eb = halve(xb);
#pragma unroll
                    for (int i = 0; i < BA; ++i) {
                        acc[i][j] += pair_term(ea[i], eb, xa[i], xb);
                        if (i & 1) __builtin_amdgcn_sched_barrier(0); // (else the scheduler spreads the pairs out until registers spill)
                    }
                }
            }
        }
    };
    if (pos < 0) walk(std::integral_constant<int, -BA>{});
    else if (PER == 1 || pos == 0) walk(std::integral_constant<int, 0>{});
    else if constexpr (PER == 2) walk(std::integral_constant<int, BA>{});
    static_assert(PER <= 2, "a case for each place of A in B");
    // workgroup reduction, pair by pair
    __shared__ float part[kSimThreads / 64][BA * BB];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < BA; ++i)
#pragma unroll
        for (int j = 0; j < BB; ++j) {
            float t = acc[i][j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
            if (lane == 0) part[wave][i * BB + j] = t;
        }
    __syncthreads();
    if (threadIdx.x < BA * BB) {
        const int i = threadIdx.x / BB, j = threadIdx.x % BB;
        const int a = A * BA + i, b = B * BB + j;
        if (a < p.L && b < p.L && a < b) {
            float js = 0.f;
            for (int w = 0; w < kSimThreads / 64; ++w) js += part[w][threadIdx.x];
            p.sim[((size_t)h * p.L + (half ? b : a)) * p.L + (half ? a : b)] = js;
        }
    }
}

// one thread per (head, a, b), a <= b: JS = sum of the two halves, mean over the rows; 1 on the diagonal
__global__ void similarity_finish_kernel(sim_params p)
{
    const unsigned i = blockIdx.x * blockDim.x + threadIdx.x, L = (unsigned)p.L, LL = L * L; // (at most 65535 layers)
    if (i >= LL) return;
    const unsigned a = i / L, b = i - a * L;
    if (a > b) return;
    float *const m = p.sim + (size_t)blockIdx.y * LL;
    const float s = a == b ? 1.f : 1.f - (m[(size_t)a * p.L + b] + m[(size_t)b * p.L + a]) / (float)p.R;
    m[(size_t)a * p.L + b] = s;
    m[(size_t)b * p.L + a] = s;
}

template <int BA, int BB>
int launch_pairs(sim_params p, hipStream_t st)
{
    p.nblk = (p.L + BB - 1) / BB;
    const int64_t pairs = (int64_t)(BB / BA) * ((int64_t)p.nblk * (p.nblk - 1) / 2 + p.nblk);
    const unsigned per_pair = (unsigned)p.H * kSimHalves, most = kSimLaunch / per_pair;
    for (int64_t lo = 0; lo < pairs; lo += most) {
        p.pair0 = (int)lo;
        const unsigned here = (unsigned)(pairs - lo < most ? pairs - lo : most);
        hipLaunchKernelGGL((similarity_kernel<BA, BB>), dim3(here * per_pair), dim3(kSimThreads), 0, st, p);
        POD_HIP_TRY(hipGetLastError());
    }
    return POD_OK;
}

} // namespace

// Blocks of 4 x 4 layers where they leave two workgroups per CU, else of 2 x 2: more workgroups, which read a row more
// often, for few heads or layers, whose rows come out of the L2 (8 layers x 4 heads: 22 us in blocks of two, 24 in blocks of four).
// 4 x 8 instead of 4 x 4 where that takes enough off the CU with most work, block pairs dealt out in order and costing their layer pairs
// and 0.9 per layer whose e's they take, times the elements of a head's rows.  Half as many workgroups with twice the sums to add
// up at their ends hide less latency, which is worth some 130 000 of these units: us, 4 x 4 -> 4 x 8 (estimate per element; units), 32 layers x 32
// heads x 65536 elements 243 -> 222 (182 -> 167; 980 000), 24000 98.5 -> 92.0, 12000 56.1 -> 54.6 (180 000), 6000 36.2 -> 35.6 (90 000), 3072 25.5 -> 27.0, 768
// 21.3 -> 23.7; 48 x 32 x 6000 65.1 -> 63.6 (190 000), 3072 42.1 -> 43.2 (100 000); 32 x 16 x 24000 60.6 -> 59.9 (170 000), 12000 37.0 -> 38.0 (86 000); 32 x 8 x 24000
// 39.2 -> 41.0 (86 000); 24 x 32, whose 768 workgroups would give a quarter of the CUs two whole block pairs and more, x 65536 154 -> 162 (112 -> 115).
pod_similarity_blocks pod_plan_similarity(int cus, int L, int H, size_t rows)
{
    auto most_work = [&](int ba, int bb) {
        const int per = bb / ba;
        const int64_t nb = (L + bb - 1) / bb, each = (int64_t)kSimHalves * H, whole = per * (nb * (nb - 1) / 2);
        int64_t ends[4] = {0, whole * each, 0, 0};
        double cost[3] = {ba * bb + 0.9 * (ba + bb), 0, 0};
        for (int pos = 0; pos < per; ++pos) { // blocks A inside their B: their own pairs, and the layers of B behind them
            const int behind = bb - (pos + 1) * ba;
            cost[1 + pos] = ba * (ba - 1) / 2 + ba * behind + 0.9 * (ba + behind);
            ends[2 + pos] = ends[1 + pos] + nb * each;
        }
        double most = 0;
        for (int at = 0; at <= per; ++at) { // (the load changes from CU to CU only where a kind begins)
            const int64_t cu = ends[at] % cus;
            double load = 0;
            for (int k = 0; k <= per; ++k) load += cost[k] * ((ends[k + 1] - cu + cus - 1) / cus - (ends[k] - cu + cus - 1) / cus);
            most = load > most ? load : most;
        }
        return most;
    };
    const int64_t nb = (L + 3) / 4;
    if (nb * (nb + 1) / 2 * kSimHalves * H < 2 * cus) return {2, 2};
    return {4, (most_work(4, 4) - most_work(4, 8)) * (double)rows > 130e3 ? 8 : 4};
}

int pod_launch_similarity(const float *att, int L, int H, int R, int n, float *sim, hipStream_t st)
{
    sim_params p;
    p.att = att; p.sim = sim; p.L = L; p.H = H; p.nblk = 0; p.pair0 = 0;
    p.rows = (size_t)R * n;
    p.R = R;
    p.heads_by_xcd = H % 8 == 0 ? 8 : 1;
    int dev = 0, cus = 0;
    POD_HIP_TRY(hipGetDevice(&dev));
    POD_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    if (L > 1) {
        const pod_similarity_blocks blocks = pod_plan_similarity(cus, L, H, p.rows);
        const int rc = blocks.a == 2 ? launch_pairs<2, 2>(p, st) : blocks.b == 8 ? launch_pairs<4, 8>(p, st) : launch_pairs<4, 4>(p, st);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(similarity_finish_kernel, dim3((unsigned)(((size_t)L * L + 255) / 256), (unsigned)H), dim3(256), 0, st, p);
    POD_HIP_TRY(hipGetLastError());
    return POD_OK;
}
