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
// A workgroup takes one head, one half of its rows and a block pair (A, B) of BL layers each (A <= B): every element of up to
// 2 BL layers is loaded once, 16 bytes per lane and layer, ahead of its use, and all the BL x BL (or, on the diagonal,
// BL (BL - 1) / 2) layer pairs are accumulated from registers.  The two halves leave their sums in the two places
// the symmetric result has for a pair; similarity_finish_kernel adds them (a fixed order: same bits on every call).
// Bound by vector issue: three and a half plain instructions and a logarithm per pair and element, plus a quarter of that for
// the e's (vector pipes 96 % busy by counter).  32 layers x 32 heads x 32 rows x 2048: 673 -> 251 us; the 673 took
// p (log p - log m) + q (log q - log m) per element, in one workgroup per head and pair of 8-layer blocks with nothing requested
// ahead.  With the pair's logarithms multiplied into e(p) + e(q) directly it takes 6 % less, but rows with the same bits then come
// out a rounding error away from 1 (one sampled row of 64 entries: every fourth).  Blocks of 8 layers read a row half as often but
// leave two waves per SIMD: 15 % slower here, 77 instead of 33 us at 8 layers.
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

template <int BL>
__global__ __launch_bounds__(kSimThreads) void similarity_kernel(sim_params p)
{
    // The block pairs of a head, off the diagonal first (they have twice the work), and inside a kind head by head: what runs at
    // the same time on an XCD are all the block pairs of a few heads, which walk the same rows and find them in its L2.
    const int x = blockIdx.x % p.heads_by_xcd, hx = p.H / p.heads_by_xcd;
    int rest = blockIdx.x / p.heads_by_xcd;
    const int h = rest % hx * p.heads_by_xcd + x;
    rest /= hx;
    const int half = rest % kSimHalves;
    rest = p.pair0 + rest / kSimHalves;
    const int noff = p.nblk * (p.nblk - 1) / 2;
    int A = rest - noff, B = A;
    if (rest < noff) {
        A = 0;
        while (rest >= p.nblk - 1 - A) { rest -= p.nblk - 1 - A; ++A; }
        B = A + 1 + rest;
    }
    const bool diag = A == B;
    const int nA = min(BL, p.L - A * BL), nB = min(BL, p.L - B * BL); // layers of the two blocks
    const size_t vec = p.rows / 4; // (the entry point takes R * n in multiples of 4 only)
    const size_t v_lo = vec * half / kSimHalves, v_hi = vec * (half + 1) / kSimHalves;
    float acc[BL][BL];
#pragma unroll
    for (int i = 0; i < BL; ++i)
#pragma unroll
        for (int j = 0; j < BL; ++j) acc[i][j] = 0.f;
    const sim_f4 *ra[BL], *rb[BL]; // (layers past the last repeat it; their sums are not formed)
#pragma unroll
    for (int i = 0; i < BL; ++i) {
        ra[i] = (const sim_f4 *)(p.att + ((size_t)(A * BL + min(i, nA - 1)) * p.H + h) * p.rows);
        rb[i] = (const sim_f4 *)(p.att + ((size_t)(B * BL + min(i, nB - 1)) * p.H + h) * p.rows);
    }
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
    sim_f4 na[BL], nb = {};
    auto request_a = [&](size_t v) {
#pragma unroll
        for (int i = 0; i < BL; ++i) na[i] = ra[i][v];
    };
    size_t v = v_lo + threadIdx.x;
    if (v < v_hi) {
        request_a(v);
        if (!diag) nb = rb[0][v];
    }
    for (; v < v_hi; v += kSimThreads) {
        const bool more = v + kSimThreads < v_hi;
        sim_f4 xa[BL];
        f2 ea[BL];
#pragma unroll
        for (int i = 0; i < BL; ++i) xa[i] = na[i];
        if (more) request_a(v + kSimThreads);
#pragma unroll
        for (int i = 0; i < BL; ++i) ea[i] = halve(xa[i]);
        if (diag) {
#pragma unroll
            for (int i = 0; i < BL; ++i)
#pragma unroll
                for (int j = i + 1; j < BL; ++j)
                    if (j < nA) acc[i][j] += pair_term(ea[i], ea[j], xa[i], xa[j]); // (wave-uniform)
        } else {
#pragma unroll
            for (int j = 0; j < BL; ++j) {
                sim_f4 xb = nb;
                if (j + 1 < BL) nb = rb[j + 1 < BL ? j + 1 : 0][v];
                else if (more) nb = rb[0][v + kSimThreads];
                if (j < nB) { // (wave-uniform)
                    const f2 eb = halve(xb);
#pragma unroll
                    for (int i = 0; i < BL; ++i) {
                        acc[i][j] += pair_term(ea[i], eb, xa[i], xb);
                        if (i & 1) __builtin_amdgcn_sched_barrier(0); // (else the scheduler spreads the pairs out until registers spill)
                    }
                }
            }
        }
    }
    // workgroup reduction, pair by pair
    __shared__ float part[kSimThreads / 64][BL * BL];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int i = 0; i < BL; ++i)
#pragma unroll
        for (int j = 0; j < BL; ++j) {
            float t = acc[i][j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
            if (lane == 0) part[wave][i * BL + j] = t;
        }
    __syncthreads();
    if (threadIdx.x < BL * BL) {
        const int i = threadIdx.x / BL, j = threadIdx.x % BL;
        const int a = A * BL + i, b = B * BL + j;
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

template <int BL>
int launch_pairs(sim_params p, hipStream_t st)
{
    p.nblk = (p.L + BL - 1) / BL;
    const int64_t pairs = (int64_t)p.nblk * (p.nblk + 1) / 2;
    const unsigned per_pair = (unsigned)p.H * kSimHalves, most = kSimLaunch / per_pair;
    for (int64_t lo = 0; lo < pairs; lo += most) {
        p.pair0 = (int)lo;
        const unsigned here = (unsigned)(pairs - lo < most ? pairs - lo : most);
        hipLaunchKernelGGL(similarity_kernel<BL>, dim3(here * per_pair), dim3(kSimThreads), 0, st, p);
        POD_HIP_TRY(hipGetLastError());
    }
    return POD_OK;
}

} // namespace

int pod_launch_similarity(const float *att, int L, int H, int R, int n, float *sim, hipStream_t st)
{
    sim_params p;
    p.att = att; p.sim = sim; p.L = L; p.H = H; p.nblk = 0; p.pair0 = 0;
    p.rows = (size_t)R * n;
    p.R = R;
    p.heads_by_xcd = H % 8 == 0 ? 8 : 1;
    // Blocks of four layers where they leave two workgroups per CU, else of two: more workgroups, which read a row more
    // often, for few heads or layers, whose rows come out of the L2 (8 layers x 4 heads: 22 us in blocks of two, 24 in blocks of four).
    int dev = 0, cus = 0;
    POD_HIP_TRY(hipGetDevice(&dev));
    POD_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    auto workgroups = [&](int bl) { const long nb = (L + bl - 1) / bl; return nb * (nb + 1) / 2 * kSimHalves * H; };
    if (L > 1) {
        const int rc = workgroups(4) >= 2 * cus ? launch_pairs<4>(p, st) : launch_pairs<2>(p, st);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(similarity_finish_kernel, dim3((unsigned)(((size_t)L * L + 255) / 256), (unsigned)H), dim3(256), 0, st, p);
    POD_HIP_TRY(hipGetLastError());
    return POD_OK;
}
