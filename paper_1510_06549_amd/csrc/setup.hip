// setup.hip -- state construction and count maintenance kernels (gfx950).
//
//   make_gw        token -> count-row index g V + w, per-(g, w) token counts
//   stirling       log S^n_{t,a} rows (fp64 recurrence of the PYP joint,
//                  Corollary 17 passage) and the folded ratio pairs used by the
//                  sampler (Eq. SPDP-sampling-w-z-r0 / -r1 with P = I)
//   init_z         initial topics from Philox (purpose INIT), r = 0
//   totals         N_gk, T_gk by an LDS-privatised histogram; B_k = sum_g T_gk
//   factors        per-(g, k) sweep constants of the conditionals
#include <climits>

#include "spdp_internal.hpp"

namespace spdp {

namespace {

constexpr int kBlock = 256;

inline int64_t blocks_for(int64_t n, int per_block)
{
    int64_t b = (n + per_block - 1) / per_block;
    return b < 1 ? 1 : b;
}

// ----------------------------------------------------------------- fills
template <typename T>
__global__ void k_fill(T *__restrict__ p, int64_t n, T v)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

template <typename T>
hipError_t fill(T *p, int64_t n, T v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    int64_t nb = blocks_for(n, kBlock);
    if (nb > 65536) nb = 65536;
    hipLaunchKernelGGL(k_fill<T>, dim3((unsigned)nb), dim3(kBlock), 0, st, p, n, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------- make_gw
// One block per document at a time: row index per token, validation, per-row
// counts.  The grid is bounded, as a launch takes fewer than 2^32 threads.
constexpr int32_t kGwBlocks = 1 << 20;
__global__ void k_make_gw(int32_t D, int32_t V, int32_t G, const int32_t *words,
                          const int64_t *__restrict__ doc_off, const int32_t *__restrict__ doc_group,
                          int32_t *gw, int32_t *__restrict__ gw_count,
                          int32_t *__restrict__ bad)
{
    for (int64_t d = blockIdx.x; d < D; d += gridDim.x) {
        const int32_t g = doc_group[d];
        const int64_t beg = doc_off[d], end = doc_off[d + 1];
        if (g < 0 || g >= G) {
            if (threadIdx.x == 0) atomicOr(bad, 1);
            continue;
        }
        for (int64_t i = beg + threadIdx.x; i < end; i += blockDim.x) {
            const int32_t w = words[i];
            if (w < 0 || w >= V) {
                atomicOr(bad, 2);
                gw[i] = 0;
                continue;
            }
            const int32_t q = g * V + w;
            gw[i] = q;
            if (gw_count) atomicAdd(gw_count + q, 1);
        }
    }
}

// ------------------------------------------------------------ narrow rows
// A row is narrow if its (group, word) pair occurs at most kNarrowMax times:
// no count of the row can then exceed kNarrowMax.
// The two counters get one pair of atomics per block, from a grid of a few
// blocks per compute unit (a pair per wavefront: 178 us for 468 000 rows).
__global__ void __launch_bounds__(kBlock) k_row_narrow(int64_t rows,
                                                       const int32_t *__restrict__ gw_count,
                                                       uint8_t *__restrict__ row_narrow,
                                                       unsigned long long *__restrict__ n)
{
    __shared__ int32_t sum[2];
    if (threadIdx.x < 2) sum[threadIdx.x] = 0;
    __syncthreads();
    int32_t c = 0, u = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < rows; q += stride) {
        const int32_t have = gw_count[q];
        row_narrow[q] = have <= kNarrowMax ? 1 : 0;
        c += have <= kNarrowMax;
        u += have > 0;
    }
    for (int o = 32; o > 0; o >>= 1) {
        c += __shfl_xor(c, o);
        u += __shfl_xor(u, o);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&sum[0], c);
        atomicAdd(&sum[1], u);
    }
    __syncthreads();
    if (threadIdx.x < 2 && sum[threadIdx.x])
        atomicAdd(n + threadIdx.x, (unsigned long long)sum[threadIdx.x]);
}

__global__ void k_tok_narrow(int64_t N, const int32_t *__restrict__ gw,
                             const uint8_t *__restrict__ row_narrow,
                             uint8_t *__restrict__ tok_narrow)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) tok_narrow[i] = row_narrow[gw[i]];
}

// --------------------------------------------------------------- max int32
__global__ void k_max_i32(const int32_t *__restrict__ x, int64_t n, int32_t *__restrict__ out)
{
    int32_t m = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        m = max(m, x[i]);
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
    __shared__ int32_t wave[kBlock / 64];
    if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) m = max(m, wave[w]);
        atomicMax(out, m);
    }
}

// --------------------------------------------------------------- Stirling
// Row n + 1 from row n,
//   S^{n+1}_t = S^n_{t-1} + (n - t a) S^n_t,  S^n_0 = [n == 0],  S^n_t = 0 (t > n),
// in log space (log-sum-exp of the two terms).  A launch takes kBand rows, a
// block the columns [t0, t0 + kBandCols) of them: an entry needs the one above
// and the one left of it, so the block also forms the kBand columns left of its
// own, one fewer each row, and blocks are independent.  The rows are a chain of
// exp and log1p either way; one workgroup for all columns was bound by its own
// compute unit instead (ncap = 808: 1.37 ms, now 0.62; 2 630: 9.1 ms, now 2.0).
// The logarithm of the factor does not depend on the chain and is taken a row ahead.
constexpr int kBand = 64, kBandCols = 192;
__global__ void __launch_bounds__(kBand + kBandCols) k_stirling_rows(int32_t n0, int32_t nmax,
                                                                     double a,
                                                                     double *__restrict__ logS)
{
    __shared__ double row[2][kBand + kBandCols + 1];
    const int32_t c = threadIdx.x;
    const int32_t t = (int32_t)blockIdx.x * kBandCols - kBand + c;  // this thread's column
    const int32_t rows = nmax - n0 < kBand ? nmax - n0 : kBand;
    if (c == 0) row[0][0] = row[1][0] = -INFINITY;
    double same = -INFINITY;
    if (t >= 0 && t <= n0) same = n0 == 0 ? 0.0 : logS[tri_index(n0, t)];
    if (n0 == 0 && t == 0 && c >= kBand) logS[0] = 0.0;
    row[0][c + 1] = same;
    // log(n - t a) of the row being formed from row n (used only for t <= n)
    double factor = t >= 0 && t <= n0 ? log((double)n0 - (double)t * a) : 0.0;
    __syncthreads();
    for (int32_t i = 0; i < rows; ++i) {
        const int32_t n = n0 + i;
        const double left = row[i & 1][c];
        double v = -INFINITY;
        if (t > 0 && t <= n + 1) {
            const double term = (t > n || same == -INFINITY) ? -INFINITY : same + factor;
            if (left == -INFINITY) v = term;
            else if (term == -INFINITY) v = left;
            else {
                const double hi = fmax(left, term), lo = fmin(left, term);
                v = hi + log1p(exp(lo - hi));
            }
        }
        if (t >= 0 && t <= n + 1) factor = log((double)(n + 1) - (double)t * a);
        same = v;
        row[(i + 1) & 1][c + 1] = v;
        if (c >= kBand && t <= n + 1) logS[tri_index(n + 1, t)] = v;
        __syncthreads();
    }
}

// Folded ratio pairs for 0 <= t <= n < nmax, computed in fp64:
//   Q0(n, t) = (n - t + 1)/(n + 1) * S^{n+1}_t / S^n_t        (outcome r = 0)
//   Q1(n, t) = (t + 1)/(n + 1) * S^{n+1}_{t+1} / S^n_t        (outcome r = 1)
// with Q(0, 0) = (0, 1); entries with t = 0 < n (no valid state) are (0, 0).
// Q holds them rounded once to fp32 (the sampling path), Q64 in fp64 (the
// boundary path), each factor evaluated as the conditional states it: the
// count ratio divided out, times the exponential of the log-table difference.
__global__ void k_stirling_pairs(int32_t nmax, const double *__restrict__ logS,
                                 float2 *__restrict__ Q, double2 *__restrict__ Q64)
{
    const int64_t n = blockIdx.y;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= nmax || t > n) return;
    float2 q;
    double2 q64;
    if (n == 0) {
        q = make_float2(0.0f, 1.0f);
        q64 = make_double2(0.0, 1.0);
    } else if (t == 0) {
        q = make_float2(0.0f, 0.0f);
        q64 = make_double2(0.0, 0.0);
    } else {
        const double base = logS[tri_index(n, t)];
        const double r0 = exp(logS[tri_index(n + 1, t)] - base);
        const double r1 = exp(logS[tri_index(n + 1, t + 1)] - base);
        const double inv = 1.0 / (double)(n + 1);
        q = make_float2((float)((double)(n - t + 1) * inv * r0), (float)((double)(t + 1) * inv * r1));
        q64 = make_double2((double)(n - t + 1) / (double)(n + 1) * r0,
                           (double)(t + 1) / (double)(n + 1) * r1);
    }
    Q[tri_index(n, t)] = q;
    Q64[tri_index(n, t)] = q64;
}

__global__ void k_lfact(int32_t nmax, double *__restrict__ lfact)
{
    const int64_t n = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (n <= nmax) lfact[n] = lgamma((double)n + 1.0);
}

// ----------------------------------------------------------------- init z
__global__ void k_init_z(int64_t N, int32_t K, uint64_t seed, int32_t *__restrict__ zr)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const uint32_t x = philox_x0(seed, (uint64_t)i, 0u, kPurposeInit);
    const int32_t z = (int32_t)(((uint64_t)x * (uint64_t)K) >> 32);
    zr[i] = zr_pack(z, 0);
}

__global__ void k_pack_zr(int64_t N, int32_t K, const int32_t *__restrict__ z,
                          const uint8_t *__restrict__ r, int32_t *__restrict__ zr,
                          int32_t *__restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    int32_t zi = z[i];
    int32_t ri = r[i];
    if (zi < 0 || zi >= K || ri > 1) {
        atomicOr(bad, 4);
        zi = 0;
        ri = 0;
    }
    zr[i] = zr_pack(zi, ri);
}

// Word associations: (z, r, s) -> zr; a head's slot must hold a source of its
// row (p > 0), a token with r = 0 stores slot 0.
__global__ void k_pack_zrs(int64_t N, int32_t K, int32_t Sp, const int32_t *__restrict__ gw,
                           const double *__restrict__ p64, const int32_t *__restrict__ z,
                           const uint8_t *__restrict__ r, const uint8_t *__restrict__ s,
                           int32_t *__restrict__ zr, int32_t *__restrict__ bad)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    int32_t zi = z[i];
    int32_t ri = r[i];
    int32_t si = s ? (int32_t)s[i] : 0;
    if (ri == 0) si = 0;
    if (zi < 0 || zi >= K || ri > 1 || si >= Sp || !(p64[(int64_t)gw[i] * Sp + si] > 0.0)) {
        atomicOr(bad, 4);
        zi = 0;
        ri = 0;
        si = 0;
    }
    zr[i] = zr_pack(zi, ri, si);
}

__global__ void k_unpack_slot(int64_t N, const int32_t *__restrict__ zr, uint8_t *__restrict__ s)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    s[i] = (uint8_t)zr_slot(zr[i]);
}

__global__ void k_unpack_zr(int64_t N, const int32_t *__restrict__ zr, int32_t *__restrict__ z,
                            uint8_t *__restrict__ r)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int32_t v = zr[i];
    if (z) z[i] = zr_topic(v);
    if (r) r[i] = (uint8_t)(v & 1);
}

// ----------------------------------------------------------------- totals
// Per block, a chunk of at most 32768 tokens is histogrammed into LDS bins of
// (g, k), each bin packing customers (low 16 bits) and tables (high 16 bits);
// non-zero bins are flushed with global atomics.  Chunks are shorter where
// there would be fewer blocks than compute units (500 000 tokens: 13 us
// in 16 blocks, 4.6 us in 244), down to a few tokens per thread.
constexpr int kTotalsChunk = 32768, kTotalsLeast = 2048;

inline int32_t totals_chunk(int64_t N)
{
    int32_t c = kTotalsChunk;
    while (c > kTotalsLeast && N / c < 256) c /= 2;
    return c;
}

__global__ void __launch_bounds__(1024) k_totals_lds(int64_t N, int32_t chunk, int32_t Kp,
                                                     int32_t bins,
                                                     FastDiv divV, const int32_t *__restrict__ gw,
                                                     const int32_t *__restrict__ zr,
                                                     int32_t *__restrict__ Ngk,
                                                     int32_t *__restrict__ Tgk)
{
    extern __shared__ uint32_t h[];
    for (int j = threadIdx.x; j < bins; j += blockDim.x) h[j] = 0u;
    __syncthreads();
    const int64_t beg = (int64_t)blockIdx.x * chunk;
    const int64_t end = min(beg + (int64_t)chunk, N);
    for (int64_t i = beg + threadIdx.x; i < end; i += blockDim.x) {
        const int32_t v = zr[i];
        const int32_t g = (int32_t)fastdiv((uint32_t)gw[i], divV);
        atomicAdd(&h[g * Kp + zr_topic(v)], 1u + ((uint32_t)(v & 1) << 16));
    }
    __syncthreads();
    for (int j = threadIdx.x; j < bins; j += blockDim.x) {
        const uint32_t x = h[j];
        if (x) {
            atomicAdd(Ngk + j, (int32_t)(x & 0xFFFFu));
            if (x >> 16) atomicAdd(Tgk + j, (int32_t)(x >> 16));
        }
    }
}

__global__ void k_totals_global(int64_t N, int32_t Kp, FastDiv divV,
                                const int32_t *__restrict__ gw, const int32_t *__restrict__ zr,
                                int32_t *__restrict__ Ngk, int32_t *__restrict__ Tgk)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const int32_t v = zr[i];
    const int32_t g = (int32_t)fastdiv((uint32_t)gw[i], divV);
    atomicAdd(Ngk + g * Kp + zr_topic(v), 1);
    if (v & 1) atomicAdd(Tgk + g * Kp + zr_topic(v), 1);
}

__global__ void k_topic_tables(int32_t G, int32_t Kp, const int32_t *__restrict__ Tgk,
                               int32_t *__restrict__ Bk)
{
    const int32_t k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= Kp) return;
    int32_t s = 0;
    for (int32_t g = 0; g < G; ++g) s += Tgk[(int64_t)g * Kp + k];
    Bk[k] = s;
}

// ---------------------------------------------------------------- factors
// Per-(g, k) constants of the conditionals, computed in fp64 and rounded once:
//   f0 = 1 / (b + N_gk),   f1 = (b + a T_gk) / (b + N_gk) / (V gamma + B_k)
// and, for the topic a token is removed from (N >= 1 there),
//   fk[0] = 1 / (b + N - 1)
//   fk[1] = (b + a T) / (b + N - 1) / (V gamma + B_k)            (r = 0 removed)
//   fk[2] = (b + a (T - 1)) / (b + N - 1) / (V gamma + B_k - 1)  (r = 1 removed)
// Padding topics (k >= K) get 0, so their outcomes carry zero weight.  fz (may
// be null) holds the same five per topic: {fk[0], fk[1], fk[2], 0}, {f0, f1, 0, 0}.
struct FactorArgs {
    const int32_t *Ngk, *Tgk;
    float *f0, *f1, *fk;
    float4 *fz;
    int64_t GK;
    int32_t K;
    double a, b, Vgamma;
};

__device__ __forceinline__ void factors_of(const FactorArgs &A, int64_t j, int32_t k, int32_t Bk)
{
    float c0 = 0.0f, c1 = 0.0f, d0 = 0.0f, d1 = 0.0f, d2 = 0.0f;
    if (k < A.K) {
        const double N = (double)A.Ngk[j], T = (double)A.Tgk[j], B = (double)Bk;
        const double inv = 1.0 / (A.b + N);
        c0 = (float)inv;
        c1 = (float)((A.b + A.a * T) * inv / (A.Vgamma + B));
        if (A.Ngk[j] >= 1) {
            const double invm = 1.0 / (A.b + N - 1.0);
            d0 = (float)invm;
            d1 = (float)((A.b + A.a * T) * invm / (A.Vgamma + B));
            if (A.Tgk[j] >= 1)
                d2 = (float)((A.b + A.a * (T - 1.0)) * invm / (A.Vgamma + B - 1.0));
        }
    }
    A.f0[j] = c0;
    A.f1[j] = c1;
    A.fk[j] = d0;
    A.fk[A.GK + j] = d1;
    A.fk[2 * A.GK + j] = d2;
    if (A.fz) {
        A.fz[2 * j] = make_float4(d0, d1, d2, 0.0f);
        A.fz[2 * j + 1] = make_float4(c0, c1, 0.0f, 0.0f);
    }
}

__global__ void k_factors(FactorArgs A, int32_t Kp, const int32_t *__restrict__ Bk)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j < A.GK) factors_of(A, j, (int32_t)(j % Kp), Bk[j % Kp]);
}

// B_k and the constants in one launch, for few groups: a block takes
// kTabTopics topics, kTabRows threads each, which share the groups of a topic.
constexpr int kTabTopics = 8, kTabRows = 32;
__global__ void __launch_bounds__(kTabTopics *kTabRows) k_tables_factors(FactorArgs A, int32_t G,
                                                                         int32_t Kp,
                                                                         int32_t *__restrict__ Bk)
{
    __shared__ int32_t part[kTabRows][kTabTopics];
    const int32_t x = threadIdx.x % kTabTopics, y = threadIdx.x / kTabTopics;
    const int32_t k = blockIdx.x * kTabTopics + x;  // (Kp is a multiple of kTabTopics)
    int32_t s = 0;
    for (int32_t g = y; g < G; g += kTabRows) s += A.Tgk[(int64_t)g * Kp + k];
    part[y][x] = s;
    __syncthreads();
    int32_t B = 0;
#pragma unroll
    for (int i = 0; i < kTabRows; ++i) B += part[i][x];
    if (y == 0) Bk[k] = B;
    for (int32_t g = y; g < G; g += kTabRows) factors_of(A, (int64_t)g * Kp + k, k, B);
}

}  // namespace

// ======================================================================
// launchers
// ======================================================================
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t st) { return fill(p, n, v, st); }
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t st) { return fill(p, n, v, st); }
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t st)
{
    return fill(p, n, v, st);
}

hipError_t launch_make_gw(const Model &m, int32_t D, const int32_t *words, const int64_t *doc_off,
                          const int32_t *doc_group, int32_t *gw, int32_t *gw_count, int32_t *bad,
                          hipStream_t st)
{
    if (D <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_make_gw, dim3((unsigned)std::min(D, kGwBlocks)), dim3(kBlock), 0, st, D,
                       m.V, m.G, words, doc_off, doc_group, gw, gw_count, bad);
    return hipGetLastError();
}

hipError_t launch_max_i32(const int32_t *x, int64_t n, int32_t *out, hipStream_t st)
{
    int64_t nb = blocks_for(n, kBlock);
    if (nb > 1024) nb = 1024;
    hipLaunchKernelGGL(k_max_i32, dim3((unsigned)nb), dim3(kBlock), 0, st, x, n, out);
    return hipGetLastError();
}

hipError_t launch_stirling(const Model &m, double *logS, float2 *Q, double2 *Q64, double *lfact,
                           hipStream_t st)
{
    const int32_t nmax = m.ncap;  // rows 0..ncap of log S; pairs for n < ncap
    for (int32_t n0 = 0; n0 < nmax; n0 += kBand) {
        const int32_t last = nmax - n0 < kBand ? nmax : n0 + kBand;  // columns 0 .. last
        hipLaunchKernelGGL(k_stirling_rows, dim3((unsigned)(last / kBandCols + 1)),
                           dim3(kBand + kBandCols), 0, st, n0, nmax, m.a, logS);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    dim3 grid((unsigned)blocks_for(nmax, kBlock), (unsigned)nmax);
    hipLaunchKernelGGL(k_stirling_pairs, grid, dim3(kBlock), 0, st, nmax, logS, Q, Q64);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_lfact, dim3((unsigned)blocks_for(nmax + 1, kBlock)), dim3(kBlock), 0, st,
                       nmax, lfact);
    return hipGetLastError();
}

hipError_t launch_init_z(const Model &m, uint64_t seed, int32_t *zr, hipStream_t st)
{
    if (m.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_init_z, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock), 0, st, m.N,
                       m.K, seed, zr);
    return hipGetLastError();
}

hipError_t launch_pack_zr(const Model &m, const int32_t *z, const uint8_t *r, int32_t *zr,
                          int32_t *bad, hipStream_t st)
{
    if (m.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_zr, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock), 0, st, m.N,
                       m.K, z, r, zr, bad);
    return hipGetLastError();
}

hipError_t launch_pack_zrs(const Model &m, const DeviceBuffers &b, const int32_t *z,
                           const uint8_t *r, const uint8_t *s, int32_t *zr, int32_t *bad,
                           hipStream_t st)
{
    if (m.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_zrs, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock), 0, st,
                       m.N, m.K, m.Sp, b.gw, b.p64, z, r, s, zr, bad);
    return hipGetLastError();
}

hipError_t launch_unpack_slot(const Model &m, const int32_t *zr, uint8_t *s, hipStream_t st)
{
    if (m.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpack_slot, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock), 0, st,
                       m.N, zr, s);
    return hipGetLastError();
}

hipError_t launch_unpack_zr(const Model &m, const int32_t *zr, int32_t *z, uint8_t *r,
                            hipStream_t st)
{
    if (m.N <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_unpack_zr, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock), 0, st,
                       m.N, zr, z, r);
    return hipGetLastError();
}

// N_gk and T_gk of the states into arrays that are zero
static hipError_t add_totals(const Model &m, const DeviceBuffers &b, const int32_t *zr,
                             int32_t *Ngk, int32_t *Tgk, hipStream_t st)
{
    if (m.N <= 0) return hipSuccess;
    const int64_t bins = (int64_t)m.G * m.Kp;
    // (if the queries fail, lds_max stays 0 and the global-atomic histogram runs)
    int dev = 0, lds_max = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    const int64_t lds = bins * (int64_t)sizeof(uint32_t);
    if (lds <= lds_max && lds <= 96 * 1024) {
        const int32_t chunk = totals_chunk(m.N);
        const unsigned nb = (unsigned)blocks_for(m.N, chunk);
        hipLaunchKernelGGL(k_totals_lds, dim3(nb), dim3(1024), (size_t)lds, st, m.N, chunk, m.Kp,
                           (int32_t)bins, m.divV, b.gw, zr, Ngk, Tgk);
    } else {
        hipLaunchKernelGGL(k_totals_global, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock),
                           0, st, m.N, m.Kp, m.divV, b.gw, zr, Ngk, Tgk);
    }
    return hipGetLastError();
}

hipError_t launch_totals(const Model &m, const DeviceBuffers &b, const int32_t *zr, hipStream_t st)
{
    hipError_t e = add_totals(m, b, zr, b.Ngk, b.Tgk, st);
    if (e != hipSuccess) return e;
    const int64_t GK = (int64_t)m.G * m.Kp;
    const FactorArgs A{b.Ngk, b.Tgk, b.f0, b.f1, b.fk, b.fz, GK,
                       m.K,   m.a,   m.b,  (double)m.V * m.gamma};
    // one launch where each thread has at most two groups of its topic
    if (m.G <= 2 * kTabRows) {
        hipLaunchKernelGGL(k_tables_factors, dim3((unsigned)(m.Kp / kTabTopics)),
                           dim3(kTabTopics * kTabRows), 0, st, A, m.G, m.Kp, b.Bk);
    } else {
        hipLaunchKernelGGL(k_topic_tables, dim3((unsigned)blocks_for(m.Kp, kBlock)), dim3(kBlock),
                           0, st, m.G, m.Kp, b.Tgk, b.Bk);
        hipLaunchKernelGGL(k_factors, dim3((unsigned)blocks_for(GK, kBlock)), dim3(kBlock), 0, st,
                           A, m.Kp, b.Bk);
    }
    return hipGetLastError();
}

hipError_t launch_totals_into(const Model &m, const DeviceBuffers &b, const int32_t *zr,
                              int32_t *Ngk, int32_t *Tgk, int32_t *Bk, hipStream_t st)
{
    hipError_t e;
    const int64_t bins = (int64_t)m.G * m.Kp;
    if ((e = fill(Ngk, bins, 0, st)) != hipSuccess) return e;
    if ((e = fill(Tgk, bins, 0, st)) != hipSuccess) return e;
    if ((e = add_totals(m, b, zr, Ngk, Tgk, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_topic_tables, dim3((unsigned)blocks_for(m.Kp, kBlock)), dim3(kBlock), 0, st,
                       m.G, m.Kp, Tgk, Bk);
    return hipGetLastError();
}

hipError_t launch_narrow_flags(const Model &m, const int32_t *gw, const int32_t *gw_count,
                               uint8_t *row_narrow, uint8_t *tok_narrow,
                               unsigned long long *n_narrow, hipStream_t st)
{
    const int64_t rows = (int64_t)m.G * m.V;
    const unsigned nb = (unsigned)std::min<int64_t>(blocks_for(rows, kBlock), 1024);
    hipLaunchKernelGGL(k_row_narrow, dim3(nb), dim3(kBlock), 0, st, rows,
                       gw_count, row_narrow, n_narrow);
    if (m.N > 0)
        hipLaunchKernelGGL(k_tok_narrow, dim3((unsigned)blocks_for(m.N, kBlock)), dim3(kBlock), 0,
                           st, m.N, gw, row_narrow, tok_narrow);
    return hipGetLastError();
}

}  // namespace spdp
