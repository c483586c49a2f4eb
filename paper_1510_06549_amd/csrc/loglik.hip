// loglik.hip -- joint log p(W, Z, R) of the current state, fp64 (gfx950).
//
// The collapsed joint of the thesis's blocked-Gibbs derivation with P = I,
// as four sums (each written as fixed-order block partials, then reduced in a
// fixed order, so the value is bit-reproducible):
//   cells     sum_{g,k,w: n>0} log S^n_{t,a} - log C(n, t)
//   base      sum_k lgamma(V gamma) - lgamma(V gamma + B_k)
//                   + sum_w lgamma(gamma + B_wk) - lgamma(gamma)
//   PYP       sum_{g,k} log (b|a)_{T_gk} - log (b)_{N_gk}
//   documents sum_d lgamma(K alpha) - lgamma(K alpha + L_d)
//                   + sum_k lgamma(alpha + n_dk) - lgamma(alpha)
// With word associations (non-identity P^g) the base counts B_wk are keyed by
// each head's source word, and the joint gains the association factor of the
// thesis's joint with the v variables: one p_{g,w,v} per table head,
//   heads     sum_{i: r_i = 1} log p_{g(i), w_i, v_i}.
// A cell with t > n or t = 0 < n (zero probability) raises the flag beside
// the value.
//
// One launch computes all parts, a range of its blocks each, and a second
// reduces them and leaves value and flag together: nine launches and two
// copies of a few microseconds each, most with too little work to fill the
// chip, made a likelihood of 3 million tokens and 100 topics about 290 us; now
// it is 39 + 6 us of kernels and the wait for the result.  What is left is
// bound by latency (a document's histogram; the gathers of log S), so the
// kernel keeps to eight waves a SIMD (57 registers: lgamma is a call and rare;
// at 205 registers, two waves, it took 63 us).
// - Counts are read where the samplers read them, a narrow row from its
//   16-bit copy, four cells a thread and four rows in flight.
// - log-gamma of alpha + c, gamma + c and K alpha + c comes from a table for
//   c < kLgammaTable, written when the state is created: the same differences
//   of lgamma values as without, and lgamma costs some 150 fp64 instructions.
#include "spdp_internal.hpp"

namespace spdp {

namespace {

constexpr int kLBlock = 256, kLWaves = kLBlock / 64;
constexpr int kDocBlocks = 2048;   // at most; two documents a wave while there are fewer
constexpr int kCellBlocks = 2048;  // at most; kCellRows rows a thread while there are fewer
constexpr int kCellRows = 4;
constexpr int kBaseBlocks = 512;
constexpr int kPypBlocks = 64;
constexpr int kHeadBlocks = 1024;  // word associations only
constexpr int kAllBlocks = kDocBlocks + kCellBlocks + kBaseBlocks + kPypBlocks + kHeadBlocks;
constexpr int kFinalBlock = 1024;

struct LogLikArgs {
    int32_t docs, cells, base, pyp;  // blocks of each part; the rest sum heads
    int32_t D, V, G, K, Kp, ncap, Sp;
    int64_t N, rows;
    double alpha, gamma, a, b;
    const double *lgt;  // [3][kLgammaTable]
    const int64_t *doc_off;
    const int32_t *zr, *nt, *B, *Bk, *Ngk, *Tgk, *gw;
    const uint16_t *nt16;
    const uint8_t *row_narrow;
    const double *logS, *lfact, *p64;
    double *partial;
    int32_t *bad;
};

template <int BLOCK>
__device__ double block_sum(double v)
{
    __shared__ double part[BLOCK / 64];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) part[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < BLOCK / 64; ++i) s += part[i];
    return s;
}

// lgamma(x + c) - lgamma(x)
__device__ __attribute__((noinline)) double lgamma_over(double x, double c)
{
    return lgamma(x + c) - lgamma(x);
}

__device__ __forceinline__ double lgamma_of(const double *__restrict__ table, double x, int64_t c)
{
    return c < kLgammaTable ? table[c] : lgamma_over(x, (double)c);
}

__global__ void k_lgamma_table(double alpha, double gamma, double Ka, double *__restrict__ lgt)
{
    const int32_t c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= kLgammaTable) return;
    lgt[c] = lgamma_over(alpha, (double)c);
    lgt[kLgammaTable + c] = lgamma_over(gamma, (double)c);
    lgt[2 * kLgammaTable + c] = lgamma_over(Ka, (double)c);
}

// log (x|y)_T = sum_{j<T} log(x + j y)
__device__ __forceinline__ double log_poch(double x, double y, int32_t T)
{
    if (T <= 0) return 0.0;
    if (y == 0.0) return (double)T * log(x);
    return (double)T * log(y) + lgamma_over(x / y, (double)T);
}

// One wave per document (LDS histogram of its topics), strided over the blocks.
__device__ double docs_part(const LogLikArgs &A, int32_t blk, int32_t *hist_all)
{
    const int32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int32_t *hist = hist_all + wave * A.Kp;
    const double Ka = (double)A.K * A.alpha;
    double acc = 0.0;
    for (int32_t d = blk * kLWaves + wave; d < A.D; d += A.docs * kLWaves) {
        const int64_t beg = A.doc_off[d], end = A.doc_off[d + 1];
        for (int32_t k = lane; k < A.K; k += 64) hist[k] = 0;
        __threadfence_block();
        __builtin_amdgcn_wave_barrier();
        for (int64_t i = beg + lane; i < end; i += 64) atomicAdd(&hist[zr_topic(A.zr[i])], 1);
        __threadfence_block();
        __builtin_amdgcn_wave_barrier();
        for (int32_t k = lane; k < A.K; k += 64) {
            const int32_t c = hist[k];
            if (c > 0) acc += lgamma_of(A.lgt, A.alpha, c);
        }
        if (lane == 0) acc -= lgamma_of(A.lgt + 2 * kLgammaTable, Ka, end - beg);
        __threadfence_block();
        __builtin_amdgcn_wave_barrier();
    }
    return acc;
}

// Four cells of a row per thread, as many rows side by side as fit the block.
__device__ double cells_part(const LogLikArgs &A, int32_t blk, bool &bad)
{
    const int32_t units = A.Kp >> 2, per = kLBlock / units;  // Kp is a multiple of 32, <= 1024
    const int32_t y = (int32_t)threadIdx.x / units, k = 4 * ((int32_t)threadIdx.x - y * units);
    if (y >= per) return 0.0;
    double acc = 0.0;
    const int64_t step = (int64_t)A.cells * per;
    for (int64_t q0 = (int64_t)blk * per + y; q0 < A.rows; q0 += kCellRows * step) {
        bool nar[kCellRows];
        uint2 lo[kCellRows], hi[kCellRows];
#pragma unroll
        for (int j = 0; j < kCellRows; ++j) {
            const int64_t q = q0 + j * step;
            nar[j] = A.row_narrow[q < A.rows ? q : q0] != 0;
        }
#pragma unroll
        for (int j = 0; j < kCellRows; ++j) {
            const int64_t q = q0 + j * step, at = (q < A.rows ? q : q0) * A.Kp + k;
            // a narrow row's four cells are one 8-byte word, a wide row's two
            const char *p = nar[j] ? reinterpret_cast<const char *>(A.nt16 + at)
                                   : reinterpret_cast<const char *>(A.nt + at);
            lo[j] = *reinterpret_cast<const uint2 *>(p);
            hi[j] = *reinterpret_cast<const uint2 *>(p + (nar[j] ? 0 : 8));
        }
#pragma unroll
        for (int j = 0; j < kCellRows; ++j) {
            if (q0 + j * step >= A.rows) break;
            const int32_t cell[4] = {
                nar[j] ? wide_of(lo[j].x & 0xFFFF) : (int32_t)lo[j].x,
                nar[j] ? wide_of(lo[j].x >> 16) : (int32_t)lo[j].y,
                nar[j] ? wide_of(lo[j].y & 0xFFFF) : (int32_t)hi[j].x,
                nar[j] ? wide_of(lo[j].y >> 16) : (int32_t)hi[j].y};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int32_t nn = cell[c] & kCountMax, tt = cell[c] >> kCountBits;
                if (cell[c] == 0) continue;
                if (tt <= 0 || tt > nn || nn > A.ncap) {
                    bad = true;
                    continue;
                }
                acc += A.logS[tri_index(nn, tt)] -
                       (A.lfact[nn] - A.lfact[tt] - A.lfact[nn - tt]);
            }
        }
    }
    return acc;
}

__device__ double base_part(const LogLikArgs &A, int32_t blk)
{
    const double *table = A.lgt + kLgammaTable;
    const int4 *B4 = reinterpret_cast<const int4 *>(A.B);
    const int64_t n4 = (int64_t)A.V * A.Kp / 4, stride = (int64_t)A.base * kLBlock;
    double acc = 0.0;
    for (int64_t i = (int64_t)blk * kLBlock + threadIdx.x; i < n4; i += stride) {
        const int4 x = B4[i];
        if (x.x > 0) acc += lgamma_of(table, A.gamma, x.x);
        if (x.y > 0) acc += lgamma_of(table, A.gamma, x.y);
        if (x.z > 0) acc += lgamma_of(table, A.gamma, x.z);
        if (x.w > 0) acc += lgamma_of(table, A.gamma, x.w);
    }
    return acc;
}

// the PYP terms, and the normalisers of the base
__device__ double pyp_part(const LogLikArgs &A, int32_t blk)
{
    const double Vg = (double)A.V * A.gamma;
    const int64_t nres = (int64_t)A.G * A.K, stride = (int64_t)A.pyp * kLBlock;
    double acc = 0.0;
    for (int64_t j = (int64_t)blk * kLBlock + threadIdx.x; j < nres; j += stride) {
        const int64_t g = j / A.K, k = j - g * A.K, idx = g * A.Kp + k;
        acc += log_poch(A.b, A.a, A.Tgk[idx]) - log_poch(A.b, 1.0, A.Ngk[idx]);
        if (g == 0) acc -= lgamma_over(Vg, (double)A.Bk[k]);
    }
    return acc;
}

// sum over table heads of log p of the head's source (word associations)
__device__ double heads_part(const LogLikArgs &A, int32_t blk, int32_t blocks)
{
    double acc = 0.0;
    const int64_t stride = (int64_t)blocks * kLBlock;
    for (int64_t i = (int64_t)blk * kLBlock + threadIdx.x; i < A.N; i += stride) {
        const int32_t v = A.zr[i];
        if (v & 1) acc += log(A.p64[(int64_t)A.gw[i] * A.Sp + zr_slot(v)]);
    }
    return acc;
}

__global__ void __launch_bounds__(kLBlock) __attribute__((amdgpu_waves_per_eu(8)))
k_ll_parts(LogLikArgs A)
{
    extern __shared__ int32_t hist[];
    int32_t blk = (int32_t)blockIdx.x, left = (int32_t)gridDim.x;
    double acc;
    bool bad = false;
    // the parts with the longest chains first
    if (blk < A.docs) acc = docs_part(A, blk, hist);
    else if ((blk -= A.docs, left -= A.docs, blk) < A.pyp) acc = pyp_part(A, blk);
    else if ((blk -= A.pyp, left -= A.pyp, blk) < A.cells) acc = cells_part(A, blk, bad);
    else if ((blk -= A.cells, left -= A.cells, blk) < A.base) acc = base_part(A, blk);
    else acc = heads_part(A, blk - A.base, left - A.base);
    const int any_bad = __syncthreads_or(bad);
    const double s = block_sum<kLBlock>(acc);
    if (threadIdx.x == 0) {
        A.partial[blockIdx.x] = s;
        A.bad[blockIdx.x] = any_bad;
    }
}

// out = {the sum, 1 if any block met a bad cell}
__global__ void __launch_bounds__(kFinalBlock) k_ll_final(int32_t n,
                                                          const double *__restrict__ partial,
                                                          const int32_t *__restrict__ bad,
                                                          double *__restrict__ out)
{
    double acc = 0.0;
    int any = 0;
#pragma unroll 4
    for (int32_t i = threadIdx.x; i < n; i += kFinalBlock) {
        acc += partial[i];
        any |= bad[i];
    }
    const int any_bad = __syncthreads_or(any);
    const double s = block_sum<kFinalBlock>(acc);
    if (threadIdx.x == 0) {
        out[0] = s;
        out[1] = any_bad ? 1.0 : 0.0;
    }
}

int32_t at_most(int64_t blocks, int32_t most)
{
    return blocks < 1 ? 1 : (blocks < most ? (int32_t)blocks : most);
}

}  // namespace

// (the flags take half a double each)
int64_t loglik_partials_needed() { return kAllBlocks + (kAllBlocks + 1) / 2; }

hipError_t launch_lgamma_table(const Model &m, double *lgt, hipStream_t st)
{
    hipLaunchKernelGGL(k_lgamma_table, dim3(kLgammaTable / kLBlock), dim3(kLBlock), 0, st, m.alpha,
                       m.gamma, (double)m.K * m.alpha, lgt);
    return hipGetLastError();
}

hipError_t launch_loglik(const Model &m, const DeviceBuffers &b, const int32_t *zr,
                         hipStream_t st)
{
    LogLikArgs A{};
    A.rows = (int64_t)m.G * m.V;
    const int64_t per = (int64_t)(kLBlock / (m.Kp / 4)) * kCellRows;
    A.docs = at_most(((int64_t)m.D + 2 * kLWaves - 1) / (2 * kLWaves), kDocBlocks);
    A.cells = at_most((A.rows + per - 1) / per, kCellBlocks);
    A.base = at_most((int64_t)m.V * m.Kp / (8 * kLBlock), kBaseBlocks);
    A.pyp = at_most(((int64_t)m.G * m.K + kLBlock - 1) / kLBlock, kPypBlocks);
    const int32_t heads = m.Sp > 0 ? kHeadBlocks : 0;
    const int32_t all = A.docs + A.cells + A.base + A.pyp + heads;
    A.D = m.D;
    A.V = m.V;
    A.G = m.G;
    A.K = m.K;
    A.Kp = m.Kp;
    A.ncap = m.ncap;
    A.Sp = m.Sp;
    A.N = m.N;
    A.alpha = m.alpha;
    A.gamma = m.gamma;
    A.a = m.a;
    A.b = m.b;
    A.lgt = b.lgt;
    A.doc_off = b.doc_off;
    A.zr = zr;
    A.nt = b.nt;
    A.B = b.B;
    A.Bk = b.Bk;
    A.Ngk = b.Ngk;
    A.Tgk = b.Tgk;
    A.gw = b.gw;
    A.nt16 = b.nt16;
    A.row_narrow = b.row_narrow;
    A.logS = b.logS;
    A.lfact = b.lfact;
    A.p64 = b.p64;
    A.partial = b.partial;
    A.bad = reinterpret_cast<int32_t *>(b.partial + kAllBlocks);
    hipLaunchKernelGGL(k_ll_parts, dim3((unsigned)all), dim3(kLBlock),
                       (size_t)kLWaves * m.Kp * sizeof(int32_t), st, A);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_ll_final, dim3(1), dim3(kFinalBlock), 0, st, all, A.partial, A.bad,
                       b.scalar);
    return hipGetLastError();
}

}  // namespace spdp
