// sample_rows.hip -- the sampler over weight rows: the plain model's instances
// of the kernel in sample_rows.hpp, the pass that computes the weight rows, the
// documents' launch order, and the choice of shape.
#include "sample_rows.hpp"

namespace spdp {

namespace {

constexpr int kBlock = 256;

struct __attribute__((packed, aligned(4))) Int4 {
    int32_t v[4];
};
struct __attribute__((packed, aligned(2))) Half4 {
    uint16_t v[4];
};
struct __attribute__((packed, aligned(4))) Float4 {
    float v[4];
};

struct WeightArgs {
    const int32_t *row_off;
    const uint8_t *row_narrow;
    const int32_t *nt;
    const uint16_t *nt16;
    const int32_t *B;
    const float *f0, *f1;
    const float2 *Q;
    const int32_t *srcrec;
    float *pw, *rho;
    int64_t rows;
    uint64_t q_last;
    FastDiv divV;
    int32_t V, K, Kp, Kw, Sp, lanes, lane_shift, kpl;
    float gamma;
};

// The weight rows of the rows that have tokens (see sample_rows.hpp).  A thread
// computes the consecutive topics of one 16-byte chunk of a row (or of one
// lane's remainder): blockDim.x threads a row, blockDim.y rows a block.  Bound
// by its bytes (a cell read, two weights written); an empty cell's ratio pair
// is (0, 1), so only cells with customers gather one.
template <bool ASSOC>
__global__ void __launch_bounds__(kBlock) k_weights(WeightArgs A)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.y + threadIdx.y;
    if (q >= A.rows || A.row_off[q] == A.row_off[q + 1]) return;
    const int32_t unit = threadIdx.x, c = unit >> A.lane_shift, l = unit - (c << A.lane_shift);
    const int32_t nc = A.kpl >> 2, rem = A.kpl & 3;
    const int32_t width = c < nc ? 4 : rem;
    const int32_t k = l * A.kpl + 4 * c;
    const int32_t g = (int32_t)fastdiv((uint32_t)q, A.divV);
    const int64_t cell = q * A.Kp + k;
    const int32_t *rec = ASSOC ? A.srcrec + q * 2 * A.Sp : nullptr;
    const int64_t w_row = (q - (int64_t)g * A.V) * A.Kp;
    int32_t x[4] = {0, 0, 0, 0};
    float beta[4] = {0.0f, 0.0f, 0.0f, 0.0f}, f0[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    float f1[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (k + 4 <= A.Kp) {  // (cells of padding topics read too: their constants are 0)
        if (A.row_narrow[q]) {
            const Half4 h = *reinterpret_cast<const Half4 *>(A.nt16 + cell);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = wide_of(h.v[i]);
        } else {
            const Int4 h = *reinterpret_cast<const Int4 *>(A.nt + cell);
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = h.v[i];
        }
        const Float4 a = *reinterpret_cast<const Float4 *>(A.f0 + (int64_t)g * A.Kp + k);
        const Float4 b = *reinterpret_cast<const Float4 *>(A.f1 + (int64_t)g * A.Kp + k);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f0[i] = a.v[i];
            f1[i] = b.v[i];
        }
        if constexpr (ASSOC) {
            for (int32_t s = 0; s < A.Sp; ++s) {
                const Int4 h =
                    *reinterpret_cast<const Int4 *>(A.B + (int64_t)rec[s] * A.Kp + k);
                const float ps = __int_as_float(rec[A.Sp + s]);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    beta[i] = __fmaf_rn(ps, A.gamma + (float)h.v[i], beta[i]);
            }
        } else {
            const Int4 h = *reinterpret_cast<const Int4 *>(A.B + w_row + k);
#pragma unroll
            for (int i = 0; i < 4; ++i) beta[i] = A.gamma + (float)h.v[i];
        }
    } else {
        for (int i = 0; i < width && k + i < A.K; ++i) {
            x[i] = A.row_narrow[q] ? wide_of(A.nt16[cell + i]) : A.nt[cell + i];
            f0[i] = A.f0[(int64_t)g * A.Kp + k + i];
            f1[i] = A.f1[(int64_t)g * A.Kp + k + i];
            if constexpr (ASSOC) {
                for (int32_t s = 0; s < A.Sp; ++s)
                    beta[i] = __fmaf_rn(__int_as_float(rec[A.Sp + s]),
                                        A.gamma + (float)A.B[(int64_t)rec[s] * A.Kp + k + i],
                                        beta[i]);
            } else {
                beta[i] = A.gamma + (float)A.B[w_row + k + i];
            }
        }
    }
    float w[4], w1[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float2 qq = make_float2(0.0f, 1.0f);
        if (x[i] != 0) {
            const uint64_t n = (uint32_t)x[i] & kCountMax, t = (uint32_t)x[i] >> kCountBits;
            const uint64_t ix = ((n * (n + 1)) >> 1) + t;
            qq = A.Q[ix < A.q_last ? ix : A.q_last];
        }
        w1[i] = f1[i] * beta[i] * qq.y;
        w[i] = w1[i] + f0[i] * qq.x;
        w1[i] = x[i] != 0 ? w1[i] / w[i] : 1.0f;  // (an empty cell has no r = 0 outcome)
    }
    const int64_t out = q * A.Kw + (c < nc ? unit * 4 : nc * A.lanes * 4 + l * rem);
    if (c < nc) {
        *reinterpret_cast<float4 *>(A.pw + out) = make_float4(w[0], w[1], w[2], w[3]);
        *reinterpret_cast<float4 *>(A.rho + out) = make_float4(w1[0], w1[1], w1[2], w1[3]);
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if (i < rem) {
                A.pw[out + i] = w[i];
                A.rho[out + i] = w1[i];
            }
        }
    }
}

// ------------------------------------------------------------ launch order
// Each XCD takes a contiguous range of documents (so that a group's rows stay
// in its L2), and within each window of kWindow documents of its range the
// longest come first, so that the documents of one wavefront have similar
// lengths and a window's longest chains start first.  A window is about what
// an XCD has in flight.  One block sorts one window (bitonic, by length and
// index, so the order is reproducible).
constexpr int kWindow = 2048;

__global__ void __launch_bounds__(kWindow / 2) k_doc_order(int32_t D, int32_t docs_per_xcd,
                                                           int32_t windows,
                                                           const int64_t *__restrict__ doc_off,
                                                           int32_t *__restrict__ order)
{
    __shared__ uint64_t key[kWindow];
    const int32_t xcd = blockIdx.x / windows, w = blockIdx.x % windows;
    const int64_t beg = (int64_t)xcd * docs_per_xcd + (int64_t)w * kWindow;
    const int64_t stop = (int64_t)(xcd + 1) * docs_per_xcd < D ? (int64_t)(xcd + 1) * docs_per_xcd : D;
    if (beg >= stop) return;
    const int32_t n = (int32_t)(stop - beg < kWindow ? stop - beg : kWindow);
    for (int32_t i = threadIdx.x; i < kWindow; i += kWindow / 2) {
        uint64_t k = ~0ull;  // (places past the end sort last)
        if (i < n) {
            const uint32_t len = (uint32_t)(doc_off[beg + i + 1] - doc_off[beg + i]);
            k = ((uint64_t)(0x7FFFFFFFu - len) << 32) | (uint32_t)i;
        }
        key[i] = k;
    }
    __syncthreads();
    for (int32_t size = 2; size <= kWindow; size <<= 1) {
        for (int32_t step = size >> 1; step > 0; step >>= 1) {
            const int32_t t = threadIdx.x;
            const int32_t a = 2 * step * (t / step) + t % step, b = a + step;
            const bool up = (a & size) == 0;
            const uint64_t ka = key[a], kb = key[b];
            if ((ka > kb) == up) {
                key[a] = kb;
                key[b] = ka;
            }
            __syncthreads();
        }
    }
    for (int32_t i = threadIdx.x; i < n; i += kWindow / 2)
        order[beg + i] = (int32_t)(beg + (int64_t)(uint32_t)key[i]);
}

// Test hook: the weights and shares of n rows topic by topic ([n][K]; 0 for a
// row without tokens), from the layout of row_pos.
__global__ void k_weight_topics(int64_t n, int32_t K, int32_t Kw, int32_t lanes, int32_t kpl,
                                const int32_t *__restrict__ row_off,
                                const float *__restrict__ pw, const float *__restrict__ rho,
                                float *__restrict__ pw_out, float *__restrict__ rho_out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * K) return;
    const int64_t q = i / K;
    const int32_t k = (int32_t)(i - q * K), l = k / kpl, j = k % kpl, c = j >> 2;
    const int32_t at = c < (kpl >> 2) ? (c * lanes + l) * 4 + (j & 3)
                                      : (kpl >> 2) * lanes * 4 + l * (kpl & 3) + (j & 3);
    const bool used = row_off[q] < row_off[q + 1];
    pw_out[i] = used ? pw[q * Kw + at] : 0.0f;
    rho_out[i] = used ? rho[q * Kw + at] : 0.0f;
}

// Topics per lane of the kernel's instances: every number up to 8, where a topic
// more is the largest share of a token's work, then 10, 12, 13, 14 and 16: a lane of
// 9, 11 or 15 takes the next, at most a ninth more than it needs (weights of 0).
// Each number is up to six kernels of some 100 KB.
int instance_kpl(int32_t topics)
{
    if (topics <= 8) return topics;
    if (topics <= 10) return 10;
    if (topics <= 12) return 12;
    if (topics <= 14) return topics;
    return 16;
}

}  // namespace

// The pass that computes the weight rows costs a few bytes per cell of the rows
// that have tokens; the token loop saves about 0.1 ns per token over count rows
// (0.25 -> 0.16 ns at 200 topics, 0.42 -> 0.34 at 500), so the weight rows pay
// where a row has enough tokens for its length.  Measured: 50 M tokens at 18
// cells per token (500 topics, 27 tokens per row) 21.2 ms over count rows, 16.9
// + 2.9 ms over weight rows; a weight costs about 3.5 ps per cell, so the line
// lies near 28 cells per token, and is drawn at 24.
// Lanes per document: 16 for many documents, 32 while those would leave each
// SIMD fewer than 8 wavefronts to cover a token's chain with (3 M tokens in
// 20 000 documents, 100 topics: 294 us with 16 lanes, 280 with 32, 350 with
// 64; 40 M tokens in 200 000, 200 topics: 6.26, 6.58 and 6.80 ms), 64 where
// there are fewer documents than two per SIMD and a lane would hold more than
// four topics.  Row offsets are 32-bit byte offsets.
RowShape row_shape(int64_t N, int32_t D, int64_t rows, int64_t rows_used, int32_t K)
{
    RowShape r;
    if (24 * N < rows_used * K) return r;
    int lanes = D > 32768 || K <= 16 ? 16 : 32;
    while (lanes < 64 && K > 16 * lanes) lanes *= 2;
    if (lanes == 32 && D < 2048 && K > 4 * 32) lanes = 64;
    r.lanes = lanes;
    r.kpl = instance_kpl((K + lanes - 1) / lanes);
    r.Kw = (lanes * r.kpl + 31) / 32 * 32;
    if (rows * r.Kw >= (1ll << 30)) r = RowShape{};
    return r;
}

hipError_t launch_doc_order(const Model &m, const int64_t *doc_off, int32_t *order,
                            hipStream_t st)
{
    const int32_t per = (m.D + 7) / 8, windows = (per + kWindow - 1) / kWindow;
    hipLaunchKernelGGL(k_doc_order, dim3(8u * (unsigned)windows), dim3(kWindow / 2), 0, st, m.D,
                       per, windows, doc_off, order);
    return hipGetLastError();
}

hipError_t launch_weights(const Model &m, const DeviceBuffers &b, hipStream_t st)
{
    WeightArgs A;
    A.row_off = b.row_off;
    A.row_narrow = b.row_narrow;
    A.nt = b.nt;
    A.nt16 = b.nt16;
    A.B = b.B;
    A.f0 = b.f0;
    A.f1 = b.f1;
    A.Q = b.Q;
    A.srcrec = b.srcrec;
    A.pw = b.pw;
    A.rho = b.rho;
    A.rows = (int64_t)m.G * m.V;
    A.q_last = (uint64_t)(tri_index(m.ncap, 0) - 1);
    A.divV = m.divV;
    A.V = m.V;
    A.K = m.K;
    A.Kp = m.Kp;
    A.Kw = m.rows.Kw;
    A.Sp = m.Sp;
    A.lanes = m.rows.lanes;
    A.lane_shift = m.rows.lanes == 16 ? 4 : (m.rows.lanes == 32 ? 5 : 6);
    A.kpl = m.rows.kpl;
    if (m.rows.kpl < 4) {
        // rows of fewer than four topics per lane are stored in topic order, so
        // they are written as whole chunks too (468 000 rows of 32 topics, one
        // per lane: 113 us when each thread wrote one, 34 us this way)
        A.lanes = m.rows.lanes * m.rows.kpl / 4;
        A.lane_shift = 30;
        A.kpl = 4;
    }
    A.gamma = (float)m.gamma;
    const unsigned units = (unsigned)(A.lanes * ((A.kpl + 3) / 4));  // at most 256
    const unsigned per = kBlock / units;
    const dim3 grid((unsigned)((A.rows + per - 1) / per)), block(units, per);
    if (m.Sp > 0) hipLaunchKernelGGL(k_weights<true>, grid, block, 0, st, A);
    else hipLaunchKernelGGL(k_weights<false>, grid, block, 0, st, A);
    return hipGetLastError();
}

hipError_t launch_weight_topics(const Model &m, const DeviceBuffers &b, int64_t row_begin,
                                int64_t n, float *pw, float *rho, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    const int64_t nb = (n * m.K + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(k_weight_topics, dim3((unsigned)nb), dim3(kBlock), 0, st, n, m.K, m.rows.Kw,
                       m.rows.lanes, m.rows.kpl, b.row_off + row_begin,
                       b.pw + row_begin * m.rows.Kw, b.rho + row_begin * m.rows.Kw, pw, rho);
    return hipGetLastError();
}

RowArgs row_args(const Model &m, const DeviceBuffers &b, const int32_t *zr_old, int32_t *zr_new,
                 uint32_t sweep, uint64_t seed)
{
    RowArgs A;
    A.gw = b.gw;
    A.doc_off = b.doc_off;
    A.doc_group = b.doc_group;
    A.order = b.order_len;
    A.zr_old = zr_old;
    A.zr_new = zr_new;
    A.nt = b.nt;
    A.nt16 = b.nt16;
    A.tok_narrow = b.tok_narrow;
    A.row_narrow = b.row_narrow;
    A.B = b.B;
    A.fz = b.fz;
    A.Q = b.Q;
    A.pw = b.pw;
    A.rho = b.rho;
    A.srcrec = b.srcrec;
    A.exact = b.exact;
    A.seed = seed;
    A.nQ = tri_index(m.ncap, 0);
    A.D = m.D;
    A.V = m.V;
    A.K = m.K;
    A.Kp = m.Kp;
    A.Kw = m.rows.Kw;
    A.Sp = m.Sp;
    A.docs_per_xcd = (m.D + 7) / 8;
    A.sweep = sweep;
    A.alpha = (float)m.alpha;
    A.gamma = (float)m.gamma;
    return A;
}

hipError_t launch_sample_rows_assoc(const RowArgs &A, int lanes, int kpl, hipStream_t st);

hipError_t launch_sample_rows(const Model &m, const DeviceBuffers &b, const int32_t *zr_old,
                              int32_t *zr_new, uint32_t sweep, uint64_t seed, hipStream_t st)
{
    if (m.D <= 0 || m.N <= 0) return hipSuccess;
    const RowArgs A = row_args(m, b, zr_old, zr_new, sweep, seed);
    if (m.Sp > 0) return launch_sample_rows_assoc(A, m.rows.lanes, m.rows.kpl, st);
    switch (m.rows.lanes) {
    case 16: return launch_rows_lanes<16, false>(A, m.rows.kpl, st);
    case 32: return launch_rows_lanes<32, false>(A, m.rows.kpl, st);
    default: return launch_rows_lanes<64, false>(A, m.rows.kpl, st);
    }
}

}  // namespace spdp
