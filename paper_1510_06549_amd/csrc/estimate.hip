// estimate.hip -- point estimates of a state and held-out perplexity (gfx950).
//
// The estimates after convergence (thesis: Eq. spdp-topic-doc-estimate,
// Eq. spdp-word-topic-estimate and Eq. spdp-group-word-topic-estimate, with
// identity transformation matrices, so q = t):
//   theta[d][k]  = (c_dk + alpha) / (L_d + K alpha)
//   phi0[w][k]   = (gamma + B_wk) / (V gamma + B_k)
//   phi[g][w][k] = (n - a t + (b + a T_gk) phi0[w][k]) / (b + N_gk)
// The group estimate weights the base by (b + a T) / (b + N), the weight of a
// new table in the Pitman-Yor seating rule; the printed a T / (b + N) would
// not sum to one over the words.
//
// Held-out perplexity (section "Perplexity"): each test document is folded in
// with phi fixed at the group estimate of the current state.  Its topics start
// uniform (first Philox word with purpose 3 at counter (test token, 0), times
// K, high 32 bits); each fold-in sweep resamples its tokens in order from
//   p(z_n = k | rest) proportional to (c_k without token n + alpha) phi[g][w_n][k]
// with the uniform of purpose 2 at counter (test token, sweep) and the first k
// whose inclusive prefix sum exceeds u * total; then
//   log p(w_d) = sum_n log sum_k phi[g][w_n][k] theta_d[k]
// with theta_d from the final counts.  All in fp64.  One wavefront per test
// document; the estimates are computed from the count rows on the fly.
//
// With word associations (non-identity P^g) phi0 is over source words and the
// base of group g's Pitman-Yor process is P^g phi0_k:
//   phi[g][w][k] = (n - a t + (b + a T_gk) sum_v p_{g,w,v} phi0[v][k]) / (b + N_gk).
#include "sampler_common.hpp"

namespace spdp {

// fp64 wave scans of the fold-in (the sampler's DPP scan, applied to both
// 32-bit halves of each value).
// Both 32-bit halves move with the same DPP control (a disabled source gives
// 0 in both halves, i.e. +0.0).
template <int CTRL, int ROW_MASK, bool BOUND>
__device__ __forceinline__ double dpp_src64(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROW_MASK, 0xF, BOUND);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROW_MASK, 0xF, BOUND);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_inclusive_sum64(double x)
{
    x += dpp_src64<0x111, 0xF, true>(x);
    x += dpp_src64<0x112, 0xF, true>(x);
    x += dpp_src64<0x114, 0xF, true>(x);
    x += dpp_src64<0x118, 0xF, true>(x);
    x += dpp_src64<0x142, 0xA, false>(x);
    x += dpp_src64<0x143, 0xC, false>(x);
    return x;
}

__device__ __forceinline__ double wave_shift_right64(double x)
{
    return dpp_src64<0x138, 0xF, true>(x);
}

__device__ __forceinline__ double readlane64(double x, int32_t l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}


namespace {

constexpr uint32_t kPurposeFoldin = 2u, kPurposeFoldinInit = 3u;

inline int64_t blocks_for(int64_t n, int per_block)
{
    int64_t b = (n + per_block - 1) / per_block;
    return b < 1 ? 1 : b;
}

// theta of training documents: a wave takes kThetaDocs documents together, so
// that their offsets and topics are in flight at once (one document a wave
// leaves a chain of three memory trips per 1.6 KB written: 80 000 documents,
// 200 topics took 53 us).
constexpr int kThetaDocs = 4;
__global__ void __launch_bounds__(64) k_theta(int32_t D, int32_t K, double alpha,
                                              const int64_t *__restrict__ doc_off,
                                              const int32_t *__restrict__ zr,
                                              double *__restrict__ theta)
{
    extern __shared__ int32_t c_all[];  // [kThetaDocs][K]
    const int32_t lane = threadIdx.x, d0 = blockIdx.x * kThetaDocs;
    int64_t beg[kThetaDocs];
    int32_t len[kThetaDocs], longest = 0;
#pragma unroll
    for (int i = 0; i < kThetaDocs; ++i) {
        const int32_t d = d0 + i < D ? d0 + i : D - 1;
        beg[i] = doc_off[d];
        len[i] = d0 + i < D ? (int32_t)(doc_off[d + 1] - beg[i]) : 0;
        longest = len[i] > longest ? len[i] : longest;
    }
    for (int32_t k = lane; k < kThetaDocs * K; k += 64) c_all[k] = 0;
    __syncthreads();
    for (int32_t x = lane; x < longest; x += 64) {
        int32_t v[kThetaDocs];
#pragma unroll
        for (int i = 0; i < kThetaDocs; ++i) v[i] = x < len[i] ? zr[beg[i] + x] : 0;
#pragma unroll
        for (int i = 0; i < kThetaDocs; ++i)
            if (x < len[i]) atomicAdd(&c_all[i * K + zr_topic(v[i])], 1);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kThetaDocs; ++i) {
        if (d0 + i >= D) break;
        const double inv = 1.0 / ((double)len[i] + (double)K * alpha);
        double *row = theta + (int64_t)(d0 + i) * K;
        for (int32_t k = lane; k < K; k += 64) row[k] = ((double)c_all[i * K + k] + alpha) * inv;
    }
}

// x / d with r = 1 / d (correctly rounded): the quotient by r, then one
// correction with the exact remainder, which rounds as the division does
// (Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", 1990).  RECIP is false where a divisor may have no reciprocal to
// correct: see launch_phi.
template <bool RECIP>
__device__ __forceinline__ double div_by(double x, double d, double r)
{
    if constexpr (!RECIP) return x / d;
    const double q = x * r;
    return __fma_rn(__fma_rn(-q, d, x), r, q);
}

struct PhiArgs {
    const int32_t *nt, *B, *Ngk, *Tgk, *Bk, *srcrec;
    const uint16_t *nt16;
    const uint8_t *row_narrow;
    const double *p64;
    double *phi0, *phi;  // either may be null
    int32_t g_begin, V, K, Kp, Sp;
    double a, b, gamma, Vgamma;
};

// phi0 as [V][K] and phi of groups [g_begin, g_end) as [g][V][K].  A thread
// takes one topic of kPhiWords words, so that every divisor and its reciprocal
// are computed once for them and their loads are in flight together: per value
// one cell read (a narrow row's 16-bit copy), a few fp64 operations and the
// write.  blockDim.x topics, blockDim.y runs of words
// a block; the groups are outside (grid z), so that writes run along words.
// 10 groups, 50 000 words, 200 topics: 309 us for phi0 and phi (2.8 TB/s written,
// where a fill reaches 6.3); 33 us and 389 us when every value took three
// divisions and a 64-bit division of its index.
constexpr int kPhiWords = 8, kPhiBlock = 1024;
template <bool ASSOC, bool RECIP>
__global__ void __launch_bounds__(kPhiBlock) k_phi(PhiArgs A)
{
    const int32_t k = blockIdx.y * blockDim.x + threadIdx.x;
    if (k >= A.K) return;
    const int32_t g = A.g_begin + (int32_t)blockIdx.z;
    const double d0 = A.Vgamma + (double)A.Bk[k], r0 = 1.0 / d0;
    double dg = 1.0, wg = 0.0;
    if (A.phi) {
        dg = A.b + (double)A.Ngk[(int64_t)g * A.Kp + k];
        wg = A.b + A.a * (double)A.Tgk[(int64_t)g * A.Kp + k];
    }
    const double rg = 1.0 / dg;
    const bool first = A.phi0 != nullptr && blockIdx.z == 0;
    double *out = A.phi ? A.phi + (int64_t)blockIdx.z * A.V * A.K : nullptr;
    // kPhiWords consecutive words per thread, their loads together (words past
    // the last one repeat it)
    const int32_t w0 = (blockIdx.x * blockDim.y + threadIdx.y) * kPhiWords;
    if (w0 >= A.V) return;
    const int32_t nw = A.V - w0 < kPhiWords ? A.V - w0 : kPhiWords;
    const uint8_t *flag = A.row_narrow + (int64_t)g * A.V + w0;
    const int32_t *base = A.B + (int64_t)w0 * A.Kp + k;
    const int64_t cell0 = ((int64_t)g * A.V + w0) * A.Kp;
    const char *wide = reinterpret_cast<const char *>(A.nt + cell0 + k);
    const char *half = reinterpret_cast<const char *>(A.nt16 + cell0 + (k & ~1));
    int32_t bw[kPhiWords], x[kPhiWords];
    bool nar[kPhiWords];
#pragma unroll
    for (int i = 0; i < kPhiWords; ++i) {
        const int32_t o = i < nw ? i : nw - 1;
        nar[i] = A.phi ? flag[o] != 0 : false;
        bw[i] = (!ASSOC || first) ? base[o * A.Kp] : 0;
    }
    // (one load whichever copy is current: the 32-bit word that holds the cell)
#pragma unroll
    for (int i = 0; i < kPhiWords; ++i) {
        const int32_t o = (i < nw ? i : nw - 1) * A.Kp;
        x[i] = A.phi ? *reinterpret_cast<const int32_t *>(nar[i] ? half + 2 * o : wide + 4 * o) : 0;
    }
    double *p_out = first ? A.phi0 + (int64_t)w0 * A.K + k : nullptr;
    if (out) out += (int64_t)w0 * A.K + k;
#pragma unroll
    for (int i = 0; i < kPhiWords; ++i) {
        if (i >= nw) break;
        double p0 = div_by<RECIP>(A.gamma + (double)bw[i], d0, r0);
        if (first) p_out[i * A.K] = p0;
        if (!A.phi) continue;
        const int32_t c =
            nar[i] ? wide_of(k & 1 ? (uint32_t)x[i] >> 16 : (uint32_t)x[i] & 0xFFFFu) : x[i];
        const double n = (double)(c & kCountMax), t = (double)(c >> kCountBits);
        if constexpr (ASSOC) {
            // the base term sums phi0 over the row's sources (padding slots
            // have p = 0)
            const int64_t q = (int64_t)g * A.V + w0 + i;
            p0 = 0.0;
            for (int32_t s = 0; s < A.Sp; ++s) {
                const double pv = A.p64[q * A.Sp + s];
                const int64_t v = A.srcrec[q * 2 * A.Sp + s];
                if (pv > 0.0)
                    p0 += pv * div_by<RECIP>(A.gamma + (double)A.B[v * A.Kp + k], d0, r0);
            }
        }
        out[i * A.K] = div_by<RECIP>(n - A.a * t + wg * p0, dg, rg);
    }
}

struct FoldArgs {
    const int32_t *gw;        // [Nt] row index g V + w of each test token
    const int64_t *doc_off;   // [Dt + 1]
    const int32_t *doc_group; // [Dt]
    int32_t *z;               // [Nt] fold-in topics
    double *ll_doc;           // [Dt] log p(w_d)
    const int32_t *nt, *B, *Ngk, *Tgk, *Bk;
    const int32_t *srcrec;    // word associations (Sp > 0): source records
    const double *p64;        //   and fp64 p of each row
    uint64_t seed;
    int32_t D, V, K, Kp, n_sweeps, Sp;
    double alpha, a, b, gamma, Vgamma;
};

// sum over the wave's 64 lanes (the last lane's inclusive prefix sum)
__device__ __forceinline__ double wave_sum(double x)
{
    return readlane64(wave_inclusive_sum64(x), 63);
}

// This lane's slices of the rows a test token's group estimate reads, loaded
// whole (padding chunks re-read the row start; their topics weigh nothing):
// the packed count row of q = g V + w and, with P = I (SP = 0), the int32
// shadow-base row of w; with word associations (SP sources per row) the
// shadow-base rows of the row's sources and their p (a padding slot repeats
// the first source with p = 0).
template <int KPL, int SP>
struct FoldRows {
    static constexpr int NB = SP > 0 ? SP : 1;
    int32_t n[KPL];
    int32_t b[NB][KPL];
    double p[NB];
};

template <int KPL, int SP>
__device__ __forceinline__ void load_fold_rows(const FoldArgs &A, int32_t q, int32_t g,
                                               int32_t kbase, FoldRows<KPL, SP> &R)
{
    load_row<KPL>(R.n, A.nt + (int64_t)q * A.Kp, kbase, A.Kp);
    if constexpr (SP == 0) {
        load_row<KPL>(R.b[0], A.B + (int64_t)(q - g * A.V) * A.Kp, kbase, A.Kp);
    } else {
#pragma unroll
        for (int s = 0; s < SP; ++s) {
            const int32_t v = A.srcrec[(int64_t)q * 2 * SP + s];
            R.p[s] = A.p64[(int64_t)q * SP + s];
            load_row<KPL>(R.b[s], A.B + (int64_t)v * A.Kp, kbase, A.Kp);
        }
    }
}

// The group estimate of this lane's topics: (n - a t)/(b + N) plus the base
// weight times (b + a T)/(b + N)/(V gamma + B_k), the base weight being
// gamma + B[w][k], or with word associations the sum over the sources, in
// slot order, of p (gamma + B[v][k]) for p > 0.
template <int KPL, int SP>
__device__ __forceinline__ void phi_from_rows(const FoldArgs &A, const FoldRows<KPL, SP> &R,
                                              const double *inv, const double *base,
                                              double (&ph)[KPL])
{
#pragma unroll
    for (int j = 0; j < KPL; ++j) {
        const double n = (double)(R.n[j] & kCountMax), t = (double)(R.n[j] >> kCountBits);
        double bw;
        if constexpr (SP == 0) {
            bw = A.gamma + (double)R.b[0][j];
        } else {
            bw = 0.0;
#pragma unroll
            for (int s = 0; s < SP; ++s)
                if (R.p[s] > 0.0) bw += R.p[s] * (A.gamma + (double)R.b[s][j]);
        }
        ph[j] = (n - A.a * t) * inv[j] + bw * base[j];  // padding topics: 0
    }
}

// The group estimates of tokens 0 .. nc - 1 of a chunk (row indices in the
// lanes of gw_c), in order, handed to f(x, ph).  Where two register sets of
// rows fit, the rows of token x + 1 are requested before token x is
// evaluated; otherwise each token's rows are loaded together, then used.
template <int KPL, int SP, typename F>
__device__ __forceinline__ void for_chunk_phi(const FoldArgs &A, int32_t g, int32_t kbase,
                                              int32_t gw_c, int32_t nc, const double *inv,
                                              const double *base, F &&f)
{
    constexpr int kRows = SP > 0 ? SP + 1 : 2;
    if constexpr (KPL * kRows > 48) {
        for (int32_t x = 0; x < nc; ++x) {
            FoldRows<KPL, SP> r;
            load_fold_rows<KPL, SP>(A, __builtin_amdgcn_readlane(gw_c, x), g, kbase, r);
            double ph[KPL];
            phi_from_rows<KPL, SP>(A, r, inv, base, ph);
            f(x, ph);
        }
    } else {
        FoldRows<KPL, SP> ra, rb;
        load_fold_rows<KPL, SP>(A, __builtin_amdgcn_readlane(gw_c, 0), g, kbase, ra);
        for (int32_t x = 0; x < nc; x += 2) {
            const int32_t x1 = x + 1 < nc ? x + 1 : x;
            load_fold_rows<KPL, SP>(A, __builtin_amdgcn_readlane(gw_c, x1), g, kbase, rb);
            {
                double ph[KPL];
                phi_from_rows<KPL, SP>(A, ra, inv, base, ph);
                f(x, ph);
            }
            if (x + 1 < nc) {
                const int32_t x2 = x + 2 < nc ? x + 2 : x + 1;
                load_fold_rows<KPL, SP>(A, __builtin_amdgcn_readlane(gw_c, x2), g, kbase, ra);
                double ph[KPL];
                phi_from_rows<KPL, SP>(A, rb, inv, base, ph);
                f(x + 1, ph);
            }
        }
    }
}

// Bound by instructions issued per token (fp64, with a wave scan on the chain
// from one token to the next).  So each lane takes one of 64 tokens' uniforms,
// as a uniform token's Philox runs on the scalar unit that four SIMDs share;
// counts and factors stay in registers, not behind an LDS round trip in the
// chain; and nothing selects on k < K, as padding topics' factors are zero.
// 8 000 documents of 200 tokens, K = 200, 10 sweeps (17.6 million draws and
// sums): 5.9 -> 4.6 ms.
template <int KPL, int SP>
__global__ void __launch_bounds__(64) k_foldin(FoldArgs A)
{
    // this lane's document counts cr, and the group's per-topic factors
    // 1/(b + N) and (b + a T)/(b + N)/(V gamma + B_k) (zero for padding topics,
    // whose group estimates and weights are then zero)
    __shared__ int32_t c[64 * KPL];
    int32_t cr[KPL];
    double inv[KPL], base[KPL];
    const int32_t d = blockIdx.x;
    if (d >= A.D) return;
    const int32_t lane = threadIdx.x, kbase = lane * KPL;
    const int64_t beg = A.doc_off[d], end = A.doc_off[d + 1];
    const int32_t g = A.doc_group[d];
#pragma unroll
    for (int j = 0; j < KPL; ++j) {
        const int32_t k = kbase + j;
        c[k] = 0;
        inv[j] = base[j] = 0.0;
        if (k < A.K) {
            const double N = (double)A.Ngk[(int64_t)g * A.Kp + k];
            const double T = (double)A.Tgk[(int64_t)g * A.Kp + k];
            inv[j] = 1.0 / (A.b + N);
            base[j] = (A.b + A.a * T) / (A.b + N) / (A.Vgamma + (double)A.Bk[k]);
        }
    }
    __syncthreads();
    // initial topics
    for (int64_t i = beg + lane; i < end; i += 64) {
        const uint32_t x = philox_x0(A.seed, (uint64_t)i, 0u, kPurposeFoldinInit);
        const int32_t z = (int32_t)(((uint64_t)x * (uint64_t)A.K) >> 32);
        A.z[i] = z;
        atomicAdd(&c[z], 1);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KPL; ++j) cr[j] = c[kbase + j];

    for (int32_t s = 0; s < A.n_sweeps; ++s) {
        // 64 tokens at a time: lane l reads and writes token cb + l, so each
        // lane sees its own earlier writes
        for (int64_t cb = beg; cb < end; cb += 64) {
            const int32_t nc = (int32_t)min((int64_t)64, end - cb);
            const bool mine = lane < nc;
            const int32_t gw_c = mine ? A.gw[cb + lane] : 0;
            int32_t z_c = mine ? A.z[cb + lane] : 0;
            // the chunk's uniforms, a token each lane
            const uint32_t x_c = philox_x0(A.seed, (uint64_t)(cb + lane), (uint32_t)s,
                                           kPurposeFoldin);
            for_chunk_phi<KPL, SP>(A, g, kbase, gw_c, nc, inv, base, [&](int32_t x,
                                                                            const double(&ph)[KPL]) {
                const int32_t k0 = __builtin_amdgcn_readlane(z_c, x);
                double pre[KPL];
                double acc = 0.0;
#pragma unroll
                for (int j = 0; j < KPL; ++j) {
                    cr[j] -= kbase + j == k0 ? 1 : 0;
                    acc += ((double)cr[j] + A.alpha) * ph[j];
                    pre[j] = acc;
                }
                const double incl = wave_inclusive_sum64(acc);
                const double excl = wave_shift_right64(incl);
                const double total = readlane64(incl, 63);
                const uint32_t xr = (uint32_t)__builtin_amdgcn_readlane((int32_t)x_c, x);
                const double target = (double)(xr >> 8) * (1.0 / 16777216.0) * total;
                const double rel = target - excl;
                int32_t cnt = 0;
#pragma unroll
                for (int j = 0; j < KPL; ++j) cnt += (pre[j] <= rel) ? 1 : 0;
                const unsigned long long cross = __ballot(cnt < KPL && kbase < A.K);
                int32_t k1 = k0;
                if (cross) {
                    const int32_t L = __ffsll((long long)cross) - 1;
                    k1 = L * KPL + __builtin_amdgcn_readlane(cnt, L);
                }
                if (k1 >= A.K) k1 = k0;  // no crossing (rounding at the very top): keep
                if (lane == x) z_c = k1;
#pragma unroll
                for (int j = 0; j < KPL; ++j) cr[j] += kbase + j == k1 ? 1 : 0;
            });
            if (mine) A.z[cb + lane] = z_c;
        }
    }

    // log p(w_d) with theta_d from the final counts
    const double tden = 1.0 / ((double)(end - beg) + (double)A.K * A.alpha);
    double th[KPL];
#pragma unroll
    for (int j = 0; j < KPL; ++j)
        th[j] = (kbase + j < A.K) ? ((double)cr[j] + A.alpha) * tden : 0.0;
    double ll = 0.0;
    for (int64_t cb = beg; cb < end; cb += 64) {
        const int32_t nc = (int32_t)min((int64_t)64, end - cb);
        const int32_t gw_c = (lane < nc) ? A.gw[cb + lane] : 0;
        for_chunk_phi<KPL, SP>(A, g, kbase, gw_c, nc, inv, base,
                                  [&](int32_t, const double(&ph)[KPL]) {
                                      double p = 0.0;
#pragma unroll
                                      for (int j = 0; j < KPL; ++j) p += ph[j] * th[j];
                                      ll += log(wave_sum(p));
                                  });
    }
    if (lane == 0) A.ll_doc[d] = ll;
}

template <int KPL>
hipError_t launch_fold(const FoldArgs &A, hipStream_t st)
{
    const dim3 grid((unsigned)A.D);
    switch (A.Sp) {
    case 0: hipLaunchKernelGGL((k_foldin<KPL, 0>), grid, dim3(64), 0, st, A); break;
    case 1: hipLaunchKernelGGL((k_foldin<KPL, 1>), grid, dim3(64), 0, st, A); break;
    case 2: hipLaunchKernelGGL((k_foldin<KPL, 2>), grid, dim3(64), 0, st, A); break;
    case 4: hipLaunchKernelGGL((k_foldin<KPL, 4>), grid, dim3(64), 0, st, A); break;
    case 8: hipLaunchKernelGGL((k_foldin<KPL, 8>), grid, dim3(64), 0, st, A); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_theta(const Model &m, const DeviceBuffers &b, const int32_t *zr, double *theta,
                        hipStream_t st)
{
    if (m.D <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_theta, dim3((unsigned)blocks_for(m.D, kThetaDocs)), dim3(64),
                       (size_t)(kThetaDocs * m.K) * sizeof(int32_t), st, m.D, m.K, m.alpha,
                       b.doc_off, zr, theta);
    return hipGetLastError();
}

hipError_t launch_phi(const Model &m, const DeviceBuffers &b, int32_t g_begin, int32_t g_end,
                      double *phi0, double *phi, hipStream_t st)
{
    if (!phi0 && (!phi || g_begin >= g_end)) return hipSuccess;
    PhiArgs A;
    A.nt = b.nt;
    A.nt16 = b.nt16;
    A.row_narrow = b.row_narrow;
    A.B = b.B;
    A.Ngk = b.Ngk;
    A.Tgk = b.Tgk;
    A.Bk = b.Bk;
    A.srcrec = b.srcrec;
    A.p64 = b.p64;
    A.phi0 = phi0;
    A.phi = phi && g_begin < g_end ? phi : nullptr;
    A.g_begin = A.phi ? g_begin : 0;
    A.V = m.V;
    A.K = m.K;
    A.Kp = m.Kp;
    A.Sp = m.Sp;
    A.a = m.a;
    A.b = m.b;
    A.gamma = m.gamma;
    A.Vgamma = (double)m.V * m.gamma;
    // topics in ranges of at most 512, and as many runs of words a block as
    // leave its last wavefront fullest
    const unsigned ranges = (unsigned)((m.K + 511) / 512);
    const unsigned x = (unsigned)((m.K + (int32_t)ranges - 1) / (int32_t)ranges);
    unsigned y = 1;
    for (unsigned c = 2; c <= 16 && c * x <= (unsigned)kPhiBlock; ++c)
        if (c * x * ((y * x + 63) / 64) >= y * x * ((c * x + 63) / 64)) y = c;
    const int64_t nb = (m.V + kPhiWords * (int64_t)y - 1) / (kPhiWords * (int64_t)y);
    const dim3 block(x, y);
    // every divisor is b or V gamma and a count below 2^31; a reciprocal that
    // overflows (a subnormal b or V gamma, no customers) or is 0 (an infinite
    // V gamma) has no correction, and the line leaves the remainder room
    auto in_range = [](double d) { return d >= 0x1p-900 && d <= 0x1p900; };
    const bool recip = in_range(A.b) && in_range(A.Vgamma);
    do {  // (a grid holds at most 65 535 groups)
        const int32_t groups = A.phi ? (g_end - A.g_begin < 32768 ? g_end - A.g_begin : 32768) : 1;
        const dim3 grid((unsigned)nb, ranges, (unsigned)groups);
        if (!recip)
            hipLaunchKernelGGL((m.Sp > 0 ? k_phi<true, false> : k_phi<false, false>), grid, block,
                               0, st, A);
        else
            hipLaunchKernelGGL((m.Sp > 0 ? k_phi<true, true> : k_phi<false, true>), grid, block, 0,
                               st, A);
        if (!A.phi) break;
        A.phi0 = nullptr;
        A.phi += (int64_t)groups * m.V * m.K;
        A.g_begin += groups;
    } while (A.g_begin < g_end);
    return hipGetLastError();
}

hipError_t launch_foldin(const Model &m, const DeviceBuffers &b, int32_t D_test,
                         const int32_t *gw, const int64_t *doc_off, const int32_t *doc_group,
                         int32_t n_sweeps, uint64_t seed, int32_t *z, double *ll_doc,
                         hipStream_t st)
{
    if (D_test <= 0) return hipSuccess;
    FoldArgs A;
    A.gw = gw;
    A.doc_off = doc_off;
    A.doc_group = doc_group;
    A.z = z;
    A.ll_doc = ll_doc;
    A.nt = b.nt;
    A.B = b.B;
    A.Ngk = b.Ngk;
    A.Tgk = b.Tgk;
    A.Bk = b.Bk;
    A.srcrec = b.srcrec;
    A.p64 = b.p64;
    A.Sp = m.Sp;
    A.seed = seed;
    A.D = D_test;
    A.V = m.V;
    A.K = m.K;
    A.Kp = m.Kp;
    A.n_sweeps = n_sweeps;
    A.alpha = m.alpha;
    A.a = m.a;
    A.b = m.b;
    A.gamma = m.gamma;
    A.Vgamma = (double)m.V * m.gamma;
    switch (sampler_kpl(m.K)) {
    case 1: return launch_fold<1>(A, st);
    case 2: return launch_fold<2>(A, st);
    case 4: return launch_fold<4>(A, st);
    case 8: return launch_fold<8>(A, st);
    case 12: return launch_fold<12>(A, st);
    default: return launch_fold<16>(A, st);
    }
}

}  // namespace spdp
