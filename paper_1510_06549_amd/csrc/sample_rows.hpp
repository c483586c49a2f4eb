// sample_rows.hpp -- the per-sweep resampling kernel over weight rows (gfx950,
// wave64), for the plain model and for word associations.
//
// Everything in a token's conditionals but the document's own counts is fixed
// for the sweep, so it is computed once per count row instead of once per
// token: for each row q = (g, w) that has tokens and each topic k,
//   pw[q][k]  = f1[g][k] beta[q][k] Q1(n, t) + f0[g][k] Q0(n, t)
//   rho[q][k] = the share of the first term (r = 1) in it
// with beta = gamma + B[w][k], or with word associations the sum over the
// row's sources of p_s (gamma + B[v_s][k]).  A token's topic weights are then
//   W(k) = (alpha + c'_k) pw[q][k],
// one load, one addition and one product per topic, and no gather.  Two things
// remain per token: its own topic, whose weights are those of the cell without
// the token, and the choice among the outcomes of the drawn topic.
//
// Layout.  LANES lanes (16, 32 or 64) share a document, so that a wavefront
// samples 64 / LANES documents in lockstep; lane l of a document owns the KPL
// contiguous topics from l KPL on, and their counts live in its registers.  A
// weight row is stored so that the document's lanes read it with whole
// 16-byte loads (row_pos).  Fewer lanes spread the fixed work of a token (the
// scan, the crossing, the bookkeeping) over more documents; more lanes
// shorten a token's chain where documents are few.
//
// Tokens are taken 16 at a time (a chunk; lane l of each row of 16 lanes stands
// for the document's token l of it, and DPP broadcasts bring a token's values
// to the row).  Ahead of a chunk each lane prepares its token: the uniform,
// and the own topic's weights from the cell's counts without the token.  After
// the chunk each lane decides its token's outcome within the drawn topic (its
// table indicator, and with word associations the source slot) from rho of
// the drawn cell.  So the serial chain of a token is the count update, KPL
// products and additions, the scan over LANES lanes and the crossing; both
// ends of a token run vectorised over the chunk, and the rows are requested
// tokens ahead.  A chunk's steps are unrolled into straight-line code, with the
// preparation's loads between them, so that every wait is for exactly the
// loads it needs.
//
// Exactness.  The draw is the first outcome, in the order (k, r = 1, slots),
// (k, r = 0), whose prefix exceeds u * total, with fp32 prefixes.  Where the
// target lies within rounding distance of a topic boundary (at the token) or
// of a boundary inside the topic (after the chunk, with the document's counts
// at the token restored from the chunk's moves), the whole decision is taken
// again with fp64 weights from the integer counts, as in the kernels over
// count rows.
#pragma once

#include "sampler_common.hpp"

namespace spdp {

struct RowArgs {
    const int32_t *gw;
    const int64_t *doc_off;
    const int32_t *doc_group;
    const int32_t *order;  // [D] documents in launch order
    const int32_t *zr_old;
    int32_t *zr_new;
    const int32_t *nt;
    const uint16_t *nt16;
    const uint8_t *tok_narrow;
    const uint8_t *row_narrow;
    const int32_t *B;
    const float4 *fz;  // [G][Kp][2] the topic's constants, see k_factors
    const float2 *Q;
    const float *pw, *rho;
    const int32_t *srcrec;
    const ExactCtx *exact;
    uint64_t seed;
    int64_t nQ;
    int32_t D, V, K, Kp, Kw, Sp;
    int32_t docs_per_xcd;
    uint32_t sweep;
    float alpha, gamma;
};

namespace {

// Position of topic k in a stored weight row: 16-byte chunks of four topics,
// chunk c of lane l at (c LANES + l) 4, then the KPL mod 4 remaining topics of
// every lane.
template <int LANES, int KPL>
__host__ __device__ __forceinline__ int32_t row_pos(int32_t k)
{
    constexpr int NC = KPL / 4, REM = KPL % 4;
    const int32_t l = k / KPL, j = k % KPL, c = j >> 2;
    return c < NC ? (c * LANES + l) * 4 + (j & 3) : NC * LANES * 4 + l * REM + (j & 3);
}

// Inclusive prefix sum over the LANES lanes of each document, the value of the
// lane before (0 in a document's first lane), and the document's total.
template <int LANES>
__device__ __forceinline__ float doc_inclusive_sum(float x)
{
    x += dpp_src<0x111, 0xF, true>(x);
    x += dpp_src<0x112, 0xF, true>(x);
    x += dpp_src<0x114, 0xF, true>(x);
    x += dpp_src<0x118, 0xF, true>(x);
    if constexpr (LANES >= 32) x += dpp_src<0x142, 0xA, false>(x);
    if constexpr (LANES >= 64) x += dpp_src<0x143, 0xC, false>(x);
    return x;
}

template <int LANES>
__device__ __forceinline__ float doc_shift_right(float x, int32_t sub)
{
    if constexpr (LANES == 16) return dpp_src<0x111, 0xF, true>(x);
    const float y = dpp_src<0x138, 0xF, true>(x);
    if constexpr (LANES == 32) return sub == 0 ? 0.0f : y;
    return y;
}

template <int LANES>
__device__ __forceinline__ float doc_total(float incl, int32_t lane)
{
    if constexpr (LANES == 16) return dpp_src<0x15F, 0xF, true>(incl);  // row_newbcast:15
    if constexpr (LANES == 32) {
        const float a = readlane_f(incl, 31), b = readlane_f(incl, 63);
        return lane < 32 ? a : b;
    }
    return readlane_f(incl, 63);
}

// Distances from a boundary, as fractions of the total, below which a decision
// is taken again in fp64.  To first order in u = 2^-24 a topic weight carries
// at most 10 relative roundings (pw's first term six: its constant, gamma, the
// sum with B, the ratio pair, two products; the sum one more; alpha, the sum with c and the
// product three), with word associations SP + 3 more (each source's p and its
// product, the sum over the sources); the summation of a boundary and of the
// total behind the target each add at most (KPL + 5)u; the target, its lane
// offset, the compared boundary and the distance one each: (2 KPL + SP + 27)u
// in all.  A boundary inside the topic is the topic's lower boundary plus a
// share of its width: both boundaries' errors enter in proportion, the share
// adds at most 16 + 2 SP roundings.
template <int KPL>
__device__ __forceinline__ float topic_margin(int32_t Sp)
{
    return (float)(2 * KPL + Sp + 40) * 5.97e-8f;
}
template <int KPL>
__device__ __forceinline__ float inner_margin(int32_t Sp)
{
    return (float)(2 * KPL + 3 * Sp + 64) * 5.97e-8f;
}

// the uniform of token t
__device__ __forceinline__ float sample_uniform(const RowArgs &A, int32_t t)
{
    const uint32_t x = philox_x0(A.seed, (uint64_t)(uint32_t)t, A.sweep, kPurposeSample);
    return (float)(x >> 8) * (1.0f / 16777216.0f);
}

// The decision of one token in fp64, by the whole wavefront (lane l takes the
// topics from l per on, per = K / 64 rounded up): weights of every outcome from
// the integer counts (cnt: the document's counts without the token, topic by
// topic, in LDS), fp64 prefix sums in outcome order, and the first outcome with
// a positive weight whose prefix exceeds u * total (the last positive one if
// rounding leaves none).  All arguments are wave-uniform; zr0 is the token's
// packed state and the result the drawn one.  A function of its own, which
// reads its context anew for every topic, so that this rare path does not set
// the registers of the token loop.
typedef const __attribute__((address_space(3))) int32_t *LdsCounts;
template <bool ASSOC>
__device__ __noinline__ int32_t decide64(const ExactCtx *ctx, int32_t q, int32_t gV, int32_t gK,
                                         int32_t zr0, float u, LdsCounts cnt)
{
    const int32_t lane = (int32_t)threadIdx.x;
    const int32_t k0 = zr_topic(zr0), r0 = zr0 & 1, s0 = zr_slot(zr0);
    const int32_t Sp = ASSOC ? ctx->Sp : 1, K = ctx->K, per = (K + 63) >> 6;
    // weights of topic k, handed to f(slot or Sp for r = 0, weight) in order
    auto topic = [&](int32_t k, auto &&f) {
        const ExactCtx *fresh = ctx;
        asm volatile("" : "+v"(fresh));
        const ExactCtx &X = *fresh;
        const int32_t del = (k == k0) ? 1 : 0;
        const int64_t at = (int64_t)q * X.Kp + k;
        const int32_t cell = X.row_narrow[q] ? wide_of(X.nt16[at]) : X.nt[at];
        const int32_t nn = (cell & kCountMax) - del, tt = (cell >> kCountBits) - del * r0;
        const double N = (double)(X.Ngk[gK + k] - del), T = (double)(X.Tgk[gK + k] - del * r0);
        const double Bt = (double)(X.Bk[k] - del * r0);
        const double doc = X.alpha + (double)cnt[k];
        const double2 qq = X.Q64[exact_q_index(X, nn, tt)];
        if constexpr (ASSOC) {
            for (int32_t s = 0; s < Sp; ++s) {
                const int32_t v = X.srcrec[(int64_t)q * 2 * Sp + s];
                const int32_t bv = X.B[(int64_t)v * X.Kp + k] - ((del && r0 && s == s0) ? 1 : 0);
                f(s, X.p64[(int64_t)q * Sp + s] * doc * (X.b + X.a * T) / (X.b + N) *
                         (X.gamma + (double)bv) / (X.Vgamma + Bt) * qq.y);
            }
        } else {
            const double bw = (double)(X.B[(int64_t)(q - gV) * X.Kp + k] - del * r0);
            f(0, doc * (X.b + X.a * T) / (X.b + N) * (X.gamma + bw) / (X.Vgamma + Bt) * qq.y);
        }
        f(Sp, doc / (X.b + N) * qq.x);
    };
    double acc = 0.0;
    int32_t last = -1;
#pragma unroll 1
    for (int j = 0; j < per; ++j) {
        const int32_t k = lane * per + j;
        if (k >= K) break;
        topic(k, [&](int32_t s, double w) {
            acc += w;
            if (w > 0.0) last = j * (Sp + 1) + s;
        });
    }
    double incl = acc;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    double run = __shfl_up(incl, 1);
    if (lane == 0) run = 0.0;
    const double target = (double)u * __shfl(incl, 63);
    int32_t cand = -1;
    if (incl > target) {
#pragma unroll 1
        for (int j = 0; j < per && cand < 0; ++j) {
            const int32_t k = lane * per + j;
            if (k >= K) break;
            topic(k, [&](int32_t s, double w) {
                run += w;
                if (cand < 0 && w > 0.0 && run > target) cand = j * (Sp + 1) + s;
            });
        }
    }
    const unsigned long long m2 = __ballot(cand >= 0), m3 = __ballot(last >= 0);
    int32_t L = 0, o = -1;
    if (m2) {
        L = __ffsll((long long)m2) - 1;
        o = readlane(cand, L);
    } else if (m3) {
        L = 63 - __clzll((long long)m3);
        o = readlane(last, L);
    }
    if (o < 0) return zr0;
    const int32_t s = o % (Sp + 1);
    return zr_pack(L * per + o / (Sp + 1), s < Sp ? 1 : 0, s < Sp && ASSOC ? s : 0);
}

// The only head of a cell that keeps other customers, with word associations:
// it stays that cell's head and redraws its source in proportion to
// p_s (gamma + B'[v_s][k0]) (fp64, one lane).
__device__ inline int32_t sole_slot64(const RowArgs &A, int32_t q, int32_t k0, int32_t s0, float u)
{
    const ExactCtx &X = *A.exact;
    auto weight = [&](int32_t s) {
        const int32_t v = A.srcrec[(int64_t)q * 2 * A.Sp + s];
        const int32_t bv = A.B[(int64_t)v * A.Kp + k0] - (s == s0 ? 1 : 0);
        return X.p64[(int64_t)q * A.Sp + s] * (X.gamma + (double)bv);
    };
    double total = 0.0;
    int32_t last = s0;
    for (int32_t s = 0; s < A.Sp; ++s) {
        const double w = weight(s);
        total += w;
        if (w > 0.0) last = s;
    }
    const double target = (double)u * total;
    double run = 0.0;
    for (int32_t s = 0; s < A.Sp; ++s) {
        const double w = weight(s);
        run += w;
        if (w > 0.0 && run > target) return s;
    }
    return last;
}

// Row buffers: a token's weight row is requested this many tokens ahead, less
// one (a divisor of the chunk).  Two buffers and three left the 40-million-token
// sampler at the memory's latency (10 MB in flight over the chip).
constexpr int kRowBuffers = 4;

// Wavefronts per SIMD that the registers are budgeted for: the plain instances
// use no scratch.  With word associations those of up to four topics a lane
// reload a few values per chunk of tokens (none per token) at five, which is
// still faster than four without: 3 sources, 1.5 million tokens in 20 000
// documents, K = 128: 542 us a sweep at five, 553 at four.  From five topics a lane on
// a reload per token, which waits for the rows requested ahead as well, costs
// more than the wavefront: K = 192 there, 764 us at five, 710 at four; plain,
// K = 224: 414 and 396.
constexpr int row_waves(int kpl) { return kpl <= 4 ? 5 : (kpl <= 13 ? 4 : 3); }

constexpr int kTok = 16;  // tokens per chunk

// the value of lane X of each row of 16 lanes, in every lane of the row
template <int X>
__device__ __forceinline__ int32_t row_bcast(int32_t x)
{
    return __builtin_amdgcn_update_dpp(0, x, 0x150 + X, 0xF, 0xF, true);
}
template <int X>
__device__ __forceinline__ float row_bcast(float x)
{
    return __int_as_float(row_bcast<X>(__float_as_int(x)));
}

// What a chunk's steps need of a lane's token; the rest waits in LDS for the
// decision after the chunk.
struct Token {
    int32_t k0;    // own topic (-1: no token)
    float p;       // the own topic's weight without the token
    float u;       // uniform (sign bit set: the token keeps its topic)
    uint32_t row;  // byte offset of its weight row
};

template <int LANES, int KPL, bool ASSOC>
struct RowWave {
    static constexpr int NG = 64 / LANES, W = LANES * KPL;
    static constexpr int BUF = kRowBuffers;
    // first lane of every document of the wavefront
    static constexpr unsigned long long kFirst =
        LANES == 64 ? 1ull : (LANES == 32 ? 0x0000000100000001ull : 0x0001000100010001ull);

    // LDS.  The draws by chunk parity, [NG][16]: x = topic, y = the target's
    // distance into it, z = its width, w = total (or -1 - (2 slot + r) when
    // decided in fp64)
    uint4 (*res)[NG * kTok];
    // tokens of three chunks (the one being drawn, the one before, whose
    // decisions are open, and the next): x = packed state, y = the r = 1 share
    // of the own topic's weight without the token, z = uniform (as in Token)
    uint4 (*tok)[64];
    int32_t *snap;  // [NG][W] document counts after the chunk
    int32_t *fix;   // [W] one document's counts at one token

    int32_t lane, sub, grp, tl, kbase, gV, gK, beg, len;
    int32_t c[KPL];
    Token cur, next;
    int32_t at_prev, at_cur, at_next;  // their places in tok

    // preparation of the next chunk
    uint32_t s_qn;  // row index, and in bit 31 whether that row is narrow
    int32_t s_zr, s_cell, s_b;
    float s_beta, s_f0, s_f1;
    float2 s_qq;

    float d_rho;  // decision of the chunk before: the drawn cell's r = 1 share

    __device__ __forceinline__ void prep0(const RowArgs &A, int32_t ch)
    {
        const int32_t t = beg + min(ch * kTok + tl, max(len - 1, 0));
        const uint32_t q = (uint32_t)A.gw[t];
        s_zr = A.zr_old[t];
        s_qn = q | ((uint32_t)A.tok_narrow[t] << 31);
    }
    // the 32-bit word that holds cell k of row q
    __device__ __forceinline__ int32_t load_cell(const RowArgs &A, int32_t q, int32_t k, bool nar)
    {
        const int64_t cell = (int64_t)q * A.Kp + k;
        const char *at = nar ? reinterpret_cast<const char *>(A.nt16) + (cell & ~1ll) * 2
                             : reinterpret_cast<const char *>(A.nt) + cell * 4;
        return *reinterpret_cast<const int32_t *>(at);
    }
    // the packed cell k from that word (Kp is even, so k's parity is the cell's)
    __device__ __forceinline__ int32_t cell_of(int32_t word, int32_t k, bool nar)
    {
        const uint32_t w = (uint32_t)word;
        return nar ? wide_of(k & 1 ? w >> 16 : w & 0xFFFFu) : word;
    }
    __device__ __forceinline__ float2 load_ratio(const RowArgs &A, int32_t cell)
    {
        const uint32_t v = (uint32_t)cell;
        const uint64_t cn = v & kCountMax, ct = v >> kCountBits;
        const uint64_t ix = ((cn * (cn + 1)) >> 1) + ct;
        const uint64_t q_last = (uint64_t)(A.nQ - 1);
        return A.Q[ix < q_last ? ix : q_last];
    }
    __device__ __forceinline__ void prep1(const RowArgs &A)
    {
        const int32_t q = (int32_t)(s_qn & 0x7FFFFFFFu);
        const int32_t k0 = zr_topic(s_zr), r0 = s_zr & 1;
        s_cell = load_cell(A, q, k0, (int32_t)s_qn < 0);
        const float4 f = A.fz[2 * (gK + k0)];
        s_f0 = f.x;
        s_f1 = r0 ? f.z : f.y;
        if constexpr (ASSOC) {
            const int32_t s0 = zr_slot(s_zr);
            const int32_t *rec = A.srcrec + (int64_t)q * 2 * A.Sp;
            float beta = 0.0f;
            for (int32_t s = 0; s < A.Sp; ++s) {
                const int32_t b = A.B[(int64_t)rec[s] * A.Kp + k0] - ((r0 && s == s0) ? 1 : 0);
                beta = __fmaf_rn(__int_as_float(rec[A.Sp + s]), A.gamma + (float)b, beta);
            }
            s_beta = beta;
        } else {
            s_b = A.B[(int64_t)(q - gV) * A.Kp + k0];
        }
    }
    __device__ __forceinline__ void prep2(const RowArgs &A)
    {
        s_cell = cell_of(s_cell, zr_topic(s_zr), (int32_t)s_qn < 0);
        s_qq = load_ratio(A, s_cell - 1 - ((s_zr & 1) << kCountBits));
        if constexpr (!ASSOC) s_beta = A.gamma + (float)(s_b - (s_zr & 1));
    }
    __device__ __forceinline__ void prep3(const RowArgs &A, int32_t ch)
    {
        const int32_t x = ch * kTok + tl;
        const bool valid = x < len;
        const int32_t n = s_cell & kCountMax, t = s_cell >> kCountBits;
        const bool sole = (s_zr & 1) && t == 1 && n > 1;
        const float p1 = s_f1 * s_beta * s_qq.y;
        next.k0 = valid ? zr_topic(s_zr) : -1;
        next.p = p1 + s_f0 * s_qq.x;
        const float u = sample_uniform(A, beg + x);
        next.u = valid && !sole ? u : __int_as_float(__float_as_int(u) | (int32_t)0x80000000);
        next.row = (s_qn & 0x7FFFFFFFu) * (uint32_t)A.Kw * 4u;
        tok[at_next][lane] =
            make_uint4((uint32_t)s_zr, __float_as_uint(p1 / next.p), __float_as_uint(next.u), 0u);
    }

    // the weight row at byte offset `row` (32 bits), this lane's topics
    __device__ __forceinline__ void fetch(const RowArgs &A, uint32_t row, float (&p)[KPL])
    {
        constexpr int NC = KPL / 4, REM = KPL % 4;
        const char *base = reinterpret_cast<const char *>(A.pw);
#pragma unroll
        for (int q = 0; q < NC; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(
                base + (uint32_t)(row + sub * 16u) + q * LANES * 16);
            p[4 * q + 0] = x.x;
            p[4 * q + 1] = x.y;
            p[4 * q + 2] = x.z;
            p[4 * q + 3] = x.w;
        }
        const float *rest = reinterpret_cast<const float *>(
            base + (uint32_t)(row + sub * (uint32_t)(REM * 4)) + NC * LANES * 16);
        if constexpr (REM == 2) {
            const float2 x = *reinterpret_cast<const float2 *>(rest);
            p[4 * NC + 0] = x.x;
            p[4 * NC + 1] = x.y;
        } else {
#pragma unroll
            for (int j = 0; j < REM; ++j) p[4 * NC + j] = rest[j];
        }
    }

    // Draws token x of chunk ch of every document (k0, po, u: its values).
    // Returns the first lanes of the documents whose draw is in doubt (the
    // target near a topic boundary, or not exactly one crossing): their counts
    // miss the draw.
    __device__ __forceinline__ unsigned long long step(const RowArgs &A, int32_t ch, int32_t x,
                                                       int32_t k0, float po, float u,
                                                       const float (&p)[KPL])
    {
        const int32_t jo = k0 - kbase;
        const bool keep = __float_as_int(u) < 0;
        float s[KPL];
        float acc = 0.0f;
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
            const bool own = jo == j;
            c[j] -= own ? 1 : 0;
            const float d = A.alpha + (float)c[j];
            acc = j == 0 ? d * (own ? po : p[j]) : acc + d * (own ? po : p[j]);
            s[j] = acc;
        }
        const float incl = doc_inclusive_sum<LANES>(acc);
        const float excl = doc_shift_right<LANES>(incl, sub);
        const float total = doc_total<LANES>(incl, lane);
        const float rel = u * total - excl;
        // prefixes are monotone: their number at or below the target, and the
        // distances of the two around it (of floats, the bits of the smallest
        // non-negative one are the smallest as unsigned integers, those of the
        // negative one nearest zero the smallest as signed integers)
        int32_t cnt = 0;
        uint32_t under = __float_as_uint(rel);  // the lane's lower boundary, prefix 0
        int32_t over = INT32_MAX;
#pragma unroll
        for (int j = 0; j < KPL; ++j) {
            const float e = rel - s[j];
            cnt += e >= 0.0f ? 1 : 0;
            under = min(under, __float_as_uint(e));
            over = min(over, __float_as_int(e));
        }
        const float below = __uint_as_float(under), above = -__int_as_float(over);
        // the first lane of each document whose prefixes pass the target
        const unsigned long long pass = __ballot(s[KPL - 1] > rel);
        const unsigned long long at = pass & ~((pass << 1) & ~kFirst);
        const float margin = topic_margin<KPL>(ASSOC ? A.Sp : 0) * total;
        const bool near = below < margin || above < margin;
        const bool here = __builtin_amdgcn_inverse_ballot_w64(at);
        int32_t kk = keep ? jo : (here ? cnt : -1);
        if (here) {
            int32_t g = grp;
            // (its address made anew where, kept over the chunk, it was one
            // register too many and was reloaded for every token)
            if constexpr (ASSOC || KPL > 4) asm volatile("" : "+v"(g));
            res[ch & 1][g * kTok + x] =
                make_uint4((uint32_t)(kbase + cnt), __float_as_uint(below),
                           __float_as_uint(below + above), __float_as_uint(total));
        }
        const unsigned long long doubt = __ballot(near) & at & ~__ballot(keep);
        unsigned long long bad = 0;
        if (doubt != 0 || __popcll(at) != NG) {
            constexpr unsigned long long kAll = LANES == 64 ? ~0ull : (1ull << (LANES & 63)) - 1;
            const int32_t crossings = __popcll((at >> (lane - sub)) & kAll);
            const bool mine = !keep && (((doubt >> (lane - sub)) & kAll) != 0 || crossings != 1);
            bad = __ballot(mine) & kFirst;
            if (mine) kk = -1;
        }
#pragma unroll
        for (int j = 0; j < KPL; ++j) c[j] += (kk == j) ? 1 : 0;
        return bad;
    }

    // After the last step of chunk ch: the load that this lane's token's
    // decision within its topic needs, and the document's counts.
    __device__ __forceinline__ void close(const RowArgs &A, int32_t ch)
    {
        __syncthreads();
        const bool drew = __float_as_int(cur.u) >= 0;
        const int32_t k = drew ? (int32_t)res[ch & 1][grp * kTok + tl].x : 0;
        const uint32_t at = cur.row + 4u * (uint32_t)row_pos<LANES, KPL>(k);
        d_rho = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(A.rho) + at);
#pragma unroll
        for (int j = 0; j < KPL; ++j) snap[grp * W + kbase + j] = c[j];
        __syncthreads();
    }
    // The table indicator (and source slot) of this lane's token of chunk ch,
    // stored; returns the lanes whose target lies near a boundary inside the
    // topic.
    __device__ __forceinline__ unsigned long long finish(const RowArgs &A, int32_t ch)
    {
        const uint4 d = res[ch & 1][grp * kTok + tl], t = tok[at_prev][lane];
        const int32_t x = ch * kTok + tl, zr0 = (int32_t)t.x;
        const bool valid = x < len && sub < kTok, drew = (int32_t)t.z >= 0;
        const int32_t k0 = zr_topic(zr0);
        const int32_t k1 = drew ? (int32_t)d.x : k0;
        const bool own = k1 == k0;
        const float at = __uint_as_float(d.y), width = __uint_as_float(d.z);
        const float total = __uint_as_float(d.w);
        const float margin = inner_margin<KPL>(ASSOC ? A.Sp : 0) * total;
        const float head = width * (own ? __uint_as_float(t.y) : d_rho);
        int32_t r1 = at < head ? 1 : 0, s1 = 0;
        bool near = fabsf(at - head) < margin;
        if constexpr (ASSOC) {
            const int32_t q = A.gw[beg + min(x, max(len - 1, 0))];
            const int32_t r0 = zr0 & 1, s0 = zr_slot(zr0);
            // source slots share the head part in proportion to p_s (gamma + B')
            if (drew && total >= 0.0f && (r1 || near)) {
                const int32_t *rec_s = A.srcrec + (int64_t)q * 2 * A.Sp;
                float beta = 0.0f;
                for (int32_t s = 0; s < A.Sp; ++s) {
                    const int32_t bc = A.B[(int64_t)rec_s[s] * A.Kp + k1] -
                                       ((own && r0 && s == s0) ? 1 : 0);
                    beta = __fmaf_rn(__int_as_float(rec_s[A.Sp + s]), A.gamma + (float)bc, beta);
                }
                const float unit = head / beta;
                float run = 0.0f;
                int32_t last = 0;
                bool found = false;
                for (int32_t s = 0; s < A.Sp; ++s) {
                    const float ps = __int_as_float(rec_s[A.Sp + s]);
                    const int32_t bc = A.B[(int64_t)rec_s[s] * A.Kp + k1] -
                                       ((own && r0 && s == s0) ? 1 : 0);
                    run = __fmaf_rn(ps, A.gamma + (float)bc, run);
                    const float edge = unit * run;
                    if (ps > 0.0f) {
                        near = near || fabsf(at - edge) < margin;
                        last = s;
                        if (!found && at < edge) {
                            found = true;
                            s1 = s;
                        }
                    }
                }
                if (!found) s1 = last;
                if (!r1) s1 = 0;
            }
            if (!drew) s1 = sole_slot64(A, q, k0, s0, fabsf(__uint_as_float(t.z)));
        }
        // decided in fp64 at the token (a token that keeps its topic may have no
        // entry of its own in res: none is written where no prefix passes its target)
        if (drew && total < 0.0f) {
            const int32_t o = (int32_t)(-1.0f - total);
            r1 = o & 1;
            s1 = o >> 1;
            near = false;
        }
        if (valid)
            A.zr_new[beg + x] = drew ? zr_pack(k1, r1, s1) : (ASSOC ? zr_pack(k0, 1, s1) : zr0);
        return __ballot(near && drew && valid);
    }
};

template <int LANES, int KPL, bool ASSOC>
__global__ void __launch_bounds__(64, row_waves(KPL)) k_sample_rows(RowArgs A)
{
    using RW = RowWave<LANES, KPL, ASSOC>;
    constexpr int BUF = RW::BUF, W = RW::W;
    static_assert(BUF == 4, "the first rows are requested below");
    __shared__ uint4 res[2][RW::NG * kTok], tok[3][64];
    __shared__ int32_t snap[64 * KPL], fix[W];

    RW w;
    w.res = res;
    w.tok = tok;
    w.snap = snap;
    w.fix = fix;
    w.lane = threadIdx.x;
    w.sub = w.lane % LANES;
    w.grp = w.lane / LANES;
    w.tl = w.lane % kTok;
    w.kbase = w.sub * KPL;
    const int32_t xcd = blockIdx.x & 7;
    const int32_t i = (int32_t)(blockIdx.x >> 3) * RW::NG + w.grp;
    const int64_t place = (int64_t)xcd * A.docs_per_xcd + i;
    w.beg = 0;
    w.len = 0;
    int32_t g = 0;
    if (i < A.docs_per_xcd && place < A.D) {
        const int32_t d = A.order[place];
        w.len = (int32_t)(A.doc_off[d + 1] - A.doc_off[d]);
        if (w.len > 0) w.beg = (int32_t)A.doc_off[d];
        g = A.doc_group[d];
    }
    int32_t longest = 0;
#pragma unroll
    for (int n = 0; n < RW::NG; ++n) longest = max(longest, readlane(w.len, n * LANES));
    if (longest == 0) return;
    // (an empty document's lanes prepare the first token of one that is not, unused)
    const int32_t some = __ffsll((long long)__ballot(w.len > 0)) - 1;
    if (w.len == 0) {
        w.beg = readlane(w.beg, some);
        g = readlane(g, some);
    }
    w.gV = g * A.V;
    w.gK = g * A.Kp;

    // document counts
#pragma unroll
    for (int j = 0; j < KPL; ++j) snap[w.lane * KPL + j] = 0;
    __syncthreads();
    for (int32_t x = w.sub; x < w.len; x += LANES)
        atomicAdd(&snap[w.grp * W + zr_topic(A.zr_old[w.beg + x])], 1);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KPL; ++j) w.c[j] = snap[w.grp * W + w.kbase + j];

    w.at_next = 0;
    w.prep0(A, 0);
    w.prep1(A);
    w.prep2(A);
    w.prep3(A, 0);
    w.cur = w.next;
    w.at_cur = 0;
    w.at_next = 1;
    w.at_prev = 2;
    float p[BUF][KPL];
    w.fetch(A, row_bcast<0>((int32_t)w.cur.row), p[0]);
    w.fetch(A, row_bcast<1>((int32_t)w.cur.row), p[1]);
    w.fetch(A, row_bcast<2>((int32_t)w.cur.row), p[2]);

    for (int32_t ch = 0;; ++ch) {
        const int32_t left = longest - ch * kTok;  // <= 0: only the last decisions are open
        unsigned long long bad = 0;
        int32_t x = 0;
        do {
            if (left <= 0) break;
#define SPDP_STEP(X)                                                                              \
    {                                                                                             \
        constexpr int kA = X + BUF - 1;                                                           \
        w.fetch(A, (uint32_t)(kA < kTok ? row_bcast<kA % kTok>((int32_t)w.cur.row)                \
                                        : row_bcast<kA % kTok>((int32_t)w.next.row)),             \
                p[kA % BUF]);                                                                     \
        bad = w.step(A, ch, X, row_bcast<X>(w.cur.k0), row_bcast<X>(w.cur.p),                     \
                     row_bcast<X>(w.cur.u), p[X % BUF]);                                          \
        x = X;                                                                                    \
        if (bad) break;                                                                           \
    }
            w.prep0(A, ch + 1);
            SPDP_STEP(0) SPDP_STEP(1) SPDP_STEP(2) SPDP_STEP(3)
            if (left <= 4) break;
            w.prep1(A);
            SPDP_STEP(4) SPDP_STEP(5) SPDP_STEP(6) SPDP_STEP(7)
            if (left <= 8) break;
            w.prep2(A);
            SPDP_STEP(8) SPDP_STEP(9) SPDP_STEP(10) SPDP_STEP(11)
            if (left <= 12) break;
            w.prep3(A, ch + 1);
            SPDP_STEP(12) SPDP_STEP(13) SPDP_STEP(14) SPDP_STEP(15)
#undef SPDP_STEP
        } while (0);
        unsigned long long late = 0;
        if (ch > 0) late = w.finish(A, ch - 1);
        if (bad | late) {
            // Draws in doubt, one at a time: a token of the chunk before, whose
            // document's counts at that token are those after that chunk with
            // its own and the later moves taken back (late), or a document's
            // token x just taken (bad).  Then the rest of this chunk, token by
            // token, and the preparations it cut short.
            const bool cut = bad != 0;
            for (;;) {
                while (late | bad) {
                    const bool now = late == 0;
                    unsigned long long &todo = now ? bad : late;
                    const int32_t L = __ffsll((long long)todo) - 1;
                    todo &= todo - 1;
                    const int32_t gd = L / LANES, xd = now ? x : L % kTok;
                    const uint4 before = tok[w.at_prev][w.lane];
                    const int32_t k1 = (int32_t)res[(ch - 1) & 1][w.grp * kTok + w.tl].x;
                    __syncthreads();
                    if (w.grp == gd) {
#pragma unroll
                        for (int j = 0; j < KPL; ++j)
                            fix[w.kbase + j] = now ? w.c[j] : snap[w.grp * W + w.kbase + j];
                    }
                    __syncthreads();
                    if (!now && w.grp == gd && w.sub < kTok && w.tl >= xd &&
                        (int32_t)before.z >= 0) {
                        atomicAdd(&fix[k1], -1);
                        if (w.tl > xd) atomicAdd(&fix[zr_topic((int32_t)before.x)], 1);
                    }
                    __syncthreads();
                    const int32_t t = readlane(w.beg, L) + (now ? ch : ch - 1) * kTok + xd;
                    const int32_t zr0 = A.zr_old[t];
                    const int32_t zr =
                        decide64<ASSOC>(A.exact, A.gw[t], readlane(w.gV, L), readlane(w.gK, L),
                                        zr0, sample_uniform(A, t), (LdsCounts)fix);
                    const int32_t k = readlane(zr_topic(zr), 0);
                    if (now) {
                        if (w.grp == gd) {
#pragma unroll
                            for (int j = 0; j < KPL; ++j)
                                w.c[j] += (k - w.kbase == j) ? 1 : 0;
                            if (w.sub == 0)
                                res[ch & 1][gd * kTok + xd] =
                                    make_uint4((uint32_t)k, 0u, 0u,
                                               __float_as_uint(-1.0f - (float)(2 * zr_slot(zr) +
                                                                               (zr & 1))));
                        }
                    } else if (w.lane == L && k == k1) {
                        A.zr_new[t] = zr;
                    }
                    __syncthreads();
                }
                if (!cut || ++x >= kTok || x >= left) break;
                const int32_t from = (w.lane & ~(kTok - 1)) + x;
                w.fetch(A, (uint32_t)__shfl((int32_t)w.cur.row, from), p[0]);
                bad = w.step(A, ch, x, __shfl(w.cur.k0, from), __shfl(w.cur.p, from),
                             __shfl(w.cur.u, from), p[0]);
            }
            // (also where nothing was cut: then no prefetch lives across the above)
            w.prep0(A, ch + 1);
            w.prep1(A);
            w.prep2(A);
            w.prep3(A, ch + 1);
            w.fetch(A, row_bcast<0>((int32_t)w.next.row), p[0]);
            w.fetch(A, row_bcast<1>((int32_t)w.next.row), p[1]);
            w.fetch(A, row_bcast<2>((int32_t)w.next.row), p[2]);
        }
        if (left <= 0) break;
        w.close(A, ch);
        w.cur = w.next;
        const int32_t at = w.at_prev;
        w.at_prev = w.at_cur;
        w.at_cur = w.at_next;
        w.at_next = at;
    }
}

template <int LANES, int KPL, bool ASSOC>
hipError_t launch_rows_shape(const RowArgs &A, hipStream_t st)
{
    constexpr int NG = 64 / LANES;
    const unsigned grid = 8u * (unsigned)((A.docs_per_xcd + NG - 1) / NG);
    hipLaunchKernelGGL((k_sample_rows<LANES, KPL, ASSOC>), dim3(grid), dim3(64), 0, st, A);
    return hipGetLastError();
}

template <int LANES, bool ASSOC>
hipError_t launch_rows_lanes(const RowArgs &A, int kpl, hipStream_t st)
{
    if constexpr (LANES < 64) {  // (64 lanes hold three topics each at least, see row_shape)
        if (kpl == 1) return launch_rows_shape<LANES, 1, ASSOC>(A, st);
        if (kpl == 2) return launch_rows_shape<LANES, 2, ASSOC>(A, st);
    }
    switch (kpl) {
    case 3: return launch_rows_shape<LANES, 3, ASSOC>(A, st);
    case 4: return launch_rows_shape<LANES, 4, ASSOC>(A, st);
    case 5: return launch_rows_shape<LANES, 5, ASSOC>(A, st);
    case 6: return launch_rows_shape<LANES, 6, ASSOC>(A, st);
    case 7: return launch_rows_shape<LANES, 7, ASSOC>(A, st);
    case 8: return launch_rows_shape<LANES, 8, ASSOC>(A, st);
    case 10: return launch_rows_shape<LANES, 10, ASSOC>(A, st);
    case 12: return launch_rows_shape<LANES, 12, ASSOC>(A, st);
    case 13: return launch_rows_shape<LANES, 13, ASSOC>(A, st);
    case 14: return launch_rows_shape<LANES, 14, ASSOC>(A, st);
    case 16: return launch_rows_shape<LANES, 16, ASSOC>(A, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

}  // namespace spdp
