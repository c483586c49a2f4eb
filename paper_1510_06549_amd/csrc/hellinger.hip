// hellinger.hip -- Hellinger distances between two topic models (gfx950).
//
// The thesis compares topic models by the Hellinger distance between every
// pair of their topics, the second model's topics re-ordered to line up with
// the first's (chapter "Experiments", subsection "Hellinger Distance").  For
// distributions p, q over the same V outcomes
//   H(p, q)^2 = 1/2 sum_v (sqrt p_v - sqrt q_v)^2 = 1 - BC(p, q),
//   BC(p, q)  = sum_v sqrt(p_v) sqrt(q_v)      (Bhattacharyya coefficient),
// so all kp x kq coefficients are one dense contraction over the outcomes,
//   BC = sqrt(P)^T sqrt(Q),   P [V][kp], Q [V][kq]  (topics contiguous),
// which runs on the fp64 matrix cores: v_mfma_f64_16x16x4 blocks, 64 x 64 or
// 128 x 128 output tiles per 256-thread block, 16 outcomes staged per step
// through LDS with the square roots taken once per staged value.  The outcome axis is
// split into slices so that the grid fills the chip even for small K; the
// slices' partial sums are added in slice order (deterministic) and
// H = sqrt(max(0, 1 - BC)).
//
// Reordering the topics to line up is read as the one-to-one matching of topics with the
// least total distance.  That linear assignment problem is solved on the host
// (shortest augmenting paths with row and column potentials, the Hungarian
// method of Kuhn and Munkres in O(kp^2 kq)): each augmentation is a chain of
// dependent minimum searches, too sequential to gain from the GPU at the
// topic counts of a topic model.
#include "spdp_internal.hpp"

#include <cmath>
#include <limits>
#include <mutex>
#include <vector>

namespace spdp {

// Partial sums of the allocation-free entry point (spdp_hellinger_noalloc):
// one array per GPU, held until the process ends.  Host code never passes
// this name to a kernel -- on the host it is only a stand-in for the symbol --
// but the device address that hellinger_scratch() looks up once per device.
static __device__ __align__(256) double scratch[kHellingerScratch];

namespace {

constexpr int kTile = 64;     // output tile of the plan's unit: kTile x kTile coefficients
constexpr int kStage = 16;    // outcomes per LDS stage (4 MFMA k-steps)
constexpr int kThreads = 256; // 4 waves, each a quarter of the tile

typedef double d4 __attribute__((ext_vector_type(4)));

// part[s][i][j] = sum over outcomes v of slice s of sqrt(P[v][i]) sqrt(Q[v][j]),
// for one TILE x TILE tile per block, each wave a quarter of it as NB x NB
// matrix-core blocks.  A stage's values are requested before the stage before
// it is multiplied, their square roots taken after it and written to the other
// LDS buffer, so one barrier per stage suffices and neither the loads' latency
// nor the square roots of one wave leave the matrix cores waiting.  The square
// roots (about 90 cycles each) are the competitor: a 64 x 64 tile takes 8 per
// thread and 16 MFMAs (64 cycles each) per stage, a 128 x 128 tile 16 and 64,
// so the larger tile is the better where the topics fill it.  Rows of kPitch
// doubles put the four k-steps of a block's reads on different LDS banks.
// 500 x 500 topics over 100 000 outcomes: 1.2 ms (42 TFLOP/s; a library product
// of 4 096^2 reaches 61 on this card), 2.28 ms with 64 x 64 tiles, one
// buffer and no prefetch (22 TFLOP/s).
template <int TILE>
__global__ void __launch_bounds__(kThreads) k_bc(const double *__restrict__ P, int32_t kp,
                                                 const double *__restrict__ Q, int32_t kq,
                                                 int64_t V, int64_t slice, int32_t tiles_j,
                                                 double *__restrict__ part)
{
    constexpr int NB = TILE / 32;                        // blocks per wave and side
    constexpr int kPitch = TILE + 16;
    constexpr int kLoads = kStage * TILE / kThreads;     // values of P (and Q) per thread
    constexpr int kRowStep = kThreads / TILE;
    __shared__ double sP[2][kStage][kPitch], sQ[2][kStage][kPitch];
    const int32_t i0 = (int32_t)(blockIdx.x / tiles_j) * TILE;
    const int32_t j0 = (int32_t)(blockIdx.x % tiles_j) * TILE;
    const int64_t v_beg = (int64_t)blockIdx.y * slice;
    const int64_t v_end = v_beg + slice < V ? v_beg + slice : V;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wi = (wave >> 1) * (TILE / 2), wj = (wave & 1) * (TILE / 2);
    // A operand: lane holds row (lane & 15) of the block at k-step (lane >> 4);
    // B operand: column (lane & 15) at k-step (lane >> 4)
    const int kr = lane >> 4, kc = lane & 15;
    // this thread stages column tc of rows tr, tr + kRowStep, ...
    const int tc = tid % TILE, tr = tid / TILE;
    const bool in_i = i0 + tc < kp, in_j = j0 + tc < kq;
    d4 acc[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};

    double rp[kLoads], rq[kLoads];
    auto request = [&](int64_t v0) {
#pragma unroll
        for (int e = 0; e < kLoads; ++e) {
            const int64_t v = v0 + tr + e * kRowStep;
            const bool in_v = v < v_end;
            rp[e] = (in_v && in_i) ? P[v * kp + i0 + tc] : 0.0;
            rq[e] = (in_v && in_j) ? Q[v * kq + j0 + tc] : 0.0;
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int e = 0; e < kLoads; ++e) {
            sP[buf][tr + e * kRowStep][tc] = sqrt(rp[e]);
            sQ[buf][tr + e * kRowStep][tc] = sqrt(rq[e]);
        }
    };
    request(v_beg);
    stage(0);
    __syncthreads();
    int buf = 0;
    for (int64_t v0 = v_beg; v0 < v_end; v0 += kStage) {
        const bool more = v0 + kStage < v_end;
        if (more) request(v0 + kStage);
#pragma unroll
        for (int ks = 0; ks < kStage; ks += 4) {
            double a[NB], b[NB];
#pragma unroll
            for (int x = 0; x < NB; ++x) {
                a[x] = sP[buf][ks + kr][wi + 16 * x + kc];
                b[x] = sQ[buf][ks + kr][wj + 16 * x + kc];
            }
#pragma unroll
            for (int x = 0; x < NB; ++x)
#pragma unroll
                for (int y = 0; y < NB; ++y)
                    acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[x], b[y], acc[x][y], 0, 0, 0);
        }
        buf ^= 1;
        if (more) stage(buf);
        __syncthreads();
    }

    // result block (fp64 layout): value r of a lane is row 4 r + (lane >> 4),
    // column lane & 15
    double *out = part + (int64_t)blockIdx.y * kp * kq;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int32_t i = i0 + wi + bi * 16 + 4 * r + kr;
                const int32_t j = j0 + wj + bj * 16 + kc;
                if (i < kp && j < kq) out[(int64_t)i * kq + j] = acc[bi][bj][r];
            }
}

__global__ void k_hell_finish(int64_t n, int32_t slices, const double *__restrict__ part,
                              double *__restrict__ h)
{
    const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    double bc = 0.0;
    for (int32_t s = 0; s < slices; ++s) bc += part[(int64_t)s * n + j];
    const double d = 1.0 - bc;
    h[j] = sqrt(d > 0.0 ? d : 0.0);
}

}  // namespace

int hellinger_scratch(int device, double **out)
{
    static std::mutex mu;
    static double *addr[kMaxDevices] = {};
    static bool looked_up[kMaxDevices] = {};
    *out = nullptr;
    if (device < 0 || device >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!looked_up[device]) {
        int cur = 0;
        hipError_t e = hipGetDevice(&cur);
        if (e == hipSuccess && cur != device) e = hipSetDevice(device);
        void *p = nullptr;
        if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return (int)e;
        addr[device] = static_cast<double *>(p);
        looked_up[device] = true;
    }
    *out = addr[device];
    return (int)hipSuccess;
}

// Tile and outcome slices.  128 x 128 tiles unless they would be filled by less
// than two thirds of what 64 x 64 tiles are (kp = 65, say), or the outcomes or
// the partial sums' room allow too few blocks of them for the chip (one block
// per compute unit at least); with them one slice per two blocks of a compute
// unit, with 64 x 64 tiles 2 048 blocks, both with at least 16 stages a slice.
HellingerPlan hellinger_plan(int32_t kp, int32_t kq, int64_t V, int64_t max_part)
{
    HellingerPlan p;
    const int64_t nh = (int64_t)kp * kq;
    if (nh == 0) return p;  // nothing to launch
    const int64_t stages = (V + kStage - 1) / kStage;
    const int64_t room = max_part / nh > 0 ? max_part / nh : 1;  // slices whose sums fit
    auto tiles_of = [&](int64_t t) { return ((kp + t - 1) / t) * ((kq + t - 1) / t); };
    auto slices_of = [&](int64_t tiles, int64_t blocks) {
        int64_t want = (blocks + tiles - 1) / tiles;
        const int64_t most = (stages + 15) / 16;
        if (want > most) want = most;
        if (want > room) want = room;
        return want < 1 ? (int64_t)1 : want;
    };
    const int64_t t64 = tiles_of(kTile), t128 = tiles_of(2 * kTile);
    const bool large = 8 * t128 <= 3 * t64 && t128 * slices_of(t128, 512) >= 256;
    p.tile = large ? 2 * kTile : kTile;
    p.tiles = large ? t128 : t64;
    p.tiles_j = (kq + p.tile - 1) / p.tile;
    const int64_t want = slices_of(p.tiles, large ? 512 : 2048);
    const int64_t per = (stages + want - 1) / want;  // stages per slice
    p.slice = per * kStage;
    p.slices = (int32_t)(V > 0 ? (V + p.slice - 1) / p.slice : 1);
    return p;
}

HellingerPlan hellinger_plan(int32_t kp, int32_t kq, int64_t V)
{
    return hellinger_plan(kp, kq, V, INT64_MAX);
}

hipError_t launch_hellinger(const HellingerPlan &p, const double *P, int32_t kp, const double *Q,
                            int32_t kq, int64_t V, double *part, double *h, hipStream_t st)
{
    const int64_t n = (int64_t)kp * kq;
    if (n == 0) return hipSuccess;
    if (V > 0) {
        const dim3 grid((unsigned)p.tiles, (unsigned)p.slices);
        if (p.tile == kTile)
            hipLaunchKernelGGL(k_bc<kTile>, grid, dim3(kThreads), 0, st, P, kp, Q, kq, V, p.slice,
                               p.tiles_j, part);
        else
            hipLaunchKernelGGL(k_bc<2 * kTile>, grid, dim3(kThreads), 0, st, P, kp, Q, kq, V,
                               p.slice, p.tiles_j, part);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int32_t slices = V > 0 ? p.slices : 0;  // no outcomes: BC = 0, H = 1
    hipLaunchKernelGGL(k_hell_finish, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n,
                       slices, part, h);
    return hipGetLastError();
}

// Least-total-cost matching of every row of c [kp][kq] (kp <= kq) to its own
// column: for each new row, a shortest augmenting path over the reduced costs
// c[i][j] - u[i] - v[j] (Dijkstra over columns), then the potentials are
// shifted so that matched pairs keep reduced cost 0 and all others stay >= 0.
double align_topics_host(const double *c, int32_t kp, int32_t kq, int32_t *match)
{
    const double inf = std::numeric_limits<double>::infinity();
    // index 0 is a virtual column / row; real rows 1..kp, columns 1..kq
    std::vector<double> u((size_t)kp + 1, 0.0), v((size_t)kq + 1, 0.0), dist((size_t)kq + 1);
    std::vector<int32_t> owner((size_t)kq + 1, 0), prev((size_t)kq + 1, 0);
    std::vector<char> done((size_t)kq + 1);
    for (int32_t row = 1; row <= kp; ++row) {
        owner[0] = row;
        int32_t col = 0;
        std::fill(dist.begin(), dist.end(), inf);
        std::fill(done.begin(), done.end(), 0);
        while (owner[col] != 0) {
            done[col] = 1;
            const int32_t i = owner[col];
            double step = inf;
            int32_t next = 0;
            for (int32_t j = 1; j <= kq; ++j) {
                if (done[j]) continue;
                const double red = c[(int64_t)(i - 1) * kq + (j - 1)] - u[i] - v[j];
                if (red < dist[j]) {
                    dist[j] = red;
                    prev[j] = col;
                }
                if (dist[j] < step) {
                    step = dist[j];
                    next = j;
                }
            }
            for (int32_t j = 0; j <= kq; ++j) {
                if (done[j]) {
                    u[owner[j]] += step;
                    v[j] -= step;
                } else {
                    dist[j] -= step;
                }
            }
            col = next;
        }
        // flip the path: every column on it takes the row of its predecessor
        while (col != 0) {
            const int32_t p = prev[col];
            owner[col] = owner[p];
            col = p;
        }
    }
    double total = 0.0;
    for (int32_t j = 1; j <= kq; ++j)
        if (owner[j] != 0) match[owner[j] - 1] = j - 1;
    for (int32_t i = 0; i < kp; ++i) total += c[(int64_t)i * kq + match[i]];
    return total;
}

}  // namespace spdp
