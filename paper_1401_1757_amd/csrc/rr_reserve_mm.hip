// Per-policy reserves as a matrix product on the FP64 matrix cores:
// r_0[policy][scenario] = sum_t f_t[policy] D_t[scenario], f the expected cash
// flows (rr_flows.h), D the discount products kept beside the curves.
#include "rr_flows.h"

#include <algorithm>
#include <type_traits>

namespace rr {

typedef double f64x4 __attribute__((ext_vector_type(4)));
// Two doubles moved by one 16-byte access, at 8-byte alignment.
typedef double f64x2 __attribute__((ext_vector_type(2), aligned(8)));

// N consecutive doubles, in 16-byte accesses where there are two or more.
template <int N>
__device__ __forceinline__ void load_run(double (&x)[N], const double *__restrict__ p)
{
    if constexpr (N == 1) {
        x[0] = p[0];
    } else {
#pragma unroll
        for (int i = 0; i < N; i += 2) {
            const f64x2 v = *reinterpret_cast<const f64x2 *>(p + i);
            x[i] = v[0];
            x[i + 1] = v[1];
        }
    }
}

// ---------------------------------------------------------------------------
// Discount products D[node][t][scen_pad], t = 0 .. n_steps, from the curves
// (and rows of zeros up to disc_rows, so that the multiplying kernel reads whole
// blocks of months).
// Sixteen wavefronts cut the months of 64 scenarios; each multiplies its chunk,
// then writes its months from the product of the chunks before it.  Bound by
// the write and the two reads of the curves (the second from the L2).
// ---------------------------------------------------------------------------
constexpr int DISC_CHUNKS = 16;

__global__ void __launch_bounds__(64 * DISC_CHUNKS) k_disc(const double *__restrict__ v, int n_steps,
                                                           int scen_pad, double *__restrict__ D)
{
    __shared__ double sh[DISC_CHUNKS][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int s = min((int)blockIdx.x * 64 + lane, scen_pad - 1);   // the last lanes repeat a column
    const double *vk = v + (size_t)blockIdx.y * n_steps * scen_pad + s;
    double *dk = D + (size_t)blockIdx.y * disc_rows(n_steps) * scen_pad + s;
    const int per = (n_steps + DISC_CHUNKS - 1) / DISC_CHUNKS;
    const int t0 = min(wave * per, n_steps), t1 = min(t0 + per, n_steps);
    constexpr int U = 8;
    double p = 1.0;
    int t = t0;
    for (; t + U <= t1; t += U) {
        double x[U];
#pragma unroll
        for (int i = 0; i < U; ++i) x[i] = vk[(size_t)(t + i) * scen_pad];
#pragma unroll
        for (int i = 0; i < U; ++i) p *= x[i];
    }
    for (; t < t1; ++t) p *= vk[(size_t)t * scen_pad];
    sh[wave][lane] = p;
    __syncthreads();
    double d = 1.0;
    for (int w = 0; w < wave; ++w) d *= sh[w][lane];
    if (wave == 0) dk[0] = 1.0;
    if (wave == DISC_CHUNKS - 1)   // rows that whole blocks of months reach
        for (t = n_steps + 1; t < disc_rows(n_steps); ++t) dk[(size_t)t * scen_pad] = 0.0;
    for (t = t0; t + U <= t1; t += U) {
        double x[U];
#pragma unroll
        for (int i = 0; i < U; ++i) x[i] = vk[(size_t)(t + i) * scen_pad];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            d *= x[i];
            dk[(size_t)(t + i + 1) * scen_pad] = d;
        }
    }
    for (; t < t1; ++t) {
        d *= vk[(size_t)t * scen_pad];
        dk[(size_t)(t + 1) * scen_pad] = d;
    }
}

hipError_t launch_discounts(const double *v, int n_nodes, int n_steps, int scen_pad, double *D, hipStream_t s)
{
    for (int k = 0; k < n_nodes; k += 65535) {
        const int nodes = std::min(n_nodes - k, 65535);
        hipLaunchKernelGGL(k_disc, dim3((scen_pad + 63) / 64, nodes), dim3(64 * DISC_CHUNKS), 0, s,
                           v + (size_t)k * n_steps * scen_pad, n_steps, scen_pad,
                           D + (size_t)k * disc_rows(n_steps) * scen_pad);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Reserves
// ---------------------------------------------------------------------------
constexpr int MM_WAVES = 4;
constexpr int MM_G = 2;          // fragments of four months per step of the pipeline

// One fragment of v_mfma_f64_16x16x4_f64: lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and of the result rows 4 i + l / 16 (i = 0..3) of column l % 16.
__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// A workgroup takes a tile of 64 policies and 16 WC NB scenarios of a node: WC
// wavefronts side by side over the scenarios, 4 / WC over the policies, each
// with its part of the reserves in accumulators.  Flows (one line of 64 a month)
// and discount products (one line of scenarios a month) go straight from memory
// into fragments, eight months ahead of their use; the workgroup's wavefronts
// share their lines in the L1.  No LDS, no barriers.  A lane's policies of all
// fragments lie side by side in the kept flows, and its NB scenarios are
// neighbours, so that every access is 16 bytes a lane (NB = 2): the L1 takes 16
// cycles for a wavefront's access of 8 bytes a lane as for one of 16 (10,000
// policies x 1,000 scenarios, the whole call: 0.189 -> 0.178 ms).
//
// Bound by the FP64 matrix pipe while the chip is full, and by the long tiles
// after that: 10,000 x 1,000 are 6.9 GFLOP with their padding in 127 us, the pipe
// busy 0.76 of the kernel's cycles.  The flows are made by a launch of their own:
// with a wavefront that makes them beside the multiplying ones, waiting for the
// matrix pipe at every FP64 operation, that call took 0.192 ms instead of 0.189.
// Tiles go longest first; the block index modulo the scenario blocks is the
// scenario block, so that (eight blocks: exactly) one XCD's L2 serves few
// columns of the discount products.
template <bool FRAC, int WC, int NB>
__global__ void __launch_bounds__(64 * MM_WAVES, 3)
k_reserve_mm(RecParams P, FlowStore st, int node_begin, int n_sb)
{
    constexpr int WR = MM_WAVES / WC, MB = 4 / WR, G = MM_G;
    const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int sb = blockIdx.x % n_sb, rank = blockIdx.x / n_sb;
    const bool all = st.tile_end - st.tile_begin == P.n_tiles;
    const int tile = all ? wave_uniform(P.tile_order[rank]) : st.tile_begin + rank;
    const int node = node_begin + blockIdx.y;
    const int first = wave_uniform(P.tiles[tile].first);
    const int smax = wave_uniform(P.tiles[tile].smax) - node * P.node_step;
    const bool frac = FRAC && wave_uniform(P.tiles[tile].flow) == FLOW_FRAC;
    const int steps = smax > 0 ? smax / (4 * G) + 1 : 0;   // the flows' whole blocks of eight months
    static_assert(4 * G == 8, "a pipeline step is a block of kept flows");
    const int wc = wave % WC, wr = wave / WC;
    const int l16 = lane & 15, lk = lane >> 4;
    const int col0 = ((sb * WC + wc) * 16 + l16) * NB;   // the lane's first scenario in the run
    const int drow = P.scen_pad;
    const double *D = P.disc + (size_t)node * disc_rows(P.n_steps) * drow + P.scen_begin;
    const double *F = st.flows + ((size_t)blockIdx.y * st.node_months + (P.tile_base[tile] - st.month_begin)) * 64;
    // The lane's elements of a fragment of four months.  Lanes past the run read
    // its last scenario (and the one after: rows are padded) and store nothing.
    const int boff = lk * drow + min(col0, P.scen_count - 1);
    const int aoff = lk * 64 + l16 * 4 + wr * MB;
    f64x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[i][n] = f64x4{0.0, 0.0, 0.0, 0.0};
    // The product over the flows at `fl`, with the discount products or (MID) for
    // flows within the month with D_t v_t^f.
    auto product = [&](const double *fl, auto mid) {
        constexpr bool MID = decltype(mid)::value;
        struct Frags {
            double a[G][MB], b[G][NB], c[MID ? G : 1][NB];
        };
        const double *vf = MID ? P.vf + (size_t)node * P.n_steps * drow + P.scen_begin : nullptr;
        auto load = [&](Frags &x, int s) {   // step s (the last one again past it: not used)
            const int t = min(s, steps - 1) * 4 * G;
#pragma unroll
            for (int k = 0; k < G; ++k) {
                load_run<MB>(x.a[k], fl + (size_t)(t + 4 * k) * 64 + aoff);
                load_run<NB>(x.b[k], D + (size_t)(t + 4 * k) * drow + boff);
                if constexpr (MID) {   // v^f has no row past the last month (its flows are 0)
                    const int row = min(t + 4 * k + lk, P.n_steps - 1) - lk;
                    load_run<NB>(x.c[k], vf + (ptrdiff_t)row * drow + boff);
                }
            }
        };
        auto multiply = [&](const Frags &x) {
#pragma unroll
            for (int k = 0; k < G; ++k)
#pragma unroll
                for (int i = 0; i < MB; ++i)
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        acc[i][n] = mfma64(x.a[k][i], MID ? x.b[k][n] * x.c[k][n] : x.b[k][n], acc[i][n]);
        };
        // Two sets of fragments by turns: the next step's are requested before a
        // step's multiplications (thousands of cycles among a SIMD's wavefronts).
        Frags x0, x1;
        load(x0, 0);
        int s = 0;
        for (; s + 1 < steps; s += 2) {
            __builtin_amdgcn_sched_barrier(0);
            load(x1, s + 1);
            __builtin_amdgcn_sched_barrier(0);
            multiply(x0);
            __builtin_amdgcn_sched_barrier(0);
            load(x0, s + 2);
            __builtin_amdgcn_sched_barrier(0);
            multiply(x1);
        }
        if (s < steps) multiply(x0);
    };
    if (steps > 0) {
        product(F, std::false_type{});
        if constexpr (FRAC) {
            if (frac) product(F + st.mid, std::true_type{});
        }
    }
    double *out = P.r0 + (size_t)(node - P.node_begin) * P.n_user * P.scen_count;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int uid = P.uidx[first + (wr * MB + i) * 16 + 4 * r + lk];
            if (uid < 0) continue;
            double *o = out + (size_t)uid * P.scen_count + col0;
            if constexpr (NB == 2) {
                if (col0 + 1 < P.scen_count) {
                    *reinterpret_cast<f64x2 *>(o) = f64x2{acc[i][0][r], acc[i][1][r]};
                    continue;
                }
            }
#pragma unroll
            for (int n = 0; n < NB; ++n)
                if (col0 + n < P.scen_count) o[n] = acc[i][n][r];
        }
}

template <int WC, int NB>
static void launch_mm(const RecParams &p, const FlowStore &st, int node_begin, int nodes, bool has_mid, hipStream_t s)
{
    const int n_sb = (p.scen_count + 16 * WC * NB - 1) / (16 * WC * NB);
    const dim3 g(n_sb * (st.tile_end - st.tile_begin), nodes), b(64 * MM_WAVES);
    if (has_mid) hipLaunchKernelGGL((k_reserve_mm<true, WC, NB>), g, b, 0, s, p, st, node_begin, n_sb);
    else hipLaunchKernelGGL((k_reserve_mm<false, WC, NB>), g, b, 0, s, p, st, node_begin, n_sb);
}

// The shape of a workgroup's part, 64 policies x 16, 32, 64 or 128 scenarios, by the
// number of workgroups: a larger part reads less a product, and keeps fewer
// CUs at work.  Whole calls, us, (WC, NB) = (1, 1) / (2, 1) / (2, 2) / (4, 2):
//   10,000 policies x 48 44 / 45 / 49 / 68, x 64 49 / 45 / 50 / 69 (471 and 628
//   parts of 16 scenarios), 1,000 x 20 nodes x 24 53 / 50 / 63 / 92;
//   10,000 x 160 73 / 58 / 60 / 78, x 200 85 / 69 / 66 / 78 (471 and 628 parts of
//   64), 30,000 x 40 78 / 68 / 63 / 91;
//   10,000 x 1,000 284 / 171 / 147 / 154 (2,512 parts of 64), 1,000 x 20 x 500
//   228 / 166 / 137 / 131 (2,560), 30,000 x 1,000 811 / 439 / 362 / 334.
// Every shape adds a reserve's products in the same order: the same bits.
hipError_t launch_reserve_mm(const RecParams &p, int node_begin, int nodes, bool has_mid, const FlowStore &st,
                             hipStream_t s)
{
    const int sc = p.scen_count;
    const long long tiles = (long long)(st.tile_end - st.tile_begin) * nodes;
    auto parts = [&](int scenarios) { return tiles * ((sc + scenarios - 1) / scenarios); };
    if (sc <= 16 || parts(16) < 512) launch_mm<1, 1>(p, st, node_begin, nodes, has_mid, s);
    else if (sc <= 32 || parts(64) < 460) launch_mm<2, 1>(p, st, node_begin, nodes, has_mid, s);
    else if (parts(64) < 2560) launch_mm<2, 2>(p, st, node_begin, nodes, has_mid, s);
    else launch_mm<4, 2>(p, st, node_begin, nodes, has_mid, s);
    return hipGetLastError();
}

}  // namespace rr
