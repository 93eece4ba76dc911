// Portfolio totals by summed cash flows: a node's expected cash flows added up
// over the policies (once for all scenarios), then the backward recurrence
// R_t = F_t + v_t R_{t+1} of that one sequence per scenario.
#include "rr_flows.h"

#include <algorithm>
#include <type_traits>

namespace rr {

constexpr int FLOW_U = 4;                  // steps loaded together
constexpr int FLOW_BLK = 8;                // steps per row reduction; rows are whole blocks
constexpr int FLOW_WAVES = 8;              // wavefronts per workgroup
constexpr int FLOW_ROW = 65;               // stage rows: 65 doubles apart, 8 columns per lane on distinct banks
constexpr int FLOW_STAGE = FLOW_BLK * FLOW_ROW;
constexpr int FLOW_RED = 64;               // rows per workgroup of the row reduction

// x + the value of the lane 16 (32) away, by the row-swap instructions: both
// outputs of a swap of x with itself, added.
__device__ __forceinline__ double add_across_16(double x)
{
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double add_across_32(double x)
{
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// A wavefront's row: flows of the 64 lanes pass through its LDS stage in
// blocks of eight steps; lane l adds eight lanes' flows of step l % 8, three
// exchanges add the eight parts, in a fixed order.  A later walk adds to what
// an earlier one wrote.  Only that branch waits for memory: a wait for the old
// values of every block would also wait for the store of the block before
// (four times the walk's time).
struct FlowRow {
    double *stage, *dst;
    int have;   // length written so far

    __device__ __forceinline__ void put(int t, double x, int lane) { stage[(t & (FLOW_BLK - 1)) * FLOW_ROW + lane] = x; }
    // After the last step of the block that ends before t.
    __device__ __forceinline__ void flush(int t, int lane)
    {
        __builtin_amdgcn_wave_barrier();
        const double *p = stage + (lane & 7) * FLOW_ROW + (lane >> 3) * 8;
        double s = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        s += dpp_f64<0x128>(s);   // row_ror:8: the lane 8 away
        s = add_across_32(add_across_16(s));
        if (lane < FLOW_BLK) {
            double *o = dst + (t - FLOW_BLK) + lane;
            if (t <= have) s += *o;
            *o = s;
        }
        __builtin_amdgcn_wave_barrier();
    }
};

// Rows of summed flows, row_len doubles each: row g of a node (grid: rows x
// nodes) takes the tiles g, g + R, ...  CHUNKS wavefronts share a row, a time
// chunk each, since the serial walk over hundreds of months is what a run waits
// for: they exchange their chunks' transfers first and then walk from the state
// these lead to.  A workgroup holds FLOW_WAVES / CHUNKS rows and one copy of the
// survival tables.  Every wavefront passes the same barriers whatever its tile's model.
//
// With `st` the flows themselves are kept too (or, without rows, only), for
// k_reserve_mm: one line of 64 policies a month.
//
// Bound by vector issue: per policy-month the table reads, about ten FP64
// operations and two multiplications for the transfer.  See flow_shape for the
// split and its figures.
template <bool LDSQ, bool VEC, int SET, int CHUNKS>
__global__ void __launch_bounds__(64 * FLOW_WAVES, SET == FLOWS_ALL ? 2 : 4)
k_flow_sums(RecParams P, int node_begin, int R, int row_len, int table_doubles, double *__restrict__ rows,
            double *__restrict__ rows_mid, FlowStore st)
{
    extern __shared__ double s_mem[];
    const int node = node_begin + blockIdx.y;
    double m = P.shock[node];
    if constexpr (LDSQ) {
        flow_stage_tables(P, s_mem, m, 64 * FLOW_WAVES);
        m = 1.0;   // the staged values are the node's own
        __syncthreads();
    }
    const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
    constexpr int SUB = FLOW_WAVES / CHUNKS;
    const int chunk = wave % CHUNKS, wave0 = wave - chunk;
    const int g = blockIdx.x * SUB + wave / CHUNKS;
    const size_t unit = (size_t)blockIdx.y * R + min(g, R - 1);
    const int shift = node * P.node_step;
    double *stage0 = s_mem + table_doubles;
    static_assert(FLOW_TR * 64 <= FLOW_STAGE, "transfers fit the stages");
    double (*s_tr)[FLOW_TR][64] = reinterpret_cast<double (*)[FLOW_TR][64]>(stage0);   // before the stages' use
    FlowRow row, mid;
    row.stage = stage0 + wave * FLOW_STAGE * (SET == FLOWS_ALL ? 2 : 1);
    row.dst = rows + unit * row_len;
    mid.stage = row.stage + FLOW_STAGE;
    mid.dst = rows_mid + unit * row_len;
    row.have = mid.have = 0;
    int done = 0, done_mid = 0;   // length of the row's longest tile so far
    for (int tile0 = st.tile_begin; tile0 < st.tile_end; tile0 += R) {
        const int tile = tile0 + g;
        const bool any = g < R && tile < st.tile_end;
        const int at = any ? tile : 0;
        const int smax = wave_uniform(P.tiles[at].smax) - shift;
        // Between a row's tiles: the stages are free again, and the next tile adds
        // to what the row's wavefronts wrote.
        if (tile0 > st.tile_begin) __syncthreads();
        if (!any || smax <= 0) {   // nothing to walk: only the two barriers
            __syncthreads();
            __syncthreads();
            continue;
        }
        const int kind = wave_uniform(P.tiles[at].kind), flow = wave_uniform(P.tiles[at].flow);
        int smin = wave_uniform(P.tiles[at].smin) - shift;
        FlowLane L;
        L.init(P, wave_uniform(P.tiles[at].first) + lane, shift);
        if (__ballot(!L.live)) smin = 0;
        const int len = (smax / FLOW_BLK + 1) * FLOW_BLK;
        const int per = ((len / FLOW_BLK + CHUNKS - 1) / CHUNKS) * FLOW_BLK;
        double *keep = nullptr;   // the lane's kept flows, month t at keep[64 t] (order: see FlowStore)
        if (st.flows) keep = st.flows + ((size_t)blockIdx.y * st.node_months + (P.tile_base[tile] - st.month_begin)) * 64 + (lane & 15) * 4 + (lane >> 4);
        flow_model<LDSQ, VEC, SET>(P, kind, flow, [&](auto tag) {
            typedef typename decltype(tag)::type W;
            typedef FlowTraits<W> X;
            constexpr bool cut = W::TR > 0;   // else one wavefront walks all of it
            const int t0 = !cut ? (chunk == 0 ? 0 : len) : min(chunk * per, len);
            const int t1 = !cut ? len : min(t0 + per, len);
            const bool lead = cut && t0 > 0;
            const int s0 = lead ? t0 - 1 : t0;   // first step walked
            W w;
            w.init(P, L, kind, shift, s0);
            if constexpr (cut) {
                double x[FLOW_TR];
                const int s1 = t1 > t0 && t1 < len ? t1 - 1 : s0;
                flow_transfer(P, s_mem, w, m, smax, s0, s1, x);
#pragma unroll
                for (int i = 0; i < W::TR; ++i) s_tr[wave][i][lane] = x[i];
                __syncthreads();
                for (int c = 0; c < chunk; ++c) {
#pragma unroll
                    for (int i = 0; i < W::TR; ++i) x[i] = s_tr[wave0 + c][i][lane];
                    w.advance(x);
                }
                w.past(s0);
            } else {
                __syncthreads();
            }
            __syncthreads();   // transfers read: the stages may be written
            row.have = done;
            mid.have = done_mid;
            if (t0 >= t1) return;
            if constexpr (X::markov) {
                // (FlowMarkov4's lanes stand in the order of the kept flows already)
                double *k = std::is_same<W, FlowMarkov4>::value && keep ? keep - (lane & 15) * 4 - (lane >> 4) + lane : keep;
                for (int t = t0; t < t1; t += FLOW_BLK) {
#pragma unroll 2
                    for (int u = 0; u < FLOW_BLK; ++u) {
                        const double f = w.step(t + u);
                        if (k) k[(size_t)(t + u) * 64] = f;
                        if (rows) row.put(t + u, f, lane);
                    }
                    if (rows) row.flush(t + FLOW_BLK, lane);
                }
            } else {
                flow_walk<FLOW_U>(
                    P, s_mem, w, m, smax, smin, t0, t1, lead,
                    [&](int t, double f) {
                        if (keep) keep[(size_t)t * 64] = f;
                        if (rows) row.put(t, f, lane);
                        if constexpr (X::frac) {
                            if (keep) keep[(size_t)t * 64 + st.mid] = w.mid;
                            if (rows) mid.put(t, w.mid, lane);
                        }
                    },
                    [&](int t) {
                        if ((t & (FLOW_BLK - 1)) || !rows) return;
                        row.flush(t, lane);
                        if constexpr (X::frac) mid.flush(t, lane);
                    });
            }
        });
        done = max(done, len);
        if (flow == FLOW_FRAC) done_mid = max(done_mid, len);
    }
    if (g >= R || chunk > 0 || !rows) return;
    for (int t = done + lane; t < row_len; t += 64) row.dst[t] = 0.0;
    if (SET == FLOWS_ALL && rows_mid != nullptr)
        for (int t = done_mid + lane; t < row_len; t += 64) mid.dst[t] = 0.0;
}

// out[node][chunk][t] = sum of the node's rows of the chunk, in a fixed order.
__global__ void __launch_bounds__(512) k_flow_reduce(const double *__restrict__ rows, int R, int row_len,
                                                     int chunk_rows, int n_chunks, double *__restrict__ out)
{
    __shared__ double sh[8][64];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int t = blockIdx.x * 64 + tx, node = blockIdx.y, chunk = blockIdx.z;
    const int r1 = min((chunk + 1) * chunk_rows, R);
    double acc = 0.0;
    if (t < row_len) {
        const double *p = rows + (size_t)node * R * row_len + t;
        for (int r = chunk * chunk_rows + ty; r < r1; r += 8) acc += p[(size_t)r * row_len];
    }
    sh[ty][tx] = acc;
    __syncthreads();
    if (ty == 0 && t < row_len) {
        double s = sh[0][tx];
#pragma unroll
        for (int i = 1; i < 8; ++i) s += sh[i][tx];
        out[((size_t)node * n_chunks + chunk) * row_len + t] = s;
    }
}

// Sum and product with their rounding error in the second part (error-free transformations of Knuth and Dekker).
struct Pair {
    double hi, lo;
};
__device__ __forceinline__ Pair exact_add(double a, double b)
{
#pragma clang fp contract(off)
    const double s = a + b, t = s - a;
    return {s, (a - (s - t)) + (b - t)};
}
__device__ __forceinline__ Pair exact_mul(double a, double b)
{
#pragma clang fp contract(off)
    const double p = a * b;
    return {p, __builtin_fma(a, b, -p)};
}
// x r + f to first order in the errors.
__device__ __forceinline__ Pair pair_step(Pair x, Pair r, Pair f)
{
    const Pair p = exact_mul(x.hi, r.hi), s = exact_add(p.hi, f.hi);
    return {s.hi, fma(x.hi, r.lo, fma(x.lo, r.hi, (p.lo + s.lo) + f.lo))};
}

// Totals of 64 scenarios of a node: R_t = F_t + vf_t M_t + v_t R_{t+1} from the
// last flow down to t = 0 (M: the flows within the month, discounted by
// vf = v^frac).  CH wavefronts take a time chunk each as the affine map
// R_lo = A R_hi + B (A the chunk's discount product), composed in order.  Reads
// every live curve value once: bound by that read at many nodes, by the chunk's
// serial chain at one.
//
// One chain carries the whole portfolio, so its rounding errors do not average
// out as those of the policies' own chains do (10,000 policies x 60 nodes:
// 1.0e-15 against 0.95e-15): the error of every operation is kept beside the
// value.
__global__ void __launch_bounds__(64 * FLOW_TOTALS_CHUNKS)
k_flow_totals(RecParams P, const double *__restrict__ sums, const double *__restrict__ sums_mid, int n_sums,
              int row_len, int max_term, int node_begin, double *__restrict__ totals)
{
    constexpr int CH = FLOW_TOTALS_CHUNKS;
    extern __shared__ double s_mem[];   // F[len + 1], then M[len + 1]
    __shared__ Pair sA[CH][64], sB[CH][64];
    const int node_rel = blockIdx.y, node = node_begin + node_rel;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int s = blockIdx.x * 64 + lane;
    const int len = max(max_term - node * P.node_step, 0);
    double *out = totals + (size_t)(node - P.node_begin) * P.scen_count;
    if (len == 0) {   // every policy has expired
        if (wave == 0 && s < P.scen_count) out[s] = 0.0;
        return;
    }
    double *F = s_mem, *M = s_mem + row_len;
    for (int t = threadIdx.x; t <= len; t += 64 * CH) {
        const double *p = sums + (size_t)node_rel * n_sums * row_len + t;
        double a = 0.0;
        for (int i = 0; i < n_sums; ++i) a += p[(size_t)i * row_len];
        F[t] = a;
        if (sums_mid) {
            const double *q = sums_mid + (size_t)node_rel * n_sums * row_len + t;
            double b = 0.0;
            for (int i = 0; i < n_sums; ++i) b += q[(size_t)i * row_len];
            M[t] = b;
        }
    }
    __syncthreads();
    const int per = (len + CH - 1) / CH;
    const int lo = wave * per, hi = min(lo + per, len);
    const size_t off = (size_t)node * P.n_steps * P.scen_pad + P.scen_begin + min(s, P.scen_count - 1);
    const double *v = P.v + off;
    Pair A{1.0, 0.0}, B{0.0, 0.0};
    auto step = [&](double x, Pair f) {
        const Pair q = exact_mul(A.hi, x);
        A = {q.hi, fma(A.lo, x, q.lo)};
        B = pair_step({x, 0.0}, B, f);
    };
    if (sums_mid) {
        const double *vf = P.vf + off;
        for (int t = hi - 1; t >= lo; --t)
            step(v[(size_t)t * P.scen_pad], pair_step({vf[(size_t)t * P.scen_pad], 0.0}, {M[t], 0.0}, {F[t], 0.0}));
    } else {
        constexpr int U = 16;   // curve values in flight
        int t = hi - 1;
        for (; t - lo >= U - 1; t -= U) {
            double x[U];
#pragma unroll
            for (int i = 0; i < U; ++i) x[i] = v[(size_t)(t - i) * P.scen_pad];
#pragma unroll
            for (int i = 0; i < U; ++i) step(x[i], {F[t - i], 0.0});
        }
        for (; t >= lo; --t) step(v[(size_t)t * P.scen_pad], {F[t], 0.0});
    }
    sA[wave][lane] = A;
    sB[wave][lane] = B;
    __syncthreads();
    if (wave == 0 && s < P.scen_count) {
        Pair R{F[len], 0.0};
#pragma unroll
        for (int w = CH - 1; w >= 0; --w) R = pair_step(sA[w][lane], R, sB[w][lane]);
        out[s] = isfinite(R.hi + R.lo) ? R.hi + R.lo : R.hi;   // (an overflow has no error term)
    }
}

// ---------------------------------------------------------------------------
// Sizes and launches
// ---------------------------------------------------------------------------
// Rows of a launch: one per tile, at most 48 MiB of them (past that a row takes
// several tiles; less where the scratch also holds the totals, at 8 bytes each).
// Sizes follow from the run alone, so every entry point adds in the same order.
constexpr size_t FLOW_ROW_BYTES = (size_t)48 << 20;
// Up to this many (node, tile) pairs a tile's months are cut in eight, past it
// in four (fewer transfers).  Totals on 16 scenarios, us, cut in eight / four: level
// books 5,000 policies (79 pairs) 34 / 43, 60,000 (938) 55 / 57, 64,000 (1,000) 58 /
// 57, 10,000 x 15 nodes (2,355) 74 / 69, x 60 137 / 105.  Above the line a single
// node would gain from eight a little longer (130,000, 2,031 pairs: 78 / 82; 200,000
// annuities with payment patterns, 3,125: 180 / 193); the flows' errors do not.
constexpr int FLOW_SPLIT_TILES = 1024;

FlowShape flow_shape(int node_count, int n_tiles, int max_term, bool has_mid, size_t own_totals)
{
    FlowShape f;
    f.row_len = (max_term / FLOW_BLK + 1) * FLOW_BLK;
    const size_t taken = std::min(own_totals * sizeof(double), (size_t)36 << 20);
    const size_t cap = (FLOW_ROW_BYTES - taken) / ((size_t)f.row_len * 8 * (has_mid ? 2 : 1));
    const int rows = (int)std::max<size_t>(1, std::min<size_t>(cap, 1 << 20));
    f.nodes = std::min({node_count, rows, 65535});
    const int most = rows / f.nodes;
    const int per = (n_tiles + most - 1) / most;   // tiles per row
    f.R = (n_tiles + per - 1) / per;
    f.chunks = (long long)node_count * n_tiles <= FLOW_SPLIT_TILES ? 8 : 4;
    f.chunk_rows = f.R > 16 * FLOW_RED ? (f.R + 15) / 16 : FLOW_RED;
    f.n_chunks = f.R <= 8 ? 0 : (f.R + f.chunk_rows - 1) / f.chunk_rows;
    const size_t rows_d = (size_t)f.nodes * f.R * f.row_len;
    const size_t sums_d = (size_t)f.nodes * f.n_chunks * f.row_len;
    f.scratch_doubles = (rows_d + sums_d) * (has_mid ? 2 : 1);
    return f;
}

// LDS of the sums kernel and of the totals kernel, in bytes.
static size_t sums_lds(const RecParams &p, int set)
{
    return ((p.q_in_lds ? (size_t)(p.n_q + 1) / 2 * 2 : 0) +
            (size_t)FLOW_WAVES * FLOW_STAGE * (set == FLOWS_ALL ? 2 : 1)) * sizeof(double);
}

bool flow_fits(const FlowShape &f, const RecParams &p, int set, bool has_mid, size_t lds_per_block)
{
    // 32 KiB of the totals kernel's LDS are its static part
    return sums_lds(p, set) <= lds_per_block &&
           (size_t)f.row_len * 8 * (has_mid ? 2 : 1) + (size_t)(32 << 10) <= lds_per_block;
}

template <bool LDSQ, int CHUNKS>
static void launch_sums(const RecParams &p, int R, int row_len, int set, int node_begin, int nodes,
                        double *rows, double *rows_mid, const FlowStore &st, hipStream_t s)
{
    constexpr int SUB = FLOW_WAVES / CHUNKS;   // rows per workgroup
    const dim3 g((R + SUB - 1) / SUB, nodes), b(64 * FLOW_WAVES);
    const size_t lds = sums_lds(p, set);
    const int td = p.q_in_lds ? (p.n_q + 1) / 2 * 2 : 0;
#define RR_SUMS(VEC, SET) \
    hipLaunchKernelGGL((k_flow_sums<LDSQ, VEC, SET, CHUNKS>), g, b, lds, s, p, node_begin, R, row_len, td, rows, \
                       rows_mid, st)
    if (set == FLOWS_ALL) RR_SUMS(true, FLOWS_ALL);
    else if (set == FLOWS_PATTERN) RR_SUMS(true, FLOWS_PATTERN);
    else if (p.has_vector) RR_SUMS(true, FLOWS_LEVEL);
    else RR_SUMS(false, FLOWS_LEVEL);
#undef RR_SUMS
}

// The walk over the tiles of st (all of them for rows) at `nodes` nodes.
static void launch_flow_walk(const RecParams &p, const FlowShape &f, int set, int node_begin, int nodes, double *rows,
                             double *rows_mid, const FlowStore &st, hipStream_t s)
{
    const int R = rows ? f.R : st.tile_end - st.tile_begin;
    auto launch = [&](auto ldsq) {
        constexpr bool L = decltype(ldsq)::value;
        if (f.chunks == 8) launch_sums<L, 8>(p, R, f.row_len, set, node_begin, nodes, rows, rows_mid, st, s);
        else launch_sums<L, 4>(p, R, f.row_len, set, node_begin, nodes, rows, rows_mid, st, s);
    };
    if (p.q_in_lds) launch(std::true_type{});
    else launch(std::false_type{});
}

hipError_t launch_flow_store(const RecParams &p, const FlowShape &f, int set, bool has_mid, int node_begin, int nodes,
                             const FlowStore &st, double *totals_scratch, hipStream_t s)
{
    double *rows = totals_scratch, *mid = nullptr;
    if (rows && has_mid) mid = rows + (size_t)f.nodes * (f.R + f.n_chunks) * f.row_len;
    launch_flow_walk(p, f, set, node_begin, nodes, rows, mid, st, s);
    return hipGetLastError();
}

hipError_t launch_flow_totals(const RecParams &p, int node_count, const FlowShape &f, int set, bool has_mid, bool kept,
                              int max_term, double *scratch, double *totals, hipStream_t s)
{
    const FlowStore none{nullptr, 0, 0, 0, 0, p.n_tiles};
    const size_t rows_d = (size_t)f.nodes * f.R * f.row_len;
    const size_t sums_d = (size_t)f.nodes * f.n_chunks * f.row_len;
    double *rows = scratch, *sums = rows + rows_d;
    double *rows_mid = has_mid ? sums + sums_d : nullptr;
    double *sums_mid = has_mid ? rows_mid + rows_d : nullptr;
    for (int k = 0; k < node_count; k += f.nodes) {
        const int nodes = node_count - k < f.nodes ? node_count - k : f.nodes;
        const int nb = p.node_begin + k;
        if (!kept) launch_flow_walk(p, f, set, nb, nodes, rows, rows_mid, none, s);
        const double *src = rows, *src_mid = rows_mid;
        int n_sums = f.R;
        if (f.n_chunks > 0) {
            const dim3 g((f.row_len + 63) / 64, nodes, f.n_chunks);
            hipLaunchKernelGGL(k_flow_reduce, g, dim3(512), 0, s, rows, f.R, f.row_len, f.chunk_rows, f.n_chunks, sums);
            if (has_mid)
                hipLaunchKernelGGL(k_flow_reduce, g, dim3(512), 0, s, rows_mid, f.R, f.row_len, f.chunk_rows, f.n_chunks, sums_mid);
            src = sums;
            src_mid = sums_mid;
            n_sums = f.n_chunks;
        }
        const dim3 g((p.scen_count + 63) / 64, nodes);
        const size_t lds = (size_t)f.row_len * sizeof(double) * (has_mid ? 2 : 1);
        hipLaunchKernelGGL(k_flow_totals, g, dim3(64 * FLOW_TOTALS_CHUNKS), lds, s, p, src, src_mid, n_sums, f.row_len, max_term,
                           nb, totals);
    }
    return hipGetLastError();
}

}  // namespace rr
