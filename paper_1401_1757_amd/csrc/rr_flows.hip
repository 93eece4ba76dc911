// Portfolio totals by summed cash flows: a node's expected cash flows added up
// over the policies (once for all scenarios), then the backward recurrence
// R_t = F_t + v_t R_{t+1} of that one sequence per scenario.
#include "rr_flows.h"

namespace rr {

constexpr int FLOW_U = 8;                  // steps per block of a walk
constexpr int FLOW_WAVES = 8;              // wavefronts per workgroup
constexpr int FLOW_ROW = 65;               // stage rows: 65 doubles apart, 8 columns per lane on distinct banks
constexpr int FLOW_STAGE = FLOW_U * FLOW_ROW;
constexpr int FLOW_RED = 64;               // rows per workgroup of the row reduction

// Sums over the policies of the tiles g, g + R, ... of a node, one row of
// row_len doubles per wavefront (unit = node * R + g).  A block of eight steps
// passes through the wavefront's LDS stage: lane l adds eight lanes' flows of
// step l % 8, three exchanges add the eight parts, in a fixed order.  A later
// tile of the wavefront adds to the row it wrote before.
//
// Bound by vector issue and LDS: per policy-month one or two table reads, one
// stage write and read and about ten FP64 operations.
template <bool LDSQ, bool VEC, bool SPECIAL>
__global__ void __launch_bounds__(64 * FLOW_WAVES, 2)
k_flow_sums(RecParams P, int node_begin, int node_count, int R, int row_len, int table_doubles,
            double *__restrict__ rows, double *__restrict__ rows_mid)
{
    extern __shared__ double s_mem[];
    if constexpr (LDSQ) {
        for (int i = threadIdx.x; i < P.n_q; i += 64 * FLOW_WAVES) s_mem[i] = P.q[i];
        __syncthreads();
    }
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int unit = wave_uniform(blockIdx.x * FLOW_WAVES + wave);
    if (unit >= node_count * R) return;
    double *stage = s_mem + table_doubles + wave * FLOW_STAGE * (SPECIAL ? 2 : 1);
    double *stage_mid = stage + FLOW_STAGE;
    const int node = node_begin + unit / R, g = unit % R;
    const int shift = node * P.node_step;
    const double m = P.shock[node];
    double *row = rows + (size_t)unit * row_len;
    double *row_mid = SPECIAL && rows_mid ? rows_mid + (size_t)unit * row_len : nullptr;
    int have = 0, have_mid = 0;   // length written so far
    const int u = lane & 7, j = lane >> 3;
    auto flush = [&](const double *st, double *dst, int t, int got) {
        __builtin_amdgcn_wave_barrier();
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < 8; ++i) s += st[u * FLOW_ROW + j * 8 + i];
        s += __shfl_xor(s, 8);
        s += __shfl_xor(s, 16);
        s += __shfl_xor(s, 32);
        if (lane < FLOW_U) dst[t + lane] = t < got ? dst[t + lane] + s : s;
        __builtin_amdgcn_wave_barrier();
    };
    for (int tile = g; tile < P.n_tiles; tile += R) {
        Tile T = P.tiles[tile];
        T.kind = wave_uniform(T.kind);
        T.first = wave_uniform(T.first);
        T.smax = wave_uniform(T.smax);
        T.smin = wave_uniform(T.smin);
        T.flow = wave_uniform(T.flow);
        const int smax = T.smax - shift;
        if (smax <= 0) continue;
        const bool mid = SPECIAL && row_mid != nullptr && T.flow == FLOW_FRAC;
        flow_tile<FLOW_U, LDSQ, VEC, SPECIAL>(
            P, s_mem, T, shift, m, lane, [&](int k, double x) { stage[k * FLOW_ROW + lane] = x; },
            [&](int k, double x) { if (SPECIAL) stage_mid[k * FLOW_ROW + lane] = x; },
            [&](int t) {
                flush(stage, row, t, have);
                if (mid) flush(stage_mid, row_mid, t, have_mid);
            });
        const int len = (smax / FLOW_U + 1) * FLOW_U;
        have = max(have, len);
        if (mid) have_mid = max(have_mid, len);
    }
    for (int t = have + lane; t < row_len; t += 64) row[t] = 0.0;
    if (row_mid)
        for (int t = have_mid + lane; t < row_len; t += 64) row_mid[t] = 0.0;
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

// Totals of 64 scenarios of a node: R_t = F_t + vf_t M_t + v_t R_{t+1} from the
// last flow down to t = 0 (M: the flows within the month, discounted by
// vf = v^frac).  CH wavefronts take a time chunk each as the affine map
// R_lo = A R_hi + B (A the chunk's discount product), composed in order; CH = 1
// is the plain recurrence, for curves whose products could leave the FP64
// range.  Reads every live curve value once: bound by that read at many nodes,
// by the chunk's serial chain at one.
template <int CH>
__global__ void __launch_bounds__(64 * CH)
k_flow_totals(RecParams P, const double *__restrict__ sums, const double *__restrict__ sums_mid, int n_sums,
              int row_len, int max_term, int node_begin, double *__restrict__ totals)
{
    extern __shared__ double s_mem[];   // F[len + 1], then M[len + 1]
    __shared__ double sA[CH][64], sB[CH][64];
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
    const int step = (len + CH - 1) / CH;
    const int lo = wave * step, hi = min(lo + step, len);
    const size_t off = (size_t)node * P.n_steps * P.scen_pad + P.scen_begin + min(s, P.scen_count - 1);
    const double *v = P.v + off;
    double A = 1.0, B = CH == 1 ? F[len] : 0.0;
    if (sums_mid) {
        const double *vf = P.vf + off;
        for (int t = hi - 1; t >= lo; --t) {
            const double x = v[(size_t)t * P.scen_pad];
            B = fma(x, B, fma(vf[(size_t)t * P.scen_pad], M[t], F[t]));
            A *= x;
        }
    } else {
        constexpr int U = 16;   // curve values in flight
        int t = hi - 1;
        for (; t - lo >= U - 1; t -= U) {
            double x[U];
#pragma unroll
            for (int i = 0; i < U; ++i) x[i] = v[(size_t)(t - i) * P.scen_pad];
#pragma unroll
            for (int i = 0; i < U; ++i) {
                B = fma(x[i], B, F[t - i]);
                A *= x[i];
            }
        }
        for (; t >= lo; --t) {
            const double x = v[(size_t)t * P.scen_pad];
            B = fma(x, B, F[t]);
            A *= x;
        }
    }
    if constexpr (CH == 1) {
        if (s < P.scen_count) out[s] = B;
        return;
    }
    sA[wave][lane] = A;
    sB[wave][lane] = B;
    __syncthreads();
    if (wave == 0 && s < P.scen_count) {
        double R = F[len];
#pragma unroll
        for (int w = CH - 1; w >= 0; --w) R = fma(sA[w][lane], R, sB[w][lane]);
        out[s] = R;
    }
}

// ---------------------------------------------------------------------------
// Sizes and launches
// ---------------------------------------------------------------------------
// Rows of a launch: enough wavefronts for four per SIMD, and at most 24 MiB of
// rows whatever the portfolio's size (a wavefront then takes several tiles).
// Sizes follow from the run alone, so every entry point adds in the same order.
constexpr int FLOW_MAX_ROWS = 4096;
constexpr size_t FLOW_ROW_BYTES = (size_t)24 << 20;

FlowShape flow_shape(int node_count, int n_tiles, int max_term, bool has_mid)
{
    FlowShape f;
    f.row_len = (max_term / FLOW_U + 1) * FLOW_U;
    const size_t cap = FLOW_ROW_BYTES / ((size_t)f.row_len * 8 * (has_mid ? 2 : 1));
    const int rows = (int)(cap < (size_t)FLOW_MAX_ROWS ? cap : (size_t)FLOW_MAX_ROWS);
    f.nodes = node_count < rows ? node_count : (rows > 0 ? rows : 1);
    const int most = rows / f.nodes > 0 ? rows / f.nodes : 1;
    const int per = (n_tiles + most - 1) / most;   // tiles per wavefront
    f.R = (n_tiles + per - 1) / per;
    f.chunk_rows = f.R > 16 * FLOW_RED ? (f.R + 15) / 16 : FLOW_RED;
    f.n_chunks = f.R <= 8 ? 0 : (f.R + f.chunk_rows - 1) / f.chunk_rows;
    const size_t rows_d = (size_t)f.nodes * f.R * f.row_len;
    const size_t sums_d = (size_t)f.nodes * f.n_chunks * f.row_len;
    f.scratch_doubles = (rows_d + sums_d) * (has_mid ? 2 : 1);
    return f;
}

// LDS of the sums kernel and of the totals kernel, in bytes.
static size_t sums_lds(const RecParams &p, bool special)
{
    return ((p.q_in_lds ? (size_t)(p.n_q + 1) / 2 * 2 : 0) +
            (size_t)FLOW_WAVES * FLOW_STAGE * (special ? 2 : 1)) * sizeof(double);
}

bool flow_fits(const FlowShape &f, const RecParams &p, bool special, bool has_mid, size_t lds_per_block)
{
    // 16 KiB of the totals kernel's LDS is its static part
    return sums_lds(p, special) <= lds_per_block &&
           (size_t)f.row_len * 8 * (has_mid ? 2 : 1) + (size_t)(16 << 10) <= lds_per_block;
}

template <bool LDSQ>
static void launch_sums(const RecParams &p, const FlowShape &f, bool special, int node_begin, int nodes,
                        double *rows, double *rows_mid, hipStream_t s)
{
    const dim3 g((nodes * f.R + FLOW_WAVES - 1) / FLOW_WAVES), b(64 * FLOW_WAVES);
    const size_t lds = sums_lds(p, special);
    const int td = p.q_in_lds ? (p.n_q + 1) / 2 * 2 : 0;
    if (special)
        hipLaunchKernelGGL((k_flow_sums<LDSQ, true, true>), g, b, lds, s, p, node_begin, nodes, f.R, f.row_len, td, rows, rows_mid);
    else if (p.has_vector)
        hipLaunchKernelGGL((k_flow_sums<LDSQ, true, false>), g, b, lds, s, p, node_begin, nodes, f.R, f.row_len, td, rows, rows_mid);
    else
        hipLaunchKernelGGL((k_flow_sums<LDSQ, false, false>), g, b, lds, s, p, node_begin, nodes, f.R, f.row_len, td, rows, rows_mid);
}

hipError_t launch_flow_totals(const RecParams &p, int node_count, const FlowShape &f, bool special, bool has_mid,
                              bool safe_curves, int max_term, double *scratch, double *totals, hipStream_t s)
{
    const size_t rows_d = (size_t)f.nodes * f.R * f.row_len;
    const size_t sums_d = (size_t)f.nodes * f.n_chunks * f.row_len;
    double *rows = scratch, *sums = rows + rows_d;
    double *rows_mid = has_mid ? sums + sums_d : nullptr;
    double *sums_mid = has_mid ? rows_mid + rows_d : nullptr;
    for (int k = 0; k < node_count; k += f.nodes) {
        const int nodes = node_count - k < f.nodes ? node_count - k : f.nodes;
        const int nb = p.node_begin + k;
        if (p.q_in_lds) launch_sums<true>(p, f, special, nb, nodes, rows, rows_mid, s);
        else launch_sums<false>(p, f, special, nb, nodes, rows, rows_mid, s);
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
        if (safe_curves)
            hipLaunchKernelGGL(k_flow_totals<16>, g, dim3(64 * 16), lds, s, p, src, src_mid, n_sums, f.row_len, max_term, nb, totals);
        else
            hipLaunchKernelGGL(k_flow_totals<1>, g, dim3(64), lds, s, p, src, src_mid, n_sums, f.row_len, max_term, nb, totals);
    }
    return hipGetLastError();
}

}  // namespace rr
