// Interest scenarios generated on the device (the interest model of Sec. 3.4
// and 3.7.2, here the Vasicek short rate): a counter-based generator, normals
// by the Box-Muller transform, and the exact joint-Gaussian step of the short
// rate and its integral over a step.
//
// The random numbers of (node k, scenario s, step t) are the Philox4x64-10
// block of the counter (t, s, k, 0) under the caller's key, so every value
// is computed independently: the normals of all steps in parallel, then the
// short-rate chain (a first-order linear recurrence in t, cut in time chunks)
// with the discount factors and their products.
#include "rr_internal.h"

#include <algorithm>
#include <cfloat>

namespace rr {

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC 2011): per round the words 0
// and 2 are multiplied by the round multipliers; the high halves are xored
// with the other two words and the key, the low halves become words 1 and 3;
// the key is bumped by the Weyl increments between rounds.
__device__ __forceinline__ void philox4x64_10(unsigned long long &c0, unsigned long long &c1,
                                              unsigned long long &c2, unsigned long long &c3,
                                              unsigned long long k0, unsigned long long k1)
{
    constexpr unsigned long long M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    constexpr unsigned long long W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const unsigned long long hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        const unsigned long long hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        const unsigned long long n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += W0;
        k1 += W1;
    }
}

__device__ __forceinline__ double u01(unsigned long long x)
{
    return ((double)(x >> 11) + 0.5) * (1.0 / 9007199254740992.0);
}

// Normals of every (node, step, scenario), stored month-major like the
// curves: z[(k * n_steps + t) * scen_pad + s].
__global__ void __launch_bounds__(256) k_vas_normals(VasParams P, double *__restrict__ z0,
                                                     double *__restrict__ z1)
{
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)P.n_nodes * P.n_steps * P.n_scen;
    if (id >= total) return;
    const int s = (int)(id % P.n_scen);
    const long long kt = id / P.n_scen;
    const int t = (int)(kt % P.n_steps);
    const int k = (int)(kt / P.n_steps);
    unsigned long long c0 = (unsigned long long)t, c1 = (unsigned long long)s,
                       c2 = (unsigned long long)k, c3 = 0;
    philox4x64_10(c0, c1, c2, c3, P.key0, P.key1);
    const double rad = sqrt(-2.0 * log(u01(c0)));
    double sn, cs;
    sincos(6.283185307179586476925286766559 * u01(c1), &sn, &cs);
    const size_t o = (size_t)kt * P.scen_pad + s;
    z0[o] = rad * cs;
    z1[o] = rad * sn;
}

// The integral of the short rate over a step that starts x above b.  One form of
// it, so that every kernel rounds alike.
__device__ __forceinline__ double vas_integral(const VasParams &P, double x, double z0, double z1)
{
    return fma(P.sd_y_perp, z1, fma(P.rho_sd_y, z0, fma(x, P.om, P.b * P.dt)));
}

// Short rates, discount factors and (D) discount products of every (node,
// scenario) in one pass over the normals.  r_t - b is a first-order linear
// recurrence, so a workgroup cuts the months of eight scenarios
// in 64 chunks of up to 16: a thread holds its chunk's normals in registers, runs
// the chunk from 0, takes its true start from the ends of the chunks before it
// (all of one length) through LDS, and runs it again for the rates and
// v = exp(-Y), Y the integral of the short rate over the step given r_t and the
// two normals.  The products of v go through LDS the same way.  Months past
// 1,024 months follow as further segments from where the last one ended.
//
// month_major: v[(k * n_steps + t) * ld + s] (the library's curve layout,
// padding scenarios set to 1), else v[(k * n_scen + s) * n_steps + t].  r (or
// null): r[(k * (n_steps + 1) + t) * scen_pad + s], t = 0 .. n_steps.  D (or
// null; month-major): D[(k * disc_rows + t) * scen_pad + s], zeros past t = n_steps;
// products beyond the FP64 range are its largest value, so that a policy whose
// flows are over by then still adds 0 x D = 0.
//
// Bound by latency at the usual sizes (a thread's loads go out together) and by
// the 32 bytes a value that it moves at many curves.  It takes the place of a
// chain a thread (600 dependent steps on 16 wavefronts), a pass for the factors
// and one for the products: 1,000 scenarios x 600 months drawn and valued for
// 10,000 policies 0.244 -> 0.196 ms.  Eight scenarios a workgroup: sixteen
// leave half of the CUs idle there and spill registers.  Instances by the months
// a thread holds: with sixteen always, chunks of one month fetched each value
// sixteen times (20,000 scenarios x 120 months: scan 94 -> 29 us).
constexpr int SCAN_S = 8, SCAN_C = 64, SCAN_LEN = 16;

// Eight scenarios are half a cache line, and consecutive blocks go to the eight
// XCDs in turn: blocks b and b + 8 take neighbours, so that one L2 sees whole
// lines (20 nodes x 500 scenarios x 600 months: scan 75 -> 65 us).
__device__ __forceinline__ int scan_block(int b, int n)
{
    const int i = b % 16;
    return b - i + 16 <= n ? b - i + (i % 8) * 2 + i / 8 : b;
}

// step(x, value) over the first c rows of a column of LDS, eight reads at a time.
template <class Step>
__device__ __forceinline__ double fold_rows(double x, const double (*rows)[SCAN_S], int lane, int c, Step step)
{
    int w = 0;
    for (; w + 8 <= c; w += 8) {
        double y[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) y[i] = rows[w + i][lane];
#pragma unroll
        for (int i = 0; i < 8; ++i) x = step(x, y[i]);
    }
    for (; w < c; ++w) x = step(x, rows[w][lane]);
    return x;
}

// LEN: months a thread holds, at least those of a chunk.
template <int LEN>
__global__ void __launch_bounds__(SCAN_S * SCAN_C)
k_vas_scan(VasParams P, int node0, const double *__restrict__ r0, const double *__restrict__ z0,
           const double *__restrict__ z1, double *__restrict__ r, double *__restrict__ v, int month_major,
           double *__restrict__ D)
{
    __shared__ double s_end[SCAN_C][SCAN_S], s_prod[SCAN_C][SCAN_S], s_dev[SCAN_S], s_disc[SCAN_S];
    const int lane = threadIdx.x % SCAN_S, c = threadIdx.x / SCAN_S, k = node0 + blockIdx.y;
    const int n_sb = P.scen_pad / SCAN_S, n = P.n_steps;
    const size_t row = P.scen_pad;
    for (int b = blockIdx.x; b < n_sb; b += gridDim.x) {
        const int s = scan_block(b, n_sb) * SCAN_S + lane;
        const bool real = s < P.n_scen;
        const double *zk0 = z0 + (size_t)k * n * row + s, *zk1 = z1 + (size_t)k * n * row + s;
        double dev0 = r0[k] - P.b, disc0 = 1.0;   // at the segment's start
        if (c == 0) {
            if (D) D[(size_t)k * disc_rows(n) * row + s] = 1.0;
            if (r && real) r[(size_t)k * (n + 1) * row + s] = r0[k];
        }
        for (int seg = 0; seg < n; seg += SCAN_C * SCAN_LEN) {
            const int per = min(SCAN_LEN, (n - seg + SCAN_C - 1) / SCAN_C);
            // Every thread walks `per` months (a month past the end repeats the last
            // one's normals, and stores nothing): only whole chunks are followed
            // by others, so what a cut one ends with is not read.
            const int t0 = seg + c * per;
            double za[LEN], zb[LEN];
#pragma unroll
            for (int i = 0; i < LEN; ++i) {
                const size_t o = (size_t)min(t0 + min(i, per - 1), n - 1) * row;
                za[i] = zk0[o];
                zb[i] = zk1[o];
            }
            double x = 0.0, e = 1.0;
#pragma unroll
            for (int i = 0; i < LEN; ++i) {
                if (i >= per) continue;
                x = fma(x, P.e, P.sd_r * za[i]);
                e *= P.e;
            }
            s_end[c][lane] = x;
            __syncthreads();
            x = fold_rows(dev0, s_end, lane, c, [&](double y, double end) { return fma(y, e, end); });
            double p = 1.0;
#pragma unroll
            for (int i = 0; i < LEN; ++i) {
                if (i >= per) continue;
                const double y = vas_integral(P, x, za[i], zb[i]);
                x = fma(x, P.e, P.sd_r * za[i]);
                za[i] = real ? exp(-y) : 1.0;
                p *= za[i];
                const int t = t0 + i;
                if (t >= n) continue;
                if (month_major) v[((size_t)k * n + t) * row + s] = za[i];
                else if (real) v[((size_t)k * P.n_scen + s) * n + t] = za[i];
                if (r && real) r[((size_t)k * (n + 1) + t + 1) * row + s] = P.b + x;
            }
            s_prod[c][lane] = p;
            if (c == SCAN_C - 1) s_dev[lane] = x;
            __syncthreads();
            dev0 = s_dev[lane];
            if (D) {
                double d = fold_rows(disc0, s_prod, lane, c, [](double y, double prod) { return y * prod; });
                double *Dk = D + (size_t)k * disc_rows(n) * row + s;
#pragma unroll
                for (int i = 0; i < LEN; ++i) {
                    if (i >= per) continue;
                    d *= za[i];
                    if (t0 + i < n) Dk[(size_t)(t0 + i + 1) * row] = fmin(d, DBL_MAX);
                }
                if (c == SCAN_C - 1) s_disc[lane] = d;
            }
            __syncthreads();   // the next segment writes what this one's threads read
            disc0 = s_disc[lane];
        }
        if (D)   // rows that whole blocks of months reach
            for (int t = n + 1 + c; t < disc_rows(n); t += SCAN_C)
                D[((size_t)k * disc_rows(n) + t) * row + s] = 0.0;
    }
}

// The same, a (node, scenario) a thread, with the scan's chunks and so its bits (a
// scenario does not depend on how many are drawn): beside the true chain runs the
// chunk's own from 0, which gives the next chunk its start.  For many curves: the
// accesses are whole rows of 64 scenarios instead of the scan's eight, and the 64
// chunks of a short run are not folded one by one.  Bound by the 32 bytes a value.
constexpr int CHAIN_U = 16;   // months loaded ahead

__global__ void __launch_bounds__(64)
k_vas_chain(VasParams P, int node0, const double *__restrict__ r0, const double *__restrict__ z0,
            const double *__restrict__ z1, double *__restrict__ r, double *__restrict__ v, int month_major,
            double *__restrict__ D)
{
    const int s = blockIdx.x * 64 + threadIdx.x, k = node0 + blockIdx.y, n = P.n_steps;
    if (s >= (month_major ? P.scen_pad : P.n_scen)) return;
    const bool real = s < P.n_scen;
    const size_t row = P.scen_pad;
    const double *zk0 = z0 + (size_t)k * n * row + s, *zk1 = z1 + (size_t)k * n * row + s;
    double *rk = r && real ? r + (size_t)k * (n + 1) * row + s : nullptr;
    double *Dk = D ? D + (size_t)k * disc_rows(n) * row + s : nullptr;
    if (Dk) Dk[0] = 1.0;
    if (rk) rk[0] = r0[k];
    double x = r0[k] - P.b, d = 1.0;              // the true chain
    double x_start = 0.0, d_start = 0.0, x_own = 0.0, d_own = 1.0, e = 1.0;   // the chunk's start, its own chain from it
    int seg = 0, per = 0, left = 0;               // start of the next segment, months a chunk, months to the chunk's end
    double za[CHAIN_U], zb[CHAIN_U];
#pragma unroll
    for (int i = 0; i < CHAIN_U; ++i) {
        za[i] = zk0[(size_t)min(i, n - 1) * row];
        zb[i] = zk1[(size_t)min(i, n - 1) * row];
    }
    for (int t0 = 0; t0 < n; t0 += CHAIN_U) {
        double na[CHAIN_U], nb[CHAIN_U];
#pragma unroll
        for (int i = 0; i < CHAIN_U; ++i) {
            const size_t o = (size_t)min(t0 + CHAIN_U + i, n - 1) * row;
            na[i] = zk0[o];
            nb[i] = zk1[o];
        }
#pragma unroll
        for (int i = 0; i < CHAIN_U; ++i) {
            const int t = t0 + i;
            if (t >= n) continue;
            if (t == seg) {
                per = min(SCAN_LEN, (n - seg + SCAN_C - 1) / SCAN_C);
                e = 1.0;
                for (int j = 0; j < per; ++j) e *= P.e;
                x_start = x;
                d_start = d;
                left = per;
                seg += SCAN_C * SCAN_LEN;
            }
            const double y = vas_integral(P, x, za[i], zb[i]);
            const double step = P.sd_r * za[i];
            x = fma(x, P.e, step);
            x_own = fma(x_own, P.e, step);
            const double f = real ? exp(-y) : 1.0;
            d *= f;
            d_own *= f;
            if (month_major) v[((size_t)k * n + t) * row + s] = f;
            else v[((size_t)k * P.n_scen + s) * n + t] = f;
            if (rk) rk[(size_t)(t + 1) * row] = P.b + x;
            if (Dk) Dk[(size_t)(t + 1) * row] = fmin(d, DBL_MAX);
            if (--left == 0) {
                x_start = fma(x_start, e, x_own);
                d_start *= d_own;
                if (t + 1 < seg) {   // (a segment starts from the chain itself)
                    x = x_start;
                    d = d_start;
                }
                x_own = 0.0;
                d_own = 1.0;
                left = per;
            }
        }
#pragma unroll
        for (int i = 0; i < CHAIN_U; ++i) {
            za[i] = na[i];
            zb[i] = nb[i];
        }
    }
    if (Dk)
        for (int t = n + 1; t < disc_rows(n); ++t) Dk[(size_t)t * row] = 0.0;
}

// Short rates in the caller's layout r_out[(k * n_scen + s) * (n_steps + 1) + t].
__global__ void __launch_bounds__(256) k_vas_rates_out(VasParams P, const double *__restrict__ r,
                                                       double *__restrict__ r_out)
{
    const long long id = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)P.n_nodes * (P.n_steps + 1) * P.n_scen;
    if (id >= total) return;
    const int s = (int)(id % P.n_scen);
    const long long kt = id / P.n_scen;
    const int t = (int)(kt % (P.n_steps + 1));
    const int k = (int)(kt / (P.n_steps + 1));
    r_out[((size_t)k * P.n_scen + s) * (P.n_steps + 1) + t] = r[(size_t)kt * P.scen_pad + s];
}

// Whether a generation of so many wavefronts of 64 scenarios goes by
// k_vas_chain.  Generation in place by the scan / by chains, us: 50 nodes x 500
// scenarios x 600 months (450 wavefronts) 364 / 351, 100 x 500 x 600 697 / 641,
// 32,000 x 120 (500) 101 / 96, but 40 x 500 x 240 (360) 113 / 132; with chunks of
// one month already 24,000 x 60 (376) 56 / 50, while 8,000 x 60 (126) 24 / 31.
static bool by_chains(long long waves, int n_steps)
{
    return waves >= (n_steps <= SCAN_C ? 256 : 440);
}

static unsigned blocks_of(long long n) { return (unsigned)((n + 255) / 256); }

hipError_t launch_vasicek(const VasParams &P, const double *r0, double *work, double *v,
                          int month_major, double *r_out, double *D, hipStream_t stream)
{
    if (P.n_nodes <= 0 || P.n_scen <= 0 || P.n_steps <= 0) return hipSuccess;
    const size_t zn = (size_t)P.n_nodes * P.n_steps * P.scen_pad;
    double *z0 = work, *z1 = work + zn, *r = r_out ? work + 2 * zn : nullptr;
    hipLaunchKernelGGL(k_vas_normals, dim3(blocks_of((long long)P.n_nodes * P.n_steps * P.n_scen)),
                       dim3(256), 0, stream, P, z0, z1);
    const int waves = (P.scen_pad + 63) / 64;
    const int per = std::min((P.n_steps + SCAN_C - 1) / SCAN_C, SCAN_LEN);   // months a chunk
    for (int k = 0; k < P.n_nodes; k += 32768) {
        const int nodes = std::min(P.n_nodes - k, 32768);
        auto launch = [&](auto kernel, int blocks, int threads) {
            hipLaunchKernelGGL(kernel, dim3(blocks, nodes), dim3(threads), 0, stream, P, k, r0, z0, z1, r, v, month_major, D);
        };
        if (by_chains((long long)waves * P.n_nodes, P.n_steps)) {
            launch(k_vas_chain, waves, 64);
        } else {
            const int blocks = std::min(P.scen_pad / SCAN_S, 1 << 16), threads = SCAN_S * SCAN_C;
            if (per <= 2) launch(k_vas_scan<2>, blocks, threads);
            else if (per <= 4) launch(k_vas_scan<4>, blocks, threads);
            else if (per <= 8) launch(k_vas_scan<8>, blocks, threads);
            else launch(k_vas_scan<SCAN_LEN>, blocks, threads);
        }
    }
    if (r_out)
        hipLaunchKernelGGL(k_vas_rates_out,
                           dim3(blocks_of((long long)P.n_nodes * (P.n_steps + 1) * P.n_scen)),
                           dim3(256), 0, stream, P, r, r_out);
    return hipGetLastError();
}

size_t vasicek_work_doubles(int n_nodes, int n_steps, int scen_pad, bool rates)
{
    return (size_t)n_nodes * scen_pad * (2 * (size_t)n_steps + (rates ? n_steps + 1 : 0));
}

}  // namespace rr
