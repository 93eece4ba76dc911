// Expected cash flows of the policies, walked forward in time (device
// templates, FP64).
//
// The reserve of Eq. (3.1) is linear in the discount products D_t = v_0 ...
// v_{t-1} (Eq. (3.5)): r_0 = sum_t f_t D_t, where f_t is the cash flow expected
// at time t.  f_t comes from the forward recurrence of the state occupancy
// (a row vector times W_t per step), the adjoint of the backward recurrence:
// the same products of survival probabilities, taken once per policy instead
// of once per policy and scenario.  What then remains per scenario is one
// multiply-add per month, and nothing per policy where only totals are asked
// for (the flows add up over the policies first).
//
// A walker holds one policy per lane.  load(t) fetches what step t needs
// (issued ahead of its use), step(t, ..) returns f_t and advances the lane
// through step t.  Steps are taken in increasing t; a lane past its term has
// flow 0.  MASK = false is the form for steps that every lane of the tile
// takes (t < the tile's smallest remaining term, no expired or padding lane).
#pragma once

#include "rr_recurrence.h"

namespace rr {

// The table values of one step; unused members cost nothing after inlining.
struct FlowIn {
    double x1, x2, x3;   // one-step survival probabilities of the lives
    double cv;           // table tiles: cash flow of the step
};

template <bool LDSQ>
__device__ __forceinline__ double flow_q(const RecParams &P, const double *__restrict__ lq, int idx)
{
    return qload<LDSQ>(lq, P.q, idx);
}

// The node's mortality shock on a survival probability (m != 1).
__device__ __forceinline__ double shocked(double p, double m) { return 1.0 - fmin(1.0, m * (1.0 - p)); }

// Stage the survival tables in LDS with the node's shock applied (n threads;
// the caller synchronises): per-step loads then need no shock.
__device__ __forceinline__ void flow_stage_tables(const RecParams &P, double *dst, double m, int n)
{
    constexpr int B = 4;
    for (int base = threadIdx.x; base < P.n_q; base += B * n) {
        double x[B];
#pragma unroll
        for (int i = 0; i < B; ++i) x[i] = P.q[min(base + i * n, P.n_q - 1)];
#pragma unroll
        for (int i = 0; i < B; ++i)
            if (base + i * n < P.n_q) dst[base + i * n] = m == 1.0 ? x[i] : shocked(x[i], m);
    }
}

// Payment factor F(T) of a pattern tile (PatLane in rr_recurrence.h), walked
// forward: the position in the policy year counts up, and the level follows by
// one multiplication by 1 + e at each anniversary passed.
struct PatWalk {
    double g, lev;
    int pos, n, annual;   // months since the last anniversary (0 at one), anniversaries so far

    __device__ __forceinline__ void init(const RecParams &P, int slot, int shift, int t0)
    {
        const int code = P.pat_code[slot];
        g = P.pat_g[slot];
        annual = code & PAT_ANNUAL;
        const unsigned w = (unsigned)(shift + ((code & PAT_ARREARS) ? 1 : 0) + t0 + 12 - (code & 255));
        n = (int)(w / 12u);
        pos = (int)(w % 12u);
        double l = 1.0, x = g;
        for (int k = n; k > 0; k >>= 1) {
            if (k & 1) l *= x;
            x *= x;
        }
        lev = l;
    }
    // F at the current step; moves on to the next one.
    __device__ __forceinline__ double next()
    {
        const double f = annual ? (pos == 0 && n > 0 ? 12.0 * lev : 0.0) : lev;
        ++pos;
        const bool ann = pos == 12;
        pos = ann ? 0 : pos;
        n += ann ? 1 : 0;
        lev = ann ? lev * g : lev;
        return f;
    }
};

// A walk may be cut in time: the walker's transfer over steps [t0, t1) is
// accumulated by tr_step from tr_init, advance(transfer), once for each chunk
// before in order, sets the state they lead to, and past(t) ends a lane whose
// term is over by then.  W::TR of FLOW_TR doubles a lane (0: walked by one
// wavefront from the start).
constexpr int FLOW_TR = 4;

// What every walker knows of its lane.
struct FlowLane {
    int slot, uid, S;    // sorted slot, upload index (-1: padding), remaining term
    bool live;
    __device__ __forceinline__ void init(const RecParams &P, int at, int shift)
    {
        slot = at;
        S = P.term[slot] - shift;
        uid = P.uidx[slot];
        live = uid >= 0 && S > 0;
    }
};

// Scalar-reserve models (one life, or two lives with the reserve in state 00):
// occupancy P, flow f_t = c_{t-1} + P_t a0 (at t = S: the boundary reserve in
// place of a0), c_t = P_t (p a1 + (1 - p) b1), P_{t+1} = P_t p.
template <bool LDSQ, bool TWO, int FLOW>
struct FlowScalar {
    int S, qa, qb;
    double occ, carry, a0, a1, b1, a1mb1, rS;
    const double *cfb;
    int cfs;
    PatWalk pat;

    __device__ __forceinline__ void init(const RecParams &P, const FlowLane &L, int, int shift, int t0)
    {
        S = L.S;
        qa = P.qoff1[L.slot] + P.age1[L.slot] + shift;
        qb = TWO ? P.qoff2[L.slot] + P.age2[L.slot] + shift : 0;
        a0 = P.coef[L.slot];
        a1 = P.coef[P.n_pad + L.slot];
        b1 = P.coef[2 * P.n_pad + L.slot];
        rS = P.coef[3 * P.n_pad + L.slot];
        a1mb1 = a1 - b1;
        occ = L.live ? 1.0 : 0.0;
        carry = 0.0;
        if constexpr (FLOW == FLOW_TABLE) {
            cfb = P.cf_t + P.pat_code[L.slot] + (ptrdiff_t)shift * P.cf_cols;
            cfs = P.cf_cols;
        }
        if constexpr (FLOW == FLOW_PATTERN) pat.init(P, L.slot, shift, t0);
    }
    __device__ __forceinline__ FlowIn load(const RecParams &P, const double *__restrict__ lq, int t) const
    {
        FlowIn in{};
        in.x1 = flow_q<LDSQ>(P, lq, qa + t);
        if constexpr (TWO) in.x2 = flow_q<LDSQ>(P, lq, qb + t);
        if constexpr (FLOW == FLOW_TABLE) in.cv = cfb[(ptrdiff_t)t * cfs];
        return in;
    }
    __device__ __forceinline__ void shock(FlowIn &in, double m) const
    {
        in.x1 = shocked(in.x1, m);
        if constexpr (TWO) in.x2 = shocked(in.x2, m);
    }
    __device__ __forceinline__ static void tr_init(double (&x)[FLOW_TR]) { x[0] = 1.0; }
    __device__ __forceinline__ static void tr_step(double (&x)[FLOW_TR], const FlowIn &in)
    {
        x[0] *= TWO ? in.x1 * in.x2 : in.x1;
    }
    static constexpr int TR = 1;
    // State after the transfer x; past the term the occupancy is 0.
    __device__ __forceinline__ void advance(const double (&x)[FLOW_TR]) { occ *= x[0]; }
    __device__ __forceinline__ void past(int t)
    {
        if (t > S) occ = 0.0;
    }
    template <bool MASK>
    __device__ __forceinline__ double step(int t, const FlowIn &in)
    {
        const double p = TWO ? in.x1 * in.x2 : in.x1;
        double c, adv = a0;
        if constexpr (FLOW == FLOW_PATTERN) {
            const double f = pat.next();
            c = p * (f * a1);
            adv = f * a0;
        } else if constexpr (FLOW == FLOW_TABLE) {
            c = p * in.cv;
        } else {
            c = fma(p, a1mb1, b1);
        }
        const bool on = !MASK || t < S;
        const double out = fma(occ, on ? adv : rS, carry);
        carry = on ? occ * c : 0.0;
        occ = on ? occ * p : 0.0;
        return out;
    }
};

// Two lives with a vector reserve: occupancy of states 00, 10 and (LAST) 01.
// ESC: every amount times the payment factor.
template <bool LDSQ, bool LAST, bool ESC>
struct FlowVector {
    int S, qa, qb;
    double o00, o01, o10, carry, cf[6], d;
    PatWalk pat;

    __device__ __forceinline__ void init(const RecParams &P, const FlowLane &L, int, int shift, int t0)
    {
        S = L.S;
        qa = P.qoff1[L.slot] + P.age1[L.slot] + shift;
        qb = P.qoff2[L.slot] + P.age2[L.slot] + shift;
#pragma unroll
        for (int j = 0; j < 6; ++j) cf[j] = P.coef[j * P.n_pad + L.slot];
        d = LAST ? P.coef[6 * P.n_pad + L.slot] : 0.0;
        o00 = L.live ? 1.0 : 0.0;
        o01 = o10 = carry = 0.0;
        if constexpr (ESC) pat.init(P, L.slot, shift, t0);
    }
    __device__ __forceinline__ FlowIn load(const RecParams &P, const double *__restrict__ lq, int t) const
    {
        FlowIn in{};
        in.x1 = flow_q<LDSQ>(P, lq, qa + t);
        in.x2 = flow_q<LDSQ>(P, lq, qb + t);
        return in;
    }
    __device__ __forceinline__ void shock(FlowIn &in, double m) const
    {
        in.x1 = shocked(in.x1, m);
        in.x2 = shocked(in.x2, m);
    }
    // Transfer from state 00: survival of each life, then the arrivals in 10 and 01.
    static constexpr int TR = LAST ? 4 : 3;
    __device__ __forceinline__ static void tr_init(double (&x)[FLOW_TR])
    {
        x[0] = x[1] = 1.0;
        x[2] = x[3] = 0.0;
    }
    __device__ __forceinline__ static void tr_step(double (&x)[FLOW_TR], const FlowIn &in)
    {
        const double w = x[0] * x[1];
        x[2] = fma(x[2], in.x2, w * ((1.0 - in.x1) * in.x2));
        if constexpr (LAST) x[3] = fma(x[3], in.x1, w * (in.x1 * (1.0 - in.x2)));
        x[0] *= in.x1;
        x[1] *= in.x2;
    }
    __device__ __forceinline__ void advance(const double (&x)[FLOW_TR])
    {
        o10 = fma(o10, x[1], o00 * x[2]);
        if constexpr (LAST) o01 = fma(o01, x[0], o00 * x[3]);
        o00 *= x[0] * x[1];
    }
    __device__ __forceinline__ void past(int t)
    {
        if (t > S) o00 = o01 = o10 = 0.0;
    }
    template <bool MASK>
    __device__ __forceinline__ double step(int t, const FlowIn &in)
    {
        if (MASK && t >= S) o00 = o01 = o10 = 0.0;
        const double px = in.x1, py = in.x2, qx = 1.0 - px, qy = 1.0 - py;
        double f = 1.0;
        if constexpr (ESC) f = pat.next();
        double adv = fma(o10, cf[4], o00 * cf[0]);
        if constexpr (LAST) adv = fma(o01, cf[2], adv);
        const double out = ESC ? fma(f, adv, carry) : carry + adv;
        const double n00 = o00 * (px * py);
        const double n10 = fma(o10, py, o00 * (qx * py));
        double arr = fma(n10, cf[5], n00 * cf[1]);
        if constexpr (LAST) {
            const double n01 = fma(o01, px, o00 * (px * qy));
            arr = fma(n01, cf[3], arr);
            // benefit on the second death: from 00 both die, from 01 and 10 the survivor
            arr = fma(fma(o10, qy, fma(o01, qx, o00 * (qx * qy))), d, arr);
            o01 = n01;
        }
        o00 = n00;
        o10 = n10;
        carry = ESC ? f * arr : arr;
        return out;
    }
};

// Three independent lives: the occupancy of every state is a product of the
// lives' survival probabilities, and "some life alive" is the sum of positive
// terms X1 + (1 - X1)(X2 + (1 - X2) X3).
template <bool LDSQ>
struct FlowThree {
    int S, qa, qb, qc;
    bool last;
    double l1, l2, l3, carry, a0all, a0, a1;

    __device__ __forceinline__ void init(const RecParams &P, const FlowLane &L, int kind, int shift, int)
    {
        S = L.S;
        last = kind == KIND_LAST;
        qa = P.qoff1[L.slot] + P.age1[L.slot] + shift;
        qb = P.qoff2[L.slot] + P.age2[L.slot] + shift;
        qc = P.qoff3[L.slot] + P.age3[L.slot] + shift;
        a0all = P.coef[L.slot];
        a1 = P.coef[P.n_pad + L.slot];
        a0 = last ? P.coef[2 * P.n_pad + L.slot] : 0.0;
        l1 = l2 = l3 = L.live ? 1.0 : 0.0;
        carry = 0.0;
    }
    __device__ __forceinline__ FlowIn load(const RecParams &P, const double *__restrict__ lq, int t) const
    {
        FlowIn in{};
        in.x1 = flow_q<LDSQ>(P, lq, qa + t);
        in.x2 = flow_q<LDSQ>(P, lq, qb + t);
        in.x3 = flow_q<LDSQ>(P, lq, qc + t);
        return in;
    }
    __device__ __forceinline__ void shock(FlowIn &in, double m) const
    {
        in.x1 = shocked(in.x1, m);
        in.x2 = shocked(in.x2, m);
        in.x3 = shocked(in.x3, m);
    }
    static constexpr int TR = 3;
    __device__ __forceinline__ static void tr_init(double (&x)[FLOW_TR]) { x[0] = x[1] = x[2] = 1.0; }
    __device__ __forceinline__ static void tr_step(double (&x)[FLOW_TR], const FlowIn &in)
    {
        x[0] *= in.x1;
        x[1] *= in.x2;
        x[2] *= in.x3;
    }
    __device__ __forceinline__ void advance(const double (&x)[FLOW_TR])
    {
        l1 *= x[0];
        l2 *= x[1];
        l3 *= x[2];
    }
    __device__ __forceinline__ void past(int t)
    {
        if (t > S) l1 = l2 = l3 = 0.0;
    }
    template <bool MASK>
    __device__ __forceinline__ double step(int t, const FlowIn &in)
    {
        if (MASK && t >= S) l1 = l2 = l3 = 0.0;
        // all alive: a0all; some alive but not all: a0 (the last survivor's)
        const double all = l1 * l2 * l3;
        const double some = fma(1.0 - l1, fma(1.0 - l2, l3, l2), l1);
        const double out = carry + fma(all, a0all - a0, some * a0);
        l1 *= in.x1;
        l2 *= in.x2;
        l3 *= in.x3;
        const double nsome = fma(1.0 - l1, fma(1.0 - l2, l3, l2), l1);
        carry = (last ? nsome : l1 * l2 * l3) * a1;
        return out;
    }
};

// One life on an uploaded Markov model of up to four states: occupancy row
// vector times the matrix at the attained age; benefits at the end of a month,
// premium in state 0.  A lane of its own per policy would read 128 scattered
// bytes a month, 512 cache lines for a wavefront, and the L1 takes them one a
// cycle.  Here four lanes share a policy: lane l holds column l % 4 of the
// matrices of the policies l / 4 + 16 s, s = 0..3 (transposed copy of the
// model), so that an access covers whole lines of sixteen policies, and the
// occupancies pass between the four lanes by quad permutations.  The matrices
// are read two months ahead.  Lane l returns the flow of policy l / 4 + 16 (l %
// 4), which is its place in a month's kept flows.
template <int Q>
__device__ __forceinline__ double quad_get(double x) { return dpp_f64<Q * 0x55>(x); }   // lane Q of the quad

struct FlowMarkov4 {
    static constexpr int TR = 0;
    int S[4], own;   // remaining terms of the four policies; which of them is the lane's own
    const double *wb[4];
    double occ[4], c[4], carry, a0;
    double w1[4][4], w2[4][4];   // columns of the step to come and the one after

    __device__ __forceinline__ void fetch(double (&w)[4][4], int t) const
    {
#pragma unroll
        for (int s = 0; s < 4; ++s) {   // (past the term: the last month's)
            const double2 *p = reinterpret_cast<const double2 *>(wb[s] + (size_t)max(min(t, S[s] - 1), 0) * 16);
            const double2 x = p[0], y = p[1];
            w[s][0] = x.x;
            w[s][1] = x.y;
            w[s][2] = y.x;
            w[s][3] = y.y;
        }
    }
    __device__ __forceinline__ void init(const RecParams &P, const FlowLane &L, int, int shift, int t0)
    {
        const int lane = threadIdx.x & 63, first = L.slot - lane, j = lane & 3;
        own = j;
        a0 = P.coef[first + j * 16 + (lane >> 2)];
        carry = 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            FlowLane K;
            K.init(P, first + s * 16 + (lane >> 2), shift);
            S[s] = K.S;
            const int model = K.live ? P.pat_code[K.slot] : 0;
            const int age0 = K.live ? P.age1[K.slot] + shift : 0;
            wb[s] = P.mk_wt + ((size_t)model * P.mk_ages + age0) * 16 + 4 * j;
            c[s] = P.coef[(1 + j) * P.n_pad + K.slot];
            occ[s] = K.live && j == 0 ? 1.0 : 0.0;
        }
        fetch(w1, t0);
        fetch(w2, t0 + 1);
    }
    // f_t
    __device__ __forceinline__ double step(int t)
    {
        double out = 0.0, arr = 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double o = t < S[s] ? occ[s] : 0.0;
            const double o0 = quad_get<0>(o), o1 = quad_get<1>(o), o2 = quad_get<2>(o), o3 = quad_get<3>(o);
            const double n = fma(o3, w1[s][3], fma(o2, w1[s][2], fma(o1, w1[s][1], o0 * w1[s][0])));
            double x = n * c[s];
            x += dpp_f64<0xb1>(x);   // the quad's sum in every lane
            x += dpp_f64<0x4e>(x);
            out = own == s ? fma(o0, a0, carry) : out;
            arr = own == s ? x : arr;
            occ[s] = n;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) w1[s][i] = w2[s][i];
        fetch(w2, t + 2);
        carry = arr;
        return out;
    }
};

// A model of more states, one policy a lane: the matrix is read a row at a time,
// which keeps the registers of the instance those of the other models.
struct FlowMarkov9 {
    static constexpr int M = MAX_MK_STATES, TR = 0;
    int S;
    const double *wb;
    double occ[M], c[M], carry, a0;

    __device__ __forceinline__ void init(const RecParams &P, const FlowLane &L, int, int shift, int)
    {
        S = L.S;
        a0 = P.coef[L.slot];
        const int model = L.live ? P.pat_code[L.slot] : 0;
        const int age0 = L.live ? P.age1[L.slot] + shift : 0;
        wb = P.mk_w + ((size_t)model * P.mk_ages + age0) * (M * M);
#pragma unroll
        for (int j = 0; j < M; ++j) {
            c[j] = P.coef[P.n_pad + L.slot] * P.mk_c[model * M + j];
            occ[j] = 0.0;
        }
        occ[0] = L.live ? 1.0 : 0.0;
        carry = 0.0;
    }
    // f_t (past the term the last month's matrix is read again)
    __device__ __forceinline__ double step(int t)
    {
        if (t >= S) {
#pragma unroll
            for (int j = 0; j < M; ++j) occ[j] = 0.0;
        }
        const double *w = wb + (size_t)max(min(t, S - 1), 0) * (M * M);
        const double out = fma(occ[0], a0, carry);
        double n[M];
#pragma unroll
        for (int j = 0; j < M; ++j) n[j] = occ[0] * w[j];
#pragma unroll 1
        for (int i = 1; i < M; ++i) {   // (the occupancies move down one place per row)
#pragma unroll
            for (int j = 0; j + 1 < M; ++j) occ[j] = occ[j + 1];
#pragma unroll
            for (int j = 0; j < M; ++j) n[j] = fma(occ[0], w[i * M + j], n[j]);
        }
        double arr = 0.0;
#pragma unroll
        for (int j = 0; j < M; ++j) {
            arr = fma(n[j], c[j], arr);
            occ[j] = n[j];
        }
        carry = arr;
        return out;
    }
};

// Annuity paid at the fraction f of the month: a second flow, discounted by
// D_t v_t^f, beside the premium's.
template <bool LDSQ, bool TWO>
struct FlowFrac {
    int S, qa, qb;
    double occ, a0, pay, f, g, mid;

    __device__ __forceinline__ void init(const RecParams &P, const FlowLane &L, int, int shift, int)
    {
        S = L.S;
        qa = P.qoff1[L.slot] + P.age1[L.slot] + shift;
        qb = TWO ? P.qoff2[L.slot] + P.age2[L.slot] + shift : 0;
        a0 = P.coef[L.slot];
        pay = P.coef[P.n_pad + L.slot];
        f = P.frac;
        g = 1.0 - P.frac;
        occ = L.live ? 1.0 : 0.0;
    }
    __device__ __forceinline__ FlowIn load(const RecParams &P, const double *__restrict__ lq, int t) const
    {
        FlowIn in{};
        in.x1 = flow_q<LDSQ>(P, lq, qa + t);
        if constexpr (TWO) in.x2 = flow_q<LDSQ>(P, lq, qb + t);
        return in;
    }
    __device__ __forceinline__ void shock(FlowIn &in, double m) const
    {
        in.x1 = shocked(in.x1, m);
        if constexpr (TWO) in.x2 = shocked(in.x2, m);
    }
    static constexpr int TR = 1;
    __device__ __forceinline__ static void tr_init(double (&x)[FLOW_TR]) { x[0] = 1.0; }
    __device__ __forceinline__ static void tr_step(double (&x)[FLOW_TR], const FlowIn &in)
    {
        x[0] *= TWO ? in.x1 * in.x2 : in.x1;
    }
    __device__ __forceinline__ void advance(const double (&x)[FLOW_TR]) { occ *= x[0]; }
    __device__ __forceinline__ void past(int t)
    {
        if (t > S) occ = 0.0;
    }
    // f_t; the flow within the month goes to mid.
    template <bool MASK>
    __device__ __forceinline__ double step(int t, const FlowIn &in)
    {
        if (MASK && t >= S) occ = 0.0;
        const double pf = TWO ? fma(f, in.x1, g) * fma(f, in.x2, g) : fma(f, in.x1, g);
        mid = occ * (pf * pay);
        const double out = occ * a0;
        occ *= TWO ? in.x1 * in.x2 : in.x1;
        return out;
    }
};

// Walk of a tile at one node over the steps [t0, t1), t0 a multiple of U: emit(t,
// flow) for each step of a block of U consecutive steps, then done(t + U) once
// per block.  Blocks are whole: steps past the last flow give 0.  The walker
// stands at step t0 (or, `lead`, at t0 - 1: that step is taken first and its flow
// dropped, so that the amounts it leaves for t0 are there).  smax: the last
// flow's time; every lane of the tile lives past smin.
template <int U, class W, class Emit, class Done>
__device__ __forceinline__ void flow_walk(const RecParams &P, const double *__restrict__ lq, W &w, double m, int smax,
                                          int smin, int t0, int t1, bool lead, Emit emit, Done done)
{
    const bool shock = m != 1.0;
    if (lead) {
        FlowIn a = w.load(P, lq, min(t0 - 1, smax - 1));
        if (shock) w.shock(a, m);
        (void)w.template step<true>(t0 - 1, a);
    }
    int t = t0;
    for (; t + U <= min(smin, t1); t += U) {
        FlowIn a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = w.load(P, lq, t + u);
        if (shock) {
#pragma unroll
            for (int u = 0; u < U; ++u) w.shock(a[u], m);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) emit(t + u, w.template step<false>(t + u, a[u]));
        done(t + U);
    }
#pragma unroll 1
    for (; t < t1; t += U) {
        FlowIn a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = w.load(P, lq, min(t + u, smax - 1));
        if (shock) {
#pragma unroll
            for (int u = 0; u < U; ++u) w.shock(a[u], m);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) emit(t + u, w.template step<true>(t + u, a[u]));
        done(t + U);
    }
}

// The transfer of a walker over the steps [t0, t1).
template <class W>
__device__ __forceinline__ void flow_transfer(const RecParams &P, const double *__restrict__ lq, const W &w, double m,
                                              int smax, int t0, int t1, double (&x)[FLOW_TR])
{
    constexpr int U = 8;
    W::tr_init(x);
    for (int t = t0; t < t1; t += U) {
        FlowIn a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = w.load(P, lq, min(t + u, smax - 1));
        if (m != 1.0) {
#pragma unroll
            for (int u = 0; u < U; ++u) w.shock(a[u], m);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (t + u < t1) W::tr_step(x, a[u]);
    }
}

// Calls visit(tag) for the tile's model, its walker the tag's type.
template <class W>
struct FlowTag {
    typedef W type;
};

// Tiles a kernel instance can hold: level ones only; payment patterns too; every kind.
enum FlowSet : int { FLOWS_LEVEL = 0, FLOWS_PATTERN = 1, FLOWS_ALL = 2 };

template <bool LDSQ, bool VEC, int SET, class Visit>
__device__ __forceinline__ void flow_model(const RecParams &P, int kind, int flow, Visit visit)
{
    if constexpr (SET >= FLOWS_PATTERN) {
        if (flow == FLOW_PATTERN) {
            if (kind == KIND_SINGLE) visit(FlowTag<FlowScalar<LDSQ, false, FLOW_PATTERN>>{});
            else if (kind == KIND_JOINT) visit(FlowTag<FlowScalar<LDSQ, true, FLOW_PATTERN>>{});
            else if (kind == KIND_REV) visit(FlowTag<FlowVector<LDSQ, false, true>>{});
            else visit(FlowTag<FlowVector<LDSQ, true, true>>{});
            return;
        }
    }
    if constexpr (SET >= FLOWS_ALL) {
        if (flow == FLOW_TABLE) {
            visit(FlowTag<FlowScalar<LDSQ, false, FLOW_TABLE>>{});
            return;
        }
        if (flow == FLOW_THREE) {
            visit(FlowTag<FlowThree<LDSQ>>{});
            return;
        }
        if (flow == FLOW_MARKOV) {
            if (P.mk_states > 4) visit(FlowTag<FlowMarkov9>{});
            else visit(FlowTag<FlowMarkov4>{});
            return;
        }
        if (flow == FLOW_FRAC) {
            if (kind == KIND_JOINT) visit(FlowTag<FlowFrac<LDSQ, true>>{});
            else visit(FlowTag<FlowFrac<LDSQ, false>>{});
            return;
        }
    }
    if (kind == KIND_SINGLE) visit(FlowTag<FlowScalar<LDSQ, false, FLOW_LEVEL>>{});
    else if (kind == KIND_JOINT) visit(FlowTag<FlowScalar<LDSQ, true, FLOW_LEVEL>>{});
    else if constexpr (VEC) {
        if (kind == KIND_REV) visit(FlowTag<FlowVector<LDSQ, false, false>>{});
        else visit(FlowTag<FlowVector<LDSQ, true, false>>{});
    }
}

template <class W>
struct FlowTraits {
    static constexpr bool markov = false, frac = false;
};
template <>
struct FlowTraits<FlowMarkov4> {
    static constexpr bool markov = true, frac = false;
};
template <>
struct FlowTraits<FlowMarkov9> {
    static constexpr bool markov = true, frac = false;
};
template <bool LDSQ, bool TWO>
struct FlowTraits<FlowFrac<LDSQ, TWO>> {
    static constexpr bool markov = false, frac = true;
};
}  // namespace rr
