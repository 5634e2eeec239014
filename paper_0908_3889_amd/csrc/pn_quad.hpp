// pn_quad.hpp -- the FP64 integration with four lanes on one inspiral, for
// batches that leave most of the chip idle: the time is then the chain of
// steps of the longest inspiral, and a step's time the instructions a wave
// issues for it.
//
// Lanes 0, 1, 2 of a quad hold S1, S2, L_hat and the stage derivatives of
// their own vector, lane 3 holds omega; what depends on omega alone is
// evaluated by all four, and vectors move between the lanes by quad
// permutations (DPP).  The stage sums, the error estimate and the norm's
// scales are a third of the one-lane kernel's.  Every number is formed by the
// same operations in the same order as there, so the results are the same
// bit for bit; a step whose fast path ends with a NaN norm is tried again with
// what the fast path leaves out of that (rhs_quad).
//
// Included by pn_lib.hip after the FP64 lane.
#pragma once

namespace pn {

template <int CTRL>
__device__ __forceinline__ double quad_perm(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int CTRL>
__device__ __forceinline__ int quad_perm(int v) {
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
constexpr int kQp(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }
constexpr int kQ0 = kQp(0, 0, 0, 0), kQ1 = kQp(1, 1, 1, 1), kQ2 = kQp(2, 2, 2, 2), kQ3 = kQp(3, 3, 3, 3);

// The coefficient row as one lane of the quad needs it, and the constants of
// the stage's cube root and log: kept in registers (a wave alone on its SIMD
// waits for every scalar move that would fetch them again).
struct RowQ {
    double M, C2, SO1, SO2, C4, SSD, C5, C6, C7, K;
    double G;          // G1 (lane 0), G2 (lane 1), 0
    double SIGM;       // lanes 0 and 1, else 0
    double LAM;        // -lambda in lane 2
};

struct PolyQ {
    double cb[10];     // cbrt1p_small_m1: q_8 .. q_0, then 1/3
    double lg[7];      // log1p_cbrt_over_w: r_5 .. r_0, then 3
};

__device__ __forceinline__ void keep(double& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ void make_poly(PolyQ& p) {
    const double cb[10] = {-0.01177066091614973521624749, 0.0135791980361245423248501, -0.01583407049188512767371284,
                           0.01900090236519766360899345, -0.0234720319593868172360808, 0.03017832676360298774987899,
                           -0.04115226337441031440928335, 0.06172839506164371309340048, -0.1111111111111111111111111,
                           1.0 / 3.0};
    const double lg[7] = {0.4297688281944602466457629, -0.5002437143231824139713031, 0.599999539072323222208094,
                          -0.7499999603441906901946652, 1.000000000035512911627931, -1.500000000000957520846056, 3.0};
#pragma unroll
    for (int i = 0; i < 10; ++i) { p.cb[i] = cb[i]; keep(p.cb[i]); }
#pragma unroll
    for (int i = 0; i < 7; ++i) { p.lg[i] = lg[i]; keep(p.lg[i]); }
}

// Growth of omega at the derivative of a step's start up to which the fast path
// is tried (omega grows faster than linearly; the polynomials reach 1/16).
constexpr double kQuadRange = 0.05;

struct LaneQ {
    double v[3];       // own vector: S1, S2, L_hat, or (omega, 0, 0)
    double k1[3];      // its derivative along the step's variable
    double w;          // omega, on every lane
    double kw;         // k1 of omega, on every lane
    double lnv, x, dt1, t, h;
    double phase;
    double range;      // a step to more than (1 + range) omega takes the general path
    RowQ r;
    int64_t idx;
    int acc, rej, nt;
    bool omega_mode, last_rej;
};

// dy/dt of the own vector at the stage point Y into d; ws: omega there, kws:
// d omega/dt (lane 3's on every lane), xo: the cube root used; returns the log
// used.  The operations are rhs_at's.  FAST: the polynomials of the cube root
// and the log alone; `far` is set where the stage point is too far from the
// step's base for them.  Otherwise such lanes take them in full.
// Lanes 0 and 1 add 0 times lane 2's sum to their derivative and lane 2 a zero
// Omega x L_hat to its own, which saves selects: nothing but a sign of zero for
// finite numbers, a NaN where the other factor is infinite.  At a stage point
// that is as good, the candidate is then not finite; a candidate far past
// omega_f may be, and its infinite derivative means a rejected step.  EXACT:
// the selects.
template <bool FAST, bool EXACT = false>
__device__ __forceinline__ double rhs_quad(const RowQ& r, const PolyQ& pc, const TermConsts& tc, const LogBase& lb,
                                           const double (&Y)[3], double (&d)[3], double& ws, double& kws, double& xo,
                                           int lane, bool& far) {
    const double w = quad_perm<kQ3>(Y[0]);
    const double u = (w - lb.w) * lb.iw;
    double q = pc.cb[0];
#pragma unroll
    for (int i = 1; i < 10; ++i) q = __builtin_fma(q, u, pc.cb[i]);
    const double c = u * q;
    double x = __builtin_fma(lb.x, c, lb.x);
    double g = pc.lg[0];
#pragma unroll
    for (int i = 1; i < 7; ++i) g = __builtin_fma(g, c, pc.lg[i]);
    double lnv = __builtin_fma(c, g, lb.lnv);
    const bool f = !(__builtin_fabs(u) <= kSmallU);
    if (FAST) far = far || f;
    else if (__ballot(f) != 0) {
        if (f) {
            const double v = r.M * w;
            x = cbrt_real(v);
            lnv = log_pos(__builtin_fabs(v));
        }
    }
    // P = L, L, S1, S1 and Q = S2, S1, S2, S2 on lanes 0 .. 3: their product is
    // L.S2, L.S1, S1.S2, S1.S2
    double P[3], Q[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        P[i] = quad_perm<kQp(2, 2, 0, 0)>(Y[i]);
        Q[i] = quad_perm<kQp(1, 0, 1, 1)>(Y[i]);
    }
    const double dot = __builtin_fma(P[0], Q[0], __builtin_fma(P[1], Q[1], P[2] * Q[2]));
    const double LS2 = quad_perm<kQ0>(dot), LS1 = quad_perm<kQ1>(dot);
    const double x2 = x * x;
    // d omega/dt (meant on lane 3, where dot = S1.S2)
    const double c3p = __builtin_fma(-r.SO2, LS2, __builtin_fma(-r.SO1, LS1, tc.c3));
    const double ssb = __builtin_fma(247.0, dot, -721.0 * (LS1 * LS2));
    const double c4p = __builtin_fma(-r.SSD, ssb, r.C4);
    const double c6p = __builtin_fma(tc.c6lnv, lnv, r.C6);
    double B = __builtin_fma(x, r.C7, c6p);
    B = __builtin_fma(x, B, r.C5);
    B = __builtin_fma(x, B, c4p);
    B = __builtin_fma(x, B, c3p);
    B = __builtin_fma(x, B, r.C2);
    B = __builtin_fma(x2, B, 1.0);
    const double ww = w * w, wx2 = w * x2;
    const double dw = (r.K * ww) * wx2 * B;
    // Omega x (own vector) on lanes 0 and 1
    const double be = r.SIGM * ww;
    const double al = __builtin_fma(r.G, wx2, -3.0 * be * dot);
    const double o0 = __builtin_fma(al, P[0], be * Q[0]), o1 = __builtin_fma(al, P[1], be * Q[1]),
                 o2 = __builtin_fma(al, P[2], be * Q[2]);
    d[0] = __builtin_fma(o1, Y[2], -o2 * Y[1]);
    d[1] = __builtin_fma(o2, Y[0], -o0 * Y[2]);
    d[2] = __builtin_fma(o0, Y[1], -o1 * Y[0]);
    // -lambda x (dS1/dt + dS2/dt) on lane 2; there and on lane 3 Omega is 0,
    // so that adding the cross product changes nothing
    const double qx = r.LAM * x;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double s = quad_perm<kQ0>(d[i]) + quad_perm<kQ1>(d[i]);
        if (EXACT) d[i] = lane < 2 ? d[i] : qx * s;
        else d[i] = __builtin_fma(qx, s, d[i]);
    }
    d[0] = lane == 3 ? dw : d[0];
    kws = quad_perm<kQ3>(dw);
    ws = w;
    xo = x;
    return lnv;
}

// omega mode: as to_omega_variable, kw on every lane
__device__ __forceinline__ void to_omega_quad(double (&k)[3], double& kw, double& dt, bool om, bool lane3) {
    const double s = om ? recip(kw) : 1.0;
#pragma unroll
    for (int i = 0; i < 3; ++i) k[i] *= s;
    if (lane3) k[0] = om ? 1.0 : k[0];
    kw = om ? 1.0 : kw;
    dt = s;
}

template <bool RECORD, bool PHASE>
struct QuadF64 {
    static __device__ __forceinline__ void gather(const double (&v)[3], double (&y)[10]) {
        y[0] = quad_perm<kQ3>(v[0]);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            y[1 + i] = quad_perm<kQ0>(v[i]);
            y[4 + i] = quad_perm<kQ1>(v[i]);
            y[7 + i] = quad_perm<kQ2>(v[i]);
        }
    }
    static __device__ __forceinline__ void own(int q, const double* y, double (&v)[3]) {
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const double a = q == 0 ? y[1 + i] : (q == 1 ? y[4 + i] : y[7 + i]);
            v[i] = q == 3 ? (i == 0 ? y[0] : 0.0) : a;
        }
    }
    static __device__ __forceinline__ void checkpoint(const Uni& u, int64_t idx, int j, int q, const double (&v)[3]) {
        double* ck = tape_of(u, idx) + 2 + u.tape_cap + (int64_t)j * 10;
        if (q == 3) ck[0] = v[0];
        else {
#pragma unroll
            for (int i = 0; i < 3; ++i) ck[1 + 3 * q + i] = v[i];
        }
    }

    // the one-lane start, on every lane; then each keeps its part
    static __device__ int load(const Io& io, const Uni& u, LaneQ& L, int64_t idx, int q) {
        L.idx = idx;
        double y[10], k1[10], m1, m2;
        const int st = read_input<PHASE>(io, u, idx, y, m1, m2);
        if (st) return st;
        Row row;
        make_row(row, m1, m2, u.terms, u.theta_literal);
        LogBase lb;
        L.lnv = rhs_x<Row, false>(row, u.tc, lb, y, k1, L.x);
        own(q, y, L.v);
        own(q, k1, L.k1);
        L.w = y[0];
        L.kw = k1[0];
        L.t = 0.0;
        L.acc = 0; L.rej = 0; L.nt = 0;
        L.omega_mode = false; L.last_rej = false;
        L.h = u.h0;
        L.dt1 = 1.0;
        L.phase = 0.0;
        L.range = kQuadRange;
        L.r.M = row[R_M]; L.r.C2 = row[R_C2]; L.r.SO1 = row[R_SO1]; L.r.SO2 = row[R_SO2]; L.r.C4 = row[R_C4];
        L.r.SSD = row[R_SSD]; L.r.C5 = row[R_C5]; L.r.C6 = row[R_C6]; L.r.C7 = row[R_C7]; L.r.K = row[R_K];
        L.r.G = q == 0 ? row[R_G1] : (q == 1 ? row[R_G2] : 0.0);
        L.r.SIGM = q < 2 ? row[R_SIGM] : 0.0;
        L.r.LAM = q == 2 ? -row[R_LAM] : 0.0;
        if (RECORD) checkpoint(u, idx, 0, q, L.v);
        return 0;
    }

    static __device__ void finish(const Io& io, const Uni& u, const LaneQ& L, int st, int q) {
        double y[10];
        gather(L.v, y);
        if (q != 0) return;
        write_out<PHASE>(io, u, L.idx, y, L.t, L.acc, L.rej, rhs_count(L, st), st, L.phase);
        if (RECORD) {
            double* tp = tape_of(u, L.idx);
            const int nt = L.omega_mode ? L.nt : L.acc;
            tp[0] = (double)nt;
            tp[1] = (double)(L.acc - nt);
        }
    }

    // error_norm over the quad: lane 0 has the scales of S1 and, by a
    // permutation, of omega (one reciprocal for the four), lanes 1 and 2 of
    // their own three; the sum runs through the lanes in the order of the
    // components
    template <bool FAST>
    static __device__ __forceinline__ double norm(const Uni& u, const LaneQ& L, const double (&Y)[3],
                                                  const double (&e)[3], int q, bool& far) {
        double sc[3], iv[3], iw;
#pragma unroll
        for (int i = 0; i < 3; ++i) sc[i] = __builtin_fma(u.tol, fmax_abs(L.v[i], Y[i]), u.tol);
        double s0 = quad_perm<kQ3>(sc[0]);
        s0 = q == 0 ? s0 : 1.0;
        bool bad = false;
        // lane 3 runs along on omega's scale three times over; nothing reads it
        rcp4(s0, sc[0], sc[1], sc[2], iw, iv[0], iv[1], iv[2], bad);
        // omega's e/scale from lane 0, where its reciprocal is
        double qw = quad_perm<kQ3>(e[0]) * quad_perm<kQ0>(iw);
        double qv[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) qv[i] = e[i] * iv[i];
        if (FAST) far = far || (bad && q != 3);
        else if (__ballot(bad && q != 3) != 0) {
            // error_norm falls back as a whole
            int b = (bad && q != 3) ? 1 : 0;
            b = quad_perm<kQ0>(b) | quad_perm<kQ1>(b) | quad_perm<kQ2>(b);
            const double w3 = e[0] * rcp_1step(sc[0]);
            const double w = quad_perm<kQ3>(w3);
            if (b) {
                qw = w;
#pragma unroll
                for (int i = 0; i < 3; ++i) qv[i] = e[i] * rcp_1step(sc[i]);
            }
        }
        double z = __builtin_fma(qw, qw, 0.0);
#pragma unroll
        for (int i = 0; i < 3; ++i) z = __builtin_fma(qv[i], qv[i], z);
        z = quad_perm<kQ0>(z);
#pragma unroll
        for (int i = 0; i < 3; ++i) z = __builtin_fma(qv[i], qv[i], z);
        z = quad_perm<kQ1>(z);
#pragma unroll
        for (int i = 0; i < 3; ++i) z = __builtin_fma(qv[i], qv[i], z);
        return quad_perm<kQ2>(z) * 0.1;
    }

    // What an attempted step of size h leaves to the step control.
    struct Tried {
        double Y[3], k7[3];        // candidate state and its derivative (own vector)
        double ws, kws, lnv, x;    // omega, its derivative, log and cube root there
        double dts, dt7, ps;       // omega mode: sum of b_j dt_j, dt_7; phase sum
        double z;
        bool fin, far;
    };

    // The stages of a step, the error norm.  FAST: no lane in omega mode, every
    // stage point near the step's base (far tells afterwards): one block of
    // straight-line code, so that the chains of the polynomials and the vector
    // work of a stage fill each other's latencies.
    template <bool FAST>
    static __device__ __forceinline__ void attempt(const Uni& u, const PolyQ& pc, const LaneQ& L, double h, int q, Tried& T) {
        const bool lane3 = q == 3, om = L.omega_mode;
        const double (&y)[3] = L.v;
        const double (&k1)[3] = L.k1;
        double Y[3], k2[3], k3[3], k4[3], k5[3], k6[3];
        double ws, kws, x7, dtj = 1.0;
        double dts = B1 * L.dt1;
        double ps = 0.0;
        bool far = false;
        if (PHASE) ps = B1 * (L.w * L.dt1);
        LogBase lb;
        lb.w = L.w;
        lb.iw = rcp_1step(L.w);
        lb.lnv = L.lnv;
        lb.x = L.x;
        {
            const double c1 = h * A21;
#pragma unroll
            for (int i = 0; i < 3; ++i) Y[i] = __builtin_fma(c1, k1[i], y[i]);
            rhs_quad<FAST>(L.r, pc, u.tc, lb, Y, k2, ws, kws, x7, q, far);
            if (!FAST) to_omega_quad(k2, kws, dtj, om, lane3);
        }
        {
            const double c1 = h * A31, c2 = h * A32;
#pragma unroll
            for (int i = 0; i < 3; ++i) Y[i] = __builtin_fma(c2, k2[i], __builtin_fma(c1, k1[i], y[i]));
            rhs_quad<FAST>(L.r, pc, u.tc, lb, Y, k3, ws, kws, x7, q, far);
            if (!FAST) { to_omega_quad(k3, kws, dtj, om, lane3); dts = __builtin_fma(B3, dtj, dts); }
            if (PHASE) ps = __builtin_fma(B3, ws * dtj, ps);
        }
        {
            const double c1 = h * A41, c2 = h * A42, c3 = h * A43;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                Y[i] = __builtin_fma(c3, k3[i], __builtin_fma(c2, k2[i], __builtin_fma(c1, k1[i], y[i])));
            rhs_quad<FAST>(L.r, pc, u.tc, lb, Y, k4, ws, kws, x7, q, far);
            if (!FAST) { to_omega_quad(k4, kws, dtj, om, lane3); dts = __builtin_fma(B4, dtj, dts); }
            if (PHASE) ps = __builtin_fma(B4, ws * dtj, ps);
        }
        {
            const double c1 = h * A51, c2 = h * A52, c3 = h * A53, c4 = h * A54;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                Y[i] = __builtin_fma(c4, k4[i], __builtin_fma(c3, k3[i],
                       __builtin_fma(c2, k2[i], __builtin_fma(c1, k1[i], y[i]))));
            rhs_quad<FAST>(L.r, pc, u.tc, lb, Y, k5, ws, kws, x7, q, far);
            if (!FAST) { to_omega_quad(k5, kws, dtj, om, lane3); dts = __builtin_fma(B5, dtj, dts); }
            if (PHASE) ps = __builtin_fma(B5, ws * dtj, ps);
        }
        {
            const double c1 = h * A61, c2 = h * A62, c3 = h * A63, c4 = h * A64, c5 = h * A65;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                Y[i] = __builtin_fma(c5, k5[i], __builtin_fma(c4, k4[i], __builtin_fma(c3, k3[i],
                       __builtin_fma(c2, k2[i], __builtin_fma(c1, k1[i], y[i])))));
            rhs_quad<FAST>(L.r, pc, u.tc, lb, Y, k6, ws, kws, x7, q, far);
            if (!FAST) { to_omega_quad(k6, kws, dtj, om, lane3); dts = __builtin_fma(B6, dtj, dts); }
            if (PHASE) ps = __builtin_fma(B6, ws * dtj, ps);
        }
        double e[3];
        {
            const double c1 = h * B1, c3 = h * B3, c4 = h * B4, c5 = h * B5, c6 = h * B6;
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                T.Y[i] = __builtin_fma(c6, k6[i], __builtin_fma(c5, k5[i], __builtin_fma(c4, k4[i],
                         __builtin_fma(c3, k3[i], __builtin_fma(c1, k1[i], y[i])))));
                e[i] = __builtin_fma(E6, k6[i], __builtin_fma(E5, k5[i], __builtin_fma(E4, k4[i],
                       __builtin_fma(E3, k3[i], E1 * k1[i]))));
            }
        }
        T.lnv = rhs_quad<FAST, !FAST>(L.r, pc, u.tc, lb, T.Y, T.k7, T.ws, T.kws, T.x, q, far);
        T.dt7 = 1.0;
        if (!FAST) to_omega_quad(T.k7, T.kws, T.dt7, om, lane3);
#pragma unroll
        for (int i = 0; i < 3; ++i) e[i] = __builtin_fma(E7, T.k7[i], e[i]);
        T.z = norm<FAST>(u, L, T.Y, e, q, far) * (h * h);
        // (a state that is not finite leaves the fast path in the norm: error_norm)
        T.fin = FAST || (finite(T.Y[0]) && finite(T.Y[1]) && finite(T.Y[2]));
        T.dts = dts;
        T.ps = ps;
        T.far = far;
    }

    // One attempted step; as F64::step.  A NaN norm on the fast path leaves
    // the inspiral where it was and its next step to the general path, by a
    // range below any step's (leaving the fast path for it within the step
    // would make that branch wait for the norm).
    static __device__ __forceinline__ int step(const Uni& u, const PolyQ& pc, LaneQ& L, bool active, bool any_w, int q) {
        const bool lane3 = q == 3;
        int st = 0;
        if (L.omega_mode ? L.dt1 <= 0 : (u.rr_on && L.kw <= 0)) st = PN_ST_OMEGADOT_NONPOSITIVE;
        if (RECORD && L.acc >= u.tape_cap) st = PN_ST_TAPE_FULL;
        if (L.acc + L.rej >= step_limit(u)) st = PN_ST_MAX_STEPS;
        const bool go = active && st == 0;
        bool last = false;
        double h = active ? L.h : 0.0;
        Tried T;
        if (__builtin_expect(any_w, 0)) {
            const double remain = L.omega_mode ? u.omega_f - L.w : 0.0;
            last = L.omega_mode && L.h >= remain;
            h = last ? remain : L.h;
            h = active ? h : 0.0;
        }
        // a step expected to leave the polynomials' range is not tried twice
        bool slow = any_w || __ballot(h * L.kw > L.range * L.w) != 0;
        if (__builtin_expect(!slow, 1)) {
            attempt<true>(u, pc, L, h, q, T);
            slow = __ballot(T.far) != 0;
        }
        if (__builtin_expect(slow, 0)) attempt<false>(u, pc, L, h, q, T);
        bool fin = T.fin;
        if (__builtin_expect(slow, 0)) {
            int f = fin ? 1 : 0;
            f = quad_perm<kQ0>(f) & quad_perm<kQ1>(f) & quad_perm<kQ2>(f) & quad_perm<kQ3>(f);
            fin = f != 0;
        }
        const double z = T.z, ws = T.ws;
        fin = fin && !__builtin_isnan(z);
        L.range = go && !fin ? -1.0 : kQuadRange;

        // as control()
        if (go && !fin && slow) st = PN_ST_NONFINITE;
        const bool ok = go && fin;
        const bool acc = ok && z <= Z_ACCEPT;
        const bool to_w = acc && !L.omega_mode && ws > u.omega_f;
        const bool take = acc && !to_w;
        const bool rej = ok && !acc;
        const double p = pow_m_tenth_scaled(fmin_k(fmax_k(z, 9.313225746154785e-10), 1.073741824e9), 0.9);
        const double lo = fmax_k(p, 0.2);
        if (__builtin_expect(__ballot(to_w) != 0, 0)) {
            const double s = to_w ? 1.0 / L.kw : 1.0;
#pragma unroll
            for (int i = 0; i < 3; ++i) L.k1[i] *= s;
            if (lane3) L.k1[0] = to_w ? 1.0 : L.k1[0];
            L.kw = to_w ? 1.0 : L.kw;
            L.dt1 = to_w ? s : L.dt1;
            L.nt = to_w ? L.acc : L.nt;
            L.h = to_w ? u.omega_f - L.w : L.h;
            L.last_rej = to_w ? false : L.last_rej;
            L.omega_mode = L.omega_mode || to_w;
        }
        if (RECORD && take) {
            if (lane3) tape_of(u, L.idx)[2 + L.acc] = h;
            if ((L.acc + 1) % u.ckpt_every == 0) checkpoint(u, L.idx, (L.acc + 1) / u.ckpt_every, q, T.Y);
        }
        const double tn = any_w && L.omega_mode ? __builtin_fma(h, T.dts, L.t) : L.t + h;
        const bool done = take && (last || (!L.omega_mode && ws == u.omega_f));
        if (take) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                L.v[i] = T.Y[i];
                L.k1[i] = T.k7[i];
            }
            L.w = ws;
            L.kw = T.kws;
            L.lnv = T.lnv;
            L.x = T.x;
            L.t = tn;
            L.dt1 = any_w ? T.dt7 : L.dt1;
            L.acc += 1;
            L.h = h * fmin_v(lo, L.last_rej ? 1.0 : 5.0);
            L.last_rej = false;
            if (PHASE) L.phase = __builtin_fma(h, T.ps, L.phase);
        }
        if (__builtin_expect(any_w, 0)) {
            if (done && L.omega_mode) {
                L.w = u.omega_f;
                L.v[0] = lane3 ? u.omega_f : L.v[0];
            }
        }
        if (__builtin_expect(__ballot(rej) != 0, 0)) {
            if (rej) {
                L.rej += 1;
                L.h = h * lo;
                L.last_rej = true;
                const double scale = L.omega_mode ? __builtin_fabs(L.w) : __builtin_fmax(1.0, __builtin_fabs(L.t));
                if (L.h < 1e-14 * scale) st = PN_ST_H_UNDERFLOW;
            }
        }
        return st != 0 ? st : (done ? 1 : 0);
    }
};

// A quad per inspiral, no refill: a wave runs until its longest inspiral ends.
// Bound by the instructions one wave issues for a step of its 16 inspirals
// (about 800 straight-line vector instructions, 190 of them permutations, and
// the step control; 4.8 cycles each for a wave alone on its SIMD).
// One wave a SIMD: blocks of four waves, the register count padded so that a
// CU takes one block (two blocks on one CU while others idle cost 690 instead
// of 450 us for 16,384 inspirals).
template <int BLOCK, bool RECORD, bool PHASE>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(1, 1)))
void integrate_quad_f64(Io io, Uni u) {
    using P = QuadF64<RECORD, PHASE>;
    const int64_t pos = ((int64_t)blockIdx.x * BLOCK + threadIdx.x) >> 2;
    const int q = threadIdx.x & 3;
    LaneQ L{};
    L.w = 1.0;                  // idle quads step on this state and discard the result
    L.range = kQuadRange;
    L.v[0] = q == 3 ? 1.0 : 0.0;
    PolyQ pc;
    make_poly(pc);
    bool active = false;
    if (pos < u.n) {
        const int64_t idx = io.order ? (int64_t)io.order[pos] : pos;
        if (idx >= 0 && idx < u.n) active = P::load(io, u, L, idx, q) == 0;
    }
    for (;;) {
        const uint64_t amask = __ballot(active);
        if (amask == 0) break;
        // inspirals in omega mode wait until all of the wave's are: their steps
        // (usually one) then take the general path once instead of one by one
        const bool run_w = __ballot(active && L.omega_mode) == amask;
        const bool act = active && (run_w || !L.omega_mode);
        const int r = P::step(u, pc, L, act, run_w, q);
        if (act && r != 0) {
            P::finish(io, u, L, r == 1 ? PN_ST_OK : r, q);
            active = false;
        }
    }
}

}  // namespace pn
