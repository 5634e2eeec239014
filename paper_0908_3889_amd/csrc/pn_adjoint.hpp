// pn_adjoint.hpp -- reverse-mode pieces of the discrete adjoint: the
// vector-Jacobian product of the right-hand side of Eqs. (1)-(4) (with
// respect to the state and to the 14-entry coefficient row), and the
// derivative of the coefficient row with respect to the masses.
#pragma once

#include "pn_device.hpp"

namespace pn {

// Adjoint of the coefficient row, accumulated over every stage of every step.
struct RowBar {
    double v[NROW];
};

// VJP of f = rhs(y) at y: given fbar = dL/df (10), writes (df/dy)^T fbar to
// ybar and adds (df/drow)^T fbar to rb.  The primal is recomputed here (same
// expansion as rhs()) but for x = (M omega)^{1/3} and lnv = ln|M omega|, which
// the replay's stage derivative left: 16 registers that the kernel has free,
// against 30 instructions.
//
// With Omega_1 = al1 L + be S2 and Omega_2 = al2 L + be S1, dS_i = Omega_i x
// S_i; the adjoint s_i of dS_i adds s_i x Omega_i to that of S_i and p_i = S_i x
// s_i to that of Omega_i, from which those of al_i, be, L and the other spin
// follow (18 operations fewer than through L x S1, L x S2 and S1 x S2).  The
// two took the adjoint of 65,536 inspirals from 1.66 to 1.58 ms.
//
// Omega mode: the stage derivative is g = (1, f_1/f_0, ..., f_9/f_0) with
// dt/domega = 1/f_0.  With omega_mode set, gbar (slot 0 unused) and gtbar
// (the weight of dt/domega) are first turned into fbar:
//   s = 1/f_0,  sbar = gtbar + sum_{c>=1} gbar_c f_c,
//   fbar_c = gbar_c s (c >= 1),  fbar_0 = -s^2 sbar.
//
// gscale multiplies gbar_in (the step size of the RK adjoint recurrence).
__device__ __forceinline__ void rhs_vjp(const Row& r, const TermConsts& tc, double x, double lnv,
                                        const double* __restrict__ y,
                                        const double* __restrict__ gbar_in, double gscale, double gtbar,
                                        bool omega_mode, double* __restrict__ ybar, RowBar& rb) {
    // ---------------- primal ----------------
    const double w = y[0];
    const double M = r[R_M];
    const double x2 = x * x;
    const double L0 = y[7], L1 = y[8], L2 = y[9];
    const double a0 = y[1], a1 = y[2], a2 = y[3];
    const double b0 = y[4], b1 = y[5], b2 = y[6];
    const double LS1 = __builtin_fma(L0, a0, __builtin_fma(L1, a1, L2 * a2));
    const double LS2 = __builtin_fma(L0, b0, __builtin_fma(L1, b1, L2 * b2));
    const double S12 = __builtin_fma(a0, b0, __builtin_fma(a1, b1, a2 * b2));
    const double c3p = __builtin_fma(-r[R_SO2], LS2, __builtin_fma(-r[R_SO1], LS1, tc.c3));
    const double ssb = __builtin_fma(247.0, S12, -721.0 * (LS1 * LS2));
    const double c4p = __builtin_fma(-r[R_SSD], ssb, r[R_C4]);
    const double c6p = __builtin_fma(tc.c6lnv, lnv, r[R_C6]);
    const double B5 = __builtin_fma(x, r[R_C7], c6p);
    const double B4 = __builtin_fma(x, B5, r[R_C5]);
    const double B3 = __builtin_fma(x, B4, c4p);
    const double B2 = __builtin_fma(x, B3, c3p);
    const double B1 = __builtin_fma(x, B2, r[R_C2]);
    const double B = __builtin_fma(x2, B1, 1.0);
    const double ww = w * w, wx2 = w * x2;
    const double Kww = r[R_K] * ww;
    const double f0 = Kww * wx2 * B;
    const double be = r[R_SIGM] * ww, m3be = -3.0 * be;
    const double al1 = __builtin_fma(r[R_G1], wx2, m3be * LS2), al2 = __builtin_fma(r[R_G2], wx2, m3be * LS1);
    const double q = -r[R_LAM] * x;

    // ---------------- seed fbar ----------------
    double fb[10];
    if (omega_mode) {
        const double u0 = __builtin_fma(L1, a2, -L2 * a1), u1 = __builtin_fma(L2, a0, -L0 * a2),
                     u2 = __builtin_fma(L0, a1, -L1 * a0);
        const double w0 = __builtin_fma(L1, b2, -L2 * b1), w1 = __builtin_fma(L2, b0, -L0 * b2),
                     w2 = __builtin_fma(L0, b1, -L1 * b0);
        const double C0 = __builtin_fma(a1, b2, -a2 * b1), C1 = __builtin_fma(a2, b0, -a0 * b2),
                     C2 = __builtin_fma(a0, b1, -a1 * b0);
        const double dS1_0 = __builtin_fma(al1, u0, -be * C0), dS1_1 = __builtin_fma(al1, u1, -be * C1),
                     dS1_2 = __builtin_fma(al1, u2, -be * C2);
        const double dS2_0 = __builtin_fma(al2, w0, be * C0), dS2_1 = __builtin_fma(al2, w1, be * C1),
                     dS2_2 = __builtin_fma(al2, w2, be * C2);
        const double s = 1.0 / f0;
        double sbar = 0.0;
        sbar = __builtin_fma(gbar_in[1], dS1_0, sbar);
        sbar = __builtin_fma(gbar_in[2], dS1_1, sbar);
        sbar = __builtin_fma(gbar_in[3], dS1_2, sbar);
        sbar = __builtin_fma(gbar_in[4], dS2_0, sbar);
        sbar = __builtin_fma(gbar_in[5], dS2_1, sbar);
        sbar = __builtin_fma(gbar_in[6], dS2_2, sbar);
        sbar = __builtin_fma(gbar_in[7], q * (dS1_0 + dS2_0), sbar);
        sbar = __builtin_fma(gbar_in[8], q * (dS1_1 + dS2_1), sbar);
        sbar = __builtin_fma(gbar_in[9], q * (dS1_2 + dS2_2), sbar);
        sbar = __builtin_fma(gscale, sbar, gtbar);
        const double gs = gscale * s;
#pragma unroll
        for (int c = 1; c < 10; ++c) fb[c] = gbar_in[c] * gs;
        fb[0] = -(s * s) * sbar;
    } else {
#pragma unroll
        for (int c = 0; c < 10; ++c) fb[c] = gbar_in[c] * gscale;
    }

    // ---------------- reverse ----------------
    const double O1_0 = __builtin_fma(al1, L0, be * b0), O1_1 = __builtin_fma(al1, L1, be * b1),
                 O1_2 = __builtin_fma(al1, L2, be * b2);
    const double O2_0 = __builtin_fma(al2, L0, be * a0), O2_1 = __builtin_fma(al2, L1, be * a1),
                 O2_2 = __builtin_fma(al2, L2, be * a2);
    const double s1b0 = __builtin_fma(q, fb[7], fb[1]), s1b1 = __builtin_fma(q, fb[8], fb[2]),
                 s1b2 = __builtin_fma(q, fb[9], fb[3]);
    const double s2b0 = __builtin_fma(q, fb[7], fb[4]), s2b1 = __builtin_fma(q, fb[8], fb[5]),
                 s2b2 = __builtin_fma(q, fb[9], fb[6]);
    // dL = q (dS1 + dS2) = q L x (al1 S1 + al2 S2)
    const double qbar = __builtin_fma(__builtin_fma(al1, a0, al2 * b0), __builtin_fma(fb[8], L2, -fb[9] * L1),
                        __builtin_fma(__builtin_fma(al1, a1, al2 * b1), __builtin_fma(fb[9], L0, -fb[7] * L2),
                                      __builtin_fma(al1, a2, al2 * b2) * __builtin_fma(fb[7], L1, -fb[8] * L0)));
    // q = -lam x
    rb.v[R_LAM] = __builtin_fma(-x, qbar, rb.v[R_LAM]);
    double xbar = -r[R_LAM] * qbar;
    const double p1_0 = __builtin_fma(a1, s1b2, -a2 * s1b1), p1_1 = __builtin_fma(a2, s1b0, -a0 * s1b2),
                 p1_2 = __builtin_fma(a0, s1b1, -a1 * s1b0);
    const double p2_0 = __builtin_fma(b1, s2b2, -b2 * s2b1), p2_1 = __builtin_fma(b2, s2b0, -b0 * s2b2),
                 p2_2 = __builtin_fma(b0, s2b1, -b1 * s2b0);
    const double al1b = __builtin_fma(p1_0, L0, __builtin_fma(p1_1, L1, p1_2 * L2));
    const double al2b = __builtin_fma(p2_0, L0, __builtin_fma(p2_1, L1, p2_2 * L2));
    const double beb = __builtin_fma(p1_0, b0, __builtin_fma(p1_1, b1, __builtin_fma(p1_2, b2,
                       __builtin_fma(p2_0, a0, __builtin_fma(p2_1, a1, p2_2 * a2)))));
    double ab0 = __builtin_fma(be, p2_0, __builtin_fma(s1b1, O1_2, -s1b2 * O1_1)),
           ab1 = __builtin_fma(be, p2_1, __builtin_fma(s1b2, O1_0, -s1b0 * O1_2)),
           ab2 = __builtin_fma(be, p2_2, __builtin_fma(s1b0, O1_1, -s1b1 * O1_0));
    double bb0 = __builtin_fma(be, p1_0, __builtin_fma(s2b1, O2_2, -s2b2 * O2_1)),
           bb1 = __builtin_fma(be, p1_1, __builtin_fma(s2b2, O2_0, -s2b0 * O2_2)),
           bb2 = __builtin_fma(be, p1_2, __builtin_fma(s2b0, O2_1, -s2b1 * O2_0));
    double Lb0 = __builtin_fma(al1, p1_0, al2 * p2_0), Lb1 = __builtin_fma(al1, p1_1, al2 * p2_1),
           Lb2 = __builtin_fma(al1, p1_2, al2 * p2_2);
    // al1 = g1 wx2 - 3 be LS2 ; al2 = g2 wx2 - 3 be LS1
    rb.v[R_G1] = __builtin_fma(wx2, al1b, rb.v[R_G1]);
    rb.v[R_G2] = __builtin_fma(wx2, al2b, rb.v[R_G2]);
    double wx2bar = __builtin_fma(r[R_G1], al1b, r[R_G2] * al2b);
    double LS2bar = m3be * al1b;
    double LS1bar = m3be * al2b;
    // be = sigM ww
    const double bebar = __builtin_fma(-3.0, __builtin_fma(LS2, al1b, LS1 * al2b), beb);
    rb.v[R_SIGM] = __builtin_fma(ww, bebar, rb.v[R_SIGM]);
    // f0 = K ww wx2 B
    const double f0b = fb[0];
    const double wB = wx2 * B;
    rb.v[R_K] = __builtin_fma(ww * wB, f0b, rb.v[R_K]);
    const double wwbar = __builtin_fma(r[R_K] * wB, f0b, r[R_SIGM] * bebar);
    const double Kf = Kww * f0b;
    wx2bar = __builtin_fma(Kf, B, wx2bar);
    const double Bbar = Kf * wx2;
    // wx2 = w x2, ww = w w
    double wbar = __builtin_fma(x2, wx2bar, 2.0 * w * wwbar);
    double x2bar = w * wx2bar;
    // B = 1 + x2 B1
    x2bar = __builtin_fma(B1, Bbar, x2bar);
    const double B1b = x2 * Bbar;
    // Horner chain
    xbar = __builtin_fma(B2, B1b, xbar);
    rb.v[R_C2] += B1b;
    const double B2b = x * B1b;
    xbar = __builtin_fma(B3, B2b, xbar);
    const double c3pb = B2b;
    const double B3b = x * B2b;
    xbar = __builtin_fma(B4, B3b, xbar);
    const double c4pb = B3b;
    const double B4b = x * B3b;
    xbar = __builtin_fma(B5, B4b, xbar);
    rb.v[R_C5] += B4b;
    const double B5b = x * B4b;
    xbar = __builtin_fma(r[R_C7], B5b, xbar);
    rb.v[R_C7] = __builtin_fma(x, B5b, rb.v[R_C7]);
    const double c6pb = B5b;
    // c6p = c6 + c6lnv lnv
    rb.v[R_C6] += c6pb;
    const double lnvbar = tc.c6lnv * c6pb;
    // c4p = c4 - ssd ssb ; ssb = 247 S12 - 721 LS1 LS2
    rb.v[R_C4] += c4pb;
    rb.v[R_SSD] = __builtin_fma(-ssb, c4pb, rb.v[R_SSD]);
    const double ssbb = -r[R_SSD] * c4pb;
    const double S12bar = 247.0 * ssbb;
    LS1bar = __builtin_fma(-721.0 * LS2, ssbb, LS1bar);
    LS2bar = __builtin_fma(-721.0 * LS1, ssbb, LS2bar);
    // c3p = c3 - so1 LS1 - so2 LS2
    rb.v[R_SO1] = __builtin_fma(-LS1, c3pb, rb.v[R_SO1]);
    rb.v[R_SO2] = __builtin_fma(-LS2, c3pb, rb.v[R_SO2]);
    LS1bar = __builtin_fma(-r[R_SO1], c3pb, LS1bar);
    LS2bar = __builtin_fma(-r[R_SO2], c3pb, LS2bar);
    // LS1 = L.a ; LS2 = L.b ; S12 = a.b
    Lb0 = __builtin_fma(a0, LS1bar, __builtin_fma(b0, LS2bar, Lb0));
    Lb1 = __builtin_fma(a1, LS1bar, __builtin_fma(b1, LS2bar, Lb1));
    Lb2 = __builtin_fma(a2, LS1bar, __builtin_fma(b2, LS2bar, Lb2));
    ab0 = __builtin_fma(L0, LS1bar, __builtin_fma(b0, S12bar, ab0));
    ab1 = __builtin_fma(L1, LS1bar, __builtin_fma(b1, S12bar, ab1));
    ab2 = __builtin_fma(L2, LS1bar, __builtin_fma(b2, S12bar, ab2));
    bb0 = __builtin_fma(L0, LS2bar, __builtin_fma(a0, S12bar, bb0));
    bb1 = __builtin_fma(L1, LS2bar, __builtin_fma(a1, S12bar, bb1));
    bb2 = __builtin_fma(L2, LS2bar, __builtin_fma(a2, S12bar, bb2));
    // x2 = x x ; lnv = ln|v| ; x = cbrt(v) ; v = M w
    xbar = __builtin_fma(2.0 * x, x2bar, xbar);
    // d lnv/dv = 1/v, dx/dv = 1/(3 x^2) = x/(3 v): one reciprocal of v
    // (hardware seed and two Newton steps; valid for either sign)
    const double v = M * w;
    const double rv = rcp_pos(v);
    const double vbar = rv * __builtin_fma(xbar, x * (1.0 / 3.0), lnvbar);
    rb.v[R_M] = __builtin_fma(w, vbar, rb.v[R_M]);
    wbar = __builtin_fma(M, vbar, wbar);

    ybar[0] = wbar;
    ybar[1] = ab0; ybar[2] = ab1; ybar[3] = ab2;
    ybar[4] = bb0; ybar[5] = bb1; ybar[6] = bb2;
    ybar[7] = Lb0; ybar[8] = Lb1; ybar[9] = Lb2;
}

// ---------------------------------------------------------------------------
// d(row)/d(m1), d(row)/d(m2): make_row() evaluated on dual numbers.
// ---------------------------------------------------------------------------
struct Dl {
    double v, d;
    __device__ Dl() : v(0), d(0) {}
    __device__ Dl(double a) : v(a), d(0) {}
    __device__ Dl(double a, double b) : v(a), d(b) {}
};
__device__ __forceinline__ Dl operator+(Dl a, Dl b) { return Dl(a.v + b.v, a.d + b.d); }
__device__ __forceinline__ Dl operator-(Dl a, Dl b) { return Dl(a.v - b.v, a.d - b.d); }
__device__ __forceinline__ Dl operator-(Dl a) { return Dl(-a.v, -a.d); }
__device__ __forceinline__ Dl operator*(Dl a, Dl b) { return Dl(a.v * b.v, a.d * b.v + a.v * b.d); }
__device__ __forceinline__ Dl operator/(Dl a, Dl b) {
    const double q = a.v / b.v;
    return Dl(q, (a.d - q * b.d) / b.v);
}
__device__ __forceinline__ Dl operator*(double a, Dl b) { return Dl(a * b.v, a * b.d); }
__device__ __forceinline__ Dl operator*(Dl a, double b) { return Dl(a.v * b, a.d * b); }
__device__ __forceinline__ Dl operator+(double a, Dl b) { return Dl(a + b.v, b.d); }
__device__ __forceinline__ Dl operator/(Dl a, double b) { return Dl(a.v / b, a.d / b); }
__device__ __forceinline__ Dl operator/(double a, Dl b) { return Dl(a) / b; }

struct RowDual {
    Dl v[NROW];
    __device__ __forceinline__ void set(int i, Dl x) { v[i] = x; }
};

// make_row() again, written on dual numbers (same expressions).
__device__ __forceinline__ void make_row_dual(RowDual& r, Dl m1, Dl m2, int terms, int theta_literal) {
    const Dl M = m1 + m2;
    const Dl iM = 1.0 / M;
    const Dl eta = m1 * m2 * iM * iM;
    const double pn = (terms & PN_TERM_PN) ? 1.0 : 0.0;
    const double fso = (terms & PN_TERM_SO_WDOT) ? 1.0 : 0.0;
    const double fss = (terms & PN_TERM_SS_WDOT) ? 1.0 : 0.0;
    r.set(R_M, M);
    r.set(R_C2, pn * ((-(743.0 + 924.0 * eta)) / 336.0));
    r.set(R_SO1, fso * ((113.0 * m1 * m1 * iM * iM + 75.0 * eta) / (12.0 * m1 * m1)));
    r.set(R_SO2, fso * ((113.0 * m2 * m2 * iM * iM + 75.0 * eta) / (12.0 * m2 * m2)));
    r.set(R_C4, pn * (34103.0 / 18144.0 + (13661.0 / 2016.0) * eta + (59.0 / 18.0) * eta * eta));
    r.set(R_SSD, fss * (eta / (48.0 * m1 * m1 * m2 * m2)));
    r.set(R_C5, pn * ((-(4159.0 + 15876.0 * eta)) * (PN_PI / 672.0)));
    const Dl theta_term = (88.0 / 3.0) * (1039.0 / 4620.0) * (theta_literal ? eta : Dl(1.0));
    const double c6c = (16447322263.0 / 139708800.0) - (1712.0 / 105.0) * PN_GAMMA_E + (16.0 / 3.0) * PN_PI * PN_PI
                     - (856.0 / 105.0) * PN_LN16;
    r.set(R_C6, pn * (c6c + (-273811877.0 / 1088640.0 + (451.0 / 48.0) * PN_PI * PN_PI - theta_term) * eta
                      + (541.0 / 896.0) * eta * eta - (5605.0 / 2592.0) * eta * eta * eta));
    r.set(R_C7, pn * ((-4415.0 / 4032.0 + (358675.0 / 6048.0) * eta + (91495.0 / 1512.0) * eta * eta) * PN_PI));
    r.set(R_K, (terms & PN_TERM_RR) ? (96.0 / 5.0) * eta * M : Dl(0.0));
    r.set(R_G1, (terms & PN_TERM_SO_PREC) ? 0.5 * (eta * (4.0 + 3.0 * m2 / m1)) : Dl(0.0));
    r.set(R_G2, (terms & PN_TERM_SO_PREC) ? 0.5 * (eta * (4.0 + 3.0 * m1 / m2)) : Dl(0.0));
    r.set(R_SIGM, (terms & PN_TERM_SS_PREC) ? 0.5 * iM : Dl(0.0));
    r.set(R_LAM, 1.0 / (eta * M * M));
}

__device__ __forceinline__ Dl operator-(double a, Dl b) { return Dl(a - b.v, -b.d); }

}  // namespace pn
