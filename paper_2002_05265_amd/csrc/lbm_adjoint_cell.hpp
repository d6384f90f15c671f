// Hand-written reverse mode of the per-cell collision in lbm_cell.hpp.
//
// Given mu = dL/dh* (the adjoint of the post-collision populations), collide_adjoint returns
// hb = dL/dh = J_C(h)^T mu and the adjoints of the relaxation coefficients.  The forward pass is
// recomputed step by step (the "tape" lives in registers) and every statement of collide is then
// reversed in the opposite order:
//
//   F1 sums of h, drho, jx, jy             R1 hb_i = mu_i + their adjoints at population i
//   F2 rho, du, u                          R2 quotient rule, u = U + du
//   F3 equilibrium differences, chained    R3 the chain in the opposite order
//   F4 d = moments of h - E                R4 (linear)
//   F5 D = relax_model(d, u, rho, coef)    R5 per-model reverse
//   F6 h* = h + P(D)                       R6 transpose of P
//
// As in the collision only the changes D are carried back, so the identity part of J_C is added at the end
// and nothing of the equilibrium but its derivative is needed.  What bounds the reverse kernels is the vector
// ALU: 304 instructions per node in FP32 for CM, 266 in FP64 (441 and 412 with
// the whole equilibrium carried back).
//
// Coefficient adjoints cb = (kpp, cpm, k11, k21, k12, k22, om), where c21, c12 and c22 = 1 + k count with their k, map to
// the rates by omega_adjoint: d/domega_nu = -kpp/2 + cpm/2 - k11 + om, d/domega_b = -kpp/2 - cpm/2, d/domega_21 =
// -k21, d/domega_12 = -k12, d/domega_22 = -k22.
#pragma once

#include "lbm_cell.hpp"

namespace lbm {

template <typename R> struct MacroBar {
    R drho, rho, jx, jy, ux, uy, dux, duy;
};

template <typename R>
__device__ __forceinline__ void zero(MacroBar<R>& b) {
    b.drho = b.rho = b.jx = b.jy = b.ux = b.uy = b.dux = b.duy = R(0);
}

// Transpose of hermite_to_pop.  Outputs the adjoints of drho, jx, jy and of the six
// post-collision Hermite differences a20 .. a22.
template <typename R>
__device__ __forceinline__ void pop_adjoint(const R (&mu)[9], MacroBar<R>& mb, R (&ab)[6]) {
    using L = Lat<R>;
    const R r0b = mu[0];
    const R r1b = (mu[1] + mu[3]) + (mu[2] + mu[4]);
    const R r5b = (mu[5] + mu[6]) + (mu[7] + mu[8]);
    const R hxb = mu[1] + mu[3], pxb = mu[1] - mu[3];
    const R hyb = mu[2] + mu[4], pyb = mu[2] - mu[4];
    const R qb = r5b;
    const R s11b = (mu[5] + mu[7]) - (mu[6] + mu[8]);
    const R s12b = (mu[5] + mu[8]) - (mu[6] + mu[7]);
    const R s21b = (mu[5] + mu[6]) - (mu[7] + mu[8]);
    const R M22b = mu[0] - R(0.5) * (hxb + hyb) + R(0.25) * qb;
    const R M20b = R(0.5) * hxb - mu[0];
    const R M02b = R(0.5) * hyb - mu[0];
    const R M12b = R(0.25) * s12b - R(0.5) * pxb;
    const R M21b = R(0.25) * s21b - R(0.5) * pyb;
    const R M11b = R(0.25) * s11b;
    mb.jx += R(0.5) * pxb + L::cs2 * M12b;
    mb.jy += R(0.5) * pyb + L::cs2 * M21b;
    mb.drho += L::w0 * r0b + L::w1 * r1b + L::w5 * r5b;
    ab[0] = M20b + L::cs2 * M22b;  // a20
    ab[1] = M02b + L::cs2 * M22b;  // a02
    ab[2] = M11b;                  // a11
    ab[3] = M21b;                  // a21
    ab[4] = M12b;                  // a12
    ab[5] = M22b;                  // a22
}

// Reverse of hermite_eq.  eb = adjoints of (e20, e02, e11, e21, e12, e22).
template <typename R>
__device__ __forceinline__ void eq_adjoint(const Macro<R>& m, const Ref<R>& r, int N, const R (&eb)[6],
                                           MacroBar<R>& mb) {
    const R a = m.ux, b = m.uy, A = r.ux, da = m.dux, db = m.duy, dr = m.drho, rs = r.rho;
    const R a2 = a * a, b2 = b * b;
    const R D20 = da * (a + A);
    const R D02 = db * (b + r.uy);
    const R e20b = eb[0], e02b = eb[1], e11b = eb[2];
    const R e21b = N >= 3 ? eb[3] : R(0), e12b = N >= 3 ? eb[4] : R(0), e22b = N >= 4 ? eb[5] : R(0);
    // direct drho terms
    mb.drho += e20b * a2 + e02b * b2 + e11b * (a * b) + e21b * (a2 * b) + e12b * (a * b2) + e22b * (a2 * b2);
    R ab = dr * (R(2) * a * e20b + b * e11b + R(2) * a * b * e21b + b2 * e12b + R(2) * a * b2 * e22b);
    R bb = dr * (R(2) * b * e02b + a * e11b + a2 * e21b + R(2) * a * b * e12b + R(2) * a2 * b * e22b);
    // reference-difference terms
    const R D22b = rs * e22b, D21b = rs * e21b, D12b = rs * e12b, D11b = rs * e11b;
    const R D20b = rs * e20b + b * D21b + b2 * D22b;
    const R D02b = rs * e02b + A * D12b + (A * A) * D22b;
    R dab = R(0), dbb = R(0);
    bb += D20 * D21b;                 // D21 = D20 b + A^2 db
    dbb += (A * A) * D21b;
    dab += b2 * D12b;                 // D12 = da b^2 + A D02
    bb += R(2) * da * b * D12b;
    bb += R(2) * b * D20 * D22b;      // D22 = D20 b^2 + A^2 D02
    dab += b * D11b;                  // D11 = da b + A db
    bb += da * D11b;
    dbb += A * D11b;
    dab += (a + A) * D20b;            // D20 = da (a + A)
    ab += da * D20b;
    dbb += (b + r.uy) * D02b;         // D02 = db (b + B)
    bb += db * D02b;
    mb.ux += ab;
    mb.uy += bb;
    mb.dux += dab;
    mb.duy += dbb;
}

// Reverse of the whole collision of one cell.  cb: adjoints of (kpp, cpm, k11, k21, k12, k22, om) (those
// the model does not have are zero).
template <int MODEL, typename R>
__device__ __forceinline__ void collide_adjoint(const R (&h)[9], const Macro<R>& m, const Ref<R>& ref,
                                                const Coef<R>& c, int N, const R (&mu)[9], R (&hb)[9],
                                                R (&cb)[7]) {
    using L = Lat<R>;
#pragma unroll
    for (int k = 0; k < 7; ++k) cb[k] = R(0);
    if constexpr (MODEL == kStreamOnly) {
#pragma unroll
        for (int i = 0; i < 9; ++i) hb[i] = mu[i];
        return;
    } else {
        constexpr bool kShifted = sizeof(R) == 4;
        constexpr bool kCentral = MODEL == kCM || MODEL == kCHM || MODEL == kK;
        constexpr bool kRawX = MODEL == kBGK || MODEL == kRM || MODEL == kCM;  // as in collide
        const R ux = m.ux, uy = m.uy;
        // F3, F4
        R e20 = m.jx * ux, e02 = m.jy * uy;
        R d11 = fmadd(-m.jx, uy, m.s.m11);
        if constexpr (kShifted) {
            e20 = fmadd(ref.jx, m.dux, e20);
            e02 = fmadd(ref.jy, m.duy, e02);
            d11 = fmadd(-ref.jx, m.duy, d11);
        }
        const R a20 = fmadd(-L::cs2, m.drho, m.s.s13 + m.s.m22);
        const R a02 = fmadd(-L::cs2, m.drho, m.s.s24 + m.s.m22);
        const R d20 = a20 - e20, d02 = a02 - e02;
        R d21 = fmadd(-L::cs2, m.jy, m.s.m21);
        R d12 = fmadd(-L::cs2, m.jx, m.s.m12);
        R d22 = fmadd(-L::cs2, kRawX ? e20 + e02 : a20 + a02, fmadd(-L::cs4, m.drho, m.s.m22));
        R e21 = R(0);
        if (kCentral || N >= 3) {
            e21 = e20 * uy;
            d12 = fmadd(-e02, ux, d12);
            if constexpr (kShifted) {
                e21 = fmadd(ref.a20, m.duy, e21);
                d12 = fmadd(-ref.a02, m.dux, d12);
            }
            d21 = d21 - e21;
            if (kCentral || N >= 4) {
                d22 = fmadd(-e21, uy, d22);
                if constexpr (kShifted) d22 = fmadd(-ref.a21, m.duy, d22);
            }
        }
        // R6: adjoints of the changes
        const Sums<R> w = sums_of(mu);
        R D20b = fmadd(R(0.5), w.s13, -mu[0]);
        R D02b = fmadd(R(0.5), w.s24, -mu[0]);
        R D11b = R(0.25) * w.m11;
        R D21b = fmadd(R(0.25), w.m21, R(-0.5) * w.d24);
        R D12b = fmadd(R(0.25), w.m12, R(-0.5) * w.d13);
        const R M22b = fmadd(R(-0.5), w.s13 + w.s24, fmadd(R(0.25), w.m22, mu[0]));
        // R5: adjoints of d (and of u and, in K, of 1 / rho)
        R d20b, d02b, d11b, d21b, d12b, d22b, uxb = R(0), uyb = R(0), invb = R(0);
        if constexpr (MODEL == kBGK) {
            d20b = -c.om * D20b;
            d02b = -c.om * D02b;
            d11b = -c.om * D11b;
            d21b = -c.om * D21b;
            d12b = -c.om * D12b;
            d22b = -c.om * M22b;
            cb[6] = -fmadd(d20, D20b, fmadd(d02, D02b, fmadd(d11, D11b, fmadd(d21, D21b, fmadd(d12, D12b, d22 * M22b)))));
        } else {
            d20b = d02b = d11b = R(0);
            if constexpr (MODEL == kHM || MODEL == kRM) {
                d21b = c.k21 * D21b;
                d12b = c.k12 * D12b;
                d22b = c.k22 * M22b;
                cb[3] = d21 * D21b;
                cb[4] = d12 * D12b;
                cb[5] = d22 * M22b;
            } else if constexpr (MODEL == kPR) {
                d21b = -D21b;
                d12b = -D12b;
                d22b = -M22b;
            } else if constexpr (MODEL == kRR) {
                const R f11 = d11 + d11;
                const R r21 = fmadd(ux, f11, uy * d20);
                const R r12 = fmadd(uy, f11, ux * d02);
                const R r22 = fmadd(ux, r12, uy * r21);
                d21b = -D21b;
                d12b = -D12b;
                d22b = -M22b;
                cb[3] = r21 * D21b;
                cb[4] = r12 * D12b;
                cb[5] = r22 * M22b;
                const R r22b = c.c22 * M22b;
                const R r21b = fmadd(uy, r22b, c.c21 * D21b);
                const R r12b = fmadd(ux, r22b, c.c12 * D12b);
                uxb = fmadd(r12, r22b, fmadd(f11, r21b, d02 * r12b));
                uyb = fmadd(r21, r22b, fmadd(f11, r12b, d20 * r21b));
                d20b = uy * r21b;
                d02b = ux * r12b;
                const R f11b = fmadd(ux, r21b, uy * r12b);
                d11b = f11b + f11b;
            } else {
                const R vx = ux + ux, vy = uy + uy;
                const R t21 = fmadd(-vx, d11, fmadd(-uy, d20, d21));
                const R t12 = fmadd(-vy, d11, fmadd(-ux, d02, d12));
                const R q21 = d21 + t21, q12 = d12 + t12;
                const R t22 = fmadd(-ux, q12, fmadd(-uy, q21, d22));
                const R D20 = fmadd(c.kpp, d20, c.cpm * d02);
                const R D02 = fmadd(c.kpp, d02, c.cpm * d20);
                const R D11 = c.k11 * d11;
                const R s21 = c.k21 * t21, s12 = c.k12 * t12;
                const R D21 = fmadd(vx, D11, fmadd(uy, D20, s21));
                const R D12 = fmadd(vy, D11, fmadd(ux, D02, s12));
                // M22 = s22 + uy (s21 + D21) + ux (s12 + D12)
                const R gy = uy * M22b, gx = ux * M22b;
                D21b += gy;
                D12b += gx;
                const R s21b = gy + D21b, s12b = gx + D12b;
                const R g11 = D11 + D11;
                uyb = fmadd(s21 + D21, M22b, fmadd(D20, D21b, g11 * D12b));
                uxb = fmadd(s12 + D12, M22b, fmadd(D02, D12b, g11 * D21b));
                D20b = fmadd(uy, D21b, D20b);
                D02b = fmadd(ux, D12b, D02b);
                D11b = fmadd(vx, D21b, fmadd(vy, D12b, D11b));
                const R t22b = c.k22 * M22b;
                if constexpr (MODEL == kK) {
                    const R n20 = d20 + D20, n02 = d02 + D02, n11 = d11 + D11;
                    const R p = fmadd(d11 + d11, d11, d20 * d02);
                    const R q = fmadd(n11 + n11, n11, n20 * n02);
                    cb[5] = fmadd(-p, m.inv_rho, t22) * M22b;
                    invb = fmadd(-c.c22, p, q) * M22b;
                    const R qb = m.inv_rho * M22b, pb = -c.c22 * qb;
                    const R n20b = qb * n02, n02b = qb * n20, n11b = (R(4) * qb) * n11;
                    D20b += n20b;
                    D02b += n02b;
                    D11b += n11b;
                    d20b = fmadd(pb, d02, n20b);
                    d02b = fmadd(pb, d20, n02b);
                    d11b = fmadd(R(4) * pb, d11, n11b);
                } else {
                    cb[5] = t22 * M22b;
                }
                cb[3] = t21 * s21b;
                cb[4] = t12 * s12b;
                // t22 = d22 - uy (d21 + t21) - ux (d12 + t12)
                d22b = t22b;
                const R ky = uy * t22b, kx = ux * t22b;
                const R t21b = fmadd(c.k21, s21b, -ky), t12b = fmadd(c.k12, s12b, -kx);
                d21b = t21b - ky;
                d12b = t12b - kx;
                uyb = fmadd(-q21, t22b, uyb);
                uxb = fmadd(-q12, t22b, uxb);
                // t21 = d21 - uy d20 - 2 ux d11, t12 = d12 - ux d02 - 2 uy d11
                const R f11 = d11 + d11;
                d20b = fmadd(-uy, t21b, d20b);
                d02b = fmadd(-ux, t12b, d02b);
                d11b = fmadd(-vx, t21b, fmadd(-vy, t12b, d11b));
                uyb = fmadd(-d20, t21b, fmadd(-f11, t12b, uyb));
                uxb = fmadd(-d02, t12b, fmadd(-f11, t21b, uxb));
            }
            if constexpr (!kRawX) {  // M22 has cs^2 (D20 + D02)
                D20b = fmadd(L::cs2, M22b, D20b);
                D02b = fmadd(L::cs2, M22b, D02b);
            }
            // second-order block, common to every moment space
            d20b = fmadd(c.kpp, D20b, fmadd(c.cpm, D02b, d20b));
            d02b = fmadd(c.kpp, D02b, fmadd(c.cpm, D20b, d02b));
            d11b = fmadd(c.k11, D11b, d11b);
            cb[0] = fmadd(D20b, d20, D02b * d02);
            cb[1] = fmadd(D20b, d02, D02b * d20);
            cb[2] = D11b * d11;
        }
        // R4, R3
        R A20b = d20b, A02b = d02b, e20b = -d20b, e02b = -d02b;
        if constexpr (kRawX) {
            e20b = fmadd(-L::cs2, d22b, e20b);
            e02b = fmadd(-L::cs2, d22b, e02b);
        } else {
            A20b = fmadd(-L::cs2, d22b, A20b);
            A02b = fmadd(-L::cs2, d22b, A02b);
        }
        R duxb = R(0), duyb = R(0);
        if (kCentral || N >= 3) {
            R e21b = -d21b;
            if (kCentral || N >= 4) {
                e21b = fmadd(-uy, d22b, e21b);
                uyb = fmadd(-e21, d22b, uyb);
                if constexpr (kShifted) duyb = -ref.a21 * d22b;
            }
            e20b = fmadd(uy, e21b, e20b);
            uyb = fmadd(e20, e21b, uyb);
            e02b = fmadd(-ux, d12b, e02b);
            uxb = fmadd(-e02, d12b, uxb);
            if constexpr (kShifted) {
                duyb = fmadd(ref.a20, e21b, duyb);
                duxb = -ref.a02 * d12b;
            }
        }
        R jxb = fmadd(ux, e20b, fmadd(-uy, d11b, -L::cs2 * d12b));
        R jyb = fmadd(uy, e02b, -L::cs2 * d21b);
        uxb = fmadd(m.jx, e20b, uxb);
        uyb = fmadd(m.jy, e02b, fmadd(-m.jx, d11b, uyb));
        if constexpr (kShifted) {
            duxb = fmadd(ref.jx, e20b, duxb);
            duyb = fmadd(ref.jy, e02b, fmadd(-ref.jx, d11b, duyb));
        }
        const R A22b = A20b + A02b;
        R drhob = fmadd(-L::cs4, d22b, -L::cs2 * A22b);
        // R2: u = U + du, du = (j - drho U) / rho, rho = rho_s + drho
        const R tx = (duxb + uxb) * m.inv_rho, ty = (duyb + uyb) * m.inv_rho;
        jxb += tx;
        jyb += ty;
        if constexpr (kShifted) drhob = fmadd(-ref.ux, tx, fmadd(-ref.uy, ty, drhob));
        drhob = fmadd(-m.dux, tx, fmadd(-m.duy, ty, drhob));
        if constexpr (MODEL == kK) drhob = fmadd(-(m.inv_rho * m.inv_rho), invb, drhob);
        // R1
        const R xb = drhob + A20b, yb = drhob + A02b, zb = drhob + (d22b + A22b);
        const R m12b = d12b + jxb, m21b = d21b + jyb;
        const R P = zb + d11b, Q = zb - d11b, S = m12b + m21b, T = m12b - m21b;
        hb[0] = mu[0] + drhob;
        hb[1] = mu[1] + (xb + jxb);
        hb[3] = mu[3] + (xb - jxb);
        hb[2] = mu[2] + (yb + jyb);
        hb[4] = mu[4] + (yb - jyb);
        hb[5] = mu[5] + (P + S);
        hb[7] = mu[7] + (P - S);
        hb[6] = mu[6] + (Q - T);
        hb[8] = mu[8] + (Q + T);
    }
}

// Adds the adjoints of the five rates, from the coefficient adjoints, to ws.
template <int MODEL, typename R>
__device__ __forceinline__ void omega_adjoint(const R (&cb)[7], double (&ws)[5]) {
    if constexpr (MODEL == kStreamOnly) {
        return;
    } else if constexpr (MODEL == kBGK) {
        ws[0] += (double)cb[6];
    } else {
        const double p = (double)cb[0], q = (double)cb[1];
        ws[0] += fma(0.5, q - p, -(double)cb[2]);
        ws[1] = fma(-0.5, p + q, ws[1]);
        if constexpr (MODEL != kPR) {
            ws[2] -= (double)cb[3];
            ws[3] -= (double)cb[4];
            ws[4] -= (double)cb[5];
        }
    }
}

}  // namespace lbm
