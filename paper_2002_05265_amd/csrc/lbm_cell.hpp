// Per-cell D2Q9 collision for gfx950: moment transform -> relax -> back-transform, in registers.
//
// Every model of Appendix B (BGK, RM, HM, CM, CHM, K, PR, RR) is written here in one common
// "deviation" form so that the same code runs in FP64 and in FP32 on shifted populations:
//
//   stored value   h_i   = f_i - f^ref_i,  f^ref = f^eq_N(rho_s, U)   (a fixed reference state;
//                                           rho_s = 0, U = 0 for plain FP64 storage)
//   density        rho   = rho_s + drho,   drho = sum_i h_i
//   velocity       u     = U + du,         du = (sum_i xi_i h_i - drho U) / rho
//   every equilibrium moment enters as its difference to the reference, built from drho and du,
//   so each quantity carried through the transform is O(du), O(drho) or O(f^neq), never O(rho).
//
// Map used by every model (the pipeline of Appendix B):
//   1. h -> raw moments (eq. RMcoll definition) -> Hermite non-equilibrium d_pq = A_pq - A^eq_pq
//   2. relax d in the model's own space (RM: raw, HM/PR: Hermite, RR: recursive Hermite
//      (eq. RRformulas_D2Q9), CHM/CM/K: central (Hermite) moments obtained by the binomial shift
//      by -u of d, whose inverse is eq. CHM2HM_Q9)
//   3. back to populations (eq. HM2RM_Q9, eq. Q9postCollVDF_RM).  Every map is linear and the density
//      and momentum do not change, so only the *changes* D_pq = d*_pq - d_pq are carried back and
//      added to the stored values: h* = h + P(D).
//
// The arithmetic is what bounds the fused kernels (vector-ALU issue in FP32 and FP16, see
// lbm_step3.hpp), so it is written for few operations:
//   - the equilibrium differences are chained through the momentum of the deviations,
//       rho a^2 - rho_s A^2     = jx a + rho_s A (a - A),       jx = rho a - rho_s A,
//       rho a^2 b - rho_s A^2 B = E20 b + rho_s A^2 (b - B),    rho a^2 b^2 - ... = E21 b + rho_s A^2 B (b - B)
//     (two operations each; every factor stays a deviation, so nothing of order one cancels), and the
//     constants rho_s A, rho_s A^2, ... come precomputed in Ref;
//   - P(D) needs neither the equilibrium nor the conserved moments;
//   - the central shifts are chained through the third order: t22 = d22 - uy (d21 + t21) - ux (d12 + t12);
//   - BGK, RM and CM relax the raw fourth moment X = d22 + cs^2 (d20 + d02), which is also what P takes.
// Relaxation vector (omega_nu, omega_b, omega_21, omega_12, omega_22): deviatoric and trace
// parts of the second-order block, then the two third-order and the fourth-order moment.
// The paper's (omega_nu, omega_3, omega_4) is omega_b = omega_nu, omega_21 = omega_12 = omega_3,
// omega_22 = omega_4 (eq. RMcoll, Section 4c).
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

enum Model : int {
    kBGK = 0, kRM = 1, kHM = 2, kCM = 3, kCHM = 4, kK = 5, kPR = 6, kRR = 7, kStreamOnly = 99
};
enum Prec : int { kF64 = 0, kF32 = 1, kF16 = 2 };

// Lattice constant c_s^2 = 1/3 and rest weights 4/9, 1/9, 1/36.
template <typename R> struct Lat {
    static constexpr R cs2 = R(1.0 / 3.0);
    static constexpr R cs4 = R(1.0 / 9.0);
    static constexpr R w0 = R(4.0 / 9.0);
    static constexpr R w1 = R(1.0 / 9.0);
    static constexpr R w5 = R(1.0 / 36.0);
};

// Velocity components, index order (0,0),(1,0),(0,1),(-1,0),(0,-1),(1,1),(-1,1),(-1,-1),(1,-1).
__host__ __device__ constexpr int cx(int i) {
    return (i == 1 || i == 5 || i == 8) ? 1 : (i == 3 || i == 6 || i == 7) ? -1 : 0;
}
__host__ __device__ constexpr int cy(int i) {
    return (i == 2 || i == 5 || i == 6) ? 1 : (i == 4 || i == 7 || i == 8) ? -1 : 0;
}
__host__ __device__ constexpr double rest_weight(int i) {
    return i == 0 ? 4.0 / 9.0 : (i < 5 ? 1.0 / 9.0 : 1.0 / 36.0);
}

// Relaxation coefficients in the form used by the kernels: factors k = -omega of the changes d* - d, with the
// second-order diagonal pair written as d20* - d20 = kpp d20 + cpm d02, d02* - d02 = cpm d20 + kpp d02, and the
// factors c = 1 - omega of the values themselves where a model needs those.
template <typename R> struct Coef {
    R cpm, c21, c12, c22, om;  // om = omega_nu (BGK)
    R kpp, k11, k21, k12, k22;
};

template <typename R>
__host__ __device__ inline Coef<R> make_coef(const double w[5]) {
    const double a = 0.5 * (1.0 - w[1]);  // trace
    const double b = 0.5 * (1.0 - w[0]);  // deviator
    Coef<R> c;
    c.cpm = R(a - b);
    c.c21 = R(1.0 - w[2]);
    c.c12 = R(1.0 - w[3]);
    c.c22 = R(1.0 - w[4]);
    c.om = R(w[0]);
    c.kpp = R(-0.5 * (w[0] + w[1]));
    c.k11 = R(-w[0]);
    c.k21 = R(-w[2]);
    c.k12 = R(-w[3]);
    c.k22 = R(-w[4]);
    return c;
}

// Reference state of the stored deviations (density rho_s, velocity U = (A, B)) and the products of
// it that the collision uses: jx = rho_s A, jy = rho_s B, a20 = rho_s A^2, a02 = rho_s B^2,
// a21 = rho_s A^2 B.
template <typename R> struct Ref {
    R rho, ux, uy;
    R jx, jy, a20, a02, a21;
};

template <typename R>
__host__ __device__ inline Ref<R> make_ref(double rho, double ux, double uy) {
    return Ref<R>{R(rho), R(ux), R(uy), R(rho * ux), R(rho * uy), R(rho * ux * ux), R(rho * uy * uy), R(rho * ux * ux * uy)};
}

// Sums and differences of the stored populations that the density, the momentum and the raw
// moments share: s13 = h1 + h3, s24 = h2 + h4, d13 = h1 - h3, d24 = h2 - h4 and the moments of the
// diagonal populations m22, m11, m21 (less h2 - h4's share of jy), m12.
template <typename R> struct Sums {
    R s13, s24, d13, d24, m22, m11, m21, m12;
};

template <typename R>
__host__ __device__ __forceinline__ Sums<R> sums_of(const R (&h)[9]) {
    const R a = h[5] + h[7], b = h[6] + h[8], p = h[5] - h[7], q = h[8] - h[6];
    Sums<R> s;
    s.s13 = h[1] + h[3];
    s.s24 = h[2] + h[4];
    s.d13 = h[1] - h[3];
    s.d24 = h[2] - h[4];
    s.m22 = a + b;
    s.m11 = a - b;
    s.m12 = p + q;
    s.m21 = p - q;
    return s;
}

// Conserved quantities of a cell: drho = rho - rho_s, (jx, jy) = rho u - rho_s U (the momentum
// of the stored deviations), u and du = u - U.
template <typename R> struct Macro {
    R drho, rho, jx, jy, ux, uy, dux, duy;
    R inv_rho;  // 1 / rho
    Sums<R> s;  // sums of the populations (macro_of; not set by macro_of_fields)
};

// Hermite equilibrium moments of order N (A^eq_pq = rho ux^p uy^q, zero above order N), as
// differences to those of the reference: E_pq = A^eq_pq(rho, u) - A^eq_pq(rho_s, U)
//   = drho u^p v^q + rho_s (u^p v^q - U^p V^q),
// the monomial differences telescoped through du so that nothing of order one cancels.
template <typename R> struct Eq {
    R e20, e02, e11, e21, e12, e22;
};

template <typename R>
__host__ __device__ __forceinline__ Eq<R> hermite_eq(const Macro<R>& m, const Ref<R>& r, int N) {
    const R a = m.ux, b = m.uy, A = r.ux, da = m.dux, db = m.duy;
    const R a2 = a * a, b2 = b * b;
    const R D20 = da * (a + A);          // a^2 - A^2
    const R D02 = db * (b + r.uy);       // b^2 - B^2
    const R D11 = da * b + A * db;       // a b - A B
    Eq<R> e;
    e.e20 = m.drho * a2 + r.rho * D20;
    e.e02 = m.drho * b2 + r.rho * D02;
    e.e11 = m.drho * (a * b) + r.rho * D11;
    if (N >= 3) {
        const R D21 = D20 * b + (A * A) * db;  // a^2 b - A^2 B
        const R D12 = da * b2 + A * D02;       // a b^2 - A B^2
        e.e21 = m.drho * (a2 * b) + r.rho * D21;
        e.e12 = m.drho * (a * b2) + r.rho * D12;
    } else {
        e.e21 = R(0);
        e.e12 = R(0);
    }
    if (N >= 4) {
        const R D22 = D20 * b2 + (A * A) * D02;  // a^2 b^2 - A^2 B^2
        e.e22 = m.drho * (a2 * b2) + r.rho * D22;
    } else {
        e.e22 = R(0);
    }
    return e;
}

// Fused multiply-add, rounded once: written out where a product feeds a sum in another
// statement, so that every kernel (and the host) computes it the same way.
template <typename R>
__host__ __device__ __forceinline__ R fmadd(R a, R b, R c) {
    if constexpr (sizeof(R) == 4)
        return fmaf(a, b, c);
    else
        return fma(a, b, c);
}

// Post-collision Hermite moments minus the reference's (equilibrium difference + relaxed
// non-equilibrium part) -> raw-moment differences (eq. HM2RM_Q9, which is linear) -> stored
// deviations (eq. Q9postCollVDF_RM; the density difference contributes drho w_i).  The pairs of
// opposite populations share their sums and differences.
template <typename R>
__host__ __device__ __forceinline__ void hermite_to_pop(const Macro<R>& m, R a20, R a02, R a11, R a21,
                                               R a12, R a22, R (&h)[9]) {
    using L = Lat<R>;
    const R tr = a20 + a02;
    const R M21 = a21 + L::cs2 * m.jy;
    const R M12 = a12 + L::cs2 * m.jx;
    const R M22 = a22 + L::cs2 * tr;
    const R r1 = m.drho * L::w1, r5 = m.drho * L::w5;
    h[0] = fmadd(m.drho, L::w0, M22 - tr);
    const R u = a20 - M22, v = m.jx - M12;  // 2 (h1 - r1), 2 (h3 - r1) = u + v, u - v
    const R p = a02 - M22, q = m.jy - M21;
    h[1] = fmadd(R(0.5), u + v, r1);
    h[3] = fmadd(R(0.5), u - v, r1);
    h[2] = fmadd(R(0.5), p + q, r1);
    h[4] = fmadd(R(0.5), p - q, r1);
    const R A = M22 + a11, B = M22 - a11, C = M12 + M21, D = M12 - M21;
    h[5] = fmadd(R(0.25), A + C, r5);
    h[6] = fmadd(R(0.25), B - D, r5);
    h[7] = fmadd(R(0.25), A - C, r5);
    h[8] = fmadd(R(0.25), B + D, r5);
}

// h += scale * P(D): the populations of the moment changes (D20, D02, D11, D21, D12) and of the raw
// fourth-moment change M22, density and momentum unchanged (eq. HM2RM_Q9, eq. Q9postCollVDF_RM); the
// pairs of opposite populations share their sums and differences.
template <typename R>
__device__ __forceinline__ void add_change(R (&h)[9], R scale, R D20, R D02, R D11, R D21, R D12, R M22) {
    const R s1 = R(0.5) * scale, s5 = R(0.25) * scale;
    const R u = D20 - M22, p = D02 - M22;
    const R A = M22 + D11, B = M22 - D11, C = D12 + D21, D = D12 - D21;
    h[0] = fmadd(scale, M22 - (D20 + D02), h[0]);
    h[1] = fmadd(s1, u - D12, h[1]);
    h[3] = fmadd(s1, u + D12, h[3]);
    h[2] = fmadd(s1, p - D21, h[2]);
    h[4] = fmadd(s1, p + D21, h[4]);
    h[5] = fmadd(s5, A + C, h[5]);
    h[6] = fmadd(s5, B - D, h[6]);
    h[7] = fmadd(s5, A - C, h[7]);
    h[8] = fmadd(s5, B + D, h[8]);
}

// Collide one cell in place.  N is the equilibrium order (2, 3 or 4; CM, CHM and K use 4).  In FP64
// the populations are stored unshifted (the reference is zero) and its terms are left out.
template <int MODEL, typename R>
__device__ __forceinline__ void collide(R (&h)[9], const Macro<R>& m, const Ref<R>& ref,
                                        const Coef<R>& c, int N) {
    using L = Lat<R>;
    if constexpr (MODEL == kStreamOnly) {
        return;
    } else {
        constexpr bool kShifted = sizeof(R) == 4;
        constexpr bool kCentral = MODEL == kCM || MODEL == kCHM || MODEL == kK;
        constexpr bool kRawX = MODEL == kBGK || MODEL == kRM || MODEL == kCM;  // relaxes X (see the top)
        const R ux = m.ux, uy = m.uy;
        // equilibrium differences and non-equilibrium moments
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
        // d22 = A22 - E22, or X = d22 + cs^2 (d20 + d02) = m22 - cs^4 drho - cs^2 (E20 + E02) - E22
        R d22 = fmadd(-L::cs2, kRawX ? e20 + e02 : a20 + a02, fmadd(-L::cs4, m.drho, m.s.m22));
        if (kCentral || N >= 3) {
            R e21 = e20 * uy;
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
        if constexpr (MODEL == kBGK) {
            add_change(h, -c.om, d20, d02, d11, d21, d12, d22);
        } else {
            // second-order block, common to every moment space
            const R D20 = fmadd(c.kpp, d20, c.cpm * d02);
            const R D02 = fmadd(c.kpp, d02, c.cpm * d20);
            const R D11 = c.k11 * d11;
            R D21, D12, M22;
            if constexpr (MODEL == kHM) {
                D21 = c.k21 * d21;
                D12 = c.k12 * d12;
                M22 = fmadd(c.k22, d22, L::cs2 * (D20 + D02));
            } else if constexpr (MODEL == kPR) {
                D21 = -d21;
                D12 = -d12;
                M22 = fmadd(L::cs2, D20 + D02, -d22);
            } else if constexpr (MODEL == kRM) {
                D21 = c.k21 * d21;
                D12 = c.k12 * d12;
                M22 = c.k22 * d22;
            } else if constexpr (MODEL == kRR) {
                // recursive non-equilibrium Hermite moments (eq. RRformulas_D2Q9)
                const R f11 = d11 + d11;
                const R r21 = fmadd(ux, f11, uy * d20);
                const R r12 = fmadd(uy, f11, ux * d02);
                const R r22 = fmadd(ux, r12, uy * r21);
                D21 = fmadd(c.c21, r21, -d21);
                D12 = fmadd(c.c12, r12, -d12);
                M22 = fmadd(c.c22, r22, fmadd(L::cs2, D20 + D02, -d22));
            } else {  // kCM, kCHM, kK: central (Hermite) moments t = shift(-u) of d, s = t* - t
                const R vx = ux + ux, vy = uy + uy;
                const R t21 = fmadd(-vx, d11, fmadd(-uy, d20, d21));
                const R t12 = fmadd(-vy, d11, fmadd(-ux, d02, d12));
                const R t22 = fmadd(-ux, d12 + t12, fmadd(-uy, d21 + t21, d22));
                const R s21 = c.k21 * t21;
                const R s12 = c.k12 * t12;
                R s22;
                if constexpr (MODEL == kCM) {
                    s22 = c.k22 * t22;  // raw central fourth moment (t22 holds t22 + cs^2 (t20 + t02))
                } else if constexpr (MODEL == kCHM) {
                    s22 = fmadd(c.k22, t22, L::cs2 * (D20 + D02));
                } else {
                    // fourth-order cumulant times rho: t22 - (t20 t02 + 2 t11^2) / rho
                    const R n20 = d20 + D20, n02 = d02 + D02, n11 = d11 + D11;
                    const R p = fmadd(d11 + d11, d11, d20 * d02);
                    const R q = fmadd(n11 + n11, n11, n20 * n02);
                    s22 = fmadd(fmadd(-c.c22, p, q), m.inv_rho, fmadd(c.k22, t22, L::cs2 * (D20 + D02)));
                }
                // back to Hermite moments (eq. CHM2HM_Q9, equilibrium parts cancel)
                D21 = fmadd(vx, D11, fmadd(uy, D20, s21));
                D12 = fmadd(vy, D11, fmadd(ux, D02, s12));
                M22 = fmadd(ux, s12 + D12, fmadd(uy, s21 + D21, s22));
            }
            add_change(h, R(1), D20, D02, D11, D21, D12, M22);
        }
    }
}

}  // namespace lbm
