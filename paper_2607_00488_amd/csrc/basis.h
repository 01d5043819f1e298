// The theta-independent basis of the recoil spectrum and its coefficients.
//
// dsigma/dT of Eqs. (xs_nsi), (xs_mm) is linear in the coupling products, and
// with eps_mumu = 0 the nu_mu and nu_tau shares of 1 - P_ee differ only by the
// constant tau_frac, so a source's S_theta(T_l) of Eq. (fT) is exactly
// sum_b c_b(theta) I_b(T_l) over kCompBasis = 7 spectra,
//   I_0 = sum nu P_ee,      I_1 = sum nu (1 - P_ee)        (g_L^2)
//   I_2 = sum nu P_ee y^2,  I_3 = sum nu (1 - P_ee) y^2    (g_R^2)
//   I_4 = sum nu P_ee x,    I_5 = sum nu (1 - P_ee) x      (-g_L g_R)
//   I_6 = sum nu (1/T - 1/E)                               (magnetic)
// with y = 1 - T/E, x = m_e T/E^2 over the reachable nodes.  The
// single-component form sums its sources in two groups of seven (fixed, and
// scaled by f_8B): kNBasis = 14.
//
// A row's factors are v_l = m_l w_l = sum_b c_b F_lb + c_const F_l,const with
// F_lb = m_l I_b(T_l) / S_SM(T_l) (0 where S_SM = 0) and F_l,const = m_l where
// S_SM = 0 (weight 1), else 0: rows of kRF = 16 doubles (14, const, 0), or of
// kRFComp = 8 (7, const) per component of the multi-component form.
#pragma once
#include "common.h"

namespace nr {

constexpr int kCompBasis = 7;
constexpr int kRF = 16;
constexpr int kRFComp = 8;

// Coefficients of one group's seven spectra (f: the group's scale).
// The multiply-adds are explicit, so that every kernel that inlines this rounds
// alike.
__device__ inline void basis_coef7(const double* th, const Phys& ph, double f, double c[7]) {
#pragma clang fp contract(off)
    const double gle = ph.gLe + th[0], gre = ph.gR + th[1];
    const double glm = ph.gLm, grm = ph.gR;
    const double glt = ph.gLm + th[2], grt = ph.gR + th[3];
    const double t = ph.tau_frac, m = 1.0 - ph.tau_frac;
    c[0] = f * gle * gle;
    c[1] = f * fma(m * glm, glm, t * glt * glt);
    c[2] = f * gre * gre;
    c[3] = f * fma(m * grm, grm, t * grt * grt);
    c[4] = -f * gle * gre;
    c[5] = -f * fma(m * glm, grm, t * glt * grt);
    c[6] = f * ph.cmm * th[4];
}

__device__ inline void basis_coef(const double* th, const Phys& ph, double c[kNBasis]) {
    basis_coef7(th, ph, 1.0, c);
    for (int b = 0; b < kCompBasis; ++b) c[kCompBasis + b] = th[5] * c[b];
}

// d(c_b)/d(theta_i) h_b summed over one group's seven spectra, i < 5.
__device__ inline void basis_dcoef7(const double* th, const Phys& ph, double f,
                                    const double h[7], double g[5]) {
    const double gle = ph.gLe + th[0], gre = ph.gR + th[1];
    const double glt = ph.gLm + th[2], grt = ph.gR + th[3];
    const double t = ph.tau_frac;
    g[0] += f * (2.0 * gle * h[0] - gre * h[4]);
    g[1] += f * (2.0 * gre * h[2] - gle * h[4]);
    g[2] += f * t * (2.0 * glt * h[1] - grt * h[5]);
    g[3] += f * t * (2.0 * grt * h[3] - glt * h[5]);
    g[4] += f * ph.cmm * h[6];
}

// The six derivatives of sum_b c_b J_b (single-component form).
__device__ inline void basis_grad(const double* th, const Phys& ph, const double J[kNBasis],
                                  double g[6]) {
    for (int i = 0; i < 6; ++i) g[i] = 0.0;
    basis_dcoef7(th, ph, 1.0, J, g);
    basis_dcoef7(th, ph, th[5], J + kCompBasis, g);
    double c[kCompBasis];
    basis_coef7(th, ph, 1.0, c);
    for (int b = 0; b < kCompBasis; ++b) g[5] += c[b] * J[kCompBasis + b];
}

}  // namespace nr
