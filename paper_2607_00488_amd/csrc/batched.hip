// Template form of the multi-component likelihood (Eqs. (Rij), (fNp_reweight),
// (mu_total)): the folds of every component's basis spectra, kept per reco bin,
// and the evaluation from them; and the finishing sum of the surrogate's
// likelihood.
#include "batched.h"
#include "lnpos.h"

#include <cmath>

namespace nr {

namespace {

// -2lnL per point: sum of the column-tile deviance partials, data constant,
// pulls (Eq. (logL)).
// x[0] + x[1] + ... + x[n - 1] in index order; with n even (so that every
// row of a [P][n] array starts 16-byte aligned) eight values at a time as
// 16-byte pairs, all in flight before the additions.
__device__ inline double row_sum(const double* x, int n) {
    double s = 0.0;
    int q = 0;
    if ((n & 1) == 0) {
        for (; q + 8 <= n; q += 8) {
            double2 v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = reinterpret_cast<const double2*>(x + q)[i];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                s += v[i].x;
                s += v[i].y;
            }
        }
    }
    for (; q < n; ++q) s += x[q];
    return s;
}

__global__ void k_finalize(FinalArgs a) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.n_pts) return;
    const double d = row_sum(a.part + (size_t)p * a.n_nt, a.n_nt);
    double pulls = 0.0;
    for (int i = 0; i < kNTheta; ++i)
        if (a.pull_sigma[i] > 0.0) {
            const double z = (a.theta[(size_t)p * kNTheta + i] - a.pull_mean[i]) / a.pull_sigma[i];
            pulls += z * z;
        }
    a.nll[p] = 2.0 * d + 2.0 * a.cdata + pulls;
}

// ------------------------------------------------------------ templates
// One thread per reco bin, one work-group row per slab of response rows: the
// FP64 sums of F_lb R_lj over the row's factors (wave-uniform).
__global__ __launch_bounds__(256) void k_tmpl_fold(TmplFoldArgs a) {
    constexpr int RL = kRFComp;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= a.n_reco) return;
    const int l0 = blockIdx.y * kTmplSlabRows;
    const int l1 = min(l0 + kTmplSlabRows, a.n_t);
    double acc[RL];
#pragma unroll
    for (int b = 0; b < RL; ++b) acc[b] = 0.0;
    for (int l = l0; l < l1; ++l) {
        const double r = a.R[(size_t)l * a.ldr + j];
        const double* f = a.rf + (size_t)l * RL;
#pragma unroll
        for (int b = 0; b < RL; ++b) acc[b] = fma(f[b], r, acc[b]);
    }
#pragma unroll
    for (int b = 0; b < RL; ++b)
        a.part[((size_t)blockIdx.y * RL + b) * a.n_reco + j] = acc[b];
}

// Slab sums in slab order, one (bin, template) per thread, into the record.
__global__ __launch_bounds__(256) void k_tmpl_records(TmplRecArgs a) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    const int b = blockIdx.y;
    if (j >= a.n_reco) return;
    double s = 0.0;
    for (int q = 0; q < a.n_slab; ++q) s += a.part[((size_t)q * a.n_cols + b) * a.n_reco + j];
    a.rec[(size_t)j * a.rl + a.dst0 + b] = s;
}

// Sums over the column slices, one (point, quantity) per thread, in slice
// order (bitwise reproducible).
__global__ __launch_bounds__(kTmplWave) void k_tmpl_reduce(TmplReduceArgs a) {
    const int p = blockIdx.x * kTmplWave + threadIdx.x;
    if (p >= a.n_pts) return;
    const int v = blockIdx.y;
    double s = 0.0;
    if (v == 0) {
        for (int q = 0; q < a.n_split; ++q) s += a.dpart[(size_t)q * a.n_pts + p];
    } else {
        for (int q = 0; q < a.n_split; ++q)
            s += a.hpart[((size_t)q * a.n_acc + v - 1) * a.n_pts + p];
    }
    a.red[(size_t)v * a.n_pts + p] = s;
}

// ------------------------------------------------ multi-component templates
// Backgrounds, mask and data of each bin after the component templates.
__global__ __launch_bounds__(256) void k_tmpl_mdata(TmplMultiDataArgs a) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= a.n_reco) return;
    double* r = a.rec + (size_t)j * a.rl;
    const int ob = kTmplCompCols * a.K;
    for (int q = 0; q < a.B; ++q) r[ob + q] = a.bkg[(size_t)q * a.n_reco + j];
    r[ob + a.B] = a.mask ? a.mask[j] : 1.0;
    r[ob + a.B + 1] = a.n[j];
}

// As k_tmpl_eval, for the multi-component record: per (point, bin) the
// component sums t_k = G0^(k) + sum_b c_b G^(k)_b (8 K products), mu from
// the rates, and for the gradient the kCompBasis + K + B contractions
//   H_b = sum_j a'_j sum_k r_k G^(k)_bj,  R_k = sum_j a'_j t_kj,
//   Q_q = sum_j a'_j B_qj,  a'_j = M_j d(-2lnL)/d mu_j.
// Loops run to compile-time maxima KM, BM with uniform predicates, so every
// accumulator stays in registers; the smaller size class (five components,
// four backgrounds: the solar species) needs fewer registers and keeps more
// waves resident.
template <bool GRAD, bool MU, int KM, int BM>
__global__ __launch_bounds__(kTmplWave) void k_tmpl_meval(TmplMultiEvalArgs a) {
    const int p = blockIdx.x * kTmplWave + threadIdx.x;
    const int sl = blockIdx.y;
    const bool ok = p < a.n_pts;
    const int pc = ok ? p : a.n_pts - 1;
    const double* th = a.theta + (size_t)pc * a.n_theta;
    double c[kCompBasis];
    basis_coef7(th, a.ph, 1.0, c);
    double rk[KM], rb[BM];
#pragma unroll
    for (int k = 0; k < KM; ++k) rk[k] = k < a.K ? th[5 + k] : 0.0;
#pragma unroll
    for (int q = 0; q < BM; ++q) rb[q] = q < a.B ? th[5 + a.K + q] : 0.0;
    const int ob = kTmplCompCols * a.K;
    const int j0 = sl * a.cols_per;
    const int j1 = min(j0 + a.cols_per, a.n_reco);
    double dsum = 0.0;
    double H[kCompBasis], Rk[KM], Qb[BM];
#pragma unroll
    for (int b = 0; b < kCompBasis; ++b) H[b] = 0.0;
#pragma unroll
    for (int k = 0; k < KM; ++k) Rk[k] = 0.0;
#pragma unroll
    for (int q = 0; q < BM; ++q) Qb[q] = 0.0;
    for (int j = j0; j < j1; ++j) {
        const double* __restrict__ r = a.rec + (size_t)j * a.rl;
        double s = 0.0, tk[KM], T[kCompBasis];
#pragma unroll
        for (int b = 0; b < kCompBasis; ++b) T[b] = 0.0;
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            tk[k] = 0.0;
            if (k < a.K) {
                const double* g = r + kTmplCompCols * k;
                double t = g[kCompBasis];
#pragma unroll
                for (int b = 0; b < kCompBasis; ++b) t = fma(c[b], g[b], t);
                if (GRAD) {  // T_b = sum_k r_k G^(k)_bj, for H_b
#pragma unroll
                    for (int b = 0; b < kCompBasis; ++b) T[b] = fma(rk[k], g[b], T[b]);
                }
                tk[k] = t;
                s = fma(rk[k], t, s);
            }
        }
#pragma unroll
        for (int q = 0; q < BM; ++q)
            if (q < a.B) s = fma(rb[q], r[ob + q], s);
        const double mask = r[ob + a.B], nj = r[ob + a.B + 1];
        const double mu = s * mask;
        const double qn = nj > 0.0 ? nj / mu : 0.0;
        double d;
        if (nj > 0.0)
            d = mu > 0.0 ? (mu - nj) + nj * ln_pos(qn) : INFINITY;
        else
            d = mu;
        dsum += d;
        if (MU && ok) a.mu[(size_t)p * a.n_reco + j] = mu;
        if (GRAD) {
            const double ap = 2.0 * (1.0 - qn) * mask;
#pragma unroll
            for (int k = 0; k < KM; ++k)
                if (k < a.K) Rk[k] = fma(ap, tk[k], Rk[k]);
#pragma unroll
            for (int b = 0; b < kCompBasis; ++b) H[b] = fma(ap, T[b], H[b]);
#pragma unroll
            for (int q = 0; q < BM; ++q)
                if (q < a.B) Qb[q] = fma(ap, r[ob + q], Qb[q]);
        }
    }
    if (!ok) return;
    a.dpart[(size_t)sl * a.n_pts + p] = dsum;
    if (GRAD) {
        const int na = kCompBasis + a.K + a.B;
        double* hp = a.hpart + (size_t)sl * na * a.n_pts + p;
#pragma unroll
        for (int b = 0; b < kCompBasis; ++b) hp[(size_t)b * a.n_pts] = H[b];
#pragma unroll
        for (int k = 0; k < KM; ++k)
            if (k < a.K) hp[(size_t)(kCompBasis + k) * a.n_pts] = Rk[k];
#pragma unroll
        for (int q = 0; q < BM; ++q)
            if (q < a.B) hp[(size_t)(kCompBasis + a.K + q) * a.n_pts] = Qb[q];
    }
}

// -2lnL and gradient of the multi-component form: d/d theta_i (i < 5) =
// sum_b dc_ib H_b, d/d r_k = R_k, d/d r_q = Q_q, plus the pulls.
__global__ __launch_bounds__(256) void k_tmpl_mfinal(TmplMultiFinalArgs a) {
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= a.n_pts) return;
    const double* th = a.theta + (size_t)p * a.n_theta;
    double pulls = 0.0;
    for (int i = 0; i < a.n_theta; ++i)
        if (a.pull_sigma[i] > 0.0) {
            const double z = (th[i] - a.pull_mean[i]) / a.pull_sigma[i];
            pulls += z * z;
        }
    a.nll[p] = 2.0 * a.red[p] + 2.0 * a.cdata + pulls;
    if (!a.grad) return;
    const double* h = a.red + a.n_pts + p;  // contraction v at h[v * n_pts]
    double* g = a.grad + (size_t)p * a.n_theta;
    double hb[kCompBasis], g5[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int b = 0; b < kCompBasis; ++b) hb[b] = h[(size_t)b * a.n_pts];
    basis_dcoef7(th, a.ph, 1.0, hb, g5);
#pragma unroll
    for (int i = 0; i < 5; ++i) g[i] = g5[i];
    for (int i = 5; i < a.n_theta; ++i) g[i] = h[(size_t)(kCompBasis + i - 5) * a.n_pts];  // R_k, Q_q
    for (int i = 0; i < a.n_theta; ++i)
        if (a.pull_sigma[i] > 0.0)
            g[i] += 2.0 * (th[i] - a.pull_mean[i]) / (a.pull_sigma[i] * a.pull_sigma[i]);
}

}  // namespace

hipError_t launch_tmpl_mdata(const TmplMultiDataArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_tmpl_mdata, dim3((a.n_reco + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tmpl_meval(const TmplMultiEvalArgs& a, int n_split, hipStream_t s) {
    if (a.K < 1 || a.K > kTmplMaxComp || a.B < 0 || a.B > kTmplMaxBkg || (a.hpart && a.mu))
        return hipErrorInvalidValue;
    const dim3 grid((a.n_pts + kTmplWave - 1) / kTmplWave, n_split);
    const bool small = a.K <= kTmplSmallComp && a.B <= kTmplSmallBkg;
    constexpr int KS = kTmplSmallComp, BS = kTmplSmallBkg, KL = kTmplMaxComp, BL = kTmplMaxBkg;
    if (a.hpart) {
        if (small) hipLaunchKernelGGL((k_tmpl_meval<true, false, KS, BS>), grid, dim3(kTmplWave), 0, s, a);
        else hipLaunchKernelGGL((k_tmpl_meval<true, false, KL, BL>), grid, dim3(kTmplWave), 0, s, a);
    } else if (a.mu) {
        hipLaunchKernelGGL((k_tmpl_meval<false, true, KL, BL>), grid, dim3(kTmplWave), 0, s, a);
    } else {
        if (small) hipLaunchKernelGGL((k_tmpl_meval<false, false, KS, BS>), grid, dim3(kTmplWave), 0, s, a);
        else hipLaunchKernelGGL((k_tmpl_meval<false, false, KL, BL>), grid, dim3(kTmplWave), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_tmpl_mfinal(const TmplMultiFinalArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_tmpl_mfinal, dim3((a.n_pts + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tmpl_fold(const TmplFoldArgs& a, int n_slab, hipStream_t s) {
    const dim3 grid((a.n_reco + 255) / 256, n_slab);
    hipLaunchKernelGGL(k_tmpl_fold, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tmpl_records(const TmplRecArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_tmpl_records, dim3((a.n_reco + 255) / 256, a.n_dst), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tmpl_reduce(const TmplReduceArgs& a, hipStream_t s) {
    const dim3 grid((a.n_pts + kTmplWave - 1) / kTmplWave, a.hpart ? 1 + a.n_acc : 1);
    hipLaunchKernelGGL(k_tmpl_reduce, grid, dim3(kTmplWave), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_finalize(const FinalArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_finalize, dim3((a.n_pts + 255) / 256), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace nr
