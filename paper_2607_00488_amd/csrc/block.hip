// Blocked fold on gfx950: the points of a list share one stream over the
// response.  Their weights (Eqs. (fT_norm), (reweight_factor)) come from the
// recoil basis of Eq. (fT); the fold of Eqs. (Rij), (fNp_reweight), (mu_total)
// is then the product of the points' weights with R on the FP64 matrix cores,
// R read once per group of up to 64 points, and the Poisson -2lnL of
// Eq. (logL) follows from its split sums.
#include "basis.h"
#include "block.h"

#include <cmath>

namespace nr {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int kThreads = 256;
constexpr int kStageQuads = 8;               // row quads per stage
constexpr int kStageRows = 4 * kStageQuads;  // 32 rows

// --------------------------------------------------------------- weights
// V^T[l][p] = sum_b F_lb c_b(theta_p), itself a product with a reduction of
// 8: two FP64 matrix instructions per 16 rows x 16 points, rows on the row operand, so that a lane's values of F are 32 contiguous
// bytes and a row's 16 points leave as one 128-byte run.  Bound by writing
// V^T: 1024 points x 16384 rows took 11 us per 64 points before, one thread
// per point with the basis broadcast from LDS.
constexpr int kWtPts = 64;   // points per work-group
constexpr int kWtRows = 64;  // rows per work-group, 16 per wave

__global__ __launch_bounds__(kThreads) void k_pts_weights(PtsWeightArgs a) {
    constexpr int RL = kRFComp;  // row length of the factors
    __shared__ double cs[kWtPts][RL + 1];
    constexpr int KS = RL / 4;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int c = blockIdx.z, l0 = blockIdx.x * kWtRows + wave * 16;
    const int p0 = blockIdx.y * kWtPts;
    if (tid < kWtPts) {
        const int p = p0 + tid;
        double v[RL];
        for (int b = 0; b < RL; ++b) v[b] = 0.0;
        if (p < a.n_pts) {
            const double* th = a.theta + (size_t)p * a.n_theta;
            const double r = th[a.rate_index + c];
            basis_coef7(th, a.ph, r, v);
            v[kCompBasis] = r;
        }
        for (int b = 0; b < RL; ++b) cs[tid][b] = v[b];
    }
    double f[KS];
    {
        const size_t l = (size_t)c * a.n_t + min(l0 + li, a.n_t - 1);
        const double2* src = reinterpret_cast<const double2*>(a.rf + l * RL + KS * lk);
#pragma unroll
        for (int s = 0; s < KS / 2; ++s) {
            const double2 t = src[s];
            f[2 * s] = t.x;
            f[2 * s + 1] = t.y;
        }
    }
    __syncthreads();
    const int nb = min(kWtPts, a.n_pad - p0) / 4;  // quads of points
    for (int b = 0; 4 * b < nb; ++b) {
        v4d acc = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < KS; ++s)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(f[s], cs[16 * b + li][KS * lk + s], acc,
                                                       0, 0, 0);
        if (16 * b + li >= 4 * nb) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int l = l0 + lk + 4 * r;
            if (l < a.n_t)
                a.wt[((size_t)c * a.n_t + l) * a.ldw + p0 + 16 * b + li] = acc[r];
        }
    }
}

// ------------------------------------------------------------------ fold
// One work-group: 16 MB points x 256 columns x the rows of one split.  Wave
// w owns 64 columns, as four sets of 16 interleaved ones: lane (li, lk)
// loads the float4 of columns 4 li .. 4 li + 3 of row 4 q + lk, which is the
// column operand of four matrix instructions (k = lk), so R goes from memory
// straight to the registers that use it, one stage (32 rows, 8 KB per wave)
// ahead.  The weights, shared by the four waves, pass through two LDS
// buffers of one stage each.  With one block of 16 points the stream over R
// is the limit (four multiply-adds per lane and R value cost a third of its
// bytes' time); with four the matrix instructions are.
template <int MB>
__device__ __forceinline__ void fold_body(const BlkFoldArgs& a, int ct, int sp, int p0,
                                          double* lds) {
    constexpr int PS = 16 * MB;                 // points = LDS row length
    constexpr int STAGE = kStageRows * PS;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lk = lane >> 4;
    const int ld4 = a.ldr >> 2;
    const int c4 = ct * (kBlkCols / 4) + wave * 16 + li;
    const float4* __restrict__ Rc =
        reinterpret_cast<const float4*>(a.R) + (c4 < ld4 ? c4 : ld4 - 1);
    const int ke0 = min(a.n_rows, (sp + 1) * a.rows_per);
    int kb = sp * a.rows_per, ke = ke0;
    if (a.band) {  // rows outside hold exact zeros in this tile's columns
        kb = max(kb, a.band[2 * ct]);
        ke = min(ke, a.band[2 * ct + 1]);
    }
    v4d acc[MB][4];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[m][e] = (v4d){0.0, 0.0, 0.0, 0.0};

    double2 wreg[MB];
    auto load_w = [&](int k) {
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int c = tid + i * kThreads;
            const int row = k + c / (PS / 2), pc = 2 * (c % (PS / 2));
            wreg[i] = row < ke ? *reinterpret_cast<const double2*>(
                                     a.wt + (size_t)row * a.ldw + p0 + pc)
                               : make_double2(0.0, 0.0);
        }
    };
    auto store_w = [&](int buf) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
            *reinterpret_cast<double2*>(lds + buf * STAGE + 2 * (tid + i * kThreads)) = wreg[i];
    };
    auto load_r = [&](int k, float4 x[kStageQuads]) {
#pragma unroll
        for (int q = 0; q < kStageQuads; ++q) {
            const int row = min(k + 4 * q + lk, a.n_rows - 1);  // past the end: weight 0
            x[q] = Rc[(size_t)row * ld4];
        }
    };
    auto compute = [&](int buf, const float4 x[kStageQuads]) {
        const double* W = lds + buf * STAGE;
#pragma unroll
        for (int q = 0; q < kStageQuads; ++q) {
            const double* wr = W + (4 * q + lk) * PS;
            double f[MB];
#pragma unroll
            for (int h = 0; h < MB / 2; ++h) {
                const double2 v = *reinterpret_cast<const double2*>(wr + 32 * h + 2 * li);
                f[2 * h] = v.x;
                f[2 * h + 1] = v.y;
            }
            if (MB & 1) f[MB - 1] = wr[16 * (MB - 1) + li];
            const double r[4] = {(double)x[q].x, (double)x[q].y, (double)x[q].z, (double)x[q].w};
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    acc[m][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[m], r[e], acc[m][e], 0, 0, 0);
        }
    };
    if (kb < ke) {
        float4 x0[kStageQuads], x1[kStageQuads];
        load_w(kb);
        load_r(kb, x0);
        store_w(0);
        __syncthreads();
        // stage in buffer `buf` and registers cur; the next one is loaded
        // before its arithmetic and its weights stored after (every wave has
        // left that buffer since the last barrier)
        auto stage = [&](int k, int buf, const float4 cur[kStageQuads], float4 nxt[kStageQuads]) {
            const bool more = k + kStageRows < ke;
            if (more) {
                load_w(k + kStageRows);
                load_r(k + kStageRows, nxt);
            }
            compute(buf, cur);
            if (more) {
                store_w(buf ^ 1);
                __syncthreads();
            }
        };
        for (int k = kb; k < ke; k += 2 * kStageRows) {
            stage(k, 0, x0, x1);
            if (k + kStageRows < ke) stage(k + kStageRows, 1, x1, x0);
        }
    }
    if (c4 >= ld4) return;
    double* out = a.part + (size_t)sp * a.split_stride + 4 * (size_t)c4;
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = lk + 4 * r;
            // blocks 2h, 2h + 1 hold alternate points (one 16-byte LDS read
            // feeds both); an odd last block holds 16 in order
            const int p = p0 + ((m | 1) < MB ? 32 * (m >> 1) + 2 * i + (m & 1) : 16 * m + i);
            double2* o = reinterpret_cast<double2*>(out + (size_t)p * a.ldr);
            o[0] = make_double2(acc[m][0][r], acc[m][1][r]);
            o[1] = make_double2(acc[m][2][r], acc[m][3][r]);
        }
}

// The points' blocks are dealt to n_groups groups of at most MAXMB.  Launch
// order: work-groups 8 apart share an XCD, and an XCD takes its (column tile,
// split) pairs in chunks of as many as leave all their groups resident at
// once, group by group: its L2 serves R to every group of a chunk, and with
// two groups of unlike size each compute unit gets one of either.
template <int MAXMB>
__global__ __launch_bounds__(kThreads, MAXMB == 4 ? 2 : MAXMB == 2 ? 3 : 4)
void k_blk_fold(BlkFoldArgs a, int n_blk, int n_groups) {
    __shared__ __attribute__((aligned(16))) double lds[2 * kStageRows * 16 * MAXMB];
    const int n_tile = a.n_ct * a.n_split, per_xcd = (n_tile + 7) / 8;
    const int tc = max(1, 64 / n_groups);
    const int u = blockIdx.x >> 3, ch = u / (tc * n_groups), ur = u - ch * tc * n_groups;
    const int cs = min(tc, per_xcd - ch * tc);
    const int g = ur / cs, t = (ch * tc + ur - g * cs) * 8 + (blockIdx.x & 7);
    if (t >= n_tile) return;
    const int ct = t % a.n_ct, sp = t / a.n_ct;
    const int b0 = (int)((long)n_blk * g / n_groups), b1 = (int)((long)n_blk * (g + 1) / n_groups);
    const int p0 = b0 * kBlkPts;
    const int nb = b1 - b0;
    if (MAXMB == 1 || nb == 1) fold_body<1>(a, ct, sp, p0, lds);
    else if (MAXMB == 2 || nb == 2) fold_body<MAXMB < 2 ? 1 : 2>(a, ct, sp, p0, lds);
    else if (nb == 3) fold_body<MAXMB < 3 ? 1 : 3>(a, ct, sp, p0, lds);
    else fold_body<MAXMB < 4 ? 1 : 4>(a, ct, sp, p0, lds);
}

// ---------------------------------------------------------------- finish
// 16 points x 32 columns per work-group, 16 lanes on a point with two columns each:
// the split sums in split order, sixteen of them in flight, then mu_j with
// backgrounds and mask, and the deviance mu - n + n ln(n / mu) as in the
// single-point reduction.  Bound by the latency of the splits' sums on short lists
// and by reading them on long ones: three points of 2048 rows x 1024 bins x 5
// components (64 splits) 7.6 us, 85 with one split's loads at a time; 100 points
// 11 us.
__global__ __launch_bounds__(kThreads) void k_blk_finish(BlkFinishArgs a) {
    static_assert(kBlkFinCols == 32, "two columns per lane");
    constexpr int U = 16;
    const int tid = threadIdx.x, pi = tid >> 4, c = tid & 15;
    const int j = blockIdx.x * kBlkFinCols + 2 * c, p = blockIdx.y * kBlkPts + pi;
    const bool okp = p < a.n_pts;
    const int pc = min(p, a.n_pts - 1);
    const double* src = a.part + (size_t)pc * a.ldr + min(j, a.ldr - 2);
    double2 s = make_double2(0.0, 0.0);
    for (int q = 0; q < a.n_split; q += U) {
        double2 t[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            t[u] = *reinterpret_cast<const double2*>(src + min(q + u, a.n_split - 1) * a.split_stride);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q + u < a.n_split) {
                s.x += t[u].x;
                s.y += t[u].y;
            }
    }
    double dsum = 0.0;
    const double* th = a.theta + (size_t)pc * a.n_theta;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int col = j + h;
        if (!okp || col >= a.n_reco) continue;
        double mu = h ? s.y : s.x;
        for (int q = 0; q < a.n_bkg; ++q)
            mu += th[a.bkg_index + q] * a.b[(size_t)q * a.n_reco + col];
        if (a.mask) mu *= a.mask[col];
        const double nj = a.n[col];
        if (a.out_mu) a.out_mu[(size_t)p * a.n_reco + col] = mu;
        if (nj > 0.0)
            dsum += mu > 0.0 ? (mu - nj + nj * log(nj / mu)) : INFINITY;
        else
            dsum += mu;
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o, 64);
    if (c == 0 && okp) a.dev[(size_t)p * a.n_ct + blockIdx.x] = dsum;
}

// -2lnL = 2 (sum of the column tiles' deviances + C_data) + pulls; 16 lanes on a
// point, each every sixteenth tile.
__global__ __launch_bounds__(64) void k_blk_final(BlkFinishArgs a) {
    const int c = threadIdx.x & 15, p = blockIdx.x * 4 + (threadIdx.x >> 4);
    const double* x = a.dev + (size_t)min(p, a.n_pts - 1) * a.n_ct;
    double d = 0.0;
#pragma unroll 8
    for (int q = c; q < a.n_ct; q += 16) d += x[q];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    if (c != 0 || p >= a.n_pts) return;
    double pulls = 0.0;
    for (int i = 0; i < a.n_theta; ++i)
        if (a.pull_sigma[i] > 0.0) {
            const double z = (a.theta[(size_t)p * a.n_theta + i] - a.pull_mean[i]) / a.pull_sigma[i];
            pulls += z * z;
        }
    a.nll[p] = 2.0 * d + 2.0 * a.cdata + pulls;
}

}  // namespace

hipError_t launch_pts_weights(const PtsWeightArgs& a, hipStream_t s) {
    if (a.n_pts <= 0 || a.n_pad < a.n_pts || a.n_pad > a.ldw || a.n_pad % 4)
        return hipErrorInvalidValue;
    const dim3 grid((a.n_t + kWtRows - 1) / kWtRows, (a.n_pad + kWtPts - 1) / kWtPts, a.n_comp);
    hipLaunchKernelGGL(k_pts_weights, grid, dim3(kThreads), 0, s, a);
    return hipGetLastError();
}

int blk_fold_lds_rows() { return kStageRows; }

hipError_t launch_blk_fold(const BlkFoldArgs& a, hipStream_t s) {
    if (a.n_pts <= 0 || a.ldw % kBlkPts || a.n_pts > a.ldw || a.ldr % 4 || a.rows_per <= 0 ||
        a.rows_per % kStageRows || (long)a.n_split * a.rows_per < a.n_rows ||
        a.n_ct != (a.ldr + kBlkCols - 1) / kBlkCols ||
        a.split_stride < (size_t)((a.n_pts + kBlkPts - 1) / kBlkPts * kBlkPts) * a.ldr)
        return hipErrorInvalidValue;
    const int n_blk = (a.n_pts + kBlkPts - 1) / kBlkPts;
    const int maxmb = n_blk == 1 ? 1 : n_blk == 2 ? 2 : 4;
    const int n_groups = (n_blk + maxmb - 1) / maxmb;
    const dim3 grid((a.n_ct * a.n_split + 7) / 8 * 8 * n_groups);
    if (maxmb == 1)
        hipLaunchKernelGGL(k_blk_fold<1>, grid, dim3(kThreads), 0, s, a, n_blk, n_groups);
    else if (maxmb == 2)
        hipLaunchKernelGGL(k_blk_fold<2>, grid, dim3(kThreads), 0, s, a, n_blk, n_groups);
    else
        hipLaunchKernelGGL(k_blk_fold<4>, grid, dim3(kThreads), 0, s, a, n_blk, n_groups);
    return hipGetLastError();
}

hipError_t launch_blk_finish(const BlkFinishArgs& a, hipStream_t s) {
    if (a.n_ct != (a.n_reco + kBlkFinCols - 1) / kBlkFinCols) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_blk_finish, dim3(a.n_ct, (a.n_pts + kBlkPts - 1) / kBlkPts),
                       dim3(kThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_blk_final, dim3((a.n_pts + 3) / 4), dim3(64), 0, s, a);
    return hipGetLastError();
}

}  // namespace nr
