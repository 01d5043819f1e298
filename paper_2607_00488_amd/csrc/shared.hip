// Basis form of the evaluation on gfx950 (shared.h): the recoil spectra of
// Eq. (fT) as folded columns shared by every point of a call, the spectra of
// Eqs. (fNp_reweight), (mu_total) and the Poisson -2lnL of Eq. (logL) with its
// gradient from them, FP64 throughout.
#include "shared.h"
#include "lnpos.h"
#include "lntab.h"

#include <algorithm>
#include <cmath>

// Every multiply-add of this file is written out: the kernels' size classes
// round alike, and a point's result does not depend on the class it falls in.
#pragma clang fp contract(off)

namespace nr {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v2d __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;

// Pointers that come out of a struct array are global memory; said so, the
// compiler emits global instead of flat accesses.
template <class T>
__device__ inline const __attribute__((address_space(1))) T* gm(const T* p) {
    return (const __attribute__((address_space(1))) T*)p;
}
template <class T>
__device__ inline __attribute__((address_space(1))) T* gm(T* p) {
    return (__attribute__((address_space(1))) T*)p;
}

// The analysis a work-group belongs to, and its index within it.
template <class P, int N>
__device__ inline int sh_find(const ShGroup<P, N>& g, int* wg) {
    int d = 0;
    if constexpr (N > 1) {
        int hi = g.n;
        while (hi - d > 1) {
            const int m = (d + hi) >> 1;
            if ((int)blockIdx.x >= g.first[m]) d = m;
            else hi = m;
        }
    }
    *wg = (int)blockIdx.x - g.first[d];
    return d;
}

// x[0] + x[st] + ... + x[(n - 1) st] in order, U of them in flight at a time.
template <int U>
__device__ inline double sum_strided(const __attribute__((address_space(1))) double* x, size_t st, int n) {
    double s = 0.0;
    for (int q = 0; q < n; q += U) {
        double v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = x[min(q + u, n - 1) * st];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q + u < n) s += v[u];
    }
    return s;
}

// ------------------------------------------------------------------ fold
// part[s][b][j] = sum over the rows l of split s of F_lb R_lj on the FP64
// matrix cores, b the row operand (15 of 16 used), the response columns the
// column operand.  Wave w owns 64 columns as four sets of 16 interleaved ones:
// lane (li, lk) loads the float4 of columns 4 li .. 4 li + 3 of row 4 q + lk,
// the column operand of four matrix instructions with k = lk, and F_{4q+lk, li}
// the same way (a row of F is 128 contiguous bytes, shared by the four waves
// through the cache), so nothing passes through LDS and no wave waits for
// another.  The next stage of 32 rows (8 KB of R per wave) is loaded
// unconditionally before the current one's arithmetic.
//
// Bound by the stream over R, with the matrix cores close behind (15 multiply-
// adds per entry: 32 us of arithmetic at 16384 x 4096, measured with R in
// cache).  16384 x 4096: 43 us, 6.2 TB/s, with one work-group per compute unit;
// two or three stages ahead 44 and 47 us; masks on the prefetched factors, which
// made every stage wait for the next one's loads, half as long again.
//
// That is W = 4.  Under band skipping only the tile x split pairs that meet the
// band have rows to fold, each bound by its own compute unit's matrix cores (1024
// rows x 256 columns: 32 us, however few of them there are).  For narrow bands W =
// 1: one set of 16 columns per wave, a float per lane and 64 rows per stage, a
// quarter of the work on four times the units; every column's sum is the same
// chain.  A stage's loads are fenced off its products, which left to itself the
// compiler moves them between (26 us where it is 16; W = 4 loses 1 us by it).
// 16384 x 4096, share of the rows of a tile inside its band 1/8: 37 -> 16 us; 5/16:
// 29; 9/16: 41 against 39, and 64 against 43 without bands.
//
// TALL: where too few tiles of 256 columns for a second split leave compute units
// idle, or just too many fill them unevenly (the rule: sh_plan).  The waves' sums are
// added in order through LDS, so that four times the work-groups write no more
// partial sums.  8000 x 34000 (133 wide tiles) 284 -> 225 us, 65536 x 36864 (144)
// 2264 -> 1847, 2048 x 40000 (157) 75 -> 67, 8000 x 49152 (192) 286 and 288.
//
// NT: responses larger than the Infinity Cache, in rows of whole cache lines, are
// read without leaving them in any cache: 20000 x 4096 59 -> 54 us, 32768 x 8192 176
// -> 162 (6.6 TB/s), 65536 x 36864 1847 -> 1731; 16384 x 4096, which just fits, 43
// against 45.  Where rows share lines, the second use would read them again: 8000 x
// 34000 225 against 241 us.
template <int N, int W, bool TALL, bool NT>
__global__ __launch_bounds__(kThreads, 2) void k_sh_fold(ShGroup<ShFold, N> g) {
    int t;
    const ShFold& a = g.p[sh_find(g, &t)];
    constexpr int ST = kShStage / 4 * (W == 1 ? 2 : 1), ROWS = 4 * ST;
    typedef float vec __attribute__((ext_vector_type(W)));
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lk = lane >> 4;
    // splits first: with their usual multiple of eight, an XCD's work-groups share
    // rows, and its L2 reads the row factors of those rows only, not of all (8 data
    // sets 71.2 -> 66.1 us a call; 100 points at 16384 x 4096 52.9 -> 52.3)
    const int ct = t / a.n_split, sp = t % a.n_split;
    const int ldr = a.ldr;
    const int col = (TALL ? ct : ct * 4 + wave) * 16 * W + W * li, cc = min(col, ldr - W);
    // the points of the call on their way to device memory: loaded here, stored
    // at the end
    const int gi = t * kThreads + tid, gn = a.n_ct * a.n_split * kThreads;
    double th = 0.0;
    if (a.th_src) {
        if (gi < a.n_th) th = gm(a.th_src)[gi];
        for (int i = gi + gn; i < a.n_th; i += gn) gm(a.th_dst)[i] = gm(a.th_src)[i];
    }
    const int rows = TALL ? a.rows_per / 4 : a.rows_per;
    int kb = sp * a.rows_per + (TALL ? wave * rows : 0), ke = min(a.n_t, kb + rows);
    if (a.band) {  // rows outside hold exact zeros in this tile's columns
        const int b = W == 4 && !TALL ? ct : ct / 4;
        kb = max(kb, gm(a.band)[2 * b]);
        ke = min(ke, gm(a.band)[2 * b + 1]);
    }
    const auto* R = (const __attribute__((address_space(1))) char*)a.R;
    const auto* F = (const __attribute__((address_space(1))) char*)a.rf;
    // byte offsets of a lane within a stage (n_reco < 2^27 columns)
    const unsigned roff = (unsigned)lk * ldr * 4u + 4u * cc;
    const unsigned foff = (lk * 16 + li) * 8u;
    const size_t rq = (size_t)ldr * 16;  // bytes of four rows
    v4d acc[W];
#pragma unroll
    for (int e = 0; e < W; ++e) acc[e] = (v4d){0.0, 0.0, 0.0, 0.0};
    struct Stage {
        vec x[ST];
        double f[ST];
    };
    auto ldx = [](const __attribute__((address_space(1))) char* p) {
        const auto* q = (const __attribute__((address_space(1))) vec*)p;
        if constexpr (NT) return __builtin_nontemporal_load(q);
        else return *q;
    };
    auto load = [&](int k, Stage& s) {
        const auto* rb = R + (size_t)k * ldr * 4;
        const auto* fb = F + (size_t)k * (kRF * 8);
#pragma unroll
        for (int q = 0; q < ST; ++q) {
            s.f[q] = *(const __attribute__((address_space(1))) double*)(fb + q * (kRF * 32) + foff);
            s.x[q] = ldx(rb + q * rq + roff);
        }
    };
    auto compute = [&](const Stage& s) {
#pragma unroll
        for (int q = 0; q < ST; ++q)
#pragma unroll
            for (int e = 0; e < W; ++e)
                acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(s.f[q], (double)s.x[q][e], acc[e], 0, 0, 0);
    };
    const int nst = kb < ke ? (ke - kb) / ROWS : 0;  // whole stages
    if (nst > 0) {  // the loads past the end repeat the last
        Stage s0, s1;
        auto at = [&](int i) { return kb + min(i, nst - 1) * ROWS; };
        load(at(0), s0);
        int i = 0;
        for (; i + 1 < nst; i += 2) {
            load(at(i + 1), s1);
            if (W == 1) __builtin_amdgcn_sched_barrier(0);
            compute(s0);
            load(at(i + 2), s0);
            if (W == 1) __builtin_amdgcn_sched_barrier(0);
            compute(s1);
        }
        if (i < nst) compute(s0);
    }
    // the last rows, all loaded at once; past the end a zero factor on the last row
    const int k0 = kb + nst * ROWS, left = ke - k0;
    if (left > 0) {
        Stage s;
#pragma unroll
        for (int q = 0; q < ST; ++q) {
            const int row = k0 + 4 * q + lk, rc = min(row, a.n_t - 1);
            s.f[q] = *(const __attribute__((address_space(1))) double*)(F + ((size_t)rc * kRF + li) * 8);
            s.x[q] = ldx(R + ((size_t)rc * ldr + cc) * 4);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < ST; ++q) {
            const double f = k0 + 4 * q + lk < ke ? s.f[q] : 0.0;
#pragma unroll
            for (int e = 0; e < W; ++e)
                acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(f, (double)s.x[q][e], acc[e], 0, 0, 0);
        }
    }
    if (a.th_src && gi < a.n_th) gm(a.th_dst)[gi] = th;
    if constexpr (TALL) {
        __shared__ __attribute__((aligned(16))) double red[4][16][kShSmallTile];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            auto* o = reinterpret_cast<v2d*>(&red[wave][lk + 4 * r][4 * li]);
            o[0] = (v2d){acc[0][r], acc[1][r]};
            o[1] = (v2d){acc[2][r], acc[3][r]};
        }
        __syncthreads();
        for (int i = tid; i < kShCols * kShSmallTile; i += kThreads) {
            const int b = i / kShSmallTile, j = i % kShSmallTile;
            if (ct * kShSmallTile + j < ldr)
                gm(a.part)[((size_t)sp * kShCols + b) * ldr + ct * kShSmallTile + j] =
                    ((red[0][b][j] + red[1][b][j]) + red[2][b][j]) + red[3][b][j];
        }
        return;
    }
    if (col >= ldr) return;
    auto* out = gm(a.part) + (size_t)sp * kShCols * ldr + col;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int b = lk + 4 * r;  // output (i, j): lane j + 16 (i % 4), register i / 4
        if (b >= kShCols) continue;
        auto* o = out + (size_t)b * ldr;
        if constexpr (W == 4) {
            ((__attribute__((address_space(1))) v2d*)o)[0] = (v2d){acc[0][r], acc[1][r]};
            ((__attribute__((address_space(1))) v2d*)o)[1] = (v2d){acc[2][r], acc[3][r]};
        } else {
            o[0] = acc[0][r];
        }
    }
}

// --------------------------------------------------------------- records
// One work-group per 16 bins: the split sums in split order, one (column, bin)
// per thread, and the bins' data; records leave as contiguous rows.  Bins past
// the last one (the tail of the last tile) get mu = 1, n = 1: a zero term.
template <int N>
__global__ __launch_bounds__(kThreads) void k_sh_rec(ShGroup<ShRec, N> g) {
    __shared__ double t[kShBins][kShRec];
    int wg;
    const ShRec& a = g.p[sh_find(g, &wg)];
    const int tid = threadIdx.x, b = tid >> 4, jl = tid & 15;
    const int j0 = wg * kShBins, j = j0 + jl;
    const bool ok = j < a.n_reco;
    if (b < kShCols) {
        double s = 0.0;
        if (ok) {
            s = sum_strided<16>(gm(a.part) + (size_t)b * a.ldr + j, (size_t)kShCols * a.ldr, a.n_split);
        } else if (b == kNBasis) {
            s = 1.0;
        }
        t[jl][b] = s;
    } else {
        const double n = ok ? gm(a.n)[j] : 1.0;
        t[jl][kShCols] = ok ? gm(a.b)[j] : 0.0;
        t[jl][kShCols + 1] = n;
        t[jl][kShCols + 2] = n > 0.0 ? 1.0 / n : 1.0;
    }
    __syncthreads();
    auto* out = gm(a.rec) + (size_t)j0 * kShRec;
    const double* src = &t[0][0];
    for (int i = tid; i < kShBins * kShRec; i += kThreads) out[i] = src[i];
}

__global__ __launch_bounds__(kThreads) void k_sh_data(ShRec a) {
    const int j = blockIdx.x * kThreads + threadIdx.x;
    if (j >= a.n_reco) return;
    double* r = a.rec + (size_t)j * kShRec;
    const double n = a.n[j];
    r[kShCols] = a.b[j];
    r[kShCols + 1] = n;
    r[kShCols + 2] = n > 0.0 ? 1.0 / n : 1.0;
}

// ---------------------------------------------------------------- points
// One wave: NB blocks of 16 points over one slice of bins, 16 bins at a time.
// mu is a product of the bins' records with the points' coefficients (16
// columns: the 14 spectra, the constant rows, b_j with f_bkg) on the FP64
// matrix cores, bins the row operand in an order that leaves a lane with the
// four consecutive bins 4 lk .. 4 lk + 3 of one point.  In that layout a_j is
// already the column operand of the gradient's contraction h = sum_j a_j G_j,
// a second product with the same records.  The vector units are left with the
// Poisson term: n ln(n / mu) as -n ln(mu (1 / n)), the logarithm of the ratio
// (near a fit's minimum the two logarithms agree to many digits, and their
// separate roundings would leave noise that stalls a line search).
//
// Bound by those vector instructions (about 25 per point and bin, 40 with the
// gradient) and the matrix instructions, which share the FP64 rate with them
// (64 cycles of about 150 per 64 elements).  65536 points x 4096 bins: 292 us in
// calls with pauses, 335-350 one after the other (the clock falls), against 510 with
// one point per lane and the series logarithm.
__device__ __constant__ const LnTable g_ln = make_ln_table();

// The terms that the fast path leaves out: an empty or underflowed spectrum, an
// overflowed one, NaN.  An empty bin's term is mu_j, its derivative 2.
__device__ __attribute__((noinline)) double2 sh_slow_term(double mu, double n) {
    double d = mu, a = 2.0;
    if (n > 0.0) {
        d = mu > 0.0 ? (isinf(mu) ? mu : mu - n + n * ln_pos(n / mu)) : INFINITY;
        a = 2.0 * (1.0 - n / mu);
    }
    return make_double2(d, a);
}

__device__ inline const __attribute__((address_space(1))) v2d* as_pair(
    const __attribute__((address_space(1))) double* p) {
    return (const __attribute__((address_space(1))) v2d*)p;
}
__device__ inline const v2d* as_pair(const double* p) { return reinterpret_cast<const v2d*>(p); }

template <int KS>
struct ShCoefs {  // the multi-component form's coefficients, a wave's 16 points
    static constexpr bool kMulti = KS != kShAcc / 4;
    double v[kMulti ? 16 : 1][kMulti ? 4 * KS + 1 : 1];
};

// One wave: the points from p0 over tiles [t0, t1) of slice sl; rec: the record of
// the first bin of tile t_rec.
template <bool GRAD, bool MU, int NB, int KS, class Rec>
__device__ __forceinline__ void sh_points(const ShEval& a, Rec rec, int t_rec, const LnTable& lt,
                                          ShCoefs<KS>& cs, int p0, int sl, int t0, int t1) {
    constexpr bool MULTI = ShCoefs<KS>::kMulti;
    constexpr int RL = 4 * KS + 2;          // record length
    constexpr int HB = (4 * KS + 15) / 16;  // blocks of 16 contractions
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4, n_pts = a.n_pts;
    // this lane's KS of each point's 4 KS coefficients (k = KS lk + s)
    double c[NB][KS];
    if constexpr (MULTI) {
        static_assert(NB == 1, "one block of points");
        const int p = min(p0 + li, n_pts - 1);
        const auto* th = gm(a.theta) + (size_t)p * a.n_theta;
        auto& row = cs.v[li];
        double t5[5], v[kCompBasis];
#pragma unroll
        for (int i = 0; i < 5; ++i) t5[i] = th[i];
        basis_coef7(t5, a.ph, 1.0, v);
        for (int k = lk; k < a.K; k += 4) {
            const double r = th[5 + k];
#pragma unroll
            for (int b = 0; b < kCompBasis; ++b) row[kShCompCols * k + b] = r * v[b];
            row[kShCompCols * k + kCompBasis] = r;
        }
        for (int q = kShCompCols * a.K + lk; q < 4 * KS; q += 4) {
            const int b = q - kShCompCols * a.K;
            row[q] = b < a.B ? th[5 + a.K + b] : 0.0;
        }
        // written and read by this wave alone
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int s = 0; s < KS; ++s) c[0][s] = row[KS * lk + s];
    } else {
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            const int p = min(p0 + 16 * x + li, n_pts - 1);
            double th[kNTheta], v[16];
#pragma unroll
            for (int i = 0; i < kNTheta; ++i) th[i] = gm(a.theta)[(size_t)p * kNTheta + i];
            basis_coef(th, a.ph, v);
            v[kNBasis] = 1.0;
            v[kNBasis + 1] = th[6];
#pragma unroll
            for (int s = 0; s < 4; ++s)
                c[x][s] = lk == 0 ? v[s] : lk == 1 ? v[4 + s] : lk == 2 ? v[8 + s] : v[12 + s];
        }
    }
    // row operand i holds bin 4 (i % 4) + i / 4: output register r of lane
    // group lk is then bin 4 lk + r
    const int fb = (4 * (li & 3) + (li >> 2)) * RL + KS * lk;
    struct Tile {
        double f[KS];      // record columns KS lk .. of this lane's row bin
        v2d n[4];          // n, 1 / n of bins 4 lk + r
        double gr[HB][4];  // columns 16 y + li of bins 4 lk + r
    };
    auto load = [&](int t, Tile& q) {
        const auto* r = rec + (t - t_rec) * (kShBins * RL);
        if constexpr (KS % 2 == 0) {
            const auto* f = as_pair(r + fb);
#pragma unroll
            for (int s = 0; s < KS / 2; ++s) {
                const v2d v = f[s];
                q.f[2 * s] = v.x;
                q.f[2 * s + 1] = v.y;
            }
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) q.f[s] = r[fb + s];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const auto* b = r + (4 * lk + e) * RL;
            q.n[e] = *as_pair(b + 4 * KS);
            if (GRAD)
#pragma unroll
                for (int y = 0; y < HB; ++y)  // the last block may end past the columns
                    q.gr[y][e] = (4 * KS) % 16 == 0 || 16 * y + li < 4 * KS ? b[16 * y + li] : 0.0;
        }
    };
    double dsum[NB];
    v4d h[NB][HB];
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        dsum[x] = 0.0;
#pragma unroll
        for (int y = 0; y < HB; ++y) h[x][y] = (v4d){0.0, 0.0, 0.0, 0.0};
    }
    const bool mu16 = MU && a.n_reco % 2 == 0 && ((size_t)a.mu & 15) == 0;
    Tile cur, nxt;
    load(t0, cur);
    for (int t = t0; t < t1; ++t) {
        load(min(t + 1, t1 - 1), nxt);
#pragma unroll
        for (int x = 0; x < NB; ++x) {
            v4d mu = (v4d){0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < KS; ++s)
                mu = __builtin_amdgcn_mfma_f64_16x16x4f64(cur.f[s], c[x][s], mu, 0, 0, 0);
            const int p = p0 + 16 * x + li, j = t * kShBins + 4 * lk;
            if (MU && p < n_pts) {
                auto* o = gm(a.mu) + (size_t)p * a.n_reco + j;
                if (mu16 && j + 3 < a.n_reco) {
                    ((__attribute__((address_space(1))) v2d*)o)[0] = (v2d){mu[0], mu[1]};
                    ((__attribute__((address_space(1))) v2d*)o)[1] = (v2d){mu[2], mu[3]};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (j + r < a.n_reco) o[r] = mu[r];
                }
            }
            double dv[4], av[4];
            bool fast = true;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double n = cur.n[r].x, q = mu[r] * cur.n[r].y;
                // positive and normal
                fast = fast && __builtin_amdgcn_class(q, 0x100);
                if (GRAD) fast = fast && __builtin_amdgcn_class(mu[r], 0x100);
                dv[r] = fma(-n, ln_tab(q, lt.e), mu[r] - n);
                if (GRAD) {
                    double y = __builtin_amdgcn_rcp(mu[r]);
                    y = fma(y, fma(-mu[r], y, 1.0), y);
                    y = fma(y, fma(-mu[r], y, 1.0), y);
                    double u = n * y;
                    u = fma(fma(-mu[r], u, n), y, u);
                    av[r] = 2.0 * (1.0 - u);
                }
            }
            if (!fast) {
#pragma unroll 1
                for (int r = 0; r < 4; ++r) {
                    const double m = r == 0 ? mu[0] : r == 1 ? mu[1] : r == 2 ? mu[2] : mu[3];
                    const double n = r == 0 ? cur.n[0].x : r == 1 ? cur.n[1].x : r == 2 ? cur.n[2].x : cur.n[3].x;
                    double2 s = sh_slow_term(m, n);
                    if (j + r >= a.n_reco) s = make_double2(0.0, 0.0);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (e == r) {
                            dv[e] = s.x;
                            if (GRAD) av[e] = s.y;
                        }
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                dsum[x] += dv[r];
                if (GRAD)
#pragma unroll
                    for (int y = 0; y < HB; ++y)
                        h[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur.gr[y][r], av[r], h[x][y],
                                                                       0, 0, 0);
            }
        }
        cur = nxt;
    }
#pragma unroll
    for (int x = 0; x < NB; ++x) {
        const int p = p0 + 16 * x + li;
        double s = dsum[x];
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (p >= n_pts) continue;
        if (lk == 0) gm(a.dpart)[(size_t)sl * n_pts + p] = s;
        if (GRAD)
#pragma unroll
            for (int y = 0; y < HB; ++y)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    gm(a.hpart)[((size_t)sl * (16 * HB) + 16 * y + lk + 4 * r) * n_pts + p] = h[x][y][r];
    }
}


template <bool GRAD, bool MU, int NB, int KS, int N>
__global__ __launch_bounds__(kThreads) void k_sh_eval(ShGroup<ShEval, N> g) {
    __shared__ LnTable lt;
    __shared__ ShCoefs<KS> cs[4];
    int wg;
    const ShEval& a = g.p[sh_find(g, &wg)];
    const int tid = threadIdx.x;
    static_assert(kThreads == kLnTab, "one table entry per thread");
    lt.e[tid] = g_ln.e[tid];
    __syncthreads();
    const int n_grp = (a.n_pts + 16 * NB - 1) / (16 * NB);
    const int w = wg * 4 + (tid >> 6), sl = w / n_grp, p0 = (w - sl * n_grp) * 16 * NB;
    if (sl >= a.n_slice) return;
    const int n_tile = (a.n_reco + kShBins - 1) / kShBins;
    const int t0 = sl * a.tiles, t1 = min(n_tile, t0 + a.tiles);
    sh_points<GRAD, MU, NB, KS>(a, gm(a.rec), 0, lt, cs[tid >> 6], p0, sl, t0, t1);
}

constexpr int kTailThreads = 64 * (kShCols + 1);

// Short lists: one launch makes the records of one slice of bins, in LDS, and
// takes every point over them, instead of a launch for either with the records in
// memory between (each costs about 4 us whatever it does).  With many points
// several work-groups share a slice, each adding up its splits again: sixteen
// splits of every column in flight at once (a wave per column; four waves of four
// columns waited twice as often: one point at 16384 x 4096 67.6 -> 66.4 us).
template <bool GRAD, bool MU, int N>
__global__ __launch_bounds__(kTailThreads) void k_sh_tail(ShGroup<ShTail, N> g) {
    __shared__ LnTable lt;
    __shared__ ShCoefs<kShAcc / 4> cs;  // unused by this form
    __shared__ __attribute__((aligned(16))) double rec[kShTailBins][kShRec];
    int wg;
    const ShTail& q = g.p[sh_find(g, &wg)];
    const ShRec& r = q.r;
    const ShEval& a = q.e;
    const int tid = threadIdx.x, wave = tid >> 6, sl = wg % a.n_slice, y = wg / a.n_slice;
    const int j0 = sl * kShTailBins;
    // one bin per lane, one column per wave (the last wave: the bin's data)
    {
        const int jl = tid & 63, j = j0 + jl, jc = min(j, r.n_reco - 1);
        const bool ok = j < r.n_reco;
        if (wave < kShCols) {
            const double s = sum_strided<16>(gm(r.part) + (size_t)wave * r.ldr + jc,
                                             (size_t)kShCols * r.ldr, r.n_split);
            rec[jl][wave] = ok ? s : wave == kNBasis ? 1.0 : 0.0;
        } else {
            const double n = ok ? gm(r.n)[jc] : 1.0;
            rec[jl][kShCols] = ok ? gm(r.b)[jc] : 0.0;
            rec[jl][kShCols + 1] = n;
            rec[jl][kShCols + 2] = n > 0.0 ? 1.0 / n : 1.0;
        }
        if (tid < kThreads) lt.e[tid] = g_ln.e[tid];
    }
    __syncthreads();
    const int n_tile = (a.n_reco + kShBins - 1) / kShBins;
    const int t0 = sl * a.tiles, t1 = min(n_tile, t0 + a.tiles);
    const int n_blk = (a.n_pts + 15) / 16;
    for (int b = wave * q.ny + y; b < n_blk; b += q.ny * (kTailThreads / 64))
        sh_points<GRAD, MU, 1, kShAcc / 4>(a, &rec[0][0], t0, lt, cs, 16 * b, sl, t0, t1);
}

// ----------------------------------------------------------------- final
// -2lnL = 2 (sum of the slices' deviances + C_data) + pulls.
__device__ inline double sh_nll(const ShFinal& a, double dev, const double th[kNTheta]) {
    double pulls = 0.0;
#pragma unroll
    for (int i = 0; i < kNTheta; ++i)
        if (a.pull_sigma[i] > 0.0) {
            const double z = (th[i] - a.pull_mean[i]) / a.pull_sigma[i];
            pulls += z * z;
        }
    return 2.0 * dev + 2.0 * a.cdata + pulls;
}

// The slices of one quantity: the two halves, each in order, by two threads.
template <class T>
__device__ inline double sh_half(const T* x, size_t st, int n, int half) {
    const int h = (n + 1) / 2, q0 = half ? h : 0, q1 = half ? n : h;
    return q0 < q1 ? sum_strided<16>(gm(x) + q0 * st, st, q1 - q0) : 0.0;
}

// The same two sums for one point by a whole wave, its many slices through LDS: read
// side by side, added in order.  One point of 40000 bins (625 slices) 5.2 us instead
// of 12.9, most of it the address arithmetic and rounds of two threads.
__device__ inline double sh_point_sum(const double* x, size_t st, int n) {
    constexpr int C = 512;
    __shared__ double buf[C];
    const int lane = threadIdx.x, h = (n + 1) / 2;
    double s = 0.0;  // lanes 0 and 1: the halves
    for (int q0 = 0; q0 < n; q0 += C) {
        double v[C / 64];
#pragma unroll
        for (int i = 0; i < C / 64; ++i) v[i] = gm(x)[min(q0 + 64 * i + lane, n - 1) * st];
        __syncthreads();  // the last piece has been added
#pragma unroll
        for (int i = 0; i < C / 64; ++i) buf[64 * i + lane] = v[i];
        __syncthreads();
        if (lane < 2) {
            const int hi = min(lane ? n : h, q0 + C) - q0;
            int q = max(lane ? h : 0, q0) - q0;
            for (; q + 16 <= hi; q += 16) {
                double y[16];
#pragma unroll
                for (int u = 0; u < 16; ++u) y[u] = buf[q + u];
#pragma unroll
                for (int u = 0; u < 16; ++u) s += y[u];
            }
            for (; q < hi; ++q) s += buf[q];
        }
    }
    return __shfl(s, 0, 64) + __shfl(s, 1, 64);
}

// 32 points per work-group; lists of one or two with many slices point by point.
template <int N>
__global__ __launch_bounds__(64) void k_sh_final(ShGroup<ShFinal, N> g) {
    int wg;
    const ShFinal& a = g.p[sh_find(g, &wg)];
    if (a.n_pts <= 2 && a.n_slice > 128) {
        for (int p = 0; p < a.n_pts; ++p) {
            double th[kNTheta];
#pragma unroll
            for (int i = 0; i < kNTheta; ++i) th[i] = gm(a.theta)[(size_t)p * kNTheta + i];
            const double d = sh_point_sum(a.dpart + p, a.n_pts, a.n_slice);
            if (threadIdx.x == 0) gm(a.nll)[p] = sh_nll(a, d, th);
        }
        return;
    }
    const int pl = threadIdx.x & 31, p = wg * 32 + pl, pc = min(p, a.n_pts - 1);
    double th[kNTheta];
#pragma unroll
    for (int i = 0; i < kNTheta; ++i) th[i] = gm(a.theta)[(size_t)pc * kNTheta + i];
    double d = sh_half(a.dpart + pc, a.n_pts, a.n_slice, threadIdx.x >> 5);
    d += __shfl_xor(d, 32, 64);
    if (threadIdx.x < 32 && p < a.n_pts) gm(a.nll)[p] = sh_nll(a, d, th);
}

// 8 points per work-group, one half of one (contraction, point) per thread; the
// constant column's contraction is not needed, its threads sum the deviances.
template <int N>
__global__ __launch_bounds__(kThreads) void k_sh_final_grad(ShGroup<ShFinal, N> g) {
    __shared__ double hs[2][8][kShAcc + 1], ths[8][kNTheta];
    int wg;
    const ShFinal& a = g.p[sh_find(g, &wg)];
    const int half = threadIdx.x >> 7, v = (threadIdx.x >> 3) & 15, pl = threadIdx.x & 7;
    const int p = wg * 8 + pl, pc = min(p, a.n_pts - 1);
    if (half == 0 && v < kNTheta) ths[pl][v] = gm(a.theta)[(size_t)pc * kNTheta + v];
    hs[half][pl][v] = v == kNBasis ? sh_half(a.dpart + pc, a.n_pts, a.n_slice, half)
                                   : sh_half(a.hpart + (size_t)v * a.n_pts + pc,
                                             (size_t)kShAcc * a.n_pts, a.n_slice, half);
    __syncthreads();
    if (threadIdx.x >= 8 || p >= a.n_pts) return;
    double th[kNTheta], gr[kNTheta], hh[kNBasis];
#pragma unroll
    for (int i = 0; i < kNTheta; ++i) th[i] = ths[pl][i];
#pragma unroll
    for (int b = 0; b < kNBasis; ++b) hh[b] = hs[0][pl][b] + hs[1][pl][b];
    basis_grad(th, a.ph, hh, gr);
    gr[6] = hs[0][pl][kNBasis + 1] + hs[1][pl][kNBasis + 1];
    gm(a.nll)[p] = sh_nll(a, hs[0][pl][kNBasis] + hs[1][pl][kNBasis], th);
#pragma unroll
    for (int i = 0; i < kNTheta; ++i) {
        double q = gr[i];
        if (a.pull_sigma[i] > 0.0)
            q += 2.0 * (th[i] - a.pull_mean[i]) / (a.pull_sigma[i] * a.pull_sigma[i]);
        gm(a.grad)[(size_t)p * kNTheta + i] = q;
    }
}

// ------------------------------------------------- multi-component form
// One thread per reco bin, one work-group row per slab of one component's
// response rows: the FP64 sums of F_lb R_lj (the row's factors wave-uniform).
__global__ __launch_bounds__(kThreads) void k_sh_mfold(ShMultiFold a) {
    const int j = blockIdx.x * kThreads + threadIdx.x;
    if (j >= a.n_reco) return;
    const int l0 = blockIdx.y * kShSlabRows, l1 = min(l0 + kShSlabRows, a.n_t);
    double acc[kRFComp];
#pragma unroll
    for (int b = 0; b < kRFComp; ++b) acc[b] = 0.0;
    for (int l = l0; l < l1; ++l) {
        const double r = a.R[(size_t)l * a.ldr + j];
        const double* f = a.rf + (size_t)l * kRFComp;
#pragma unroll
        for (int b = 0; b < kRFComp; ++b) acc[b] = fma(f[b], r, acc[b]);
    }
#pragma unroll
    for (int b = 0; b < kRFComp; ++b)
        a.part[((size_t)blockIdx.y * kRFComp + b) * a.n_reco + j] = acc[b];
}

// Slab sums in slab order, times the mask, into the component's columns.
__global__ __launch_bounds__(kThreads) void k_sh_mrec(ShMultiRec a) {
    const int j = blockIdx.x * kThreads + threadIdx.x, b = blockIdx.y;
    if (j >= a.n_reco) return;
    double s = 0.0;
    for (int q = 0; q < a.n_slab; ++q) s += a.part[((size_t)q * kRFComp + b) * a.n_reco + j];
    a.rec[(size_t)j * (a.cols + 2) + kShCompCols * a.comp + b] = a.mask ? s * a.mask[j] : s;
}

// Backgrounds, zero columns and data.  Bins past the last one hold zeros: their
// mu = 0 takes the points kernel's slow term, which leaves them out.
__global__ __launch_bounds__(kThreads) void k_sh_mdata(ShMultiData a) {
    const int j = blockIdx.x * kThreads + threadIdx.x;
    const int n_pad = (a.n_reco + kShBins - 1) / kShBins * kShBins;
    if (j >= n_pad) return;
    double* r = a.rec + (size_t)j * (a.cols + 2);
    const bool ok = j < a.n_reco;
    const double m = ok && a.mask ? a.mask[j] : 1.0;
    if (!ok)
        for (int q = 0; q < kShCompCols * a.K; ++q) r[q] = 0.0;
    for (int q = kShCompCols * a.K; q < a.cols; ++q) {
        const int b = q - kShCompCols * a.K;
        r[q] = ok && b < a.B ? a.bkg[(size_t)b * a.n_reco + j] * m : 0.0;
    }
    const double n = ok ? a.n[j] : 0.0;
    r[a.cols] = n;
    r[a.cols + 1] = n > 0.0 ? 1.0 / n : 1.0;
}

template <class T>
__device__ inline double sh_mnll(const ShMultiFinal& a, const T* th, double dev) {
    double pulls = 0.0;
    for (int i = 0; i < a.n_theta; ++i)
        if (a.pull_sigma[i] > 0.0) {
            const double z = (th[i] - a.pull_mean[i]) / a.pull_sigma[i];
            pulls += z * z;
        }
    return 2.0 * dev + 2.0 * a.cdata + pulls;
}

__global__ __launch_bounds__(64) void k_sh_mfinal(ShMultiFinal a) {
    const int p = blockIdx.x * 64 + threadIdx.x;
    if (p >= a.n_pts) return;
    const double d = sh_half(a.dpart + p, a.n_pts, a.n_slice, 0) +
                     sh_half(a.dpart + p, a.n_pts, a.n_slice, 1);
    gm(a.nll)[p] = sh_mnll(a, gm(a.theta) + (size_t)p * a.n_theta, d);
}

// 16 points per work-group: the slices of every contraction, then
//   d/d theta_i (i < 5) = sum_k r_k sum_b dc_ib h_kb,
//   d/d r_k = sum_b c_b h_kb + h_k,const,  d/d r_q = h_q,
// written as whole rows.
template <int COLS>
__global__ __launch_bounds__(kThreads) void k_sh_mfinal_grad(ShMultiFinal a) {
    constexpr int ACC = (COLS + 15) / 16 * 16;
    __shared__ double hs[16][COLS + 1];
    __shared__ double dv[16];
    __shared__ double gs[16][kMaxTheta + 1], ths[16][kMaxTheta + 1];
    const int v0 = threadIdx.x >> 4, pl = threadIdx.x & 15, p0 = blockIdx.x * 16, p = p0 + pl;
    const int n_col = kShCompCols * a.K + a.B;
    const int n_row = min(16, a.n_pts - p0);
    for (int i = threadIdx.x; i < n_row * a.n_theta; i += kThreads)
        ths[i / a.n_theta][i % a.n_theta] = gm(a.theta)[(size_t)p0 * a.n_theta + i];
    if (p < a.n_pts) {
        for (int v = v0; v <= n_col; v += 16) {  // v = n_col: the deviance
            const bool dev = v == n_col;
            const double* x = dev ? a.dpart + p : a.hpart + (size_t)v * a.n_pts + p;
            const size_t st = (size_t)(dev ? 1 : ACC) * a.n_pts;
            const double s = sh_half(x, st, a.n_slice, 0) + sh_half(x, st, a.n_slice, 1);
            if (dev) dv[pl] = s;
            else hs[pl][v] = s;
        }
    }
    __syncthreads();
    if (v0 == 0 && p < a.n_pts) {
        const double* th = ths[pl];
        double t5[5], c[kCompBasis], H[kCompBasis], g5[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        for (int i = 0; i < 5; ++i) t5[i] = th[i];
        basis_coef7(t5, a.ph, 1.0, c);
        for (int b = 0; b < kCompBasis; ++b) H[b] = 0.0;
        for (int k = 0; k < a.K; ++k) {
            const double* h = &hs[pl][kShCompCols * k];
            const double r = th[5 + k];
            double R = h[kCompBasis];
            for (int b = 0; b < kCompBasis; ++b) {
                H[b] = fma(r, h[b], H[b]);
                R = fma(c[b], h[b], R);
            }
            gs[pl][5 + k] = R;
        }
        basis_dcoef7(t5, a.ph, 1.0, H, g5);
        for (int i = 0; i < 5; ++i) gs[pl][i] = g5[i];
        for (int q = 0; q < a.B; ++q) gs[pl][5 + a.K + q] = hs[pl][kShCompCols * a.K + q];
        for (int i = 0; i < a.n_theta; ++i)
            if (a.pull_sigma[i] > 0.0)
                gs[pl][i] += 2.0 * (th[i] - a.pull_mean[i]) / (a.pull_sigma[i] * a.pull_sigma[i]);
        gm(a.nll)[p] = sh_mnll(a, th, dv[pl]);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n_row * a.n_theta; i += kThreads)
        gm(a.grad)[(size_t)p0 * a.n_theta + i] = gs[i / a.n_theta][i % a.n_theta];
}

// One analysis travels in a struct of its own size, several in one of
// kShGroup (at most 4 KB of kernel arguments).
template <class P, int N, class Wgs>
ShGroup<P, N> make_group(const P* p, int n, Wgs wgs) {
    static_assert(sizeof(ShGroup<P, N>) <= 4096, "kernel arguments");
    ShGroup<P, N> g;
    g.n = n;
    g.first[0] = 0;
    for (int d = 0; d < n; ++d) {
        g.p[d] = p[d];
        g.first[d + 1] = g.first[d] + wgs(p[d]);
    }
    return g;
}

#define SH_LAUNCH(KERNEL, P, THREADS, WGS)                                              \
    do {                                                                                \
        if (n == 1) {                                                                   \
            const ShGroup<P, 1> g_ = make_group<P, 1>(p, 1, WGS);                       \
            hipLaunchKernelGGL(KERNEL(1), dim3(g_.first[1]), dim3(THREADS), 0, s, g_);  \
        } else {                                                                        \
            const ShGroup<P, kShGroup> g_ = make_group<P, kShGroup>(p, n, WGS);         \
            hipLaunchKernelGGL(KERNEL(kShGroup), dim3(g_.first[n]), dim3(THREADS), 0, s, g_); \
        }                                                                               \
    } while (0)

template <int W, bool TALL, bool NT>
void launch_fold(const ShFold* p, int n, hipStream_t s) {
#define SH_K(M) (k_sh_fold<M, W, TALL, NT>)
    SH_LAUNCH(SH_K, ShFold, kThreads, [](const ShFold& f) { return f.n_ct * f.n_split; });
#undef SH_K
}

template <bool GRAD, bool MU, int NB, int KS = kShAcc / 4>
void launch_eval(const ShEval* p, int n, hipStream_t s) {
    const auto wgs = [](const ShEval& e) {
        const int grp = (e.n_pts + 16 * NB - 1) / (16 * NB);
        return (int)(((long)grp * e.n_slice + 3) / 4);
    };
    if constexpr (KS == kShAcc / 4) {
#define SH_K(M) (k_sh_eval<GRAD, MU, NB, KS, M>)
        SH_LAUNCH(SH_K, ShEval, kThreads, wgs);
#undef SH_K
    } else {
        const ShGroup<ShEval, 1> g = make_group<ShEval, 1>(p, 1, wgs);
        hipLaunchKernelGGL((k_sh_eval<GRAD, MU, NB, KS, 1>), dim3(g.first[1]), dim3(kThreads), 0, s, g);
    }
}

template <bool GRAD, bool MU>
void launch_eval_nb(const ShEval* p, int n, hipStream_t s) {
    if (p[0].K) {
        // every column is a step of both products: one component, 1500 bins, 20000 points
        // with the gradient 171 us by the former kernel, which skipped absent columns,
        // 238 with the 44 of the solar species, 125 with 12
        const int cols = sh_cols(p[0].K, p[0].B);
        if (cols == kShTiny) launch_eval<GRAD, MU, 1, kShTiny / 4>(p, n, s);
        else if (cols == kShSmall) launch_eval<GRAD, MU, 1, kShSmall / 4>(p, n, s);
        else launch_eval<GRAD, MU, 1, kShLarge / 4>(p, n, s);
        return;
    }
    long waves = 0;  // of one block of 16 points each
    for (int d = 0; d < n; ++d) waves += (long)((p[d].n_pts + 15) / 16) * p[d].n_slice;
    // more blocks per wave share the record loads, but only once the chip's
    // 1024 SIMDs stay full
    if (waves >= 16384) launch_eval<GRAD, MU, 4>(p, n, s);
    else if (waves >= 8192) launch_eval<GRAD, MU, 2>(p, n, s);
    else launch_eval<GRAD, MU, 1>(p, n, s);
}

}  // namespace

hipError_t launch_sh_fold(const ShFold* p, int n, hipStream_t s) {
    if (n < 1 || n > kShGroup) return hipErrorInvalidValue;
    for (int d = 0; d < n; ++d)
        if (p[d].ldr % 4 || p[d].rows_per <= 0 || p[d].rows_per % kShStage || p[d].ldr >= (1 << 27) ||
            p[d].n_ct != sh_tiles(p[d].ldr, p[d].kind) || p[d].n_split < 1 ||
            (p[d].kind == kShTall && p[d].rows_per % (4 * kShStage)) ||
            (long)p[d].n_split * p[d].rows_per < p[d].n_t)
            return hipErrorInvalidValue;
    // one launch for each kind of tile and load
    for (const ShKind kind : {kShWide, kShNarrow, kShTall})
        for (const bool nt : {false, true}) {
            ShFold q[kShGroup];
            int m = 0;
            for (int d = 0; d < n; ++d)
                if (p[d].kind == kind && (kind != kShNarrow && p[d].stream) == nt) q[m++] = p[d];
            if (!m) continue;
            if (kind == kShNarrow) launch_fold<1, false, false>(q, m, s);
            else if (kind == kShWide && nt) launch_fold<4, false, true>(q, m, s);
            else if (kind == kShWide) launch_fold<4, false, false>(q, m, s);
            else if (nt) launch_fold<4, true, true>(q, m, s);
            else launch_fold<4, true, false>(q, m, s);
        }
    return hipGetLastError();
}

hipError_t launch_sh_rec(const ShRec* p, int n, hipStream_t s) {
    if (n < 1 || n > kShGroup) return hipErrorInvalidValue;
#define SH_K(M) (k_sh_rec<M>)
    SH_LAUNCH(SH_K, ShRec, kThreads, [](const ShRec& r) { return (r.n_reco + kShBins - 1) / kShBins; });
#undef SH_K
    return hipGetLastError();
}

hipError_t launch_sh_data(const ShRec& p, hipStream_t s) {
    hipLaunchKernelGGL(k_sh_data, dim3((p.n_reco + kThreads - 1) / kThreads), dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_sh_eval(const ShEval* p, int n, hipStream_t s) {
    if (n < 1 || n > kShGroup) return hipErrorInvalidValue;
    for (int d = 0; d < n; ++d)
        if (p[d].n_pts < 1 || !p[d].hpart != !p[0].hpart || !p[d].mu != !p[0].mu ||
            (p[d].hpart && p[d].mu) || (p[d].K && (n > 1 || p[d].K > kShMaxComp || p[d].B > kShMaxBkg ||
                                                   p[d].n_theta != 5 + p[d].K + p[d].B)) ||
            (long)p[d].tiles * p[d].n_slice * kShBins < p[d].n_reco)
            return hipErrorInvalidValue;
    if (p[0].hpart) launch_eval_nb<true, false>(p, n, s);
    else if (p[0].mu) launch_eval_nb<false, true>(p, n, s);
    else launch_eval_nb<false, false>(p, n, s);
    return hipGetLastError();
}

hipError_t launch_sh_tail(const ShTail* p, int n, hipStream_t s) {
    if (n < 1 || n > kShGroup) return hipErrorInvalidValue;
    for (int d = 0; d < n; ++d)
        if (p[d].ny < 1 || p[d].e.tiles * kShBins != kShTailBins || p[d].e.K ||
            !p[d].e.hpart != !p[0].e.hpart || !p[d].e.mu != !p[0].e.mu ||
            (p[d].e.hpart && p[d].e.mu) || p[d].r.n_reco != p[d].e.n_reco ||
            (long)kShTailBins * p[d].e.n_slice < p[d].e.n_reco)
            return hipErrorInvalidValue;
    const auto wgs = [](const ShTail& t) { return t.e.n_slice * t.ny; };
    if (p[0].e.hpart) {
#define SH_K(M) (k_sh_tail<true, false, M>)
        SH_LAUNCH(SH_K, ShTail, kTailThreads, wgs);
#undef SH_K
    } else if (p[0].e.mu) {
#define SH_K(M) (k_sh_tail<false, true, M>)
        SH_LAUNCH(SH_K, ShTail, kTailThreads, wgs);
#undef SH_K
    } else {
#define SH_K(M) (k_sh_tail<false, false, M>)
        SH_LAUNCH(SH_K, ShTail, kTailThreads, wgs);
#undef SH_K
    }
    return hipGetLastError();
}

hipError_t launch_sh_final(const ShFinal* p, int n, hipStream_t s) {
    if (n < 1 || n > kShGroup) return hipErrorInvalidValue;
    for (int d = 0; d < n; ++d)
        if (!p[d].grad != !p[0].grad || (p[d].grad && !p[d].hpart)) return hipErrorInvalidValue;
    if (p[0].grad) {
#define SH_K(M) (k_sh_final_grad<M>)
        SH_LAUNCH(SH_K, ShFinal, kThreads, [](const ShFinal& f) { return (f.n_pts + 7) / 8; });
#undef SH_K
    } else {
#define SH_K(M) (k_sh_final<M>)
        SH_LAUNCH(SH_K, ShFinal, 64, [](const ShFinal& f) { return (f.n_pts + 31) / 32; });
#undef SH_K
    }
    return hipGetLastError();
}

hipError_t launch_sh_mfold(const ShMultiFold& p, hipStream_t s) {
    hipLaunchKernelGGL(k_sh_mfold, dim3((p.n_reco + kThreads - 1) / kThreads,
                                        (p.n_t + kShSlabRows - 1) / kShSlabRows),
                       dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_sh_mrec(const ShMultiRec& p, hipStream_t s) {
    hipLaunchKernelGGL(k_sh_mrec, dim3((p.n_reco + kThreads - 1) / kThreads, kRFComp),
                       dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_sh_mdata(const ShMultiData& p, hipStream_t s) {
    hipLaunchKernelGGL(k_sh_mdata, dim3((p.n_reco + kShBins + kThreads - 1) / kThreads),
                       dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_sh_mfinal(const ShMultiFinal& p, hipStream_t s) {
    if (p.K < 1 || p.K > kShMaxComp || p.B > kShMaxBkg || (p.grad && !p.hpart))
        return hipErrorInvalidValue;
    if (!p.grad)
        hipLaunchKernelGGL(k_sh_mfinal, dim3((p.n_pts + 63) / 64), dim3(64), 0, s, p);
    else if (sh_cols(p.K, p.B) == kShTiny)
        hipLaunchKernelGGL(k_sh_mfinal_grad<kShTiny>, dim3((p.n_pts + 15) / 16), dim3(kThreads), 0, s, p);
    else if (sh_cols(p.K, p.B) == kShSmall)
        hipLaunchKernelGGL(k_sh_mfinal_grad<kShSmall>, dim3((p.n_pts + 15) / 16), dim3(kThreads), 0, s, p);
    else
        hipLaunchKernelGGL(k_sh_mfinal_grad<kShLarge>, dim3((p.n_pts + 15) / 16), dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

// Slices of 64 bins up to 4096 points (fixed by the response's shape, so that a
// point's result does not depend on its list); beyond, as few as fill whole rounds
// of resident waves of 64 points, since every slice writes its sums for every
// point: 6144 are two rounds of the likelihood kernel's three waves per SIMD and
// three of the gradient's two (65536 x 4096: 3072 to 16384 waves within 5 %).
// The multi-component form writes three to five times as many: one round of its
// gradient's two waves of 16 points per SIMD.
constexpr int kSliceTiles = 4;       // of short lists
constexpr int kShortPts = 4096;
constexpr int kWaves = 6144, kMultiWaves = 2048;

void sh_slices(int n_pts, int n_reco, bool multi, int* tiles, int* n_slice) {
    const int n_tile = (n_reco + kShBins - 1) / kShBins;
    int t = kSliceTiles;
    const int grp = multi ? (n_pts + 15) / 16 : (n_pts + 63) / 64;
    if (multi || n_pts > kShortPts) {
        const int ns = std::max(1, (multi ? kMultiWaves : kWaves) / grp);
        t = std::max(t, (n_tile + ns - 1) / ns);
    }
    *tiles = t;
    *n_slice = (n_tile + t - 1) / t;
}

// As few slices as fill the waves, but at least one, and never more than the
// shortest ones: at most the waves' points, the list's, or those times the latter.
size_t sh_sums(int n_pts, int n_reco, bool multi) {
    const size_t n = n_pts, most = (n_reco + kSliceTiles * kShBins - 1) / (kSliceTiles * kShBins);
    const size_t resident = multi ? (size_t)kMultiWaves * 16 : (size_t)kWaves * 64;
    const size_t s = std::min(most * n, std::max(resident, n));
    return multi ? s : std::max(s, most * std::min(n, (size_t)kShortPts));
}

}  // namespace nr
