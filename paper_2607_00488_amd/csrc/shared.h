// Internal declarations of the basis form of the evaluation.
//
// A point's row factors are v_l = sum_b c_b(theta) F_lb (basis.h), so the fold
// of any number of points is a product of three matrices,
//   mu = C (F^T R) + f_bkg b,   C [points][15], F [rows][15], R [rows][bins],
// and taking F^T R first costs one pass over R per call, whatever the number of
// points: 15 multiply-adds per response entry instead of one (two with the
// gradient) per entry and point.  The gradient needs nothing more of R:
//   d(-2lnL)/d theta_i = sum_b dc_b/d theta_i h_b, h_b = sum_j a_j (F^T R)_bj.
// Launches: fold; records (split sums and data, one record per bin) and points
// (mu, deviance, h), together for short lists; final.
#pragma once
#include "basis.h"

namespace nr {

constexpr int kShCols = kNBasis + 1;  // folded columns: 14 spectra, constant rows
constexpr int kShTile = 256;          // response columns per fold work-group
constexpr int kShSmallTile = 64;      // of the two other kinds
constexpr int kShStage = 32;          // rows per stage of the fold
// Work-groups of the fold: four waves side by side over 256 columns, the same with
// narrow waves over 64, four waves over the same 64 columns and a quarter of the
// split's rows each.
enum ShKind { kShWide, kShNarrow, kShTall };
constexpr int kShRec = 18;            // record: 15 columns, b_j, n_j, 1 / n_j
constexpr int kShBins = 16;           // bins per tile of the points kernel
constexpr int kShAcc = 16;            // contractions h per point (the last: b_j)
constexpr int kShGroup = 16;          // analyses per grouped launch

struct ShFold {
    const float* R;    // [n_t][ldr]
    const double* rf;  // [n_t][kRF]
    double* part;      // [n_split][kShCols][ldr]
    // per column tile the rows [lo, hi) that hold its non-zero responses (lo a
    // multiple of four), or null (every row)
    const int* band;
    // points to copy to device memory beside the fold, or null
    const double* th_src;
    double* th_dst;
    int n_th;  // values
    int ldr, n_t, n_ct, n_split, rows_per;
    ShKind kind;
    bool stream;  // read R past the caches (kinds of 64 columns per wave)
};

struct ShRec {
    const double* part;
    const double* n;  // [n_reco]
    const double* b;  // [n_reco]
    double* rec;      // [n_reco rounded up to kShBins][kShRec]
    int n_split, ldr, n_reco;
};

// The multi-component likelihood is the same product with a record of 8 columns
// per component (seven spectra and the constant rows, coefficients r_k c_b and
// r_k) and one per background (coefficient r_q), all times the common mask M_j:
//   mu_j = M_j [sum_k r_k (G0^(k)_j + sum_b c_b G^(k)_bj) + sum_q r_q B_qj].
// Its columns are padded with zeros to a multiple of four: three size classes, the
// smallest for one component, the next for five and four backgrounds (the solar
// species).
constexpr int kShMaxComp = 8;
constexpr int kShMaxBkg = 8;
constexpr int kShCompCols = kCompBasis + 1;
constexpr int kShTiny = 12, kShSmall = 44, kShLarge = 72;  // columns of the classes

struct ShEval {
    const double* rec;
    const double* theta;  // [n_pts][n_theta]
    double* dpart;        // [n_slice][n_pts] deviance sums
    double* hpart;        // [n_slice][n_acc][n_pts], or null (no gradient)
    double* mu;           // [n_pts][n_reco], or null
    Phys ph;
    int n_pts, n_reco, tiles, n_slice;  // tiles of kShBins bins per slice
    // multi-component form: components, backgrounds (K = 0: single-component)
    int K, B, n_theta;
};

// Columns of a record and contractions of the gradient (whole blocks of 16).
inline int sh_cols(int K, int B) {
    const int n = kShCompCols * K + B;
    return K == 0 ? kShAcc : n <= kShTiny ? kShTiny : n <= kShSmall ? kShSmall : kShLarge;
}
inline int sh_acc(int K, int B) { return (sh_cols(K, B) + 15) / 16 * 16; }

// Records and points of a short list in one launch; slices of kShTailBins bins,
// their points dealt to ny work-groups each.
constexpr int kShTailBins = 64;
struct ShTail {
    ShRec r;
    ShEval e;
    int ny;
};

struct ShFinal {
    const double* dpart;
    const double* hpart;
    const double* theta;
    double* nll;
    double* grad;  // [n_pts][7] or null
    double cdata;
    double pull_mean[kNTheta];
    double pull_sigma[kNTheta];
    Phys ph;
    int n_pts, n_slice;
};

// Multi-component likelihood and gradient.
struct ShMultiFinal {
    const double* dpart;
    const double* hpart;
    const double* theta;
    double* nll;
    double* grad;  // [n_pts][n_theta] or null
    double cdata;
    double pull_mean[kMaxTheta];
    double pull_sigma[kMaxTheta];
    Phys ph;
    int n_pts, n_slice, K, B, n_theta;
};

// Columns of one component folded (slabs of rows, see launch_sh_mfold) and the
// data of a multi-component record.
struct ShMultiFold {
    const float* R;    // this component's rows
    const double* rf;  // [n_t][kRFComp]
    double* part;      // [n_slab][kRFComp][n_reco]
    int ldr, n_t, n_reco;
};
struct ShMultiRec {
    const double* part;
    const double* mask;  // [n_reco] or null
    double* rec;         // [..][cols + 2]
    int n_slab, n_reco, comp, cols;
};
struct ShMultiData {
    const double* n;
    const double* bkg;   // [B][n_reco]
    const double* mask;  // [n_reco] or null
    double* rec;
    int n_reco, K, B, cols;
};

// N analyses of one launch, by value: first[d] is the first work-group of d.
template <class P, int N>
struct ShGroup {
    int n;
    int first[N + 1];
    P p[N];
};

// Each takes n <= kShGroup analyses (all with or all without gradient / mu).
hipError_t launch_sh_fold(const ShFold* p, int n, hipStream_t s);
hipError_t launch_sh_rec(const ShRec* p, int n, hipStream_t s);
hipError_t launch_sh_eval(const ShEval* p, int n, hipStream_t s);
hipError_t launch_sh_tail(const ShTail* p, int n, hipStream_t s);
hipError_t launch_sh_final(const ShFinal* p, int n, hipStream_t s);
hipError_t launch_sh_mfinal(const ShMultiFinal& p, hipStream_t s);
constexpr int kShSlabRows = 64;  // response rows per multi-component fold work-group
hipError_t launch_sh_mfold(const ShMultiFold& p, hipStream_t s);
hipError_t launch_sh_mrec(const ShMultiRec& p, hipStream_t s);
hipError_t launch_sh_mdata(const ShMultiData& p, hipStream_t s);
// New data beside folded columns that stay.
hipError_t launch_sh_data(const ShRec& p, hipStream_t s);

// Column tiles of the fold.
inline int sh_tiles(int ldr, ShKind kind) {
    const int cols = kind == kShWide ? kShTile : kShSmallTile;
    return (ldr + cols - 1) / cols;
}
// Column slices of an evaluation of n_pts points over n_reco bins.
void sh_slices(int n_pts, int n_reco, bool multi, int* tiles, int* n_slice);
// Slices x points of any list of up to n_pts points (fewer points may take more
// slices), at least.
size_t sh_sums(int n_pts, int n_reco, bool multi);

}  // namespace nr
