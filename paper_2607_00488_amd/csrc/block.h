// Internal declarations of the blocked fold: many parameter points of a
// multi-component context share one stream over the response.
#pragma once
#include "common.h"

namespace nr {

constexpr int kBlkPts = 16;    // points of one matrix-instruction block
constexpr int kBlkCols = 256;  // response columns per fold work-group
constexpr int kBlkFinCols = 32;  // columns per likelihood work-group

// Weights of a list of points from the row factors (basis.h):
// wt[r][p] = v_r(theta_p) for p < n_pts, 0 for n_pts <= p < n_pad.
struct PtsWeightArgs {
    const double* rf;     // [n_comp n_t][kRFComp]
    int n_t, n_comp;
    const double* theta;  // [n_pts][n_theta]
    int n_theta, rate_index;  // theta index of component 0's rate
    int n_pts, n_pad, ldw;
    Phys ph;
    double* wt;           // [n_comp n_t][ldw]
};

// part[s][p][j] = sum over the rows l of split s of wt[l][p] R[l][j]:
// n_split splits of rows_per rows, points padded to 16, columns to ldr.
struct BlkFoldArgs {
    const double* wt;
    int ldw;
    const float* R;
    int ldr, n_rows, n_pts;
    int n_ct, n_split, rows_per;
    double* part;
    size_t split_stride;  // doubles between splits
    // per column tile the rows [lo, hi) that hold its non-zero responses (lo a
    // multiple of four), or null (every row)
    const int* band;
};

// mu_j and deviance of every point from the splits, then -2lnL.
struct BlkFinishArgs {
    const double* part;
    size_t split_stride;
    int n_split, ldr, n_reco, n_pts, n_ct;
    const double* theta;  // [n_pts][n_theta]
    int n_theta, bkg_index, n_bkg;
    const double* n;
    const double* b;      // [n_bkg][n_reco]
    const double* mask;   // [n_reco] or null
    double* dev;          // [n_pts][n_ct] deviance sums
    double* out_mu;       // [n_pts][n_reco] or null
    double cdata;
    double pull_mean[kMaxTheta];
    double pull_sigma[kMaxTheta];
    double* nll;          // [n_pts]
};

int blk_fold_lds_rows();
hipError_t launch_pts_weights(const PtsWeightArgs& a, hipStream_t s);
hipError_t launch_blk_fold(const BlkFoldArgs& a, hipStream_t s);
hipError_t launch_blk_finish(const BlkFinishArgs& a, hipStream_t s);

}  // namespace nr
