// Internal declarations of the surrogate's training step for hidden layers of
// kFusedHidden outputs: five launches, each reading operands that are contiguous
// along the reduction (the producers write what the weight gradients need
// transposed as well).
#pragma once
#include "mlp.h"

namespace nr {

// Fragment order of a matrix X[row][k], k its reduction index: blocks of 32 rows x
// 16 k are 1 KB runs, lane (row % 32) + 32 ((k / 8) % 2) of a wave at 16 bytes
// each, so that a matrix operand is one contiguous load.  (From rows a load
// touched 32 bytes of 32 rows, and the rest of those cache lines was gone before
// its turn came.)  Rows are padded to 32, k to 16.
constexpr int kFragRows = 32, kFragK = 16;
inline __host__ __device__ int frag_steps(int K) { return (K + kFragK - 1) / kFragK; }
inline __host__ __device__ size_t frag_at(int row, int k, int steps) {
    return (((size_t)(row >> 5) * steps + (k >> 4)) * 64 + (row & 31) + 32 * ((k >> 3) & 1)) * 8 +
           (k & 7);
}
inline size_t frag_size(int rows, int K) {
    return (size_t)((rows + kFragRows - 1) / kFragRows) * kFragRows * frag_steps(K) * kFragK;
}

// Buffers of one step, all BF16 ones in fragment order; `steps`: 16-point steps of
// those whose reduction runs over the points.
struct TrainBufs {
    bf16* xt;     // [32][points] network input (normalised theta, 1, zeros)
    bf16* ht[3];  // [kFusedHidden + 8][points] activations; row kFusedHidden is 1,
                  // the rows after it 0
    bf16* h2;     // [points][kFusedHidden + 8] last activations (same columns)
    float* z[3];  // [points][kFusedHidden], rows
    bf16* dy;     // [points][N]
    bf16* dyt;    // [N][points]
    bf16* dz2;    // [points][kFusedHidden]
    bf16* dzt[3]; // [kFusedHidden][points]
    int steps;
};

// The weights of one layer, W[m][n] of output m and input n (bias and padding
// included), and their copies in fragment order: by outputs and by inputs.
struct TrainPack {
    const bf16* w;
    bf16 *wf, *wt;  // [M][N], [N][M]
    int M, N;
};

struct TrainFwd {
    const double* theta;  // [..][7]
    const long long* idx; // [B] rows of theta, or null (0 .. B - 1)
    double lo[kNTheta], hi[kNTheta];
    const bf16* wf[3];
    int B;
    TrainBufs b;
};

struct TrainMse {
    const bf16* wf;    // output weights
    const float* t;    // [..][N] targets, rows
    const long long* idx;  // [B] rows of t, or null
    int B, N;
    float scale;
    double* tile_loss; // [ceil(B / 128)][ceil(N / 128)]
    TrainBufs b;
};

// A product whose reduction is summed in n_split chunks of `chunk`, each chunk
// by itself and the chunks in order: the sums of the K-split GEMM.
struct TrainSplit {
    int chunk, n_split;
};

struct TrainDh {
    const bf16* wt;  // output weights by inputs
    int B, N;
    TrainSplit sp;
    TrainBufs b;
};

struct TrainHidden {
    const bf16* wt[2];  // weights of layers 2 and 1 by inputs
    int B;
    TrainSplit sp;
    TrainBufs b;
};

// Weight gradient of one layer, G[m][n] = sum_p A[m][p] B[n][p], and Adam.
struct TrainLayer {
    const bf16* A;   // [M][points]
    const bf16* Bm;  // [N][points]
    int M, N;        // outputs; inputs with the bias column and padding
    TrainSplit sp;
    float *w, *g, *m, *v;  // [M][N]
    bf16* w16;             // [M][N]
    bf16 *wf, *wt;         // fragment order (TrainPack)
    int first;             // first work-group
};
struct TrainW {
    TrainLayer l[4];
    int B, steps;
    float lr, b1, b2, eps, bc1, bc2;
};

hipError_t launch_train_fwd(const TrainFwd& a, hipStream_t s);
hipError_t launch_train_mse(const TrainMse& a, hipStream_t s);
hipError_t launch_train_dh(const TrainDh& a, hipStream_t s);
hipError_t launch_train_hidden(const TrainHidden& a, hipStream_t s);
hipError_t launch_train_w(TrainW a, hipStream_t s);
// rows kFusedHidden .. + 7 of ht: one row of ones, seven of zeros
hipError_t launch_train_ones(bf16* ht, int steps, hipStream_t s);
hipError_t launch_train_pack(const TrainPack& a, hipStream_t s);

}  // namespace nr
