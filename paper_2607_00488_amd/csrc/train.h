// Internal declarations of the surrogate's training step for hidden layers of
// kFusedHidden outputs: five launches, each reading operands that are contiguous
// along the reduction (the producers write what the weight gradients need
// transposed as well).
#pragma once
#include "mlp.h"

namespace nr {

// Buffers of one step.  Transposed ones have rows of `ldt` >= B values.
struct TrainBufs {
    bf16* xt;     // [32][ldt] network input (normalised theta, 1, zeros)
    bf16* ht[3];  // [kFusedHidden + 8][ldt] activations; row kFusedHidden is 1,
                  // the rows after it 0
    bf16* h2;     // [B][kFusedHidden + 8] last activations (with the same columns)
    float* z[3];  // [B][kFusedHidden]
    bf16* dy;     // [B][N]
    bf16* dyt;    // [N][ldt]
    bf16* dz2;    // [B][kFusedHidden]
    bf16* dzt[3]; // [kFusedHidden][ldt]
    int ldt;
};

struct TrainFwd {
    const double* theta;  // [B][7]
    double lo[kNTheta], hi[kNTheta];
    const bf16* w[3];     // [kFusedHidden][k_l]
    int k[3];
    int B;
    TrainBufs b;
};

struct TrainMse {
    const bf16* w;     // [N][kFusedHidden + 8]
    const float* t;    // [B][N] targets
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
    const bf16* wt;  // [kFusedHidden + 8][N] output weights, transposed
    int B, N;
    TrainSplit sp;
    TrainBufs b;
};

struct TrainHidden {
    const bf16* wt[2];  // transposed weights of layers 2 and 1, [k][kFusedHidden]
    int B;
    TrainSplit sp;
    TrainBufs b;
};

// Weight gradient of one layer, G[m][n] = sum_p A[m][p] B[n][p], and Adam.
struct TrainLayer {
    const bf16* A;   // [M][ldt]
    const bf16* Bm;  // [N][ldt]
    int M, N;        // outputs; inputs with the bias column and padding
    TrainSplit sp;
    float *w, *g, *m, *v;  // [M][N]
    bf16 *w16, *w16t;      // [M][N]; [N][M] or null
    int first;             // first work-group
};
struct TrainW {
    TrainLayer l[4];
    int B, ldt;
    float lr, b1, b2, eps, bc1, bc2;
};

hipError_t launch_train_fwd(const TrainFwd& a, hipStream_t s);
hipError_t launch_train_mse(const TrainMse& a, hipStream_t s);
hipError_t launch_train_dh(const TrainDh& a, hipStream_t s);
hipError_t launch_train_hidden(const TrainHidden& a, hipStream_t s);
hipError_t launch_train_w(TrainW a, hipStream_t s);
// rows [row0, row0 + 8) of a transposed buffer: one row of ones, seven of zeros
hipError_t launch_train_ones(bf16* ht, int row0, int ldt, hipStream_t s);

}  // namespace nr
