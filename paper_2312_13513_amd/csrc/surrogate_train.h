// Training kernels of one network with widths up to kTrainMaxWidth
// (surrogate_train.hip).  Layer l: out_l[l] x in_l[l] weights at off_W[l] of the
// padded parameter vector, biases at off_b[l].
#pragma once

#include "surrogate.h"

namespace chem {

constexpr int kTrainMaxWidth = 512;

bool train_fused_supported(const int in_l[4], const int out_l[4]);

// Forward pass, loss and errors of `rows` rows (order[start + i], or start + i).
struct TrainArgs {
    const bf16_t *X;            // rows of 64
    const int32_t *order;       // NULL: rows in place
    int64_t start, rows;
    const float *Y;             // targets, rows of ldy
    int64_t ldy;
    int K;
    float scale;                // 2 / (rows K)
    const bf16_t *W[4];         // weights in fragment order
    const bf16_t *WT[3];        // WT[l]: transpose of layer l + 1 in fragment order, its columns padded to 64
    const float *b[4];
    int in_l[4], out_l[4];
    // out: [unit][row] matrices of ldT columns in fragment order, ldT a multiple
    // of 32 and at least rows rounded up to 32 (errors of the padding rows are 0)
    bf16_t *Xt, *Ht[3], *Dt[4];
    int64_t ldT;
    double *loss_part;          // squared errors per block of 16 rows
};
hipError_t launch_train_rows(const TrainArgs &a, hipStream_t s);

// Weight and bias gradients from those copies into g (padded parameter vector).
struct GradArgs {
    const bf16_t *Xt, *Ht[3], *Dt[4];
    int64_t ldT, rows;
    int in_l[4], out_l[4];
    int tiles[4], all_tiles;    // 32 x 32 tiles of each layer and their sum
    int64_t off_W[4], off_b[4];
    float *g;
};
hipError_t launch_train_grad(const GradArgs &a, hipStream_t s);

// With `weights` the BF16 copies of the parameters o.p, after an Adam step if
// `adam`; *loss += the sum of loss_part (unless NULL).  Layers of any width, in_l
// multiples of 64 and out_l of 16.
// wbf: row by row; wfrag: each layer's [out_l][in_l] matrix in fragment order, the
// 16 x 32 operand of rows 16 jb .. and columns 32 ks .. as 512 values at
// (jb in_l / 32 + ks) 512, lane by lane, 8 each; wfragT (unless NULL): the transposes
// of layers 2..4 in that order, at off_T, their columns padded to 64.
struct UpdateArgs {
    int64_t n_pad;
    int weights, adam;
    AdamArgs o;
    bf16_t *wbf, *wfrag, *wfragT;
    int in_l[4], out_l[4];
    int64_t off_W[4], off_T[4];
    const double *loss_part;
    int loss_blocks;
    double *loss;
};
hipError_t launch_train_update(const UpdateArgs &a, hipStream_t s);

}  // namespace chem
