// One-launch kernels for small layers and batches (lmkan_gather.hip).
#pragma once

#include "lmkan_slab_common.h"

namespace lmkan {

struct GatherArgs {
    const void *P;
    const float *x;
    const float *gy;
    float *out;       // y or grad_x
    float *gcoef;
    CoefMap map;      // of P
    GridTab tab;
    ConvGeom cg;
    int64_t B;
    int n_in;
    int n_out;
    int K;
    int W;
    int col_limit;    // columns >= col_limit do not exist in the coefficient tensor
    int conv;         // x (and grad_x) is an image, rows are its windows
    int n_ct;         // forward: column tiles
    int log_per_row;  // items of a row that a wave locates at once
    int log_spw, log_wpr;  // forward: slots of a wave and waves that share a row
    int64_t groups;   // forward: row groups
    int items, k_chunks;  // input gradient: items of a wave, waves along the pairs
    int overlap;      // input gradient: windows overlap
    int coef_ct, coef_blocks;  // coefficient gradient: column tiles; workgroups, where both gradients share a launch
    int parts, spn;   // coefficient gradient: workgroups that share a (pair, tile)'s nodes; lane groups that share a node's samples
    int accumulate;
};

bool forward_gather_shape_ok(const LayerShape &s);
// of a shape that head_forward_shape_ok(), on rows
bool forward_gather_beats_head(const LayerShape &s);
bool backward_input_gather_shape_ok(const LayerShape &s);
bool backward_coef_gather_shape_ok(const LayerShape &s);
// both gradients from one launch
bool backward_gather_shape_ok(const LayerShape &s);
// the forward pass and the input gradient read the table 16 bytes at a time
bool gather_table_aligned(const void *coef);
// x: rows, 8-byte aligned, or (conv) an image; the same for grad_x
void launch_forward_gather(const LayerShape &s, const GridTab &tab, const float *x, const void *coef, float *y,
                           hipStream_t stream, const ConvGeom *conv);
void launch_backward_input_gather(const LayerShape &s, const GridTab &tab, const float *x, const void *coef,
                                  const float *gy, float *gx, hipStream_t stream, const ConvGeom *conv);
void launch_backward_gather(const LayerShape &s, const GridTab &tab, const float *x, const void *coef, const float *gy,
                            float *gx, float *gcoef, bool accumulate, hipStream_t stream, const ConvGeom *conv);
void launch_backward_coef_gather(const LayerShape &s, const GridTab &tab, const float *x, const float *gy, float *gcoef,
                                 bool accumulate, hipStream_t stream, const ConvGeom *conv);

}  // namespace lmkan
