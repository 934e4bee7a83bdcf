// nn.h -- launches of the warm-start network's kernels (k_nn.hip), shared with
// its host orchestration (net.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>

namespace clh {

// Place of a BF16 or FP32 activation tensor's values: voxels in [z][y][x] order
// vs elements apart, 16-channel chunks cs elements apart.
struct NNLayout {
    int vs;
    long cs;
};
inline NNLayout nn_channels_last(int C) { return {C, 16}; }
// [C / 16][voxels][16]
inline NNLayout nn_chunked(size_t voxels) { return {16, (long)voxels * 16}; }

void nn_pack_weights(const float *w, unsigned short *out, int Ci, int Co, int flip, hipStream_t s);
// mask: see k_conv3 (NULL: none)
void nn_conv3(const unsigned short *in, const void *wp, const float *bias, void *out, int out_f32,
              const unsigned short *mask, NNLayout li, NNLayout lo, int D, int H, int W, int Ci, int Co, int act,
              float slope, hipStream_t s);
// 16 -> Co, the input as two channels per voxel (nn_pack_two), the others zero
void nn_conv3_two(const unsigned short *in, const void *wp, const float *bias, unsigned short *out, NNLayout lo, int D,
                  int H, int W, int Co, int act, float slope, hipStream_t s);
size_t nn_packed_weight_elems(int Ci, int Co);
size_t nn_dw_workspace_floats(int D, int H, int W, int Ci, int Co);
void nn_conv3_dw(const unsigned short *X, const unsigned short *dZ, float *partial, float *gw, float *gb, NNLayout lx,
                 NNLayout lz, int D, int H, int W, int Ci, int Co, hipStream_t s);
// 16-channel tensors [D][H][W][16] (chunks stacked along z), D, H, W of the
// finer grid; through the LeakyReLU of Y: the gradient is rounded to BF16, then
// multiplied by 1 or slope by the sign of Y
void nn_pool2(const unsigned short *in, unsigned short *out, int D, int H, int W, hipStream_t s);
void nn_pool2_bwd(const unsigned short *gpool, unsigned short *g, const unsigned short *Y, float slope, int D, int H,
                  int W, hipStream_t s);
void nn_up2(const unsigned short *a, unsigned short *out, int D, int H, int W, hipStream_t s);
void nn_up2_bwd(const unsigned short *g, unsigned short *ga, const unsigned short *Y, float slope, int D, int H, int W,
                hipStream_t s);
void nn_head(const unsigned short *in, const float *w, const float *b, float *out, size_t P, int Ci, hipStream_t s);
void nn_head_bwd(const unsigned short *in, const float *gout, const float *w, float slope, unsigned short *gin,
                 double *partials, int nparts, double *dst_dev, size_t P, hipStream_t s);
void nn_mse(const float *pred, const float *label, size_t n, float inv, float *grad, double *partials, int nparts,
            hipStream_t s);
void nn_adam(float *p, const float *g, float *m, float *v, size_t n, float lr, float b1, float b2, float eps, float c1,
             float c2, hipStream_t s);
void nn_pack_input(const float *a, const float *b, unsigned short *out, size_t P, hipStream_t s);
void nn_pack_two(const float *a, const float *b, unsigned short *out, size_t P, hipStream_t s);

} // namespace clh
