// hexsv_nn.h — launchers of the surrogate's kernels (hexsv_nn.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hexsv {
namespace nn {

enum { EPI_RELU = 0, EPI_LIN = 1 };
constexpr int OUT_STRIDE = 4;  // floats per cell of the network output (3 used)
constexpr int FEATURES = 11;     // network input channels
constexpr int FEATURES_PAD = 16; // stored input channels per cell (bf16, zero padded)

// Which raster positions a tap may reach, as in the neighbour table of the
// scheme: periodic sides wrap (perq: q, perr: r), positions outside the raster
// are zero, and with an active mask (per raster cell, nonzero = in the domain;
// nullable: every cell) a tap t >= 1 reads its neighbour only when both the cell
// and the neighbour are in the domain (tap 0, the cell itself, is always read).
// The rule is symmetric, so the transposed stencil of the data gradient uses it
// unchanged.
struct ConvMask {
    const uint8_t *active;
    int perq, perr;
};

// Workgroups (tiles of 64 x 4 cells) of one conv launch over a batch.
int conv_tiles(int nq, int nr, int batch);

// Hex convolution of channels-last bf16 x (cinp channels) with the MFMA
// weight layout wm[t][coutp][cinp]; epilogue per EPI_* (see hexsv_nn.hip).
// Built for (cinp, coutp, epi) in {(16,32,RELU), (32,32,RELU), (32,16,LIN)}.
// live (nullable, device): the launch does nothing unless *live != 0.
hipError_t launch_conv(int cinp, int coutp, int epi, const __bf16 *x, const __bf16 *wm,
                       const float *bias, void *out, int nq, int nr, int batch, int cout_real,
                       const ConvMask &cm, hipStream_t st, const int32_t *live = nullptr);
// The 4-layer network with 32 hidden channels in one launch, a sweep (k_hexnet4): weights
// and biases of each layer as for launch_conv (layer 0: 16 -> 32, layers 1-2:
// 32 -> 32, layer 3: 32 -> 16 with 3 outputs written, FP32, OUT_STRIDE per cell;
// w4: and a zero); x: the FP32 features (f32in) or the packed bf16 input; keep
// (with f32in, no mask): also what the gradient reads.  All equal the layer-by-layer
// launch_conv chain's bit for bit.
struct Net4 {
    const __bf16 *wm[4];
    const float *bias[4];
};
// What the gradient reads of a forward: the packed input and the hidden activations.
struct Net4Keep {
    __bf16 *x0, *act[3];
};
hipError_t launch_net4(const void *x, bool f32in, const Net4 &nw, float *out, bool w4, int nq,
                       int nr, int batch, const ConvMask &cm, hipStream_t st,
                       const int32_t *live = nullptr, const Net4Keep *keep = nullptr);
// The same network by 16 x 16 tiles (k_hexnet4_tile) from the packed input; three floats a cell.
hipError_t launch_net4_tiles(const __bf16 *x, const Net4 &nw, float *out, int nq, int nr, int batch,
                             const ConvMask &cm, hipStream_t st, const int32_t *live = nullptr);
// Which way is the fastest for these samples (of a forward call, a gradient's forward, a surrogate
// window)?  chain_too: the layers may also run one by one.
enum Net4Use { NET4_FORWARD, NET4_KEEP, NET4_WINDOW };
enum Net4Route { NET4_CHAIN, NET4_SWEEP, NET4_TILES };
Net4Route net4_route(int nq, int nr, int batch, bool masked, Net4Use use, bool chain_too);
// Weight-gradient partials: one record (7*coutp*cinp + coutp floats) per workgroup of
// the launch, which sweeps the tiles with its sums in registers.  WGRAD_WGS workgroups
// are two per CU, all resident: more would only add records to reduce (half as many with the
// data gradient, whose workgroups fill a CU).  Layers with 32
// input channels (not the first): the data gradient dx through x's ReLU as well, with the
// transposed stencil's weights wt[t][cinp][coutp].
constexpr int WGRAD_WGS = 512;
int wgrad_records(int nq, int nr, int batch, bool dx);
hipError_t launch_wgrad(int cinp, int coutp, const __bf16 *x, const __bf16 *dy, float *part,
                        const __bf16 *wt, __bf16 *dx, int nq, int nr, int batch,
                        const ConvMask &cm, hipStream_t st);
// All layers' records into the flat gradient; block0 is set by the launcher.
constexpr int MAX_LAYERS = 16;
struct WgradLayer {
    const float *part;
    int64_t off;  // of the layer's W in the flat parameters
    int cinp, coutp, cin, cout, nrec, block0;
};
struct WgradTable {
    int layers;
    WgradLayer y[MAX_LAYERS];
};
hipError_t launch_wgrad_reduce(WgradTable tab, float *grad, hipStream_t st);
hipError_t launch_prepare_weights(const float *p, int cin, int cout, int cinp, int coutp,
                                  __bf16 *wm, __bf16 *wt, float *bias, hipStream_t st);
hipError_t launch_adam(float *p, float *m, float *v, const float *g, int64_t n, float lr,
                       int step, hipStream_t st);
hipError_t launch_l1_loss(const float *pred, const float *target, int64_t ncell, double inv_count,
                          __bf16 *dy, double *part, int nparts, hipStream_t st);
hipError_t launch_pack_features(const float *f, int64_t ncell, __bf16 *x, hipStream_t st);

}  // namespace nn
}  // namespace hexsv
