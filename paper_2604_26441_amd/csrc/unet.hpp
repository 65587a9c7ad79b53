// Launchers of the U-Net kernels (kernels_unet.hip).
#pragma once
#include "common.hpp"

struct sgmg_hierarchy;

namespace sgmg {

// A batch of samples on one mesh for the energy-norm training score.
struct EnergyBatch {
  Grid g;                  // fine node grid (all samples)
  const uint8_t* fixn;     // clamp bits per node
  const double* ke;        // K_e of the unit-modulus cube (576)
  const double* E;         // N x nel element moduli
  const double* f;         // N x ndof loads
  const double* cstar;     // N compliances f.u*
  double* u;               // N x ndof: network output as DOF vectors
  double* Ku;              // N x ndof
  double* part;            // N x nb x 2 block partials
  double* scal;            // N x 4: score, gradient factor, a / b, 0
  int N, nb;               // samples, node blocks of 256 per sample
  int Dp, Hp, Wp;          // padded voxel grid of the network
};
void launch_energy_loss(const EnergyBatch& e, const float* y, float* gy, hipStream_t s);

// Fine-level view of a hierarchy (runtime.hip) for the network's training.
struct FineView {
  Grid g;
  const uint8_t* fixn;
  const double* ke;
  int is_modulus;
  double E0, Emin, penal;
};
int hierarchy_fine_view(const ::sgmg_hierarchy* h, FineView* v);

// Every layer's parameters (or gradients) on the device; off: first index of
// each layer in the flat order of the C ABI, then the total.
struct ParamTable {
  static constexpr int kLayers = 8;
  const float* w[kLayers];
  const float* b[kLayers];
  int ci[kLayers], co[kLayers], k3[kLayers], cop[kLayers], off[kLayers + 1];
};
void launch_export_params(const ParamTable& t, float* out, hipStream_t s);

void launch_conv_fwd(int K, const float* x, int N, int Ci, int Co, int D, int H, int W,
                     const float* w, const float* b, int relu, float* rpre, const float* add,
                     float* y, hipStream_t s);
// Packed 3x3x3 weights (uint4 words) of a layer that reads its input as stored
// (up = 0) or upsampled (up = 1).
size_t conv3_packed_words(int up, int Ci, int Co);
void launch_pack_conv3(const float* w, int up, int Ci, int Co, uint4* wp, hipStream_t s);
// Packed weights of the data gradients of up to eight 3x3x3 layers: w, the
// layer's channels and wp (conv3_packed_words(0, Co, Ci)) are given.
struct ConvPacks {
  struct One {
    const float* w;
    uint4* wp;
    int Ci, Co, Cip, Cop, total;
  } p[8];
  int n;
};
void launch_pack_conv3_flip(ConvPacks ps, hipStream_t s);
// up = 1: x is stored at (D/2, H/2, W/2) and read as its nearest x2 upsampling
// (Ci a multiple of 8); with hw (up = 1, Co = 16) the 1x1x1 head's three
// channels hw, hb of the result are written to hy, and y may be NULL.
void launch_conv3_mfma(const float* x, int up, int N, int Ci, int Co, int D, int H, int W,
                       const uint4* wp, const float* b, int relu, const float* add, float* y,
                       hipStream_t s, const float* hw = nullptr, const float* hb = nullptr,
                       float* hy = nullptr);
// The training pass's forward: one order of every sum, also with up = 1 (wp
// packed with up 0).
void launch_conv3_train(const float* x, int up, int N, int Ci, int Co, int D, int H, int W,
                        const uint4* wp, const float* b, int relu, float* rpre, const float* add,
                        float* y, hipStream_t s);
void launch_weight_transpose(const float* w, int Ci, int Co, int K, float* wt, hipStream_t s);
size_t conv_wgrad_part_floats(int N, int Ci, int Co, int D, int H, int W, int K);
void launch_conv_wgrad(int K, const float* x, int up, const float* dy, int N, int Ci, int Co, int D,
                       int H, int W, float* part, float* dw, float* db, hipStream_t s);
void launch_pool(const float* x, int NC, int D, int H, int W, float* y, hipStream_t s);
// y = scale * x upsampled + extra where r > 0 (the adjoints of the pooling, the
// skip and the ReLU), and the eightfold sums of x (into y, unless NULL) where r
// > 0 (those of the upsampling and the ReLU, into dr).
void launch_expand_relu(const float* x, int NC, int D, int H, int W, float scale, const float* r,
                        const float* extra, float* y, hipStream_t s);
void launch_sum8_relu(const float* x, int NC, int D, int H, int W, const float* r, float* y, float* dr,
                      hipStream_t s);
void launch_relu_bwd(const float* dy, const float* r, long n, float* dr, hipStream_t s);
void launch_add(const float* a, const float* b, long n, float* y, hipStream_t s);
void launch_mse(const float* y, const float* t, const float* mask, int N, int C, int DHW, float* dy,
                RedWs ws, double* sums, hipStream_t s);
void launch_adam(float* p, float* pq, const float* g, float* m, float* v, long n, float lr, float b1,
                 float b2, float eps, int step, int quantize, hipStream_t s);
void launch_round_bf16(const float* p, float* q, long n, hipStream_t s);
void launch_unet_input(const Grid& g, const double* rho, const double* f, const uint8_t* fixn,
                       double* fmax_scratch, int Dp, int Hp, int Wp, float* in, hipStream_t s);
void launch_unet_output(const Grid& g, const float* out, const uint8_t* fixn, int Dp, int Hp,
                        int Wp, double* u, hipStream_t s);
void launch_unet_target(const Grid& g, const double* u, double* umax_scratch, int Dp, int Hp, int Wp,
                        float* t, float* m, hipStream_t s);
void launch_scale_by_ratio(double* u, int n, const double* num, const double* den, double* alpha,
                           hipStream_t s);

}  // namespace sgmg
