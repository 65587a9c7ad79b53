// Training and inference kernels of the warm-start 3D U-Net (extension, not
// a passage of the paper).  Tensors are (N, C, D, H, W) in FP32; weights are
// held in BF16 precision (values rounded to BF16, stored as FP32 so the
// arithmetic is FP32 accumulation of BF16-exact weights) in the layout
// w[(ci * K^3 + tap) * Cop + co], Cop = output channels padded to 16, so the
// 16 weights of one (ci, tap) are contiguous and read with uniform loads.
#include "kernels.hpp"
#include "node_ops.hpp"
#include "unet.hpp"

namespace sgmg {

constexpr int kCOB = 16;   // output channels per thread
// Blocks of a convolution below which channel tiles are split over more blocks.
constexpr long kConvBlocks = 1024;

// y[n, co] = epi(b[co] + sum_{ci, tap} w * x[n, ci, v + tap - r]) for co in a
// block of 16; epi: optional ReLU, optional stored pre-add value r, optional
// skip add.  Zero padding outside the volume.
template <int K>
__global__ __launch_bounds__(256) void k_conv_fwd(const float* __restrict__ x, int Ci, int Co,
                                                  int Cop, int D, int H, int W,
                                                  const float* __restrict__ w,
                                                  const float* __restrict__ bias, int relu,
                                                  float* __restrict__ rpre,
                                                  const float* __restrict__ add,
                                                  float* __restrict__ y) {
  constexpr int R = K / 2;
  constexpr int K3 = K * K * K;
  const int HW = H * W, DHW = D * HW;
  const int v = blockIdx.x * 256 + threadIdx.x;
  const int co0 = blockIdx.y * kCOB;
  const int n = blockIdx.z;
  if (v >= DHW) return;
  const int d = v / HW, hh = (v / W) % H, ww = v % W;
  float acc[kCOB];
#pragma unroll
  for (int c = 0; c < kCOB; ++c) acc[c] = 0.f;
  const float* xn = x + (size_t)n * Ci * DHW;
  for (int ci = 0; ci < Ci; ++ci) {
    const float* xc = xn + (size_t)ci * DHW;
    const float* wc = w + (size_t)ci * K3 * Cop + co0;
#pragma unroll
    for (int t = 0; t < K3; ++t) {
      const int dz = t / (K * K) - R, dy = (t / K) % K - R, dx = t % K - R;
      const int zz = d + dz, yy = hh + dy, xx = ww + dx;
      const bool ok = (unsigned)zz < (unsigned)D && (unsigned)yy < (unsigned)H &&
                      (unsigned)xx < (unsigned)W;
      const float xv = ok ? xc[(size_t)zz * HW + yy * W + xx] : 0.f;
      const float* wt = wc + (size_t)t * Cop;
#pragma unroll
      for (int c = 0; c < kCOB; ++c) acc[c] += wt[c] * xv;
    }
  }
#pragma unroll
  for (int c = 0; c < kCOB; ++c) {
    const int co = co0 + c;
    if (co >= Co) break;
    float val = acc[c] + (bias ? bias[co] : 0.f);
    if (relu) val = fmaxf(val, 0.f);
    const size_t o = ((size_t)n * Co + co) * DHW + v;
    if (rpre) rpre[o] = val;
    if (add) val += add[o];
    y[o] = val;
  }
}

void launch_conv_fwd(int K, const float* x, int N, int Ci, int Co, int D, int H, int W,
                     const float* w, const float* b, int relu, float* rpre, const float* add,
                     float* y, hipStream_t s) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB;
  dim3 grid(div_up((long)D * H * W, 256), Cop / kCOB, N);
  if (K == 3)
    k_conv_fwd<3><<<grid, 256, 0, s>>>(x, Ci, Co, Cop, D, H, W, w, b, relu, rpre, add, y);
  else
    k_conv_fwd<1><<<grid, 256, 0, s>>>(x, Ci, Co, Cop, D, H, W, w, b, relu, rpre, add, y);
}

// ---------------------------------------------------------------------------
// 3x3x3 convolutions as implicit GEMMs on the matrix cores
// (v_mfma_f32_16x16x32_bf16, FP32 accumulation).  Per MFMA the A operand is
// 16 output channels x 32 reduction slots and the B operand 32 reduction
// slots x 16 output voxels (one x-run of a tile row); a lane holds 8 slots,
// the same 8 input channels at one tap.  The activations are FP32: each value
// is split exactly into three BF16 terms (truncation: hi, then the
// remainder's hi, then what is left, 8 + 8 + 8 significand bits), and the
// three products with the BF16 weight are exact in FP32, so the result is an
// FP32 sum of the exact products (the accuracy of the FP32 vector-ALU form).
//
// Block: an output tile of 16 (x) x 4 (y) x 4 (z) voxels of one sample and
// COT tiles of 16 output channels; wave w owns the 4 tile rows of z = w.
// The input the tile reads is staged in LDS as the three term planes, 8
// channels (16 B) per voxel, so one ds_read_b128 is a lane's B operand; zero
// outside the volume (the padding).  The next stage's values are loaded while
// this one is multiplied.
constexpr int kCTX = 16, kCTY = 4, kCTZ = 4;
constexpr int kCHX = kCTX + 2, kCHY = kCTY + 2, kCHZ = kCTZ + 2;
constexpr int kCHV = kCHX * kCHY * kCHZ;       // 648 halo voxels
constexpr int kCSteps = 7;                     // k-steps of 4 taps

typedef __bf16 cbf16x8 __attribute__((ext_vector_type(8)));
typedef float cf32x4 __attribute__((ext_vector_type(4)));

// exact three-term BF16 split of v; returns the terms' bit patterns
__device__ inline void split3(float v, unsigned& t0, unsigned& t1, unsigned& t2) {
  const unsigned b = __float_as_uint(v);
  const unsigned h = b & 0xffff0000u;
  const float r1 = v - __uint_as_float(h);
  const unsigned m = __float_as_uint(r1) & 0xffff0000u;
  const float r2 = r1 - __uint_as_float(m);
  t0 = h >> 16;
  t1 = m >> 16;
  t2 = __float_as_uint(r2) >> 16;
}

// Eight channels of a voxel, split, into entry e of the three planes.
__device__ inline void stage_split(const float (&v)[8], uint4* p0, uint4* p1, uint4* p2, int e) {
  unsigned t0[4], t1[4], t2[4];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    unsigned a0, a1, a2, b0, b1, b2;
    split3(v[j], a0, a1, a2);
    split3(v[j + 1], b0, b1, b2);
    t0[j >> 1] = a0 | (b0 << 16);
    t1[j >> 1] = a1 | (b1 << 16);
    t2[j >> 1] = a2 | (b2 << 16);
  }
  p0[e] = uint4{t0[0], t0[1], t0[2], t0[3]};
  p1[e] = uint4{t1[0], t1[1], t1[2], t1[3]};
  p2[e] = uint4{t2[0], t2[1], t2[2], t2[3]};
}

// A row's sums of the first terms and of the smaller two: kept apart until the
// end, so that a sum of full size is rounded once per step and not three
// times (output error against FP64 5.4e-7 -> 2.8e-7 on the 104^3 grid), and two
// chains of products run side by side.
template <int COT>
struct ConvAcc {
  cf32x4 hi[COT], lo[COT];
};

template <int COT>
__device__ inline void conv_zero(ConvAcc<COT> (&acc)[kCTY]) {
#pragma unroll
  for (int r = 0; r < kCTY; ++r)
#pragma unroll
    for (int c = 0; c < COT; ++c) acc[r].hi[c] = acc[r].lo[c] = cf32x4{0.f, 0.f, 0.f, 0.f};
}

// SEQ: all three terms into one sum, smallest first (lo stays zero).
template <int COT, bool SEQ = false>
__device__ inline void mfma3(const uint4 (&a)[COT], const cbf16x8 b0, const cbf16x8 b1,
                             const cbf16x8 b2, ConvAcc<COT>& acc) {
#pragma unroll
  for (int c = 0; c < COT; ++c) {
    const cbf16x8 av = __builtin_bit_cast(cbf16x8, a[c]);
    if constexpr (SEQ) {
      acc.hi[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b2, acc.hi[c], 0, 0, 0);
      acc.hi[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b1, acc.hi[c], 0, 0, 0);
      acc.hi[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b0, acc.hi[c], 0, 0, 0);
      continue;
    }
    acc.lo[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b2, acc.lo[c], 0, 0, 0);
    acc.hi[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b0, acc.hi[c], 0, 0, 0);
    acc.lo[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b1, acc.lo[c], 0, 0, 0);
  }
}

// Where a convolution's result goes: y = relu?(acc + bias) (kept in rpre) plus
// add; with hw, the three channels of the 1x1x1 head on that (16 channels,
// hw[ci * 16 + co], hb) go to hy, and y may be NULL.
struct ConvOut {
  const float* bias;
  int relu;
  float* rpre;
  const float* add;
  float* y;
  const float* hw;
  const float* hb;
  float* hy;
};

// Epilogue: lane holds output channels 16 c + 4 q + i of voxel column col.
template <int COT, bool HEAD>
__device__ inline void conv_store(const ConvAcc<COT> (&acc)[kCTY], const ConvOut& o, int n, int Co,
                                  int ct0, int gx, int y0, int gz, int H, int W, int D) {
  const int lane = threadIdx.x & 63, q = lane >> 4;
  const size_t HW = (size_t)H * W, DHW = D * HW;
  const bool in = gx < W && gz < D;
  float bias[COT][4], hw[4][3];
#pragma unroll
  for (int c = 0; c < COT; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int co = (ct0 + c) * 16 + 4 * q + i;
      bias[c][i] = o.bias && co < Co ? o.bias[co] : 0.f;
    }
  if constexpr (HEAD) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int k = 0; k < 3; ++k) hw[i][k] = o.hw[(4 * q + i) * 16 + k];
  }
#pragma unroll
  for (int r = 0; r < kCTY; ++r) {
    const int gy = y0 + r;
    if (gy >= H) break;
    // a uniform part (sample, channel 16 c + i) and this lane's part
    const size_t vox = in ? gz * HW + (size_t)gy * W + gx : 0, lane_at = 4 * q * DHW + vox;
    float head[3] = {0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < COT; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int cu = (ct0 + c) * 16 + i;
        if (cu + 4 * q >= Co || !in) continue;
        const size_t at = ((size_t)n * Co + cu) * DHW;
        float val = (acc[r].hi[c][i] + acc[r].lo[c][i]) + bias[c][i];
        if (o.relu) val = fmaxf(val, 0.f);
        if (o.rpre) (o.rpre + at)[lane_at] = val;
        if (o.add) val += (o.add + at)[lane_at];
        if (o.y) (o.y + at)[lane_at] = val;
        if constexpr (HEAD) {
#pragma unroll
          for (int k = 0; k < 3; ++k) head[k] += hw[i][k] * val;
        }
      }
    if constexpr (HEAD) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        head[k] += __shfl_xor(head[k], 16, 64);
        head[k] += __shfl_xor(head[k], 32, 64);
      }
      const float v = q == 0 ? head[0] : (q == 1 ? head[1] : head[2]);
      if (q < 3 && in) o.hy[((size_t)n * 3 + q) * DHW + vox] = v + o.hb[q];
    }
  }
}

// Input at the output's resolution.  The 32 slots are 4 taps x 8 channels: lane
// group q takes tap 4 s + q of k-step s (7 steps cover the 27 taps, tap 27 has
// zero weights); one chunk of 8 channels is staged at a time, the 18 x 6 x 6
// halo.  Bound: with 16 output channels a B operand feeds one MFMA, and its
// LDS read (8 cycles of the CU) outweighs the MFMA (16 cycles on each of four
// SIMDs).  Measured, layers 1-4 on a 1 x 104^3 grid: 62, 35, 28, 47 us with every
// stage's loads waited for -> 54, 32, 23, 33 us.
// SEQ: the training pass's forward.  A ReLU's mask is a step function of the
// value before it, so a mask that flips with the rounding moves the gradient by
// 1e-5 and more (about one pass in fifteen); its sums keep one fixed order of the
// terms, and the decoder's layers (up = 1: x stored at half resolution) the order
// of this kernel.
template <int COT, bool SEQ>
__global__ __launch_bounds__(256) void k_conv3_mfma(const float* __restrict__ x, int up, int Ci,
                                                    int Co, int Cop, int D, int H, int W, int tx, int ty,
                                                    const uint4* __restrict__ wp, ConvOut out) {
  constexpr int kPer = (kCHV + 255) / 256;
  __shared__ uint4 lds[3][kCHV];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 15, q = lane >> 4;
  const unsigned lane_w = col * 4 + q;       // this lane's packed weights
  const int tile = xcd_block(blockIdx.x, gridDim.x);
  const int n = blockIdx.y, ct0 = blockIdx.z * COT;
  const int bx = tile % tx, by = (tile / tx) % ty, bz = tile / (tx * ty);
  const int x0 = bx * kCTX, y0 = by * kCTY, z0 = bz * kCTZ;
  const size_t HWi = (size_t)(H >> up) * (W >> up), DHWi = (D >> up) * HWi;
  const float* xn = x + (size_t)n * Ci * DHWi;
  const int nchunk = (Ci + 7) >> 3;

  unsigned voff[kPer];                       // this thread's halo voxels
  bool vin[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int v = threadIdx.x + 256 * u;
    const int gx = x0 - 1 + v % kCHX, gy = y0 - 1 + (v / kCHX) % kCHY, gz = z0 - 1 + v / (kCHX * kCHY);
    vin[u] = v < kCHV && (unsigned)gx < (unsigned)W && (unsigned)gy < (unsigned)H &&
             (unsigned)gz < (unsigned)D;
    voff[u] = vin[u] ? (unsigned)((gz >> up) * HWi + (size_t)(gy >> up) * (W >> up) + (gx >> up)) : 0u;
  }
  float stage[kPer][8];
  auto load = [&](int ch) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float* xc = xn + (size_t)min(8 * ch + j, Ci - 1) * DHWi;
#pragma unroll
      for (int u = 0; u < kPer; ++u) stage[u][j] = xc[voff[u]];
    }
  };

  ConvAcc<COT> acc[kCTY];
  conv_zero(acc);

  load(0);
  for (int ch = 0; ch < nchunk; ++ch) {
    const uint4* wc = wp + ((size_t)ch * kCSteps * Cop + ct0 * 16) * 4;
    auto weights = [&](int s, uint4 (&a)[COT]) {
#pragma unroll
      for (int c = 0; c < COT; ++c) a[c] = (wc + ((size_t)s * Cop + c * 16) * 4)[lane_w];
    };
    auto step = [&](int s, const uint4 (&a)[COT]) {
      // tap 27 (weights zero) reads tap 26's voxel, a staged finite value
      const int t = 4 * s + q < 27 ? 4 * s + q : 26;
      const int dx = t % 3, dy = (t / 3) % 3, dz = t / 9;
      const int base = ((w + dz) * kCHY + dy) * kCHX + col + dx;
#pragma unroll
      for (int r = 0; r < kCTY; ++r) {
        const int v = base + r * kCHX;
        mfma3<COT, SEQ>(a, __builtin_bit_cast(cbf16x8, lds[0][v]),
                        __builtin_bit_cast(cbf16x8, lds[1][v]),
                        __builtin_bit_cast(cbf16x8, lds[2][v]), acc[r]);
      }
    };
    // one channel tile: all of the chunk's weights are loaded before the
    // staging, which hides them; more: two steps' weights alternate
    constexpr int kA = COT == 1 ? kCSteps : 2;
    uint4 a[kA][COT];
#pragma unroll
    for (int s = 0; s < (COT == 1 ? kCSteps : 1); ++s) weights(s, a[s]);
    __syncthreads();                         // the previous chunk's reads are done
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int v = threadIdx.x + 256 * u;
      if (v >= kCHV) break;
#pragma unroll
      for (int j = 0; j < 8; ++j) stage[u][j] = vin[u] && 8 * ch + j < Ci ? stage[u][j] : 0.f;
      stage_split(stage[u], lds[0], lds[1], lds[2], v);
    }
    __syncthreads();
    if (ch + 1 < nchunk) load(ch + 1);
    if constexpr (COT == 1) {
#pragma unroll
      for (int s = 0; s < kCSteps; ++s) step(s, a[s]);
    } else {
#pragma unroll 1
      for (int s = 0; s + 1 < kCSteps; s += 2) {
        weights(s + 1, a[1]);
        step(s, a[0]);
        weights(s + 2, a[0]);
        step(s + 1, a[1]);
      }
      step(kCSteps - 1, a[0]);
    }
  }
  conv_store<COT, false>(acc, out, n, Co, ct0, x0 + col, y0, z0 + w, H, W, D);
}

// Input stored at half resolution and read as its nearest-neighbour upsampling
// (voxel v of the output grid reads v / 2), Ci a multiple of 8.  The 10 x 4 x 4
// stored voxels of 32 channels are staged at a time, so each value is loaded
// and split once, not once per output voxel that reads it.  The 32 slots are 32
// channels at one tap (lane group q: channels 8 q .. 8 q + 7): the six tile rows
// r + dy read only four stored rows, so 4 B operands and the weights of the
// three dy serve 12 products.  Bound: the matrix cores (36 products of 16
// cycles per 12 LDS reads of 8 cycles a CU).
// Measured, layers 5-7 on a 1 x 104^3 grid: 94, 111, 175 us in the form above on
// an 18 x 6 x 6 halo, the head 25 us -> 44, 58, 98 us with the head in the last.
// (The weights two steps ahead, all steps unrolled: 48, 66, 124 us, an occupancy
// step lost.)
constexpr int kUX = kCTX / 2 + 2, kUY = kCTY / 2 + 2, kUZ = kCTZ / 2 + 2;
constexpr int kUV = kUX * kUY * kUZ;           // 160 stored voxels
constexpr int kUP = kUV + 8;                   // pitch of a channel group: its banks rotate

template <bool HEAD>
__global__ __launch_bounds__(256) void k_conv3_up(const float* __restrict__ x, int Ci, int Co,
                                                  int Cop, int D, int H, int W, int tx, int ty,
                                                  const uint4* __restrict__ wp, ConvOut out) {
  constexpr int kPer = (4 * kUV + 255) / 256;
  __shared__ uint4 lds[3][4 * kUP];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int col = lane & 15, q = lane >> 4;
  const unsigned lane_w = col * 4 + q;       // this lane's packed weights
  const int tile = xcd_block(blockIdx.x, gridDim.x);
  const int n = blockIdx.y, ct0 = blockIdx.z;
  const int bx = tile % tx, by = (tile / tx) % ty, bz = tile / (tx * ty);
  const int x0 = bx * kCTX, y0 = by * kCTY, z0 = bz * kCTZ;
  const int Wi = W >> 1, Hi = H >> 1, Di = D >> 1;
  const size_t HWi = (size_t)Hi * Wi, DHWi = Di * HWi;
  const float* xn = x + (size_t)n * Ci * DHWi;
  const int nstage = (Ci + 31) >> 5;

  // this thread's staged entries, lds[.][group * kUP + voxel] for channel
  // group e / kUV: element offset in a stage's 32 channels
  size_t voff[kPer];
  int vgrp[kPer];
  bool vin[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {
    const int e = threadIdx.x + 256 * u, v = e % kUV;
    vgrp[u] = e / kUV;
    const int gx = (x0 >> 1) - 1 + v % kUX, gy = (y0 >> 1) - 1 + (v / kUX) % kUY,
              gz = (z0 >> 1) - 1 + v / (kUX * kUY);
    vin[u] = e < 4 * kUV && (unsigned)gx < (unsigned)Wi && (unsigned)gy < (unsigned)Hi &&
             (unsigned)gz < (unsigned)Di;
    voff[u] = vin[u] ? 8 * vgrp[u] * DHWi + gz * HWi + (size_t)gy * Wi + gx : 0;
  }
  float stage[kPer][8];
  auto load = [&](int st) {
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const bool in = vin[u] && 32 * st + 8 * vgrp[u] < Ci;
      const float* p = xn + (in ? (size_t)32 * st * DHWi + voff[u] : 0);
#pragma unroll
      for (int j = 0; j < 8; ++j) stage[u][j] = p[j * DHWi];
#pragma unroll
      for (int j = 0; j < 8; ++j) stage[u][j] = in ? stage[u][j] : 0.f;
    }
  };

  ConvAcc<1> acc[kCTY];
  conv_zero(acc);

  load(0);
  for (int st = 0; st < nstage; ++st) {
    const uint4* wc = wp + ((size_t)st * 27 * Cop + ct0 * 16) * 4;
    // weights of the three dy at (dz, dx) = (i / 3, i % 3)
    auto weights = [&](int i, uint4 (&a)[3][1]) {
#pragma unroll
      for (int dy = 0; dy < 3; ++dy)
        a[dy][0] = (wc + (size_t)(9 * (i / 3) + 3 * dy + i % 3) * Cop * 4)[lane_w];
    };
    auto step = [&](int i, const uint4 (&a)[3][1]) {
      const int hz = ((w + i / 3 - 1) >> 1) + 1, hx = ((col + i % 3 - 1) >> 1) + 1;
      const int base = q * kUP + hz * kUY * kUX + hx;
#pragma unroll
      for (int hy = 0; hy < kUY; ++hy) {
        const cbf16x8 b0 = __builtin_bit_cast(cbf16x8, lds[0][base + hy * kUX]);
        const cbf16x8 b1 = __builtin_bit_cast(cbf16x8, lds[1][base + hy * kUX]);
        const cbf16x8 b2 = __builtin_bit_cast(cbf16x8, lds[2][base + hy * kUX]);
#pragma unroll
        for (int r = 0; r < kCTY; ++r)
#pragma unroll
          for (int dy = 0; dy < 3; ++dy)
            if (((r + dy - 1) >> 1) + 1 == hy) mfma3<1>(a[dy], b0, b1, b2, acc[r]);
      }
    };
    uint4 a[2][3][1];
    weights(0, a[0]);
    __syncthreads();                         // the previous stage's reads are done
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = threadIdx.x + 256 * u;
      if (e >= 4 * kUV) break;
      stage_split(stage[u], lds[0], lds[1], lds[2], e + vgrp[u] * (kUP - kUV));
    }
    __syncthreads();
    if (st + 1 < nstage) load(st + 1);
#pragma unroll 1
    for (int i = 0; i < 8; i += 2) {         // each step's weights are loaded a step ahead
      weights(i + 1, a[1]);
      step(i, a[0]);
      weights(i + 2, a[0]);
      step(i + 1, a[1]);
    }
    step(8, a[0]);
  }
  conv_store<1, HEAD>(acc, out, n, Co, ct0, x0 + col, y0, z0 + w, H, W, D);
}

// Packed A operands from the BF16-exact FP32 layout w[(ci * 27 + tap) * Cop +
// co].  up 0: wp[((ch * 7 + s) * Cop + co) * 4 + q] holds input channels 8 ch ..
// 8 ch + 7 at tap 4 s + q for output channel co; up 1: wp[((st * 27 + t) * Cop +
// co) * 4 + q] holds channels 32 st + 8 q .. + 7 at tap t.  Zero past Ci and
// for tap 27.
__global__ void k_pack_conv3(const float* __restrict__ w, int up, int Ci, int Cop, int total,
                             uint4* __restrict__ wp) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int q = i & 3, co = (i >> 2) % Cop, k = i / (4 * Cop);
  const int t = up ? k % 27 : 4 * (k % kCSteps) + q;
  const int c0 = up ? 32 * (k / 27) + 8 * q : 8 * (k / kCSteps);
  unsigned p[4];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    const int c = c0 + j;
    const float a = t < 27 && c < Ci ? w[((size_t)c * 27 + t) * Cop + co] : 0.f;
    const float b = t < 27 && c + 1 < Ci ? w[((size_t)(c + 1) * 27 + t) * Cop + co] : 0.f;
    p[j >> 1] = (__float_as_uint(a) >> 16) | (__float_as_uint(b) & 0xffff0000u);
  }
  wp[i] = uint4{p[0], p[1], p[2], p[3]};
}

size_t conv3_packed_words(int up, int Ci, int Co) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB;
  return (size_t)(up ? (Ci + 31) / 32 * 27 : (Ci + 7) / 8 * kCSteps) * Cop * 4;
}

void launch_pack_conv3(const float* w, int up, int Ci, int Co, uint4* wp, hipStream_t s) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB;
  const int total = (int)conv3_packed_words(up, Ci, Co);
  k_pack_conv3<<<div_up(total, 256), 256, 0, s>>>(w, up, Ci, Cop, total, wp);
}

void launch_conv3_mfma(const float* x, int up, int N, int Ci, int Co, int D, int H, int W,
                       const uint4* wp, const float* b, int relu, const float* add, float* y,
                       hipStream_t s, const float* hw, const float* hb, float* hy) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB, ntile = Cop / 16;
  const int tx = div_up(W, kCTX), ty = div_up(H, kCTY), tz = div_up(D, kCTZ);
  const long tiles = (long)tx * ty * tz;
  const ConvOut o{b, relu, nullptr, add, y, hw, hb, hy};
  // channel tiles per block: the largest power of two dividing ntile (<= 4;
  // one for upsampled inputs, whose operands serve three products anyway: two
  // took 73 us instead of 58 for the 64 -> 32 layer of the 104^3 grid), halved
  // while the grid has fewer than kConvBlocks blocks
  int cot = 1;
  while (!up && cot < 4 && ntile % (2 * cot) == 0) cot *= 2;
  while (cot > 1 && tiles * N * (ntile / cot) < kConvBlocks) cot /= 2;
  dim3 grid((unsigned)tiles, N, ntile / cot);
  if (up) {
    if (hw) k_conv3_up<true><<<grid, 256, 0, s>>>(x, Ci, Co, Cop, D, H, W, tx, ty, wp, o);
    else k_conv3_up<false><<<grid, 256, 0, s>>>(x, Ci, Co, Cop, D, H, W, tx, ty, wp, o);
    return;
  }
#define SGMG_CONV3(COT, SEQ) \
  k_conv3_mfma<COT, SEQ><<<grid, 256, 0, s>>>(x, 0, Ci, Co, Cop, D, H, W, tx, ty, wp, o)
  switch (cot) {
    case 4: SGMG_CONV3(4, false); break;
    case 2: SGMG_CONV3(2, false); break;
    default: SGMG_CONV3(1, false); break;
  }
#undef SGMG_CONV3
}

void launch_conv3_train(const float* x, int up, int N, int Ci, int Co, int D, int H, int W,
                        const uint4* wp, const float* b, int relu, float* rpre, const float* add,
                        float* y, hipStream_t s) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB, ntile = Cop / 16;
  const int tx = div_up(W, kCTX), ty = div_up(H, kCTY), tz = div_up(D, kCTZ);
  const long tiles = (long)tx * ty * tz;
  const ConvOut o{b, relu, rpre, add, y, nullptr, nullptr, nullptr};
  int cot = 1;                               // as above
  while (cot < 4 && ntile % (2 * cot) == 0) cot *= 2;
  while (cot > 1 && tiles * N * (ntile / cot) < kConvBlocks) cot /= 2;
  const dim3 grid((unsigned)tiles, N, ntile / cot);
#define SGMG_CONV3(COT, SEQ) \
  k_conv3_mfma<COT, SEQ><<<grid, 256, 0, s>>>(x, up, Ci, Co, Cop, D, H, W, tx, ty, wp, o)
  switch (cot) {
    case 4: SGMG_CONV3(4, true); break;
    case 2: SGMG_CONV3(2, true); break;
    default: SGMG_CONV3(1, true); break;
  }
#undef SGMG_CONV3
}

// The same operands (up 0) for the data gradients, whose weights are w with the
// channels swapped and the taps flipped, straight from w[(ci * 27 + tap) * Cop +
// co]: all layers in one launch (a transposed copy and a pack per layer took
// 12 launches of 4.6 us).
__global__ void k_pack_conv3_flip(ConvPacks ps) {
  int i = blockIdx.x * blockDim.x + threadIdx.x, l = 0;
  while (l < ps.n && i >= ps.p[l].total) i -= ps.p[l++].total;
  if (l == ps.n) return;
  const ConvPacks::One& p = ps.p[l];
  const int q = i & 3, ci = (i >> 2) % p.Cip, k = i / (4 * p.Cip);
  const int t = 4 * (k % kCSteps) + q, c0 = 8 * (k / kCSteps);
  unsigned v[4];
#pragma unroll
  for (int j = 0; j < 8; j += 2) {
    float f[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int co = c0 + j + h;
      f[h] = t < 27 && co < p.Co && ci < p.Ci ? p.w[((size_t)ci * 27 + 26 - t) * p.Cop + co] : 0.f;
    }
    v[j >> 1] = (__float_as_uint(f[0]) >> 16) | (__float_as_uint(f[1]) & 0xffff0000u);
  }
  p.wp[i] = uint4{v[0], v[1], v[2], v[3]};
}

void launch_pack_conv3_flip(ConvPacks ps, hipStream_t s) {
  long total = 0;
  for (int l = 0; l < ps.n; ++l) {
    ConvPacks::One& p = ps.p[l];
    p.Cop = (p.Co + kCOB - 1) / kCOB * kCOB;
    p.Cip = (p.Ci + kCOB - 1) / kCOB * kCOB;
    p.total = (int)conv3_packed_words(0, p.Co, p.Ci);
    total += p.total;
  }
  k_pack_conv3_flip<<<div_up(total, 256), 256, 0, s>>>(ps);
}

// Weights for the data gradient: wt[(co * K3 + (K3 - 1 - t)) * Cip + ci] =
// w[(ci * K3 + t) * Cop + co]  (channels swapped, taps flipped).
__global__ void k_weight_transpose(const float* __restrict__ w, int Ci, int Co, int Cop, int K3,
                                   int Cip, float* __restrict__ wt) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Co * K3 * Cip) return;
  const int ci = i % Cip, t = (i / Cip) % K3, co = i / (Cip * K3);
  wt[i] = ci < Ci ? w[((size_t)ci * K3 + (K3 - 1 - t)) * Cop + co] : 0.f;
}

void launch_weight_transpose(const float* w, int Ci, int Co, int K, float* wt, hipStream_t s) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB;
  const int Cip = (Ci + kCOB - 1) / kCOB * kCOB;
  const int K3 = K * K * K;
  k_weight_transpose<<<div_up((long)Co * K3 * Cip, 256), 256, 0, s>>>(w, Ci, Co, Cop, K3, Cip, wt);
}

// Weight and bias gradients of the 1x1x1 layer, first stage: block (ci,
// co-quad, chunk) sums dy[n, co, v] * x[n, ci, v] over its voxel chunk for 4
// output channels; the block totals go to part[chunk][...] and a second
// kernel adds the chunks in order (deterministic).
constexpr int kWGChunk = 4096;

__global__ __launch_bounds__(256) void k_conv1_wgrad(const float* __restrict__ x,
                                                     const float* __restrict__ dy, int N, int Ci,
                                                     int Co, long DHW, float* __restrict__ part) {
  __shared__ float red[4][8];
  const long total = (long)N * DHW;
  const int ci = blockIdx.x, co0 = blockIdx.y * 4, chunk = blockIdx.z;
  float acc[4] = {}, accb[4] = {};
  const long beg = (long)chunk * kWGChunk;
  const long end = beg + kWGChunk < total ? beg + kWGChunk : total;
  for (long g = beg + threadIdx.x; g < end; g += 256) {
    const int n = (int)(g / DHW);
    const long v = g % DHW;
    const float xv = x[((size_t)n * Ci + ci) * DHW + v];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float gy = co0 + c < Co ? dy[((size_t)n * Co + co0 + c) * DHW + v] : 0.f;
      acc[c] += gy * xv;
      accb[c] += gy;
    }
  }
  // fixed-order block reduction: wave sums, then the 4 wave totals in order
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    float s = c < 4 ? acc[c] : accb[c - 4];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) red[wv][c] = s;
  }
  __syncthreads();
  // layout of part: [chunk][ci][co-quad][8]
  const int nq = (Co + 3) / 4;
  float* dst = part + (((size_t)chunk * Ci + ci) * nq + blockIdx.y) * 8;
  const int i = threadIdx.x;
  if (i < 8) dst[i] = red[0][i] + red[1][i] + red[2][i] + red[3][i];
}

// Second stage: dw[ci * Cop + co] and db[co] (db taken from ci = 0).
__global__ void k_conv1_wgrad_sum(const float* __restrict__ part, int nchunks, int Ci, int Co,
                                  int Cop, float* __restrict__ dw, float* __restrict__ db) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const int nq = (Co + 3) / 4;
  if (i >= Ci * nq * 8) return;
  const int j = i % 8, q = (i / 8) % nq, ci = i / (8 * nq);
  float s = 0.f;
  for (int c0 = 0; c0 < nchunks; c0 += 16) {       // sixteen loads together, the adds in order
    float v[16];
#pragma unroll
    for (int c = 0; c < 16; ++c)
      v[c] = part[(((size_t)min(c0 + c, nchunks - 1) * Ci + ci) * nq + q) * 8 + j];
#pragma unroll
    for (int c = 0; c < 16; ++c)
      if (c0 + c < nchunks) s += v[c];
  }
  const int co = q * 4 + (j & 3);
  if (co >= Co) return;
  if (j < 4) dw[(size_t)ci * Cop + co] = s;
  else if (ci == 0) db[co] = s;
}

// Weight and bias gradients of the 3x3x3 layers on the matrix cores
// (v_mfma_f32_16x16x4_f32: FP32 operands, FP32 accumulation):
//   dw[ci, t, co] = sum_v dy[co, v] x[ci, v + t - 1],  db[co] = sum_v dy[co, v].
// Per MFMA A is 16 output channels x 4 voxels of dy, B 4 voxels x 16 input
// channels of x at one tap; the four voxels follow each other in x.
//
// Block: 16 input channels x 16 output channels x all taps, over a run of
// spatial tiles of 16 (x) x 4 x 4 voxels.  Per tile the dy voxels and the 18 x
// 6 x 6 halo of x are staged in LDS, channels innermost with a pitch of 17
// floats (the staging writes run along voxels, the operand reads along
// channels: neither meets a bank twice); a tile outside the volume holds
// zeros, and rows and x-quads past its end are skipped.  Wave w accumulates
// taps 7 w .. 7 w + 6 (seven independent 16 x 16 sums); the 28th is dy times
// ones, the bias gradient.  The run's sums go to part[run][...], and a
// second kernel adds the runs in FP64 in a fixed order (deterministic).
// Bound: the FP32 matrix rate (157 TFLOP/s: 32 cycles per MFMA, 8 of LDS
// reads). A tile is summed by itself (64 steps of the matrix cores) and added
// to the run's sum, which keeps the FP32 chains short. The next tile is loaded
// while this one is multiplied, and the operands of the next four voxels are
// read a step ahead.
// Measured, 8 samples of a 32^3 mesh (40^3 voxels), seven layers: 2565 us
// (vector ALU, one input and four output channels per block, 31 neighbour
// loads per voxel) -> 639 us, the sums 118 -> 42 us.
constexpr int kWgPitch = 17;

//
// NC = 5 (at most five input channels): a column is (channel, x tap), column 3
// ci + dx, so one product serves three taps and ten sums (nine (y, z) taps and
// the bias) replace 28; wave w takes sums w, w + 4, w + 8.  The 5 -> 16 layer:
// 118 us with 11 of 16 columns empty, 62 us.  Same bits.
template <int NC>
__global__ __launch_bounds__(256, 2) void k_conv3_wgrad(const float* __restrict__ x, int up,
                                                     const float* __restrict__ dy, int Ci, int Co,
                                                     int Cop, int D, int H, int W, int tx, int ty,
                                                     int tz, int tiles, int run,
                                                     float* __restrict__ part) {
  __shared__ float xs[kCHV * kWgPitch];
  __shared__ float ds[kCTX * kCTY * kCTZ * kWgPitch];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int col = lane & 15, k = lane >> 4;
  const int ci0 = blockIdx.y * 16, co0 = blockIdx.z * 16;
  const int HW = H * W, Wi = W >> up, HWi = (H >> up) * Wi;
  const size_t DHW = (size_t)D * HW, DHWi = (size_t)(D >> up) * HWi;
  constexpr bool kPack = NC < 16;
  constexpr int NS = kPack ? 3 : 7;             // sums of a wave
  auto sum_of = [&](int j) { return kPack ? w + 4 * j : 7 * w + j; };
  int off[NS];                                  // LDS offset of this lane's operand per sum
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int t = kPack ? 3 * min(sum_of(j), 8) + min(col, 14) % 3 : min(sum_of(j), 26);
    const int dx = t % 3, dyy = (t / 3) % 3, dz = t / 9;
    off[j] = ((dz * kCHY + dyy) * kCHX + dx + k) * kWgPitch + (kPack ? min(col, 14) / 3 : col);
  }
  constexpr int jb = kPack ? 2 : 6;             // the bias gradient: this sum of
  const bool ones = w == (kPack ? 1 : 3);       // this wave
  cf32x4 acc[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) acc[j] = cf32x4{0.f, 0.f, 0.f, 0.f};

  // the staged voxels of a tile that this thread loads: three of the halo
  // (the third only for the first 136 threads), one of dy
  float xq[3][NC], dq[16];
  auto load = [&](int tile) {
    const int bx = tile % tx, by = (tile / tx) % ty, bz = (tile / (tx * ty)) % tz,
              n = tile / (tx * ty * tz);
    const int x0 = bx * kCTX, y0 = by * kCTY, z0 = bz * kCTZ;
    const float* xn = x + ((size_t)n * Ci + ci0) * DHWi;
    const float* dn = dy + ((size_t)n * Co + co0) * DHW;
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int v = tid + 256 * u;
      const int hx = v % kCHX, hy = (v / kCHX) % kCHY, hz = v / (kCHX * kCHY);
      const int gx = x0 - 1 + hx, gy = y0 - 1 + hy, gz = z0 - 1 + hz;
      const bool in = v < kCHV && (unsigned)gx < (unsigned)W && (unsigned)gy < (unsigned)H &&
                      (unsigned)gz < (unsigned)D;
      const size_t o = in ? (size_t)(gz >> up) * HWi + (size_t)(gy >> up) * Wi + (gx >> up) : 0;
#pragma unroll
      for (int c = 0; c < NC; ++c) xq[u][c] = xn[min(c, Ci - 1 - ci0) * DHWi + o];
#pragma unroll
      for (int c = 0; c < NC; ++c) xq[u][c] = in && ci0 + c < Ci ? xq[u][c] : 0.f;
    }
    const int gx = x0 + (tid & 15), gy = y0 + ((tid >> 4) & 3), gz = z0 + (tid >> 6);
    const bool in = gx < W && gy < H && gz < D;
    const size_t o = in ? (size_t)gz * HW + (size_t)gy * W + gx : 0;
#pragma unroll
    for (int c = 0; c < 16; ++c) dq[c] = dn[min(c, Co - 1 - co0) * DHW + o];
#pragma unroll
    for (int c = 0; c < 16; ++c) dq[c] = in && co0 + c < Co ? dq[c] : 0.f;
  };

  const int last = min((int)(blockIdx.x + 1) * run, tiles);
  load(blockIdx.x * run);
  for (int tile = blockIdx.x * run; tile < last; ++tile) {
    __syncthreads();                            // the previous tile's reads are done
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int v = tid + 256 * u;
      if (v < kCHV) {
#pragma unroll
        for (int c = 0; c < NC; ++c) xs[v * kWgPitch + c] = xq[u][c];
      }
    }
#pragma unroll
    for (int c = 0; c < 16; ++c) ds[tid * kWgPitch + c] = dq[c];
    __syncthreads();
    if (tile + 1 < last) load(tile + 1);        // in flight during this tile's products
    const int nx = min(kCTX, W - (tile % tx) * kCTX), ny = min(kCTY, H - (tile / tx) % ty * kCTY),
              nz = min(kCTZ, D - (tile / (tx * ty)) % tz * kCTZ);
    // operands one step of four voxels ahead of the products
    float av[2], bv[2][NS];
    auto read = [&](int b, int z, int yy, int g) {
      const int dr = (z * kCTY + yy) * kCTX + g, xr = (z * kCHY + yy) * kCHX + g;
      av[b] = ds[(dr + k) * kWgPitch + col];
#pragma unroll
      for (int j = 0; j < NS; ++j) bv[b][j] = xs[xr * kWgPitch + off[j]];
      bv[b][jb] = ones ? 1.f : bv[b][jb];
    };
    cf32x4 sum[NS];                             // this tile's
#pragma unroll
    for (int j = 0; j < NS; ++j) sum[j] = cf32x4{0.f, 0.f, 0.f, 0.f};
    int z = 0, yy = 0, g = 0;
    auto next = [&]() {
      g += 4;
      if (g >= nx) { g = 0; if (++yy >= ny) { yy = 0; ++z; } }
    };
    auto products = [&](int b) {
#pragma unroll
      for (int j = 0; j < NS; ++j)
        sum[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[b], bv[b][j], sum[j], 0, 0, 0);
    };
    read(0, 0, 0, 0);
    next();
    while (true) {
      if (z >= nz) { products(0); break; }
      read(1, z, yy, g);
      next();
      products(0);
      if (z >= nz) { products(1); break; }
      read(0, z, yy, g);
      next();
      products(1);
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) acc[j] += sum[j];
  }
  // result: lane holds output channels 4 (lane / 16) + i of input channel col
  const size_t nw = (size_t)Ci * 27 * Cop;
  float* dst = part + (size_t)blockIdx.x * (nw + Cop);
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int q = sum_of(j), co = co0 + 4 * k;
    const bool bias = q == (kPack ? 9 : 27);
    const int ci = ci0 + (kPack ? col / 3 : col), t = kPack ? 3 * q + col % 3 : q;
    if (bias ? ci0 + col == 0 : q < (kPack ? 9 : 27) && ci < Ci && (!kPack || col < 15)) {
      float* o = bias ? dst + nw + co : dst + ((size_t)ci * 27 + t) * Cop + co;
      *(float4*)o = make_float4(acc[j][0], acc[j][1], acc[j][2], acc[j][3]);
    }
  }
}

// Sum of the runs' parts, 64 values per block, run r in slice r % 16, the
// slices added in order; values past nw are the bias gradient.
__global__ __launch_bounds__(1024) void k_conv3_wgrad_sum(const float* __restrict__ part, int runs,
                                                          size_t nw, int Cop, int Co,
                                                          float* __restrict__ dw,
                                                          float* __restrict__ db) {
  __shared__ double red[16][64];
  const int a = threadIdx.x & 63, sl = threadIdx.x >> 6;
  const size_t i = (size_t)blockIdx.x * 64 + a, n = nw + Cop;
  double s = 0.0;
  if (i < n) {
#pragma unroll 4
    for (int r = sl; r < runs; r += 16) s += (double)part[(size_t)r * n + i];
  }
  red[sl][a] = s;
  __syncthreads();
  if (sl != 0 || i >= n) return;
  s = 0.0;
#pragma unroll
  for (int q = 0; q < 16; ++q) s += red[q][a];
  if (i < nw) dw[i] = (float)s;
  else if ((int)(i - nw) < Co) db[i - nw] = (float)s;
}

// Spatial tiles, tiles per run and runs of a 3x3x3 weight gradient: the
// shortest runs with at most 512 blocks, two per compute unit, so that the
// whole grid is resident at once (the 32 -> 16 layer: 236 us with 1200 blocks
// in runs of four tiles, 229 us).
constexpr int kWgBlocks = 512;
struct WgradPlan {
  int tx, ty, tz, tiles, run, runs, gy, gz;
};
static WgradPlan wgrad_plan(int N, int Ci, int Co, int D, int H, int W) {
  WgradPlan p;
  p.tx = div_up(W, kCTX);
  p.ty = div_up(H, kCTY);
  p.tz = div_up(D, kCTZ);
  p.tiles = p.tx * p.ty * p.tz * N;
  p.gy = div_up(Ci, 16);
  p.gz = div_up(Co, 16);
  p.run = div_up(p.tiles, std::max(1, kWgBlocks / (p.gy * p.gz)));
  p.runs = div_up(p.tiles, p.run);
  return p;
}

size_t conv_wgrad_part_floats(int N, int Ci, int Co, int D, int H, int W, int K) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB;
  if (K == 3)
    return (size_t)wgrad_plan(N, Ci, Co, D, H, W).runs * ((size_t)Ci * 27 * Cop + Cop);
  const long total = (long)N * D * H * W;
  const long nchunks = (total + kWGChunk - 1) / kWGChunk;
  return (size_t)nchunks * Ci * ((Co + 3) / 4) * 8;
}

void launch_conv_wgrad(int K, const float* x, int up, const float* dy, int N, int Ci, int Co, int D,
                       int H, int W, float* part, float* dw, float* db, hipStream_t s) {
  const int Cop = (Co + kCOB - 1) / kCOB * kCOB;
  if (K == 3) {
    const WgradPlan p = wgrad_plan(N, Ci, Co, D, H, W);
    const dim3 grid(p.runs, p.gy, p.gz);
    if (Ci <= 5)
      k_conv3_wgrad<5><<<grid, 256, 0, s>>>(x, up, dy, Ci, Co, Cop, D, H, W, p.tx, p.ty, p.tz,
                                            p.tiles, p.run, part);
    else
      k_conv3_wgrad<16><<<grid, 256, 0, s>>>(x, up, dy, Ci, Co, Cop, D, H, W, p.tx, p.ty, p.tz,
                                             p.tiles, p.run, part);
    const size_t nw = (size_t)Ci * 27 * Cop;
    k_conv3_wgrad_sum<<<div_up((long)(nw + Cop), 64), 1024, 0, s>>>(part, p.runs, nw, Cop, Co, dw, db);
    return;
  }
  const long total = (long)N * D * H * W;
  const int nchunks = (int)((total + kWGChunk - 1) / kWGChunk);
  const int nq = (Co + 3) / 4;
  k_conv1_wgrad<<<dim3(Ci, nq, nchunks), 256, 0, s>>>(x, dy, N, Ci, Co, (long)D * H * W, part);
  k_conv1_wgrad_sum<<<div_up((long)Ci * nq * 8, 256), 256, 0, s>>>(part, nchunks, Ci, Co, Cop, dw, db);
}

// 2x2x2 mean pooling and its adjoint; nearest x2 upsampling and its adjoint.
// Grid: x over (volume nc, output plane d), y over the voxels of the plane;
// the plane and volume indices are uniform over a block.
__global__ void k_pool(const float* __restrict__ x, int D, int H, int W, float* __restrict__ y) {
  const int Do = D >> 1, Ho = H >> 1, Wo = W >> 1;
  const int j = blockIdx.y * blockDim.x + threadIdx.x;
  if (j >= Ho * Wo) return;
  const int dd = blockIdx.x % Do, nc = blockIdx.x / Do;
  const int ho = j / Wo, wo = j - ho * Wo;
  const float* b = x + ((size_t)nc * D + 2 * dd) * H * W + (size_t)(2 * ho) * W + 2 * wo;
  float s = 0.f;
  for (int a = 0; a < 8; ++a) s += b[(size_t)(a >> 2) * H * W + ((a >> 1) & 1) * W + (a & 1)];
  y[((size_t)nc * Do + dd) * Ho * Wo + j] = s * 0.125f;
}

// The adjoint of the pooling (scale 1/8), the skip's gradient and the ReLU mask in
// one pass over the fine grid (16 channels of 8 x 40^3: 42 us in two, 22 us).
__global__ void k_expand_relu(const float* __restrict__ x, int D, int H, int W, float scale,
                              const float* __restrict__ r, const float* __restrict__ extra,
                              float* __restrict__ y) {
  const int j = blockIdx.y * blockDim.x + threadIdx.x;
  if (j >= H * W) return;
  const int d = blockIdx.x % D, nc = blockIdx.x / D;
  const int h = j / W, w = j - h * W;
  const int Hc = H >> 1, Wc = W >> 1;
  const size_t i = ((size_t)nc * D + d) * H * W + j;
  const float g =
      extra[i] + scale * x[(((size_t)nc * (D >> 1) + (d >> 1)) * Hc + (h >> 1)) * Wc + (w >> 1)];
  y[i] = r[i] > 0.f ? g : 0.f;
}
__global__ void k_sum8_relu(const float* __restrict__ x, int D, int H, int W,
                            const float* __restrict__ r, float* __restrict__ y,
                            float* __restrict__ dr) {
  const int Do = D >> 1, Ho = H >> 1, Wo = W >> 1;
  const int j = blockIdx.y * blockDim.x + threadIdx.x;
  if (j >= Ho * Wo) return;
  const int dd = blockIdx.x % Do, nc = blockIdx.x / Do;
  const int ho = j / Wo, wo = j - ho * Wo;
  const float* b = x + ((size_t)nc * D + 2 * dd) * H * W + (size_t)(2 * ho) * W + 2 * wo;
  float s = 0.f;
  for (int a = 0; a < 8; ++a) s += b[(size_t)(a >> 2) * H * W + ((a >> 1) & 1) * W + (a & 1)];
  const size_t i = ((size_t)nc * Do + dd) * Ho * Wo + j;
  if (y) y[i] = s;
  dr[i] = r[i] > 0.f ? s : 0.f;
}

void launch_pool(const float* x, int NC, int D, int H, int W, float* y, hipStream_t s) {
  k_pool<<<dim3(NC * (D / 2), div_up((H / 2) * (W / 2), 256)), 256, 0, s>>>(x, D, H, W, y);
}
void launch_expand_relu(const float* x, int NC, int D, int H, int W, float scale, const float* r,
                        const float* extra, float* y, hipStream_t s) {
  k_expand_relu<<<dim3(NC * D, div_up(H * W, 256)), 256, 0, s>>>(x, D, H, W, scale, r, extra, y);
}
void launch_sum8_relu(const float* x, int NC, int D, int H, int W, const float* r, float* y, float* dr,
                      hipStream_t s) {
  k_sum8_relu<<<dim3(NC * (D / 2), div_up((H / 2) * (W / 2), 256)), 256, 0, s>>>(x, D, H, W, r, y, dr);
}

// dr = dy * (r > 0)
__global__ void k_relu_bwd(const float* __restrict__ dy, const float* __restrict__ r, long n,
                           float* __restrict__ dr) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dr[i] = r[i] > 0.f ? dy[i] : 0.f;
}

void launch_relu_bwd(const float* dy, const float* r, long n, float* dr, hipStream_t s) {
  k_relu_bwd<<<div_up(n, 256), 256, 0, s>>>(dy, r, n, dr);
}

__global__ void k_add(const float* __restrict__ a, const float* __restrict__ b, long n,
                      float* __restrict__ y) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = a[i] + b[i];
}

void launch_add(const float* a, const float* b, long n, float* y, hipStream_t s) {
  k_add<<<div_up(n, 256), 256, 0, s>>>(a, b, n, y);
}

// Masked MSE: loss = sum m (y - t)^2 / sum m over (N, 3, DHW), m = mask[n, v]
// broadcast over the channels; dy = 2 m (y - t) / sum m.  Deterministic:
// block partials + launch_finalize.
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ y, const float* __restrict__ t,
                                             const float* __restrict__ mask, int N, int C, int DHW,
                                             float* __restrict__ dy, RedWs ws) {
  const long total = (long)N * C * DHW;
  double se = 0.0, sm = 0.0;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    const int v = (int)(i % DHW);
    const int n = (int)(i / ((long)C * DHW));
    const float m = mask ? mask[(size_t)n * DHW + v] : 1.f;
    const float e = y[i] - t[i];
    se += (double)m * e * e;
    sm += m;
    dy[i] = m * e;            // scaled in k_mse_scale once sum m is known
  }
  const double vv[2] = {se, sm};
  grid_sum<2>(vv, ws);
}

__global__ void k_mse_scale(float* __restrict__ dy, long n, const double* __restrict__ sums) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dy[i] = (float)(2.0 / sums[1]) * dy[i];
}

void launch_mse(const float* y, const float* t, const float* mask, int N, int C, int DHW, float* dy,
                RedWs ws, double* sums, hipStream_t s) {
  const long total = (long)N * C * DHW;
  const unsigned grid = (unsigned)std::min<long>(div_up(total, 256), 1024);
  k_mse<<<grid, 256, 0, s>>>(y, t, mask, N, C, DHW, dy, ws);
  launch_finalize(ws, grid, 2, sums, s);
  k_mse_scale<<<div_up(total, 256), 256, 0, s>>>(dy, total, sums);
}

// Adam on FP32 master weights; the compute copy is the master value rounded
// to BF16 (round to nearest even), stored as FP32.
__device__ inline float round_bf16(float v) {
  return (float)(__bf16)v;
}

__global__ void k_adam(float* __restrict__ p, float* __restrict__ pq, const float* __restrict__ g,
                       float* __restrict__ m, float* __restrict__ v, long n, float lr, float b1,
                       float b2, float eps, float c1, float c2, int quantize) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float upd = lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  const float np = p[i] - upd;
  p[i] = np;
  if (pq) pq[i] = quantize ? round_bf16(np) : np;
}

void launch_adam(float* p, float* pq, const float* g, float* m, float* v, long n, float lr, float b1,
                 float b2, float eps, int step, int quantize, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  k_adam<<<div_up(n, 256), 256, 0, s>>>(p, pq, g, m, v, n, lr, b1, b2, eps, c1, c2, quantize);
}

__global__ void k_round_bf16(const float* __restrict__ p, float* __restrict__ q, long n) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) q[i] = round_bf16(p[i]);
}

void launch_round_bf16(const float* p, float* q, long n, hipStream_t s) {
  k_round_bf16<<<div_up(n, 256), 256, 0, s>>>(p, q, n);
}

// Network input on the padded node grid (Dp, Hp, Wp >= Nz, Ny, Nx):
// channel 0 = mean density of the elements around the node, 1..3 = load
// divided by max |f|, 4 = 1 where any DOF of the node is clamped.
__global__ void k_unet_input(Grid g, const double* __restrict__ rho, const double* __restrict__ f,
                             const uint8_t* __restrict__ fixn, const double* __restrict__ fmax,
                             int Dp, int Hp, int Wp, float* __restrict__ in) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long vol = (long)Dp * Hp * Wp;
  if (i >= vol) return;
  const int x = i % Wp, y = (i / Wp) % Hp, z = i / ((long)Wp * Hp);
  float ch[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
  if (x < g.Nx && y < g.Ny && z < g.Nz) {
    double s = 0.0;
    int c = 0;
    for (int q = 0; q < 8; ++q) {
      const int ex = x - 1 + (q & 1), ey = y - 1 + ((q >> 1) & 1), ez = z - 1 + (q >> 2);
      if (ex < 0 || ey < 0 || ez < 0 || ex >= g.nx || ey >= g.ny || ez >= g.nz) continue;
      s += rho[ex + g.nx * (ey + g.ny * ez)];
      ++c;
    }
    ch[0] = (float)(c ? s / c : 0.0);
    const int node = x + g.Nx * (y + g.Ny * z);
    const double sc = *fmax > 0.0 ? 1.0 / *fmax : 0.0;
    for (int k = 0; k < 3; ++k) ch[1 + k] = (float)(f[3 * (size_t)node + k] * sc);
    ch[4] = fixn[node] ? 1.f : 0.f;
  }
  for (int k = 0; k < 5; ++k) in[k * vol + i] = ch[k];
}

__global__ void k_absmax(const double* __restrict__ a, int n, unsigned long long* __restrict__ out) {
  double m = 0.0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    m = fmax(m, fabs(a[i]));
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(out, (unsigned long long)__double_as_longlong(m));
}

__global__ void k_zero_u64(unsigned long long* p) { *p = 0ull; }

void launch_unet_input(const Grid& g, const double* rho, const double* f, const uint8_t* fixn,
                       double* fmax_scratch, int Dp, int Hp, int Wp, float* in, hipStream_t s) {
  k_zero_u64<<<1, 1, 0, s>>>((unsigned long long*)fmax_scratch);
  k_absmax<<<256, 256, 0, s>>>(f, g.n, (unsigned long long*)fmax_scratch);
  k_unet_input<<<div_up((long)Dp * Hp * Wp, 256), 256, 0, s>>>(g, rho, f, fixn, fmax_scratch, Dp,
                                                               Hp, Wp, in);
}

// Network output (3 channels on the padded grid) -> FP64 DOF vector, zero on
// clamped DOFs.
__global__ void k_unet_output(Grid g, const float* __restrict__ out, const uint8_t* __restrict__ fixn,
                              int Dp, int Hp, int Wp, double* __restrict__ u) {
  const int node = blockIdx.x * blockDim.x + threadIdx.x;
  if (node >= g.Nn) return;
  const int x = node % g.Nx, y = (node / g.Nx) % g.Ny, z = node / (g.Nx * g.Ny);
  const long vol = (long)Dp * Hp * Wp;
  const long v = ((long)z * Hp + y) * Wp + x;
  const unsigned fx = fixn[node];
  for (int k = 0; k < 3; ++k)
    u[3 * (size_t)node + k] = (fx >> k) & 1u ? 0.0 : (double)out[k * vol + v];
}

void launch_unet_output(const Grid& g, const float* out, const uint8_t* fixn, int Dp, int Hp, int Wp,
                        double* u, hipStream_t s) {
  k_unet_output<<<div_up(g.Nn, 256), 256, 0, s>>>(g, out, fixn, Dp, Hp, Wp, u);
}

// Training target: u / max|u| on the padded grid (3 channels) and a mask that
// is 1 on the nodes of the mesh.
__global__ void k_unet_target(Grid g, const double* __restrict__ u, const double* __restrict__ umax,
                              int Dp, int Hp, int Wp, float* __restrict__ t, float* __restrict__ m) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long vol = (long)Dp * Hp * Wp;
  if (i >= vol) return;
  const int x = i % Wp, y = (i / Wp) % Hp, z = i / ((long)Wp * Hp);
  const bool in = x < g.Nx && y < g.Ny && z < g.Nz;
  const double sc = *umax > 0.0 ? 1.0 / *umax : 0.0;
  const size_t node = in ? (size_t)(x + g.Nx * (y + g.Ny * z)) : 0;
  for (int k = 0; k < 3; ++k) t[k * vol + i] = in ? (float)(u[3 * node + k] * sc) : 0.f;
  if (m) m[i] = in ? 1.f : 0.f;
}

void launch_unet_target(const Grid& g, const double* u, double* umax_scratch, int Dp, int Hp, int Wp,
                        float* t, float* m, hipStream_t s) {
  k_zero_u64<<<1, 1, 0, s>>>((unsigned long long*)umax_scratch);
  k_absmax<<<256, 256, 0, s>>>(u, g.n, (unsigned long long*)umax_scratch);
  k_unet_target<<<div_up((long)Dp * Hp * Wp, 256), 256, 0, s>>>(g, u, umax_scratch, Dp, Hp, Wp, t, m);
}

// ---------------------------------------------------------------------------
// Energy-norm training score of the network's displacement shapes.  Sample
// n's output channels on the node voxels give u (zero on clamped DOFs); with
// a = f.u, b = u.K u and the compliance c = f.u* the best multiple (a / b) u
// leaves the squared energy-norm error c - a^2 / b, so the score
// 1 - a^2 / (b c) is 0 for the exact shape and 1 for u = 0.  The batch loss is
// the mean score; its output gradient is -(2 a / (b c N)) (f - (a / b) K u) on
// free DOFs.
__global__ void k_energy_u(EnergyBatch e, const float* __restrict__ y) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const Grid& g = e.g;
  if (i >= (long)e.N * g.Nn) return;
  const int n = (int)(i / g.Nn), node = (int)(i % g.Nn);
  const int x = node % g.Nx, yy = (node / g.Nx) % g.Ny, z = node / (g.Nx * g.Ny);
  const long vol = (long)e.Dp * e.Hp * e.Wp;
  const long v = ((long)z * e.Hp + yy) * e.Wp + x;
  const unsigned fx = e.fixn[node];
  double* u = e.u + (size_t)n * g.n + 3 * (size_t)node;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    u[c] = (fx >> c) & 1u ? 0.0 : (double)y[((size_t)n * 3 + c) * vol + v];
}

__global__ __launch_bounds__(256) void k_energy_Ku(EnergyBatch e) {
  __shared__ double lds[32];
  const Grid& g = e.g;
  const int n = blockIdx.y;
  const int node = blockIdx.x * 256 + threadIdx.x;
  double a = 0.0, b = 0.0;
  if (node < g.Nn) {
    const size_t off = (size_t)n * g.n, base = off + 3 * (size_t)node;
    double acc[3], xo[3];
    fine_node_Ku<double>(g, e.E + (size_t)n * g.nel, e.ke, e.u + off, node, acc, xo);
    const unsigned fx = e.fixn[node];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double kv = (fx >> c) & 1u ? 0.0 : acc[c];
      e.Ku[base + c] = kv;
      a += e.f[base + c] * xo[c];
      b += xo[c] * kv;
    }
  }
  a = block_sum(a, lds);
  b = block_sum(b, lds + 16);
  if (threadIdx.x == 0) {
    double* p = e.part + ((size_t)n * e.nb + blockIdx.x) * 2;
    p[0] = a;
    p[1] = b;
  }
}

// one block per sample: the block partials in a fixed order, then the score
// and the gradient factors (score 1 and the gradient -f / (c N) when u.K u is
// not positive)
__global__ __launch_bounds__(256) void k_energy_final(EnergyBatch e) {
  __shared__ double lds[32];
  const int n = blockIdx.x;
  double a = 0.0, b = 0.0;
  for (int i = threadIdx.x; i < e.nb; i += 256) {
    a += e.part[((size_t)n * e.nb + i) * 2];
    b += e.part[((size_t)n * e.nb + i) * 2 + 1];
  }
  a = block_sum(a, lds);
  b = block_sum(b, lds + 16);
  if (threadIdx.x != 0) return;
  const double c = e.cstar[n];
  double* sc = e.scal + 4 * (size_t)n;
  if (b > 0.0 && c > 0.0 && isfinite(a) && isfinite(b)) {
    sc[0] = 1.0 - a * a / (b * c);
    sc[1] = -2.0 * a / (b * c * e.N);
    sc[2] = a / b;
  } else {
    sc[0] = 1.0;
    sc[1] = c > 0.0 ? -1.0 / (c * e.N) : 0.0;
    sc[2] = 0.0;
  }
  sc[3] = 0.0;
}

__global__ void k_energy_grad(EnergyBatch e, float* __restrict__ gy) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  const long vol = (long)e.Dp * e.Hp * e.Wp;
  if (i >= (long)e.N * 3 * vol) return;
  const Grid& g = e.g;
  const int n = (int)(i / (3 * vol)), c = (int)((i / vol) % 3);
  const long v = i % vol;
  const int x = (int)(v % e.Wp), yy = (int)((v / e.Wp) % e.Hp), z = (int)(v / ((long)e.Wp * e.Hp));
  double val = 0.0;
  if (x < g.Nx && yy < g.Ny && z < g.Nz) {
    const int node = x + g.Nx * (yy + g.Ny * z);
    if (!((e.fixn[node] >> c) & 1u)) {
      const size_t d = (size_t)n * g.n + 3 * (size_t)node + c;
      const double* sc = e.scal + 4 * (size_t)n;
      val = sc[1] * (e.f[d] - sc[2] * e.Ku[d]);
    }
  }
  gy[i] = (float)val;
}

void launch_energy_loss(const EnergyBatch& e, const float* y, float* gy, hipStream_t s) {
  k_energy_u<<<div_up((long)e.N * e.g.Nn, 256), 256, 0, s>>>(e, y);
  k_energy_Ku<<<dim3(e.nb, e.N), 256, 0, s>>>(e);
  k_energy_final<<<e.N, 256, 0, s>>>(e);
  k_energy_grad<<<div_up((long)e.N * 3 * e.Dp * e.Hp * e.Wp, 256), 256, 0, s>>>(e, gy);
}

// All layers' weights and biases (or their gradients) in the order of the C
// ABI, per layer w[co][ci][tap] then b[co], from the device layout
// w[(ci * K3 + tap) * Cop + co].
__global__ void k_export_params(ParamTable t, float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= t.off[ParamTable::kLayers]) return;
  int l = 0;
  while (i >= t.off[l + 1]) ++l;
  const int j = i - t.off[l], nw = t.co[l] * t.ci[l] * t.k3[l];
  if (j >= nw) {
    out[i] = t.b[l][j - nw];
    return;
  }
  const int tap = j % t.k3[l], ci = (j / t.k3[l]) % t.ci[l], co = j / (t.k3[l] * t.ci[l]);
  out[i] = t.w[l][((size_t)ci * t.k3[l] + tap) * t.cop[l] + co];
}

void launch_export_params(const ParamTable& t, float* out, hipStream_t s) {
  k_export_params<<<div_up(t.off[ParamTable::kLayers], 256), 256, 0, s>>>(t, out);
}

// x0 = alpha u0 with alpha = (f . u0) / (u0 . K u0) (sums[0], sums[1]).
__global__ void k_scale_by_ratio(double* __restrict__ u, int n, const double* __restrict__ num,
                                 const double* __restrict__ den, double* __restrict__ alpha_out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  const double a = *den > 0.0 ? *num / *den : 0.0;
  if (i == 0 && alpha_out) *alpha_out = a;
  if (i < n) u[i] *= a;
}

void launch_scale_by_ratio(double* u, int n, const double* num, const double* den, double* alpha,
                           hipStream_t s) {
  k_scale_by_ratio<<<div_up(n, 256), 256, 0, s>>>(u, n, num, den, alpha);
}

}  // namespace sgmg
