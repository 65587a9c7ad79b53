// Coarsest level (Sec. 3.2, Sec. 4.1): dense K_L + eps I on the free DOFs,
// explicit inverse by a blocked in-place Gauss-Jordan sweep (no pivoting:
// the matrix is SPD), and the per-cycle solve as a gather-GEMV-scatter.
#include "kernels.hpp"

namespace sgmg {

constexpr int kNB = 64;       // pivot block width

// One matrix row per blockIdx.x.  Columns further away than one stencil reach
// in DOF order are zeros, decided before any index is split.
__global__ __launch_bounds__(256) void k_dense_assemble(Grid g, const double* __restrict__ S,
                                                        const int* __restrict__ free_idx, int nf,
                                                        int ld, double* __restrict__ A) {
  const int i = blockIdx.x;
  const int j = blockIdx.y * 256 + threadIdx.x;
  if (j >= nf) return;
  const int di = free_idx[i], dj = free_idx[j];
  const int ni = di / 3, d = di % 3, reach = 1 + g.Nx + g.Nx * g.Ny;
  const int nj = dj / 3, e = dj - 3 * nj;
  double v = 0.0;
  if (nj - ni <= reach && ni - nj <= reach) {
    const int ix = ni % g.Nx, iy = (ni / g.Nx) % g.Ny, iz = ni / (g.Nx * g.Ny);
    const int jx = nj % g.Nx, jy = (nj / g.Nx) % g.Ny, jz = nj / (g.Nx * g.Ny);
    const int ox = jx - ix, oy = jy - iy, oz = jz - iz;
    if (ox >= -1 && ox <= 1 && oy >= -1 && oy <= 1 && oz >= -1 && oz <= 1) {
      const int o = (ox + 1) + 3 * (oy + 1) + 9 * (oz + 1);
      v = S[(size_t)(o * 9 + 3 * d + e) * g.Nn + ni];
    }
  }
  A[(size_t)i * ld + j] = v;
}

void launch_dense_assemble(const Grid& g, const double* S, const int* free_idx, int nf, int ld, double* A,
                           hipStream_t s) {
  k_dense_assemble<<<dim3(nf, div_up(nf, 256)), 256, 0, s>>>(g, S, free_idx, nf, ld, A);
}

__global__ void k_dense_diag_sum(const double* __restrict__ A, int nf, int ld, RedWs ws, double* out) {
  double s = 0.0;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nf; i += gridDim.x * blockDim.x)
    s += A[(size_t)i * ld + i];
  const double v[1] = {s};
  grid_sum<1>(v, ws);
}

void launch_dense_diag_sum(const double* A, int nf, int ld, RedWs ws, double* out, hipStream_t s) {
  k_dense_diag_sum<<<1, 256, 0, s>>>(A, nf, ld, ws, out);
  launch_finalize(ws, 1, 1, out, s);
}

// eps = max(mean diag * 1e-8, 1e-14) added to the diagonal (Sec. 4.1).
__global__ void k_dense_add_diag(double* __restrict__ A, int nf, int ld, const double* __restrict__ dsum,
                                 double* __restrict__ eps_out) {
  const double eps = fmax(*dsum / nf * 1e-8, 1e-14);
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0 && eps_out) *eps_out = eps;
  if (i < nf) A[(size_t)i * ld + i] += eps;
}

void launch_dense_add_diag(double* A, int nf, int ld, const double* mean_diag_sum, hipStream_t s,
                           double* eps_out) {
  k_dense_add_diag<<<div_up(nf, 256), 256, 0, s>>>(A, nf, ld, mean_diag_sum, eps_out);
}

// --- blocked Gauss-Jordan sweep --------------------------------------------
// For pivot block K: Q = A_KK^-1; A_KJ <- Q A_KJ (J != K);
// A_IJ <- A_IJ - A_IK(old) A_KJ(new) (I, J != K); A_IK <- -A_IK(old) Q.
// After all blocks A holds its inverse.
//
// The pivots form one serial chain, so a pivot block's own update and its
// inversion run in the first block of the launch that updates the rest of
// the matrix, and two pivot blocks share one pass over it:
//   panel(K)        : the row and the column of block K, and both rewritten
//                     in matrix-core operand order (R = A_KJ, C = A_IK old)
//   update, K alone : row and column K + 1 only; inverts pivot K + 1
//   panel(K + 1)
//   update, both    : A_IJ - C_K R_K - C_{K+1} R_{K+1} for everything else,
//                     one read and one write of A; inverts pivot K + 2
// Every element sees the same operations in the same order as with one full
// update per block, so the split changes no bit of the result.
// Measured per two pivot blocks at n = 3630: panels 10 + 11 us, cross 25 us (the
// pivot's chain), the pass over A 76 us (46 us of matrix-core work beside 43 us
// of copy rate); whole inverse 7.5 -> 3.55 ms. One launch each for column copy, pivot, row panel and update of a
// single block took 131 us per block. n = 1944: 2.7 -> 1.15 ms, n = 1344: 1.67 ->
// 0.75 ms, both bound by the chain of pivots (25 us each with its tile).
//
// FP64 matrix-core operand layouts (v_mfma_f64_16x16x4_f64): A lane l = (row
// l % 16, k l / 16), B lane l = (k l / 16, column l % 16), result register i
// of lane l = (row 4 i + l / 16, column l % 16).  The operands of 16 rows (or
// columns) for two k-steps of 4 are 64 consecutive pairs of doubles, in lane
// order, so they are one coalesced 16-byte load and the update needs no LDS
// (8-byte loads kept the address units busier than the matrix cores): element
// (16-row group g, k-step t, lane l) of a panel is at
// ((8 g + t / 2) * 64 + l) * 2 + t % 2.
typedef double f64x4_gj __attribute__((ext_vector_type(4)));
constexpr int kLdP = 68;       // LDS pitch (doubles): 8 rows x 4 k of a wave in distinct banks


// The row panel (blocks 0 .. nb - 1, J) and the column panel (blocks nb ..
// 2 nb - 1, I) of pivot block K.  Q: its inverse, 64 x 64, zero past nbw
// (the block's width).  CF of row block K and RF of column block K are zeros,
// so an update with them leaves row and column K as they are.
__global__ __launch_bounds__(256) void k_gj_panel(double* __restrict__ A, int n, int ld, int nb, int K,
                                                  const double* __restrict__ Q,
                                                  double* __restrict__ CF,
                                                  double* __restrict__ RF) {
  __shared__ double Qs[kNB][kLdP];
  __shared__ double Vs[kNB][kLdP];
  const bool row = (int)blockIdx.x < nb;
  const int B = row ? blockIdx.x : blockIdx.x - nb;
  const int k0 = K * kNB, b0 = B * kNB, nbw = min(kNB, n - k0);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  double* F = (row ? RF : CF) + (size_t)B * kNB * kNB;
  if (B == K) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int e = tid + 256 * u, r = e / kNB, c = e % kNB;
      F[e] = 0.0;
      if (row && r < nbw && c < nbw) A[(size_t)(k0 + r) * ld + k0 + c] = Q[e];
    }
    return;
  }
  double2* F2 = (double2*)F + 512 * w + lane;      // the wave's group of 16 rows or columns
  const int r0 = row ? k0 : b0, c0 = row ? b0 : k0;
  double qv[16], vv[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int e = tid + 256 * u, r = e / kNB, c = e % kNB;
    qv[u] = Q[e];
    vv[u] = A[(size_t)min(r0 + r, n - 1) * ld + min(c0 + c, n - 1)];
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int e = tid + 256 * u, r = e / kNB, c = e % kNB;
    if (row) Qs[c][r] = qv[u];                     // transposed: a thread's rows are adjacent
    else Qs[r][c] = -qv[u];
    Vs[r][c] = r0 + r < n && c0 + c < n ? vv[u] : 0.0;
  }
  __syncthreads();
  if (row) {
    // a 4 x 4 register tile per thread (rows 2 tr + {0, 1, 32, 33}, columns
    // 2 tc + {0, 1, 32, 33}: 16-byte LDS reads), the 64 products in order
    const int tr = tid / 16, tc = tid % 16;
    double acc[4][4] = {};
#pragma unroll 4
    for (int t = 0; t < kNB; ++t) {
      double a[4], b[4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double2 x = *(const double2*)&Qs[t][2 * tr + 32 * h];
        const double2 y = *(const double2*)&Vs[t][2 * tc + 32 * h];
        a[2 * h] = x.x; a[2 * h + 1] = x.y;
        b[2 * h] = y.x; b[2 * h + 1] = y.y;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < 4; ++p) acc[q][p] = __builtin_fma(a[q], b[p], acc[q][p]);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *(double2*)&Vs[2 * tr + 32 * (q / 2) + q % 2][2 * tc + 32 * h] =
            make_double2(acc[q][2 * h], acc[q][2 * h + 1]);
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 8; ++t)
      F2[64 * t] = make_double2(Vs[8 * t + lk][16 * w + lr], Vs[8 * t + 4 + lk][16 * w + lr]);
  } else {
    f64x4_gj acc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = f64x4_gj{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int t = 0; t < 16; t += 2) {
      const double2 a = make_double2(Vs[16 * w + lr][4 * t + lk], Vs[16 * w + lr][4 * t + 4 + lk]);
      F2[32 * t] = a;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, Qs[4 * t + lk][16 * q + lr], acc[q], 0, 0, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, Qs[4 * t + 4 + lk][16 * q + lr], acc[q], 0, 0, 0);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) Vs[16 * w + 4 * i + lk][16 * q + lr] = acc[q][i];
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    const int e = tid + 256 * u, r = e / kNB, c = e % kNB;
    if (r0 + r < n && c0 + c < n) A[(size_t)(r0 + r) * ld + c0 + c] = Vs[r][c];
  }
}

template <int NW>
struct PivotLds {
  double P[kNB][kNB + 1];
  double g[2][kNB / NW][kNB];  // 1 / a_pp in lane p, -a_rp / a_pp elsewhere, by parity
};

// Inverse of the 64 x 64 block S.P by in-place Gauss-Jordan (SPD: no
// pivoting), NW waves: lane r of wave w keeps the CW = 64 / NW columns CW w .. of
// row r.  Pivot p:
//   r == p : a_pc <- a_pc / a_pp (c != p),  a_pp <- 1 / a_pp
//   r != p : a_rc <- a_rc - (a_rp / a_pp) a_pc (c != p),  a_rp <- -a_rp / a_pp
// The wave that owns CW pivot columns runs their CW steps alone (row p
// reaches the lanes through scalar registers), publishes the multipliers,
// and after one barrier the other waves apply these steps to their own
// columns in the same order; the next owner goes on with its own steps while
// the others still apply.  Bound: the owners' chain, a division and the
// columns of one wave per pivot: 22 us with 16 waves and four columns each,
// taken where nothing hides it.
// Writes Q, zero past nbw.
template <int NW>
__device__ inline void gj_pivot(PivotLds<NW>& S, int nbw, double* __restrict__ Q, int* __restrict__ flag) {
  const int r = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int CW = kNB / NW;
  __syncthreads();
  double v[CW];
#pragma unroll
  for (int c = 0; c < CW; ++c) v[c] = S.P[r][CW * w + c];
  bool bad = false;
  for (int b = 0; b < NW; ++b) {
    const int buf = b & 1;
    if (w == b) {
#pragma unroll
      for (int sp = 0; sp < CW; ++sp) {
        const int p = CW * b + sp;
        const double pv = lane_value(v[sp], p);
        bad |= !(pv > 0.0);
        const double inv = 1.0 / pv;
        const bool me = r == p;
        const double g = v[sp] * inv;            // a_rp / a_pp
        const double f = me ? inv : -g;
#pragma unroll
        for (int c = 0; c < CW; ++c) {
          if (c == sp) continue;
          v[c] = __builtin_fma(f, lane_value(v[c], p), me ? 0.0 : v[c]);
        }
        v[sp] = f;
        S.g[buf][sp][r] = f;
      }
    }
    __syncthreads();
    if (w != b) {
#pragma unroll
      for (int sp = 0; sp < CW; ++sp) {
        const int p = CW * b + sp;
        const bool me = r == p;
        const double f = S.g[buf][sp][r];
#pragma unroll
        for (int c = 0; c < CW; ++c)
          v[c] = __builtin_fma(f, lane_value(v[c], p), me ? 0.0 : v[c]);
      }
    }
  }
  if (bad && r == 0) *flag = 1;
#pragma unroll
  for (int c = 0; c < CW; ++c) S.P[r][CW * w + c] = v[c];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < kNB / NW; ++u) {
    const int e = threadIdx.x + 64 * NW * u, a = e / kNB, c = e % kNB;
    Q[e] = a < nbw && c < nbw ? S.P[a][c] : 0.0;
  }
}

// acc[NR][NC] = C R over one panel for 16 NR rows and 16 NC columns, the k
// steps in order.
template <int NR, int NC>
__device__ inline void gj_product(const double2* __restrict__ c, const double2* __restrict__ r,
                                  f64x4_gj (&acc)[NR][NC]) {
#pragma unroll
  for (int q = 0; q < NR; ++q)
#pragma unroll
    for (int p = 0; p < NC; ++p) acc[q][p] = f64x4_gj{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
  for (int t = 0; t < 8; ++t) {
    double2 a[NR], b[NC];
#pragma unroll
    for (int q = 0; q < NR; ++q) a[q] = c[q * 512 + t * 64];
#pragma unroll
    for (int p = 0; p < NC; ++p) b[p] = r[p * 512 + t * 64];
#pragma unroll
    for (int q = 0; q < NR; ++q)
#pragma unroll
      for (int p = 0; p < NC; ++p)
        acc[q][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].x, b[p].x, acc[q][p], 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NR; ++q)
#pragma unroll
      for (int p = 0; p < NC; ++p)
        acc[q][p] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[q].y, b[p].y, acc[q][p], 0, 0, 0);
  }
}

// A wave's tile: rows i0 .., columns j0 .. : old - C_0 R_0 (- C_1 R_1).
template <int NR, int NC, class Out>
__device__ inline void gj_tile(const double* __restrict__ A, int n, int ld, int i0, int j0, int panels,
                               const double* __restrict__ CF, const double* __restrict__ RF,
                               size_t panel_stride, Out&& out) {
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  double v[NR][NC][4];
#pragma unroll
  for (int q = 0; q < NR; ++q)
#pragma unroll
    for (int p = 0; p < NC; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int a = i0 + 16 * q + 4 * i + lk, b = j0 + 16 * p + lr;
        v[q][p][i] = A[(size_t)min(a, n - 1) * ld + min(b, n - 1)];
      }
  for (int m = 0; m < panels; ++m) {
    f64x4_gj acc[NR][NC];
    gj_product<NR, NC>((const double2*)(CF + m * panel_stride + (size_t)(i0 >> 4) * 1024) + lane,
                       (const double2*)(RF + m * panel_stride + (size_t)(j0 >> 4) * 1024) + lane, acc);
#pragma unroll
    for (int q = 0; q < NR; ++q)
#pragma unroll
      for (int p = 0; p < NC; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[q][p][i] -= acc[q][p][i];
  }
#pragma unroll
  for (int q = 0; q < NR; ++q)
#pragma unroll
    for (int p = 0; p < NC; ++p)
#pragma unroll
      for (int i = 0; i < 4; ++i) out(i0 + 16 * q + 4 * i + lk, j0 + 16 * p + lr, v[q][p][i]);
}

// Update by the last `panels` panels (K, or K - 1 and K), 32 x 32 per wave.
// cross: only row and column K + 1, blocks 1 .. nj the row's tiles and nj + 1 ..
// 2 nj the column's; otherwise every tile outside row and column K.  Block 0
// forms and inverts pivot block K + 1 (left out of the tiles).  NW = 16: tiles
// of 128 x 128.  NW = 8: 128 x 64, so two blocks share a compute unit and one
// loads while the other multiplies, and the last round of blocks is a smaller
// part of the launch (see dense_spd_inverse).
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_gj_update(double* __restrict__ A, int n, int ld, int nb,
                                                       int K, int panels, int cross,
                                                       const double* __restrict__ CF,
                                                       const double* __restrict__ RF,
                                                       size_t panel_stride, double* __restrict__ Q,
                                                       int* __restrict__ flag) {
  constexpr int WC = NW / 4;                       // waves along the columns
  __shared__ PivotLds<NW> S;
  const int w = threadIdx.x >> 6;
  if (blockIdx.x == 0) {
    if (K + 1 >= nb) return;
    const int k1 = (K + 1) * kNB;
    for (int q = w; q < 16; q += NW)
      gj_tile<1, 1>(A, n, ld, k1 + 16 * (q >> 2), k1 + 16 * (q & 3), panels, CF, RF, panel_stride,
                    [&](int a, int b, double v) {
                      S.P[a - k1][b - k1] = a < n && b < n ? v : (a == b ? 1.0 : 0.0);
                    });
    gj_pivot<NW>(S, min(kNB, n - k1), Q, flag);
    return;
  }
  const int nj = (nb + 1) / 2, t = blockIdx.x - 1, mid = (K + 1) / 2;
  int Ip, Jp;
  if (!cross) {
    // each XCD's share is about one band of four tile rows, column by column:
    // its L2 keeps the band's C and streams R (all of both is 7.4 MB at n =
    // 3630, more than the 4 MB an XCD has)
    const int nc = NW == 16 ? nj : nb;             // tile columns
    const int u = xcd_block(t, nj * nc), band = u / (4 * nc), in = u - band * 4 * nc;
    const int rows = min(4, nj - 4 * band);
    Ip = 4 * band + in % rows;
    Jp = in / rows;
  } else {
    Ip = t < nj ? mid : t - nj;
    Jp = t < nj ? t : mid;
    if (t >= nj && Ip == mid) return;              // among the row's tiles
  }
  const int i0 = 128 * Ip + 32 * (w / WC), j0 = 32 * WC * Jp + 32 * (w % WC);
  const int I = i0 / kNB, J = j0 / kNB;
  if (I >= nb || J >= nb || I == K || J == K || (I == K + 1 && J == K + 1)) return;
  if (cross && I != K + 1 && J != K + 1) return;
  gj_tile<2, 2>(A, n, ld, i0, j0, panels, CF, RF, panel_stride,
                [&](int a, int b, double v) {
                  if (a < n && b < n) A[(size_t)a * ld + b] = v;
                });
}

size_t dense_inverse_scratch(int n) {
  return (4 * (size_t)div_up(n, kNB) + 1) * kNB * kNB;
}

int dense_spd_inverse(double* A, int n, int ld, double* scratch, int* d_flag, hipStream_t s) {
  const int nb = div_up(n, kNB), nj = (nb + 1) / 2;
  const size_t ps = 2 * (size_t)nb * kNB * kNB;      // two panels, C and R each
  double* CF = scratch;
  double* RF = scratch + (size_t)nb * kNB * kNB;
  double* Q = scratch + 2 * ps;
  auto panel = [&](int K, int m) {
    k_gj_panel<<<2 * nb, 256, 0, s>>>(A, n, ld, nb, K, Q, CF + m * ps, RF + m * ps);
  };
  auto update = [&](int K, int panels, int cross, int blocks) {
    k_gj_update<16><<<1 + blocks, 1024, 0, s>>>(A, n, ld, nb, K, panels, cross, CF, RF, ps, Q, d_flag);
  };
  auto cross = [&](int K, int panels, int blocks) { update(K, panels, 1, blocks); };
  // Up to one tile of 128 x 128 per compute unit the launch lasts as long as
  // its pivot, which sixteen waves invert fastest (n = 1944: 29 us, with eight
  // 39 us); beyond that the tiles hide the pivot (n = 3630: 84 us with 128 x
  // 128, 76 us with 128 x 64).
  auto full = [&](int K, int panels) {
    if (nj * nj <= 256)
      update(K, panels, 0, nj * nj);
    else
      k_gj_update<8><<<1 + nj * nb, 512, 0, s>>>(A, n, ld, nb, K, panels, 0, CF, RF, ps, Q, d_flag);
  };
  cross(-1, 0, 0);                                   // pivot block 0
  for (int K = 0; K < nb; K += 2) {
    panel(K, 0);
    if (K + 1 < nb) {
      cross(K, 1, 2 * nj);
      panel(K + 1, 1);
      full(K + 1, 2);
    } else if (nb > 1) {
      full(K, 1);
    }
  }
  return 0;
}

// ---------------------------------------------------------------------------
// Symmetric form of the coarsest solve.  The explicit inverse of the SPD
// matrix K_L + eps I is symmetric, so only its upper triangle is read per
// cycle: it is packed once per factorisation into 64 x 64 tiles (I, J),
// I <= J, tile t(I, J) = I nb - I (I - 1) / 2 + (J - I), each tile row-major
// and zero-padded past nf.  A cycle reads every stored coefficient once:
//   pass 1, one workgroup per tile: row sums A_IJ x_J (towards y_I) and, off
//           the diagonal, column sums A_IJ^T x_I (towards y_J), written as
//           per-tile partials;
//   pass 2, per output block I: y_I = the sum over J of the column partial
//           of tile (J, I) for J < I and the row partial of tile (I, J) for
//           J >= I, in a fixed order.
// x is gathered through the free-DOF list inside pass 1, and y is scattered
// by pass 2, so no separate gather launch remains.  Fixed summation order:
// deterministic.
constexpr int kTile = 64;

int sym_tiles(int nf) {
  const int nb = div_up(nf, kTile);
  return nb * (nb + 1) / 2;
}

__device__ inline int tile_index(int I, int J, int nb) { return I * nb - I * (I - 1) / 2 + (J - I); }

// Inverse of tile_index: the block row from the quadratic's root, corrected
// by at most a step either way against rounding.
__device__ inline void tile_ij(int t, int nb, int& I, int& J) {
  const double b = 2.0 * nb + 1.0;
  int i = (int)((b - sqrt(b * b - 8.0 * t)) * 0.5);
  i = max(0, min(i, nb - 1));
  while (i > 0 && tile_index(i, i, nb) > t) --i;
  while (i + 1 < nb && tile_index(i + 1, i + 1, nb) <= t) ++i;
  I = i;
  J = i + (t - tile_index(i, i, nb));
}

__global__ __launch_bounds__(256) void k_dense_pack(const double* __restrict__ A, int nf, int ld, int nb,
                                                   double* __restrict__ P) {
  int I, J;
  tile_ij(blockIdx.x, nb, I, J);
  double* T = P + (size_t)blockIdx.x * kTile * kTile;
  for (int e = threadIdx.x; e < kTile * kTile; e += 256) {
    const int a = e / kTile, b = e % kTile;
    const int i = I * kTile + a, j = J * kTile + b;
    T[e] = (i < nf && j < nf) ? A[(size_t)i * ld + j] : 0.0;
  }
}

__global__ __launch_bounds__(256) void k_dense_symv_tiles(const double* __restrict__ P, int nf,
                                                         int nb, const int* __restrict__ free_idx,
                                                         const double* __restrict__ r,
                                                         double* __restrict__ prow,
                                                         double* __restrict__ pcol) {
  __shared__ double tile[kTile][kTile + 1];
  __shared__ double xs[2][kTile];
  __shared__ double red[4][kTile];
  const int t = blockIdx.x;
  int I, J;
  tile_ij(t, nb, I, J);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const double* T = P + (size_t)t * kTile * kTile;
  double v[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = T[(w + 4 * k) * kTile + lane];
  if (w < 2) {
    const int i = (w == 0 ? I : J) * kTile + lane;
    xs[w][lane] = i < nf ? r[free_idx[i]] : 0.0;
  }
  __syncthreads();
  // column partial over this wave's 16 rows (towards y_J)
  double pc = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    pc += v[k] * xs[0][w + 4 * k];
    tile[w + 4 * k][lane] = v[k];
  }
  red[w][lane] = pc;
  __syncthreads();
  if (w == 0 && I != J)
    pcol[(size_t)t * kTile + lane] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
  __syncthreads();
  // row partial: lane = row, this wave's 16 columns (towards y_I)
  double pr = 0.0;
#pragma unroll
  for (int k = 0; k < 16; ++k) pr += tile[lane][16 * w + k] * xs[1][16 * w + k];
  red[w][lane] = pr;
  __syncthreads();
  if (w == 0)
    prow[(size_t)t * kTile + lane] = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
}

// One block of 4 waves per output block I: wave w adds the partials of
// J = w, w + 4, ... (tile indices in closed form, loads independent), then
// the four wave sums are added in a fixed order.
__global__ __launch_bounds__(256) void k_dense_symv_sum(int nf, int nb,
                                                       const int* __restrict__ free_idx,
                                                       const double* __restrict__ prow,
                                                       const double* __restrict__ pcol,
                                                       double* __restrict__ z) {
  __shared__ double red[4][kTile];
  const int I = blockIdx.x, a = threadIdx.x & 63, w = threadIdx.x >> 6;
  double y0 = 0.0, y1 = 0.0;
  int J = w;
  for (; J + 4 < nb; J += 8) {
    const int J1 = J + 4;
    y0 += J < I ? pcol[(size_t)tile_index(J, I, nb) * kTile + a]
                : prow[(size_t)tile_index(I, J, nb) * kTile + a];
    y1 += J1 < I ? pcol[(size_t)tile_index(J1, I, nb) * kTile + a]
                 : prow[(size_t)tile_index(I, J1, nb) * kTile + a];
  }
  if (J < nb)
    y0 += J < I ? pcol[(size_t)tile_index(J, I, nb) * kTile + a]
                : prow[(size_t)tile_index(I, J, nb) * kTile + a];
  red[w][a] = y0 + y1;
  __syncthreads();
  if (w == 0) {
    const int i = I * kTile + a;
    if (i < nf) z[free_idx[i]] = (red[0][a] + red[1][a]) + (red[2][a] + red[3][a]);
  }
}

void launch_dense_pack(const double* A, int nf, int ld, double* P, hipStream_t s) {
  if (nf <= 0) return;
  k_dense_pack<<<sym_tiles(nf), 256, 0, s>>>(A, nf, ld, div_up(nf, kTile), P);
}

void launch_dense_symv(const double* P, const int* free_idx, int nf, const double* r,
                       double* partials, double* z, hipStream_t s) {
  if (nf <= 0) return;
  const int nb = div_up(nf, kTile), nt = sym_tiles(nf);
  double* prow = partials;
  double* pcol = partials + (size_t)nt * kTile;
  k_dense_symv_tiles<<<nt, 256, 0, s>>>(P, nf, nb, free_idx, r, prow, pcol);
  k_dense_symv_sum<<<nb, 256, 0, s>>>(nf, nb, free_idx, prow, pcol, z);
}

}  // namespace sgmg
