// gfx950 kernels of the learned warm start: per-cell frame and features, network
// inference and training (forward, loss, backward, gradient reduction, Adam).
//
// One workgroup carries one cell at a time; node-wise products with the 64 x 64 (or 64 x
// 128) weight blocks run on the matrix cores (v_mfma_f32_16x16x32_bf16).  Meshes of up to
// 768 rows run with their activations resident in LDS (net_resident_kernel, and for training
// net_chain_kernel and net_wgrad_kernel); larger ones gather from memory
// (net_forward_kernel, net_backward_kernel).  Every partial gradient sum goes to its own slot
// and the slots are reduced in a fixed order, so training is deterministic.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "npfem_internal.h"
#include "npfem_net_internal.h"

namespace npfem {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kRS = 16;     // reduction stride (values per wave)
constexpr int kTP = 40;     // LDS row pitch (BF16) of the transposed 32-node chunks
constexpr int kNetUnrollDeg = 6;   // neighbour gathers issued together (the icosphere degree)

__device__ inline int tid() { return threadIdx.x; }

__device__ inline float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ inline uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ inline bf16x8 ld8(const uint16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }
__device__ inline bf16x8 zero8() {
  const __bf16 z = (__bf16)0.f;
  return bf16x8{z, z, z, z, z, z, z, z};
}

template <int N>
__device__ inline void wg_sum(double (&v)[N], double* red) {
  static_assert(N <= kRS, "wg_sum: too many values");
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double x = v[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    v[i] = x;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) red[wave * kRS + i] = v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) t += red[w * kRS + i];
    v[i] = t;
  }
}

// Orthogonal polar factor of a 3x3 matrix with positive determinant (scaled Newton
// iteration X <- (g X + X^-T / g) / 2, g = (|X^-1|_F / |X|_F)^(1/2); Higham 1986).
// This is the Kabsch rotation: C = U S V^T -> U V^T.  Identity for det <= 0.
__device__ void polar3(const double* C, double* R) {
  double X[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) X[k] = C[k];
  const double d0 = X[0] * (X[4] * X[8] - X[5] * X[7]) - X[1] * (X[3] * X[8] - X[5] * X[6]) +
                    X[2] * (X[3] * X[7] - X[4] * X[6]);
  if (!(d0 > 0.0) || !isfinite(d0)) {
#pragma unroll
    for (int k = 0; k < 9; ++k) R[k] = (k % 4 == 0) ? 1.0 : 0.0;
    return;
  }
  for (int it = 0; it < 60; ++it) {
    double cof[9];
    cof[0] = X[4] * X[8] - X[5] * X[7];
    cof[1] = X[5] * X[6] - X[3] * X[8];
    cof[2] = X[3] * X[7] - X[4] * X[6];
    cof[3] = X[2] * X[7] - X[1] * X[8];
    cof[4] = X[0] * X[8] - X[2] * X[6];
    cof[5] = X[1] * X[6] - X[0] * X[7];
    cof[6] = X[1] * X[5] - X[2] * X[4];
    cof[7] = X[2] * X[3] - X[0] * X[5];
    cof[8] = X[0] * X[4] - X[1] * X[3];
    const double d = X[0] * cof[0] + X[1] * cof[1] + X[2] * cof[2];
    const double id = 1.0 / d;
    double nx = 0.0, nc = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      nx += X[k] * X[k];
      nc += cof[k] * cof[k];
    }
    const double g = sqrt(sqrt(nc * id * id / nx));          // (|X^-1|_F / |X|_F)^(1/2)
    const double cg = 0.5 * id / g, xg = 0.5 * g;
    double diff = 0.0;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double xn = xg * X[k] + cg * cof[k];
      diff += (xn - X[k]) * (xn - X[k]);
      X[k] = xn;
    }
    if (diff <= 1e-30) break;
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = X[k];
}

// ---------------------------------------------------------------------------------
// Forward: frame, features, encoder, message-passing layers, decoder.
// ---------------------------------------------------------------------------------

// Frame (mass-weighted centroids, covariance with the rest shape, Kabsch) and the node
// features of cell k, written as BF16 rows of 32 (zero padded) to feat.  Leaves R and
// s in fr[0..9] (LDS) and ends with a barrier.
template <typename Real>
__device__ void cell_features(const NetFwdArgs<Real>& A, const NetMeshDev& M, int k, const Real* x, const Real* v,
                              const Real* f, uint16_t* feat, double* red, double* fr) {
  const int n = M.n, np = M.n_pad;
  double s1[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = tid(); i < n; i += kBlock) {
    const double m = M.mass[i];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      s1[c] += m * (double)x[3 * i + c];
      s1[3 + c] += m * (double)v[3 * i + c];
      s1[6 + c] += (double)f[3 * i + c];
    }
  }
  wg_sum<9>(s1, red);
  const double ims = 1.0 / M.mass_sum;
  const double xc[3] = {s1[0] * ims, s1[1] * ims, s1[2] * ims};
  const double vc[3] = {s1[3] * ims, s1[4] * ims, s1[5] * ims};
  const double ac[3] = {s1[6] * ims, s1[7] * ims, s1[8] * ims};
  double s2[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = tid(); i < n; i += kBlock) {
    const double m = M.mass[i];
    double d[3], fd[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      d[c] = (double)x[3 * i + c] - xc[c];
      fd[c] = (double)f[3 * i + c] - m * ac[c];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) s2[3 * a + b] += m * d[a] * M.Xc[3 * i + b];
    s2[9] += fd[0] * fd[0] + fd[1] * fd[1] + fd[2] * fd[2];
  }
  wg_sum<10>(s2, red);
  if (tid() == 0) {
    double R[9];
    polar3(s2, R);
    const double s = A.h * A.h * (sqrt(s2[9] / n) + A.W.force_floor) / M.mass_mean;
#pragma unroll
    for (int q = 0; q < 9; ++q) fr[q] = R[q];
    fr[9] = s;
    if (A.S.frame) {
#pragma unroll
      for (int q = 0; q < 10; ++q) A.S.frame[(size_t)k * kNetFrame + q] = fr[q];
    }
  }
  __syncthreads();
  double R[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) R[q] = fr[q];
  const double s = fr[9];
  const double hs = A.h / s, h2s = A.h * A.h / s, iq = 1.0 / A.W.shape_scale;
  for (int i = tid(); i < np; i += kBlock) {
    float fv[kNetFeat];
#pragma unroll
    for (int q = 0; q < kNetFeat; ++q) fv[q] = 0.f;
    if (i < n) {
      const double m = M.mass[i];
      double d[3], dv[3], df[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        d[c] = (double)x[3 * i + c] - xc[c];
        dv[c] = (double)v[3 * i + c] - vc[c];
        df[c] = (double)f[3 * i + c] - m * ac[c];
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        double rd = 0.0, rv = 0.0, rf = 0.0;                 // (R^T w)_a = sum_b R[b][a] w_b
#pragma unroll
        for (int b = 0; b < 3; ++b) {
          rd += R[3 * b + a] * d[b];
          rv += R[3 * b + a] * dv[b];
          rf += R[3 * b + a] * df[b];
        }
        const double Xa = M.Xc[3 * i + a];
        fv[a] = (float)((rd - Xa) * iq);
        fv[3 + a] = (float)(rv * hs);
        fv[6 + a] = (float)(rf * h2s / m);
        fv[9 + a] = (float)(Xa * M.inv_rho);
      }
    }
    bf16x8 w0, w1;
#pragma unroll
    for (int e = 0; e < 8; ++e) w0[e] = (__bf16)fv[e];
#pragma unroll
    for (int e = 0; e < 8; ++e) w1[e] = (__bf16)(e < 4 ? fv[8 + e] : 0.f);
    uint16_t* fp = feat + (size_t)i * kNetFeatPad;
    *reinterpret_cast<bf16x8*>(fp) = w0;
    *reinterpret_cast<bf16x8*>(fp + 8) = w1;
    *reinterpret_cast<bf16x8*>(fp + 16) = zero8();
    *reinterpret_cast<bf16x8*>(fp + 24) = zero8();
  }
  __syncthreads();
}

// Encoder rows of this wave: h0 = relu(W_e f + b_e) into H; training also stores z0 to Z.
__device__ void encoder_rows(const NetWeights& W, const uint16_t* feat, int n, int np, uint16_t* H,
                             uint16_t* Z) {
  const int lane = tid() & 63, wave = tid() >> 6, l16 = lane & 15, kq = lane >> 4;
  bf16x8 bq[4];
  float bias[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    bq[cb] = ld8(W.We + (size_t)(cb * 16 + l16) * kNetFeatPad + 8 * kq);
    bias[cb] = W.theta[W.lay.off_be + cb * 16 + l16];
  }
  for (int rb = wave; rb < (np >> 4); rb += kBlock / 64) {
    const bf16x8 aq = ld8(feat + (size_t)(rb * 16 + l16) * kNetFeatPad + 8 * kq);
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const floatx4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, bq[cb], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = rb * 16 + 4 * kq + i, col = cb * 16 + l16;
        const float z = row < n ? acc[i] + bias[cb] : 0.f;
        H[(size_t)row * kNetH + col] = f2bf(fmaxf(z, 0.f));
        if (Z) Z[(size_t)row * kNetH + col] = f2bf(z);
      }
    }
  }
}

// Decoder on the matrix cores: o = W_d h + b_d (3 outputs padded to one 16-column
// block); lanes l16 = 0, 1, 2 of each 16-lane group hold the components of a row and
// exchange them to form the correction s R o (world frame) and/or store o.
template <typename Real>
__device__ void decoder_rows(const NetFwdArgs<Real>& A, int k, int64_t voff, int n, int np, const uint16_t* H,
                             const double* fr) {
  const int lane = tid() & 63, wave = tid() >> 6, l16 = lane & 15, kq = lane >> 4;
  double R[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) R[q] = fr[q];
  const double s = fr[9];
  bf16x8 bq[2];
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2) bq[s2] = l16 < 3 ? ld8(A.W.Wd + (size_t)l16 * kNetH + 32 * s2 + 8 * kq) : zero8();
  const float bias = l16 < 3 ? A.W.theta[A.W.lay.off_bd + l16] : 0.f;
  for (int rb = wave; rb < (np >> 4); rb += kBlock / 64) {
    const int row = rb * 16 + l16;
    floatx4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(H + (size_t)row * kNetH + 8 * kq), bq[0],
                                                          floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ld8(H + (size_t)row * kNetH + 32 + 8 * kq), bq[1], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float o = acc[i] + bias;                    // o[4kq + i][l16]
      const float o0 = __shfl(o, kq * 16, 64), o1 = __shfl(o, kq * 16 + 1, 64), o2 = __shfl(o, kq * 16 + 2, 64);
      const int r2 = rb * 16 + 4 * kq + i;
      if (r2 < n && l16 < 3) {
        if (A.delta) {
          const double da = s * (R[3 * l16] * o0 + R[3 * l16 + 1] * o1 + R[3 * l16 + 2] * o2);
          A.delta[3 * (voff + r2) + l16] = (Real)da;
        }
        if (A.S.out) A.S.out[((size_t)k * A.S.n_pad_max + r2) * 3 + l16] = o;
      }
    }
  }
}

// One message-passing layer over the row blocks of this wave: reads h and its
// neighbour means, writes h + relu(z) to Hout and z to Zout.
// Neighbour j of row i: nbr(q, i) for q < deg(i).
template <typename NbrF, typename DegF>
__device__ void layer_rows(const NetWeights& W, int l, int n, int np, int width, const uint16_t* Hin,
                           uint16_t* Hout, uint16_t* Zout, NbrF nbr, DegF deg) {
  const int lane = tid() & 63, wave = tid() >> 6, l16 = lane & 15, kq = lane >> 4;
  const uint16_t* Wl = W.Wl + (size_t)l * kNetH * 2 * kNetH;
  bf16x8 bq[4][4];
  float bias[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) bq[s4][cb] = ld8(Wl + (size_t)(cb * 16 + l16) * 2 * kNetH + 32 * s4 + 8 * kq);
    bias[cb] = W.theta[W.lay.b(l) + cb * 16 + l16];
  }
  for (int rb = wave; rb < (np >> 4); rb += kBlock / 64) {
    const int row = rb * 16 + l16;
    bf16x8 aq[4];
    if (row < n) {
      aq[0] = ld8(Hin + (size_t)row * kNetH + 8 * kq);
      aq[1] = ld8(Hin + (size_t)row * kNetH + 32 + 8 * kq);
      float g0[8], g1[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) g0[e] = g1[e] = 0.f;
      const int dg = deg(row);
      // the first kNetUnrollDeg ELL columns are loaded unconditionally (ELL padding points
      // at the row itself, so every address is valid) and masked by the degree; wider
      // meshes continue in a rolled loop
#pragma unroll
      for (int q = 0; q < kNetUnrollDeg; ++q) {
        const int j = q < width ? nbr(q, row) : row;
        const float w = q < dg ? 1.f : 0.f;
        const bf16x8 h0 = ld8(Hin + (size_t)j * kNetH + 8 * kq);
        const bf16x8 h1 = ld8(Hin + (size_t)j * kNetH + 32 + 8 * kq);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          g0[e] += w * (float)h0[e];
          g1[e] += w * (float)h1[e];
        }
      }
      for (int q = kNetUnrollDeg; q < dg; ++q) {
        const int j = nbr(q, row);
        const bf16x8 h0 = ld8(Hin + (size_t)j * kNetH + 8 * kq);
        const bf16x8 h1 = ld8(Hin + (size_t)j * kNetH + 32 + 8 * kq);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          g0[e] += (float)h0[e];
          g1[e] += (float)h1[e];
        }
      }
      const float inv = 1.0f / (float)dg;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        aq[2][e] = (__bf16)(g0[e] * inv);
        aq[3][e] = (__bf16)(g1[e] * inv);
      }
    } else {
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) aq[s4] = zero8();
    }
    floatx4 acc[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) acc[cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq[s4], bq[s4][cb], acc[cb], 0, 0, 0);
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r2 = rb * 16 + 4 * kq + i, col = cb * 16 + l16;
        const float z = r2 < n ? acc[cb][i] + bias[cb] : 0.f;
        const float hn = r2 < n ? bf2f(Hin[(size_t)r2 * kNetH + col]) + fmaxf(z, 0.f) : 0.f;
        Hout[(size_t)r2 * kNetH + col] = f2bf(hn);
        if (Zout) Zout[(size_t)r2 * kNetH + col] = f2bf(z);
      }
    }
  }
}

// Variant for any mesh size: activations ping-pong in memory, neighbours from CSR.
template <typename Real>
__global__ void __launch_bounds__(kBlock) net_forward_kernel(NetFwdArgs<Real> A) {
  __shared__ double red[4 * kRS];
  __shared__ double fr[10];
  const NetLayout L = A.W.lay;
  const bool train = A.S.train != 0;
  const size_t plane = (size_t)A.S.n_pad_max * kNetH;
  const int nh = train ? L.layers + 1 : 2;
  for (int k = blockIdx.x; k < A.n_cells; k += gridDim.x) {
    const int cell = A.cells ? A.cells[k] : k;
    const NetMeshDev& M = A.meshes[A.cell_mesh[cell]];
    const int n = M.n, np = M.n_pad;
    const int64_t voff = A.cell_voff[cell];
    const size_t slot = train ? (size_t)k : (size_t)blockIdx.x;
    uint16_t* feat = A.S.feat + slot * A.S.n_pad_max * kNetFeatPad;
    uint16_t* Hs = A.S.H + slot * nh * plane;
    uint16_t* Zs = train ? A.S.Z + slot * (L.layers + 1) * plane : nullptr;
    cell_features<Real>(A, M, k, A.x + 3 * voff, A.v + 3 * voff, A.f + 3 * voff, feat, red, fr);
    encoder_rows(A.W, feat, n, np, Hs, Zs);   // training: z0 for the backward pass
    __syncthreads();
    auto nbr = [&](int q, int i) { return M.nb_ell[q * np + i]; };
    auto deg = [&](int i) { return M.nb_ptr[i + 1] - M.nb_ptr[i]; };
    for (int l = 0; l < L.layers; ++l) {
      const uint16_t* Hin = Hs + (size_t)(train ? l : (l & 1)) * plane;
      uint16_t* Hout = Hs + (size_t)(train ? l + 1 : ((l + 1) & 1)) * plane;
      layer_rows(A.W, l, n, np, M.nb_deg, Hin, Hout, train ? Zs + (size_t)(l + 1) * plane : nullptr,
                              nbr, deg);
      __syncthreads();
    }
    const uint16_t* HL = Hs + (size_t)(train ? L.layers : (L.layers & 1)) * plane;
    decoder_rows<Real>(A, k, voff, n, np, HL, fr);
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------
// The frame of every cell (one wave per cell), then the network with the cell's
// activations resident in LDS and updated in place (inference, and the training forward).
// ---------------------------------------------------------------------------------

__device__ inline double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Per cell k: R (rest -> world, row-major), the displacement scale s, and the centroid,
// mean velocity and mean acceleration used by the features (kNetFrame doubles).
template <typename Real>
__global__ void __launch_bounds__(256) net_frame_kernel(NetFwdArgs<Real> A) {
  const int lane = tid() & 63;
  const int k = blockIdx.x * 4 + (tid() >> 6);
  if (k >= A.n_cells) return;
  const int cell = A.cells ? A.cells[k] : k;
  const NetMeshDev& M = A.meshes[A.cell_mesh[cell]];
  const int n = M.n;
  const int64_t voff = A.cell_voff[cell];
  const Real* x = A.x + 3 * voff;
  const Real* v = A.v + 3 * voff;
  const Real* f = A.f + 3 * voff;
  double s1[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = lane; i < n; i += 64) {
    const double m = M.mass[i];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      s1[c] += m * (double)x[3 * i + c];
      s1[3 + c] += m * (double)v[3 * i + c];
      s1[6 + c] += (double)f[3 * i + c];
    }
  }
#pragma unroll
  for (int q = 0; q < 9; ++q) s1[q] = wave_sum(s1[q]);
  const double ims = 1.0 / M.mass_sum;
  double fr[kNetFrame];
#pragma unroll
  for (int q = 0; q < 9; ++q) fr[10 + q] = s1[q] * ims;      // x_c, v_c, a_c
  double s2[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (int i = lane; i < n; i += 64) {
    const double m = M.mass[i];
    double d[3], fd[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      d[c] = (double)x[3 * i + c] - fr[10 + c];
      fd[c] = (double)f[3 * i + c] - m * fr[16 + c];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int b = 0; b < 3; ++b) s2[3 * a + b] += m * d[a] * M.Xc[3 * i + b];
    s2[9] += fd[0] * fd[0] + fd[1] * fd[1] + fd[2] * fd[2];
  }
#pragma unroll
  for (int q = 0; q < 10; ++q) s2[q] = wave_sum(s2[q]);
  polar3(s2, fr);                                          // every lane, the same values
  fr[9] = A.h * A.h * (sqrt(s2[9] / n) + A.W.force_floor) / M.mass_mean;
  fr[19] = 0.0;
  double* out = A.cframe + (size_t)k * kNetFrame;
#pragma unroll
  for (int q = 0; q < kNetFrame; ++q)
    if (lane == q) out[q] = fr[q];
}

// The network with one cell per workgroup, its activations in LDS ([n_pad][kHP] BF16) and
// the nodes taken in a reverse Cuthill-McKee order of the mesh, 16 positions per row block.
// Every product has the node as the matrix instruction's column, z^T = W_s h^T + W_n mean^T.
// Row 4 kq + i of result tile c stands for feature 32 (c / 2) + 8 kq + 4 (c % 2) + i, so that
// a lane of group kq ends up with eight consecutive features per 32 of its node: its results
// are the next product's operand, nothing is exchanged between lanes, and activations move
// as 16-byte LDS accesses.  The neighbour sums run on the matrix unit too: a neighbour's row
// is an operand as it is read, and a constant 0/1 operand picks a result tile's features from
// it, so each instruction adds one neighbour per node in FP32, in the order of the mesh's list
// (a row's neighbour positions stay in registers).
//
// Bound: the LDS.  A row block reads 14 rows of 128 bytes per node, the neighbours' from
// arbitrary rows (about two lanes to a bank), 9 k of a layer's 15 k cycles at n = 642.
// 100,000 cells: 15.5 ms; one row block per wave of the earlier layout (sums by dot2 on the
// vector unit, 2-byte LDS results, 151 KB) took 33.0 ms, dot2 sums in this layout 15.9.  The
// sums as a contraction with the adjacency over a window of nodes (transposing LDS reads, no
// random rows) reach 13.0 ms, but add in another order: 40 cells of 100,000 then change in a
// BF16 rounding, up to 4e-3 of a result.
constexpr int kHP = 72;                        // LDS row pitch (BF16): 16 rows fall on distinct banks

// A workgroup barrier that orders LDS accesses only: global loads and stores stay in flight.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Four rows x 16 columns of BF16 per 16-lane group, transposed: lane i passes the address of
// row i / 4, columns 4 (i % 4) .. + 3, and receives column i of the four rows.
typedef short short4_t __attribute__((ext_vector_type(4)));
__device__ inline uint2 ld_tr(const uint16_t* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                       (__attribute__((address_space(3))) short4_t*)const_cast<uint16_t*>(p)));
}
__device__ inline bf16x8 join8(uint2 a, uint2 b) { return __builtin_bit_cast(bf16x8, uint4{a.x, a.y, b.x, b.y}); }
__device__ inline uint2 ld4(const uint16_t* p) { return *reinterpret_cast<const uint2*>(p); }
__device__ inline uint4 ldw(const uint16_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ inline void stw(uint16_t* p, uint2 a, uint2 b) { *reinterpret_cast<uint4*>(p) = uint4{a.x, a.y, b.x, b.y}; }
__device__ inline uint32_t pack2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}
__device__ inline uint32_t pack2(double a, double b) {      // rounded once
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}
__device__ inline float half_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ inline float half_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// The nodes of a k step as masks, 0xffff or 0 each: bits j and j + 16 of a lane's word
// (shifted right by four per k step) are the nodes of dword j.
__device__ inline uint4 adj_mask(uint32_t word) {
  uint32_t d[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) d[j] = __umul24((word >> j) & 0x00010001u, 0xffffu);
  return uint4{d[0], d[1], d[2], d[3]};
}

// First feature of a lane's result tile c, and of its eight consecutive ones of 32-step s.
__device__ inline int tile_feature(int c, int kq) { return 32 * (c >> 1) + 8 * kq + 4 * (c & 1); }

// h^T operands (result tiles c) of the 32-node k step starting at row `row0`.
__device__ inline void ld_nodes_t(const uint16_t* H, int row0, int l16, int kq, bf16x8 (&a)[4]) {
  const uint16_t* p = H + (row0 + 8 * kq + (l16 >> 2)) * kHP + 8 * (l16 & 3);
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int o = 32 * (c >> 1) + 4 * (c & 1);
    a[c] = join8(ld_tr(p + o), ld_tr(p + o + 4 * kHP));
  }
}

// One layer's [W_s | W_n] operands and biases, copied to LDS by the whole workgroup with
// loads that bypass the registers.
constexpr int kLayerOps = 16 * 512 + 2 * kNetH;    // in BF16 slots; the biases are FP32
template <int NW>
__device__ inline void stage_weights(const NetWeights& W, int l, uint16_t* dst) {
  const uint16_t* src = W.WlA + (size_t)l * 16 * 512;
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6), lane = tid() & 63;
#pragma unroll
  for (int q = 0; q < 16 / NW; ++q) {
    const int f = wave + NW * q;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + f * 512 + lane * 8),
                                     (__attribute__((address_space(3))) void*)(dst + f * 512), 16, 0, 0);
  }
  if (wave == 0)
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(W.theta + W.lay.b(l) + lane),
                                     (__attribute__((address_space(3))) void*)(dst + 16 * 512), 4, 0, 0);
}
__device__ inline void wait_staged() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0)

// NW waves of up to RR row blocks each (n_pad <= 16 NW RR); a wave past the last one repeats
// it without storing, so that the rounds are free of branches.  TRAIN keeps what the backward
// pass reads: per layer the activations, the neighbour means and the signs of the
// pre-activations.  F: the precision in which the features are formed (before BF16 rounds them):
// FP64 in training, and in inference but for the small regular meshes (net_features32).
template <typename Real, int NW, int RR, bool TRAIN, typename F>
__global__ void __launch_bounds__(NW * 64, 2) net_resident_kernel(NetFwdArgs<Real> A) {
  extern __shared__ __align__(16) unsigned char lds[];
  constexpr bool kF64 = std::is_same<F, double>::value;
  constexpr int kPairs = kNetUnrollDeg / 2;
  const int zero_row = A.S.n_pad_max;          // a row of zeros: where a neighbour list has ended
  uint16_t* H = reinterpret_cast<uint16_t*>(lds);
  // two layers' operands of [W_s | W_n]: a wave's copy comes from here, the next layer's is
  // on its way meanwhile
  uint16_t* Wb = H + (zero_row + 1) * kHP;
  const int lane = tid() & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const NetLayout L = A.W.lay;
  const size_t plane = (size_t)A.S.n_pad_max * kNetH;
  // picks a result tile's features from a 32-feature operand (even and odd tiles)
  bf16x8 pick[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 8; ++e) pick[t][e] = (__bf16)(kq == (l16 >> 2) && e == 4 * t + (l16 & 3) ? 1.f : 0.f);
  if (tid() < kHP) H[zero_row * kHP + tid()] = 0;
  // of this wave's rows, while the mesh stays the same: the vertex, the inverse degree and the
  // first kNetUnrollDeg neighbours
  int mesh = -1, vert[RR];
  float inv[RR];
  uint32_t nbr[RR][kPairs];
  for (int k = blockIdx.x; k < A.n_cells; k += gridDim.x) {
    const int cell = A.cells ? A.cells[k] : k;
    const int mi = A.cell_mesh[cell];
    const NetMeshDev& M = A.meshes[mi];
    const int n = M.n, np = M.n_pad, nrb = np >> 4, pairs = (M.nb_deg + 1) >> 1;
    if (mi != mesh) {
      mesh = mi;
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const int row = min(wave + NW * r, nrb - 1) * 16 + l16;
        vert[r] = row < n ? M.perm[row] : 0;
        inv[r] = M.ideg[row];
#pragma unroll
        for (int q = 0; q < kPairs; ++q) {
          const uint32_t w = q < pairs ? M.nbp[q * np + row] : 0xffffffffu;
          const uint32_t a = w & 0xffffu, b = w >> 16;
          nbr[r][q] = (a == 0xffffu ? zero_row : a) | (b == 0xffffu ? zero_row : b) << 16;
        }
      }
    }
    const int64_t voff = A.cell_voff[cell];
    const double* fr = A.cframe + (size_t)k * kNetFrame;
    uint16_t* Hs = TRAIN ? A.S.H + (size_t)k * (L.layers + 1) * plane : nullptr;
    uint16_t* As = TRAIN ? A.S.Am + (size_t)k * L.layers * plane : nullptr;
    uint16_t* Ms = TRAIN ? A.S.mask + (size_t)k * (L.layers + 1) * (plane / 16) : nullptr;
    uint2 out[RR][4];                          // new activations of this wave's rows, BF16
    // ---- encoder: lane group kq forms features 3 kq .. + 2 of its row -----------------
    {
      double cen[3];
      F R[9];
#pragma unroll
      for (int c = 0; c < 3; ++c) cen[c] = kq == 0 ? fr[10 + c] : (kq == 1 ? fr[13 + c] : fr[16 + c]);
#pragma unroll
      for (int q = 0; q < 9; ++q) R[q] = (F)fr[q];
      const double s = fr[9];
      const F scl = kq == 0 ? (F)(1.0 / A.W.shape_scale)
                            : (kq == 1 ? (F)(A.h / s) : (kq == 2 ? (F)(A.h * A.h / s) : (F)M.inv_rho));
      const Real* src = kq == 0 ? A.x : (kq == 1 ? A.v : A.f);
      Real raw[RR][3];                         // every row is requested first
#pragma unroll
      for (int r = 0; r < RR; ++r)
#pragma unroll
        for (int c = 0; c < 3; ++c) raw[r][c] = src[3 * (voff + vert[r]) + c];
      stage_weights<NW>(A.W, 0, Wb);
      bf16x8 we[4];
      float4 bias[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        we[c] = ld8(A.W.WeA + c * 512 + lane * 8);
        bias[c] = *reinterpret_cast<const float4*>(A.W.theta + L.off_be + tile_feature(c, kq));
      }
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        if (NW * r >= nrb) continue;
        const int rb = min(wave + NW * r, nrb - 1), row = rb * 16 + l16;
        const bool own = wave + NW * r < nrb, tail = rb * 16 + 16 > n;   // uniform
        __builtin_amdgcn_sched_barrier(0);     // one row block's registers at a time
        // (R^T x - X) / shape, R^T v h / s, R^T f h^2 / (s m) or X / rho: one lane group each
        F w[3], Xr[3], fv[3];
        const double m = M.rest[4 * row + 3];
        float im = 0.f;
        if constexpr (kF64) {
#pragma unroll
          for (int a = 0; a < 3; ++a) Xr[a] = M.rest[4 * row + a];
        } else {
          const float4 q = *reinterpret_cast<const float4*>(M.restf + 4 * row);
          Xr[0] = q.x, Xr[1] = q.y, Xr[2] = q.z, im = q.w;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) w[c] = (F)fma(kq == 2 ? -m : -1.0, cen[c], (double)raw[r][c]);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const F Xa = Xr[a];
          const F t = fma(R[6 + a], w[2], fma(R[3 + a], w[1], R[a] * w[0]));     // (R^T w)_a
          F g = (kq == 3 ? Xa : t) - (kq == 0 ? Xa : F(0));
          g *= scl;
          if constexpr (kF64) g /= kq == 2 ? m : 1.0;
          else g *= kq == 2 ? im : 1.f;
          fv[a] = g;
          if (tail) fv[a] = row < n ? fv[a] : F(0);
        }
        // features 0-7 to lane group 0, 8-11 to group 1: the operand's k slots
        const uint32_t p0 = pack2(fv[0], fv[1]), p1 = pack2(fv[2], F(0));
        const uint32_t q0 = __shfl(p0, lane + 16, 64), q1 = __shfl(p1, lane + 16, 64);
        const uint32_t r0 = __shfl(p0, lane + 32, 64), r1 = __shfl(p1, lane + 32, 64);
        uint4 fw = {0u, 0u, 0u, 0u};
        if (kq == 0) fw = uint4{p0, p1 | q0 << 16, q0 >> 16 | q1 << 16, r0};
        if (kq == 1) fw = uint4{q1 | r0 << 16, r0 >> 16 | r1 << 16, 0u, 0u};
        if (TRAIN && own) *reinterpret_cast<uint4*>(A.S.feat + ((size_t)k * A.S.n_pad_max + row) * kNetFeatPad + 8 * kq) = fw;
        uint32_t bits = 0;
        uint2 o[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const floatx4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(we[c], __builtin_bit_cast(bf16x8, fw),
                                                                      floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          float z[4] = {acc[0] + bias[c].x, acc[1] + bias[c].y, acc[2] + bias[c].z, acc[3] + bias[c].w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (tail) z[i] = row < n ? z[i] : 0.f;
            if (TRAIN) bits |= z[i] > 0.f ? 1u << (4 * c + i) : 0u;
            z[i] = fmaxf(z[i], 0.f);
          }
          o[c] = uint2{pack2(z[0], z[1]), pack2(z[2], z[3])};
        }
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          if (own) stw(H + row * kHP + 32 * s2 + 8 * kq, o[2 * s2], o[2 * s2 + 1]);
          if (TRAIN && own) stw(Hs + (size_t)row * kNetH + 32 * s2 + 8 * kq, o[2 * s2], o[2 * s2 + 1]);
        }
        if (TRAIN && own) Ms[(size_t)rb * 64 + lane] = (uint16_t)bits;
      }
    }
    wait_staged();
    lds_barrier();
    // ---- message-passing layers ---------------------------------------------------------
    for (int l = 0; l < L.layers; ++l) {
      bf16x8 wf[4][4];                         // [k step: W_s 0, 1, W_n 0, 1][output tile]
      const uint16_t* Wl = Wb + (l & 1) * kLayerOps + lane * 8;
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) wf[s][c] = ld8(Wl + (c * 4 + s) * 512);
      if (l + 1 < L.layers) stage_weights<NW>(A.W, l + 1, Wb + ((l + 1) & 1) * kLayerOps);
      const float* bias_l = reinterpret_cast<const float*>(Wb + (l & 1) * kLayerOps + 16 * 512) + 8 * kq;
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        if (NW * r >= nrb) continue;
        const int rb = min(wave + NW * r, nrb - 1), row = rb * 16 + l16;
        const bool own = wave + NW * r < nrb, tail = rb * 16 + 16 > n;
        __builtin_amdgcn_sched_barrier(0);     // one row block's registers at a time
        floatx4 ag[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) ag[c] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto add = [&](int j) {
          const bf16x8 h0 = ld8(H + j * kHP + 8 * kq), h1 = ld8(H + j * kHP + 32 + 8 * kq);
#pragma unroll
          for (int c = 0; c < 4; ++c)
            ag[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick[c & 1], c < 2 ? h0 : h1, ag[c], 0, 0, 0);
        };
#pragma unroll
        for (int q = 0; q < kPairs; ++q) {
          add((int)(nbr[r][q] & 0xffffu));
          add((int)(nbr[r][q] >> 16));
        }
        // vertices of higher degree, up to the row block's longest list (a mesh with two
        // vertices of degree 200 has 598 of degree up to 8: going through the mesh's longest
        // list in every block, 2000 cells took 4.35 ms, now 1.18)
        for (int q = kPairs; q < pairs; ++q) {
          const uint32_t w = M.nbp[q * np + row];
          if (!__any(w != 0xffffffffu)) break;
          add((w & 0xffffu) == 0xffffu ? zero_row : (int)(w & 0xffffu));
          add((w >> 16) == 0xffffu ? zero_row : (int)(w >> 16));
        }
        uint4 h[2], m[2];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          h[s2] = ldw(H + row * kHP + 32 * s2 + 8 * kq);
          const floatx4 u = ag[2 * s2] * inv[r], v = ag[2 * s2 + 1] * inv[r];
          m[s2] = uint4{pack2(u[0], u[1]), pack2(u[2], u[3]), pack2(v[0], v[1]), pack2(v[2], v[3])};
          if (TRAIN && own) *reinterpret_cast<uint4*>(As + (size_t)l * plane + (size_t)row * kNetH + 32 * s2 + 8 * kq) = m[s2];
        }
        const uint32_t hw[8] = {h[0].x, h[0].y, h[0].z, h[0].w, h[1].x, h[1].y, h[1].z, h[1].w};
        const bf16x8 op[4] = {__builtin_bit_cast(bf16x8, h[0]), __builtin_bit_cast(bf16x8, h[1]),
                              __builtin_bit_cast(bf16x8, m[0]), __builtin_bit_cast(bf16x8, m[1])};
        uint32_t bits = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[s][c], op[s], acc, 0, 0, 0);
          const float4 bv = *reinterpret_cast<const float4*>(bias_l + 32 * (c >> 1) + 4 * (c & 1));
          const float z[4] = {acc[0] + bv.x, acc[1] + bv.y, acc[2] + bv.z, acc[3] + bv.w};
          const float ho[4] = {half_lo(hw[2 * c]), half_hi(hw[2 * c]), half_lo(hw[2 * c + 1]), half_hi(hw[2 * c + 1])};
          float hn[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            hn[i] = ho[i] + fmaxf(z[i], 0.f);
            if (tail) hn[i] = row < n ? hn[i] : 0.f;
            if (TRAIN) bits |= z[i] > 0.f ? 1u << (4 * c + i) : 0u;
          }
          out[r][c] = uint2{pack2(hn[0], hn[1]), pack2(hn[2], hn[3])};
        }
        if (TRAIN && own) {
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2)
            stw(Hs + (size_t)(l + 1) * plane + (size_t)row * kNetH + 32 * s2 + 8 * kq, out[r][2 * s2], out[r][2 * s2 + 1]);
          Ms[(size_t)(l + 1) * (plane / 16) + (size_t)rb * 64 + lane] = (uint16_t)bits;
        }
      }
      lds_barrier();                           // every wave is done reading the old activations
      if (l + 1 == L.layers) break;            // the decoder takes the last ones from registers
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        if (wave + NW * r >= nrb) continue;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
          stw(H + ((wave + NW * r) * 16 + l16) * kHP + 32 * s2 + 8 * kq, out[r][2 * s2], out[r][2 * s2 + 1]);
      }
      wait_staged();
      lds_barrier();
    }
    // ---- decoder: o = W_d h + b_d; lanes kq = 0 hold the three outputs of node l16 ------
    {
      const bf16x8 wd0 = ld8(A.W.WdA + lane * 8), wd1 = ld8(A.W.WdA + 512 + lane * 8);
      const float* bd = A.W.theta + L.off_bd;
      double R[9];
#pragma unroll
      for (int q = 0; q < 9; ++q) R[q] = fr[q];
      const double s = fr[9];
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        if (wave + NW * r >= nrb) continue;
        floatx4 acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wd0, join8(out[r][0], out[r][1]),
                                                              floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wd1, join8(out[r][2], out[r][3]), acc, 0, 0, 0);
        if (kq == 0 && (wave + NW * r) * 16 + l16 < n) {
          const int v = vert[r];
          const float o[3] = {acc[0] + bd[0], acc[1] + bd[1], acc[2] + bd[2]};
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            if (A.delta) {
              const double da = s * (R[3 * c] * o[0] + R[3 * c + 1] * o[1] + R[3 * c + 2] * o[2]);
              A.delta[3 * (voff + v) + c] = (Real)da;
            }
            if (TRAIN) A.S.out[((size_t)k * A.S.n_pad_max + v) * 3 + c] = o[c];
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------
// Loss: target t = R^T delta* / s with delta* = x_{n+1} - x_n - u0 = x_{n+1} - y_n,
// squared error, dLoss/do.
// ---------------------------------------------------------------------------------
template <typename Real>
__global__ void __launch_bounds__(kBlock) net_loss_kernel(NetLossArgs<Real> A) {
  __shared__ double red[4 * kRS];
  for (int k = blockIdx.x; k < A.n_cells; k += gridDim.x) {
    const int cell = A.cells ? A.cells[k] : k;
    const NetMeshDev& M = A.meshes[A.cell_mesh[cell]];
    const int n = M.n, np = M.n_pad;
    const int64_t voff = A.cell_voff[cell];
    const double* fr = A.S.frame + (size_t)k * kNetFrame;
    double R[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) R[q] = fr[q];
    const double is = 1.0 / fr[9];
    double acc[1] = {0.0};
    for (int i = tid(); i < np; i += kBlock) {
      float* dO = A.dout + ((size_t)k * A.S.n_pad_max + i) * 3;
      if (i < n) {
        const int64_t g = 3 * (voff + i);
        double d[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) d[c] = ((double)A.x_next[g + c] - (double)A.x[g + c]) - (double)A.u0[g + c];
        const float* o = A.S.out + ((size_t)k * A.S.n_pad_max + i) * 3;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const double t = (R[a] * d[0] + R[3 + a] * d[1] + R[6 + a] * d[2]) * is;
          const double r = (double)o[a] - t;
          acc[0] += r * r;
          dO[a] = (float)(2.0 * r * A.inv_count);
        }
      } else {
        dO[0] = dO[1] = dO[2] = 0.f;
      }
    }
    wg_sum<1>(acc, red);
    if (tid() == 0) A.cell_loss[k] = acc[0];
  }
}

// ---------------------------------------------------------------------------------
// Backward: per cell, decoder then layers in reverse then encoder; weight gradients
// added to this workgroup's slot of the partial sums.
// ---------------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) net_backward_kernel(NetBwdArgs A) {
  __shared__ __align__(16) uint16_t tz[kNetH * kTP];   // dz^T of a 32-node chunk
  __shared__ __align__(16) uint16_t th[kNetH * kTP];   // h^T (or features^T)
  __shared__ __align__(16) uint16_t ta[kNetH * kTP];   // (neighbour mean of h)^T
  const NetLayout L = A.W.lay;
  const int lane = tid() & 63, wave = tid() >> 6, l16 = lane & 15, kq = lane >> 4;
  const size_t plane = (size_t)A.S.n_pad_max * kNetH;
  float* part = A.partial + (size_t)blockIdx.x * L.count;
  float* dHa = A.dH + (size_t)blockIdx.x * 2 * plane;
  float* dHb = dHa + plane;
  float* Qb = A.Q + (size_t)blockIdx.x * plane;
  uint16_t* dZ = A.dZ + (size_t)blockIdx.x * plane;

  for (int k = blockIdx.x; k < A.n_cells; k += gridDim.x) {
    const int cell = A.cells ? A.cells[k] : k;
    const NetMeshDev& M = A.meshes[A.cell_mesh[cell]];
    const int n = M.n, np = M.n_pad;
    const uint16_t* Hs = A.S.H + (size_t)k * (L.layers + 1) * plane;
    const uint16_t* Zs = A.S.Z + (size_t)k * (L.layers + 1) * plane;
    const uint16_t* feat = A.S.feat + (size_t)k * A.S.n_pad_max * kNetFeatPad;
    const float* dO = A.dout + (size_t)k * A.S.n_pad_max * 3;

    // ---- decoder ---------------------------------------------------------------------
    const uint16_t* HL = Hs + (size_t)L.layers * plane;
    if (tid() < 3 * kNetH) {
      const int c = tid() / kNetH, q = tid() % kNetH;
      float acc = 0.f;
      for (int i = 0; i < n; ++i) acc += dO[3 * i + c] * bf2f(HL[(size_t)i * kNetH + q]);
      part[L.off_Wd + tid()] += acc;
    } else if (tid() < 3 * kNetH + 3) {
      const int c = tid() - 3 * kNetH;
      float acc = 0.f;
      for (int i = 0; i < n; ++i) acc += dO[3 * i + c];
      part[L.off_bd + c] += acc;
    }
    for (int e = tid(); e < np * kNetH; e += kBlock) {
      const int i = e / kNetH, q = e % kNetH;
      float g = 0.f;
      if (i < n)
        g = dO[3 * i] * bf2f(A.W.Wd[q]) + dO[3 * i + 1] * bf2f(A.W.Wd[kNetH + q]) +
            dO[3 * i + 2] * bf2f(A.W.Wd[2 * kNetH + q]);
      dHa[e] = g;
    }
    __syncthreads();

    float* dcur = dHa;
    float* dnext = dHb;
    for (int l = L.layers - 1; l >= -1; --l) {            // l = -1: the encoder
      const uint16_t* Z = Zs + (size_t)(l + 1) * plane;
      const uint16_t* Hin = l >= 0 ? Hs + (size_t)l * plane : nullptr;
      // dz = dh * [z > 0], and the bias gradient
      for (int e = tid(); e < np * kNetH; e += kBlock) {
        const int i = e / kNetH;
        const float dz = (i < n && bf2f(Z[e]) > 0.f) ? dcur[e] : 0.f;
        dZ[e] = f2bf(dz);
      }
      if (tid() < kNetH) {
        float acc = 0.f;
        for (int i = 0; i < n; ++i) {
          const size_t e = (size_t)i * kNetH + tid();
          if (bf2f(Z[e]) > 0.f) acc += dcur[e];
        }
        part[(l >= 0 ? L.b(l) : L.off_be) + tid()] += acc;
      }
      __syncthreads();
      // weight gradients: dW_s = dz^T h, dW_n = dz^T mean_N(h)  (dW_e = dz^T f)
      floatx4 gs[4], gn[4];
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) gs[kb] = gn[kb] = floatx4{0.f, 0.f, 0.f, 0.f};
      for (int c0 = 0; c0 < np; c0 += 32) {
        for (int e = tid(); e < 32 * kNetH; e += kBlock) {
          const int nd = e >> 6, q = e & 63, i = c0 + nd;
          tz[q * kTP + nd] = dZ[(size_t)i * kNetH + q];
          if (l >= 0) {
            th[q * kTP + nd] = Hin[(size_t)i * kNetH + q];
            float a = 0.f;
            if (i < n) {
              const int p0 = M.nb_ptr[i], p1 = M.nb_ptr[i + 1];
              for (int p = p0; p < p1; ++p) a += bf2f(Hin[(size_t)M.nb_idx[p] * kNetH + q]);
              a /= (float)(p1 - p0);
            }
            ta[q * kTP + nd] = f2bf(a);
          } else if (q < kNetFeatPad) {
            th[q * kTP + nd] = feat[(size_t)i * kNetFeatPad + q];
          }
        }
        __syncthreads();
        const bf16x8 aq = ld8(tz + (wave * 16 + l16) * kTP + 8 * kq);
        if (l >= 0) {
#pragma unroll
          for (int kb = 0; kb < 4; ++kb) {
            gs[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, ld8(th + (kb * 16 + l16) * kTP + 8 * kq), gs[kb], 0, 0, 0);
            gn[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, ld8(ta + (kb * 16 + l16) * kTP + 8 * kq), gn[kb], 0, 0, 0);
          }
        } else {
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
            gs[kb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aq, ld8(th + (kb * 16 + l16) * kTP + 8 * kq), gs[kb], 0, 0, 0);
        }
        __syncthreads();
      }
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int o = wave * 16 + 4 * kq + i, q = kb * 16 + l16;
          if (l >= 0) {
            part[L.Ws(l) + o * kNetH + q] += gs[kb][i];
            part[L.Wn(l) + o * kNetH + q] += gn[kb][i];
          } else if (kb < 2 && q < kNetFeat) {
            part[L.off_We + o * kNetFeat + q] += gs[kb][i];
          }
        }
      }
      if (l < 0) break;
      // dh_prev = dh + W_s^T dz + (mean_N)^T (W_n^T dz)
      {
        const uint16_t* WsT = A.W.WsT + (size_t)l * kNetH * kNetH;
        const uint16_t* WnT = A.W.WnT + (size_t)l * kNetH * kNetH;
        bf16x8 bs[2][4], bn[2][4];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) {
            bs[s2][cb] = ld8(WsT + (size_t)(cb * 16 + l16) * kNetH + 32 * s2 + 8 * kq);
            bn[s2][cb] = ld8(WnT + (size_t)(cb * 16 + l16) * kNetH + 32 * s2 + 8 * kq);
          }
        for (int rb = wave; rb < (np >> 4); rb += 4) {
          const int row = rb * 16 + l16;
          const bf16x8 a0 = ld8(dZ + (size_t)row * kNetH + 8 * kq);
          const bf16x8 a1 = ld8(dZ + (size_t)row * kNetH + 32 + 8 * kq);
          floatx4 ap[4], an[4];
#pragma unroll
          for (int cb = 0; cb < 4; ++cb) {
            ap[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bs[0][cb], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            ap[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bs[1][cb], ap[cb], 0, 0, 0);
            an[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, bn[0][cb], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            an[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, bn[1][cb], an[cb], 0, 0, 0);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int r2 = rb * 16 + 4 * kq + i;
            const float ideg = r2 < n ? 1.0f / (float)(M.nb_ptr[r2 + 1] - M.nb_ptr[r2]) : 0.f;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
              const size_t o = (size_t)r2 * kNetH + cb * 16 + l16;
              dnext[o] = r2 < n ? dcur[o] + ap[cb][i] : 0.f;
              Qb[o] = an[cb][i] * ideg;
            }
          }
        }
      }
      __syncthreads();
      for (int e = tid(); e < n * kNetH; e += kBlock) {
        const int j = e / kNetH, q = e % kNetH;
        float acc = 0.f;
        for (int p = M.nb_ptr[j]; p < M.nb_ptr[j + 1]; ++p) acc += Qb[(size_t)M.nb_idx[p] * kNetH + q];
        dnext[e] += acc;
      }
      __syncthreads();
      float* t = dcur;
      dcur = dnext;
      dnext = t;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------------
// Backward with the cell resident (meshes of n_pad <= 768), in the layout of
// net_resident_kernel.  net_chain_kernel carries one cell's dLoss/dh through the layers in
// registers (FP32) and leaves each layer's dz (BF16) in memory; net_wgrad_kernel forms the
// weight gradients, sums over every node of the minibatch, from the stored planes.
//
// The chain is bound by one cell's latency (a minibatch of 256 cells has one workgroup per
// CU): 114 us for 642 vertices, 4 layers; with the weight gradients (82 us), their sum (9) and
// the forward (106) a minibatch takes 350 us, against 5.8 ms when one workgroup of four waves
// went through a cell's layers in memory, sums over nodes running serially in 64 threads.  The neighbour term (mean_N)^T (W_n^T dz) = W_n^T sum_{i in N(j)} dz_i / deg_i is
// formed with the sum first: dz_i and 1 / deg_i, split into three BF16 parts, in one
// contraction over the window's nodes, then the FP32 sums, split likewise, against W_n; three
// parts hold 24 bits, so both keep FP32 accuracy.
// ---------------------------------------------------------------------------------
__device__ inline float row16_sum(float x) {                // over the 16 lanes of a row
  auto dpp = [](float y, auto ctrl) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), decltype(ctrl)::value, 0xf, 0xf, false));
  };
  x += dpp(x, std::integral_constant<int, 0xB1>{});         // quad_perm [1,0,3,2]
  x += dpp(x, std::integral_constant<int, 0x4E>{});         // quad_perm [2,3,0,1]
  x += dpp(x, std::integral_constant<int, 0x141>{});        // row_half_mirror
  x += dpp(x, std::integral_constant<int, 0x140>{});        // row_mirror
  return x;
}

template <int NW, int RR>
__global__ void __launch_bounds__(NW * 64, 2) net_chain_kernel(NetChainArgs A) {
  extern __shared__ __align__(16) unsigned char lds[];
  const int np_max = A.S.n_pad_max;
  uint16_t* D = reinterpret_cast<uint16_t*>(lds);            // dz of the layer, [n_pad][kHP]
  uint16_t* wdeg = D + (size_t)np_max * kHP;                 // [3][n_pad] parts of 1 / degree
  float* red = reinterpret_cast<float*>(wdeg + (size_t)3 * np_max);    // [NW][256]
  const int lane = tid() & 63, l16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid() >> 6);
  const NetLayout L = A.W.lay;
  const size_t plane = (size_t)np_max * kNetH;
  for (int k = blockIdx.x; k < A.n_cells; k += gridDim.x) {
    const int cell = A.cells ? A.cells[k] : k;
    const NetMeshDev& M = A.meshes[A.cell_mesh[cell]];
    const int n = M.n, np = M.n_pad, nblk = np >> 5;
    const uint16_t* Ms = A.S.mask + (size_t)k * (L.layers + 1) * (plane / 16);
    uint16_t* Zs = A.S.Z + (size_t)k * (L.layers + 1) * plane;          // receives dz
    float* part = A.cellpart + (size_t)k * net_cell_part(L.layers);
    for (int e = tid(); e < 3 * np; e += NW * 64) wdeg[e] = M.wdeg[e];
    // ---- decoder: dh = W_d^T dO, and the gradients of W_d and b_d ---------------------
    floatx4 dh[RR][2][4];
    {
      const uint16_t* HL = A.S.H + ((size_t)k * (L.layers + 1) + L.layers) * plane;
      float gw[3][16], gb[3] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int q = 0; q < 16; ++q) gw[c][q] = 0.f;
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const int blk = wave + NW * r;
        if (blk >= nblk) break;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int row = blk * 32 + 16 * b + l16;
          const float* o = A.dout + ((size_t)k * np_max + (row < n ? M.perm[row] : row)) * 3;   // zero on padding
          const float d0 = o[0], d1 = o[1], d2 = o[2];
          gb[0] += d0;
          gb[1] += d1;
          gb[2] += d2;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int ft = tile_feature(c, kq);
            const uint2 h = ld4(HL + (size_t)row * kNetH + ft);
            const uint2 q0 = ld4(A.W.Wd + ft), q1 = ld4(A.W.Wd + kNetH + ft), q2 = ld4(A.W.Wd + 2 * kNetH + ft);
            const float hv[4] = {half_lo(h.x), half_hi(h.x), half_lo(h.y), half_hi(h.y)};
            const float v0[4] = {half_lo(q0.x), half_hi(q0.x), half_lo(q0.y), half_hi(q0.y)};
            const float v1[4] = {half_lo(q1.x), half_hi(q1.x), half_lo(q1.y), half_hi(q1.y)};
            const float v2[4] = {half_lo(q2.x), half_hi(q2.x), half_lo(q2.y), half_hi(q2.y)};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              gw[0][4 * c + i] += d0 * hv[i];
              gw[1][4 * c + i] += d1 * hv[i];
              gw[2][4 * c + i] += d2 * hv[i];
              dh[r][b][c][i] = d0 * v0[i] + d1 * v1[i] + d2 * v2[i];
            }
          }
        }
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const float t = row16_sum(gw[c][q]);
          if (l16 == 0) red[wave * 256 + c * kNetH + tile_feature(q >> 2, kq) + (q & 3)] = t;
        }
        const float t = row16_sum(gb[c]);
        if (lane == 0) red[wave * 256 + 3 * kNetH + c] = t;
      }
      lds_barrier();
      if (tid() < 3 * kNetH + 3) {
        float t = 0.f;
        for (int w = 0; w < NW; ++w) t += red[w * 256 + tid()];
        part[(L.layers + 1) * kNetH + tid()] = t;
      }
      lds_barrier();
    }
    for (int l = L.layers - 1; l >= -1; --l) {               // l = -1: the encoder
      // dz = dh * [z > 0] to LDS and memory, and the bias gradient
      float bs[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) bs[q] = 0.f;
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const int blk = wave + NW * r;
        if (blk >= nblk) break;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int row = blk * 32 + 16 * b + l16;
          const uint32_t bits = Ms[(size_t)(l + 1) * (plane / 16) + (size_t)(blk * 2 + b) * 64 + lane];
          uint2 w[4];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            float dz[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              dz[i] = (bits >> (4 * c + i)) & 1u ? dh[r][b][c][i] : 0.f;
              bs[4 * c + i] += dz[i];
            }
            w[c] = uint2{pack2(dz[0], dz[1]), pack2(dz[2], dz[3])};
          }
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2) {
            stw(D + row * kHP + 32 * s2 + 8 * kq, w[2 * s2], w[2 * s2 + 1]);
            stw(Zs + (size_t)(l + 1) * plane + (size_t)row * kNetH + 32 * s2 + 8 * kq, w[2 * s2], w[2 * s2 + 1]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const float t = row16_sum(bs[q]);
        if (l16 == 0) red[wave * 256 + tile_feature(q >> 2, kq) + (q & 3)] = t;
      }
      lds_barrier();
      if (tid() < kNetH) {
        float t = 0.f;
        for (int w = 0; w < NW; ++w) t += red[w * 256 + tid()];
        part[(l + 1) * kNetH + tid()] = t;
      }
      if (l < 0) break;
      // dh_prev = dh + W_s^T dz + W_n^T sum_{i in N} dz_i / deg_i
      bf16x8 ws[2][4], wn[2][4];
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          ws[s][c] = ld8(A.W.WsTA + (size_t)((l * 4 + c) * 2 + s) * 512 + lane * 8);
          wn[s][c] = ld8(A.W.WnTA + (size_t)((l * 4 + c) * 2 + s) * 512 + lane * 8);
        }
#pragma unroll
      for (int r = 0; r < RR; ++r) {
        const int blk = wave + NW * r;
        if (blk >= nblk) break;
        __builtin_amdgcn_sched_barrier(0);     // one block's registers at a time
        const int lo = M.blk[2 * blk], ks = M.blk[2 * blk + 1];
        const uint32_t* adj = M.adj + (size_t)blk * M.adj_dw * 128 + lane;
        floatx4 ag[2][4];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int c = 0; c < 4; ++c) ag[b][c] = floatx4{0.f, 0.f, 0.f, 0.f};
        uint32_t w0 = 0, w1 = 0;
#pragma unroll 1
        for (int s = 0; s < ks; ++s) {
          const int at = lo + 32 * s;
          bf16x8 a[4];
          ld_nodes_t(D, at, l16, kq, a);
          if ((s & 3) == 0) {
            w0 = adj[(size_t)(s >> 2) * 128];
            w1 = adj[(size_t)(s >> 2) * 128 + 64];
          }
          const uint4 m0 = adj_mask(w0), m1 = adj_mask(w1);
          w0 >>= 4;
          w1 >>= 4;
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            const uint4 w = *reinterpret_cast<const uint4*>(wdeg + (size_t)p * np + at + 8 * kq);
            const bf16x8 b0 = __builtin_bit_cast(bf16x8, uint4{m0.x & w.x, m0.y & w.y, m0.z & w.z, m0.w & w.w});
            const bf16x8 b1 = __builtin_bit_cast(bf16x8, uint4{m1.x & w.x, m1.y & w.y, m1.z & w.z, m1.w & w.w});
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              ag[0][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], b0, ag[0][c], 0, 0, 0);
              ag[1][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c], b1, ag[1][c], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int row = blk * 32 + 16 * b + l16;
          const bf16x8 z0 = ld8(D + row * kHP + 8 * kq), z1 = ld8(D + row * kHP + 32 + 8 * kq);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            dh[r][b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ws[0][c], z0, dh[r][b][c], 0, 0, 0);
            dh[r][b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ws[1][c], z1, dh[r][b][c], 0, 0, 0);
          }
#pragma unroll
          for (int p = 0; p < 3; ++p) {                      // the sums' leading, middle and last bits
            uint2 t[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              t[c] = uint2{pack2(ag[b][c][0], ag[b][c][1]), pack2(ag[b][c][2], ag[b][c][3])};
              ag[b][c][0] -= half_lo(t[c].x);
              ag[b][c][1] -= half_hi(t[c].x);
              ag[b][c][2] -= half_lo(t[c].y);
              ag[b][c][3] -= half_hi(t[c].y);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              dh[r][b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wn[0][c], join8(t[0], t[1]), dh[r][b][c], 0, 0, 0);
              dh[r][b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wn[1][c], join8(t[2], t[3]), dh[r][b][c], 0, 0, 0);
            }
          }
        }
      }
      lds_barrier();                                         // every wave is done reading D
    }
    lds_barrier();                                           // and red, before the next cell
  }
}

// Weight gradients dz^T h and dz^T mean (dz^T features for the encoder, plane 0): contractions
// over the nodes of the cells k = blockIdx.x, + gridDim.x, ..., each wave taking every fourth
// 32-node chunk.  A lane loads eight consecutive nodes x four columns (whole 128-byte rows
// per 16 lanes) and picks its operands' node-contiguous halves with byte permutes, so a
// tile's rows (columns) are 4 (row) + cc; nothing is transposed through LDS.  The four waves'
// sums are added in LDS in a fixed order and written to this workgroup's slot.
// Bound: memory, 385 MB for 256 cells of 642 vertices in 82 us (the copy rate).  Both products
// of a layer in one workgroup read dz once (300 MB) but leave two waves per SIMD: 91 us.
constexpr int kWgPitch = 68;
__global__ void __launch_bounds__(256, 4) net_wgrad_kernel(NetChainArgs A) {
  __shared__ __align__(16) float acc_s[kNetH * kWgPitch];
  const int lane = tid() & 63, wave = tid() >> 6, l16 = lane & 15, kq = lane >> 4;
  const NetLayout L = A.W.lay;
  // blockIdx.y: 0 the encoder, 2 l + 1 and 2 l + 2 the two products of layer l
  const int np_max = A.S.n_pad_max, pl = (blockIdx.y + 1) >> 1, mean = pl > 0 && (blockIdx.y & 1) == 0;
  const size_t plane = (size_t)np_max * kNetH;
  const int pitch = pl == 0 ? kNetFeatPad : kNetH;
  floatx4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto operand = [](const uint2 (&v)[8], int cc) {
    uint32_t d[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t a = cc < 2 ? v[2 * j].x : v[2 * j].y, b = cc < 2 ? v[2 * j + 1].x : v[2 * j + 1].y;
      d[j] = __builtin_amdgcn_perm(b, a, (cc & 1) ? 0x07060302u : 0x05040100u);
    }
    return __builtin_bit_cast(bf16x8, uint4{d[0], d[1], d[2], d[3]});
  };
  for (int k = blockIdx.x; k < A.n_cells; k += gridDim.x) {
    const int cell = A.cells ? A.cells[k] : k;
    const int nch = A.meshes[A.cell_mesh[cell]].n_pad >> 5;
    const uint16_t* Z = A.S.Z + ((size_t)k * (L.layers + 1) + pl) * plane + 4 * l16;
    const uint16_t* B = pl == 0 ? A.S.feat + (size_t)k * np_max * kNetFeatPad + 4 * (l16 & 7)
                                : (mean ? A.S.Am + ((size_t)k * L.layers + pl - 1) * plane
                                        : A.S.H + ((size_t)k * (L.layers + 1) + pl - 1) * plane) + 4 * l16;
    for (int c = wave; c < nch; c += 4) {
      const int row = c * 32 + 8 * kq;
      uint2 vz[8], vb[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        vz[j] = ld4(Z + (row + j) * kNetH);
        vb[j] = ld4(B + (row + j) * pitch);
      }
      bf16x8 za[4];
#pragma unroll
      for (int a = 0; a < 4; ++a) za[a] = operand(vz, a);
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const bf16x8 o = operand(vb, b);
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(za[a], o, acc[a][b], 0, 0, 0);
      }
    }
  }
  for (int w = 0; w < 4; ++w) {
    if (wave == w) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            float* p = acc_s + (4 * (4 * kq + i) + a) * kWgPitch + 4 * l16 + b;
            *p = w == 0 ? acc[a][b][i] : *p + acc[a][b][i];
          }
    }
    __syncthreads();
  }
  float* part = A.partial + (size_t)blockIdx.x * L.count;
  if (pl == 0) {
    for (int e = tid(); e < kNetH * kNetFeat; e += 256) part[L.off_We + e] = acc_s[e / kNetFeat * kWgPitch + e % kNetFeat];
  } else {
    float* o = part + (mean ? L.Wn(pl - 1) : L.Ws(pl - 1));
    for (int e = tid(); e < kNetH * kNetH; e += 256) o[e] = acc_s[e / kNetH * kWgPitch + e % kNetH];
  }
}

// The minibatch gradient: weights summed over the slots of net_wgrad_kernel, biases and the
// decoder over the cells' sums of net_chain_kernel, in FP64, four strided partial sums per
// parameter added in a fixed order.
__global__ void __launch_bounds__(256) net_gather_kernel(NetChainArgs A, int slots, float* grad) {
  __shared__ double sh[4][64];
  const NetLayout L = A.W.lay;
  const int g = tid() >> 6;
  const int64_t p = (int64_t)blockIdx.x * 64 + (tid() & 63);
  double t = 0.0;
  if (p < L.count) {
    const int np_ = net_cell_part(L.layers);
    int at = -1;                                             // index into a cell's sums
    if (p >= L.off_Wd) at = (L.layers + 1) * kNetH + (int)(p - L.off_Wd);
    else if (p >= L.off_be && p < L.off_Ws0) at = (int)(p - L.off_be);
    else if (p >= L.off_Ws0) {
      const int64_t l = (p - L.off_Ws0) / L.layer_stride, q = (p - L.off_Ws0) % L.layer_stride - 2 * kNetH * kNetH;
      if (q >= 0) at = (int)((l + 1) * kNetH + q);
    }
    if (at >= 0) {
#pragma unroll 8
      for (int k = g; k < A.n_cells; k += 4) t += (double)A.cellpart[(size_t)k * np_ + at];
    } else {
#pragma unroll 8
      for (int s = g; s < slots; s += 4) t += (double)A.partial[(size_t)s * L.count + p];
    }
  }
  sh[g][tid() & 63] = t;
  __syncthreads();
  if (g == 0 && p < L.count) grad[p] = (float)((sh[0][tid()] + sh[1][tid()]) + (sh[2][tid()] + sh[3][tid()]));
}

__global__ void net_reduce_kernel(const float* __restrict__ partial, int grid, int64_t count, float* grad) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  double s = 0.0;
  for (int g = 0; g < grid; ++g) s += (double)partial[(size_t)g * count + p];
  grad[p] = (float)s;
}

__global__ void net_adam_kernel(float* theta, float* m, float* v, const float* grad, int64_t count, float lr,
                                float b1, float b2, float eps, float c1, float c2) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= count) return;
  const float g = grad[p];
  const float mn = b1 * m[p] + (1.f - b1) * g;
  const float vn = b2 * v[p] + (1.f - b2) * g * g;
  m[p] = mn;
  v[p] = vn;
  theta[p] -= lr * (mn / c1) / (sqrtf(vn / c2) + eps);
}

// BF16 copies of the weight blocks in the layouts the kernels read: by rows for the
// any-size kernels, and as operands of the resident ones ([..][lane][8], row l16 of tile c
// standing for feature tile_feature(c, l16 / 4) + l16 % 4, eight consecutive k per lane).
__global__ void net_pack_kernel(NetWeights w, NetPackDst d) {
  const NetLayout L = w.lay;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nWe = (int64_t)kNetH * kNetFeatPad, nL = (int64_t)L.layers * kNetH * kNetH;
  const int le = (int)(e & 511), l16 = (le >> 3) & 15, kk = 8 * (le >> 7) + (le & 7);
  auto row = [&](int c) { return tile_feature(c, l16 >> 2) + (l16 & 3); };
  if (e < nWe) {
    const int o = (int)(e / kNetFeatPad), c = (int)(e % kNetFeatPad);
    d.We[e] = c < kNetFeat ? f2bf(w.theta[L.off_We + o * kNetFeat + c]) : (uint16_t)0;
    d.WeA[e] = kk < kNetFeat ? f2bf(w.theta[L.off_We + row((int)(e >> 9)) * kNetFeat + kk]) : (uint16_t)0;
  }
  if (e < nL) {
    const int l = (int)(e / (kNetH * kNetH)), r = (int)(e % (kNetH * kNetH));
    const int o = r / kNetH, q = r % kNetH;
    const float ws = w.theta[L.Ws(l) + r], wn = w.theta[L.Wn(l) + r];
    d.Wl[(size_t)l * kNetH * 2 * kNetH + (size_t)o * 2 * kNetH + q] = f2bf(ws);
    d.Wl[(size_t)l * kNetH * 2 * kNetH + (size_t)o * 2 * kNetH + kNetH + q] = f2bf(wn);
    d.WsT[(size_t)l * kNetH * kNetH + (size_t)q * kNetH + o] = f2bf(ws);
    d.WnT[(size_t)l * kNetH * kNetH + (size_t)q * kNetH + o] = f2bf(wn);
    const int f = (int)(e >> 9) & 7, in = row(f >> 1), k = 32 * (f & 1) + kk;   // [l][input tile][k step]
    d.WsTA[e] = f2bf(w.theta[L.Ws(l) + k * kNetH + in]);
    d.WnTA[e] = f2bf(w.theta[L.Wn(l) + k * kNetH + in]);
  }
  if (e < 2 * nL) {
    const int l = (int)(e / (2 * kNetH * kNetH)), f = (int)(e >> 9) & 15, s = f & 3;
    d.WlA[e] = f2bf(w.theta[(s < 2 ? L.Ws(l) : L.Wn(l)) + row(f >> 2) * kNetH + 32 * (s & 1) + kk]);
  }
  if (e < 3 * kNetH) d.Wd[e] = f2bf(w.theta[L.off_Wd + e]);
  if (e < 1024) d.WdA[e] = l16 < 3 ? f2bf(w.theta[L.off_Wd + l16 * kNetH + 32 * (int)(e >> 9) + kk]) : (uint16_t)0;
}

__global__ void fill_zero_kernel(float* p, int64_t count) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < count) p[e] = 0.f;
}

inline int blocks_for(int64_t count, int threads) { return (int)((count + threads - 1) / threads); }

}  // namespace

template <typename Real>
hipError_t launch_net_forward(const NetFwdArgs<Real>& a, int grid, hipStream_t s) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(net_forward_kernel<Real>, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

// Waves per workgroup of the resident kernels: four, and two workgroups per CU, while the LDS
// holds two (the 18 row blocks of a 258-vertex mesh would leave eight waves a third round of
// two), else eight with at most six row blocks each.
static int resident_waves(int n_pad) { return n_pad <= 320 ? 4 : 8; }

size_t net_resident_lds_bytes(int n_pad) {
  return n_pad <= 768 ? (size_t)(n_pad + 1) * kHP * 2 + 2 * kLayerOps * 2 : 0;
}
size_t net_chain_lds_bytes(int n_pad) {
  if (n_pad > 768) return 0;     // three blocks per wave
  return ((size_t)n_pad * (kHP + 3) * 2 + (size_t)resident_waves(n_pad) * 256 * 4 + 15) / 16 * 16;
}
// FP32 features in inference: meshes of up to 704 rows and degree eight.  They round to the other
// BF16 value in about one feature of 5,500 (measured at 642 vertices); larger meshes and those of high
// degree have FP64 features (2,000 cells of 742 vertices: 435 us with FP32, 448 with FP64).
bool net_features32(int n_pad, int nb_deg) { return n_pad <= 704 && nb_deg <= 8; }

int net_resident_per_cu(int n_pad) { return resident_waves(n_pad) == 4 ? 2 : 1; }

template <typename K, typename... Args>
static hipError_t launch_lds(K kernel, dim3 grid, int threads, size_t lds, hipStream_t s, Args... args) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, dim3(threads), lds, s, args...);
  return hipGetLastError();
}

template <typename Real>
hipError_t launch_net_resident(const NetFwdArgs<Real>& a, int grid, int train, hipStream_t s) {
  (void)hipGetLastError();
  const int np = a.S.n_pad_max;
  const size_t lds = net_resident_lds_bytes(np);
  if (!a.cframe || a.n_cells < 1 || grid < 1 || lds == 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(net_frame_kernel<Real>, dim3((a.n_cells + 3) / 4), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (resident_waves(np) == 4) {
    if (train) return launch_lds(net_resident_kernel<Real, 4, 5, true, double>, dim3(grid), 256, lds, s, a);
    return a.features32 ? launch_lds(net_resident_kernel<Real, 4, 5, false, float>, dim3(grid), 256, lds, s, a)
                        : launch_lds(net_resident_kernel<Real, 4, 5, false, double>, dim3(grid), 256, lds, s, a);
  }
  if (train) return launch_lds(net_resident_kernel<Real, 8, 6, true, double>, dim3(grid), 512, lds, s, a);
  return a.features32 ? launch_lds(net_resident_kernel<Real, 8, 6, false, float>, dim3(grid), 512, lds, s, a)
                      : launch_lds(net_resident_kernel<Real, 8, 6, false, double>, dim3(grid), 512, lds, s, a);
}

hipError_t launch_net_chain(const NetChainArgs& a, int grid, int slots, float* grad, hipStream_t s) {
  (void)hipGetLastError();
  const size_t lds = net_chain_lds_bytes(a.S.n_pad_max);
  if (a.n_cells < 1 || grid < 1 || slots < 1 || slots > a.n_cells || lds == 0) return hipErrorInvalidValue;
  hipError_t e = resident_waves(a.S.n_pad_max) == 4 ? launch_lds(net_chain_kernel<4, 3>, dim3(grid), 256, lds, s, a)
                                                    : launch_lds(net_chain_kernel<8, 3>, dim3(grid), 512, lds, s, a);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(net_wgrad_kernel, dim3(slots, 2 * a.W.lay.layers + 1), dim3(256), 0, s, a);
  hipLaunchKernelGGL(net_gather_kernel, dim3(blocks_for(a.W.lay.count, 64)), dim3(256), 0, s, a, slots, grad);
  return hipGetLastError();
}

template <typename Real>
hipError_t launch_net_loss(const NetLossArgs<Real>& a, hipStream_t s) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(net_loss_kernel<Real>, dim3(a.n_cells), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_net_backward(const NetBwdArgs& a, int grid, hipStream_t s) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(net_backward_kernel, dim3(grid), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_net_reduce(const float* partial, int grid, int64_t count, float* grad, hipStream_t s) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(net_reduce_kernel, dim3(blocks_for(count, 256)), dim3(256), 0, s, partial, grid, count, grad);
  return hipGetLastError();
}

hipError_t launch_net_adam(float* theta, float* m, float* v, const float* grad, int64_t count, double lr,
                           double b1, double b2, double eps, int t, hipStream_t s) {
  (void)hipGetLastError();
  const float c1 = (float)(1.0 - std::pow(b1, t)), c2 = (float)(1.0 - std::pow(b2, t));
  hipLaunchKernelGGL(net_adam_kernel, dim3(blocks_for(count, 256)), dim3(256), 0, s, theta, m, v, grad, count,
                     (float)lr, (float)b1, (float)b2, (float)eps, c1, c2);
  return hipGetLastError();
}

hipError_t launch_net_pack(const NetWeights& w, const NetPackDst& d, hipStream_t s) {
  (void)hipGetLastError();
  const int64_t n = std::max<int64_t>((int64_t)w.lay.layers * kNetH * 2 * kNetH, (int64_t)kNetH * kNetFeatPad);
  hipLaunchKernelGGL(net_pack_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, w, d);
  return hipGetLastError();
}

hipError_t launch_fill_zero(float* p, int64_t count, hipStream_t s) {
  (void)hipGetLastError();
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks_for(count, 256)), dim3(256), 0, s, p, count);
  return hipGetLastError();
}

template hipError_t launch_net_forward<float>(const NetFwdArgs<float>&, int, hipStream_t);
template hipError_t launch_net_forward<double>(const NetFwdArgs<double>&, int, hipStream_t);
template hipError_t launch_net_resident<float>(const NetFwdArgs<float>&, int, int, hipStream_t);
template hipError_t launch_net_resident<double>(const NetFwdArgs<double>&, int, int, hipStream_t);
template hipError_t launch_net_loss<float>(const NetLossArgs<float>&, hipStream_t);
template hipError_t launch_net_loss<double>(const NetLossArgs<double>&, hipStream_t);

}  // namespace npfem
