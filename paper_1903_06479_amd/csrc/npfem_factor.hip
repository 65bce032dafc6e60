// Batched banded Cholesky substitution: the paper's own route to the products with the
// constant matrices (section 2.1.1 factors H~ once and solves with the factor in every
// iteration).  A = H~ or M~/h^2 is factored on the host as P A P^T = L L^T, P the
// reverse Cuthill-McKee order of the mesh, so that L is banded (half bandwidth b); each
// right-hand side q then needs L y = P q and L^T z = y, out = P^T z.
//
// A wave takes 16 (FP32) or 64 (FP64) right-hand sides.  They are brought into the order and
// transposed to [position][right-hand side] once, through an LDS tile, into the caller's
// workspace, which then holds y and z; the result goes back the same way.  The solved
// positions still inside the band sit in an LDS ring (one value per position and right-hand
// side).
//   FP32: the matrix cores, blocks of 16 positions (band_solve_mfma_kernel).
//   FP64: the vector units, one lane per right-hand side, blocks of 8 positions; the
//         factor entries are uniform across the wave and are read through the scalar
//         unit, every ring read feeds eight FMAs and the 8 x 8 diagonal block is solved
//         in registers (band_solve_kernel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "npfem_factor.h"

namespace npfem {
namespace {

constexpr int kRhs = 64;        // right-hand sides per wave in FP64 (one per lane)
constexpr int kTileRow = 65;    // padded row of the 64 x 64 transpose tile

// acc[k] += sum over jj < B of C[jj][k] * ring[(base + jj) mod W] (the factor entries are
// stored negated; the ring holds W = B + 16 positions), one position at a time: the next
// position's factor entries (scalar loads) and ring value (LDS) are requested before the
// current position's FMAs.
template <typename Real>
__device__ __forceinline__ void band_dot(Real (&acc)[kFactorRows], const Real* __restrict__ C, const Real* win,
                                         int base, int W, int B, int lane) {
  int slot = ((base % W) + W) % W;
  Real c[kFactorRows], v = win[slot * kRhs + lane];
#pragma unroll
  for (int k = 0; k < kFactorRows; ++k) c[k] = C[k];
  for (int g = 0; g < B; ++g) {
    Real cc[kFactorRows], vv = v;
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) cc[k] = c[k];
    if (g + 1 < B) {
      slot = slot + 1 == W ? 0 : slot + 1;
      v = win[slot * kRhs + lane];
#pragma unroll
      for (int k = 0; k < kFactorRows; ++k) c[k] = C[(g + 1) * kFactorRows + k];
    }
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) acc[k] = fma(cc[k], vv, acc[k]);
  }
}

// in[r][k] -> Y[iperm[k]][r - r0] for the wave's 64 right-hand sides r0 .. r0+63, through
// the LDS tile `lds` ([64][65]): rows read whole, written back one position per row.
// Addresses are clamped into range (and the values past the end dropped) so that the
// loads carry no branches and issue back to back; the chunk's iperm entries are read
// once, one per lane, and handed out with readlane.
template <typename Real>
__device__ __forceinline__ void load_rhs(const Real* __restrict__ in, Real* __restrict__ Y, Real* lds,
                                         const int* __restrict__ iperm, int np, int rows, int64_t r0, int lane) {
  const int64_t r_last = rows - 1;
  for (int k0 = 0; k0 < np; k0 += kRhs) {
    const int k = min(k0 + lane, np - 1);
    const bool k_ok = k0 + lane < np;
    const int ip = iperm[k];
#pragma unroll 16
    for (int rr = 0; rr < kRhs; ++rr) {
      const int64_t r = r0 + rr;
      const Real val = in[min(r, r_last) * np + k];
      lds[rr * kTileRow + lane] = (r <= r_last && k_ok) ? val : Real(0);
    }
    __syncthreads();
    const int kn = min(kRhs, np - k0);
    for (int kk = 0; kk < kn; ++kk) {
      const int pos = __builtin_amdgcn_readlane(ip, kk);
      Y[(size_t)pos * kRhs + lane] = lds[lane * kTileRow + kk];
    }
    __syncthreads();
  }
}

// out[r][k] = Y[iperm[k]][r - r0], the same way back.
template <typename Real>
__device__ __forceinline__ void store_solution(const Real* __restrict__ Y, Real* lds, const int* __restrict__ iperm,
                                               Real* __restrict__ out, int np, int rows, int64_t r0, int lane) {
  for (int k0 = 0; k0 < np; k0 += kRhs) {
    const int ip = iperm[min(k0 + lane, np - 1)];
#pragma unroll 16
    for (int kk = 0; kk < kRhs; ++kk) {       // past np: a repeat of the last position, not stored
      const int pos = __builtin_amdgcn_readlane(ip, kk);
      lds[lane * kTileRow + kk] = Y[(size_t)pos * kRhs + lane];
    }
    __syncthreads();
    const int k = k0 + lane;
    if (k < np) {
      const int rn = (int)min((int64_t)kRhs, rows - r0);
      for (int rr = 0; rr < rn; ++rr) out[(r0 + rr) * np + k] = lds[rr * kTileRow + lane];
    }
    __syncthreads();
  }
}

// The pointers are kernel arguments (not struct members) so that their no-alias
// guarantee lets uniform entries (the FP64 factor, the diagonal blocks) be fetched by
// scalar loads.
template <typename Real>
__global__ __launch_bounds__(kRhs) void band_solve_kernel(const Real* __restrict__ F, const Real* __restrict__ G,
                                                          const Real* __restrict__ T, const int* __restrict__ iperm,
                                                          const Real* __restrict__ in, Real* __restrict__ out,
                                                          Real* __restrict__ work, int np, int B, int W,
                                                          int rows) {
  extern __shared__ __align__(16) unsigned char smem[];
  Real* lds = reinterpret_cast<Real*>(smem);
  const int lane = threadIdx.x;
  const int nblk = np / kFactorRows;
  const int64_t r0 = (int64_t)blockIdx.x * kRhs;
  Real* __restrict__ Y = work + (size_t)blockIdx.x * np * kRhs;

  load_rhs(in, Y, lds, iperm, np, rows, r0, lane);

  Real* win = lds;              // ring of the last solved positions, [W][64]
  Real nxt[kFactorRows], x[kFactorRows];

  // forward: L y = P q, positions ascending
  for (int s = 0; s < W; ++s) win[s * kRhs + lane] = Real(0);
#pragma unroll
  for (int k = 0; k < kFactorRows; ++k) nxt[k] = Y[(size_t)k * kRhs + lane];
  for (int blk = 0; blk < nblk; ++blk) {
    const int i0 = blk * kFactorRows;
    Real acc[kFactorRows];
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) acc[k] = nxt[k];
    if (blk + 1 < nblk) {
#pragma unroll
      for (int k = 0; k < kFactorRows; ++k) nxt[k] = Y[(size_t)(i0 + kFactorRows + k) * kRhs + lane];
    }
    band_dot(acc, F + (size_t)blk * B * kFactorRows, win, i0 - B, W, B, lane);
    const Real* __restrict__ Tb = T + (size_t)blk * kFactorDiag;
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) {
      Real s = acc[k];
#pragma unroll
      for (int l = 0; l < k; ++l) s = fma(-Tb[kFactorRows + k * kFactorRows + l], x[l], s);
      x[k] = s * Tb[k];
    }
    const int slot = i0 % W;                              // i0 and W are multiples of 8
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) {
      win[(slot + k) * kRhs + lane] = x[k];
      Y[(size_t)(i0 + k) * kRhs + lane] = x[k];
    }
  }

  // backward: L^T z = y, positions descending
  for (int s = 0; s < W; ++s) win[s * kRhs + lane] = Real(0);
#pragma unroll
  for (int k = 0; k < kFactorRows; ++k) nxt[k] = Y[(size_t)(np - kFactorRows + k) * kRhs + lane];
  for (int blk = nblk - 1; blk >= 0; --blk) {
    const int i0 = blk * kFactorRows;
    Real acc[kFactorRows];
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) acc[k] = nxt[k];
    if (blk > 0) {
#pragma unroll
      for (int k = 0; k < kFactorRows; ++k) nxt[k] = Y[(size_t)(i0 - kFactorRows + k) * kRhs + lane];
    }
    band_dot(acc, G + (size_t)blk * B * kFactorRows, win, i0 + kFactorRows, W, B, lane);
    const Real* __restrict__ Tb = T + (size_t)blk * kFactorDiag;
#pragma unroll
    for (int k = kFactorRows - 1; k >= 0; --k) {
      Real s = acc[k];
#pragma unroll
      for (int l = k + 1; l < kFactorRows; ++l) s = fma(-Tb[kFactorRows + l * kFactorRows + k], x[l], s);
      x[k] = s * Tb[k];
    }
    const int slot = i0 % W;                              // i0 and W are multiples of 8
#pragma unroll
    for (int k = 0; k < kFactorRows; ++k) {
      win[(slot + k) * kRhs + lane] = x[k];
      Y[(size_t)(i0 + k) * kRhs + lane] = x[k];
    }
  }
  __syncthreads();

  store_solution(Y, lds, iperm, out, np, rows, r0, lane);
}

// FP32 substitution on the matrix cores (v_mfma_f32_16x16x4_f32), blocks of 16 positions and
// 16 right-hand sides per wave.  A block's update from the solved window,
// acc -= L[block][window] x[window], is a 16 x B by B x 16 product: A operand the factor,
// B operand the ring, both with four steps per 16-byte read; lane l holds rows
// 4 (l >> 4) .. +3 of column l & 15 of the result.  The 16 x 16 diagonal block is applied as
// its inverse, 4 more matrix instructions; the right-hand sides reach the B layout through the
// ring slots of the block's 16 positions (the oldest of the window, which nothing needs after
// the update).
// Bound: one wave's chain of dependent matrix instructions and LDS turns per block, so what
// counts is the number of waves: with 64 right-hand sides per wave a ring of 48 KB left three
// waves per CU, a quarter of whose SIMDs idled (60,000 rows of 2562 vertices: 5.44 ms); 16 of
// them need 11 KB, 14 waves per CU, and share the factor through the caches (2.49 ms; 2.86 with
// four groups of the factor in flight, 3.98 with one).  The factor stream
// runs kAhead 16-position groups ahead across blocks, the ring one group, Y and the diagonal
// inverse one block.
typedef float floatx4_t __attribute__((ext_vector_type(4)));
constexpr int kRhsM = 16;       // right-hand sides per wave
constexpr int kAhead = 8;

template <bool kFwd>
__device__ __forceinline__ void mfma_pass(const floatx4_t* __restrict__ A, const floatx4_t* __restrict__ D,
                                          float* __restrict__ Y, floatx4_t* win, int np, int B, int lane) {
  const int l16 = lane & 15, kq = lane >> 4;
  const int nb = np / kFactorMfmaRows, ng = B / 16;
  for (int s = 0; s < ng; ++s) win[s * 64 + lane] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // kAhead groups of the factor in flight, group g of a block in a[g % kAhead] (registers that
  // wait for a load are never copied: a copy would wait for it)
  floatx4_t a[kAhead];
#pragma unroll
  for (int k = 0; k < kAhead; ++k) a[k] = A[((size_t)(kFwd ? 0 : nb - 1) * ng + min(k, ng - 1)) * 64 + lane];
  auto rows = [&](int bi) {
    floatx4_t v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = Y[(bi * 16 + 4 * kq + r) * kRhsM + l16];
    return v;
  };
  auto put = [&](int slot, const floatx4_t& v) {       // rows 4 kq + r -> operand layout
    float* w = reinterpret_cast<float*>(win);
#pragma unroll
    for (int r = 0; r < 4; ++r) w[(slot * 64 + r * 16 + l16) * 4 + kq] = v[r];
  };
  const int b_first = kFwd ? 0 : nb - 1;
  floatx4_t nxt = rows(b_first), dn = D[b_first * 64 + lane];
  int own = kFwd ? 0 : b_first % ng;                   // ring slot (of 16 positions) of the block
  // the window's slots in the order of the factor's steps (ascending positions): forward from
  // the oldest, which is the block's own slot; backward from the block's successor
  auto next_slot = [&](int s) { return s + 1 == ng ? 0 : s + 1; };
  floatx4_t bn = win[(kFwd ? own : next_slot(own)) * 64 + lane];
  for (int it = 0; it < nb; ++it) {
    const int bi = kFwd ? it : nb - 1 - it;
    const int bnx = it + 1 < nb ? (kFwd ? bi + 1 : bi - 1) : bi;
    floatx4_t acc = nxt;
    const floatx4_t d = dn;
    nxt = rows(bnx);
    dn = D[bnx * 64 + lane];
    int sb = kFwd ? own : next_slot(own);
    for (int g0 = 0; g0 < ng; g0 += kAhead) {
#pragma unroll
      for (int u = 0; u < kAhead; ++u) {
        const int g = g0 + u;
        if (g >= ng) break;
        const floatx4_t bv = bn;
        sb = next_slot(sb);
        bn = win[sb * 64 + lane];                      // past the last group: not used
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][q], bv[q], acc, 0, 0, 0);
        // in its place the group kAhead on, or the next block's
        const bool in = g + kAhead < ng;
        a[u] = A[((size_t)(in ? bi : bnx) * ng + (in ? g + kAhead : u)) * 64 + lane];
      }
    }
    // the diagonal block: x = L_D^-1 acc (forward) or L_D^-T acc (backward)
    put(own, acc);
    const floatx4_t yv = win[own * 64 + lane];
    floatx4_t x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 4; ++q) x = __builtin_amdgcn_mfma_f32_16x16x4f32(d[q], yv[q], x, 0, 0, 0);
    put(own, x);
#pragma unroll
    for (int r = 0; r < 4; ++r) Y[(bi * 16 + 4 * kq + r) * kRhsM + l16] = x[r];
    own = kFwd ? next_slot(own) : (own == 0 ? ng - 1 : own - 1);
    // the next block's first group, which may hold the positions just solved
    bn = win[(kFwd ? own : next_slot(own)) * 64 + lane];
  }
}

__global__ __launch_bounds__(64) void band_solve_mfma_kernel(const floatx4_t* __restrict__ FA,
                                                             const floatx4_t* __restrict__ GA,
                                                             const floatx4_t* __restrict__ DA,
                                                             const floatx4_t* __restrict__ DB,
                                                             const int* __restrict__ iperm,
                                                             const float* __restrict__ in, float* __restrict__ out,
                                                             float* __restrict__ work, int np, int B, int rows) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* lds = reinterpret_cast<float*>(smem);
  const int lane = threadIdx.x, l16 = lane & 15, kq = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kRhsM;
  float* __restrict__ Y = work + (size_t)blockIdx.x * np * kRhsM;
  const int rn = (int)min((int64_t)kRhsM, rows - r0);
  const float* __restrict__ src = in + r0 * np;
  // in[r][k] -> Y[iperm[k]][r - r0] through a [16][65] tile; the next 64 columns are on their
  // way while these are written (rows past the end repeat the last, and are zero in Y)
  float v[kRhsM];
  auto request = [&](int k0) {
    const int k = min(k0 + lane, np - 1);
#pragma unroll
    for (int r = 0; r < kRhsM; ++r) v[r] = src[min(r, rn - 1) * np + k];
  };
  request(0);
  for (int k0 = 0; k0 < np; k0 += 64) {
    const int ip = iperm[min(k0 + lane, np - 1)];
#pragma unroll
    for (int r = 0; r < kRhsM; ++r) lds[r * kTileRow + lane] = r < rn ? v[r] : 0.f;
    if (k0 + 64 < np) request(k0 + 64);
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 64; kk += 4) {
      const int pos = __shfl(ip, kk + kq);
      if (k0 + kk + kq < np) Y[pos * kRhsM + l16] = lds[l16 * kTileRow + kk + kq];
    }
    __syncthreads();
  }
  mfma_pass<true>(FA, DA, Y, reinterpret_cast<floatx4_t*>(lds), np, B, lane);
  mfma_pass<false>(GA, DB, Y, reinterpret_cast<floatx4_t*>(lds), np, B, lane);
  __syncthreads();
  // and back
  float* __restrict__ dst = out + r0 * np;
  for (int k0 = 0; k0 < np; k0 += 64) {
    const int ip = iperm[min(k0 + lane, np - 1)];
#pragma unroll
    for (int kk = 0; kk < 64; kk += 4) lds[l16 * kTileRow + kk + kq] = Y[__shfl(ip, kk + kq) * kRhsM + l16];
    __syncthreads();
    if (k0 + lane < np) {
#pragma unroll
      for (int r = 0; r < kRhsM; ++r)
        if (r < rn) dst[r * np + k0 + lane] = lds[r * kTileRow + lane];
    }
    __syncthreads();
  }
}

}  // namespace

template <typename Real>
size_t band_solve_lds_bytes(int ring) {
  return (size_t)std::max(ring, kTileRow) * kRhs * sizeof(Real);
}

size_t band_solve_work_bytes(int n_pad, int rows, int real_bytes) {
  return (size_t)((rows + kRhs - 1) / kRhs) * kRhs * n_pad * real_bytes;
}

template <typename Real>
hipError_t launch_band_solve(const BandFactorDev<Real>& f, int which, int n_pad, const Real* in, Real* out,
                             Real* work, int rows, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  size_t lds = band_solve_lds_bytes<Real>(f.ring);
  if (lds > kBandSolveMaxLds) return hipErrorInvalidValue;
  const int rhs = std::is_same<Real, float>::value ? kRhsM : kRhs;
  const int grid = (rows + rhs - 1) / rhs;
  const void* fn;
  if constexpr (std::is_same<Real, float>::value) {
    fn = reinterpret_cast<const void*>(&band_solve_mfma_kernel);
    lds = (size_t)std::max(f.B, kTileRow) * kRhsM * sizeof(float);
  } else {
    fn = reinterpret_cast<const void*>(&band_solve_kernel<double>);
  }
  if (lds > 64 * 1024) {          // above the default dynamic LDS limit (set on the current device)
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if constexpr (std::is_same<Real, float>::value)
    hipLaunchKernelGGL(band_solve_mfma_kernel, dim3(grid), dim3(64), lds, s,
                       reinterpret_cast<const floatx4_t*>(f.FA[which]), reinterpret_cast<const floatx4_t*>(f.GA[which]),
                       reinterpret_cast<const floatx4_t*>(f.DA[which]), reinterpret_cast<const floatx4_t*>(f.DB[which]),
                       f.iperm, in, out, work, n_pad, f.B, rows);
  else
    hipLaunchKernelGGL(band_solve_kernel<double>, dim3(grid), dim3(kRhs), lds, s, f.F[which], f.G[which],
                       f.T[which], f.iperm, in, out, work, n_pad, f.B, f.ring, rows);
  return hipGetLastError();
}

template size_t band_solve_lds_bytes<float>(int);
template size_t band_solve_lds_bytes<double>(int);
template hipError_t launch_band_solve<float>(const BandFactorDev<float>&, int, int, const float*, float*, float*,
                                             int, hipStream_t);
template hipError_t launch_band_solve<double>(const BandFactorDev<double>&, int, int, const double*, double*,
                                              double*, int, hipStream_t);

}  // namespace npfem
