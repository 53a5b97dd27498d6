// Filtered back-projection (Methods, "Reconstruction procedure"): ramp
// filtering of every detector row of every projection, then back-projection
// of each slice over the angles in [0, pi).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "pwf_device.h"
#include "pwf_kernels.h"

namespace pwf {

// Rows of the projections, zero-padded: dst[(j ny + y) n_pad + i] = psi_j[y][i]
// for i < nx, 0 up to n_pad.
__global__ void fbp_pad_kernel(const float2* const* __restrict__ psi, int nx, int ny, int n_pad,
                               float2* __restrict__ dst, size_t total) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const size_t row = i / n_pad;
    const int col = (int)(i - row * n_pad);
    const int j = (int)(row / ny), y = (int)(row - (size_t)j * ny);
    dst[i] = col < nx ? psi[j][(size_t)y * nx + col] : make_float2(0.f, 0.f);
  }
}

// Multiply every padded row spectrum by the real ramp response (already
// divided by n_pad, the normalisation of the inverse transform).
__global__ void fbp_ramp_kernel(float2* __restrict__ a, const float* __restrict__ h, int n_pad, size_t total) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const float w = h[i % n_pad];
    a[i] = make_float2(a[i].x * w, a[i].y * w);
  }
}

// One 16 (x) by 32 (z) tile of voxels of one slice per workgroup, two voxels
// per lane (rows z and z + 16).  Voxel centres X, Z = k + 1/2 - n_out/2;
// detector index u + nx/2 - 1/2 with u = X cos - Z sin, linear interpolation,
// 0 outside the detector.  For a chunk of angles the detector samples the tile
// can reach are staged in LDS first: over the tile u spans 15 |cos| + 31 |sin|
// < 35 pixels, so kFbpSeg samples from one below the smallest corner value
// cover every voxel's pair (zeros stand for samples outside the detector).
// Each staged entry holds a sample and the step to the next one, so that a
// voxel's interpolation is one LDS read and two FMAs per part, instead of a
// gather through the vector-memory path once per angle; the lane's second
// voxel shares the per-angle reads and sits 16 sin below the first.
constexpr int kFbpSeg = 40;     // staged samples per angle
constexpr int kFbpChunk = 32;   // angles per staged chunk
constexpr int kFbpThreads = 256;
constexpr int kFbpTileZ = 32;

__global__ void __launch_bounds__(kFbpThreads) fbp_backproject_kernel(const float2* __restrict__ q, int n_proj, int nx,
                                                                      int ny, int n_pad, const float2* __restrict__ cs,
                                                                      int n_out, float scale, float2* __restrict__ vol) {
  __shared__ float4 seg[kFbpChunk * kFbpSeg];  // sample k, then sample k + 1 minus sample k
  __shared__ float2 csl[kFbpChunk];  // cos, sin
  __shared__ float t0l[kFbpChunk];   // detector index of the tile's first voxel minus base
  __shared__ int base[kFbpChunk];
  const int tiles_x = n_out / 16, tiles_z = (n_out + kFbpTileZ - 1) / kFbpTileZ;
  const int y = blockIdx.x / (tiles_x * tiles_z);
  const int tile = blockIdx.x - y * tiles_x * tiles_z;
  const int tx = tile % tiles_x, tz = tile / tiles_x;
  const float h = 0.5f * (float)n_out;
  const float dx = (float)(threadIdx.x & 15), dz = (float)(threadIdx.x >> 4);  // first voxel within the tile
  const float X0 = (float)(tx * 16) + 0.5f - h, Z0 = (float)(tz * kFbpTileZ) + 0.5f - h;
  const float off = 0.5f * (float)nx - 0.5f;
  float2 acc0 = make_float2(0.f, 0.f), acc1 = make_float2(0.f, 0.f);
  for (int j0 = 0; j0 < n_proj; j0 += kFbpChunk) {
    const int na = min(kFbpChunk, n_proj - j0);
    __syncthreads();  // the previous chunk's reads are done
    if ((int)threadIdx.x < na) {
      const float2 c = cs[j0 + threadIdx.x];
      const float xe = X0 + 15.f, ze = Z0 + (float)(kFbpTileZ - 1);
      const float ta = X0 * c.x - Z0 * c.y, tb = xe * c.x - Z0 * c.y;
      const float tc = X0 * c.x - ze * c.y, td = xe * c.x - ze * c.y;
      const int b0 = (int)floorf(fminf(fminf(ta, tb), fminf(tc, td)) + off) - 1;
      base[threadIdx.x] = b0;
      // u + nx/2 - 1/2 - base = (ta + off - base) + dx cos - dz sin: small numbers,
      // so the index and the weight keep more bits than from u itself
      csl[threadIdx.x] = c;
      t0l[threadIdx.x] = (ta + off) - (float)b0;
    }
    __syncthreads();
    // every load of the chunk is issued before the first LDS write
    constexpr int kPer = (kFbpChunk * kFbpSeg + kFbpThreads - 1) / kFbpThreads;
    float2 r0[kPer], r1[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (int)threadIdx.x + u * kFbpThreads;
      const int a = e / kFbpSeg, i = base[a < kFbpChunk ? a : 0] + e % kFbpSeg;
      const float2* row = q + ((size_t)(j0 + a) * ny + y) * n_pad;
      const bool ok = e < kFbpChunk * kFbpSeg && a < na;
      r0[u] = (ok && i >= 0 && i < nx) ? row[i] : make_float2(0.f, 0.f);
      r1[u] = (ok && i + 1 >= 0 && i + 1 < nx) ? row[i + 1] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int e = (int)threadIdx.x + u * kFbpThreads;
      if (e < kFbpChunk * kFbpSeg)
        seg[e] = make_float4(r0[u].x, r0[u].y, r1[u].x - r0[u].x, r1[u].y - r0[u].y);
    }
    __syncthreads();
    for (int a = 0; a < na; ++a) {
      const float2 c = csl[a];
      const float t = fmaf(dx, c.x, fmaf(-dz, c.y, t0l[a]));
      const float t2 = fmaf(-16.f, c.y, t);
      // t, t2 >= 1 by the choice of base (up to rounding), so truncation is the floor
      const float w = __builtin_amdgcn_fractf(t), w2 = __builtin_amdgcn_fractf(t2);
      const int k = min(max((int)t, 0), kFbpSeg - 1), k2 = min(max((int)t2, 0), kFbpSeg - 1);
      const float4 p = seg[a * kFbpSeg + k], p2 = seg[a * kFbpSeg + k2];
      acc0.x = fmaf(w, p.z, acc0.x + p.x);
      acc0.y = fmaf(w, p.w, acc0.y + p.y);
      acc1.x = fmaf(w2, p2.z, acc1.x + p2.x);
      acc1.y = fmaf(w2, p2.w, acc1.y + p2.y);
    }
  }
  const int ix = tx * 16 + (threadIdx.x & 15), iz = tz * kFbpTileZ + (threadIdx.x >> 4);
  if (iz < n_out) vol[((size_t)y * n_out + iz) * n_out + ix] = make_float2(acc0.x * scale, acc0.y * scale);
  if (iz + 16 < n_out)
    vol[((size_t)y * n_out + iz + 16) * n_out + ix] = make_float2(acc1.x * scale, acc1.y * scale);
}

hipError_t launch_fbp_pad(const float2* const* psi, int n_proj, int nx, int ny, int n_pad, float2* dst,
                          hipStream_t st) {
  const size_t total = (size_t)n_proj * ny * n_pad;
  hipLaunchKernelGGL(fbp_pad_kernel, dim3(4096), dim3(256), 0, st, psi, nx, ny, n_pad, dst, total);
  return hipGetLastError();
}

hipError_t launch_fbp_ramp(float2* a, const float* h, int n_pad, size_t rows, hipStream_t st) {
  hipLaunchKernelGGL(fbp_ramp_kernel, dim3(4096), dim3(256), 0, st, a, h, n_pad, rows * n_pad);
  return hipGetLastError();
}

hipError_t launch_fbp_backproject(const float2* q, int n_proj, int nx, int ny, int n_pad, const float2* cs, int n_out,
                                  float scale, float2* vol, hipStream_t st) {
  const size_t blocks = (size_t)ny * (n_out / 16) * ((n_out + kFbpTileZ - 1) / kFbpTileZ);
  hipLaunchKernelGGL(fbp_backproject_kernel, dim3((unsigned)blocks), dim3(kFbpThreads), 0, st, q, n_proj, nx, ny, n_pad,
                     cs, n_out, scale, vol);
  return hipGetLastError();
}

}  // namespace pwf

namespace pwf {

// Quadratic background removal after tomography (Methods, "Reconstruction
// procedure"): per slice, the least-squares quadratic in x, z (voxel-centre
// coordinates over n/2) fitted separately to the real and imaginary parts of
// the voxels at radius >= r_bg, subtracted from the whole slice.  The normal
// matrix depends only on the grid and the radius; the host inverts it once.
// Each slice is split into kBgRows-row bands, one workgroup per band.
constexpr int kBgThreads = 256;

__device__ __forceinline__ void bg_monomials(double x, double z, double (&m)[6]) {
  m[0] = 1.0;
  m[1] = x;
  m[2] = z;
  m[3] = x * x;
  m[4] = x * z;
  m[5] = z * z;
}

// partial[(slice * bands + band) * 12 + p * 6 + k] = sum over the band's
// background voxels of monomial k times part p (0 real, 1 imaginary).
__global__ void __launch_bounds__(kBgThreads) bg_moments_kernel(const float2* __restrict__ vol, int n, int rows,
                                                               double r2_bg, double* __restrict__ partial) {
  const int bands = n / rows;
  const int slice = blockIdx.x / bands, band = blockIdx.x - slice * bands;
  const double h = 0.5 * n, inv_h = 1.0 / h;
  double acc[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) acc[k] = 0.0;
  // kBgCols columns per lane at a time, their loads issued before the sums
  constexpr int kBgCols = 4;
  for (int r = 0; r < rows; ++r) {
    const int iz = band * rows + r;
    const double Z = (double)iz + 0.5 - h;
    const float2* row = vol + ((size_t)slice * n + iz) * n;
    for (int ix0 = threadIdx.x; ix0 < n; ix0 += kBgCols * kBgThreads) {
      float2 v[kBgCols];
      bool bg[kBgCols];
#pragma unroll
      for (int u = 0; u < kBgCols; ++u) {
        const int ix = ix0 + u * kBgThreads;
        const double X = (double)ix + 0.5 - h;
        bg[u] = ix < n && X * X + Z * Z >= r2_bg;
        v[u] = bg[u] ? row[ix] : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < kBgCols; ++u) {
        if (!bg[u]) continue;
        double m[6];
        bg_monomials(((double)(ix0 + u * kBgThreads) + 0.5 - h) * inv_h, Z * inv_h, m);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          acc[k] = fma(m[k], (double)v[u].x, acc[k]);
          acc[6 + k] = fma(m[k], (double)v[u].y, acc[6 + k]);
        }
      }
    }
  }
  // fixed-order reduction: wave butterflies, then the waves in order
  __shared__ double red[kBgThreads / 64][12];
#pragma unroll
  for (int k = 0; k < 12; ++k) {
    double a = acc[k];
    for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][k] = a;
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    double a = 0.0;
    for (int w = 0; w < kBgThreads / 64; ++w) a += red[w][threadIdx.x];
    partial[(size_t)blockIdx.x * 12 + threadIdx.x] = a;
  }
}

// Coefficients of every slice (band sums in order, times the inverse normal
// matrix), then the surface subtracted over the band.  coef[slice * 12 + p * 6
// + k]: coefficient k of part p, written by the slice's first band.
__global__ void __launch_bounds__(kBgThreads) bg_subtract_kernel(float2* __restrict__ vol, int n, int rows,
                                                                const double* __restrict__ partial,
                                                                const double* __restrict__ minv,
                                                                double* __restrict__ coef) {
  const int bands = n / rows;
  const int slice = blockIdx.x / bands, band = blockIdx.x - slice * bands;
  __shared__ double mom[12], c[12];
  if (threadIdx.x < 12) {
    double a = 0.0;
    for (int b = 0; b < bands; ++b) a += partial[((size_t)slice * bands + b) * 12 + threadIdx.x];
    mom[threadIdx.x] = a;
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    const int p = threadIdx.x / 6, k = threadIdx.x % 6;
    double a = 0.0;
    for (int j = 0; j < 6; ++j) a = fma(minv[k * 6 + j], mom[p * 6 + j], a);
    c[threadIdx.x] = a;
    if (band == 0) coef[(size_t)slice * 12 + threadIdx.x] = a;
  }
  __syncthreads();
  const double h = 0.5 * n, inv_h = 1.0 / h;
  for (int r = 0; r < rows; ++r) {
    const int iz = band * rows + r;
    const double z = ((double)iz + 0.5 - h) * inv_h;
    float2* row = vol + ((size_t)slice * n + iz) * n;
    for (int ix = threadIdx.x; ix < n; ix += kBgThreads) {
      double m[6];
      bg_monomials(((double)ix + 0.5 - h) * inv_h, z, m);
      double bre = 0.0, bim = 0.0;
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        bre = fma(c[k], m[k], bre);
        bim = fma(c[6 + k], m[k], bim);
      }
      const float2 v = row[ix];
      row[ix] = make_float2((float)((double)v.x - bre), (float)((double)v.y - bim));
    }
  }
}

int bg_rows_per_band(int n) { return n % 64 == 0 ? 64 : 16; }

hipError_t launch_bg_moments(const float2* vol, int n_slices, int n, double r_bg, double* partial, hipStream_t st) {
  const int rows = bg_rows_per_band(n);
  const size_t blocks = (size_t)n_slices * (n / rows);
  hipLaunchKernelGGL(bg_moments_kernel, dim3((unsigned)blocks), dim3(kBgThreads), 0, st, vol, n, rows, r_bg * r_bg,
                     partial);
  return hipGetLastError();
}

hipError_t launch_bg_subtract(float2* vol, int n_slices, int n, const double* partial, const double* minv,
                              double* coef, hipStream_t st) {
  const int rows = bg_rows_per_band(n);
  const size_t blocks = (size_t)n_slices * (n / rows);
  hipLaunchKernelGGL(bg_subtract_kernel, dim3((unsigned)blocks), dim3(kBgThreads), 0, st, vol, n, rows, partial,
                     minv, coef);
  return hipGetLastError();
}

}  // namespace pwf
