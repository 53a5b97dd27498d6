// Filtered back-projection (Methods, "Reconstruction procedure"): ramp
// filtering of every detector row of every projection, then back-projection
// of each slice over the angles in [0, pi).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "pwf_kernels.h"
#include "pwf_sweeps.h"

namespace pwf {

// ------------------------------------------------------------------ ramp filter
//
// One pass over the projections: read a detector row, zero-pad it in registers
// to N = n_pad points, transform, multiply by the real ramp response (already
// divided by N), transform back and write the nx samples at positions 1 .. nx
// of a row of `pitch` elements, with zeros at positions 0 and nx + 1 (for
// every index outside the detector).  Bound by 8 bytes in and 8 out per
// sample; padding, transform, product and inverse transform as passes of
// their own moved 104 (n_pad = 2 nx).  180 x 128 rows
// of 1024: 0.59 -> 0.15 ms.  Half of the padded row (the first radix's upper
// inputs) is zero at compile time, and so is not loaded.
template <int N> struct FbpRowCfg : RowCfg<N> {};
template <> struct FbpRowCfg<1024> : RowCfgAlt2<1024> {};   // 64 lanes a row: 16 elements each, not 32
template <> struct FbpRowCfg<2048> : RowCfgAlt<2048> {};

template <int N>
__global__ void __launch_bounds__(FbpRowCfg<N>::T * FbpRowCfg<N>::RW)
fbp_filter_kernel(const float2* const* __restrict__ psi, int nx, int ny, int pitch, const float* __restrict__ ramp,
                  float2* __restrict__ dst, const float2* __restrict__ pass, const float2* __restrict__ full) {
  using C = FbpRowCfg<N>;
  using Plan = typename C::Plan;
  using TS = TwSel<Plan, (N > 1024 ? 4 : 1), true>;
  constexpr int T = C::T, RW = C::RW, E = N / T;
  constexpr int R1 = Plan::radix[0], RL = Plan::radix[Plan::NPASS - 1];
  constexpr int M1 = N / R1, ML = N / RL;
  constexpr bool WAVE = T <= 64;
  __shared__ float2 lds[RW * lds_len(N)];
  __shared__ float2 twl[TS::kLds];
  const int t = (int)threadIdx.x % T, rw = (int)threadIdx.x / T;
  const size_t row = (size_t)blockIdx.x * RW + rw;   // projection row / ny, detector row row % ny
  const LdsView lv{lds + rw * lds_len(N), 1};
  TwStage<TS::kLds, T * RW> tws;
  tws.load(TS::staged_from(pass, full));
  // (RW divides 32 and so ny: the workgroup's rows are one projection's)
  const int j = (int)((size_t)blockIdx.x * RW / ny);
  const float2* __restrict__ src = psi[j] + (row - (size_t)j * ny) * nx;
  float2 v[E];
  static_for<0, E>([&](auto ee) {
    constexpr int e = decltype(ee)::value, q = e % R1;
    v[e] = make_float2(0.f, 0.f);
    if constexpr (q < R1 / 2) {   // positions q M1 + (0 .. M1 - 1): below N/2
      const int x = t + T * (e / R1) + q * M1;
      if (x < nx) v[e] = gld(src, (uint32_t)x);
    }
  });
  tws.store(twl);
  if constexpr (WAVE) __syncthreads();
  fft_forward<Plan, T, WAVE>(v, t, TS::forward(twl, pass), lv);
  static_for<0, E>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    v[e] = cscale(v[e], gldf(ramp, (uint32_t)(t + T * (e / RL) + (e % RL) * ML)));
  });
  fft_inverse<Plan, T, WAVE>(v, t, TS::inverse(twl, pass), lv);
  float2* __restrict__ out = dst + row * pitch;
  static_for<0, E>([&](auto ee) {
    constexpr int e = decltype(ee)::value, q = e % R1;
    if constexpr (q < R1 / 2) {
      const int x = t + T * (e / R1) + q * M1;
      if (x < nx) gst(out, (uint32_t)(x + 1), v[e]);
    }
  });
  if (t == 0) {
    gst(out, 0, make_float2(0.f, 0.f));
    gst(out, (uint32_t)(nx + 1), make_float2(0.f, 0.f));
  }
}

template <int N>
static hipError_t fbp_filter_run(const float2* const* psi, int n_proj, int nx, int ny, int pitch, const float* ramp,
                                 float2* dst, const float2* pass, const float2* full, hipStream_t st) {
  using C = FbpRowCfg<N>;
  const size_t rows = (size_t)n_proj * ny;
  hipLaunchKernelGGL((fbp_filter_kernel<N>), dim3((unsigned)(rows / C::RW)), dim3(C::T * C::RW), 0, st, psi, nx, ny,
                     pitch, ramp, dst, pass, full);
  return hipGetLastError();
}

hipError_t launch_fbp_filter(const float2* const* psi, int n_proj, int nx, int ny, int n_pad, int pitch,
                             const float* ramp, float2* dst, const float2* tw_row, const float2* twn, hipStream_t st) {
  switch (n_pad) {
    case 128: return fbp_filter_run<128>(psi, n_proj, nx, ny, pitch, ramp, dst, tw_row, twn, st);
    case 256: return fbp_filter_run<256>(psi, n_proj, nx, ny, pitch, ramp, dst, tw_row, twn, st);
    case 512: return fbp_filter_run<512>(psi, n_proj, nx, ny, pitch, ramp, dst, tw_row, twn, st);
    case 1024: return fbp_filter_run<1024>(psi, n_proj, nx, ny, pitch, ramp, dst, tw_row, twn, st);
    case 2048: return fbp_filter_run<2048>(psi, n_proj, nx, ny, pitch, ramp, dst, tw_row, twn, st);
    default: return hipErrorInvalidValue;
  }
}

// ------------------------------------------------------------------ back-projection
//
// A workgroup takes a tile of 16 VX (x) by 16 VZ (z) voxels of S neighbouring
// slices; a lane takes VX VZ voxels, 16 apart, in all S slices.  Voxel centres
// X, Z = k + 1/2 - n_out/2; detector index u + nx/2 - 1/2 with u = X cos - Z
// sin, linear interpolation, 0 outside the detector.  For a chunk of angles
// the detector samples the tile can reach are staged in LDS: over the tile u
// spans at most (16 VX - 1) |cos| + (16 VZ - 1) |sin|, so kSeg samples from
// one below the smallest corner value cover every voxel's pair (zeros stand
// for samples outside the detector).  Each staged entry holds a sample and the
// step to the next one: one 16-byte LDS read and four FP32 operations per
// voxel, angle and slice.
// Bound by the vector ALU: index, weight and address cost as much again as the
// interpolation, and are the same for every slice (the slices differ by a
// constant LDS offset), so S slices share them.  128 slices of 1024^2 from 180
// angles: 10.5 operations per voxel, angle and slice with one slice and two
// voxels a lane, 6.12 ms; 4.6 and 0.6 for staging with S = 8, 2 x 2 voxels,
// 4.05 ms (6.0e12 interpolations a second, the vector ALU issuing in 93% of the cycles).  Copying straight
// to LDS took 4.8 ms, the next chunk's loads held in registers 4.5 ms.
constexpr int kFbpThreads = 256;
constexpr int kFbpChunk = 4;     // angles per staged chunk
constexpr int kFbpHead = 64;     // angles whose cos, sin and segment start are prepared at a time

// Entries per angle and slice: the smallest corner's index is in [1, 2), so
// indices stay below 2 + span.
template <int VX, int VZ> constexpr int fbp_seg() {
  // span <= sqrt((16 VX - 1)^2 + (16 VZ - 1)^2): 21.3 (1 x 1), 34.5 (1 x 2), 43.9 (2 x 2)
  return VX * VZ == 1 ? 24 : VX * VZ == 2 ? 40 : 48;
}

template <int S, int VX, int VZ>
__global__ void __launch_bounds__(kFbpThreads, 4)
fbp_backproject_kernel(const float2* __restrict__ q, int n_proj, int nx, int ny, int pitch,
                       const float2* __restrict__ cs, int n_out, float scale, float2* __restrict__ vol) {
  constexpr int SEG = fbp_seg<VX, VZ>(), V = VX * VZ;
  constexpr int kLen = kFbpChunk * S * SEG;
  __shared__ float4 seg[kLen];             // [angle][slice][k]: sample k and the step to sample k + 1
  __shared__ float4 head[2 * kFbpHead];        // cos, sin, detector index of the tile's first voxel minus base, base
  const int tiles_x = (n_out + 16 * VX - 1) / (16 * VX), tiles_z = (n_out + 16 * VZ - 1) / (16 * VZ);
  const int b = xcd_contiguous<false>(blockIdx.x, gridDim.x);
  const int yg = b / (tiles_x * tiles_z), y0 = yg * S;
  const int tile = b - yg * tiles_x * tiles_z;
  const int tx = tile % tiles_x, tz = tile / tiles_x;
  const float h = 0.5f * (float)n_out;
  const float dx = (float)(threadIdx.x & 15), dz = (float)(threadIdx.x >> 4);  // first voxel within the tile
  const float X0 = (float)(tx * 16 * VX) + 0.5f - h, Z0 = (float)(tz * 16 * VZ) + 0.5f - h;
  const float off = 0.5f * (float)nx - 0.5f;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  float2 acc[V][S];
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int s = 0; s < S; ++s) acc[v][s] = make_float2(0.f, 0.f);
  auto prepare = [&](int j) {   // head of angles j .. j + kFbpHead - 1 (j a multiple of that)
    if ((int)threadIdx.x < min(kFbpHead, n_proj - j)) {
      const float2 c = cs[j + threadIdx.x];
      const float xe = X0 + (float)(16 * VX - 1), ze = Z0 + (float)(16 * VZ - 1);
      const float ta = X0 * c.x - Z0 * c.y, tb = xe * c.x - Z0 * c.y;
      const float tc = X0 * c.x - ze * c.y, td = xe * c.x - ze * c.y;
      const int b0 = (int)floorf(fminf(fminf(ta, tb), fminf(tc, td)) + off) - 1;
      // u + nx/2 - 1/2 - base = (ta + off - base) + dx cos - dz sin: small numbers,
      // so the index and the weight keep more bits than from u itself
      head[(j & kFbpHead) + threadIdx.x] = make_float4(c.x, c.y, (ta + off) - (float)b0, __int_as_float(b0));
    }
  };
  // Filtered rows to registers, an (angle, slice) segment per wave at a time,
  // so that everything but the clamped position is wave-uniform; the step to
  // the next sample comes from the next lane.
  constexpr int kPer = kFbpChunk * S / 4;
  static_assert(SEG < 64, "a segment and the sample after it in one wave");
  float2 r[kPer];
  auto load = [&](int j0) {
    static_for<0, kPer>([&](auto uu) {
      constexpr int u = decltype(uu)::value;
      // segment (angle, slice) wave + 4 u; the angle is a constant where a slice group spans the waves
      const int a = S >= 4 ? 4 * u / S : (wave + 4 * u) / S, s = S >= 4 ? wave + 4 * u % S : (wave + 4 * u) % S;
      const int j = min(j0 + a, n_proj - 1);
      const int i = __builtin_amdgcn_readfirstlane(__float_as_int(head[j & (2 * kFbpHead - 1)].w)) + lane;
      const uint32_t pos = j0 + a < n_proj ? (uint32_t)min(max(i + 1, 0), nx + 1) : 0u;   // (element 0 is zero)
      r[u] = gld(q + ((size_t)j * ny + y0 + s) * pitch, pos);
    });
  };
  auto store = [&]() {
    static_for<0, kPer>([&](auto uu) {
      constexpr int u = decltype(uu)::value;
      const int xi = (int)__float_as_uint(r[u].x), yi = (int)__float_as_uint(r[u].y);
      const float nx_ = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, xi, 0x130, 0xf, 0xf, true));
      const float ny_ = __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, yi, 0x130, 0xf, 0xf, true));
      if (lane < SEG) seg[(wave + 4 * u) * SEG + lane] = make_float4(r[u].x, r[u].y, nx_ - r[u].x, ny_ - r[u].y);
    });
  };
  for (int j0 = 0; j0 < n_proj; j0 += kFbpChunk) {
    if (j0 % kFbpHead == 0) {   // (the other half of head: its last readers passed the last barrier)
      prepare(j0);
      __syncthreads();
    }
    load(j0);
    store();
    __syncthreads();
    // (angles past the last one of the final chunk are staged as zeros, with the
    // last angle's geometry: they add nothing, and the loop has no remainder)
#pragma unroll
    for (int a = 0; a < kFbpChunk; ++a) {
      const float4 c = head[min(j0 + a, n_proj - 1) & (2 * kFbpHead - 1)];
      const float t0 = fmaf(dx, c.x, fmaf(-dz, c.y, c.z));
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int vx = v % VX, vz = v / VX;
        const float t = vx ? (vz ? fmaf(-16.f, c.y, fmaf(16.f, c.x, t0)) : fmaf(16.f, c.x, t0))
                           : (vz ? fmaf(-16.f, c.y, t0) : t0);
        // 1 <= t < SEG by the choice of base and SEG (up to rounding, far below
        // the margins of 1 and 0.7): truncation is the floor
        const float w = __builtin_amdgcn_fractf(t);
        const float4* p = seg + a * S * SEG + (int)t;
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float4 g = p[s * SEG];
          acc[v][s].x = fmaf(w, g.z, acc[v][s].x + g.x);
          acc[v][s].y = fmaf(w, g.w, acc[v][s].y + g.y);
        }
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int ix = tx * 16 * VX + (threadIdx.x & 15) + 16 * (v % VX);
    const int iz = tz * 16 * VZ + (threadIdx.x >> 4) + 16 * (v / VX);
    if (ix < n_out && iz < n_out) {
#pragma unroll
      for (int s = 0; s < S; ++s)
        vol[((size_t)(y0 + s) * n_out + iz) * n_out + ix] = make_float2(acc[v][s].x * scale, acc[v][s].y * scale);
    }
  }
}

template <int S, int VX, int VZ>
static hipError_t fbp_backproject_run(const float2* q, int n_proj, int nx, int ny, int pitch, const float2* cs,
                                      int n_out, float scale, float2* vol, hipStream_t st) {
  const size_t blocks =
      (size_t)(ny / S) * ((n_out + 16 * VX - 1) / (16 * VX)) * ((n_out + 16 * VZ - 1) / (16 * VZ));
  hipLaunchKernelGGL((fbp_backproject_kernel<S, VX, VZ>), dim3((unsigned)blocks), dim3(kFbpThreads), 0, st, q, n_proj,
                     nx, ny, pitch, cs, n_out, scale, vol);
  return hipGetLastError();
}

hipError_t launch_fbp_backproject(const float2* q, int n_proj, int nx, int ny, int pitch, const float2* cs, int n_out,
                                  float scale, float2* vol, hipStream_t st) {
  // The more voxels and slices a workgroup takes, the fewer operations and
  // staged bytes per voxel (128 slices of 1024^2: 4.05 ms with 8 x 2 x 2, 4.2
  // with 4 x 2 x 2, 5.0 with 4 x 1 x 2), as long as three workgroups per CU are
  // there to overlap staging with interpolation.  (ny is a multiple of 32, n_out
  // of 16.)
  const size_t want = 768;
  const size_t t32 = (size_t)((n_out + 31) / 32), t16 = (size_t)(n_out / 16);
  if (t32 * t32 * (ny / 8) >= want) return fbp_backproject_run<8, 2, 2>(q, n_proj, nx, ny, pitch, cs, n_out, scale, vol, st);
  if (t32 * t32 * (ny / 4) >= want) return fbp_backproject_run<4, 2, 2>(q, n_proj, nx, ny, pitch, cs, n_out, scale, vol, st);
  if (t16 * t32 * (ny / 4) >= want) return fbp_backproject_run<4, 1, 2>(q, n_proj, nx, ny, pitch, cs, n_out, scale, vol, st);
  if (t16 * t32 * (ny / 2) >= want) return fbp_backproject_run<2, 1, 2>(q, n_proj, nx, ny, pitch, cs, n_out, scale, vol, st);
  return fbp_backproject_run<1, 1, 1>(q, n_proj, nx, ny, pitch, cs, n_out, scale, vol, st);
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
