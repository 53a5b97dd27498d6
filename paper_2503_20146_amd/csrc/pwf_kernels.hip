// Element-wise, reduction and utility kernels of libpwf, and the host-side
// dispatch of the per-side sweep instantiations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "pwf_device.h"
#include "pwf_kernels.h"

namespace pwf {

__device__ __forceinline__ float2 cexp_c(float2 p) {
  float s, c;
  sincosf(p.y, &s, &c);
  const float a = expf(p.x);
  return make_float2(a * c, a * s);
}

// Multiply a natural-order spectrum by one of the Algorithm S2 windows and 1/m.
__global__ void plain_window(float2* __restrict__ a, const Inst* __restrict__ ip, int which) {
  const Inst& I = *ip;
  const int nx = I.nx, ny = I.ny;
  const size_t m = (size_t)nx * ny;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < m; i += (size_t)gridDim.x * blockDim.x) {
    const int ky = (int)(i / nx), kx = (int)(i - (size_t)ky * nx);
    const float fx = freq_of(kx, nx), fy = freq_of(ky, ny);
    float2 val = a[i];
    switch (which) {
      case PLAIN_W_Q1: val = cmul(val, transfer(I.chirp1_rev, I.s_coef, I.series, fx, fy, false)); break;
      case PLAIN_W_Q2: val = cmul(val, transfer(I.chirp2_rev, I.s_coef, I.series, fx, fy, false)); break;
      case PLAIN_W_Q2C: val = cmul(val, transfer(I.chirp2_rev, I.s_coef, I.series, fx, fy, true)); break;
      case PLAIN_W_Q1C: val = cmul(val, transfer(I.chirp1_rev, I.s_coef, I.series, fx, fy, true)); break;
      case PLAIN_W_IOTF: val = cscale(val, iotf_at(I, kx, ky)); break;
      case PLAIN_W_PINV: val = cscale(val, pinv_of(I, fx, fy)); break;
      case PLAIN_W_GAMMA2: val = cscale(val, gamma2_at(I, kx, ky)); break;
      default: break;
    }
    a[i] = cscale(val, I.inv_m);
  }
}

// Element-wise steps of Algorithm S2 in natural layout.
__global__ void plain_elementwise(int op, size_t m, const float2* __restrict__ a, const float2* __restrict__ b,
                                  float2* __restrict__ c, float2* __restrict__ out,
                                  const Inst* __restrict__ ip, const double* beta, int iter,
                                  double* __restrict__ partial) {
  const Inst& I = *ip;
  double acc = 0.0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < m; i += (size_t)gridDim.x * blockDim.x) {
    switch (op) {
      case PLAIN_EXP: out[i] = cexp_c(a[i]); break;
      case PLAIN_MUL_T: out[i] = cmul(a[i], I.t[i]); break;
      case PLAIN_MUL_CONJ_T: out[i] = cmulc(a[i], I.t[i]); break;
      case PLAIN_ABS2: out[i] = make_float2(a[i].x * a[i].x + a[i].y * a[i].y, 0.f); break;
      case PLAIN_REAL: out[i] = make_float2(a[i].x, 0.f); break;
      case PLAIN_NEG_ERR: {  // -e = f - y, and the loss sum of e^2
        const float e = I.y[i] - a[i].x;
        acc += (double)e * (double)e;
        out[i] = make_float2(-e, 0.f);
        break;
      }
      case PLAIN_MUL: out[i] = cmul(a[i], make_float2(b[i].x, 0.f)); break;  // v * Re(h)
      case PLAIN_GRAD: out[i] = cscale(cmulc(a[i], b[i]), 1.0f / *I.maxt2); break;  // b * conj(x) / max|t|^2
      case PLAIN_IMAG: out[i] = make_float2(a[i].y, 0.f); break;
      case PLAIN_DIRECTION: {  // d = Re g + i Re(Filter(Im g, P)) + Re a Re(rho) + i Im a Im(rho)
        out[i] = make_float2(a[i].x + (I.alpha_c1 + I.alpha_c2) * c[i].x,
                             b[i].x + (I.alpha_c1 - I.alpha_c2) * c[i].y);
        break;
      }
      case PLAIN_NESTEROV: {  // a = psi (in/out via out), b = d, c = z (updated in place)
        const float bf = (float)beta[iter];
        const float2 zp = c[i];
        const float2 z = make_float2(a[i].x - I.eta * b[i].x, a[i].y - I.eta * b[i].y);
        c[i] = z;
        out[i] = make_float2(z.x + bf * (z.x - zp.x), z.y + bf * (z.y - zp.y));
        break;
      }
      default: break;
    }
  }
  if (op == PLAIN_NEG_ERR) {
    __shared__ double red[16];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      double sum = 0.0;
      for (int i = 0; i < (int)(blockDim.x >> 6); ++i) sum += red[i];
      partial[blockIdx.x] = sum;
    }
  }
}

__global__ void plain_loss_final(const double* partial, int np, double* dst, int iter, int32_t* status) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < np; ++i) s += partial[i];
    if (dst) dst[iter] = s;
    if (!isfinite(s)) atomicOr(status, 1);
  }
}

// Loss of every instance from its column-tile partials (fixed order, FP64),
// when no back-blur sweep follows to sum them: one workgroup per instance.
__global__ void loss_final_kernel(const Inst* __restrict__ insts, int32_t* status) {
  const Inst& I = insts[blockIdx.x];
  if (threadIdx.x == 0 && I.loss_dst) {
    double s = 0.0;
    for (int i = 0; i < I.n_partials; ++i) s += I.loss_partial[i];
    s *= I.inv_m_d;
    I.loss_dst[0] = s;
    if (!isfinite(s)) atomicOr(status, 1);
  }
}

// ------------------------------------------------------------------ utilities

// Maximum of the workgroup's (256 lanes') non-negative values into *out, which
// other workgroups raise too.  Order-free, so deterministic.
__device__ __forceinline__ void block_max_to(float mx, float* out) {
  __shared__ float red[4];
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) {
    mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    atomicMax((unsigned int*)out, __float_as_uint(mx));
  }
}

__global__ void fill_zero_kernel(float4* __restrict__ p, size_t n16) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
    p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// max |t|^2 of up to kMaxabs2Batch diffusers (blockIdx.y = diffuser) into out[d],
// which hold 0 on entry: workgroup maxima, then an integer maximum of their
// bits (the values are not negative), so no second launch has to wait for the
// first.  (A launch in which one thread took the maximum of 256 partials was
// 11 us of every gradient, step and solve.)
__global__ void __launch_bounds__(256) maxabs2_kernel(Maxabs2Batch B) {
  const int d = blockIdx.y;
  const float2* __restrict__ t = B.t[d];
  const size_t m = B.m[d];
  float mx = 0.f;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < m; i += (size_t)gridDim.x * blockDim.x) {
    const float2 a = t[i];
    mx = fmaxf(mx, a.x * a.x + a.y * a.y);
  }
  block_max_to(mx, B.out[d]);
}

// 1-D factors of the separable windows of one instance (FP64 arguments).
__device__ __forceinline__ void build_tables(const Inst& I) {
  for (int k = threadIdx.x; k < I.nx + I.ny; k += blockDim.x) {
    const bool isx = k < I.nx;
    const int kk = isx ? k : k - I.nx;
    const int n = isx ? I.nx : I.ny;
    const double f = (double)(kk < (n >> 1) ? kk : kk - n) / (double)n;
    const double f2 = f * f;
    float2 q[2];
    const double a[2] = {I.chirp1_rev, I.chirp2_rev};
    for (int j = 0; j < 2; ++j) {
      double rev = -a[j] * f2;
      rev -= rint(rev);
      float sn, cs;
      sincosf((float)(rev * 6.283185307179586476925), &sn, &cs);
      q[j] = make_float2(cs, sn);
    }
    const float cio = isx ? I.iotf_cx : I.iotf_cy;
    const float cst = isx ? I.stf_cx : I.stf_cy;
    const float ff = (float)f2;
    // IOTF factor and 1 - STF factor: Eq. 5 / Eq. 14 in closed form, or from the
    // caller's separable IOTF with STF = IOTF^(2 gamma)
    const float* src = isx ? I.src_ix : I.src_iy;
    float iotf, g2;
    if (src) {
      iotf = src[kk];
      g2 = 1.f - powf(fmaxf(iotf, 0.f), I.two_gamma);
    } else {
      iotf = expf(-cio * ff);
      g2 = -expm1f(-cst * ff);
    }
    if (isx) {
      I.qx1[kk] = q[0];
      I.qx2[kk] = q[1];
      // (y factors below carry the 1/m of the inverse 2-D transform: exact, m = 2^k)
      I.ix[kk] = iotf;
      I.gx[kk] = g2;
    } else {
      I.qy1[kk] = make_float2(q[0].x * I.inv_m, q[0].y * I.inv_m);
      I.qy2[kk] = make_float2(q[1].x * I.inv_m, q[1].y * I.inv_m);
      I.iy[kk] = iotf;
      I.gy[kk] = g2;
    }
  }
}

__global__ void build_tables_kernel(const Inst* __restrict__ insts) { build_tables(insts[blockIdx.x]); }

// Set-up of a call on few instances in one launch: the descriptors come as
// kernel arguments, so that no copy engine and no staging buffer are involved,
// and go to device memory for the sweeps; the window tables are built from
// them, and `clear` 32-bit words at `words` (status flag, maxima) are zeroed.
__global__ void __launch_bounds__(256) setup_kernel(const SetupArgs A) {
  const Inst& I = A.inst[blockIdx.x];
  const uint32_t* src = (const uint32_t*)&I;
  uint32_t* dst = (uint32_t*)(A.dst + blockIdx.x);
  for (int i = threadIdx.x; i < (int)(sizeof(Inst) / 4); i += 256) dst[i] = src[i];
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < A.clear; i += 256) A.words[i] = 0u;
  build_tables(I);
}

hipError_t launch_setup(const SetupArgs& A, int n, hipStream_t st) {
  if (n < 1 || n > kSetupInsts) return hipErrorInvalidValue;
  hipLaunchKernelGGL(setup_kernel, dim3(n), dim3(256), 0, st, A);
  return hipGetLastError();
}

hipError_t launch_build_tables(const Inst* insts, int n, hipStream_t st) {
  hipLaunchKernelGGL(build_tables_kernel, dim3(n), dim3(256), 0, st, insts);
  return hipGetLastError();
}

// ------------------------------------------------------------------ host dispatch

#define PWF_DECLARE_SIDE(N)                                                                              \
  template <int M> hipError_t launch_row_n(int op, int plan, int nblocks, const Sweep& S, hipStream_t st); \
  template <int M> hipError_t launch_col_n(int w, int op, int nblocks, const Sweep& S, hipStream_t st); \
  template <int M> hipError_t plain_rows_n(int dir, const float2* src, float2* dst, int ny,             \
                                           const float2* tw, hipStream_t st);                          \
  template <int M> hipError_t plain_cols_n(int dir, float2* a, int nx, const float2* tw, hipStream_t st); \
  template <int M> int plan_twiddles_n(int which, float2* out);                                       \
  extern template hipError_t launch_row_n<N>(int, int, int, const Sweep&, hipStream_t);                \
  extern template hipError_t launch_col_n<N>(int, int, int, const Sweep&, hipStream_t);                \
  extern template hipError_t plain_rows_n<N>(int, const float2*, float2*, int, const float2*, hipStream_t); \
  extern template hipError_t plain_cols_n<N>(int, float2*, int, const float2*, hipStream_t); \
  extern template int plan_twiddles_n<N>(int, float2*);
PWF_DECLARE_SIDE(128)
PWF_DECLARE_SIDE(256)
PWF_DECLARE_SIDE(512)
PWF_DECLARE_SIDE(1024)
PWF_DECLARE_SIDE(2048)
#undef PWF_DECLARE_SIDE

bool row_alt_default_n(int n, int op) {
  switch (n) {
    case 128: return row_alt_default<128>(op);
    case 256: return row_alt_default<256>(op);
    case 512: return row_alt_default<512>(op);
    case 1024: return row_alt_default<1024>(op);
    case 2048: return row_alt_default<2048>(op);
    default: return false;
  }
}

int row_plan_count_n(int n) {
  switch (n) {
    case 128: return row_plan_count<128>();
    case 256: return row_plan_count<256>();
    case 512: return row_plan_count<512>();
    case 1024: return row_plan_count<1024>();
    case 2048: return row_plan_count<2048>();
    default: return 0;
  }
}

template <int N> int rows_per_block_of(int plan) {
  return plan == 2 ? RowCfgAlt2<N>::RW : plan == 1 ? RowCfgAlt<N>::RW : RowCfg<N>::RW;
}

int row_rows_per_block(int n, int plan) {
  switch (n) {
    case 128: return rows_per_block_of<128>(plan);
    case 256: return rows_per_block_of<256>(plan);
    case 512: return rows_per_block_of<512>(plan);
    case 1024: return rows_per_block_of<1024>(plan);
    case 2048: return rows_per_block_of<2048>(plan);
    default: return 0;
  }
}

int col_default_width(int n) {
  switch (n) {
    case 128: return ColSweepCfg<128>::WA;
    case 256: return ColSweepCfg<256>::WA;
    case 512: return ColSweepCfg<512>::WA;
    case 1024: return ColSweepCfg<1024>::WA;
    case 2048: return ColSweepCfg<2048>::WA;
    default: return 0;
  }
}

bool col_width_supported(int n, int w) {
  switch (n) {
    case 128: return w == ColSweepCfg<128>::WA || w == ColSweepCfg<128>::WB;
    case 256: return w == ColSweepCfg<256>::WA || w == ColSweepCfg<256>::WB;
    case 512: return w == ColSweepCfg<512>::WA || w == ColSweepCfg<512>::WB;
    case 1024: return w == ColSweepCfg<1024>::WA || w == ColSweepCfg<1024>::WB;
    case 2048: return w == ColSweepCfg<2048>::WA || w == ColSweepCfg<2048>::WB;
    default: return false;
  }
}

int col_alt_width(int n) {
  switch (n) {
    case 128: return ColSweepCfg<128>::WB;
    case 256: return ColSweepCfg<256>::WB;
    case 512: return ColSweepCfg<512>::WB;
    case 1024: return ColSweepCfg<1024>::WB;
    case 2048: return ColSweepCfg<2048>::WB;
    default: return 0;
  }
}

hipError_t launch_row(int nx, int op, int plan, int nblocks, const Sweep& S, hipStream_t st) {
  switch (nx) {
    case 128: return launch_row_n<128>(op, plan, nblocks, S, st);
    case 256: return launch_row_n<256>(op, plan, nblocks, S, st);
    case 512: return launch_row_n<512>(op, plan, nblocks, S, st);
    case 1024: return launch_row_n<1024>(op, plan, nblocks, S, st);
    case 2048: return launch_row_n<2048>(op, plan, nblocks, S, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_col(int ny, int width, int op, int nblocks, const Sweep& S, hipStream_t st) {
  switch (ny) {
    case 128: return launch_col_n<128>(width, op, nblocks, S, st);
    case 256: return launch_col_n<256>(width, op, nblocks, S, st);
    case 512: return launch_col_n<512>(width, op, nblocks, S, st);
    case 1024: return launch_col_n<1024>(width, op, nblocks, S, st);
    case 2048: return launch_col_n<2048>(width, op, nblocks, S, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_plain_rows(int nx, int dir, const float2* src, float2* dst, int ny, const float2* tw,
                             hipStream_t st) {
  switch (nx) {
    case 128: return plain_rows_n<128>(dir, src, dst, ny, tw, st);
    case 256: return plain_rows_n<256>(dir, src, dst, ny, tw, st);
    case 512: return plain_rows_n<512>(dir, src, dst, ny, tw, st);
    case 1024: return plain_rows_n<1024>(dir, src, dst, ny, tw, st);
    case 2048: return plain_rows_n<2048>(dir, src, dst, ny, tw, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_plain_cols(int ny, int dir, float2* a, int nx, const float2* tw, hipStream_t st) {
  switch (ny) {
    case 128: return plain_cols_n<128>(dir, a, nx, tw, st);
    case 256: return plain_cols_n<256>(dir, a, nx, tw, st);
    case 512: return plain_cols_n<512>(dir, a, nx, tw, st);
    case 1024: return plain_cols_n<1024>(dir, a, nx, tw, st);
    case 2048: return plain_cols_n<2048>(dir, a, nx, tw, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_plain_window(float2* a, const Inst* inst, int which, size_t m, hipStream_t st) {
  const int blocks = (int)((m + 255) / 256 < 4096 ? (m + 255) / 256 : 4096);
  hipLaunchKernelGGL(plain_window, dim3(blocks), dim3(256), 0, st, a, inst, which);
  return hipGetLastError();
}

int plain_elementwise_blocks() { return 1024; }

hipError_t launch_plain_elementwise(int op, size_t m, const float2* a, const float2* b, float2* c, float2* out,
                                    const Inst* inst, const double* beta, int iter, double* partial,
                                    hipStream_t st) {
  hipLaunchKernelGGL(plain_elementwise, dim3(plain_elementwise_blocks()), dim3(256), 0, st, op, m, a, b, c, out,
                     inst, beta, iter, partial);
  return hipGetLastError();
}

hipError_t launch_plain_loss_final(const double* partial, int np, double* dst, int iter, int32_t* status,
                                   hipStream_t st) {
  hipLaunchKernelGGL(plain_loss_final, dim3(1), dim3(64), 0, st, partial, np, dst, iter, status);
  return hipGetLastError();
}

hipError_t launch_loss_final(const Inst* insts, int n, int32_t* status, hipStream_t st) {
  hipLaunchKernelGGL(loss_final_kernel, dim3(n), dim3(64), 0, st, insts, status);
  return hipGetLastError();
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t st) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  const size_t want = (n16 + 255) / 256;
  const int blocks = (int)(want < 8192 ? want : 8192);
  hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(256), 0, st, (float4*)p, n16);
  return hipGetLastError();
}

// Joint diffuser refinement: normalisation sum_j max|u1_j|^2 from the S2
// workgroup maxima (n instances, `count` maxima each, `stride` floats apart).
// One workgroup per instance takes its maximum (order-free, so deterministic)
// and leaves it in the instance's first entry, which the next S2 rewrites;
// one thread then sums the n maxima in instance order in FP64.
__global__ void __launch_bounds__(256) joint_max_kernel(float* __restrict__ u1max, int count, size_t stride) {
  float* p = u1max + (size_t)blockIdx.x * stride;
  __shared__ float red[4];
  float mx = 0.f;
  for (int b = threadIdx.x; b < count; b += blockDim.x) mx = fmaxf(mx, p[b]);
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  if (threadIdx.x == 0) p[0] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

__global__ void __launch_bounds__(256) joint_norm_kernel(const float* __restrict__ u1max, int n, size_t stride,
                                                         double* __restrict__ dsum, float* __restrict__ maxt2) {
  __shared__ float v[256];
  double acc = 0.0;
  for (int j0 = 0; j0 < n; j0 += 256) {  // maxima gathered in parallel, summed in order
    const int m = min(256, n - j0);
    if ((int)threadIdx.x < m) v[threadIdx.x] = u1max[(size_t)(j0 + threadIdx.x) * stride];
    __syncthreads();
    if (threadIdx.x == 0)
      for (int j = 0; j < m; ++j) acc += (double)v[j];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *dsum = acc;
    *maxt2 = 0.f;   // (this iteration's gradient has read it; joint_update_kernel raises it again)
  }
}

__device__ __forceinline__ float4 ld_nt(const float4* p) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  const f4 a = __builtin_nontemporal_load((const f4*)p);
  return make_float4(a.x, a.y, a.z, a.w);
}

// t <- t - eta_t sum_j G_j / dsum, G_j = conj(u1_j) a2_j of instance j (fields
// `stride` elements apart); the sum over instances runs in order, in FP64.
// Two elements per lane and eight instances' loads in flight at a time: bound
// by reading the n fields (40 x 1024^2: 91 -> 61 us, 5.8 TB/s).  Leaves max |t|^2 of the
// new t for the next gradient.
__global__ void __launch_bounds__(256) joint_update_kernel(const float4* __restrict__ g, int n, size_t stride2,
                                                           size_t m2, float2* __restrict__ t, double eta_t,
                                                           const double* __restrict__ dsum, float* __restrict__ maxt2) {
  const double scale = eta_t / *dsum;
  float mx = 0.f;
  // (a contiguous range of the field per XCD: with the blocks dealt over all of it, 105 us)
  const unsigned blk = (gridDim.x & 7) ? blockIdx.x : (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  for (size_t r = blk * (size_t)blockDim.x + threadIdx.x; r < m2; r += (size_t)gridDim.x * blockDim.x) {
    double s[4] = {0.0, 0.0, 0.0, 0.0};
    auto add = [&](float4 a) {
      s[0] += a.x;
      s[1] += a.y;
      s[2] += a.z;
      s[3] += a.w;
    };
    int j = 0;
    for (; j + 8 <= n; j += 8) {
      float4 a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = ld_nt(g + (size_t)(j + u) * stride2 + r);
#pragma unroll
      for (int u = 0; u < 8; ++u) add(a[u]);
    }
    for (; j < n; ++j) add(ld_nt(g + (size_t)j * stride2 + r));
    const float2 t0 = t[2 * r], t1 = t[2 * r + 1];   // (the caller's: aligned to 8 bytes only)
    const float4 w = make_float4((float)((double)t0.x - scale * s[0]), (float)((double)t0.y - scale * s[1]),
                                 (float)((double)t1.x - scale * s[2]), (float)((double)t1.y - scale * s[3]));
    t[2 * r] = make_float2(w.x, w.y);
    t[2 * r + 1] = make_float2(w.z, w.w);
    mx = fmaxf(mx, fmaxf(w.x * w.x + w.y * w.y, w.z * w.z + w.w * w.w));
  }
  block_max_to(mx, maxt2);
}

hipError_t launch_joint_update(float* u1max, int n, int count, size_t max_stride, const float2* g,
                               size_t field_stride, size_t m, float2* t, double eta_t, double* dsum, float* maxt2,
                               hipStream_t st) {
  hipLaunchKernelGGL(joint_max_kernel, dim3(n), dim3(256), 0, st, u1max, count, max_stride);
  hipLaunchKernelGGL(joint_norm_kernel, dim3(1), dim3(256), 0, st, u1max, n, max_stride, dsum, maxt2);
  const int blocks = (int)std::min<size_t>((m / 2 + 255) / 256, 2048);
  hipLaunchKernelGGL(joint_update_kernel, dim3(blocks), dim3(256), 0, st, (const float4*)g, n, field_stride / 2, m / 2,
                     t, eta_t, dsum, maxt2);
  return hipGetLastError();
}

// Speckle autocorrelation sums (Siegert calibration): sum I, and for every
// shift d the sums of I(x, y) I(x + d, y) and I(x, y) I(x, y + d) (circular),
// in FP64 (the products too), in a fixed order.
// A workgroup stages tiles of ROWS x 64 pixels and the kMaxShift pixels right
// of and below them in LDS.  In a wave, lanes 0 .. 31 own the x shifts 1 .. 32
// and lanes 32 .. 63 the y shifts: the wave walks the pixels of its rows, and
// each lane multiplies the pixel (broadcast from the lane that holds its
// column) by its own shifted one.  So a lane keeps one sum instead of 67, and
// nothing is reduced across lanes but sum I and sum I^2.  Bound by the vector
// ALU (four operations per pixel and wave).  With all 67 sums in every thread
// the reductions and the one thread that added 512 partials of each sum were
// 0.21 ms at 1024^2; 27 us now.
constexpr int kSpkCols = 64, kSpkPitch = kSpkCols + kMaxShift + 1;   // (odd: y lanes hit distinct banks)
constexpr int kSpkValues = 1 + 2 * (kMaxShift + 1);

template <int ROWS>
__global__ void __launch_bounds__(256) speckle_sums_kernel(const float* __restrict__ img, int nx, int ny,
                                                           int max_shift, double* __restrict__ partial) {
  static_assert(kMaxShift == 32, "one lane per shift and axis");
  __shared__ float tile[(ROWS + kMaxShift) * kSpkPitch];
  __shared__ double red[4][66];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d = (lane & 31) + 1;
  const int off = lane < 32 ? d : d * kSpkPitch;
  const int tx = (nx + kSpkCols - 1) / kSpkCols, ty = (ny + ROWS - 1) / ROWS;
  double acc[4] = {0.0, 0.0, 0.0, 0.0}, s1 = 0.0, s2 = 0.0;
  for (int b = blockIdx.x; b < tx * ty; b += gridDim.x) {
    const int y0 = (b / tx) * ROWS, x0 = (b % tx) * kSpkCols;
    const int rows = min(ROWS, ny - y0), cols = min(kSpkCols, nx - x0);
    const int wc = cols + max_shift, n = (rows + max_shift) * wc;   // staged: at most one wrap each way
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += 256) {
      const int r = i / wc, c = i - r * wc;
      int y = y0 + r, x = x0 + c;
      y = y < ny ? y : y - ny;
      x = x < nx ? x : x - nx;
      tile[r * kSpkPitch + c] = img[(size_t)y * nx + x];
    }
    __syncthreads();
    for (int r = wave; r < rows; r += 4) {
      const float* t = tile + r * kSpkPitch;
      const float v = lane < cols ? t[lane] : 0.f;
      s1 += (double)v;
      s2 = fma((double)v, (double)v, s2);
      if (cols == kSpkCols && max_shift == kMaxShift) {
#pragma unroll
        for (int c = 0; c < kSpkCols; ++c) {
          const double vc = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), c));
          acc[c & 3] = fma(vc, (double)t[c + off], acc[c & 3]);
        }
      } else if (d <= max_shift) {   // (lanes of shifts that were not asked for have nothing staged)
        for (int c = 0; c < cols; ++c) acc[c & 3] = fma((double)t[c], (double)t[c + off], acc[c & 3]);
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) {
    s1 += __shfl_xor(s1, o, 64);
    s2 += __shfl_xor(s2, o, 64);
  }
  red[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
  if (lane == 0) {
    red[wave][64] = s1;
    red[wave][65] = s2;
  }
  __syncthreads();
  if (threadIdx.x < 66) {
    const int i = threadIdx.x;
    const double t = ((red[0][i] + red[1][i]) + red[2][i]) + red[3][i];
    double* p = partial + (size_t)blockIdx.x * kSpkValues;
    if (i < 64) {
      p[(i < 32 ? 1 : 2 + kMaxShift) + (i & 31) + 1] = t;
    } else if (i == 64) {
      p[0] = t;
    } else {
      p[1] = t;                 // d = 0 is the same sum on both axes
      p[2 + kMaxShift] = t;
    }
  }
}

// out[j] = sum over rows b of partial[b][j], 64 values per workgroup: each of
// 16 waves sums every 16th row, then the waves' sums are added in order.
__global__ void __launch_bounds__(1024) sum_rows_kernel(const double* __restrict__ partial, int rows, int len,
                                                        double* __restrict__ out) {
  __shared__ double red[16][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + lane;
  double t = 0.0;
  if (j < len) {
#pragma unroll 8
    for (int b = wave; b < rows; b += 16) t += partial[(size_t)b * len + j];
  }
  red[wave][lane] = t;
  __syncthreads();
  if (wave == 0 && j < len) {
    for (int w = 1; w < 16; ++w) t += red[w][lane];
    out[j] = t;
  }
}

hipError_t launch_sum_rows(const double* partial, int rows, int len, double* out, hipStream_t st) {
  hipLaunchKernelGGL(sum_rows_kernel, dim3((len + 63) / 64), dim3(1024), 0, st, partial, rows, len, out);
  return hipGetLastError();
}

int speckle_sum_blocks() { return 512; }

hipError_t launch_speckle_sums(const float* img, int nx, int ny, int max_shift, double* partial, double* out,
                               hipStream_t st) {
  if (max_shift < 0 || max_shift > kMaxShift) return hipErrorInvalidValue;
  // tiles of 32 rows where they fill the CUs, else of 16: twice the workgroups
  const long tx = (nx + kSpkCols - 1) / kSpkCols;
  const bool tall = tx * ((ny + 31) / 32) >= 256;
  const long tiles = tx * ((ny + (tall ? 31 : 15)) / (tall ? 32 : 16));
  const int blocks = (int)std::min<long>(tiles, speckle_sum_blocks());
  if (tall)
    hipLaunchKernelGGL(speckle_sums_kernel<32>, dim3(blocks), dim3(256), 0, st, img, nx, ny, max_shift, partial);
  else
    hipLaunchKernelGGL(speckle_sums_kernel<16>, dim3(blocks), dim3(256), 0, st, img, nx, ny, max_shift, partial);
  return launch_sum_rows(partial, blocks, kSpkValues, out, st);
}

hipError_t launch_maxabs2(const Maxabs2Batch& B, hipStream_t st) {
  if (B.n < 1 || B.n > kMaxabs2Batch) return hipErrorInvalidValue;
  hipLaunchKernelGGL(maxabs2_kernel, dim3(256, B.n), dim3(256), 0, st, B);
  return hipGetLastError();
}

int plan_twiddles(int n, int which, float2* out) {
  switch (n) {
    case 128: return plan_twiddles_n<128>(which, out);
    case 256: return plan_twiddles_n<256>(which, out);
    case 512: return plan_twiddles_n<512>(which, out);
    case 1024: return plan_twiddles_n<1024>(which, out);
    case 2048: return plan_twiddles_n<2048>(which, out);
    default: return -1;
  }
}

}  // namespace pwf
