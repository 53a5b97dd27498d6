// Fourier shell correlation (Methods, Eq. 16) of the chosen parts (0 real, 1
// imaginary) a, b of two complex volumes (n^3) or images (n^2).
//
// Three or four passes over memory, all bound by it:
//   rows    two rows of a in one complex transform (and two of b in another),
//           split by Hermitian symmetry: both real fields' half spectra
//           kx = 0 .. n/2 - 1, interleaved as (A, B) pairs, fill exactly one
//           complex n^dims array.  Real values at kx = 0 and n/2 share
//           position 0 (A(0) + i A(n/2) per row), as in the sweeps' half form.
//   columns along y (per z plane) and, in 3-D, along z, in place.
//   shells  sums per shell of Re(A* B), |A|^2, |B|^2, reading the array once.
// That is 24 + 16 + 16 + 8 bytes per voxel.  The earlier form put a and b as
// real and imaginary part of one field: it read both inputs once more for
// their RMS (the two had to be brought to one size first), wrote the packed
// field, transformed all kx and read C(k) and C(-k) for the shells, 104 bytes
// per voxel.  Here each field has transforms of its own, so neither's
// rounding reaches the other whatever their sizes.
// Measured at 512^3: 3.60 -> 1.69 ms a call (one thread per shell summing the
// workgroups' partials was 0.23 of the 3.60, one summing the RMS partials 0.07).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "pwf_sweeps.h"

namespace pwf {

namespace {

constexpr int kFscThreads = 256;

// ------------------------------------------------------------------ rows

template <int N> struct FscRowCfg : RowCfg<N> {};
template <> struct FscRowCfg<1024> : RowCfgAlt2<1024> {};   // 64 lanes a row: 16 elements each, not 32
template <> struct FscRowCfg<2048> : RowCfgAlt<2048> {};

template <int N> struct FscRowTw {
  using TS = TwSel<typename FscRowCfg<N>::Plan, (N > 1024 ? 4 : 1), true>;
};

// Workgroup: RW transforms = RW/2 row pairs x {a, b}.  Bound by its 24 bytes
// per voxel, 16 of them the interleaved inputs of which it uses one part.
template <int N>
__global__ void __launch_bounds__(FscRowCfg<N>::T * FscRowCfg<N>::RW)
fsc_rows_kernel(const float2* __restrict__ g1, const float2* __restrict__ g2, int part, float s1, float s2,
                float4* __restrict__ dst, const float2* __restrict__ pass, const float2* __restrict__ full) {
  using C = FscRowCfg<N>;
  using Plan = typename C::Plan;
  using TS = typename FscRowTw<N>::TS;
  constexpr int T = C::T, RW = C::RW, E = N / T;
  constexpr int R1 = Plan::radix[0], RL = Plan::radix[Plan::NPASS - 1];
  constexpr int M1 = N / R1, ML = N / RL;
  constexpr bool WAVE = T <= 64;
  static_assert(RW % 2 == 0 && (N / 2) % (2 * T) == 0, "row pairs");
  __shared__ float2 lds[RW * lds_len(N)];
  __shared__ float2 twl[TS::kLds];
  const int b = xcd_contiguous<false>(blockIdx.x, gridDim.x);
  const int t = (int)threadIdx.x % T, q = (int)threadIdx.x / T;
  TwStage<TS::kLds, T * RW> tws;
  tws.load(TS::staged_from(pass, full));
  {
    const float s = (q & 1) ? s2 : s1;
    const size_t r0 = 2 * ((size_t)b * (RW / 2) + (q >> 1));
    const float* __restrict__ src = (const float*)(((q & 1) ? g2 : g1) + r0 * N) + part;
    const LdsView lv{lds + q * lds_len(N), 1};
    float2 v[E];
    static_for<0, E>([&](auto ee) {
      constexpr int e = decltype(ee)::value;
      const uint32_t x = (uint32_t)(t + T * (e / R1) + (e % R1) * M1);
      v[e] = make_float2(gldf(src, 2 * x), gldf(src, 2 * x + 2 * N));
    });
    tws.store(twl);
    if constexpr (WAVE) __syncthreads();
    static_for<0, E>([&](auto ee) { v[decltype(ee)::value] = cscale(v[decltype(ee)::value], s); });
    fft_forward<Plan, T, WAVE>(v, t, TS::forward(twl, pass), lv);
    static_for<0, E>([&](auto ee) {
      constexpr int e = decltype(ee)::value;
      lv.at(t + T * (e / RL) + (e % RL) * ML) = v[e];
    });
  }
  __syncthreads();
  // split: with C = F{row0 + i row1}, 2 F{row0} = C(k) + conj C(-k) and
  // 2 F{row1} = (C(k) - conj C(-k)) / i (the common factor leaves the correlation unchanged; a sum of two
  // FP32 numbers is rounded once, as an FP64 one would be when it is stored)
  const int pl = (int)threadIdx.x / (2 * T), u = (int)threadIdx.x % (2 * T);
  const LdsView la{lds + 2 * pl * lds_len(N), 1}, lb{lds + (2 * pl + 1) * lds_len(N), 1};
  float4* __restrict__ out = dst + 2 * ((size_t)b * (RW / 2) + pl) * (N / 2);
  static_for<0, (N / 2) / (2 * T)>([&](auto jj) {
    constexpr int j = decltype(jj)::value;
    const int k = u + j * 2 * T, m = k ? N - k : N / 2;
    const float2 a = la.at(k), am = la.at(m), c = lb.at(k), cm = lb.at(m);
    float4 o0 = make_float4(a.x + am.x, a.y - am.y, c.x + cm.x, c.y - cm.y);
    float4 o1 = make_float4(a.y + am.y, am.x - a.x, c.y + cm.y, cm.x - c.x);
    if (j == 0 && k == 0) {   // real values at kx = 0 and n/2
      o0 = make_float4(2.f * a.x, 2.f * am.x, 2.f * c.x, 2.f * cm.x);
      o1 = make_float4(2.f * a.y, 2.f * am.y, 2.f * c.y, 2.f * cm.y);
    }
    out[k] = o0;
    out[N / 2 + k] = o1;
  });
}

// ------------------------------------------------------------------ columns

// Forward transforms of every column, in place, of `planes` [N][nx] planes
// plane_stride elements apart (tiles of W columns; nx a multiple of W).  The
// twiddles are staged in LDS as in the column sweeps; tiles that share
// 128-byte lines run on one XCD.
template <int N>
__global__ void __launch_bounds__(ColCfg<N>::T * ColCfg<N>::WA, 2)
fsc_cols_kernel(float2* __restrict__ a, size_t nx, size_t plane_stride, int tiles, const float2* __restrict__ pass,
                const float2* __restrict__ full) {
  using C = ColCfg<N>;
  using Plan = typename C::Plan;
  using TS = TwSel<Plan, (N > 1024 ? 2 : 1), true>;
  constexpr int T = C::T, W = C::WA, E = N / T;
  constexpr int R1 = Plan::radix[0], RL = Plan::radix[Plan::NPASS - 1];
  constexpr int M1 = N / R1, ML = N / RL;
  __shared__ float2 lds[W * lds_len(N)];
  __shared__ float2 twl[TS::kLds];
  const int b = xcd_contiguous<false>(blockIdx.x, gridDim.x);
  const int plane = b / tiles, tile = b - plane * tiles;
  const int w = (int)threadIdx.x % W, t = (int)threadIdx.x / W;
  const LdsView lv{lds + w, W};
  TwStage<TS::kLds, T * W> tws;
  tws.load(TS::staged_from(pass, full));
  float2* __restrict__ base = a + plane * plane_stride + (size_t)tile * W + w + (size_t)t * nx;
  float2 v[E];
  static_for<0, E>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    v[e] = base[(size_t)(T * (e / R1) + (e % R1) * M1) * nx];
  });
  tws.store(twl);
  fft_forward<Plan, T>(v, t, TS::forward(twl, pass), lv);
  static_for<0, E>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    base[(size_t)(T * (e / RL) + (e % RL) * ML) * nx] = v[e];
  });
}

// ------------------------------------------------------------------ shells

// Shell sums of Re(A* B), |A|^2, |B|^2 over kappa = round(|k|) (signed index
// frequencies of an n^dims grid), kappa <= n/2, in a fixed order (the result is
// bit-reproducible), from the half spectra of fsc_rows_kernel.  The rows
// (+-ky, +-kz) hold the same kappa along kx: a wave takes all of them at once
// (four in 3-D, two in 2-D; a row that is its own mirror counts its share), so
// that one pass of the run logic below serves up to four rows, and its loads
// are all in flight together.  Columns kx > 0 stand for -kx too (weight 2);
// position 0 is split into kx = 0 and kx = n/2 with the mirrored row.
// Every wave owns a private histogram of the three sums in LDS and walks its
// share of the row groups in chunks of 64 K consecutive elements, K per lane
// (64 K divides n/2).  kappa is monotone in kx, so equal kappa form runs of
// consecutive elements:
//  * each lane sums its own K elements run by run; a run that starts and ends
//    inside the lane is complete and goes to the histogram at once (no other
//    lane holds that kappa);
//  * the lane's first and last runs may continue runs of its neighbours.  A
//    lane whose K elements are one run passes the sum arriving from the left
//    on (when kappa matches) plus its own; any other lane starts afresh with
//    its last run.  That is the map x -> A x + B per lane (A = 1 for a
//    continuing single-run lane, else 0), composed over the wave by an
//    inclusive scan in a fixed butterfly order;
//  * a lane with several runs adds the sum arriving from the left to its first
//    run and writes that; a lane whose last run the next lane does not
//    continue writes its scan value.
// The kappa written by the lanes of one store are distinct, so no two lanes
// of a wave touch one entry at once, and the stores follow program order.
// The workgroup then adds its waves' histograms in wave order and writes one
// row of partials.  Four waves per workgroup up to n = 1024 and two at 2048
// keep the histograms at 49 KB of LDS.
__device__ __forceinline__ void shell_add(double (&s)[3], double ax, double ay, double bx, double by, double w) {
  s[0] += w * (ax * bx + ay * by);
  s[1] += w * (ax * ax + ay * ay);
  s[2] += w * (bx * bx + by * by);
}

template <int N, int K, int DIMS>
__global__ void __launch_bounds__(kFscThreads) fsc_shell_kernel(const float4* __restrict__ spec,
                                                                double* __restrict__ partial) {
  extern __shared__ double sh[];
  constexpr int H = N / 2, nsh = H + 1;
  constexpr int CPR = H / (64 * K);         // chunks per row
  constexpr int NR = DIMS == 3 ? 4 : 2;     // rows of a group
  constexpr int groups = DIMS == 3 ? (H + 1) * (H + 1) : H + 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
  for (int i = threadIdx.x; i < waves * 3 * nsh; i += blockDim.x) sh[i] = 0.0;
  __syncthreads();
  double* h = sh + wave * 3 * nsh;
  // (each sum converts its operands itself: held for all four sums they took 18 more registers and, at
  // 512^3, a wave per SIMD: 1.69 -> 1.77 ms)
  auto sum = [](float a, float b) {
    asm volatile("" : "+v"(a), "+v"(b));
    return (double)a + (double)b;
  };
  auto put = [&](int k, double x0, double x1, double x2) {
    if (k < nsh) {
      h[k] += x0;
      h[nsh + k] += x1;
      h[2 * nsh + k] += x2;
    }
  };
  for (int c = (int)blockIdx.x * waves + wave; c < groups * CPR; c += (int)gridDim.x * waves) {
    const int g = c / CPR, kx0 = (c - g * CPR) * 64 * K + lane * K;
    const int ky = g % (H + 1), kz = g / (H + 1);   // 0 .. n/2; kz = 0 in 2-D
    const float fx0 = (float)((c - g * CPR) * 64 * K);
    const float r2 = (float)ky * (float)ky + (float)kz * (float)kz;
    if (fx0 * fx0 + r2 > ((float)H + 0.5f) * ((float)H + 0.5f)) continue;   // (uniform) the whole chunk lies outside
    int sk[K];
#pragma unroll
    for (int j = 0; j < K; ++j) {
      const float fx = (float)(kx0 + j);
      const int k = (int)rintf(sqrtf(fx * fx + r2));
      sk[j] = k < nsh ? k : nsh;  // nsh: outside the last shell
    }
    // rows (ky, kz), (-ky, kz), (ky, -kz), (-ky, -kz): row i and row NR - 1 - i mirror each other
    float4 p[NR][K];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int yy = (i & 1) ? (N - ky) & (N - 1) : ky, zz = (i & 2) ? (N - kz) & (N - 1) : kz;
      const float4* __restrict__ row = spec + ((size_t)zz * N + yy) * H + kx0;
#pragma unroll
      for (int j = 0; j < K; ++j) p[i][j] = sk[0] < nsh ? row[j] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    // a self-mirrored row is loaded twice and counted half each
    const double wr = (((ky & (H - 1)) == 0) ? 0.5 : 1.0) * ((DIMS == 3 && (kz & (H - 1)) == 0) ? 0.5 : 1.0);
    // runs inside the lane: f = first run, q = current run
    double f0 = 0.0, f1 = 0.0, f2 = 0.0, q0 = 0.0, q1 = 0.0, q2 = 0.0;
    int sf = sk[0], sq = sk[0];
    bool multi = false;
#pragma unroll
    for (int j = 0; j < K; ++j) {
      double v[3] = {0.0, 0.0, 0.0};
      if (j == 0 && kx0 == 0) {
        double ny[3] = {0.0, 0.0, 0.0};   // kx = n/2
#pragma unroll
        for (int i = 0; i < NR / 2; ++i) {
          // P = X0 + i Xn with X0, Xn Hermitian: 2 X0 = P(k) + conj P(-k), 2 Xn = (P(k) - conj P(-k)) / i,
          // separated in FP64 (the weight takes the factor of 2)
          const float4 u = p[i][j], m = p[NR - 1 - i][j];
          shell_add(v, sum(u.x, m.x), sum(u.y, -m.y), sum(u.z, m.z), sum(u.w, -m.w), 0.5 * wr);
          shell_add(ny, sum(u.y, m.y), sum(m.x, -u.x), sum(u.w, m.w), sum(m.z, -u.z), 0.5 * wr);
        }
        put((int)rintf(sqrtf((float)H * (float)H + r2)), ny[0], ny[1], ny[2]);   // (this lane alone)
      } else {
#pragma unroll
        for (int i = 0; i < NR; ++i)
          shell_add(v, p[i][j].x, p[i][j].y, p[i][j].z, p[i][j].w, 2.0 * wr);
      }
      if (sk[j] == nsh) v[0] = v[1] = v[2] = 0.0;
      if (j == 0) {
        f0 = v[0];
        f1 = v[1];
        f2 = v[2];
      } else if (sk[j] == sq) {
        if (multi) {
          q0 += v[0];
          q1 += v[1];
          q2 += v[2];
        } else {
          f0 += v[0];
          f1 += v[1];
          f2 += v[2];
        }
      } else {
        if (multi) put(sq, q0, q1, q2);  // a run inside the lane is complete
        multi = true;
        sq = sk[j];
        q0 = v[0];
        q1 = v[1];
        q2 = v[2];
      }
    }
    const int sl = multi ? sq : sf;  // kappa of the lane's last run
    const int sl_prev = __shfl_up(sl, 1, 64);
    const bool join = lane > 0 && sl_prev == sf;
    int A = !multi && join ? 1 : 0;
    double B0 = multi ? q0 : f0, B1 = multi ? q1 : f1, B2 = multi ? q2 : f2;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int Ap = __shfl_up(A, d, 64);
      const double P0 = __shfl_up(B0, d, 64);
      const double P1 = __shfl_up(B1, d, 64);
      const double P2 = __shfl_up(B2, d, 64);
      if (lane >= d) {
        if (A) {
          B0 += P0;
          B1 += P1;
          B2 += P2;
        }
        A &= Ap;
      }
    }
    // B is now the sum of this lane's last run and the run it continues
    const double in0 = __shfl_up(B0, 1, 64), in1 = __shfl_up(B1, 1, 64), in2 = __shfl_up(B2, 1, 64);
    if (multi) put(sf, join ? f0 + in0 : f0, join ? f1 + in1 : f1, join ? f2 + in2 : f2);
    const int sf_next = __shfl_down(sf, 1, 64);
    if (!(lane < 63 && sf_next == sl)) put(sl, B0, B1, B2);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 3 * nsh; i += blockDim.x) {
    double t = sh[i];
    for (int w = 1; w < waves; ++w) t += sh[w * 3 * nsh + i];
    partial[(size_t)blockIdx.x * 3 * nsh + i] = t;
  }
}

template <int N>
hipError_t fsc_run(const float2* g1, const float2* g2, int dims, int part, float s1, float s2, float2* X,
                   const float2* tw_row, const float2* tw_col, const float2* twn, double* partial, double* out,
                   hipStream_t st) {
  using R = FscRowCfg<N>;
  using C = ColCfg<N>;
  const size_t rows = dims == 3 ? (size_t)N * N : (size_t)N;
  hipLaunchKernelGGL((fsc_rows_kernel<N>), dim3((unsigned)(rows / R::RW)), dim3(R::T * R::RW), 0, st, g1, g2, part, s1,
                     s2, (float4*)X, tw_row, twn);
  const int tiles = N / C::WA, planes = dims == 3 ? N : 1;
  hipLaunchKernelGGL((fsc_cols_kernel<N>), dim3(tiles * planes), dim3(C::T * C::WA), 0, st, X, (size_t)N,
                     (size_t)N * N, tiles, tw_col, twn);
  if (dims == 3)
    hipLaunchKernelGGL((fsc_cols_kernel<N>), dim3(tiles * N), dim3(C::T * C::WA), 0, st, X, (size_t)N * N, (size_t)0,
                       tiles * N, tw_col, twn);
  // four elements per lane where 256 divides n/2, else one (64 divides n/2 from n = 128)
  constexpr int K = N >= 512 ? 4 : 1, H = N / 2;
  const int threads = N > 1024 ? kFscThreads / 2 : kFscThreads, waves = threads / 64;
  const size_t lds = sizeof(double) * waves * 3 * (H + 1);
  const int chunks = (dims == 3 ? (H + 1) * (H + 1) : H + 1) * (H / (64 * K));
  // a wave takes four chunks or more, up to three workgroups per CU: fewer rows of partials for small inputs
  const int blocks = std::min(fsc_blocks(), (chunks + 4 * waves - 1) / (4 * waves));
  if (dims == 3)
    hipLaunchKernelGGL((fsc_shell_kernel<N, K, 3>), dim3(blocks), dim3(threads), lds, st, (const float4*)X, partial);
  else
    hipLaunchKernelGGL((fsc_shell_kernel<N, K, 2>), dim3(blocks), dim3(threads), lds, st, (const float4*)X, partial);
  if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  return launch_sum_rows(partial, blocks, 3 * (H + 1), out, st);
}

}  // namespace

// three 49 KB workgroups per CU: one round over the 256 CUs
int fsc_blocks() { return 768; }

hipError_t launch_fsc(const float2* g1, const float2* g2, int n, int dims, int part, float s1, float s2, float2* X,
                      const float2* tw_row, const float2* tw_col, const float2* twn, double* partial, double* out,
                      hipStream_t st) {
  switch (n) {
    case 128: return fsc_run<128>(g1, g2, dims, part, s1, s2, X, tw_row, tw_col, twn, partial, out, st);
    case 256: return fsc_run<256>(g1, g2, dims, part, s1, s2, X, tw_row, tw_col, twn, partial, out, st);
    case 512: return fsc_run<512>(g1, g2, dims, part, s1, s2, X, tw_row, tw_col, twn, partial, out, st);
    case 1024: return fsc_run<1024>(g1, g2, dims, part, s1, s2, X, tw_row, tw_col, twn, partial, out, st);
    case 2048: return fsc_run<2048>(g1, g2, dims, part, s1, s2, X, tw_row, tw_col, twn, partial, out, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pwf
