// Bandwidth-bound kernels of the path: the MPO mixing stage of H_eff and of
// the environment updates, and the Lanczos vector operations (dot products,
// classical Gram-Schmidt updates, norms) with fixed-order reductions so that
// every result is bitwise reproducible from run to run.
#include "internal.h"

namespace tna {
namespace {

constexpr int NT = 256;
constexpr int MAXPART = 512;  // partial sums per reduction

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// sum over the 256 threads of a block, fixed order; result valid in thread 0
__device__ inline double block_sum(double v, double *sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0) r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return r;
}

int n_parts(int64_t n) {
  int64_t g = (n + 4095) / 4096;
  if (g < 1) g = 1;
  if (g > MAXPART) g = MAXPART;
  return (int)g;
}

// ------------------------------------------------------------------ mixing
struct MixDev {
  int n0, n1, I1, I2, J1, J2, ich1, ich2, och1, och2;
  int64_t is0, is1, os0, os1;
  const void *in;
  void *out;
  const double *M;
};

// One thread per (o0, o1).  Every thread of the launch reads M at the same addresses: through the
// constant address space those are scalar loads shared by the wave.  The channel counts are template
// constants for the MPOs in use: as the guarded 32 x 32 products of run-time counts, with a scalar load waited
// for in each, they took 34 us for the 256 elements of a chi = 16 bond.
// SPLIT: one j1 per grid row instead of all (CJ1 times the threads, x read as often): a launch with fewer
// blocks than keep the chip busy is bound by each thread's walk over M (203 x 331, 32 channels: 33 us
// without, 20 us with).
template <typename T, int CI1, int CI2, int CJ1, int CJ2, bool SPLIT>
__global__ __launch_bounds__(NT) void mix_kernel(MixDev a) {
  constexpr int I = CI1 * CI2, J = SPLIT ? CJ2 : CJ1 * CJ2;
  const int j1 = SPLIT ? blockIdx.y : 0;
  const int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x;
  const int64_t total = (int64_t)a.n0 * a.n1;
  if (idx >= total) return;
  const int64_t o0 = idx / a.n1, o1 = idx - o0 * a.n1;
  const T *in = static_cast<const T *>(a.in) + o0 * a.is0 + o1 * a.is1;
  T *out = static_cast<T *>(a.out) + o0 * a.os0 + o1 * a.os1;
  const double __attribute__((address_space(4))) *M =
      (const double __attribute__((address_space(4))) *)a.M + (SPLIT ? j1 * CJ2 * I : 0);
  if (SPLIT) out += (int64_t)j1 * a.och1;
  T x[I];
#pragma unroll
  for (int i = 0; i < I; ++i) x[i] = in[(i / CI2) * a.ich1 + (i % CI2) * a.ich2];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    T acc = T(0);
#pragma unroll
    for (int i = 0; i < I; ++i) acc += (T)M[j * I + i] * x[i];
    out[(j / CJ2) * a.och1 + (j % CJ2) * a.och2] = acc;
  }
}

// The same for any channel counts up to 32.  M goes through LDS, its rows filled up with zeros to 32 entries, so
// that a row's products need a bound only every four channels and no load is waited for alone; the
// channel offsets are stepped, not divided.
// H_eff of 203 x 331 with it, and with divided offsets and scalar loads of M: d = 2, D = 7, FP64 106 / 149 us;
// d = 1, D = 32 274 / 323 us; 4 x 4 with d = 3, D = 3 in FP32 23.9 / 60 us.
template <typename T>
__global__ __launch_bounds__(NT) void mix_any_kernel(MixDev a) {
  constexpr int CH = 32;
  __shared__ T Ms[CH * CH];
  const int I = a.I1 * a.I2, J = a.J1 * a.J2;
  for (int e = threadIdx.x; e < J * CH; e += NT) {
    const int j = e / CH, i = e % CH;
    Ms[e] = i < I ? (T)a.M[j * I + i] : T(0);
  }
  __syncthreads();
  const int64_t idx = (int64_t)blockIdx.x * NT + threadIdx.x;
  const int64_t total = (int64_t)a.n0 * a.n1;
  if (idx >= total) return;
  const int64_t o0 = idx / a.n1, o1 = idx - o0 * a.n1;
  const T *in = static_cast<const T *>(a.in) + o0 * a.is0 + o1 * a.is1;
  T *out = static_cast<T *>(a.out) + o0 * a.os0 + o1 * a.os1;
  T x[CH];
  int c2 = 0, at = 0;  // channel (c1, c2) and its offset
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    x[i] = i < I ? in[at] : T(0);
    c2 = c2 + 1 < a.I2 ? c2 + 1 : 0;
    at += c2 > 0 ? a.ich2 : a.ich1 - (a.I2 - 1) * a.ich2;
  }
  c2 = at = 0;
#pragma unroll 1
  for (int j = 0; j < J; ++j) {
    T acc = T(0);
#pragma unroll
    for (int i0 = 0; i0 < CH; i0 += 4)
      if (i0 < I)  // uniform
#pragma unroll
        for (int i = i0; i < i0 + 4; ++i) acc += Ms[j * CH + i] * x[i];
    out[at] = acc;
    c2 = c2 + 1 < a.J2 ? c2 + 1 : 0;
    at += c2 > 0 ? a.och2 : a.och1 - (a.J2 - 1) * a.och2;
  }
}

__global__ void build_mix_kernel(int mode, int d, int D, const double *W1, const double *W2, double *M) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (mode == 0) {
    const int I = D * d * d, J = d * d * D;
    if (t >= I * J) return;
    const int j = t / I, i = t % I;
    const int s = j / (d * D), tt = (j / D) % d, wq = j % D;
    const int w = i / (d * d), sp = (i / d) % d, tp = i % d;
    double acc = 0.0;
    for (int wp = 0; wp < D; ++wp)
      acc += W1[((w * D + wp) * d + s) * d + sp] * W2[((wp * D + wq) * d + tt) * d + tp];
    M[t] = acc;
  } else {
    const int I = D * d, J = d * D;
    if (t >= I * J) return;
    const int j = t / I, i = t % I;
    const int s = j / D, wo = j % D;  // output (s, w') or (t, w)
    const int wi = i / d, sp = i % d;  // input (w, s') or (w'', t')
    // mode 1: W[w_in][w_out][s][s']   mode 2: W[w_out][w_in][t][t']
    M[t] = (mode == 1) ? W1[((wi * D + wo) * d + s) * d + sp] : W1[((wo * D + wi) * d + s) * d + sp];
  }
}

// ------------------------------------------------------------------ reductions
__global__ __launch_bounds__(NT) void multidot_kernel(const double *V, int64_t ldv, int nv, const double *w,
                                                      int64_t n, double *part) {
  __shared__ double sh[4];
  const int G = gridDim.x;
  const int64_t chunk = (n + G - 1) / G;
  const int64_t beg = chunk * blockIdx.x;
  const int64_t end = beg + chunk < n ? beg + chunk : n;
  for (int i0 = 0; i0 < nv; i0 += 8) {
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t e = beg + threadIdx.x; e < end; e += NT) {
      const double wv = w[e];
#pragma unroll
      for (int g = 0; g < 8; ++g)
        if (i0 + g < nv) acc[g] += V[(int64_t)(i0 + g) * ldv + e] * wv;
    }
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      if (i0 + g < nv) {  // uniform
        double r = block_sum(acc[g], sh);
        if (threadIdx.x == 0) part[(int64_t)(i0 + g) * G + blockIdx.x] = r;
      }
    }
  }
}

// h[i] = <V_i, w> with one block per vector (short vectors), fixed order
__global__ __launch_bounds__(NT) void multidot_small_kernel(const double *V, int64_t ldv, const double *w, int64_t n,
                                                            double *h) {
  __shared__ double sh[4];
  const int i = blockIdx.x;
  const double *v = V + (int64_t)i * ldv;
  double acc = 0.0;
  for (int64_t e = threadIdx.x; e < n; e += NT) acc += v[e] * w[e];
  acc = block_sum(acc, sh);
  if (threadIdx.x == 0) h[i] = acc;
}

// out[i] = sum_b part[i*G + b], one block per i, fixed tree
__global__ __launch_bounds__(NT) void reduce_parts_kernel(const double *part, int G, double *out) {
  __shared__ double sh[4];
  const int i = blockIdx.x;
  double v = 0.0;
  for (int b = threadIdx.x; b < G; b += NT) v += part[(int64_t)i * G + b];
  v = block_sum(v, sh);
  if (threadIdx.x == 0) out[i] = v;
}

__global__ __launch_bounds__(NT) void axpy_multi_kernel(const double *V, int64_t ldv, int nv, const double *h,
                                                        double *w, int64_t n, double *part) {
  __shared__ double sh[4];
  const int G = gridDim.x;
  const int64_t chunk = (n + G - 1) / G;
  const int64_t beg = chunk * blockIdx.x;
  const int64_t end = beg + chunk < n ? beg + chunk : n;
  double loc = 0.0;
  for (int64_t e = beg + threadIdx.x; e < end; e += NT) {
    double acc = 0.0;
    for (int i = 0; i < nv; ++i) acc += h[i] * V[(int64_t)i * ldv + e];
    const double v = w[e] - acc;
    w[e] = v;
    loc += v * v;
  }
  if (part) {
    double r = block_sum(loc, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = r;
  }
}

__global__ __launch_bounds__(NT) void combine_kernel(const double *V, int64_t ldv, int nv, const double *c,
                                                     double *y, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) {
    double acc = 0.0;
    for (int i = 0; i < nv; ++i) acc += c[i] * V[(int64_t)i * ldv + e];
    y[e] = acc;
  }
}

__global__ __launch_bounds__(NT) void norm2_kernel(const double *x, int64_t n, double *part) {
  __shared__ double sh[4];
  const int G = gridDim.x;
  const int64_t chunk = (n + G - 1) / G;
  const int64_t beg = chunk * blockIdx.x;
  const int64_t end = beg + chunk < n ? beg + chunk : n;
  double loc = 0.0;
  for (int64_t e = beg + threadIdx.x; e < end; e += NT) loc += x[e] * x[e];
  double r = block_sum(loc, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = r;
}

__global__ __launch_bounds__(NT) void scale_kernel(const double *x, double *y, int64_t n, const double *nrm2,
                                                   double scal) {
  const double f = nrm2 ? 1.0 / sqrt(*nrm2) : scal;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) y[e] = x[e] * f;
}

__global__ __launch_bounds__(NT) void finite_kernel(const double *x, int64_t n, int *flag) {
  int bad = 0;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT)
    bad |= !isfinite(x[e]);
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicAdd(flag, 1);
}

__global__ __launch_bounds__(NT) void cvt_kernel(const double *x, float *y, int64_t n) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) y[e] = (float)x[e];
}

__global__ __launch_bounds__(NT) void fill_kernel(double *x, int64_t n, double v) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) x[e] = v;
}

__global__ __launch_bounds__(NT) void fill_int_kernel(int *x, int64_t n, int v) {
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) x[e] = v;
}

template <typename T>
__global__ __launch_bounds__(NT) void transpose_kernel(const T *A, int m, int n, double *B) {
  __shared__ double tile[32][33];
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;  // bx over n, by over m
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    int i = by + r, j = bx + tx;
    tile[r][tx] = (i < m && j < n) ? (double)A[(int64_t)i * n + j] : 0.0;
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    int j = bx + r, i = by + tx;
    if (j < n && i < m) B[(int64_t)j * m + i] = tile[tx][r];
  }
}

__global__ __launch_bounds__(NT) void identity_kernel(double *J, int n, int ld, int64_t stride) {
  double *Jb = J + stride * blockIdx.y;
  const int64_t total = (int64_t)n * ld;
  for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < total; e += (int64_t)gridDim.x * NT) {
    int64_t r = e / ld, c = e - r * ld;
    Jb[e] = (r == c) ? 1.0 : 0.0;
  }
}

int grid_for(int64_t n) {
  int64_t g = (n + NT - 1) / NT;
  if (g < 1) g = 1;
  if (g > 4096) g = 4096;
  return (int)g;
}

}  // namespace

// ---------------------------------------------------------------------- API
tna_status mix(const MixArgs &a, hipStream_t s) {
  const int I = a.I1 * a.I2, J = a.J1 * a.J2;
  if (I < 1 || I > 32 || J < 1 || J > 32 || a.n0 < 0 || a.n1 < 0) {
    set_error("mix: bad channel count");
    return TNA_ERR_ARG;
  }
  int64_t total = (int64_t)a.n0 * a.n1;
  if (total == 0) return TNA_OK;
  const MixDev d{a.n0, a.n1, a.I1, a.I2, a.J1, a.J2, a.ich1, a.ich2, a.och1, a.och2, a.is0, a.is1, a.os0, a.os1,
                 a.in, a.out, a.M};
  dim3 grid((unsigned)((total + NT - 1) / NT));
  const char *name = a.type_in == G_F64 ? "mix.f64" : "mix.f32";
  timer_begin(name, s);
  if (a.type_in != a.type_out) {
    set_error("mix: type combination not built");
    return TNA_ERR_UNSUPPORTED;
  }
  const bool split = grid.x < 1024;  // fewer than four blocks per compute unit
  auto launch = [&](auto kd, auto kf, bool rows) {
    const dim3 g(grid.x, rows ? a.J1 : 1);
    if (a.type_in == G_F64) hipLaunchKernelGGL(kd, g, dim3(NT), 0, s, d);
    else hipLaunchKernelGGL(kf, g, dim3(NT), 0, s, d);
  };
#define TNA_MIX_CASE(b, c, e, f)                                                                        \
  if (a.I1 == b && a.I2 == c && a.J1 == e && a.J2 == f) {                                             \
    if (split) launch(mix_kernel<double, b, c, e, f, true>, mix_kernel<float, b, c, e, f, true>, true); \
    else launch(mix_kernel<double, b, c, e, f, false>, mix_kernel<float, b, c, e, f, false>, false);    \
  } else
  TNA_MIX_CASE(5, 4, 4, 5)
  TNA_MIX_CASE(5, 2, 2, 5)
  TNA_MIX_CASE(8, 4, 4, 8)
  TNA_MIX_CASE(8, 2, 2, 8)
  TNA_MIX_CASE(3, 4, 4, 3)
  TNA_MIX_CASE(3, 2, 2, 3)
  launch(mix_any_kernel<double>, mix_any_kernel<float>, false);
#undef TNA_MIX_CASE
  const int es = a.type_in == G_F64 ? 8 : 4;
  timer_end(name, 2.0 * I * J * (double)total, (double)total * (I + J) * es, s);
  TNA_LAUNCHED("vec.hip:1");
  return TNA_OK;
}

tna_status build_mix_matrix(int mode, int d, int D, const double *W1, const double *W2, double *M, hipStream_t s) {
  int n = (mode == 0) ? (D * d * d) * (D * d * d) : (D * d) * (D * d);
  hipLaunchKernelGGL(build_mix_kernel, dim3((n + 255) / 256), dim3(256), 0, s, mode, d, D, W1, W2, M);
  TNA_LAUNCHED("vec.hip:2");
  return TNA_OK;
}

tna_status multidot(const double *V, int64_t ldv, int nv, const double *w, int64_t n, double *h, double *part,
                    hipStream_t s) {
  if (nv <= 0) return TNA_OK;
  int G = n_parts(n);
  if (n <= 65536) {  // short vectors: a block per vector, no second pass
    timer_begin("vec.multidot", s);
    hipLaunchKernelGGL(multidot_small_kernel, dim3(nv), dim3(NT), 0, s, V, ldv, w, n, h);
    timer_end("vec.multidot", 2.0 * nv * (double)n, 8.0 * (nv + 1) * (double)n, s);
    TNA_LAUNCHED("vec.multidot");
    return TNA_OK;
  }
  timer_begin("vec.multidot", s);
  hipLaunchKernelGGL(multidot_kernel, dim3(G), dim3(NT), 0, s, V, ldv, nv, w, n, part);
  timer_end("vec.multidot", 2.0 * nv * (double)n, 8.0 * (nv + 1) * (double)n, s);
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(nv), dim3(NT), 0, s, part, G, h);
  TNA_LAUNCHED("vec.hip:3");
  return TNA_OK;
}

tna_status axpy_multi(const double *V, int64_t ldv, int nv, const double *h, double *w, int64_t n, double *nrm2,
                      double *part, hipStream_t s) {
  int G = n_parts(n);
  timer_begin("vec.axpy", s);
  hipLaunchKernelGGL(axpy_multi_kernel, dim3(G), dim3(NT), 0, s, V, ldv, nv, h, w, n, nrm2 ? part : nullptr);
  timer_end("vec.axpy", 2.0 * nv * (double)n, 8.0 * (nv + 2) * (double)n, s);
  if (nrm2) hipLaunchKernelGGL(reduce_parts_kernel, dim3(1), dim3(NT), 0, s, part, G, nrm2);
  TNA_LAUNCHED("vec.hip:4");
  return TNA_OK;
}

tna_status combine(const double *V, int64_t ldv, int nv, const double *c, double *y, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(combine_kernel, dim3(grid_for(n)), dim3(NT), 0, s, V, ldv, nv, c, y, n);
  TNA_LAUNCHED("vec.hip:5");
  return TNA_OK;
}

tna_status norm2(const double *x, int64_t n, double *out, double *part, hipStream_t s) {
  int G = n_parts(n);
  hipLaunchKernelGGL(norm2_kernel, dim3(G), dim3(NT), 0, s, x, n, part);
  hipLaunchKernelGGL(reduce_parts_kernel, dim3(1), dim3(NT), 0, s, part, G, out);
  TNA_LAUNCHED("vec.hip:6");
  return TNA_OK;
}

tna_status scale(const double *x, double *y, int64_t n, const double *nrm2, double scal, hipStream_t s) {
  hipLaunchKernelGGL(scale_kernel, dim3(grid_for(n)), dim3(NT), 0, s, x, y, n, nrm2, scal);
  TNA_LAUNCHED("vec.hip:7");
  return TNA_OK;
}

tna_status check_finite(const double *x, int64_t n, int *flag, hipStream_t s) {
  hipLaunchKernelGGL(finite_kernel, dim3(grid_for(n)), dim3(NT), 0, s, x, n, flag);
  TNA_LAUNCHED("vec.hip:8");
  return TNA_OK;
}

tna_status convert_f64_f32(const double *x, float *y, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(cvt_kernel, dim3(grid_for(n)), dim3(NT), 0, s, x, y, n);
  TNA_LAUNCHED("vec.hip:9");
  return TNA_OK;
}

tna_status fill(double *x, int64_t n, double v, hipStream_t s) {
  if (n <= 0) return TNA_OK;
  hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(NT), 0, s, x, n, v);
  TNA_LAUNCHED("vec.hip:10");
  return TNA_OK;
}

tna_status fill_int(int *x, int64_t n, int v, hipStream_t s) {
  if (n <= 0) return TNA_OK;
  hipLaunchKernelGGL(fill_int_kernel, dim3(grid_for(n)), dim3(NT), 0, s, x, n, v);
  TNA_LAUNCHED("vec.hip:11");
  return TNA_OK;
}

tna_status copy_transpose(const void *A, int m, int n, int type, double *B, hipStream_t s) {
  dim3 grid((n + 31) / 32, (m + 31) / 32);
  if (type == G_F64)
    hipLaunchKernelGGL(transpose_kernel<double>, grid, dim3(NT), 0, s, static_cast<const double *>(A), m, n, B);
  else
    hipLaunchKernelGGL(transpose_kernel<float>, grid, dim3(NT), 0, s, static_cast<const float *>(A), m, n, B);
  TNA_LAUNCHED("vec.hip:12");
  return TNA_OK;
}

tna_status set_identity(double *J, int n, int ld, int batch, int64_t stride, hipStream_t s) {
  int64_t total = (int64_t)n * ld;
  dim3 grid((unsigned)grid_for(total), batch);
  hipLaunchKernelGGL(identity_kernel, grid, dim3(NT), 0, s, J, n, ld, stride);
  TNA_LAUNCHED("vec.hip:13");
  return TNA_OK;
}

}  // namespace tna
