// The two-site effective Hamiltonian (Eq. 18) of short bonds in one launch.
//
//   X[(a,w)][(s',t',c')] = sum_a' L[a][w][a'] theta[a'][(s',t',c')]
//   Z[(a,s,t)][(w'',c')] = sum_i M[(s,t,w'')][i] X[a][i][c'],  i = (w,s',t')
//   out[(a,s,t)][c]      = sum_(w'',c') Z[(a,s,t)][(w'',c')] R[c][(w'',c')]
//
// A left index a needs nothing from the others beyond theta and R, so a workgroup takes `ac` of them
// (as many as fill one 16-row MFMA tile of each product) through all three steps: its rows of L, M
// (formed from W1 and W2 in place), X and Z stay in LDS, theta and R are read from L2 as MFMA operands.
// Products run in the order of the general path (k ascending in steps of four, one accumulator; the
// mixing sum over i ascending), so both give the same bits, in FP64 and in the FP32-operator form.
// Bound by latency: operand loads of a tile, then few waves for the last product's chr / 16 tiles.
// D = 5, FP64: 7.5 us a call at chi = 16 (15 us in four launches, 44 us before the mixing had
// compile-time channel counts), 17.5 us at 48 (18.6 us).
#include <algorithm>
#include <cstdint>

#include "dev_tile.h"
#include "internal.h"

namespace tna {
namespace {

constexpr int NT = 512;  // eight waves: their operand loads in flight hide each other's latency

struct HeffSmall {
  int chl, chr, D, ac;
  const double *L, *W1, *W2, *R, *theta;
  double *out;
};

// odd strides: sixteen lanes reading down the rows of an MFMA operand fall on distinct LDS banks
__host__ __device__ inline int odd(int x) { return x | 1; }
__host__ __device__ inline size_t lds_elems(int chl, int chr, int D, int ac) {
  const int I = 4 * D;
  return (size_t)ac * D * odd(chl) + (size_t)I * I + (size_t)ac * I * chr + (size_t)ac * 4 * odd(D * chr);
}

// One 16 x 16 tile, C(i, j) = sum_k A(i, k) B(k, j), k ascending.  Lane (lr, lk) supplies A(lr, k + lk)
// (LDS) and B(k + lk, lr) (device memory); B of the next UN steps is loaded while the current ones are
// multiplied.
template <class T, class FA, class FB>
__device__ __forceinline__ typename Mma<T>::acc tile(int K, int lk, FA a_at, FB b_at) {
  constexpr int UN = 16;
  typename Mma<T>::acc c = {0, 0, 0, 0};
  T b[UN], nb[UN];
  auto load = [&](T(&v)[UN], int k0) {
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int k = k0 + 4 * u + lk;
      v[u] = k < K ? (T)b_at(k) : T(0);
    }
  };
  load(b, 0);
  for (int k0 = 0; k0 < K; k0 += 4 * UN) {
    if (k0 + 4 * UN < K) load(nb, k0 + 4 * UN);
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int k = k0 + 4 * u + lk;
      if (k0 + 4 * u < K) c = Mma<T>::step(k < K ? a_at(k) : T(0), b[u], c);
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) b[u] = nb[u];
  }
  return c;
}

// CD: the MPO's bond dimension where it is one of those in use (0: p.D)
template <class T, int CD>
__global__ __launch_bounds__(NT) void heff_small_kernel(HeffSmall p) {
  extern __shared__ double lds_raw[];
  const int chl = p.chl, chr = p.chr, D = CD > 0 ? CD : p.D, I = 4 * D, N1 = 4 * chr, K3 = D * chr;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int a0 = blockIdx.x * p.ac, na = min(p.ac, chl - a0);
  const int ldl = odd(chl), ldz = odd(K3);
  T *Ls = reinterpret_cast<T *>(lds_raw);  // rows (a, w)
  T *Ms = Ls + p.ac * D * ldl;             // rows (s, t, w'')
  T *Xs = Ms + I * I;                      // [al][i][c']
  T *Zs = Xs + (size_t)p.ac * I * chr;     // rows (al, s, t)
  for (int e = tid; e < na * D * chl; e += NT) Ls[(e / chl) * ldl + e % chl] = (T)p.L[(size_t)a0 * D * chl + e];
  for (int e = tid; e < I * I; e += NT) {
    const int j = e / I, i = e - j * I;
    const int s = j / (2 * D), t = (j / D) & 1, wq = j % D;
    const int w = i >> 2, sp = (i >> 1) & 1, tp = i & 1;
    double acc = 0.0;
    for (int wp = 0; wp < D; ++wp)
      acc += p.W1[((w * D + wp) * 2 + s) * 2 + sp] * p.W2[((wp * D + wq) * 2 + t) * 2 + tp];
    Ms[e] = (T)acc;
  }
  __syncthreads();
  const int r1 = min(lr, na * D - 1), r3 = min(lr, na * 4 - 1);
  for (int j0 = 16 * wave; j0 < N1; j0 += NT / 4) {  // X: rows al D + w, columns (s', t', c')
    const int j = j0 + lr, jc = min(j, N1 - 1);
    const typename Mma<T>::acc c = tile<T>(
        chl, lk, [&](int k) { return Ls[r1 * ldl + k]; }, [&](int k) { return (T)p.theta[(size_t)k * N1 + jc]; });
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = Mma<T>::row(lk, r);
      if (row < na * D && j < N1) Xs[row * N1 + j] = c[r];  // al I chr + (4 w + s't') chr + c'
    }
  }
  __syncthreads();
  {  // Z: a wave takes one (s, t), its rows of M (the same for every lane) against EL columns (al, c') a lane
    constexpr int EL = 2, DM = CD > 0 ? CD : 8;
    const int nac = na * chr, st = wave & 3, part = wave >> 2, parts = NT / 256;
    const T *Mst = Ms + st * D * I;
    for (int x0 = part * 64 * EL; x0 < nac; x0 += parts * 64 * EL) {
      T acc[EL][DM];
      const T *xi[EL];
      int zo[EL];
#pragma unroll
      for (int e = 0; e < EL; ++e) {
        const int x = x0 + 64 * e + lane, xc = x < nac ? x : nac - 1, al = xc / chr, cc = xc - al * chr;
        xi[e] = Xs + al * I * chr + cc;
        zo[e] = x < nac ? (al * 4 + st) * ldz + cc : -1;
#pragma unroll
        for (int u = 0; u < DM; ++u) acc[e][u] = T(0);
      }
#pragma unroll 4
      for (int i = 0; i < I; ++i) {
        T v[EL];
#pragma unroll
        for (int e = 0; e < EL; ++e) v[e] = xi[e][i * chr];
#pragma unroll
        for (int u = 0; u < DM; ++u)
          if (CD > 0 || u < D) {
            const T m = Mst[u * I + i];
#pragma unroll
            for (int e = 0; e < EL; ++e) acc[e][u] += m * v[e];
          }
      }
#pragma unroll
      for (int e = 0; e < EL; ++e)
        if (zo[e] >= 0)
#pragma unroll
          for (int u = 0; u < DM; ++u)
            if (CD > 0 || u < D) Zs[zo[e] + u * chr] = acc[e][u];
    }
  }
  __syncthreads();
  for (int j0 = 16 * wave; j0 < chr; j0 += NT / 4) {  // out: rows al 4 + st, columns c
    const int j = j0 + lr, jc = min(j, chr - 1);
    const typename Mma<T>::acc c = tile<T>(
        K3, lk, [&](int k) { return Zs[r3 * ldz + k]; }, [&](int k) { return (T)p.R[(size_t)jc * K3 + k]; });
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = Mma<T>::row(lk, r);
      if (row < na * 4 && j < chr) p.out[((size_t)a0 * 4 + row) * chr + j] = (double)c[r];
    }
  }
}

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + nb && y < x + na;
}

}  // namespace

bool heff_small_takes(int chl, int chr, int d, int D, const double *L, const double *W1, const double *W2,
                      const double *R, const double *theta, const double *out, int prec) {
  if (d != 2 || D < 1 || D > 8 || !heff_small_bond(chl, chr)) return false;
  if (prec != TNA_HEFF_F64 && prec != TNA_HEFF_F32) return false;
  // the general path has read L, W1 and W2 whole before it writes out; a caller may rely on that
  const size_t w = sizeof(double) * 4 * (size_t)D * D, no = sizeof(double) * 4 * (size_t)chl * chr;
  return !overlap(out, no, L, sizeof(double) * (size_t)chl * D * chl) && !overlap(out, no, W1, w) &&
         !overlap(out, no, W2, w) && !overlap(out, no, R, sizeof(double) * (size_t)chr * D * chr) &&
         !overlap(out, no, theta, no);
}

tna_status heff_small(int chl, int chr, int D, const double *L, const double *W1, const double *W2, const double *R,
                      const double *theta, double *out, int prec, hipStream_t s) {
  HeffSmall p{chl, chr, D, std::min(std::max(1, 16 / D), 4), L, W1, W2, R, theta, out};
  const size_t es = prec == TNA_HEFF_F64 ? sizeof(double) : sizeof(float);
  const size_t lds = es * lds_elems(chl, chr, D, p.ac);
  const dim3 grid((chl + p.ac - 1) / p.ac);
  timer_begin("heff.small", s);
  auto go = [&](auto fn) -> tna_status {
    if (lds > 64 * 1024)
      TNA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds));
    hipLaunchKernelGGL(fn, grid, dim3(NT), lds, s, p);
    return TNA_OK;
  };
  auto by_d = [&](auto t) -> tna_status {
    using T = decltype(t);
    switch (D) {
      case 3: return go(heff_small_kernel<T, 3>);
      case 5: return go(heff_small_kernel<T, 5>);
      case 8: return go(heff_small_kernel<T, 8>);
      default: return go(heff_small_kernel<T, 0>);
    }
  };
  TNA_TRY(prec == TNA_HEFF_F64 ? by_d(0.0) : by_d(0.0f));
  const double n = (double)chl * chr;
  timer_end("heff.small", 8.0 * D * n * (chl + chr) + 32.0 * D * D * n,
            8.0 * ((double)D * (chl * (double)chl + chr * (double)chr) + 8.0 * n), s);
  TNA_LAUNCHED("heff.small");
  return TNA_OK;
}

}  // namespace tna
