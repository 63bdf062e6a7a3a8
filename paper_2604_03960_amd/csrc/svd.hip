// Truncated SVD (Eq. 3 / Eq. 19) by blocked one-sided Jacobi on gfx950, and
// the spectrum sums of Eq. (4)-(5).
//
// The R = min(m,n) rows of length C = max(m,n) of A (or of A^T when m > n)
// are orthogonalised; the product of the rotations is accumulated in Jt
// (R x R, starts at I).  Rows are grouped in blocks of 32; one Jacobi sweep
// visits every pair of blocks once in round-robin order (nb-1 steps of nb/2
// disjoint pairs).  Per step three launches:
//   gram   G = [B_p; B_q][B_p; B_q]^T (64 x 64) on the FP64 MFMA, K split
//          across workgroups, partial sums in fixed order;
//   eigen  a two-sided Jacobi sweep of the 64 x 64 symmetric G in registers
//          (odd-even transposition order), eigenvectors sorted by eigenvalue
//          (larger rows to the lower block); skipped when every off-diagonal
//          already satisfies |g_ij| <= tol sqrt(g_ii g_jj);
//   apply  [B_p; B_q] <- Q^T [B_p; B_q] and [J_p; J_q] <- Q^T [J_p; J_q] on the
//          MFMA, column slab by column slab, in place.
// A sweep with no rotating pair ends the iteration (one 4-byte host read per
// sweep).  Afterwards sigma_r = |row r|, a bitonic sort orders them, and the
// factors are written with the sign gauge (largest-magnitude entry of each
// left vector positive) and Gram-Schmidt completion of null vectors.
#include <hip/hip_cooperative_groups.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "dev_reduce.h"
#include "dev_tile.h"
#include "internal.h"

namespace tna {

tna_status DevBuf::ensure(size_t need) {
  if (need <= bytes) return TNA_OK;
  if (borrowed) {
    set_error("workspace too small for this call");
    return TNA_ERR_NOMEM;
  }
  release();
  size_t want = need + need / 4;
  if (hipMalloc(&ptr, want) != hipSuccess) {
    ptr = nullptr;
    bytes = 0;
    set_error("device allocation failed");
    return TNA_ERR_NOMEM;
  }
  bytes = want;
  return TNA_OK;
}

void DevBuf::release() {
  if (ptr && !borrowed) (void)hipFree(ptr);
  ptr = nullptr;
  bytes = 0;
  borrowed = false;
}

namespace {

// Jacobi rotation (c, s) zeroing the off-diagonal g of a symmetric 2 x 2 block [[a, g], [g, b]], by its half angle:
// cos 2u = |b - a| / sqrt((b - a)^2 + 4 g^2), c = sqrt((1 + cos 2u) / 2), two reciprocal square roots long, with
// tg = (s / c) g for the new diagonal (a - tg, b + tg).  Identity (c, s, tg = 1, 0, 0) where a row is at or below
// floor2 or the coupling is at the rounding level.  It is a chain of dependent operations cut into eight stages, so
// that a caller can issue other work between them; each reciprocal square root takes the hardware estimate y
// (relative error below 2^-22) and one third-order step y (1 + e/2 + 3 e^2/8), e = 1 - x y^2, which cubes the
// error: c^2 + s^2 = 1 to a few ulp without the long correctly rounded division and square-root sequences.
// The rotation depends on the ratios of a, b and g alone, so they are first multiplied by the power of two that
// brings the largest into [1, 2) (exact): the squares of squared norms would underflow for rows of norm
// 1e-77 (also for a block of such rows in a matrix of norm 1) and overflow at 1e77.  The eigen step of 331 x 517 takes
// 36.3 us a launch so, 35.0 without (mean of all sweeps).
struct RotChain {
  double a, b, g;  // inputs: the 2 x 2 block [[a, g], [g, b]]
  double as, bs, gs;  // the block, scaled
  double dl, x, y, e, ir, c2, ic, c, s, tg;
  bool act;
  // g^2 > tol^2 a b
  __device__ __forceinline__ bool coupled(double tol2) const { return gs * gs > tol2 * fabs(as * bs); }
  // (TEST off: the caller decides whether the rotation acts)
  template <int K, bool TEST = true>
  __device__ __forceinline__ void stage(double floor2) {
    constexpr double tol_in = 4.0 * 1.1102230246251565e-16;
    if constexpr (K == 0) {
      constexpr int EXP = 0x7ff00000;
      const int m = max(max(__double2hiint(a) & EXP, __double2hiint(b) & EXP), __double2hiint(g) & EXP);
      const double sc = __hiloint2double(0x7fe00000 - m, 0);  // 2^1023 for an all-zero block
      as = a * sc;
      bs = b * sc;
      gs = g * sc;
      dl = bs - as;
      x = fma(dl, dl, 4.0 * gs * gs);
    } else if constexpr (K == 1) {
      y = __builtin_amdgcn_rsq(x);
      act = TEST ? (a > floor2 && b > floor2 && coupled(tol_in * tol_in)) : true;
    } else if constexpr (K == 2) {
      e = fma(-(x * y), y, 1.0);
    } else if constexpr (K == 3) {
      ir = fma(y * e, fma(0.375, e, 0.5), y);
    } else if constexpr (K == 4) {
      c2 = fma(0.5 * fabs(dl), ir, 0.5);
      s = (dl >= 0.0 ? gs : -gs) * ir;
      y = __builtin_amdgcn_rsq(c2);
    } else if constexpr (K == 5) {
      e = fma(-(c2 * y), y, 1.0);
    } else if constexpr (K == 6) {
      ic = fma(y * e, fma(0.375, e, 0.5), y);
    } else {
      c = act ? c2 * ic : 1.0;
      s = s * ic;
      tg = act ? s * ic * g : 0.0;
      s = act ? s : 0.0;
    }
  }
};

constexpr double EPS53 = 1.1102230246251565e-16;
constexpr int BS = 32;  // rows per block

// v_mfma_f64_16x16x4_f64: A[i][k] in lane i + 16k, B[k][j] in lane j + 16k,
// result D[i][j] in lane j + 16(i%4), register i/4.
__device__ inline v4d mfma16(double a, double b, v4d c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// round-robin pairing of nb blocks (nb even): step s in [0, nb-1), pair t in [0, nb/2)
__device__ inline void rr_pair(int nb, int s, int t, int &p, int &q) {
  const int n1 = nb - 1;
  int a, b;
  if (t == 0) { a = s % n1; b = n1; }
  else { a = (s + t) % n1; b = (s - t + n1) % n1; }
  p = a < b ? a : b;
  q = a < b ? b : a;
}

__device__ inline int block_rows(int R, int blk) {
  int r = R - blk * BS;
  return r < 0 ? 0 : (r > BS ? BS : r);
}

__device__ inline double wave_sum_d(double v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ inline double bsum256(double v, double *red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  const double r = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return r;
}

// -------------------------------------------------------------- gram
// 64 x 64 Gram of the rows of blocks p and q over columns [kb, ke) on MFMA:
// wave (qi, qj) holds the 32 x 32 quadrant (qi, qj) as 2 x 2 16 x 16 tiles.
constexpr int GBK = 64;
// The next 64-column slab (32 KB of the pair's rows) is loaded into registers while the current
// one is multiplied.
__device__ inline void gram_acc(const SvdMat &a, int p, int q, int np, int nq, int64_t kb, int64_t ke,
                                double (*Ts)[65], v4d acc[2][2]) {
  constexpr int RS = 256 / GBK, NU = 64 / RS;  // row stride of a thread's loads, rows per thread
  const double *B = a.bw;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int qi = wave >> 1, qj = wave & 1;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v4d{0, 0, 0, 0};
  // thread tid loads column tid % GBK of rows tid / GBK + RS u, u < NU
  const int col = tid % GBK, r0 = tid / GBK;
  const double *rowp[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int r = r0 + RS * u;
    const bool valid = r < 32 ? (r < np) : (r - 32 < nq);
    const int grow = r < 32 ? p * BS + r : q * BS + (r - 32);
    rowp[u] = valid ? B + (int64_t)grow * a.C : nullptr;
  }
  double nx[NU];
  auto load = [&](int64_t k0) {
    const int64_t gc = k0 + col;
#pragma unroll
    for (int u = 0; u < NU; ++u) nx[u] = (rowp[u] && gc < ke) ? rowp[u][gc] : 0.0;
  };
  if (kb < ke) load(kb);
  for (int64_t k0 = kb; k0 < ke; k0 += GBK) {
#pragma unroll
    for (int u = 0; u < NU; ++u) Ts[col][r0 + RS * u] = nx[u];
    __syncthreads();
    if (k0 + GBK < ke) load(k0 + GBK);  // in flight during the products below
#pragma unroll
    for (int kk = 0; kk < GBK; kk += 4) {
      double av[2], bv[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) av[i] = Ts[kk + lk][32 * qi + 16 * i + lr];
#pragma unroll
      for (int j = 0; j < 2; ++j) bv[j] = Ts[kk + lk][32 * qj + 16 * j + lr];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }
}

// G[row * 64 + col] = acc (f64 result layout)
__device__ inline void gram_store(const v4d acc[2][2], double *G, int ldg) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  const int qi = wave >> 1, qj = wave & 1;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 32 * qi + 16 * i + 4 * r + lk, col = 32 * qj + 16 * j + lr;
        G[row * ldg + col] = acc[i][j][r];
      }
}

// grid (pairs, ksplit, matrices)
__global__ __launch_bounds__(256) void gram_kernel(const SvdMat *mats, int step) {
  __shared__ double Ts[GBK][64 + 1];
  const SvdMat &a = mats[blockIdx.z];
  const int pair = blockIdx.x, ks = blockIdx.y;
  if (!a.active || a.fused || step >= a.nb - 1 || pair >= a.nb / 2 || ks >= a.ksplit) return;
  int p, q;
  rr_pair(a.nb, step, pair, p, q);
  const int np = block_rows(a.Ra, p), nq = block_rows(a.Ra, q);
  int64_t chunk = (a.C + a.ksplit - 1) / a.ksplit;
  chunk = (chunk + GBK - 1) / GBK * GBK;
  const int64_t kb = chunk * ks;
  const int64_t ke = kb + chunk < a.C ? kb + chunk : a.C;
  v4d acc[2][2];
  gram_acc(a, p, q, np, nq, kb, ke, Ts, acc);
  gram_store(acc, a.gram + ((int64_t)pair * a.ksplit + ks) * 4096, 64);
}

// -------------------------------------------------------------- eigen
// Rows whose squared norm is at or below row_floor2 = (0.1 eps C)^2 |A|_F^2 are at the
// rounding level of the rotations: their directions are noise, so pairs with such a
// row are neither tested nor rotated (the relative test could never settle on them).
// Skipping a coupling g_ij <= sigma_i sigma_floor moves sigma_i by at most
// sigma_floor^2 / sigma_i; kept vectors below the floor are completed afterwards.
// After the QR start such rows do settle under the relative test, but only after many
// more sweeps (a numerically low-rank matrix can need twice as many), so the floor is
// used there only when the factor built from the rows leaves scaled by the singular
// values (rows_scaled): then nothing needs their directions.  An input that carries
// noise of noise_rel |A|_F (rows_scaled only) raises the floor to that level.  Otherwise rows after the QR start
// keep their place down to 1e-77 |A|_F: rows at one level that outnumber their columns (what is left of equal
// rows) have to shrink by a rounding a sweep until they are out of the test, from 1e-77 to the end of the range in
// more sweeps than the cap.  Below 1e-150 the Gram's entries lose their digits to underflow.
__device__ inline double row_floor2(const SvdMat &a, double fro2) {
  if (a.precond && !a.rows_scaled) return fmax(1e-154 * fro2, 1e-300);
  const double f = fmax(0.1 * EPS53 * (double)a.C, a.rows_scaled ? a.noise_rel : 0.0);
  return f * f * fro2;
}

// ---- two-sided Jacobi sweep of an N x N Gram held in registers
// Odd-even transposition order: the even rounds rotate the slot pairs (2t, 2t+1), the odd rounds the
// pairs (2t+1, 2t+2), and the two elements of a pair change places after every rotation (also after
// an identity one).  N rounds bring every pair of elements together once and leave the order of
// the slots reversed.  The moves are between neighbours only, so nothing travels through LDS but
// the rotations themselves and, in the odd rounds, the rows at the edges of the row groups.
//
// Layout: lane t of a group of N / 2 lanes holds columns 2t and 2t+1 of the HR rows HR rg ..
// HR rg + HR - 1 of its row group rg, of G and of Q alike (Q's rows stay, its columns move).  An
// even round's column pairs lie inside a lane, an odd round's in neighbouring lanes (two DPP moves
// per value); row pairs lie in registers of one lane except those across two groups.  Every lane
// also carries the diagonal elements of its columns (d0, d1), updated from the rotations (a - t g,
// b + t g), so a round needs one coupling per pair, read in place by the lanes that hold it.  Per
// round: the owners form their pairs' rotations and put them in LDS, one barrier, and every lane
// reads its columns' and its rows' rotations and updates HR x 2 elements of G and of Q.
constexpr int OE_QD = 4;  // of eight rows of Q, those updated behind a round's LDS reads (2, 6, 8: within 3 %)
template <int N, int NW>
struct OeShape {
  static constexpr int LPG = N / 2, GPW = 64 / LPG, NG = NW * GPW, HR = N / NG, PH = HR / 2;
  static_assert(64 % LPG == 0 && N % NG == 0 && HR >= 2 && HR % 2 == 0, "odd-even shape");
};
template <int N, int NW>
struct OeLds {
  // per parity: rotation (c, s) of pair t at [t + 1] and its new diagonal elements, lower slot first;
  // lanes that own no pair write to the 64 entries behind
  double2 cs[2][N / 2 + 1 + 64];
  double2 nd[2][N / 2 + 1 + 64];
  double edge[2][OeShape<N, NW>::NG][N];  // first and last row of every group
};

// value of the next / previous lane (lanes at the ends of a group get another group's value or
// zero, which their identity coefficients discard)
__device__ inline double lane_next(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xf, 0xf, true);  // wave_shl:1
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ inline double lane_prev(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, true);  // wave_shr:1
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// One sweep of N rounds by the whole workgroup (NW waves).  Rows at or below floor2 and pairs whose
// coupling is at the rounding level are not rotated; returns whether this lane's pairs rotated.
// A round's update first brings the couplings of the next round up to date and starts the next
// rotations' dependent chain, whose stages are issued between the updates of the other elements.
template <int N, int NW>
__device__ inline int oe_sweep(OeLds<N, NW> &L, double (&g)[OeShape<N, NW>::HR][2],
                               double (&q)[OeShape<N, NW>::HR][2], double &d0, double &d1, double floor2) {
  using S = OeShape<N, NW>;
  constexpr int HR = S::HR, PH = S::PH, LPG = S::LPG, NG = S::NG;
  constexpr int NST = 8;  // stages of a rotation
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t = lane & (LPG - 1), rg = wave * S::GPW + lane / LPG;
  const int rp = rg > 0 ? rg - 1 : 0, rn = rg < NG - 1 ? rg + 1 : NG - 1;  // neighbouring groups (clamped)
  // even rounds: pair t = slots (2t, 2t+1), row 2t is row 2 (t % PH) of group t / PH;
  // odd rounds: pair t = slots (2t+1, 2t+2), row 2t+2 is row 2 ((t+1) % PH) of group (t+1) / PH
  const bool own0 = t / PH == rg, own1 = t < LPG - 1 && (t + 1) / PH == rg;
  const int w0 = own0 ? t + 1 : N / 2 + 1 + lane, w1 = own1 ? t + 1 : N / 2 + 1 + lane;
  const int k0 = t % PH, k1 = (t + 1) % PH;
  if (threadIdx.x == 0) {  // the edge slots of an odd round sit it out: read after the first barrier below
    L.cs[1][0] = make_double2(0.0, -1.0);
    L.cs[1][N / 2] = make_double2(0.0, 1.0);
  }
  int rot = 0;
  RotChain r;
  // g[2 k][1], k per lane: selected word by word (a select of whole elements becomes a load at a
  // selected address, and the array would leave the registers)
  auto coupling = [&](int k) {
    int lo = __double2loint(g[0][1]), hi = __double2hiint(g[0][1]);
    static_for<1, PH>([&](auto m) {
      lo = k == m ? __double2loint(g[2 * m][1]) : lo;
      hi = k == m ? __double2hiint(g[2 * m][1]) : hi;
    });
    return __hiloint2double(hi, lo);
  };
  r.a = d0;
  r.b = d1;
  r.g = coupling(k0);
  static_for<0, NST>([&](auto st) { r.stage<st>(floor2); });
  // the first QD rows of Q take a round's column rotations in the next round, while its LDS reads
  // are on their way; the others between the stages of the rotation
  constexpr int QD = OE_QD * HR / 8, QI = HR - QD;
  double2 C = make_double2(0.0, 0.0), Cu = make_double2(0.0, -1.0), Cl = make_double2(0.0, 1.0);
  auto q_even = [&](auto i) {
    const double x = q[i][0], y = q[i][1];
    q[i][0] = C.x * y + C.y * x;
    q[i][1] = C.x * x - C.y * y;
  };
  auto q_odd = [&](auto i) {
    const double x = q[i][0], y = q[i][1];
    q[i][0] = Cu.x * lane_prev(y) - Cu.y * x;
    q[i][1] = Cl.x * lane_next(x) + Cl.y * y;
  };
#pragma unroll 1
  for (int rr = 0; rr < N / 2; ++rr) {
    {  // even round
      L.cs[0][w0] = make_double2(r.c, r.s);
      L.nd[0][w0] = make_double2(r.b + r.tg, r.a - r.tg);
      rot |= own0 && r.act;
      __syncthreads();
      const double2 Cn = L.cs[0][t + 1], nd = L.nd[0][t + 1];
      double2 P[PH];
#pragma unroll
      for (int k = 0; k < PH; ++k) P[k] = L.cs[0][rg * PH + k + 1];
      static_for<0, QD>(q_odd);
      __builtin_amdgcn_sched_barrier(0);
      C = Cn;
      d0 = nd.x;
      d1 = nd.y;
      double lo[PH][2];  // rows 2k+1 before the row rotation leaves
#pragma unroll
      for (int k = 0; k < PH; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const double x = g[2 * k][h], y = g[2 * k + 1][h];
          g[2 * k][h] = P[k].x * y + P[k].y * x;
          lo[k][h] = P[k].x * x - P[k].y * y;
        }
#pragma unroll
      for (int k = 0; k < PH; ++k) {  // columns of the rows 2k: the next couplings
        const double x = g[2 * k][0], y = g[2 * k][1];
        g[2 * k][0] = C.x * y + C.y * x;
        g[2 * k][1] = C.x * x - C.y * y;
      }
      r.a = d1;
      r.b = lane_next(d0);
      r.g = coupling(k1);
      static_for<0, NST>([&](auto st) {
        r.stage<st>(floor2);
        __builtin_amdgcn_sched_barrier(0);
        static_for<QD + st * QI / NST, QD + (st + 1) * QI / NST>(q_even);
        static_for<st * PH / NST, (st + 1) * PH / NST>([&](auto k) {
          const double x = lo[k][0], y = lo[k][1];
          g[2 * k + 1][0] = C.x * y + C.y * x;
          g[2 * k + 1][1] = C.x * x - C.y * y;
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    }
    {  // odd round
      L.cs[1][w1] = make_double2(r.c, r.s);
      L.nd[1][w1] = make_double2(r.b + r.tg, r.a - r.tg);
      rot |= own1 && r.act;
      *reinterpret_cast<double2 *>(&L.edge[0][rg][2 * t]) = make_double2(g[0][0], g[0][1]);
      *reinterpret_cast<double2 *>(&L.edge[1][rg][2 * t]) = make_double2(g[HR - 1][0], g[HR - 1][1]);
      __syncthreads();
      const double2 Cun = L.cs[1][t], Cln = L.cs[1][t + 1];
      const double2 nu = L.nd[1][t], nl = L.nd[1][t + 1];
      double2 P[PH + 1];
#pragma unroll
      for (int k = 0; k <= PH; ++k) P[k] = L.cs[1][rg * PH + k];
      const double2 ep = *reinterpret_cast<const double2 *>(&L.edge[1][rp][2 * t]);
      const double2 en = *reinterpret_cast<const double2 *>(&L.edge[0][rn][2 * t]);
      static_for<0, QD>(q_even);
      __builtin_amdgcn_sched_barrier(0);
      Cu = Cun;
      Cl = Cln;
      d0 = t > 0 ? nu.y : d0;
      d1 = t < LPG - 1 ? nl.x : d1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const double first = P[0].x * (h ? ep.y : ep.x) - P[0].y * g[0][h];
        const double last = P[PH].x * (h ? en.y : en.x) + P[PH].y * g[HR - 1][h];
#pragma unroll
        for (int k = 0; k + 1 < PH; ++k) {
          const double x = g[2 * k + 1][h], y = g[2 * k + 2][h];
          g[2 * k + 1][h] = P[k + 1].x * y + P[k + 1].y * x;
          g[2 * k + 2][h] = P[k + 1].x * x - P[k + 1].y * y;
        }
        g[0][h] = first;
        g[HR - 1][h] = last;
      }
#pragma unroll
      for (int k = 0; k < PH; ++k) {
        const double x = g[2 * k][0], y = g[2 * k][1];
        g[2 * k][0] = Cu.x * lane_prev(y) - Cu.y * x;
        g[2 * k][1] = Cl.x * lane_next(x) + Cl.y * y;
      }
      r.a = d0;
      r.b = d1;
      r.g = coupling(k0);
      static_for<0, NST>([&](auto st) {
        r.stage<st>(floor2);
        __builtin_amdgcn_sched_barrier(0);
        static_for<QD + st * QI / NST, QD + (st + 1) * QI / NST>(q_odd);
        static_for<st * PH / NST, (st + 1) * PH / NST>([&](auto k) {
          const double x = g[2 * k + 1][0], y = g[2 * k + 1][1];
          g[2 * k + 1][0] = Cu.x * lane_prev(y) - Cu.y * x;
          g[2 * k + 1][1] = Cl.x * lane_next(x) + Cl.y * y;
        });
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
  static_for<0, QD>(q_odd);
  return rot;
}

// The parts of the eigen step around the sweeps, for a workgroup of EIG_NW waves.
constexpr int EIG_NW = 4, EIG_NT = 64 * EIG_NW;
using EigShape = OeShape<64, EIG_NW>;
using EigRegs = double[EigShape::HR][2];
__device__ inline int eig_t() { return threadIdx.x & (EigShape::LPG - 1); }
__device__ inline int eig_rg() { return threadIdx.x / EigShape::LPG; }

// From G in registers: its diagonal (through diag[64]), Q = I, and whether any pair of rows above the
// floor fails the outer test |g_ij| <= tol sqrt(g_ii g_jj), with the roots taken one by one (the product
// of two squared norms leaves the range of FP64 at norms of 1e-81 and 1e77; through L's edge rows, free before
// a sweep).  Contains barriers.
__device__ inline int oe_start(OeLds<64, EIG_NW> &L, const EigRegs &g, EigRegs &q, double &d0, double &d1,
                               double *diag, double tol, double floor2) {
  const int t = eig_t(), rg = eig_rg();
  double *const root = &L.edge[0][0][0];
#pragma unroll
  for (int i = 0; i < EigShape::HR; ++i) {
    const int r = EigShape::HR * rg + i;
    if (r == 2 * t) diag[r] = g[i][0];
    if (r == 2 * t + 1) diag[r] = g[i][1];
  }
  __syncthreads();
  if (threadIdx.x < 64) root[threadIdx.x] = sqrt(diag[threadIdx.x]);
  __syncthreads();
  d0 = diag[2 * t];
  d1 = diag[2 * t + 1];
  const double t0 = tol * root[2 * t], t1 = tol * root[2 * t + 1];
  int need = 0;
  const double lo2 = fmax(floor2, 0.0);
#pragma unroll
  for (int i = 0; i < EigShape::HR; ++i) {
    const int r = EigShape::HR * rg + i;
    const double dr = diag[r], sr = root[r];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const double dc = h ? d1 : d0, tc = h ? t1 : t0;
      need |= (int)(r != 2 * t + h) & (int)(dr > lo2) & (int)(dc > lo2) & (int)(fabs(g[i][h]) > tc * sr);
      q[i][h] = r == 2 * t + h ? 1.0 : 0.0;
    }
  }
  return need;
}

// Sweeps until one rotates nothing (or inner_max); e0, e1: the elements left in the lane's slots (a
// sweep reverses their order).
__device__ inline void oe_sweeps(OeLds<64, EIG_NW> &L, EigRegs &g, EigRegs &q, double &d0, double &d1, int inner_max,
                                 double floor2, int &e0, int &e1) {
  int rev = 0;
  for (int sweep = 0; sweep < inner_max; ++sweep) {
    const int rot = oe_sweep<64, EIG_NW>(L, g, q, d0, d1, floor2);
    rev ^= 1;
    if (inner_max > 1 && !__syncthreads_or(rot)) break;
  }
  const int t = eig_t();
  e0 = rev ? 63 - 2 * t : 2 * t;
  e1 = rev ? e0 - 1 : e0 + 1;
}

// rank[e]: the output row of element e, eigenvalues in decreasing order (ties: lower element first),
// the np largest to block p (rows 0..), the others to block q (rows 32..).  Four lanes per element,
// each counting a quarter of the others.
__device__ inline void oe_rank(double d0, double d1, int e0, int e1, double *diag, int *rank, int np, int nq) {
  const int tid = threadIdx.x;
  auto valid = [&](int r) { return r < 32 ? (r < np) : (r - 32 < nq); };
  if (eig_rg() == 0) {
    diag[e0] = d0;
    diag[e1] = d1;
  }
  __syncthreads();
  constexpr int LPE = EIG_NT / 64, PER = 64 / LPE;
  static_assert(LPE == 4, "the shuffles below sum four lanes");
  const int e = tid / LPE, o0 = (tid % LPE) * PER;
  const double mine = diag[e];
  int cnt = 0;
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int o = o0 + m;
    const double x = diag[o];
    cnt += (int)valid(o) & ((int)(x > mine) | ((int)(x == mine) & (int)(o < e)));
  }
  cnt += __shfl_xor(cnt, 1, 64);
  cnt += __shfl_xor(cnt, 2, 64);
  if (o0 == 0) rank[e] = cnt < np ? cnt : 32 + (cnt - np);
  __syncthreads();
}

// The eigen step of a block pair: the K-split partial Grams summed, the outer test, one odd-even sweep
// (or inner_max) and the pair's rotation Qt with its rows in decreasing order of the eigenvalues.
// Bound by the chain of 64 rounds on one compute unit: about 0.5 us a round, of which the FP64
// instructions of the four waves (one per SIMD, 64 values a lane) issue for about 0.37 us and the
// rotations' way through LDS and the barrier take the rest.  Four waves: with eight the rotation chain
// and its LDS reads are repeated by twice as many waves (41.0 against 39.3 us a launch).  Measured at 331 x 517
// (six pairs): 84 us a launch with the matrix in LDS, 41 us in this form.
// grid (pairs, matrices)
__global__ __launch_bounds__(EIG_NT) __attribute__((amdgpu_waves_per_eu(1, 2))) void eigen_kernel(const SvdMat *mats, int step) {
  using S = EigShape;
  __shared__ OeLds<64, EIG_NW> L;
  __shared__ double diag[64];   // by slot while testing, by element while ranking
  __shared__ int rank[64];
  const SvdMat &a = mats[blockIdx.y];
  const int pair = blockIdx.x;
  if (!a.active || a.fused || step >= a.nb - 1 || pair >= a.nb / 2) return;
  const int tid = threadIdx.x, t = eig_t(), rg = eig_rg();
  int p, q;
  rr_pair(a.nb, step, pair, p, q);
  const int np = block_rows(a.Ra, p), nq = block_rows(a.Ra, q);
  int *skip = a.skip + pair;
  if (np + nq == 0) {
    if (tid == 0) *skip = 1;
    return;
  }
  auto valid = [&](int r) { return r < 32 ? (r < np) : (r - 32 < nq); };
  // the K-split partial Grams summed in split order; this lane's elements are 16-byte pairs of HR rows
  const double *Gp = a.gram + (int64_t)pair * a.ksplit * 4096 + (int64_t)S::HR * rg * 64 + 2 * t;
  const int nks = a.ksplit;
  double g[S::HR][2], v[S::HR][2];
#pragma unroll
  for (int i = 0; i < S::HR; ++i) g[i][0] = g[i][1] = 0.0;
  int ks = 0;
  for (; ks + 4 <= nks; ks += 4) {
    double2 part[4][S::HR];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < S::HR; ++i)
        part[u][i] = *reinterpret_cast<const double2 *>(Gp + (int64_t)(ks + u) * 4096 + 64 * i);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < S::HR; ++i) {
        g[i][0] += part[u][i].x;
        g[i][1] += part[u][i].y;
      }
  }
  for (; ks < nks; ++ks)
#pragma unroll
    for (int i = 0; i < S::HR; ++i) {
      const double2 x = *reinterpret_cast<const double2 *>(Gp + (int64_t)ks * 4096 + 64 * i);
      g[i][0] += x.x;
      g[i][1] += x.y;
    }
  const double floor2 = row_floor2(a, *a.fro2);
  double d0, d1;
  const int need = oe_start(L, g, v, d0, d1, diag, a.tol, floor2);
  if (!__syncthreads_or(need)) {
    if (tid == 0) *skip = 1;
    return;
  }
  if (tid == 0) atomicAdd(a.ctr, 1);
  int e0, e1;
  oe_sweeps(L, g, v, d0, d1, a.inner_max, floor2, e0, e1);
  oe_rank(d0, d1, e0, e1, diag, rank, np, nq);
  // Qt row rank[e] <- column of element e: this lane's HR consecutive entries of it
  double *Qt = a.qt + (int64_t)pair * 4096;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int e = h ? e1 : e0;
    const bool ve = valid(e);
    double *row = Qt + (ve ? rank[e] : 0) * 64 + S::HR * rg;
    if (ve)
#pragma unroll
      for (int i = 0; i < S::HR; i += 2)
        *reinterpret_cast<double2 *>(row + i) = make_double2(v[i][h], v[i + 1][h]);
  }
  // rows and columns of the slots without a row are zero
  for (int e = tid; e < 4096; e += EIG_NT)
    if (!valid(e >> 6)) Qt[e] = 0.0;
  if (tid == 0) *skip = 0;
}

// -------------------------------------------------------------- apply
// rows of X (valid slots, row grow(slot)) columns [c0, c0 + 64) <- Qt X, with
// As[k][i] = Qt[i][k] in LDS; Xs is the staging tile
template <class Valid, class Grow>
__device__ inline void apply_tile(double *X, int ld, int c0, double (*As)[65], double (*Xs)[65], Valid valid,
                                  Grow grow) {
  const int tid = threadIdx.x;
  for (int e = tid; e < 4096; e += 256) {
    const int i = e >> 6, k = e & 63;
    Xs[i][k] = (valid(i) && c0 + k < ld) ? X[(int64_t)grow(i) * ld + c0 + k] : 0.0;
  }
  __syncthreads();
  const int lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  v4d acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = v4d{0, 0, 0, 0};
#pragma unroll 4
  for (int kk = 0; kk < 64; kk += 4) {
    const double av = As[kk + lk][16 * wave + lr];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = mfma16(av, Xs[kk + lk][16 * t + lr], acc[t]);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int so = 16 * wave + 4 * r + lk, col = 16 * t + lr;  // f64 result layout
      if (valid(so) && c0 + col < ld) X[(int64_t)grow(so) * ld + c0 + col] = acc[t][r];
    }
}

// grid (pairs, groups of tpw column tiles of B then of Jt, matrices).  Each wave
// keeps its 16 rows of the pair's rotation Qt as MFMA A-operands in registers (read once);
// the 64 x 64 tile of X passes through LDS, and the next tile of the group is loaded into
// registers while the current one is multiplied and written back, so one workgroup keeps
// a tile's loads in flight at all times.  33 KB of LDS: four workgroups per CU.
__global__ __launch_bounds__(256) void apply_kernel(const SvdMat *mats, int step, int tpw) {
  __shared__ double Xs[64][65];  // Xs[k][j] = X[row(k)][c0 + j]
  const SvdMat &a = mats[blockIdx.z];
  const int pair = blockIdx.x;
  const int ntile_b = (a.C + 63) / 64, ntile_j = (a.R + 63) / 64;
  const int t0 = blockIdx.y * tpw;
  if (!a.active || a.fused || step >= a.nb - 1 || pair >= a.nb / 2 || t0 >= ntile_b + ntile_j) return;
  if (a.skip[pair]) return;
  int p, q;
  rr_pair(a.nb, step, pair, p, q);
  const int np = block_rows(a.Ra, p), nq = block_rows(a.Ra, q);
  auto valid = [&](int r) { return r < 32 ? (r < np) : (r - 32 < nq); };
  auto grow = [&](int r) { return r < 32 ? p * BS + r : q * BS + (r - 32); };
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 15, lk = lane >> 4;
  // A(i, k) = Qt[i][k] for the wave's output rows i = 16 wave + lr, k = 4 kk + lk
  const double *Qt = a.qt + (int64_t)pair * 4096 + (16 * wave + lr) * 64 + lk;
  double aq[16];
#pragma unroll
  for (int kk = 0; kk < 16; ++kk) aq[kk] = Qt[4 * kk];
  const int t1 = t0 + tpw < ntile_b + ntile_j ? t0 + tpw : ntile_b + ntile_j;
  // thread tid loads rows (tid >> 6) + 4u, u < 16, at column tid & 63 of a tile
  const int lrow = tid >> 6, lcol = tid & 63;
  auto tile_of = [&](int tile, double *&X, int &ld, int &c0) {
    if (tile < ntile_b) { X = a.bw; ld = a.C; c0 = tile * 64; }
    else { X = a.jt; ld = a.R; c0 = (tile - ntile_b) * 64; }
  };
  double nx[16];
  auto load = [&](int tile) {
    double *X;
    int ld, c0;
    tile_of(tile, X, ld, c0);
    const bool colok = c0 + lcol < ld;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      const int k = lrow + 4 * u;
      nx[u] = (colok && valid(k)) ? X[(int64_t)grow(k) * ld + c0 + lcol] : 0.0;
    }
  };
  load(t0);
  for (int tile = t0; tile < t1; ++tile) {
    __syncthreads();  // the previous tile's products have read Xs
#pragma unroll
    for (int u = 0; u < 16; ++u) Xs[lrow + 4 * u][lcol] = nx[u];
    __syncthreads();
    if (tile + 1 < t1) load(tile + 1);  // in flight during the products below
    v4d acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = v4d{0, 0, 0, 0};
#pragma unroll
    for (int kk = 0; kk < 16; ++kk)
#pragma unroll
      for (int t = 0; t < 4; ++t) acc[t] = mfma16(aq[kk], Xs[4 * kk + lk][16 * t + lr], acc[t]);
    double *X;
    int ld, c0;
    tile_of(tile, X, ld, c0);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int so = 16 * wave + 4 * r + lk, col = 16 * t + lr;  // f64 result layout
        if (valid(so) && c0 + col < ld) X[(int64_t)grow(so) * ld + c0 + col] = acc[t][r];
      }
  }
}

// -------------------------------------------------------------- whole Jacobi, one workgroup
// Matrices with at most 64 rows to orthogonalise (one block pair) run every
// sweep inside one workgroup: Gram on MFMA into LDS, the outer test, the Jacobi
// sweep in registers, then the rotation of B and Jt, until a sweep needs no
// rotation.  Bound by the 64 rounds of the sweep (about 33 us) and the walk over
// B's column tiles; 64 rows of 64 to 128: 370 us, 1000 us with the Gram in LDS.
// ctr[0] = 0 when converged (1 otherwise), ctr[1] = sweeps.  grid (matrices)
__global__ __launch_bounds__(EIG_NT) __attribute__((amdgpu_waves_per_eu(1, 2))) void jacobi_fused_kernel(
    const SvdMat *mats, int max_sweeps) {
  __shared__ OeLds<64, EIG_NW> L;
  __shared__ double diag[64];
  __shared__ int rank[64];
  __shared__ double Gs[64][65];  // the Gram, then Qt's columns
  __shared__ double Xs[64][65];  // Gram staging, then apply tiles
  const SvdMat &a = mats[blockIdx.x];
  if (!a.active || a.fused != 1) return;
  const int tid = threadIdx.x, t = eig_t(), rg = eig_rg();
  const int np = block_rows(a.R, 0), nq = block_rows(a.R, 1);
  auto valid = [&](int r) { return r < 32 ? (r < np) : (r - 32 < nq); };
  auto grow = [](int r) { return r; };  // blocks 0 and 1: slot r is row r
  const double floor2 = row_floor2(a, *a.fro2);
  int sw = 0, conv = 0;
  while (sw < max_sweeps) {
    ++sw;
    {
      v4d acc[2][2];
      gram_acc(a, 0, 1, np, nq, 0, a.C, Xs, acc);
      gram_store(acc, &Gs[0][0], 65);
    }
    __syncthreads();
    double g[EigShape::HR][2], v[EigShape::HR][2], d0, d1;
#pragma unroll
    for (int i = 0; i < EigShape::HR; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) g[i][h] = Gs[EigShape::HR * rg + i][2 * t + h];
    const int need = oe_start(L, g, v, d0, d1, diag, a.tol, floor2);
    if (!__syncthreads_or(need)) {
      conv = 1;
      break;
    }
    int e0, e1;
    oe_sweeps(L, g, v, d0, d1, a.inner_max, floor2, e0, e1);
    oe_rank(d0, d1, e0, e1, diag, rank, np, nq);
    // Gs[k][i] = Qt[i][k], over the Gram
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = h ? e1 : e0;
      if (valid(e)) {
        const int col = rank[e];
#pragma unroll
        for (int i = 0; i < EigShape::HR; ++i) Gs[EigShape::HR * rg + i][col] = v[i][h];
      }
    }
    __syncthreads();
    const int ntile_b = (a.C + 63) / 64;
    for (int tl = 0; tl < ntile_b; ++tl) {
      apply_tile(a.bw, a.C, 64 * tl, Gs, Xs, valid, grow);
      __syncthreads();
    }
    apply_tile(a.jt, a.R, 0, Gs, Xs, valid, grow);
    __syncthreads();
  }
  if (tid == 0) {
    a.ctr[0] = conv ? 0 : 1;
    a.ctr[1] = sw;
  }
}

// -------------------------------------------------------------- one-sided Jacobi, tiny matrices
// At most 32 rows of at most 64 columns: the one-sided (Hestenes) method directly on the rows, held
// in registers with Jt.  Odd-even transposition order as in oe_sweep: group t of 16 lanes (one DPP row)
// holds the rows in the slots 2t and 2t+1, a lane up to 4 columns of B and 2 of Jt of each; a rotation
// leaves its two rows exchanged.  Between the rounds one row of every group moves to its neighbour
// through LDS: the lower one down before an odd round (pairs (2t+1, 2t+2)), the upper one up after it,
// one barrier each.  Rotation and tests as in the blocked method, outer tolerance a.tol, rows at
// the rounding floor left alone.  ctr[0] = 0 when converged, ctr[1] = sweeps.
// It reads A itself (its Frobenius norm is formed on the way) and ends with the spectrum record, so such a
// matrix takes one launch up to its spectrum.  Bound by the chain of R rounds a sweep on one compute
// unit: dot products, their sums over 16 lanes, the rotation and the move, about 120 instructions and
// two trips through LDS a round, 0.35 us.  64 matrices of 32 x 32 (10 sweeps): 122 us; with the rows in LDS
// and the norm and spectrum in launches of their own 214 + 35 us.  grid (matrices), 256 threads.
constexpr int TINY_NV = 3;  // 16-byte values of a row that a lane passes on
struct TinyLds {
  double2 down[17][16][TINY_NV], up[17][16][TINY_NV];
  double red[4];
  double sig[32], key[32];
};

// CU columns of B and JU of Jt per lane: C <= 16 CU, R <= 16 JU.  Leaves bw, jt and sig[r] = |row r|.
template <int CU, int JU>
__device__ __forceinline__ void jacobi_tiny_rows(const SvdMat &a, int max_sweeps, TinyLds &L, int &sw, int &conv) {
  constexpr int NR = CU + JU, NV = (NR + 1) / 2;
  static_assert(NV <= TINY_NV, "row in LDS");
  const int tid = threadIdx.x, t = tid >> 4, l = tid & 15;
  const int R = a.R, C = a.C, P = (R + 1) >> 1;
  double x[2 * NV], y[2 * NV];  // lower and upper row: B values, then Jt values
  auto load = [&](int r, double(&z)[2 * NV]) {  // row r of A (of A^T when trans), Jt = I
    static_for<0, 2 * NV>([&](auto u) {
      z[u] = 0.0;
      if constexpr (u < CU) {
        const int c = l + 16 * u;
        if (r < R && c < C) {
          const int e = a.trans ? c * a.n + r : r * a.n + c;
          z[u] = a.dtype == TNA_F64 ? static_cast<const double *>(a.A)[e]
                                    : (double)static_cast<const float *>(a.A)[e];
        }
      } else if constexpr (u < NR) {
        z[u] = (r < R && l + 16 * (u - CU) == r) ? 1.0 : 0.0;
      }
    });
  };
  auto put = [&](double2(*to)[TINY_NV], const double(&z)[2 * NV]) {
    static_for<0, NV>([&](auto v) { to[l][v] = make_double2(z[2 * v], z[2 * v + 1]); });
  };
  auto get = [&](double2(*from)[TINY_NV], double(&z)[2 * NV]) {
    static_for<0, NV>([&](auto v) {
      const double2 w = from[l][v];
      z[2 * v] = w.x;
      z[2 * v + 1] = w.y;
    });
  };
  load(2 * t, x);
  load(2 * t + 1, y);
  if (tid < 16) static_for<0, NV>([&](auto v) { L.down[16][l][v] = make_double2(0.0, 0.0); });
  double ss = 0.0;
  static_for<0, CU>([&](auto u) { ss += x[u] * x[u] + y[u] * y[u]; });
  const double fro2 = bsum256(ss, L.red);
  if (tid == 0) a.fro2[0] = fro2;
  const double floor2 = row_floor2(a, fro2);
  const double tol2 = a.tol * a.tol;
  // rotates x against y if their coupling fails the test, and exchanges them; `idle` leaves x and
  // zeroes y (the last slot's odd round: y is the empty row)
  auto rotate = [&](int &rot, bool idle) {
    double al = 0.0, be = 0.0, ga = 0.0;
    static_for<0, CU>([&](auto u) {
      al = fma(x[u], x[u], al);
      be = fma(y[u], y[u], be);
      ga = fma(x[u], y[u], ga);
    });
    row16_sum3(al, be, ga);
    RotChain r;
    r.a = al;
    r.b = be;
    r.g = ga;
    static_for<0, 8>([&](auto st) { r.template stage<st, false>(floor2); });
    const bool act = al > floor2 && be > floor2 && r.coupled(tol2);
    const double c = act ? r.c : idle ? 0.0 : 1.0, s = act ? r.s : idle ? 1.0 : 0.0;
    rot |= act;
    static_for<0, NR>([&](auto u) {
      const double p = x[u], q = y[u];
      x[u] = c * q + s * p;
      y[u] = c * p - s * q;
    });
  };
  // what a group reads in place of a neighbour it lacks: the empty row above the last slot, and the
  // first group its own lower row back
  double2(*const from_above)[TINY_NV] = L.down[t + 1 < P ? t + 1 : 16];
  double2(*const from_below)[TINY_NV] = t > 0 ? L.up[t] : L.down[0];
  const bool last = t + 1 >= P;
  sw = conv = 0;
  while (sw < max_sweeps) {
    ++sw;
    int rot = 0;
#pragma unroll 1
    for (int rr = 0; rr < P; ++rr) {
      rotate(rot, false);
      put(L.down[t], x);
      __syncthreads();
      static_for<0, 2 * NV>([&](auto u) { x[u] = y[u]; });
      get(from_above, y);
      rotate(rot, last);
      put(L.up[t + 1], y);
      __syncthreads();
      static_for<0, 2 * NV>([&](auto u) { y[u] = x[u]; });
      get(from_below, x);
    }
    if (!__syncthreads_or(rot && t < P)) {
      conv = 1;
      break;
    }
  }
  // an odd number of sweeps leaves the slots reversed: with an odd R the empty slot is then the first
  const int shift = R & sw & 1;
  auto store = [&](int r, const double(&z)[2 * NV]) {
    double n2 = 0.0;
    static_for<0, CU>([&](auto u) { n2 = fma(z[u], z[u], n2); });
    n2 = row16_sum(n2);
    if (r < 0 || r >= R) return;
    if (l == 0) L.sig[r] = sqrt(n2);
    static_for<0, NR>([&](auto u) {
      if constexpr (u < CU) {
        if (l + 16 * u < C) a.bw[r * C + l + 16 * u] = z[u];
      } else {
        if (l + 16 * (u - CU) < R) a.jt[r * R + l + 16 * (u - CU)] = z[u];
      }
    });
  };
  store(2 * t - shift, x);
  store(2 * t + 1 - shift, y);
}

__global__ __launch_bounds__(256) void jacobi_tiny_kernel(const SvdMat *mats, int max_sweeps) {
  __shared__ TinyLds L;
  const SvdMat &a = mats[blockIdx.x];
  if (!a.active || a.fused != 2) return;
  const int tid = threadIdx.x, R = a.R;
  int sw, conv;
  if (R <= 16) {
    if (a.C <= 16) jacobi_tiny_rows<1, 1>(a, max_sweeps, L, sw, conv);
    else jacobi_tiny_rows<4, 1>(a, max_sweeps, L, sw, conv);
  } else {
    if (a.C <= 32) jacobi_tiny_rows<2, 2>(a, max_sweeps, L, sw, conv);
    else jacobi_tiny_rows<4, 2>(a, max_sweeps, L, sw, conv);
  }
  double *const sig = L.sig, *const key = L.key;
  if (tid == 0) {
    a.ctr[0] = conv ? 0 : 1;
    a.ctr[1] = sw;
  }
  __syncthreads();
  // the spectrum record of sort_kernel, for at most 32 values: ranks counted, sums by the first wave.
  // With a NaN among them nothing is ranked (the caller stops at the NaN sums).
  if (tid < 64) {
    const double mine = tid < R ? sig[tid] : 0.0;
    const bool nan = __any(!(mine == mine));
    int k = 0;
    for (int o = 0; o < R; ++o) k += (sig[o] > mine || (sig[o] == mine && o < tid)) ? 1 : 0;
    if (tid < R) {
      key[nan ? tid : k] = mine;
      a.perm[nan ? tid : k] = tid;
    }
  }
  __syncthreads();
  if (tid < 64) {
    const double s0 = key[0], v = tid < R ? key[tid] : 0.0;
    if (tid < R) a.S[tid] = v;
    const double Z = wave_sum_d(v * v);
    const double p = v * v / Z;
    const double ent = wave_sum_d(tid < R && p > 0.0 ? -p * log(p) : 0.0);
    if (tid == 0) {
      a.spec[0] = Z;
      a.spec[1] = Z == Z ? ent : Z;
      a.spec[7] = conv ? (double)sw : -(double)sw;
    }
    if (tid < 16) a.spec[8 + tid] = v;
    const unsigned long long above = __ballot(tid < R && v > a.thr);
    const unsigned long long rank = __ballot(tid < R && v > (a.noise_rel > 0.0 ? a.noise_rel : 1e-12) * s0);
    if (tid == 0) {
      if (a.thr > 0.0) a.spec[24] = (double)__popcll(above);
      a.spec[25] = (double)__popcll(rank);
    }
    if (a.eps_target > 0.0) {
      double tail = v * v;  // sum over this value and the later ones
#pragma unroll
      for (int off = 1; off < 32; off <<= 1) {
        const double o = __shfl_down(tail, off, 64);
        tail += tid + off < 32 ? o : 0.0;
      }
      const unsigned long long meets = __ballot(tid < R && tail <= a.eps_target * a.eps_target);
      const int first = meets ? __ffsll((unsigned long long)meets) - 1 : R;
      if (tid == 0) a.spec[6] = (double)(first < 1 ? 1 : first);
    }
  }
}

// -------------------------------------------------------------- load / init
// grid (tiles, 1, matrices): rows of A (or of A^T) into bw as double; Jt = I
__global__ __launch_bounds__(256) void load_kernel(const SvdMat *mats) {
  __shared__ double tile[32][33];
  const SvdMat &a = mats[blockIdx.z];
  if (a.fused == 2) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int ntj = (a.n + 31) / 32, nti = (a.m + 31) / 32;
  const int t = blockIdx.x;
  if (t < nti * ntj) {
    const int by = (t / ntj) * 32, bx = (t % ntj) * 32;  // by over m, bx over n
    for (int r = ty; r < 32; r += 8) {
      const int i = by + r, j = bx + tx;
      double v = 0.0;
      if (i < a.m && j < a.n)
        v = a.dtype == TNA_F64 ? static_cast<const double *>(a.A)[(int64_t)i * a.n + j]
                               : (double)static_cast<const float *>(a.A)[(int64_t)i * a.n + j];
      tile[r][tx] = v;
    }
    __syncthreads();
    if (!a.trans) {
      for (int r = ty; r < 32; r += 8) {
        const int i = by + r, j = bx + tx;
        if (i < a.m && j < a.n) a.bw[(int64_t)i * a.n + j] = tile[r][tx];
      }
    } else {
      for (int r = ty; r < 32; r += 8) {
        const int j = bx + r, i = by + tx;
        if (j < a.n && i < a.m) a.bw[(int64_t)j * a.m + i] = tile[tx][r];
      }
    }
  } else {
    const int64_t e0 = (int64_t)(t - nti * ntj) * 1024, tot = (int64_t)a.R * a.R;
    for (int64_t e = e0 + threadIdx.x; e < e0 + 1024 && e < tot; e += 256) {
      const int64_t r = e / a.R, c = e - r * a.R;
      a.jt[e] = (r == c) ? 1.0 : 0.0;
    }
  }
}

// |A|_F^2 of the loaded rows in two fixed-order stages: partials of 4096 elements or more by up to
// FRO_BLOCKS blocks into the Gram area (free until the first sweep), then one block per matrix
// sums them
constexpr int FRO_BLOCKS = 256;
__host__ __device__ inline int fro_blocks(int R, int C) {
  const int64_t b = ((int64_t)R * C + 4095) / 4096;
  return b < 1 ? 1 : b > FRO_BLOCKS ? FRO_BLOCKS : (int)b;
}
__global__ __launch_bounds__(256) void fro_partial_kernel(const SvdMat *mats) {
  __shared__ double red[4];
  const SvdMat &a = mats[blockIdx.z];
  const int nb = fro_blocks(a.R, a.C);
  if (a.fused == 2 || (int)blockIdx.x >= nb) return;
  const int64_t tot = (int64_t)a.R * a.C;
  const int64_t chunk = (tot + nb - 1) / nb;
  const int64_t beg = chunk * blockIdx.x, end = beg + chunk < tot ? beg + chunk : tot;
  double v = 0.0;
  for (int64_t e = beg + threadIdx.x; e < end; e += 256) v += a.bw[e] * a.bw[e];
  v = bsum256(v, red);
  if (threadIdx.x == 0) a.gram[blockIdx.x] = v;
}
__global__ __launch_bounds__(256) void fro_kernel(const SvdMat *mats) {
  __shared__ double red[4];
  const SvdMat &a = mats[blockIdx.x];
  if (a.fused == 2) return;
  double v = (int)threadIdx.x < fro_blocks(a.R, a.C) ? a.gram[threadIdx.x] : 0.0;
  v = bsum256(v, red);
  if (threadIdx.x == 0) *a.fro2 = v;
}

// What the host decides on, written straight into its pinned memory (one store each instead of one
// copy command per matrix): counters at hctr[2 z], hctr[2 z + 1], the two norms at hfro[2 z],
// hfro[2 z + 1].  With reset, the counter of rotating pairs is cleared for the next sweep.
__global__ void status_kernel(const SvdMat *mats, int nmat, int *hctr, double *hfro, int reset) {
  const int z = blockIdx.x * blockDim.x + threadIdx.x;
  if (z >= nmat) return;
  const SvdMat &a = mats[z];
  if (hctr) {
    hctr[2 * z] = a.ctr[0];
    hctr[2 * z + 1] = a.ctr[1];
  }
  if (hfro) {
    hfro[2 * z] = a.fro2[0];
    hfro[2 * z + 1] = a.fro2[1];
  }
  if (reset && a.active && !a.fused) a.ctr[0] = 0;
}

// -------------------------------------------------------------- QR start
// A Householder QR of the loaded rows, B = Q Rf, turns the start state (B, Jt) =
// (A, I) into (Rf, Q^T): B = Jt A still holds, and the one-sided Jacobi needs far
// fewer sweeps on the rows of Rf than on A itself.  Blocked: each panel of 32
// columns is factored by one workgroup per matrix where at most 1024 rows are left
// (qr_panel_wg_kernel), by a grid above that (qr_panel_coop_kernel, qr_col_kernel);
// the trailing columns take the panel's block reflector in three launches
// (qr_wy_kernel, qr_wy_solve_kernel, qr_wy_update_kernel), and Q^T is formed from
// the stored reflectors the same way.  No column pivoting: on the
// prescribed-spectrum matrices it did not lower the sweep count; cperm / pinv keep
// the column order explicit (the identity, or by decreasing norm, see below).
constexpr int QR_MIN_ROWS_DEV = 256;
// The products of a block reflector with 32 rows (S = V V^T and W = V X) are long in K and short
// in M: K is cut into up to QR_SPLIT pieces, and the pieces are summed in order afterwards.
constexpr int QR_SPLIT = 8;

// grid (column blocks, 1, matrices): the identity column order
__global__ __launch_bounds__(256) void qr_init_kernel(const SvdMat *mats) {
  const SvdMat &a = mats[blockIdx.z];
  if (!a.active || !a.precond) return;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j < a.C) a.cperm[j] = j;
  if (j == 0) a.ctr[2] = 0;  // arrival counter of qr_col_kernel
}

// A rows_scaled matrix whose QR start may stop early takes its columns in order of decreasing
// norm (ties: lower index first), decided once before the factorisation: the panels then meet
// the heavy columns first, so the rows below the factored panels fall to the rounding level at
// about the numerical rank whatever the input's column order (a two-site matrix is ordered
// physical index first, so half of its columns by weight sit at the end).
__device__ inline bool qr_sorts_columns(const SvdMat &a) { return a.active && a.precond && a.rows_scaled; }

// grid (32-column blocks, 1, matrices): squared column norms of B into qws[2048 ..) (free until the QR);
// eight threads a column, each every eighth row (with one thread a column and 256 columns a block, four
// blocks walked 1024 rows one after the other: 226 us at 1024 x 1024)
__global__ __launch_bounds__(256) void colnorm_kernel(const SvdMat *mats) {
  __shared__ double part[8][33];
  const SvdMat &a = mats[blockIdx.z];
  if (!qr_sorts_columns(a)) return;
  const int cl = threadIdx.x & 31, g = threadIdx.x >> 5, c = blockIdx.x * 32 + cl;
  double ss = 0.0;
  if (c < a.C) {
#pragma unroll 8
    for (int r = g; r < a.R; r += 8) {
      const double v = a.bw[(int64_t)r * a.C + c];
      ss = fma(v, v, ss);
    }
  }
  part[g][cl] = ss;
  __syncthreads();
  if (g == 0 && c < a.C) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) t += part[k][cl];
    a.qws[2048 + c] = t;
  }
}

// A NaN compares with nothing: it would move the entries that fill a sort up to a power of two, whose
// indices lie past the matrix, among the real ones.
__device__ inline double sort_key(double v) { return v == v ? v : __builtin_huge_val(); }

// one block per matrix: cperm <- columns by decreasing norm (bitonic sort of (norm, index))
__global__ __launch_bounds__(1024) void colsort_kernel(const SvdMat *mats) {
  __shared__ double key[4096];
  __shared__ int idx[4096];
  const SvdMat &a = mats[blockIdx.x];
  if (!qr_sorts_columns(a)) return;
  int P = 1;
  while (P < a.C) P <<= 1;
  for (int i = threadIdx.x; i < P; i += 1024) {
    key[i] = i < a.C ? sort_key(a.qws[2048 + i]) : -1.0;
    idx[i] = i;
  }
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < P; i += 1024) {
        const int l = i ^ j;
        if (l > i) {
          const bool i_before_l = key[i] > key[l] || (key[i] == key[l] && idx[i] < idx[l]);
          if ((i & k) == 0 ? !i_before_l : i_before_l) {
            const double tk = key[i]; key[i] = key[l]; key[l] = tk;
            const int ti = idx[i]; idx[i] = idx[l]; idx[l] = ti;
          }
        }
      }
      __syncthreads();
    }
  for (int i = threadIdx.x; i < a.C; i += 1024) a.cperm[i] = idx[i];
}

// grid (tiles, 1, matrices): B[r][c] <- row r of A (A^T when trans) at column cperm[c], read again
// from the input (the natural-order load served the norms)
__global__ __launch_bounds__(256) void permute_load_kernel(const SvdMat *mats) {
  __shared__ double tile[32][33];
  const SvdMat &a = mats[blockIdx.z];
  if (!qr_sorts_columns(a)) return;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
  const int ntc = (a.C + 31) / 32, ntr = (a.R + 31) / 32;
  const int t = blockIdx.x;
  if (t >= ntr * ntc) return;
  const int r0 = (t / ntc) * 32, c0 = (t % ntc) * 32;
  auto in = [&](int64_t e) {
    return a.dtype == TNA_F64 ? static_cast<const double *>(a.A)[e] : (double)static_cast<const float *>(a.A)[e];
  };
  if (!a.trans) {  // B row r = A row r (length n = C): gather along the row
    for (int rr = ty; rr < 32; rr += 8) {
      const int r = r0 + rr, c = c0 + tx;
      if (r < a.R && c < a.C) a.bw[(int64_t)r * a.C + c] = in((int64_t)r * a.n + a.cperm[c]);
    }
  } else {  // B row r = A column r; B column c = A row cperm[c]: read A rows along r, write through LDS
    for (int cc = ty; cc < 32; cc += 8) {
      const int c = c0 + cc, r = r0 + tx;
      tile[cc][tx] = (c < a.C && r < a.R) ? in((int64_t)a.cperm[c] * a.n + r) : 0.0;
    }
    __syncthreads();
    for (int rr = ty; rr < 32; rr += 8) {
      const int r = r0 + rr, c = c0 + tx;
      if (r < a.R && c < a.C) a.bw[(int64_t)r * a.C + c] = tile[tx][rr];
    }
  }
}

// The scalars of the reflector that takes a column x, |x|^2 = t, x_0 = xn, to (alpha, 0, ...): v = x - alpha e_0 is
// stored times the power of two sc that brings |x| into [1, 2), and beta = 2 / |sc v|^2, so that no norm squared
// twice is formed.  A column below 1e-150, whose squares soon lose their digits, has no reflector (beta = sc = 0):
// its entries under the diagonal count as zero.
constexpr double QR_NULL2 = 1e-300;
struct Reflector {
  double alpha, beta, v0, sc;
  __device__ __forceinline__ Reflector(double t, double xn) {
    const double nx = sqrt(t);
    const bool null = !(t > QR_NULL2);
    alpha = xn >= 0.0 ? -nx : nx;
    v0 = xn - alpha;
    sc = null ? 0.0 : __hiloint2double(0x7fe00000 - (__double2hiint(nx) & 0x7ff00000), 0);
    const double ns = nx * sc;
    beta = null ? 0.0 : 1.0 / (ns * (ns + fabs(xn * sc)));
  }
  // coefficient of v in a later column whose product with v is y
  __device__ __forceinline__ double coef(double y) const { return beta * (y * sc) * sc; }
};

// Householder QR of the panel of columns k0 .. k0+31 of B (rows k0..), one column after the
// other: x = B[k:R, k], alpha = -sign(x_0) |x|, v = x - alpha e_0 (stored as row k of qv),
// beta = 2 / v^T v = 1 / (|x| (|x| + |x_0|)) (stored in qws), both scaled as Reflector says;
// B[k:, k] <- (alpha, 0, ...); then every later column c of the panel: B[k:, c] -= beta (v^T B[k:, c]) v.
// The trailing columns are updated afterwards with the block reflector (qr_block_apply).
//
// Spread over row chunks of QC_ROWS rows, one launch per column: launch k applies reflector k to
// the panel columns right of it and forms the chunk partials that reflector k+1 needs
// (|B[k+1:, k+1]|^2 and the dots B[k+2:, k+1] . B[k+2:, c]); the last chunk to arrive (arrival
// counter, device-scope fences, no waiting) sums the partials in chunk order and writes alpha, beta,
// v_{k+1,k+1} = x0 - alpha and w_c = beta (v . B[:, c]) for the next launch.  The start launch
// (k = k0 - 1) forms the partials of column k0 only.  Scratch: chunk partials (33 per chunk) at
// qws[2048 ..), the scalars at qws[2048 + 64 C + R ..).  grid (chunks, 1, matrices), 256 threads.
constexpr int QC_ROWS = 128;
__global__ __launch_bounds__(256) void qr_col_kernel(const SvdMat *mats, int k0, int k) {
  __shared__ double red[8][33];
  __shared__ int last;
  const SvdMat &a = mats[blockIdx.z];
  if (!a.active || !a.precond || k0 >= a.Ra) return;
  const int R = a.R, C = a.C;
  const int kend = k0 + 32 < R ? k0 + 32 : R, cend = k0 + 32 < C ? k0 + 32 : C;
  if (k >= kend) return;
  const int G = (R - k0 + QC_ROWS - 1) / QC_ROWS, blk = blockIdx.x;
  if (blk >= G) return;
  const int tid = threadIdx.x, lane = tid & 63, cl = tid & 31, rsub = tid >> 5;
  const int c = k0 + cl;
  const bool colok = c < cend;
  double *B = a.bw;
  double *part = a.qws + 2048, *betas = a.qws + 2048 + 64 * (int64_t)C, *sc = betas + R;
  const bool start = k < k0;
  if (start) {
    // reflector rows k0 .. kend-1 start as zero (launch k writes its entries from row k on)
    const int64_t tot = (int64_t)(kend - k0) * R;
    for (int64_t e = (int64_t)blk * 256 + tid; e < tot; e += (int64_t)G * 256) a.qv[(int64_t)k0 * R + e] = 0.0;
    if (blk == 0 && tid == 0) a.fro2[1] = 0.0;  // trailing-row maximum of this panel (qr_tail_kernel)
  }
  double alpha = 0.0, beta = 0.0, vk = 0.0, x0 = 0.0, vsc = 0.0, wc = 0.0;
  const int kc = k - k0;
  if (!start) {
    alpha = sc[0];
    beta = sc[1];
    vk = sc[2];
    x0 = sc[3];
    vsc = sc[36];
    wc = (cl > kc && colok) ? sc[4 + cl] : 0.0;
  }
  double val[QC_ROWS / 8];
#pragma unroll
  for (int m = 0; m < QC_ROWS / 8; ++m) {
    const int i = k0 + blk * QC_ROWS + rsub + 8 * m;
    double x = (i < R && colok) ? B[(int64_t)i * C + c] : 0.0;
    if (!start) {
      const double bk = __shfl(x, (lane & 32) | kc, 64);  // this row's column-k entry
      if (i < R && i >= k && colok && cl >= kc) {
        const double vi = (i == k) ? vk : bk;
        if (cl > kc) {
          x -= wc * vi;
        } else {
          x = (i == k) ? (beta != 0.0 ? alpha : x0) : 0.0;
          a.qv[(int64_t)k * R + i] = vi * vsc;
        }
        B[(int64_t)i * C + c] = x;
      }
    }
    val[m] = x;
  }
  const int nk = k + 1, nc = nk - k0;
  if (nk >= kend) return;
  double acc = 0.0;
#pragma unroll
  for (int m = 0; m < QC_ROWS / 8; ++m) {
    const int i = k0 + blk * QC_ROWS + rsub + 8 * m;
    const double y = val[m];
    const double ynk = __shfl(y, (lane & 32) | nc, 64);
    if (i < R && i >= nk) {
      if (cl == nc) acc += y * y;                    // |B[nk:, nk]|^2
      else if (cl > nc && i > nk) acc += ynk * y;    // B[nk+1:, nk] . B[nk+1:, c]
    }
  }
  red[rsub][cl] = acc;
  __syncthreads();
  if (tid < 32 && cl >= nc) {
    double t = 0.0;
#pragma unroll
    for (int g = 0; g < 8; ++g) t += red[g][cl];
    part[(int64_t)blk * 33 + 1 + cl] = t;
  }
  __threadfence();
  __syncthreads();
  if (tid == 0) last = atomicAdd(&a.ctr[2], 1) == G - 1;
  __syncthreads();
  if (!last) return;
  __threadfence();
  if (tid < 32 && cl >= nc) {
    double t = 0.0;
    for (int b = 0; b < G; ++b) t += part[(int64_t)b * 33 + 1 + cl];
    red[0][cl] = t;
  }
  __syncthreads();
  if (tid < 32) {
    const double xn = B[(int64_t)nk * C + nk];
    const Reflector h(red[0][nc], xn);
    if (cl > nc && colok) sc[4 + cl] = h.coef(red[0][cl] + h.v0 * B[(int64_t)nk * C + c]);
    if (cl == 0) {
      sc[0] = h.alpha;
      sc[1] = h.beta;
      sc[2] = h.v0;
      sc[3] = xn;
      sc[36] = h.sc;
      betas[nk] = h.beta;
      a.ctr[2] = 0;
    }
  }
}

// The same panel factorisation as qr_col_kernel in one cooperative launch per panel: each
// workgroup keeps its QC_ROWS-row chunk of the panel in registers for all 32 columns, and one grid
// barrier per column replaces a launch.  Per column every workgroup writes its chunk partials
// (|B[k+1:, k+1]|^2, the dots B[k+2:, k+1] . B[k+2:, c], and, for the chunk holding row k+1,
// that row's entries) into one of two alternating buffers, passes the barrier, and sums all
// chunks' partials in chunk order itself, so every workgroup forms the same reflector scalars
// with the additions of the per-launch path (row k+1's entries come from one chunk, the other
// chunks add exact zeros).  The chunk is written back to B after the last column.  Must be
// launched with hipLaunchCooperativeKernel (all workgroups resident); every workgroup of the
// grid passes the same 33 barriers whatever its matrix.  Scratch: 2 x 65 partials per chunk at
// qws[2048 ..).  grid (chunks, 1, matrices), 256 threads.
constexpr int QC_GROUP = 64;
__global__ __launch_bounds__(256) void qr_panel_coop_kernel(const SvdMat *mats, int k0) {
  __shared__ double pl[QC_GROUP * 64];
  __shared__ double red[8][33];
  __shared__ double rowv[32];
  __shared__ double scs[4 + 32 + 1];
  cooperative_groups::grid_group grid = cooperative_groups::this_grid();
  const SvdMat &a = mats[blockIdx.z];
  const int R = a.R, C = a.C;
  const bool on = a.active && a.precond && k0 < a.Ra && k0 < R;
  const int kend = k0 + 32 < R ? k0 + 32 : R, cend = k0 + 32 < C ? k0 + 32 : C;
  const int G = on ? (R - k0 + QC_ROWS - 1) / QC_ROWS : 0, blk = blockIdx.x;
  const bool mine = blk < G;
  const int tid = threadIdx.x, lane = tid & 63, cl = tid & 31, rsub = tid >> 5;
  const int c = k0 + cl;
  const bool colok = c < cend;
  double *B = a.bw;
  double *part = a.qws + 2048, *betas = a.qws + 2048 + 64 * (int64_t)C;
  double val[QC_ROWS / 8];
  if (mine) {
    // reflector rows k0 .. kend-1 start as zero (column k writes its entries from row k on)
    const int64_t tot = (int64_t)(kend - k0) * R;
    for (int64_t e = (int64_t)blk * 256 + tid; e < tot; e += (int64_t)G * 256) a.qv[(int64_t)k0 * R + e] = 0.0;
    if (blk == 0 && tid == 0) a.fro2[1] = 0.0;  // trailing-row maximum of this panel (qr_tail_kernel)
  }
#pragma unroll
  for (int m = 0; m < QC_ROWS / 8; ++m) {
    const int i = k0 + blk * QC_ROWS + rsub + 8 * m;
    val[m] = (mine && i < R && colok) ? B[(int64_t)i * C + c] : 0.0;
  }
  for (int it = 0; it <= 32; ++it) {
    const int k = k0 - 1 + it;
    if (mine && it > 0 && k < kend) {  // apply reflector k to the chunk
      const int kc = k - k0;
      const double alpha = scs[0], beta = scs[1], vk = scs[2], x0 = scs[3], vsc = scs[36];
      const double wc = (cl > kc && colok) ? scs[4 + cl] : 0.0;
#pragma unroll
      for (int m = 0; m < QC_ROWS / 8; ++m) {
        const int i = k0 + blk * QC_ROWS + rsub + 8 * m;
        double x = val[m];
        const double bk = __shfl(x, (lane & 32) | kc, 64);  // this row's column-k entry
        if (i < R && i >= k && colok && cl >= kc) {
          const double vi = (i == k) ? vk : bk;
          if (cl > kc) {
            x -= wc * vi;
          } else {
            x = (i == k) ? (beta != 0.0 ? alpha : x0) : 0.0;
            a.qv[(int64_t)k * R + i] = vi * vsc;
          }
        }
        val[m] = x;
      }
    }
    const int nk = k + 1, nc = nk - k0;
    const bool more = mine && nk < kend;
    double *pp = part + (int64_t)(it & 1) * G * 65;
    if (more) {
      double acc = 0.0;
#pragma unroll
      for (int m = 0; m < QC_ROWS / 8; ++m) {
        const int i = k0 + blk * QC_ROWS + rsub + 8 * m;
        const double y = val[m];
        const double ynk = __shfl(y, (lane & 32) | nc, 64);
        if (i < R && i >= nk) {
          if (cl == nc) acc += y * y;                    // |B[nk:, nk]|^2
          else if (cl > nc && i > nk) acc += ynk * y;    // B[nk+1:, nk] . B[nk+1:, c]
        }
      }
      red[rsub][cl] = acc;
      __syncthreads();
      if (tid < 32) {
        double t = 0.0;
#pragma unroll
        for (int g = 0; g < 8; ++g) t += red[g][cl];
        pp[(int64_t)blk * 65 + 1 + cl] = cl >= nc ? t : 0.0;
      }
      // row nk's entries from the chunk that holds the row, exact zeros from the others
      const int own = (nk - k0) / QC_ROWS, ro = (nk - k0) % QC_ROWS;
      if (blk != own) {
        if (tid < 32) pp[(int64_t)blk * 65 + 33 + cl] = 0.0;
      } else if (rsub == ro % 8) {
#pragma unroll
        for (int m = 0; m < QC_ROWS / 8; ++m)
          if (m == ro / 8) pp[(int64_t)blk * 65 + 33 + cl] = colok ? val[m] : 0.0;
      }
    }
    grid.sync();  // device-scope release and acquire: the partials written above are visible after it
    if (more) {
      // the chunks' partials come in through LDS, QC_GROUP chunks at a time with every thread
      // loading (the far-memory latency paid once per group), and are summed in chunk order
      double t = 0.0;
      for (int b0 = 0; b0 < G; b0 += QC_GROUP) {
        const int nb = G - b0 < QC_GROUP ? G - b0 : QC_GROUP;
        for (int e = tid; e < nb * 64; e += 256) pl[e] = pp[(int64_t)(b0 + (e >> 6)) * 65 + 1 + (e & 63)];
        __syncthreads();
        if (tid < 64)
          for (int b = 0; b < nb; ++b) t += pl[b * 64 + tid];
        __syncthreads();
      }
      if (tid < 64) {
        if (tid < 32) red[0][tid] = t;
        else rowv[tid - 32] = t;
      }
      __syncthreads();
      if (tid < 32) {
        const double xn = rowv[nc];
        const Reflector h(red[0][nc], xn);
        if (cl > nc && colok) scs[4 + cl] = h.coef(red[0][cl] + h.v0 * rowv[cl]);
        if (cl == 0) {
          scs[0] = h.alpha;
          scs[1] = h.beta;
          scs[2] = h.v0;
          scs[3] = xn;
          scs[36] = h.sc;
          if (blk == 0) betas[nk] = h.beta;
        }
      }
      __syncthreads();
    }
  }
  if (mine) {
#pragma unroll
    for (int m = 0; m < QC_ROWS / 8; ++m) {
      const int i = k0 + blk * QC_ROWS + rsub + 8 * m;
      if (i < R && colok) B[(int64_t)i * C + c] = val[m];
    }
  }
}

// The same panel factorisation for at most 1024 rows below k0, in one workgroup: no grid barriers, the
// whole panel in registers.  Wave w holds the rows 64 w + 4 m + lk (m < 16, lk = lane / 16) at the columns
// lr and lr + 16 (lr = lane % 16); a column's entries reach the other columns of their rows by a
// DPP row broadcast, the dots with the other columns are summed over lk and the waves through LDS,
// and the first wave forms the reflector's scalars.  After column k the registers hold R above the diagonal
// and the reflectors on and below it; both are written out at the end.
// Bound by its instructions on one compute unit: per column 16 x (broadcast, two products, two updates) a
// wave and two barriers; 34 to 40 us a panel with 512 threads.  The form with 1024, which has 128 registers a lane,
// keeps 184 B a lane in scratch and takes 77 us.  grid (1, 1, matrices), 64 x waves threads.
constexpr int QP_M = 16, QP_ROWS = 1024;
template <int N>
__device__ inline double row_bcast16(double v) {  // lane N of every 16-lane row to the whole row
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + N, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + N, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
template <int NT>
__global__ __launch_bounds__(NT) void qr_panel_wg_kernel(const SvdMat *mats, int k0) {
  __shared__ double red[NT / 64][4][33];
  __shared__ double rowk[32], ws[32];
  __shared__ double alphas[32], vscs[32], sc_vk;
  const SvdMat &a = mats[blockIdx.z];
  if (!a.active || !a.precond || k0 >= a.Ra || k0 >= a.R) return;
  const int R = a.R, C = a.C, K = R - k0;
  const int ncol = C - k0 < 32 ? C - k0 : 32, nref = K < 32 ? K : 32;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  double *B = a.bw + (int64_t)k0 * C + k0;
  double *betas = a.qws + 2048 + 64 * (int64_t)C + k0;
  if (tid == 0) a.fro2[1] = 0.0;  // trailing-row maximum of this panel (qr_tail_kernel)
  double val[QP_M][2];
#pragma unroll
  for (int m = 0; m < QP_M; ++m) {
    const int i = 64 * wave + 4 * m + lk;
#pragma unroll
    for (int h = 0; h < 2; ++h) val[m][h] = (i < K && lr + 16 * h < ncol) ? B[(int64_t)i * C + lr + 16 * h] : 0.0;
  }
  static_for<0, 32>([&](auto kc_c) {
    constexpr int kc = kc_c, kh = kc / 16, kl = kc % 16, km = kc / 4, kk = kc % 4;
    if (kc < nref) {  // uniform
      // x: column kc's entries of this lane's rows, zero above row kc
      double x[QP_M];
      double s0 = 0.0, s1 = 0.0;
      static_for<0, QP_M>([&](auto m) {
        double v = row_bcast16<kl>(val[m][kh]);
        if constexpr (m < 8) v = (wave == 0 && 4 * m + lk < kc) ? 0.0 : v;
        x[m] = v;
        s0 = fma(v, val[m][0], s0);
        s1 = fma(v, val[m][1], s1);
      });
      red[wave][lk][lr] = s0;
      red[wave][lk][lr + 16] = s1;
      if (wave == 0 && lk == kk) {
        rowk[lr] = val[km][0];
        rowk[lr + 16] = val[km][1];
      }
      __syncthreads();
      if (wave == 0) {  // lanes: column lane % 32, halves of the partials
        const int c = lane & 31, half = lane >> 5;
        double t = 0.0;
        for (int w = 0; w < nw; ++w) t += red[w][2 * half][c] + red[w][2 * half + 1][c];
        t += __shfl_xor(t, 32, 64);
        const double xn = rowk[kc];
        const Reflector h(__shfl(t, kc, 64), xn);
        if (lane < 32) ws[c] = c > kc ? h.coef(t - h.alpha * rowk[c]) : 0.0;
        if (lane == 0) {
          alphas[kc] = h.beta != 0.0 ? h.alpha : xn;
          vscs[kc] = h.sc;
          sc_vk = h.v0;
          betas[kc] = h.beta;
        }
      }
      __syncthreads();
      const double w0 = ws[lr], w1 = ws[lr + 16], vk = sc_vk;
      static_for<0, QP_M>([&](auto m) {
        double v = x[m];
        if constexpr (m == km) v = (wave == 0 && lk == kk) ? vk : v;  // the reflector's own entry of row kc
        val[m][0] = fma(-w0, v, val[m][0]);
        val[m][1] = fma(-w1, v, val[m][1]);
        if constexpr (m == km) val[m][kh] = (wave == 0 && lk == kk && lr == kl) ? vk : val[m][kh];
      });
    }
  });
  // R on and above the diagonal to B, the reflectors as rows to qv (from column k0 on, which is all
  // their readers look at)
  double *qv = a.qv + (int64_t)k0 * R;
#pragma unroll
  for (int m = 0; m < QP_M; ++m) {
    const int i = 64 * wave + 4 * m + lk;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = lr + 16 * h;
      if (i < K && c < ncol) {
        const double v = val[m][h];
        B[(int64_t)i * C + c] = i < c ? v : i == c ? alphas[c] : 0.0;
        if (c < nref) qv[(int64_t)c * R + k0 + i] = i < c ? 0.0 : v * vscs[c];
      }
    }
  }
}

// ---- the panel's block reflector I - V T V^T applied from the left, X <- X - V^T W2 with V as 32 rows
// of length K, in three launches over all matrices: W = V X and S = V V^T in pieces of K (qr_wy_kernel),
// the pieces summed in order and W2 = T^T W by forward substitution (qr_wy_solve_kernel: T^-1 has 1 / beta on
// its diagonal and S above it, so W2_i = beta_i (W_i - sum_{j<i} S_ji W2_j) and T is never formed),
// and the update (qr_wy_update_kernel).  X is the trailing columns of B (on_b) or all of Jt.
// MFMA operands come straight from L2, where V, W2 and a tile of X stay.  Scratch in qws: S pieces at
// [2048 ..), W2 (32 x N) at [2048 + 32 C ..), W pieces (32 x N each) behind the betas.
// Measured at 331 x 517: 58 us a panel in seven launches per matrix with T formed column by column,
// about 15 us in this form.
struct WyX {
  double *X;
  int ld, N, K, nref;
  const double *V;
};
__device__ inline bool wy_operands(const SvdMat &a, int k0, bool on_b, WyX &o) {
  if (!a.active || !a.precond || k0 >= a.Ra || (on_b && k0 + 32 >= a.C)) return false;
  o.K = a.R - k0;
  o.nref = o.K < 32 ? o.K : 32;
  o.V = a.qv + (int64_t)k0 * a.R + k0;
  o.X = on_b ? a.bw + (int64_t)k0 * a.C + k0 + 32 : a.jt + (int64_t)k0 * a.R;
  o.ld = on_b ? a.C : a.R;
  o.N = on_b ? a.C - k0 - 32 : a.R;
  return true;
}
// grid (64-column tiles of X and, last, the S tile, pieces, matrices), 256 threads: a wave 16 columns
__global__ __launch_bounds__(256) void qr_wy_kernel(const SvdMat *mats, int k0, int on_b, int kc) {
  const SvdMat &a = mats[blockIdx.z];
  WyX o;
  if (!wy_operands(a, k0, on_b != 0, o)) return;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, wave = threadIdx.x >> 6;
  const int nt = (o.N + 63) / 64, piece = blockIdx.y;
  const bool is_s = blockIdx.x == gridDim.x - 1;
  if (!is_s && (int)blockIdx.x >= nt) return;
  if (is_s && wave >= 2) return;
  const int kb = piece * kc, ke = kb + kc < o.K ? kb + kc : o.K;
  const int c = is_s ? 16 * wave + lr : 64 * blockIdx.x + 16 * wave + lr;
  const int R = a.R, r0 = lr < o.nref ? lr : 0, r1 = lr + 16 < o.nref ? lr + 16 : 0;  // rows past nref: discarded
  const int cc = is_s ? (c < o.nref ? c : 0) : (c < o.N ? c : o.N - 1);
  v4d acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
  constexpr int UN = 8;
  for (int k = kb; k < ke; k += 4 * UN) {
    double v0[UN], v1[UN], x[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      const int kk = k + 4 * u + lk;
      const bool in = kk < ke;
      v0[u] = in ? o.V[(int64_t)r0 * R + kk] : 0.0;
      v1[u] = in ? o.V[(int64_t)r1 * R + kk] : 0.0;
      x[u] = in ? (is_s ? o.V[(int64_t)cc * R + kk] : o.X[(int64_t)kk * o.ld + cc]) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      acc0 = mfma16(v0[u], x[u], acc0);
      acc1 = mfma16(v1[u], x[u], acc1);
    }
  }
  const int N = is_s ? 32 : o.N;
  double *out = is_s ? a.qws + 2048 + (int64_t)piece * 1024
                     : a.qws + 2048 + 64 * (int64_t)a.C + 2 * (int64_t)R + (int64_t)piece * 32 * o.N;
  if (c < N) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      out[(int64_t)(4 * r + lk) * N + c] = acc0[r];
      out[(int64_t)(16 + 4 * r + lk) * N + c] = acc1[r];
    }
  }
}
// grid (64-column tiles, 1, matrices), 256 threads
__global__ __launch_bounds__(256) void qr_wy_solve_kernel(const SvdMat *mats, int k0, int on_b, int kc) {
  __shared__ double St[32][34];  // St[i][j] = S[j][i]
  __shared__ double Ws[32][65];
  const SvdMat &a = mats[blockIdx.z];
  WyX o;
  if (!wy_operands(a, k0, on_b != 0, o)) return;
  const int c0 = 64 * blockIdx.x, tid = threadIdx.x;
  if (c0 >= o.N) return;
  const int np = (o.K + kc - 1) / kc;
  const double *sp = a.qws + 2048, *wp = a.qws + 2048 + 64 * (int64_t)a.C + 2 * (int64_t)a.R;
  // every piece's loads are in flight before the first sum
  const int col = tid & 63;
  const int cn = c0 + col < o.N ? c0 + col : o.N - 1;
  double sv[QR_SPLIT][4], wv[QR_SPLIT][8];
#pragma unroll
  for (int p = 0; p < QR_SPLIT; ++p) {
#pragma unroll
    for (int u = 0; u < 4; ++u) sv[p][u] = p < np ? sp[p * 1024 + tid + 256 * u] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) wv[p][u] = p < np ? wp[((int64_t)p * 32 + (tid >> 6) + 4 * u) * o.N + cn] : 0.0;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int e = tid + 256 * u;
    double v = 0.0;
#pragma unroll
    for (int p = 0; p < QR_SPLIT; ++p) v += sv[p][u];
    St[e & 31][e >> 5] = v;
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    double v = 0.0;
#pragma unroll
    for (int p = 0; p < QR_SPLIT; ++p) v += wv[p][u];
    Ws[(tid >> 6) + 4 * u][col] = v;
  }
  __syncthreads();
  if (tid >= 64) return;
  const double *betas = a.qws + 2048 + 64 * (int64_t)a.C + k0;
  double *W2 = a.qws + 2048 + 32 * (int64_t)a.C;
  double w[32], be[32];
  static_for<0, 32>([&](auto i) { be[i] = i < o.nref ? betas[i] : 0.0; });
  static_for<0, 32>([&](auto i) {
    double v = Ws[i][tid];
    static_for<0, i>([&](auto j) { v = fma(-St[i][j], w[j], v); });
    w[i] = be[i] * v;
    if (c0 + tid < o.N) W2[(int64_t)i * o.N + c0 + tid] = w[i];
  });
}
// grid (64-column tiles, 64-row tiles, matrices), 256 threads: a wave 16 rows
__global__ __launch_bounds__(256) void qr_wy_update_kernel(const SvdMat *mats, int k0, int on_b) {
  const SvdMat &a = mats[blockIdx.z];
  WyX o;
  if (!wy_operands(a, k0, on_b != 0, o)) return;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4, wave = threadIdx.x >> 6;
  const int c0 = 64 * blockIdx.x, i0 = 64 * blockIdx.y + 16 * wave;
  if (c0 >= o.N || i0 >= o.K) return;
  const double *W2 = a.qws + 2048 + 32 * (int64_t)a.C;
  const int i = i0 + lr < o.K ? i0 + lr : o.K - 1;
  double av[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int r = 4 * u + lk;
    av[u] = r < o.nref ? o.V[(int64_t)r * a.R + i] : 0.0;
  }
  double bv[4][8];
  v4d acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = c0 + 16 * t + lr, cn = c < o.N ? c : o.N - 1;
#pragma unroll
    for (int u = 0; u < 8; ++u) bv[t][u] = W2[(int64_t)(4 * u + lk) * o.N + cn];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = i0 + 4 * r + lk;
      acc[t][r] = (row < o.K && c < o.N) ? -o.X[(int64_t)row * o.ld + c] : 0.0;
    }
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int u = 0; u < 8; ++u) acc[t] = mfma16(av[u], bv[t][u], acc[t]);
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int c = c0 + 16 * t + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = i0 + 4 * r + lk;
      if (row < o.K && c < o.N) o.X[(int64_t)row * o.ld + c] = -acc[t][r];
    }
  }
}

// grid (ceil((R - k1) / 4), 1, matrices): fro2[1] <- the largest squared norm of the rows k1.. of B
// after the panels before k1 (their entries left of column k1 are zero), one wave per row.  Run
// only while the QR start of a rows_scaled matrix is still going; the maximum is taken on the bit
// patterns of the non-negative sums, which order like the values.
__global__ __launch_bounds__(256) void qr_tail_kernel(const SvdMat *mats, int k1) {
  const SvdMat &a = mats[blockIdx.z];
  if (!a.active || !a.precond || !a.rows_scaled || k1 >= a.Ra) return;
  const int r = k1 + blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (r >= a.R) return;
  const double *row = a.bw + (int64_t)r * a.C;
  double ss = 0.0;
  for (int c = k1 + lane; c < a.C; c += 64) ss += row[c] * row[c];
  ss = wave_sum_d(ss);
  if (lane == 0)
    atomicMax(reinterpret_cast<unsigned long long *>(a.fro2 + 1), (unsigned long long)__double_as_longlong(ss));
}

// grid (column blocks, 1, matrices)
__global__ __launch_bounds__(256) void qr_pinv_kernel(const SvdMat *mats) {
  const SvdMat &a = mats[blockIdx.z];
  if (!a.active || !a.precond) return;
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c < a.C) a.pinv[a.cperm[c]] = c;
}

// -------------------------------------------------------------- finish
// grid (ceil(R/4), 1, matrices): sigma_r = |row r|, one wave per row
__global__ __launch_bounds__(256) void norms_kernel(const SvdMat *mats) {
  const SvdMat &a = mats[blockIdx.z];
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (a.fused == 2 || r >= a.R) return;
  const double *row = a.bw + (int64_t)r * a.C;
  double s = 0.0;
  for (int c = lane; c < a.C; c += 64) s += row[c] * row[c];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane == 0) a.sig[r] = sqrt(s);
}

// one block per matrix: bitonic sort of (sigma desc, index asc), then Z and the entropy
__global__ __launch_bounds__(1024) void sort_kernel(const SvdMat *mats) {
  __shared__ double key[4096];
  __shared__ int idx[4096];
  __shared__ double red[16];
  const SvdMat &a = mats[blockIdx.x];
  if (a.fused == 2) return;
  int P = 1;
  while (P < a.R) P <<= 1;
  for (int i = threadIdx.x; i < P; i += 1024) {
    key[i] = i < a.R ? sort_key(a.sig[i]) : -1.0;
    idx[i] = i;
  }
  __syncthreads();
  for (int k = 2; k <= P; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < P; i += 1024) {
        const int l = i ^ j;
        if (l > i) {
          const bool i_before_l = key[i] > key[l] || (key[i] == key[l] && idx[i] < idx[l]);
          const bool up = (i & k) == 0;
          if (up ? !i_before_l : i_before_l) {
            const double tk = key[i]; key[i] = key[l]; key[l] = tk;
            const int ti = idx[i]; idx[i] = idx[l]; idx[l] = ti;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int i = threadIdx.x; i < a.R; i += 1024) {
    a.perm[i] = idx[i];
    key[i] = a.sig[idx[i]];
    a.S[i] = key[i];
  }
  __syncthreads();
  // Z = sum S^2 and S_vN = -sum p ln p (p = S^2 / Z), fixed-order block sums
  double z2 = 0.0;
  for (int i = threadIdx.x; i < a.R; i += 1024) z2 += key[i] * key[i];
  for (int off = 32; off > 0; off >>= 1) z2 += __shfl_xor(z2, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = z2;
  __syncthreads();
  double Z = 0.0;
  for (int w = 0; w < 16; ++w) Z += red[w];
  __syncthreads();
  double e = 0.0;
  for (int i = threadIdx.x; i < a.R; i += 1024) {
    const double p = key[i] * key[i] / Z;
    if (p > 0.0) e -= p * log(p);
  }
  for (int off = 32; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
  __syncthreads();
  if (threadIdx.x == 0) {
    double ent = 0.0;
    for (int w = 0; w < 16; ++w) ent += red[w];
    a.spec[0] = Z;
    a.spec[1] = ent;
  }
  if (threadIdx.x < 16) a.spec[8 + threadIdx.x] = (int)threadIdx.x < a.R ? key[threadIdx.x] : 0.0;
  // spec[7]: sweeps of the single-workgroup Jacobi paths, negative when not converged (0 otherwise)
  if (threadIdx.x == 0) a.spec[7] = a.fused ? (a.ctr[0] ? -(double)a.ctr[1] : (double)a.ctr[1]) : 0.0;
  // spec[24] (thr > 0 only): how many values exceed thr, for threshold truncation
  if (a.thr > 0.0) {
    __shared__ int cnt_w[16];
    int cnt = 0;
    for (int i = threadIdx.x; i < a.R; i += 1024) cnt += key[i] > a.thr;
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    if ((threadIdx.x & 63) == 0) cnt_w[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
      int c = 0;
      for (int w = 0; w < 16; ++w) c += cnt_w[w];
      a.spec[24] = (double)c;
    }
  }
  // spec[25]: numerical rank, the number of values above 1e-12 S_0
  {
    __shared__ int nr_w[16];
    const double cut = (a.noise_rel > 0.0 ? a.noise_rel : 1e-12) * key[0];
    int cnt = 0;
    for (int i = threadIdx.x; i < a.R; i += 1024) cnt += key[i] > cut;
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    if ((threadIdx.x & 63) == 0) nr_w[threadIdx.x >> 6] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
      int c = 0;
      for (int w = 0; w < 16; ++w) c += nr_w[w];
      a.spec[25] = (double)c;
    }
  }
  // spec[6]: smallest k >= 1 with sqrt(sum_{j>=k} S_j^2) <= eps_target (k = R always qualifies)
  if (a.eps_target > 0.0) {
    __shared__ double csum[1024];
    __shared__ int best[16];
    const int t = threadIdx.x, R = a.R;
    const double eps2 = a.eps_target * a.eps_target;
    const int L = (R + 1023) / 1024;
    const int beg = t * L, end = beg + L < R ? beg + L : R;
    double c = 0.0;
    for (int j = beg; j < end; ++j) c += key[j] * key[j];
    // sums over the chunks after this one: inclusive suffix scan in a fixed tree order
    double v = c;
    for (int off = 1; off < 1024; off <<= 1) {
      csum[t] = v;
      __syncthreads();
      if (t + off < 1024) v += csum[t + off];
      __syncthreads();
    }
    csum[t] = v;
    __syncthreads();
    const double after = t + 1 < 1024 ? csum[t + 1] : 0.0;
    int kmin = R;
    double tsum = after;
    for (int j = end - 1; j >= beg; --j) {
      tsum += key[j] * key[j];
      if (tsum <= eps2) kmin = j;
    }
    if (kmin < 1) kmin = 1;
    for (int off = 32; off > 0; off >>= 1) kmin = min(kmin, __shfl_xor(kmin, off, 64));
    if ((t & 63) == 0) best[t >> 6] = kmin;
    __syncthreads();
    if (t == 0) {
      int b = best[0];
      for (int w = 1; w < 16; ++w) b = min(b, best[w]);
      a.spec[6] = (double)b;
    }
  }
}

// one block per matrix: spec[2..5] for the kept rank k
__global__ __launch_bounds__(256) void trunc_kernel(const SvdMat *mats) {
  __shared__ double red[4];
  const SvdMat &a = mats[blockIdx.x];
  if (a.k < 1 || a.fused == 2) return;
  const double *s = a.S;
  const int R = a.R, k = a.k, t = threadIdx.x;
  double tl = 0.0, hd = 0.0;
  for (int i = t; i < R; i += 256) {
    if (i >= k) tl += s[i] * s[i];
    else hd += s[i] * s[i];
  }
  const double tail = bsum256(tl, red);
  const double head = bsum256(hd, red);
  if (t == 0) {
    const double Z = a.spec[0];
    a.spec[2] = sqrt(tail);
    a.spec[3] = tail / Z;
    a.spec[4] = sqrt(head);
    a.spec[5] = (k < R && s[0] > 0.0) ? (s[k - 1] - s[k]) / s[0] : 1.0;
    a.spec[26] = s[k - 1];
  }
}

// Kept values at or below this are null: at the rounding level of sigma_0 or under the
// Jacobi row floor (whose rows were never orthogonalised against the others).  With the
// QR start (rows_scaled off) that floor is far lower.
__device__ inline double null_threshold(const SvdMat &a) {
  if (a.precond && !a.rows_scaled) return sqrt(row_floor2(a, *a.fro2));
  const double C = (double)(a.m > a.n ? a.m : a.n);
  return EPS53 * C * fmax(a.S[0], 0.1 * sqrt(*a.fro2));
}

// U (m x k) and Vt (k x n), unscaled; null Bw-derived vectors are zeroed.
// grid (chunks, 2, matrices): y = 0 writes U, y = 1 writes Vt
template <typename T>
__device__ inline void write_factors(const SvdMat &a, int which, int64_t e0, int64_t stride) {
  const double thr = null_threshold(a);
  if (which == 0) {
    T *U = static_cast<T *>(a.U);
    const int64_t total = (int64_t)a.m * a.k;
    for (int64_t e = e0; e < total; e += stride) {
      const int i = (int)(e / a.k), j = (int)(e % a.k);
      const int r = a.perm[j];
      double v;
      if (!a.trans) v = a.jt[(int64_t)r * a.R + i];
      else v = (a.S[j] > thr && a.S[j] > 0.0) ? a.bw[(int64_t)r * a.C + (a.pinv ? a.pinv[i] : i)] / a.S[j] : 0.0;
      U[e] = (T)v;
    }
  } else {
    T *Vt = static_cast<T *>(a.Vt);
    const int64_t total = (int64_t)a.k * a.n;
    for (int64_t e = e0; e < total; e += stride) {
      const int j = (int)(e / a.n), c = (int)(e % a.n);
      const int r = a.perm[j];
      double v;
      if (a.trans) v = a.jt[(int64_t)r * a.R + c];
      else v = (a.S[j] > thr && a.S[j] > 0.0) ? a.bw[(int64_t)r * a.C + (a.pinv ? a.pinv[c] : c)] / a.S[j] : 0.0;
      Vt[e] = (T)v;
    }
  }
}

__global__ __launch_bounds__(256) void write_kernel(const SvdMat *mats) {
  const SvdMat &a = mats[blockIdx.z];
  if (a.k < 1 || a.fused == 2) return;
  const int64_t e0 = (int64_t)blockIdx.x * 256 + threadIdx.x, stride = (int64_t)gridDim.x * 256;
  if (a.out_type == TNA_F64) write_factors<double>(a, blockIdx.y, e0, stride);
  else write_factors<float>(a, blockIdx.y, e0, stride);
}

// Gram-Schmidt completion of kept null vectors with unit vectors e_0, e_1, ...
// (Vt rows when rows of A were orthogonalised, U columns otherwise); one block per matrix.  A unit vector is taken
// when more than half of its length is left.  A complement of few dimensions may hold no such one, but always one
// with more than 1 / sqrt(L): when none is left the search starts again with half of that.
template <typename T>
__device__ void complete_one(const SvdMat &a, double *vec, double *red, int *ok) {
  const double thr = null_threshold(a);
  const int L = a.trans ? a.m : a.n;
  T *base;
  int64_t es, vs;
  if (a.trans) { base = static_cast<T *>(a.U); es = a.k; vs = 1; }
  else { base = static_cast<T *>(a.Vt); es = 1; vs = a.n; }
  const int tid = threadIdx.x;
  int e = 0, again = 0;
  double least = 0.5;
  for (int j = 0; j < a.k; ++j) {
    if (a.S[j] > thr && a.S[j] > 0.0) continue;
    for (;; ++e) {
      if (e == L) {
        if (again) break;
        again = 1;
        least = 0.5 / sqrt((double)L);
        e = 0;
      }
      for (int i = tid; i < L; i += 256) vec[i] = (i == e) ? 1.0 : 0.0;
      __syncthreads();
      for (int pass = 0; pass < 2; ++pass)
        for (int qv = 0; qv < a.k; ++qv) {
          if (qv == j) continue;
          if (!((a.S[qv] > thr && a.S[qv] > 0.0) || qv < j)) continue;
          double h = 0.0;
          for (int i = tid; i < L; i += 256) h += (double)base[qv * vs + (int64_t)i * es] * vec[i];
          h = bsum256(h, red);
          for (int i = tid; i < L; i += 256) vec[i] -= h * (double)base[qv * vs + (int64_t)i * es];
          __syncthreads();
        }
      double nr = 0.0;
      for (int i = tid; i < L; i += 256) nr += vec[i] * vec[i];
      nr = sqrt(bsum256(nr, red));
      if (tid == 0) *ok = nr > least;
      __syncthreads();
      const int good = *ok;
      __syncthreads();
      if (good) {
        for (int i = tid; i < L; i += 256) base[j * vs + (int64_t)i * es] = (T)(vec[i] / nr);
        __syncthreads();
        ++e;
        break;
      }
    }
  }
}

__global__ __launch_bounds__(256) void complete_kernel(const SvdMat *mats) {
  __shared__ double vec[4096];
  __shared__ double red[4];
  __shared__ int ok;
  const SvdMat &a = mats[blockIdx.x];
  if (a.k < 1 || a.fused == 2 || a.rows_scaled) return;  // the factor to complete leaves scaled by (near-)zero values
  // only matrices with a kept null vector do any work
  const double thr = null_threshold(a);
  if (a.S[a.k - 1] > thr && a.S[a.k - 1] > 0.0) return;
  if (a.out_type == TNA_F64) complete_one<double>(a, vec, red, &ok);
  else complete_one<float>(a, vec, red, &ok);
}

// sign gauge (largest-|.| entry of U[:, j] positive, ties: lowest row), then
// scaling by S_j/|S_k| of Vt rows (scale_mode 1) or U columns (scale_mode 2)
template <typename T>
__device__ void gauge_one(const SvdMat &a, int j, double *bv, int *bi, double *sgn) {
  const int tid = threadIdx.x;
  T *U = static_cast<T *>(a.U);
  T *Vt = static_cast<T *>(a.Vt);
  double best = -1.0;
  int bidx = 0x7fffffff;
  for (int i = tid; i < a.m; i += 256) {
    const double v = fabs((double)U[(int64_t)i * a.k + j]);
    if (v > best) { best = v; bidx = i; }
  }
  for (int off = 32; off > 0; off >>= 1) {
    const double ov = __shfl_xor(best, off, 64);
    const int oi = __shfl_xor(bidx, off, 64);
    if (ov > best || (ov == best && oi < bidx)) { best = ov; bidx = oi; }
  }
  if ((tid & 63) == 0) { bv[tid >> 6] = best; bi[tid >> 6] = bidx; }
  __syncthreads();
  if (tid == 0) {
    double b = bv[0];
    int ii = bi[0];
    for (int w = 1; w < 4; ++w)
      if (bv[w] > b || (bv[w] == b && bi[w] < ii)) { b = bv[w]; ii = bi[w]; }
    // (a column without a comparable entry has no largest one)
    *sgn = (ii < a.m && (double)U[(int64_t)ii * a.k + j] < 0.0) ? -1.0 : 1.0;
  }
  __syncthreads();
  const double nk = a.spec[4];
  const double f = (a.scale_mode != 0 && nk > 0.0) ? a.S[j] / nk : 1.0;
  const double fu = *sgn * (a.scale_mode == 2 ? f : 1.0);
  const double fv = *sgn * (a.scale_mode == 1 ? f : 1.0);
  if (fu != 1.0)
    for (int i = tid; i < a.m; i += 256) U[(int64_t)i * a.k + j] = (T)((double)U[(int64_t)i * a.k + j] * fu);
  if (fv != 1.0)
    for (int c = tid; c < a.n; c += 256) Vt[(int64_t)j * a.n + c] = (T)((double)Vt[(int64_t)j * a.n + c] * fv);
}

// grid (max k, 1, matrices)
__global__ __launch_bounds__(256) void gauge_kernel(const SvdMat *mats) {
  __shared__ double bv[4];
  __shared__ int bi[4];
  __shared__ double sgn;
  const SvdMat &a = mats[blockIdx.z];
  const int j = blockIdx.x;
  if (j >= a.k || a.fused == 2) return;
  if (a.out_type == TNA_F64) gauge_one<double>(a, j, bv, bi, &sgn);
  else gauge_one<float>(a, j, bv, bi, &sgn);
}

// The outputs of a matrix of at most 32 rows and 64 columns (fused == 2) in one workgroup: truncation sums,
// U and Vt through LDS, gauge and scaling; the rare matrix with kept null vectors to complete goes
// through the general steps on its outputs instead.
template <typename T>
__device__ void finish_small(const SvdMat &a, double (*Us)[33], double (*Vs)[65], double *sc, double *red, double *vec,
                             int *ok) {
  const int tid = threadIdx.x, m = a.m, n = a.n, k = a.k, R = a.R, C = a.C;
  T *U = static_cast<T *>(a.U);
  T *Vt = static_cast<T *>(a.Vt);
  const double thr = null_threshold(a);
  if (tid < 64) {
    const double s = tid < R ? a.S[tid] : 0.0;
    const double tail = wave_sum_d(tid >= k ? s * s : 0.0), head = wave_sum_d(tid < k ? s * s : 0.0);
    const double s0 = __shfl(s, 0, 64), sk1 = __shfl(s, k - 1, 64), sk = __shfl(s, k < 64 ? k : 63, 64);
    if (tid == 0) {
      a.spec[2] = sqrt(tail);
      a.spec[3] = tail / a.spec[0];
      a.spec[4] = sqrt(head);
      a.spec[5] = (k < R && s0 > 0.0) ? (sk1 - sk) / s0 : 1.0;
      a.spec[26] = sk1;
      sc[0] = sqrt(head);
    }
  }
  // the rotations give one factor, the rows over their norms the other
  auto from_rows = [&](int j, int c) {
    const double s = a.S[j];
    return (s > thr && s > 0.0) ? a.bw[a.perm[j] * C + c] / s : 0.0;
  };
  auto from_rot = [&](int j, int c) { return a.jt[a.perm[j] * R + c]; };
  for (int e = tid; e < k * m; e += 256) {
    const int j = e / m, i = e - j * m;
    Us[i][j] = a.trans ? from_rows(j, i) : from_rot(j, i);
  }
  for (int e = tid; e < k * n; e += 256) {
    const int j = e / n, c = e - j * n;
    Vs[j][c] = a.trans ? from_rot(j, c) : from_rows(j, c);
  }
  __syncthreads();
  const bool complete = !a.rows_scaled && !(a.S[k - 1] > thr && a.S[k - 1] > 0.0);
  if (complete) {
    for (int e = tid; e < m * k; e += 256) U[e] = (T)Us[e / k][e % k];
    for (int e = tid; e < k * n; e += 256) Vt[e] = (T)Vs[e / n][e % n];
    __syncthreads();
    complete_one<T>(a, vec, red, ok);
    __syncthreads();
    for (int e = tid; e < m * k; e += 256) Us[e / k][e % k] = (double)U[e];
    for (int e = tid; e < k * n; e += 256) Vs[e / n][e % n] = (double)Vt[e];
    __syncthreads();
  }
  {  // eight lanes per column of U: its largest entry, ties to the lowest row
    const int j = tid >> 3;
    double best = -1.0;
    int at = 0x7fffffff;
    if (j < k)
      for (int i = tid & 7; i < m; i += 8) {
        const double v = fabs((double)(T)Us[i][j]);
        if (v > best) { best = v; at = i; }
      }
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) {
      const double ov = __shfl_xor(best, off, 64);
      const int oi = __shfl_xor(at, off, 64);
      if (ov > best || (ov == best && oi < at)) { best = ov; at = oi; }
    }
    if (j < k && (tid & 7) == 0) {
      const double sg = at < m && Us[at][j] < 0.0 ? -1.0 : 1.0;
      const double f = (a.scale_mode != 0 && sc[0] > 0.0) ? a.S[j] / sc[0] : 1.0;
      sc[1 + j] = sg * (a.scale_mode == 2 ? f : 1.0);
      sc[33 + j] = sg * (a.scale_mode == 1 ? f : 1.0);
    }
  }
  __syncthreads();
  for (int e = tid; e < m * k; e += 256) U[e] = (T)((double)(T)Us[e / k][e % k] * sc[1 + e % k]);
  for (int e = tid; e < k * n; e += 256) Vt[e] = (T)((double)(T)Vs[e / n][e % n] * sc[33 + e / n]);
}

// grid (matrices)
__global__ __launch_bounds__(256) void finish_small_kernel(const SvdMat *mats) {
  __shared__ double Us[64][33], Vs[32][65];
  __shared__ double sc[1 + 2 * 32], red[4], vec[64];
  __shared__ int ok;
  const SvdMat &a = mats[blockIdx.x];
  if (a.k < 1 || a.fused != 2) return;
  if (a.out_type == TNA_F64) finish_small<double>(a, Us, Vs, sc, red, vec, &ok);
  else finish_small<float>(a, Us, Vs, sc, red, vec, &ok);
}

int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }
constexpr int QR_MIN_ROWS = QR_MIN_ROWS_DEV;

}  // namespace

// ====================================================================== host
tna_status svd_plan_mat(int m, int n, int dtype, int batch_hint, SvdMat *a, int orient) {
  if (m < 1 || n < 1) {
    set_error("svd: dimensions must be positive");
    return TNA_ERR_ARG;
  }
  *a = SvdMat{};
  a->m = m;
  a->n = n;
  a->trans = m > n || (m == n && orient == 2);
  a->R = m < n ? m : n;
  a->C = m < n ? n : m;
  a->Ra = a->R;
  a->dtype = dtype;
  if (a->C > 4096) {
    set_error("svd: max(m,n) > 4096 is not supported");
    return TNA_ERR_UNSUPPORTED;
  }
  int nb = (a->R + BS - 1) / BS;
  if (nb < 2) nb = 2;
  if (nb & 1) ++nb;
  a->nb = nb;
  const int npairs = nb / 2;
  int ks = ceil_div(1024, (int64_t)npairs * (batch_hint > 0 ? batch_hint : 1));
  const int kmax = ceil_div(a->C, 256);
  if (ks > kmax) ks = kmax;
  if (ks < 1) ks = 1;
  a->ksplit = ks;
  // Outer convergence: every off-diagonal |g_ij| <= tol sqrt(g_ii g_jj).  Applying a
  // 64-row block rotation and re-forming the Gram leave a rounding floor of about
  // (64 + C) ulps whatever C is, so the bound sits at twice that floor.
  a->tol = 2.0 * (64.0 + (double)a->C) * EPS53;
  static const int inner_env = [] {
    const char *e = std::getenv("TNA_SVD_INNER");
    return e ? std::atoi(e) : 0;
  }();
  a->fused = (a->R <= 32 && a->C <= 64) ? 2 : ((nb == 2 && a->C <= 1024) ? 1 : 0);
  a->precond = (!a->fused && a->R >= QR_MIN_ROWS) ? 1 : 0;
  // Two inner sweeps per block pair (one after the QR start and in the
  // single-workgroup form) cost few extra outer sweeps and far less than diagonalising
  // each pair
  a->inner_max = inner_env > 0 ? inner_env : ((a->fused || a->precond) ? 1 : 2);
  a->active = 1;
  return TNA_OK;
}

// [2048 ..) S pieces (QR_SPLIT x 32 x 32, at most 32 C), W2 (32 x C); betas (R), scalars of the per-column
// panels (R), then the pieces of W (QR_SPLIT x 32 x C)
static size_t qws_doubles(const SvdMat &a) {
  return 2048 + 64 * (size_t)a.C + 2 * (size_t)a.R + QR_SPLIT * 32 * (size_t)a.C;
}
size_t svd_work_doubles(const SvdMat &a) {
  const size_t npairs = a.nb / 2;
  return (size_t)a.R * a.C + (size_t)a.R * a.R + npairs * a.ksplit * 4096 + npairs * 4096 + a.R + 8 +
         (a.precond ? (size_t)a.R * a.R + qws_doubles(a) : 0);
}
size_t svd_work_ints(const SvdMat &a) { return (size_t)a.nb / 2 + a.R + 4 + (a.precond ? 2 * (size_t)a.C : 0); }

// gram, qt and qws (the Grams of a small group after its QR start) are accessed in 16-byte pairs: they come
// first, from an aligned address on, each an even number of doubles.  The double that may cost comes out of
// fro2's eight, of which two are used.
void svd_bind_work(SvdMat *a, double *dw, int *iw) {
  const size_t npairs = a->nb / 2;
  dw += (reinterpret_cast<uintptr_t>(dw) / sizeof(double)) & 1;
  a->gram = dw;
  dw += npairs * a->ksplit * 4096;
  a->qt = dw;
  dw += npairs * 4096;
  if (a->precond) {
    a->qws = dw;
    dw += qws_doubles(*a);
    a->qv = dw;
    dw += (size_t)a->R * a->R;
  } else {
    a->qv = a->qws = nullptr;
  }
  a->bw = dw;
  dw += (size_t)a->R * a->C;
  a->jt = dw;
  dw += (size_t)a->R * a->R;
  a->sig = dw;
  dw += a->R;
  a->fro2 = dw;
  a->skip = iw;
  iw += npairs;
  a->perm = iw;
  iw += a->R;
  a->ctr = iw;
  iw += 4;
  a->cperm = a->precond ? iw : nullptr;
  a->pinv = a->precond ? iw + a->C : nullptr;
}

// The descriptors through one of SvdGroup::NSTAGE pinned buffers in turn: a buffer is written again only
// when its last copy is done, which with several of them costs no wait in the course of a group.
static tna_status upload(const std::vector<SvdMat> &mats, SvdGroup &g, hipStream_t s) {
  const size_t bytes = sizeof(SvdMat) * mats.size();
  TNA_TRY(g.desc.ensure(bytes));
  SvdGroup::Stage &st = g.stage[g.next_stage];
  g.next_stage = (g.next_stage + 1) % SvdGroup::NSTAGE;
  if (!st.done) TNA_HIP(hipEventCreateWithFlags(&st.done, hipEventDisableTiming));
  else TNA_HIP(hipEventSynchronize(st.done));
  if (st.cap < bytes) {
    if (st.host) (void)hipHostFree(st.host);
    st.host = nullptr;
    st.cap = 0;
    TNA_HIP(hipHostMalloc(&st.host, bytes * 2, hipHostMallocDefault));
    st.cap = bytes * 2;
  }
  std::memcpy(st.host, mats.data(), bytes);
  TNA_HIP(hipMemcpyAsync(g.desc.ptr, st.host, bytes, hipMemcpyHostToDevice, s));
  TNA_HIP(hipEventRecord(st.done, s));
  return TNA_OK;
}

// X[k0:, :] <- (I - V T^T V^T) X[k0:, :] for the 32 reflectors k0.. of every QR-started matrix, X the
// trailing columns of B (on_b) or all of Jt.  K is cut into at most QR_SPLIT pieces, as many as bring
// the first launch to about two workgroups per compute unit.
static tna_status qr_block_apply(const std::vector<SvdMat> &mats, const SvdMat *d, int nm, int k0, bool on_b,
                                 hipStream_t s) {
  int maxk = 0, maxn = 0;
  for (auto &a : mats) {
    if (!a.precond || k0 >= a.Ra || (on_b && k0 + 32 >= a.C)) continue;
    maxk = std::max(maxk, a.R - k0);
    maxn = std::max(maxn, on_b ? a.C - k0 - 32 : a.R);
  }
  if (maxk == 0) return TNA_OK;
  const int nt = ceil_div(maxn, 64);
  int np = std::min(QR_SPLIT, std::max(1, ceil_div(512, (int64_t)nt * nm)));
  np = std::min(np, ceil_div(maxk, 64));
  const int kc = ceil_div(ceil_div(maxk, np), 32) * 32;
  hipLaunchKernelGGL(qr_wy_kernel, dim3(nt + 1, ceil_div(maxk, kc), nm), dim3(256), 0, s, d, k0, on_b ? 1 : 0, kc);
  hipLaunchKernelGGL(qr_wy_solve_kernel, dim3(nt, 1, nm), dim3(256), 0, s, d, k0, on_b ? 1 : 0, kc);
  hipLaunchKernelGGL(qr_wy_update_kernel, dim3(nt, ceil_div(maxk, 64), nm), dim3(256), 0, s, d, k0, on_b ? 1 : 0);
  TNA_LAUNCHED("svd.qr_apply");
  return TNA_OK;
}

tna_status svd_group_run(std::vector<SvdMat> &mats, SvdGroup &g, int max_sweeps, std::vector<int> &sweeps,
                         hipStream_t s, bool defer_fused) {
  const int nm = (int)mats.size();
  if (nm == 0) return TNA_OK;
  sweeps.assign(nm, 0);
  int max_tiles_load = 0, max_pairs = 0, max_ks = 0, max_tiles = 0, max_steps = 0, max_r4 = 0;
  for (auto &a : mats) {
    a.active = 1;
    max_tiles_load = std::max(max_tiles_load, ceil_div(a.m, 32) * ceil_div(a.n, 32) + ceil_div((int64_t)a.R * a.R, 1024));
    max_pairs = std::max(max_pairs, a.nb / 2);
    max_ks = std::max(max_ks, a.ksplit);
    max_tiles = std::max(max_tiles, ceil_div(a.C, 64) + ceil_div(a.R, 64));
    max_steps = std::max(max_steps, a.nb - 1);
    max_r4 = std::max(max_r4, ceil_div(a.R, 4));
  }
  if (nm > 4096) {
    set_error("svd: at most 4096 matrices per group");
    return TNA_ERR_ARG;
  }
  if (!g.host_ctr) TNA_HIP(hipHostMalloc((void **)&g.host_ctr, sizeof(int) * 2 * 4096, hipHostMallocDefault));
  if (!g.host_fro) TNA_HIP(hipHostMalloc((void **)&g.host_fro, sizeof(double) * 2 * 4096, hipHostMallocDefault));
  TNA_TRY(upload(mats, g, s));
  const SvdMat *d = g.desc.as<SvdMat>();
  int n_two = 0, n_tiny = 0;
  for (auto &a : mats) {
    n_two += a.fused == 1;
    n_tiny += a.fused == 2;
  }
  const int nfused = n_two + n_tiny;
  auto read_status = [&](bool ctr, bool fro, int reset) -> tna_status {
    hipLaunchKernelGGL(status_kernel, dim3(ceil_div(nm, 64)), dim3(64), 0, s, d, nm, ctr ? g.host_ctr : nullptr,
                       fro ? g.host_fro : nullptr, reset);
    TNA_LAUNCHED("svd.status");
    TNA_HIP(hipStreamSynchronize(s));
    return TNA_OK;
  };
  // a NaN or Inf anywhere in an input shows in its squared Frobenius norm; the callers that defer
  // their reads (the sweep engine) check the spectrum sums they read anyway
  auto check_finite_norms = [&]() -> tna_status {
    for (int z = 0; z < nm; ++z)
      if (!std::isfinite(g.host_fro[2 * z])) {
        set_error("svd: non-finite entry in input matrix " + std::to_string(z));
        return TNA_ERR_NONFINITE;
      }
    return TNA_OK;
  };
  if (n_tiny < nm) {
    int fro_b = 1;
    for (auto &a : mats) fro_b = std::max(fro_b, fro_blocks(a.R, a.C));
    hipLaunchKernelGGL(load_kernel, dim3(max_tiles_load, 1, nm), dim3(256), 0, s, d);
    hipLaunchKernelGGL(fro_partial_kernel, dim3(fro_b, 1, nm), dim3(256), 0, s, d);
    hipLaunchKernelGGL(fro_kernel, dim3(nm), dim3(256), 0, s, d);
    TNA_LAUNCHED("svd.load");
  }
  // with every matrix on a single-workgroup path the norms are read with the sweep counts below
  if (!defer_fused && nfused < nm) {
    if (n_tiny > 0) {  // these form their norms in their only launch
      timer_begin("svd.fused", s);
      hipLaunchKernelGGL(jacobi_tiny_kernel, dim3(nm), dim3(256), 0, s, d, max_sweeps);
      timer_end("svd.fused", 0.0, 0.0, s);
      TNA_LAUNCHED("svd.fused");
    }
    TNA_TRY(read_status(false, true, 0));
    TNA_TRY(check_finite_norms());
  }
  // QR start for the larger matrices
  int qr_rows = 0, qr_cblk = 0;
  for (auto &a : mats)
    if (a.precond) {
      qr_rows = std::max(qr_rows, a.R);
      qr_cblk = std::max(qr_cblk, ceil_div(a.C, 256));
    }
  if (qr_rows > 0) {
    hipLaunchKernelGGL(qr_init_kernel, dim3(qr_cblk, 1, nm), dim3(256), 0, s, d);
    int sorted = 0, ptiles = 0;
    for (auto &a : mats)
      if (a.precond && a.rows_scaled) {
        ++sorted;
        ptiles = std::max(ptiles, ceil_div(a.R, 32) * ceil_div(a.C, 32));
      }
    if (sorted > 0) {
      hipLaunchKernelGGL(colnorm_kernel, dim3(8 * qr_cblk, 1, nm), dim3(256), 0, s, d);
      hipLaunchKernelGGL(colsort_kernel, dim3(nm), dim3(1024), 0, s, d);
      hipLaunchKernelGGL(permute_load_kernel, dim3(ptiles, 1, nm), dim3(256), 0, s, d);
      TNA_LAUNCHED("svd.qr_order");
    }
    double qr_bytes = 0.0;
    for (auto &a : mats)
      if (a.precond) qr_bytes += 16.0 * ((double)a.R * a.C / 3.0 + (double)a.R * a.R / 2.0);
    // Blocked Householder QR (no column pivoting: the start it gives converges as fast on
    // these matrices, and the trailing update becomes matrix products): each 32-column panel is
    // factored, then B[k0:, k0+32:] <- (I - V T^T V^T) B[k0:, k0+32:].
    // A rows_scaled matrix stops its QR start once every row below the factored panels is at the
    // rounding level (row_floor2): such rows are never rotated, so the sweeps run on the rows
    // above (Ra), and a numerically low-rank matrix pays for the panels of its rank only.
    std::vector<int> watch(nm, 0);
    int nwatch = 0;
    for (int z = 0; z < nm; ++z)
      if (mats[z].precond && mats[z].rows_scaled) {
        watch[z] = 1;
        ++nwatch;
      }
    // the panel factorisation: one workgroup per matrix for at most 1024 rows; above, one cooperative
    // launch per panel where the runtime admits the grid (all workgroups resident), else one launch
    // per column.  TNA_QR_PANEL=col forces the per-column launches and TNA_QR_PANEL=coop the cooperative
    // ones, whose refusal is then an error.
    const char *qp = std::getenv("TNA_QR_PANEL");
    const bool force_coop = qp && std::strcmp(qp, "coop") == 0;
    bool coop = !(qp && std::strcmp(qp, "col") == 0);
    timer_begin("svd.qr", s);
    for (int k0 = 0; k0 < qr_rows; k0 += 32) {
      const int chunks = ceil_div(qr_rows - k0, QC_ROWS);
      bool panel_done = false;
      if (!qp && qr_rows - k0 <= QP_ROWS) {
        const int nw = ceil_div(qr_rows - k0, 64);
        if (nw <= 8) hipLaunchKernelGGL(qr_panel_wg_kernel<512>, dim3(1, 1, nm), dim3(64 * nw), 0, s, d, k0);
        else hipLaunchKernelGGL(qr_panel_wg_kernel<1024>, dim3(1, 1, nm), dim3(64 * nw), 0, s, d, k0);
        panel_done = true;
      } else if (coop) {
        int kk0 = k0;
        void *args[] = {(void *)&d, (void *)&kk0};
        const hipError_t e = hipLaunchCooperativeKernel(reinterpret_cast<const void *>(qr_panel_coop_kernel),
                                                        dim3(chunks, 1, nm), dim3(256), args, 0, s);
        if (e == hipSuccess) {
          panel_done = true;
        } else {
          (void)hipGetLastError();  // not admitted: the per-column launches from here on
          if (force_coop) {
            set_error("svd: cooperative QR panel launch not admitted");
            return TNA_ERR_UNSUPPORTED;
          }
          coop = false;
        }
      }
      if (!panel_done)
        for (int k = k0 - 1; k < k0 + 32 && k < qr_rows; ++k)
          hipLaunchKernelGGL(qr_col_kernel, dim3(chunks, 1, nm), dim3(256), 0, s, d, k0, k);
      TNA_TRY(qr_block_apply(mats, d, nm, k0, true, s));
      const int k1 = k0 + 32;
      int tail = 0;
      for (int z = 0; z < nm; ++z)
        if (watch[z] && k1 < mats[z].R) tail = std::max(tail, mats[z].R - k1);
      if (tail == 0) continue;
      hipLaunchKernelGGL(qr_tail_kernel, dim3(ceil_div(tail, 4), 1, nm), dim3(256), 0, s, d, k1);
      TNA_TRY(read_status(false, true, 0));
      bool stopped = false;
      for (int z = 0; z < nm; ++z) {
        if (!watch[z]) continue;
        SvdMat &a = mats[z];
        const double f = std::fmax(0.1 * EPS53 * (double)a.C, a.noise_rel);
        const double floor2 = f * f * g.host_fro[2 * z];
        if (g.host_fro[2 * z + 1] <= floor2) {
          a.Ra = k1;
          stopped = true;
        }
        if (a.Ra < a.R || k1 + 32 >= a.R) {
          watch[z] = 0;
          --nwatch;
        }
      }
      if (stopped) TNA_TRY(upload(mats, g, s));
      if (nwatch == 0 && std::all_of(mats.begin(), mats.end(), [&](const SvdMat &a) {
            return !a.precond || a.Ra < a.R || k1 >= a.R;
          }))
        break;
    }
    timer_end("svd.qr", 0.0, qr_bytes, s);
    hipLaunchKernelGGL(qr_pinv_kernel, dim3(qr_cblk, 1, nm), dim3(256), 0, s, d);
    // Jt = Q^T = H_{R-1} ... H_0: 32 reflectors at a time, Jt <- (I - V T^T V^T) Jt
    timer_begin("svd.qr_form", s);
    for (int k0 = 0; k0 < qr_rows; k0 += 32) TNA_TRY(qr_block_apply(mats, d, nm, k0, false, s));
    timer_end("svd.qr_form", 0.0, 0.0, s);
    TNA_LAUNCHED("svd.qr");
    // The sweeps of a stopped matrix pair blocks of its Ra rows.  A group too small for the chip (under one
    // Gram workgroup per compute unit with 256 columns each) cuts its Grams finer, down to 64 columns
    // (six pairs of 331 x 517: 10.8 us a launch in three pieces, 6.3 in six); the pieces then go where
    // the QR start's blocked products were, if that holds more of them than the area planned for them.
    bool replan = false;
    for (auto &a : mats) {
      if (!a.precond) continue;
      const int nb0 = a.nb, ks0 = a.ksplit;
      int slots = (a.nb / 2) * a.ksplit;
      if (a.Ra < a.R) {
        a.nb = std::max(2, ceil_div(a.Ra, BS));
        a.nb += a.nb & 1;
      }
      const int pairs = a.nb / 2;
      const size_t wy = qws_doubles(a);
      int ks = std::min(ceil_div(1024, (int64_t)pairs * nm), ceil_div(a.C, 256));
      if ((int64_t)pairs * nm * ks < 256) {
        ks = std::min(ceil_div(256, (int64_t)pairs * nm), ceil_div(a.C, 64));
        if (ks * pairs > slots && (int)(wy / 4096) > slots) {
          slots = (int)(wy / 4096);
          a.gram = a.qws;
        }
      }
      ks = std::max(std::min(ks, slots / pairs), 1);
      const int chunk = ceil_div(ceil_div(a.C, ks), GBK) * GBK;  // as the kernel cuts it
      a.ksplit = ceil_div(a.C, chunk);
      replan = replan || a.nb != nb0 || a.ksplit != ks0;
    }
    if (replan) TNA_TRY(upload(mats, g, s));
  }
  max_pairs = max_ks = 0;
  double gram_flops = 0, gram_bytes = 0, apply_flops = 0, apply_bytes = 0;
  for (auto &a : mats) {
    max_pairs = std::max(max_pairs, a.nb / 2);
    max_ks = std::max(max_ks, a.ksplit);
    const double pairs = a.nb / 2, b2 = 4096.0;
    gram_flops += 2.0 * b2 * a.C * pairs;
    gram_bytes += 8.0 * (double)a.Ra * a.C;
    apply_flops += 2.0 * b2 * (double)(a.C + a.R) * pairs;
    apply_bytes += 16.0 * ((double)a.Ra * a.C + (double)a.Ra * a.R);
  }
  // one block pair: every sweep inside one workgroup, no host round trip per sweep
  const bool tiny_done = !defer_fused && nfused < nm;
  if (n_two > 0 || (n_tiny > 0 && !tiny_done)) {
    timer_begin("svd.fused", s);
    if (n_two) hipLaunchKernelGGL(jacobi_fused_kernel, dim3(nm), dim3(EIG_NT), 0, s, d, max_sweeps);
    if (n_tiny && !tiny_done) hipLaunchKernelGGL(jacobi_tiny_kernel, dim3(nm), dim3(256), 0, s, d, max_sweeps);
    timer_end("svd.fused", 0.0, 0.0, s);
    TNA_LAUNCHED("svd.fused");
  }
  // column tiles per workgroup of the apply: four keep a tile's loads in flight behind another's products,
  // where that still leaves two workgroups per compute unit; one spreads a small group (331 x 517, six
  // pairs: 17.5 us a launch with four, 8.2 with one; 16 x 512 x 512: 33 against 39)
  int tpw = 4;
  while (tpw > 1 && (int64_t)max_pairs * nm * ceil_div(max_tiles, tpw) < 512) tpw /= 2;
  std::vector<int> live(nm);
  int active = 0;
  max_steps = 0;
  for (int z = 0; z < nm; ++z) {
    live[z] = !mats[z].fused;
    active += live[z];
    if (live[z]) max_steps = std::max(max_steps, mats[z].nb - 1);
  }
  if (active > 0)
    hipLaunchKernelGGL(status_kernel, dim3(ceil_div(nm, 64)), dim3(64), 0, s, d, nm, (int *)nullptr,
                       (double *)nullptr, 1);
  for (int sw = 1; sw <= max_sweeps && active > 0; ++sw) {
    for (int step = 0; step < max_steps; ++step) {
      timer_begin("svd.gram", s);
      hipLaunchKernelGGL(gram_kernel, dim3(max_pairs, max_ks, nm), dim3(256), 0, s, d, step);
      timer_end("svd.gram", gram_flops, gram_bytes, s);
      timer_begin("svd.eigen", s);
      hipLaunchKernelGGL(eigen_kernel, dim3(max_pairs, nm), dim3(EIG_NT), 0, s, d, step);
      timer_end("svd.eigen", 0.0, 0.0, s);
      timer_begin("svd.apply", s);
      hipLaunchKernelGGL(apply_kernel, dim3(max_pairs, ceil_div(max_tiles, tpw), nm), dim3(256), 0, s, d, step, tpw);
      timer_end("svd.apply", apply_flops, apply_bytes, s);
    }
    TNA_LAUNCHED("svd.sweep");
    TNA_TRY(read_status(true, false, 1));
    static const int dbg = [] {
      const char *e = std::getenv("TNA_DEBUG_SVD");
      return e && e[0] == '1';
    }();
    if (dbg) std::fprintf(stderr, "svd sweep %d: rotating pairs of matrix 0 = %d\n", sw, g.host_ctr[0]);
    bool changed = false;
    for (int z = 0; z < nm; ++z) {
      if (!live[z]) continue;
      sweeps[z] = sw;
      if (g.host_ctr[2 * z] == 0) {
        mats[z].active = 0;
        live[z] = 0;
        --active;
        changed = true;
      }
    }
    if (changed && active > 0) {
      TNA_TRY(upload(mats, g, s));
      max_steps = 0;
      for (int z = 0; z < nm; ++z)
        if (live[z]) max_steps = std::max(max_steps, mats[z].nb - 1);
    }
  }
  // with defer_fused the caller takes the sweep counts and convergence of the single-workgroup
  // paths from spec[7] after its own read of the spectra (no synchronisation here)
  if (nfused > 0 && !defer_fused) {
    TNA_TRY(read_status(true, nfused == nm, 0));
    if (nfused == nm) TNA_TRY(check_finite_norms());
    double fl = 0.0, by = 0.0;
    for (int z = 0; z < nm; ++z)
      if (mats[z].fused) {
        sweeps[z] = g.host_ctr[2 * z + 1];
        if (g.host_ctr[2 * z] != 0) ++active;  // not converged within max_sweeps
        // per sweep: Gram 2 R^2 C, rotation of B and Jt 2 R^2 (C + R); B read for the Gram,
        // B and Jt read and written by the rotation
        const double R = mats[z].R, C = mats[z].C, sw = sweeps[z];
        fl += sw * (2.0 * R * R * C + 2.0 * R * R * (C + R));
        by += sw * 8.0 * (R * C + 2.0 * (R * C + R * R));
      }
    timer_add_work("svd.fused", fl, by);
  }
  bool reup = false;  // finishing kernels run on every matrix
  for (auto &a : mats) {
    reup = reup || !a.active;
    a.active = 1;
  }
  if (reup) TNA_TRY(upload(mats, g, s));
  if (n_tiny < nm) {
    hipLaunchKernelGGL(norms_kernel, dim3(max_r4, 1, nm), dim3(256), 0, s, d);
    hipLaunchKernelGGL(sort_kernel, dim3(nm), dim3(1024), 0, s, d);
    TNA_LAUNCHED("svd.finish");
  }
  return active > 0 ? TNA_ERR_NOCONV : TNA_OK;
}

tna_status svd_group_outputs(std::vector<SvdMat> &mats, SvdGroup &g, hipStream_t s) {
  const int nm = (int)mats.size();
  if (nm == 0) return TNA_OK;
  int max_k = 1, n_tiny = 0;
  int64_t max_el = 1;
  for (auto &a : mats) {
    n_tiny += a.fused == 2;
    max_k = std::max(max_k, a.k);
    max_el = std::max<int64_t>(max_el, std::max<int64_t>((int64_t)a.m * a.k, (int64_t)a.k * a.n));
  }
  TNA_TRY(upload(mats, g, s));
  const SvdMat *d = g.desc.as<SvdMat>();
  if (n_tiny > 0) hipLaunchKernelGGL(finish_small_kernel, dim3(nm), dim3(256), 0, s, d);
  if (n_tiny < nm) {
    hipLaunchKernelGGL(trunc_kernel, dim3(nm), dim3(256), 0, s, d);
    hipLaunchKernelGGL(write_kernel, dim3((unsigned)std::min<int64_t>(ceil_div(max_el, 256), 2048), 2, nm),
                       dim3(256), 0, s, d);
    hipLaunchKernelGGL(complete_kernel, dim3(nm), dim3(256), 0, s, d);
    hipLaunchKernelGGL(gauge_kernel, dim3(max_k, 1, nm), dim3(256), 0, s, d);
  }
  TNA_LAUNCHED("svd.outputs");
  return TNA_OK;
}

void SvdGroup::release() {
  desc.release();
  work_d.release();
  work_i.release();
  for (Stage &st : stage) {
    if (st.host) (void)hipHostFree(st.host);
    if (st.done) (void)hipEventDestroy(st.done);
    st = Stage{};
  }
  if (host_ctr) (void)hipHostFree(host_ctr);
  if (host_fro) (void)hipHostFree(host_fro);
  host_ctr = nullptr;
  host_fro = nullptr;
}

}  // namespace tna
