// Multipole-to-local translation (M->L over V lists) by rotation: every
// V-list source multipole is rotated so that the translation vector lies on
// the z axis, translated along z (an O(p^3) operator that keeps the order m),
// and rotated back.  The paper's FMM diagonalises this step with exponential
// expansions (arXiv:1711.02976, Sec. 1 and 3.2); this kernel computes the
// same truncated operator as the dense M->L instead.
//
// Coefficients are handled in the paper's normalisation (Sec. 2: Y_n^m =
// sqrt((n-|m|)!/(n+|m|)!) P_n^|m| e^{i m phi}), where a rotation is a real
// orthogonal matrix per degree.  For the offset t = (rho, theta, phi) the
// whole M->L is
//   Phi(phi - pi/2) R^-1 Phi(theta) R Z(rho) R^-1 Phi(-theta) R Phi(pi/2 - phi)
// with Phi(a) = diag(e^{-i m a}), R the fixed rotation by +90 degrees about y
// (inverse S R S, S = diag((-1)^m)) and Z(rho) the translation along +z,
//   L'_k^l = rho^-(k+1) sum_n H_l[k][n] rho^-n M'_n^l,
//   H_l[k][n] = (-1)^{n+l} (n+k)! / (s_k^l s_n^l),  s_n^m = sqrt((n-m)!(n+m)!).
//
// GPU organisation (k_m2l_rot).  One block of RW waves per target box and
// right-hand side (the block-to-box map balances the V-list work over the
// XCDs, see make_m2l_map); its V-list (source, density) pairs are the columns,
// taken 64 at a time into an LDS array X[coefficient][column].  Each batch
// runs four phases separated by barriers:
//   0. all threads gather the columns' multipoles into X;
//   1. per degree n: Phi(pi/2-phi), R, Phi(-theta), S R S;
//   2. per order l: the z translation;
//   3. per degree n: R, Phi(theta), S R S, Phi(phi - pi/2);
// then every thread sums the columns of the outputs it owns into FP64
// accumulators kept in registers across batches.  A wave processes whole
// degrees (or orders), one column per lane, so the rotation and translation
// matrices are the same for every lane: they are read as scalar operands,
// and each lane's coefficients of one degree stay in registers.  Degrees and
// orders are assigned to waves by a host-side longest-first schedule.  Orders
// whose 64 columns do not fit the LDS run in k_m2l_rows below.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <vector>

#include "fmm.h"

namespace rpy {

namespace {

constexpr int MAXW = 16;       // most waves per block
constexpr int ROT_NC = 64;     // columns per batch of k_m2l_rot, one per lane
constexpr int MAXK = MAX_ORDER + 1;

template <class R> struct Cx;
template <> struct Cx<double> { using T = double2; };
template <> struct Cx<float> { using T = float2; };

// Degrees (phases 1 and 3) and orders (phase 2) handled by each wave.
struct RotSched {
  unsigned char deg[MAXW][MAXK];
  unsigned char ord[MAXW][MAXK];
  unsigned char ndeg[MAXW];
  unsigned char nord[MAXW];
};

// Per-column data of a batch, in LDS (structure of arrays, one slot per lane),
// in the kernel's precision.
template <class R>
struct ColData {
  int* src;  // source box, -1 for an empty column
  R* e1x;    // e^{-i(pi/2 - phi)}
  R* e1y;
  R* e2x;    // e^{i theta}
  R* e2y;
  R* rinv;   // 1/rho (box units)
  R* wx;     // source centre - target centre (re-centres the fourth density)
  R* wy;
  R* wz;
};

__host__ __device__ constexpr int rot_block(int n) { return n * (n + 1) * (2 * n + 1) / 6; }  // sum_{j<n} (j+1)^2

// One row of the real-split rotation of degree N whose A+ part uses the
// inputs of parity Q: yr = sum A+ Re x, yi = sum A- Im x over the nonzero
// entries, stored in that order in the row a.
template <int N, int Q, class R>
__device__ inline void rot_row(const R* __restrict__ a, const R* xr, const R* xi, R& yr, R& yi) {
  constexpr int NP = N >= Q ? (N - Q) / 2 + 1 : 0;
  constexpr int MS = Q == 1 ? 2 : 1;
  constexpr int NM = N >= MS ? (N - MS) / 2 + 1 : 0;
  R r = 0, i = 0;
#pragma unroll
  for (int j = 0; j < NP; ++j) r = fma(a[j], xr[Q + 2 * j], r);
#pragma unroll
  for (int j = 0; j < NM; ++j) i = fma(a[NP + j], xi[MS + 2 * j], i);
  yr = r;
  yi = i;
}

// Stores (SR yr + i SI yi) times e (if PH) to col[mp] and advances e by (bx, by).
// The phase e^{i m a} is advanced by recurrence in the kernel's precision: in
// FP32 its error grows like m ulp, and it multiplies coefficients of degree
// n >= m, which the V-list separation makes smaller by a factor of at least
// 0.43^n than the degree-0 term.
template <bool PH, int SR, int SI, class R>
__device__ inline void put_row(typename Cx<R>::T* col, int mp, int ld, R yr, R yi, R& fr, R& fi, R bx, R by) {
  typename Cx<R>::T o;
  if (SR < 0) yr = -yr;
  if (SI < 0) yi = -yi;
  if (PH) {
    o.x = yr * fr - yi * fi;
    o.y = yr * fi + yi * fr;
    const R tr = fr * bx - fi * by;
    fi = fr * by + fi * bx;
    fr = tr;
  } else {
    o.x = yr;
    o.y = yi;
  }
  col[mp * ld] = o;
}

// A row of K table entries by scalar loads, issued before the previous row's
// multiply-adds: in the FP64 form, whose tables (28 KB at p = 16) outgrow the
// scalar cache, one load wait per two rows is covered that way (p = 16,
// 778k beads, 20 right-hand sides: 59.9 ms with a row pair loaded and then used,
// 57.9 now; 100k beads: 389 and 373 us).  A wait before each issue, which leaves
// none open, costs more in scalar instructions than it gains.
template <int K, class R>
__device__ inline void load_row(const R* __restrict__ a, R* r) {
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int j = 0; j < K; ++j) r[j] = a[j];
  __builtin_amdgcn_sched_barrier(0);
}

// col[mp] = e^{mp} (SR Re(R x)_mp + i SI Im(R x)_mp) for mp = 0..N, with
// e = (bx, by) when PH (else 1); SR = SI = 1 gives R, SR = (-1)^N and
// SI = -(-1)^N give the inverse rotation S R S on the same table.
template <int N, bool PH, int SR, int SI, class R>
__device__ inline void rot_apply(const R* __restrict__ A, const R* xr, const R* xi, R bx, R by,
                                 typename Cx<R>::T* col, int ld) {
  constexpr int K = N + 1;
  R fr = 1, fi = 0;
  if constexpr (sizeof(R) == 8) {
    R ra[K], rb[K], yr, yi;
    load_row<K, R>(A, ra);
#pragma unroll 1
    for (int mp = 0; mp < K - 1; mp += 2) {
      load_row<K, R>(A + (mp + 1) * K, rb);
      rot_row<N, (N & 1), R>(ra, xr, xi, yr, yi);
      put_row<PH, SR, SI, R>(col, mp, ld, yr, yi, fr, fi, bx, by);
      load_row<K, R>(A + min(mp + 2, K - 1) * K, ra);
      rot_row<N, ((N + 1) & 1), R>(rb, xr, xi, yr, yi);
      put_row<PH, SR, SI, R>(col, mp + 1, ld, yr, yi, fr, fi, bx, by);
    }
    if (K & 1) {
      rot_row<N, (N & 1), R>(ra, xr, xi, yr, yi);
      put_row<PH, SR, SI, R>(col, N, ld, yr, yi, fr, fi, bx, by);
    }
    return;
  }
#pragma unroll 1
  for (int mp = 0; mp < K - 1; mp += 2) {
    R yr, yi;
    rot_row<N, (N & 1), R>(A + mp * K, xr, xi, yr, yi);
    put_row<PH, SR, SI, R>(col, mp, ld, yr, yi, fr, fi, bx, by);
    rot_row<N, ((N + 1) & 1), R>(A + (mp + 1) * K, xr, xi, yr, yi);
    put_row<PH, SR, SI, R>(col, mp + 1, ld, yr, yi, fr, fi, bx, by);
  }
  if (K & 1) {
    R yr, yi;
    rot_row<N, (N & 1), R>(A + N * K, xr, xi, yr, yi);
    put_row<PH, SR, SI, R>(col, N, ld, yr, yi, fr, fi, bx, by);
  }
}

template <int N, class R>
__device__ inline void load_col(const typename Cx<R>::T* col, int ld, R* xr, R* xi) {
#pragma unroll
  for (int m = 0; m <= N; ++m) {
    const auto v = col[m * ld];
    xr[m] = v.x;
    xi[m] = v.y;
  }
}

// Phase 1 for degree N of column c (the column's coefficients are already in
// X, scaled to the paper's normalisation): Phi(pi/2 - phi), R, Phi(-theta),
// S R S.
template <int N, class R>
__device__ void first_half(int c, int ld, const ColData<R>& cd, const R* __restrict__ A, typename Cx<R>::T* X) {
  using C = typename Cx<R>::T;
  constexpr int K = N + 1, t0 = N * (N + 1) / 2;
  constexpr int SG = (N & 1) ? -1 : 1;
  C* col = X + t0 * ld + c;
  R xr[K], xi[K];
  {
    const R ax = (R)cd.e1x[c], ay = (R)cd.e1y[c];
    R er = 1, ei = 0;
#pragma unroll
    for (int m = 0; m < K; ++m) {
      const C v = col[m * ld];
      xr[m] = v.x * er - v.y * ei;
      xi[m] = v.x * ei + v.y * er;
      const R tr = er * ax - ei * ay;
      ei = er * ay + ei * ax;
      er = tr;
    }
  }
  rot_apply<N, true, 1, 1, R>(A, xr, xi, (R)cd.e2x[c], (R)cd.e2y[c], col, ld);
  load_col<N, R>(col, ld, xr, xi);
  rot_apply<N, false, SG, -SG, R>(A, xr, xi, 0.0, 0.0, col, ld);
}

// Phase 2: z translation of order l (KK = p - l + 1 degrees) of column c.
template <int KK, class R>
__device__ void ztrans(int l, int c, int ld, const ColData<R>& cd, const R* __restrict__ H, typename Cx<R>::T* X) {
  using C = typename Cx<R>::T;
  const R ri = (R)cd.rinv[c];
  R s = 1;
  for (int j = 0; j < l; ++j) s *= ri;
  R vr[KK], vi[KK];
#pragma unroll
  for (int j = 0; j < KK; ++j) {
    const int n = l + j;
    C v = X[(n * (n + 1) / 2 + l) * ld + c];
    vr[j] = v.x * s;
    vi[j] = v.y * s;
    s *= ri;
  }
  R so = 1;
  for (int j = 0; j <= l; ++j) so *= ri;
  const auto row = [&](int kk, const R* h) {
    R ar = 0, ai = 0;
#pragma unroll
    for (int j = 0; j < KK; ++j) {
      ar = fma(h[j], vr[j], ar);
      ai = fma(h[j], vi[j], ai);
    }
    const int k = l + kk;
    C o;
    o.x = ar * so;
    o.y = ai * so;
    X[(k * (k + 1) / 2 + l) * ld + c] = o;
    so *= ri;
  };
  if constexpr (sizeof(R) == 8) {
    R ha[KK], hb[KK];
    load_row<KK, R>(H, ha);
#pragma unroll 1
    for (int kk = 0; kk < KK - 1; kk += 2) {
      load_row<KK, R>(H + (kk + 1) * KK, hb);
      row(kk, ha);
      load_row<KK, R>(H + min(kk + 2, KK - 1) * KK, ha);
      row(kk + 1, hb);
    }
    if (KK & 1) row(KK - 1, ha);
    return;
  }
#pragma unroll 2
  for (int kk = 0; kk < KK; ++kk) row(kk, H + kk * KK);
}

// Phase 3 for degree N of column c: R, Phi(theta), S R S, Phi(phi - pi/2).
template <int N, class R>
__device__ void second_half(int c, int ld, const ColData<R>& cd, const R* __restrict__ A, typename Cx<R>::T* X) {
  using C = typename Cx<R>::T;
  constexpr int K = N + 1, t0 = N * (N + 1) / 2;
  constexpr int SG = (N & 1) ? -1 : 1;
  C* col = X + t0 * ld + c;
  R xr[K], xi[K];
  load_col<N, R>(col, ld, xr, xi);
  rot_apply<N, true, 1, 1, R>(A, xr, xi, (R)cd.e2x[c], -(R)cd.e2y[c], col, ld);
  load_col<N, R>(col, ld, xr, xi);
  rot_apply<N, true, SG, -SG, R>(A, xr, xi, (R)cd.e1x[c], -(R)cd.e1y[c], col, ld);
}

// Degree (order) cases compiled into a kernel: 0..16, 17..21 and 22..27, as
// far as the PM it is built for.
#define RPY_DEG_CASES(X) \
  X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)
#define RPY_DEG_CASES_HI(X) X(17) X(18) X(19) X(20) X(21)
#define RPY_DEG_CASES_HI2(X) X(22) X(23) X(24) X(25) X(26) X(27)

}  // namespace

// PM: highest degree compiled in.  RW: waves per block.  MINW: waves per SIMD
// the register allocation must allow.  A block translates ND of the box's nd_all densities, starting
// at density ND * blockIdx.y.
template <int ND, class R, int PM, int RW, int MINW>
__global__ void __launch_bounds__(64 * RW, MINW) k_m2l_rot(int p, int nd_all, Tree t, List V, RotSched sched,
                                                const R* __restrict__ rot, const R* __restrict__ zt, int rot_len,
                                                const double* __restrict__ geo, const double* __restrict__ sf,
                                                const double2* __restrict__ M, const float2* __restrict__ M32,
                                                double2* __restrict__ L, const int* __restrict__ bmap) {
  using C = typename Cx<R>::T;
  constexpr int RT = 64 * RW;
  constexpr int NACC = (ND * ncoef(PM) + RT - 1) / RT;
  extern __shared__ double2 smem[];
  const int T = ncoef(p);
  constexpr int nc = ROT_NC;
  constexpr int ld = nc + 1;  // padded row: column-wise and row-wise LDS accesses both avoid bank conflicts
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = bmap[blockIdx.x];
  if (b < 0) return;  // whole block, before any barrier
  const int d0 = ND * blockIdx.y;
  C* X = reinterpret_cast<C*>(smem);
  ColData<R> cd;
  {
    R* dq = reinterpret_cast<R*>(X + (size_t)T * ld);
    cd.e1x = dq; dq += nc;
    cd.e1y = dq; dq += nc;
    cd.e2x = dq; dq += nc;
    cd.e2y = dq; dq += nc;
    cd.rinv = dq; dq += nc;
    cd.wx = dq; dq += nc;
    cd.wy = dq; dq += nc;
    cd.wz = dq; dq += nc;
    cd.src = reinterpret_cast<int*>(dq);
  }
  double2 acc[NACC];
#pragma unroll
  for (int r = 0; r < NACC; ++r) acc[r] = make_double2(0.0, 0.0);

  const int e0 = V.off[b], e1 = V.off[b + 1];
  const int ncols = (e1 - e0) * ND;
  const int bx = t.ax[b], by = t.ay[b], bz = t.az[b];
  const double cbx = t.cx[b], cby = t.cy[b], cbz = t.cz[b];

  for (int c0 = 0; c0 < ncols; c0 += nc) {
    if (tid < nc) {
      const int g = c0 + tid;
      int S = -1;
      double q0 = 1.0, q1 = 0.0, q2 = 1.0, q3 = 0.0, q4 = 0.5, w0 = 0.0, w1 = 0.0, w2 = 0.0;
      if (g < ncols) {
        S = V.ent[e0 + g / ND];
        const int o = (t.ax[S] - bx + 3) * 49 + (t.ay[S] - by + 3) * 7 + (t.az[S] - bz + 3);
        const double* gq = geo + (size_t)o * 8;
        q0 = gq[0];
        q1 = gq[1];
        q2 = gq[2];
        q3 = gq[3];
        q4 = gq[4];
        w0 = t.cx[S] - cbx;
        w1 = t.cy[S] - cby;
        w2 = t.cz[S] - cbz;
      }
      cd.src[tid] = S;
      cd.e1x[tid] = q0;
      cd.e1y[tid] = q1;
      cd.e2x[tid] = q2;
      cd.e2y[tid] = q3;
      cd.rinv[tid] = q4;
      cd.wx[tid] = w0;
      cd.wy[tid] = w1;
      cd.wz[tid] = w2;
    }
    __syncthreads();
    // phase 0: gather the batch's multipoles (coefficient-contiguous reads),
    // convert to the paper's normalisation (times s_n^m) and store them
    // column-wise.  A thread takes the four densities of one right-hand side
    // of one source at one coefficient, so the fourth density is re-centred
    // on this machine from registers: M4 + (c_S - c_B) . (M1, M2, M3).
    {
      const int ng = nc / 4;  // (source, rhs) groups in the batch
      for (int it = tid; it < ng * T; it += RT) {
        const int g = it / T, f = it - (it / T) * T;
        const int c = 4 * g, S = cd.src[c];
        C o[4];
        if (S >= 0 && sizeof(R) == 4) {
          // FP32: multipoles already scaled and rounded (k_m2l_prep)
          const float2* src = M32 + ((int64_t)S * nd_all + d0 + (c % ND)) * T + f;
          float2 v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = src[k * T];
          const float w0 = (float)cd.wx[c], w1 = (float)cd.wy[c], w2 = (float)cd.wz[c];
          v[3].x += w0 * v[0].x + w1 * v[1].x + w2 * v[2].x;
          v[3].y += w0 * v[0].y + w1 * v[1].y + w2 * v[2].y;
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            o[k].x = (R)v[k].x;
            o[k].y = (R)v[k].y;
          }
        } else if (S >= 0) {
          const double2* src = M + ((int64_t)S * nd_all + d0 + (c % ND)) * T + f;
          double2 v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = src[k * T];
          const double w0 = cd.wx[c], w1 = cd.wy[c], w2 = cd.wz[c];
          v[3].x += w0 * v[0].x + w1 * v[1].x + w2 * v[2].x;
          v[3].y += w0 * v[0].y + w1 * v[1].y + w2 * v[2].y;
          const double s = sf[f];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            o[k].x = (R)(v[k].x * s);
            o[k].y = (R)(v[k].y * s);
          }
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) o[k].x = o[k].y = 0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) X[f * ld + c + k] = o[k];
      }
    }
    __syncthreads();
    {
      const int nd = sched.ndeg[wv];
      for (int i = 0; i < nd; ++i) {
        const int n = sched.deg[wv][i];
        const R* A = rot + rot_block(n);
        switch (n) {
#define RPY_P1(k) \
  case k: if (k <= PM) first_half<(k <= PM ? k : 0), R>(lane, ld, cd, A, X); break;
          RPY_DEG_CASES(RPY_P1)
          RPY_DEG_CASES_HI(RPY_P1)
#undef RPY_P1
          default: break;
        }
      }
    }
    __syncthreads();
    {
      const int no = sched.nord[wv];
      for (int i = 0; i < no; ++i) {
        const int l = sched.ord[wv][i];
        const int kk = p - l + 1;
        // rows of orders below l: sum_{l' < l} (p - l' + 1)^2
        const int zo = (p + 1) * (p + 2) * (2 * p + 3) / 6 - kk * (kk + 1) * (2 * kk + 1) / 6;
        switch (kk) {
#define RPY_P2(k) \
  case k + 1: if (k <= PM) ztrans<(k <= PM ? k : 0) + 1, R>(l, lane, ld, cd, zt + zo, X); break;
          RPY_DEG_CASES(RPY_P2)
          RPY_DEG_CASES_HI(RPY_P2)
#undef RPY_P2
          default: break;
        }
      }
    }
    __syncthreads();
    {
      const int nd = sched.ndeg[wv];
      for (int i = 0; i < nd; ++i) {
        const int n = sched.deg[wv][i];
        const R* A = rot + rot_block(n);
        switch (n) {
#define RPY_P3(k) \
  case k: if (k <= PM) second_half<(k <= PM ? k : 0), R>(lane, ld, cd, A, X); break;
          RPY_DEG_CASES(RPY_P3)
          RPY_DEG_CASES_HI(RPY_P3)
#undef RPY_P3
          default: break;
        }
      }
    }
    __syncthreads();
    // sum the columns of each (coefficient, density) into the accumulators
#pragma unroll
    for (int r = 0; r < NACC; ++r) {
      const int i = tid + r * RT;
      if (i < ND * T) {
        const int d = i / T, f = i - d * T;  // lanes walk a column: one bank per lane
        const C* row = X + (size_t)f * ld + d;
        double sx = 0.0, sy = 0.0;
        for (int j = 0; j < nc; j += ND) {
          const C v = row[j];
          sx += (double)v.x;
          sy += (double)v.y;
        }
        acc[r].x += sx;
        acc[r].y += sy;
      }
    }
    __syncthreads();
  }
  // paper normalisation -> stored normalisation (times s_k^l)
  double2* Lb = L + ((int64_t)b * nd_all + d0) * T;
#pragma unroll
  for (int r = 0; r < NACC; ++r) {
    const int i = tid + r * RT;
    if (i < ND * T) {
      const int d = i / T, f = i - d * T;
      const double s = sf[f];
      Lb[(size_t)d * T + f] = make_double2(acc[r].x * s, acc[r].y * s);
    }
  }
}


// ------------------------------------------ several rows of a degree per wave --
// k_m2l_rot gives each lane a column, so its batches need 64 columns of LDS.
// Where only 32 or 16 fit the wave's 64 / NC lane groups take different rows of
// the same degree (or order) of NC columns here, so that no lane idles.  The
// matrix entries then differ between the groups; they are read by vector loads,
// 16 entries of a group's row per load into its rows of 16 lanes, and each
// multiply-add broadcasts one of them over the row (DPP row_newbcast).  The
// azimuthal phases depend on the order alone: the first is applied by the
// gather and the last by the column sums, one complex product each from a
// table per V-list offset.  What bounds it is instruction issue: 12 to 16
// instructions per row beside its multiply-adds (phases, the LDS store, loop),
// which is why k_m2l_rot, with two rows per trip and scalar operands, stays
// where its 64 columns fit (order 16, FP64: 61 ms there, 71 with 64 columns
// here).

namespace {

template <int NC>
struct RowTab {
  static constexpr int G = 64 / NC;
  // rotation rows of degree n come by parity s = 0, 1 of m', G at a time
  static constexpr int steps(int n, int s) { return n >= s ? ((n - s) / 2 + G) / G : 0; }
  static constexpr int chunks(int n) { return n < 16 ? 1 : 2; }  // A+ in entries 0.., A- in 8.. or in the second 16
  static constexpr int rot_off(int n, int s) {
    int o = 0;
    for (int k = 0; k < n; ++k) o += (steps(k, 0) + steps(k, 1)) * chunks(k);
    return (o + (s ? steps(n, 0) * chunks(n) : 0)) * 16 * G;
  }
  // z-translation rows of an order with kk degrees, G at a time
  static constexpr int zsteps(int kk) { return (kk + G - 1) / G; }
  static constexpr int zchunks(int kk) { return kk <= 16 ? 1 : 2; }
  static constexpr int z_off(int kk) {
    int o = 0;
    for (int k = 1; k < kk; ++k) o += zsteps(k) * zchunks(k);
    return o * 16 * G;
  }
};

// Multiply-adds y += m[K + i] x[i], i < N + TAIL, and z += w[L + i] v[i],
// i < N, the entries broadcast over each row of 16 lanes, in blocks of up to 8
// pairs.  A block starts with the two wait states a DPP operand needs after a
// vector write.
#define RPY_PAIR(T_, i)                                                                                 \
  "v_fmac_" T_ "_dpp %0, %2, %[x" #i "] row_newbcast:%[k" #i "] row_mask:0xf bank_mask:0xf\n\t"         \
  "v_fmac_" T_ "_dpp %1, %3, %[v" #i "] row_newbcast:%[l" #i "] row_mask:0xf bank_mask:0xf\n\t"
#define RPY_TAIL(T_) "v_fmac_" T_ "_dpp %0, %2, %[t] row_newbcast:%[kt] row_mask:0xf bank_mask:0xf\n\t"
#define RPY_ARG(i) [x##i] "v"(x[i]), [v##i] "v"(v[i]), [k##i] "n"(K + i), [l##i] "n"(L + i)
#define RPY_DOT(N_, PAIRS, ...)                                                                         \
  if constexpr (N == N_) {                                                                              \
    if constexpr (TAIL)                                                                                 \
      asm("s_nop 1\n\t" PAIRS RPY_TAIL(RPY_T)                                                           \
          : "+v"(y), "+v"(z)                                                                            \
          : "v"(m), "v"(w), __VA_ARGS__, [t] "v"(x[N_]), [kt] "n"(K + N_));                             \
    else                                                                                                \
      asm("s_nop 1\n\t" PAIRS : "+v"(y), "+v"(z) : "v"(m), "v"(w), __VA_ARGS__);                        \
  }
#define RPY_DOT_FOR(R_)                                                                                 \
  template <int N, int TAIL, int K, int L>                                                              \
  __device__ inline void dot2(R_ m, R_ w, const R_* x, const R_* v, R_& y, R_& z) {                     \
    if constexpr (N > 8) {                                                                              \
      dot2<8, 0, K, L>(m, w, x, v, y, z);                                                               \
      dot2<N - 8, TAIL, K + 8, L + 8>(m, w, x + 8, v + 8, y, z);                                        \
    }                                                                                                   \
    if constexpr (N == 0 && TAIL)                                                                       \
      asm("s_nop 1\n\t" RPY_TAIL(RPY_T) : "+v"(y), "+v"(z) : "v"(m), "v"(w), [t] "v"(x[0]), [kt] "n"(K)); \
    RPY_DOT(1, RPY_PAIR(RPY_T, 0), RPY_ARG(0))                                                          \
    RPY_DOT(2, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1), RPY_ARG(0), RPY_ARG(1))                           \
    RPY_DOT(3, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1) RPY_PAIR(RPY_T, 2), RPY_ARG(0), RPY_ARG(1), RPY_ARG(2)) \
    RPY_DOT(4, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1) RPY_PAIR(RPY_T, 2) RPY_PAIR(RPY_T, 3), RPY_ARG(0), RPY_ARG(1), \
            RPY_ARG(2), RPY_ARG(3))                                                                     \
    RPY_DOT(5, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1) RPY_PAIR(RPY_T, 2) RPY_PAIR(RPY_T, 3) RPY_PAIR(RPY_T, 4), \
            RPY_ARG(0), RPY_ARG(1), RPY_ARG(2), RPY_ARG(3), RPY_ARG(4))                                 \
    RPY_DOT(6, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1) RPY_PAIR(RPY_T, 2) RPY_PAIR(RPY_T, 3) RPY_PAIR(RPY_T, 4) \
                RPY_PAIR(RPY_T, 5), RPY_ARG(0), RPY_ARG(1), RPY_ARG(2), RPY_ARG(3), RPY_ARG(4), RPY_ARG(5)) \
    RPY_DOT(7, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1) RPY_PAIR(RPY_T, 2) RPY_PAIR(RPY_T, 3) RPY_PAIR(RPY_T, 4) \
                RPY_PAIR(RPY_T, 5) RPY_PAIR(RPY_T, 6), RPY_ARG(0), RPY_ARG(1), RPY_ARG(2), RPY_ARG(3),  \
            RPY_ARG(4), RPY_ARG(5), RPY_ARG(6))                                                         \
    RPY_DOT(8, RPY_PAIR(RPY_T, 0) RPY_PAIR(RPY_T, 1) RPY_PAIR(RPY_T, 2) RPY_PAIR(RPY_T, 3) RPY_PAIR(RPY_T, 4) \
                RPY_PAIR(RPY_T, 5) RPY_PAIR(RPY_T, 6) RPY_PAIR(RPY_T, 7), RPY_ARG(0), RPY_ARG(1), RPY_ARG(2), \
            RPY_ARG(3), RPY_ARG(4), RPY_ARG(5), RPY_ARG(6), RPY_ARG(7))                                 \
  }
#define RPY_T "f64"
RPY_DOT_FOR(double)
#undef RPY_T
#define RPY_T "f32"
RPY_DOT_FOR(float)
#undef RPY_T
#undef RPY_DOT_FOR
#undef RPY_DOT
#undef RPY_ARG
#undef RPY_TAIL
#undef RPY_PAIR

// What a lane keeps of its column's source through a batch: the phases
// e^{i m' theta} of its first row of either parity and of a row step, and
// 1/rho.  FP32 reads the phases and the powers of 1/rho from LDS tables
// instead, made by the recurrences of k_m2l_rot.
template <class R>
struct LaneCol {
  R e0x, e0y, e1x, e1y, sx, sy;  // FP64
  R ri;                          // FP64
  const typename Cx<R>::T* th;   // FP32: e^{i m theta} at m = 2 g
  const R* rp;                   // FP32: (1/rho)^n
};

template <class R>
__device__ inline R ipow(R x, int n) {
  R r = 1;
  for (; n; n >>= 1) {
    if (n & 1) r *= x;
    x *= x;
  }
  return r;
}

// Rows m' = S, S + 2, .. of the rotation of degree N on the lane's column
// (xr + i xi), G at a time: written with the phase e^{+-i m' theta} (ph, cj =
// +-1 on the imaginary part) or, for the inverse rotation S R S, with its signs
// and a factor.  A loop, not unrolled: a wave runs through the code of its
// degrees once per batch, and the code of all degrees has to stay in the
// instruction cache (unrolled, 100 KB in FP64 at p = 16, it took 1.3x as long
// with 20 % fewer instructions).  Row groups past the last row write to `dump`.
template <int N, int S, int NC, class R>
__device__ inline void rows_class(const LaneCol<R>& lc, bool ph, R cj, R fac, const R* __restrict__ tab, unsigned lo,
                                  int g, int ld, const R* xr, const R* xi, typename Cx<R>::T* col,
                                  typename Cx<R>::T* dump) {
  using C = typename Cx<R>::T;
  using RT = RowTab<NC>;
  constexpr int G = RT::G, CH = RT::chunks(N), KB = CH > 1 ? 0 : 8;
  constexpr R SG = (N & 1) ? -1 : 1;
  // A+ acts on the real parts of orders Q, Q + 2, ..; A- on the imaginary
  // parts of the others from 1 on
  constexpr int Q = (N + S) & 1, M0 = Q == 1 ? 2 : 1;
  constexpr int NP = N >= Q ? (N - Q) / 2 + 1 : 0, NM = N >= M0 ? (N - M0) / 2 + 1 : 0;
  constexpr int cnt = N >= S ? (N - S) / 2 + 1 : 0, steps = RT::steps(N, S);
  static_assert(NP == NM || NP == NM + 1, "one more real input at most");
  if constexpr (steps == 0) return;
  R a[NP + 1], b[NM + 1];
#pragma unroll
  for (int j = 0; j < NP; ++j) a[j] = xr[Q + 2 * j];
#pragma unroll
  for (int j = 0; j < NM; ++j) b[j] = xi[M0 + 2 * j];
  R ex = S ? lc.e1x : lc.e0x, ey = (S ? lc.e1y : lc.e0y) * cj;
  const R sy = lc.sy * cj;
  const R* row = tab + RT::rot_off(N, S);
  R mp = row[lo], mm = CH > 1 ? (row + 16 * G)[lo] : mp;  // the next step's entries are loaded ahead
  col += S * ld;
  int left = cnt - g;  // this group's rows are left while positive
#pragma unroll 1
  for (int j = 0; j < steps; ++j) {
    row += CH * 16 * G;
    const R np = row[lo], nm = CH > 1 ? (row + 16 * G)[lo] : np;
    R yr = 0, yi = 0;
    dot2<NM, NP - NM, 0, KB>(mp, mm, a, b, yr, yi);
    mp = np;
    mm = nm;
    C o;
    if (ph) {
      if constexpr (sizeof(R) == 4) {
        const C e = lc.th[S + 2 * j * G];
        ex = e.x;
        ey = e.y * cj;
      }
      o.x = fma(yr, ex, -(yi * ey));
      o.y = fma(yr, ey, yi * ex);
      if constexpr (sizeof(R) == 8) {
        const R tr = ex * lc.sx - ey * sy;
        ey = ex * sy + ey * lc.sx;
        ex = tr;
      }
    } else {
      o.x = SG * yr * fac;
      o.y = -SG * yi * fac;
    }
    *(cnt % G == 0 || left > 0 ? col : dump) = o;
    left -= G;
    col += 2 * G * ld;
  }
}

// Orders a wave's own LDS accesses: its lane groups read rows that others of them
// wrote, and write rows that others have read.  The LDS takes a wave's accesses in
// the order of its instructions, so no wait is needed, but the compiler must keep
// that order, which a lane's own accesses alone would not require of it.
__device__ inline void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); }

// The tables' base as an opaque offset: otherwise the addresses of all
// degrees are kept in registers through the loop over batches.
__device__ inline int opaque_zero() {
  int z = 0;
  asm volatile("" : "+s"(z));
  return z;
}

// R with the phases, then S R S, of degree N in place.
template <int N, int NC, class R>
__device__ inline void rows_degree(const LaneCol<R>& lc, R cj, bool scale, const R* __restrict__ tab, unsigned lo,
                                   int g, int c, int ld, typename Cx<R>::T* X, typename Cx<R>::T* dump) {
  asm volatile("" : "+v"(c), "+v"(lo), "+v"(g));
  tab += opaque_zero();
  typename Cx<R>::T* col = X + N * (N + 1) / 2 * ld + c;
  R fac = 1;
  if constexpr (sizeof(R) == 4) {
    if (scale) fac = lc.rp[N];
  } else {
    R ri = lc.ri;
    asm volatile("" : "+v"(ri));
    if (scale) fac = ipow(ri, N);
  }
#pragma unroll 1
  for (int k = 0; k < 2; ++k) {
    R xr[N + 1], xi[N + 1];
    wave_order();  // the first pass's rows are written
    load_col<N, R>(col, ld, xr, xi);
    wave_order();  // all rows are read before any is written
    rows_class<N, 0, NC, R>(lc, k == 0, cj, fac, tab, lo, g, ld, xr, xi, col + 2 * g * ld, dump);
    rows_class<N, 1, NC, R>(lc, k == 0, cj, fac, tab, lo, g, ld, xr, xi, col + 2 * g * ld, dump);
  }
}

// z translation of order l (KK degrees) on inputs already times rho^-n; rows
// in steps of G.
template <int KK, int NC, class R>
__device__ inline void rows_ztrans(int l, const LaneCol<R>& lc, const R* __restrict__ tab, unsigned lo, int g, int c,
                                   int ld, typename Cx<R>::T* X, typename Cx<R>::T* dump) {
  using C = typename Cx<R>::T;
  using RT = RowTab<NC>;
  constexpr int G = RT::G, CH = RT::zchunks(KK), K0 = KK < 16 ? KK : 16;
  asm volatile("" : "+v"(c), "+v"(lo), "+v"(g));
  tab += opaque_zero();
  X += c;
  R vr[KK], vi[KK];
  C* x = X + (l * (l + 1) / 2 + l) * ld;  // coefficient (l, l); the next degree's is n + 1 further on
#pragma unroll
  for (int j = 0; j < KK; ++j) {
    const C v = x[(j * l + j * (j + 1) / 2) * ld];
    vr[j] = v.x;
    vi[j] = v.y;
  }
  wave_order();  // all degrees are read before any is written
  const R* row = tab + RT::z_off(KK);
  R so = 1, st = 1;
  if constexpr (sizeof(R) == 8) {
    R ri = lc.ri;
    asm volatile("" : "+v"(ri));
    so = ipow(ri, l + 1 + g);
    st = ipow(ri, G);
  }
  R m0 = row[lo], m1 = CH > 1 ? (row + 16 * G)[lo] : m0;
  int kk = g;
  C* y = x + (g * l + g * (g + 1) / 2) * ld;  // coefficient (l + kk, l)
  int dy = (G * l + g * G + G * (G + 1) / 2) * ld;
#pragma unroll 1
  for (int j = 0; j < RT::zsteps(KK); ++j, kk += G) {
    row += CH * 16 * G;
    const R n0 = row[lo], n1 = CH > 1 ? (row + 16 * G)[lo] : n0;
    R ar = 0, ai = 0;
    dot2<K0, 0, 0, 0>(m0, m0, vr, vi, ar, ai);
    if constexpr (KK > 16) dot2<KK - 16, 0, 0, 0>(m1, m1, vr + 16, vi + 16, ar, ai);
    m0 = n0;
    m1 = n1;
    if constexpr (sizeof(R) == 4) so = lc.rp[min(l + kk, l + KK - 1) + 1];
    C o;
    o.x = ar * so;
    o.y = ai * so;
    *(KK % G == 0 || kk < KK ? y : dump) = o;
    y += dy;
    dy += G * G * ld;
    if constexpr (sizeof(R) == 8) so *= st;
  }
}

}  // namespace

// Phases e^{-i m (pi/2 - phi)} (ph1) and e^{i m theta} (ph2), m = 0..p, of
// every V-list offset, by the recurrences of k_m2l_rot in the kernel's
// precision.
template <class R>
__global__ void k_m2l_phases(int p, const double* geo, typename Cx<R>::T* ph) {
  const int o = threadIdx.x + blockIdx.x * blockDim.x, w = blockIdx.y;
  if (o >= 343) return;
  const R ax = (R)geo[8 * o + 2 * w], ay = (R)geo[8 * o + 2 * w + 1];
  R er = 1, ei = 0;
  for (int m = 0; m <= p; ++m) {
    typename Cx<R>::T e;
    e.x = er;
    e.y = ei;
    ph[((int64_t)w * 343 + o) * (p + 1) + m] = e;
    const R tr = fma(er, ax, -(ei * ay));
    ei = fma(er, ay, ei * ax);
    er = tr;
  }
}

// One right-hand side (four densities) of one target box per block: grid
// (boxes, right-hand sides).
template <class R, int PM, int NC, int RW, int MINW>
__global__ void __launch_bounds__(64 * RW, MINW) k_m2l_rows(int p, int nd_all, Tree t, List V, RotSched sched,
                                                 const R* __restrict__ rtab, const R* __restrict__ ztab,
                                                 const double* __restrict__ geo,
                                                 const typename Cx<R>::T* __restrict__ ph,
                                                 const double* __restrict__ sf, const double2* __restrict__ M,
                                                 const float2* __restrict__ M32, double2* __restrict__ L,
                                                 const int* __restrict__ bmap) {
  using C = typename Cx<R>::T;
  constexpr int RT = 64 * RW, NS = NC / 4, ld = NC + 1;
  constexpr int NACC = (4 * ncoef(PM) + RT - 1) / RT;
  constexpr bool F32 = sizeof(R) == 4;
  extern __shared__ double2 smem[];
  const int T = ncoef(p), tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int b = bmap[blockIdx.x];
  if (b < 0) return;  // whole block, before any barrier
  const int d0 = 4 * blockIdx.y;
  C* X = reinterpret_cast<C*>(smem);
  C* dump = X + (size_t)T * ld;
  R* wsh = reinterpret_cast<R*>(dump + 1);            // [2][3][NS] source centre - target centre
  int* src = reinterpret_cast<int*>(wsh + 6 * NS);    // [2][NS] source box, -1 for none
  int* off = src + 2 * NS;                            // [2][NS] its offset's slot
  C* thT = reinterpret_cast<C*>(off + 2 * NS);        // FP32: [NS][p+1] e^{i m theta}
  R* rpT = reinterpret_cast<R*>(thT + NS * (p + 1));  // FP32: [NS][p+2] rho^-n
  double2 acc[NACC];
#pragma unroll
  for (int r = 0; r < NACC; ++r) acc[r] = make_double2(0.0, 0.0);
  const int e0 = V.off[b], e1 = V.off[b + 1];
  const int bx = t.ax[b], by = t.ay[b], bz = t.az[b];
  const double cbx = t.cx[b], cby = t.cy[b], cbz = t.cz[b];
  const int c = lane % NC, g = lane / NC;  // column and row group
  // the gather's sources gj, gj + gn, .. at coefficient gf (order gm); the
  // sums' coefficients' orders
  const auto order_of = [](int f) {
    int n = 0;
    while (tri(n + 1) <= f) ++n;
    return f - tri(n);
  };
  static_assert(RT >= ncoef(PM), "a thread per coefficient");
  const int gn = RT / T, gj = tid / T, gf = tid - gj * T, gm = order_of(gf);
  const double gs = F32 ? 1.0 : sf[gf];
  int om[NACC];
#pragma unroll
  for (int r = 0; r < NACC; ++r) om[r] = order_of((tid + r * RT) % T);
  const unsigned lo = g * 16 + (lane & 15);  // this lane's entry of a group of rows
  int par = 0;
  for (int s0 = e0; s0 < e1; s0 += NS, par ^= NS) {
    if (tid < NS) {
      const bool have = s0 + tid < e1;
      const int S = have ? V.ent[s0 + tid] : -1;
      int o = 0;
      double w0 = 0.0, w1 = 0.0, w2 = 0.0;
      if (have) {
        o = (t.ax[S] - bx + 3) * 49 + (t.ay[S] - by + 3) * 7 + (t.az[S] - bz + 3);
        w0 = t.cx[S] - cbx;
        w1 = t.cy[S] - cby;
        w2 = t.cz[S] - cbz;
      }
      src[par + tid] = S;
      off[par + tid] = o;
      wsh[3 * par + tid] = (R)w0;
      wsh[3 * par + NS + tid] = (R)w1;
      wsh[3 * par + 2 * NS + tid] = (R)w2;
      if (F32) {
        const R ri = have ? (R)geo[8 * o + 4] : (R)0.5;
        R x = 1;
        for (int n = 0; n <= p + 1; ++n) {
          rpT[tid * (p + 2) + n] = x;
          x *= ri;
        }
      }
    }
    __syncthreads();
    if (F32)
      for (int i = tid; i < NS * (p + 1); i += RT) {
        const int j = i / (p + 1);
        thT[i] = ph[(int64_t)(343 + off[par + j]) * (p + 1) + i - j * (p + 1)];
      }
    // gather: the multipoles in the paper's normalisation, the fourth density
    // re-centred on this machine, times the first phase, into their columns; a
    // thread keeps its coefficient
    for (int j = gj; j < NS && gj < gn; j += gn) {
      const int S = src[par + j];
      C o[4];
      if (S >= 0) {
        const C e = ph[(int64_t)off[par + j] * (p + 1) + gm];
        const R w0 = wsh[3 * par + j], w1 = wsh[3 * par + NS + j], w2 = wsh[3 * par + 2 * NS + j];
        C v[4];
        if constexpr (F32) {  // already scaled and rounded (k_m2l_prep)
          const float2* sp = M32 + ((int64_t)S * nd_all + d0) * T + gf;
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = sp[k * T];
          v[3].x += w0 * v[0].x + w1 * v[1].x + w2 * v[2].x;
          v[3].y += w0 * v[0].y + w1 * v[1].y + w2 * v[2].y;
        } else {
          const double2* sp = M + ((int64_t)S * nd_all + d0) * T + gf;
#pragma unroll
          for (int k = 0; k < 4; ++k) v[k] = sp[k * T];
          v[3].x += w0 * v[0].x + w1 * v[1].x + w2 * v[2].x;
          v[3].y += w0 * v[0].y + w1 * v[1].y + w2 * v[2].y;
        }
        const R ex = F32 ? e.x : (R)(e.x * gs), ey = F32 ? e.y : (R)(e.y * gs);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          o[k].x = fma(v[k].x, ex, -(v[k].y * ey));
          o[k].y = fma(v[k].x, ey, v[k].y * ex);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) o[k].x = o[k].y = 0;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) X[gf * ld + 4 * j + k] = o[k];
    }
    LaneCol<R> lc;
    if constexpr (F32) {
      lc.th = thT + (c >> 2) * (p + 1) + 2 * g;
      lc.rp = rpT + (c >> 2) * (p + 2);
    } else {
      const bool have = src[par + (c >> 2)] >= 0;
      const double* gq = geo + 8 * off[par + (c >> 2)];
      const double wx = have ? gq[2] : 1.0, wy = have ? gq[3] : 0.0;
      lc.ri = have ? gq[4] : 0.5;
      double x2 = wx * wx - wy * wy, y2 = 2.0 * wx * wy;  // e^{2 i theta}
      lc.e0x = 1.0;
      lc.e0y = 0.0;
      lc.sx = 1.0;
      lc.sy = 0.0;
      for (int k = 0; k < RowTab<NC>::G; ++k) {
        if (k == g) {
          lc.e0x = lc.sx;
          lc.e0y = lc.sy;
        }
        const double tr = lc.sx * x2 - lc.sy * y2;
        lc.sy = lc.sx * y2 + lc.sy * x2;
        lc.sx = tr;
      }
      lc.e1x = lc.e0x * wx - lc.e0y * wy;
      lc.e1y = lc.e0x * wy + lc.e0y * wx;
    }
    __syncthreads();
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
      // half 0: R, Phi(-theta), S R S, rho^-n; half 1: R, Phi(theta), S R S
      const R cj = half ? (R)-1 : (R)1;
      const int nd = sched.ndeg[wv];
      for (int i = 0; i < nd; ++i) {
        switch (sched.deg[wv][i]) {
#define RPY_P1(k) \
  case k: if (k <= PM) rows_degree<(k <= PM ? k : 0), NC, R>(lc, cj, half == 0, rtab, lo, g, c, ld, X, dump); break;
          RPY_DEG_CASES(RPY_P1)
          RPY_DEG_CASES_HI(RPY_P1)
          RPY_DEG_CASES_HI2(RPY_P1)
#undef RPY_P1
          default: break;
        }
      }
      __syncthreads();
      if (half == 0) {
        const int no = sched.nord[wv];
        for (int i = 0; i < no; ++i) {
          const int l = sched.ord[wv][i];
          switch (p - l + 1) {
#define RPY_P2(k) \
  case k + 1: if (k <= PM) rows_ztrans<(k <= PM ? k : 0) + 1, NC, R>(l, lc, ztab, lo, g, c, ld, X, dump); break;
            RPY_DEG_CASES(RPY_P2)
            RPY_DEG_CASES_HI(RPY_P2)
            RPY_DEG_CASES_HI2(RPY_P2)
#undef RPY_P2
            default: break;
          }
        }
        __syncthreads();
      }
    }
    // sum the columns of each (density, coefficient), times the last phase
#pragma unroll
    for (int r = 0; r < NACC; ++r) {
      const int i = tid + r * RT;
      if (i < 4 * T) {
        const int d = i / T, f = i - d * T;
        double sx = 0.0, sy = 0.0;
        for (int j = 0; j < NS; ++j) {
          if (src[par + j] < 0) break;
          const C v = X[f * ld + 4 * j + d], e = ph[(int64_t)off[par + j] * (p + 1) + om[r]];
          const R fi = -e.y;
          sx += (double)fma(v.x, e.x, -(v.y * fi));
          sy += (double)fma(v.x, fi, v.y * e.x);
        }
        acc[r].x += sx;
        acc[r].y += sy;
      }
    }
  }
  // paper normalisation -> stored normalisation (times s_k^l)
  double2* Lb = L + ((int64_t)b * nd_all + d0) * T;
#pragma unroll
  for (int r = 0; r < NACC; ++r) {
    const int i = tid + r * RT;
    if (i < 4 * T) {
      const double s = sf[i % T];
      Lb[i] = make_double2(acc[r].x * s, acc[r].y * s);
    }
  }
}

// Columns per batch of k_m2l_rows (0: k_m2l_rot is used), which also fix its
// tables.
static int rows_cols(int p, size_t real) {
  if (real == 4) return p <= 21 ? 0 : 32;
  return p <= 16 ? 0 : (p <= 21 ? 32 : 16);
}

template <int NC>
static void rows_tables(int p, const std::vector<double>& rot, const std::vector<double>& zt, std::vector<double>& tr,
                        std::vector<double>& tz) {
  using RT = RowTab<NC>;
  constexpr int G = RT::G;
  // one step of rows past the end is loaded and not used
  tr.assign(RT::rot_off(p + 1, 0) + 32 * G, 0.0);
  for (int n = 0; n <= p; ++n)
    for (int mp = 0; mp <= n; ++mp) {
      const int s = mp & 1, j = (mp / 2) / G, g = (mp / 2) % G, q = (n + mp) & 1;
      const double* row = rot.data() + rot_block(n) + mp * (n + 1);
      const int NP = n >= q ? (n - q) / 2 + 1 : 0, MS = q == 1 ? 2 : 1, NM = n >= MS ? (n - MS) / 2 + 1 : 0;
      double* o = tr.data() + RT::rot_off(n, s) + (j * RT::chunks(n) * G + g) * 16;
      for (int k = 0; k < NP; ++k) o[k] = row[k];
      double* om = RT::chunks(n) > 1 ? o + 16 * G : o + 8;
      for (int k = 0; k < NM; ++k) om[k] = row[NP + k];
    }
  tz.assign(RT::z_off(p + 2) + 32 * G, 0.0);
  for (int l = 0, off = 0; l <= p; off += (p - l + 1) * (p - l + 1), ++l) {
    const int K = p - l + 1;
    for (int kk = 0; kk < K; ++kk)
      for (int j = 0; j < K; ++j)
        tz[RT::z_off(K) + ((kk / G * RT::zchunks(K) + j / 16) * G + kk % G) * 16 + j % 16] = zt[off + kk * K + j];
  }
}

// Longest-first assignment of degrees (cost (n+1)^2) and orders (cost
// (p-l+1)^2) to the block's waves.
static RotSched make_sched(int p, int RW) {
  RotSched s{};
  for (int pass = 0; pass < 2; ++pass) {
    long load[MAXW] = {0};
    for (int j = p; j >= 0; --j) {
      // items in decreasing cost: degree j, or order p - j
      const int item = pass == 0 ? j : p - j;
      int w = 0;
      for (int k = 1; k < RW; ++k)
        if (load[k] < load[w]) w = k;
      load[w] += (long)(j + 1) * (j + 1);
      if (pass == 0) s.deg[w][s.ndeg[w]++] = (unsigned char)item;
      else s.ord[w][s.nord[w]++] = (unsigned char)item;
    }
  }
  return s;
}

static size_t rot_smem_bytes(int p, size_t real) {
  return (size_t)ncoef(p) * (ROT_NC + 1) * 2 * real + (size_t)ROT_NC * (8 * real + sizeof(int));
}

// ND densities per block, nsplit blocks per target box (nsplit ND densities
// per box in M and L).
template <class R, int ND, int PM, int RW, int MINW>
static hipError_t launch_nd(const Launch& l, Exp e, const R* rot, const R* zt, int part, int nsplit) {
  const Built* B = l.B;
  const RotSched sc = make_sched(l.p, RW);
  const size_t shm = rot_smem_bytes(l.p, sizeof(R));
  if (shm > 160 * 1024) return hipErrorInvalidValue;
  auto kern = k_m2l_rot<ND, R, PM, RW, MINW>;
  hipError_t he = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  if (he != hipSuccess) return he;
  if (!B->m2l_map || B->m2l_part[2] < B->tree.nbox) return hipErrorInvalidValue;
  const int b0 = part == 1 ? B->m2l_part[1] : 0, b1 = part == 0 ? B->m2l_part[1] : B->m2l_part[2];
  // the map runs are whole multiples of 8 blocks, so every density group of
  // a box lands on the same XCD
  for (int64_t b = b0; he == hipSuccess && b < b1; b += launch_blocks(64 * RW)) {
    const unsigned nb = (unsigned)std::min<int64_t>(b1 - b, launch_blocks(64 * RW));
    kern<<<dim3(nb, nsplit), 64 * RW, shm, l.s>>>(l.p, ND * nsplit, B->tree, B->lists[LV], sc, rot, zt, l.tb->rot_len,
                                                  l.tb->geo, l.tb->sfac, e.M, e.M32, e.L, B->m2l_map + b);
    he = hipGetLastError();
  }
  return he;
}

// The FP32 M->L reads the multipoles of its source boxes in the paper's
// normalisation, scaled and rounded once per pass here instead of per
// V-list entry: boxes [b0, b1), all nd densities.
__global__ void k_m2l_prep(int T, int nd, int64_t b0, int64_t b1, const double* __restrict__ sf,
                           const double2* __restrict__ M, float2* __restrict__ M32) {
  const int64_t i = b0 * nd * T + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= b1 * nd * T) return;
  const double s = sf[i % T];
  const double2 v = M[i];
  M32[i] = make_float2((float)(v.x * s), (float)(v.y * s));
}

template <class R, int PM, int NC, int RW, int MINW>
static hipError_t launch_rows(const Launch& l, int nrc, Exp e, int part) {
  const Built* B = l.B;
  const int p = l.p;
  const RotSched sc = make_sched(p, RW);
  const size_t cx = 2 * sizeof(R);
  const size_t shm = cx * (ncoef(p) * (NC + 1) + 1) + sizeof(R) * 6 * (NC / 4) + sizeof(int) * 4 * (NC / 4) +
                     (sizeof(R) == 4 ? cx * (NC / 4) * (p + 1) + sizeof(R) * (NC / 4) * (p + 2) : 0);
  auto kern = k_m2l_rows<R, PM, NC, RW, MINW>;
  hipError_t he = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                      hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
  if (he != hipSuccess) return he;
  if (!B->m2l_map || B->m2l_part[2] < B->tree.nbox || !l.tb->rows_rot || l.tb->rows_nc != NC) return hipErrorInvalidValue;
  const int b0 = part == 1 ? B->m2l_part[1] : 0, b1 = part == 0 ? B->m2l_part[1] : B->m2l_part[2];
  for (int64_t b = b0; he == hipSuccess && b < b1; b += launch_blocks(64 * RW)) {
    const unsigned nb = (unsigned)std::min<int64_t>(b1 - b, launch_blocks(64 * RW));
    kern<<<dim3(nb, nrc), 64 * RW, shm, l.s>>>(
        p, 4 * nrc, B->tree, B->lists[LV], sc, static_cast<const R*>(l.tb->rows_rot),
        static_cast<const R*>(l.tb->rows_zt), l.tb->geo, static_cast<const typename Cx<R>::T*>(l.tb->rows_ph),
        l.tb->sfac, e.M, e.M32, e.L, B->m2l_map + b);
    he = hipGetLastError();
  }
  return he;
}

template <class R>
static hipError_t launch_rot(const Launch& l, int nrc, Exp e, const R* rot, const R* zt, int part) {
  const int p = l.p;
  if (p < 0 || p > MAX_ORDER) return hipErrorInvalidValue;
  if (l.B->tree.nbox == 0) return hipSuccess;
  if (sizeof(R) == 4) {
    // sources of the deepest level's targets (part 0) are on that level, those
    // of the other targets (part 1) above it
    if (!e.M32) return hipErrorInvalidValue;
    const Built* B = l.B;
    const int64_t deep = B->level_start.empty() ? 0 : B->level_start[B->depth];
    const int64_t b0 = part == 1 ? 0 : (part == 0 ? deep : 0), b1 = part == 1 ? deep : B->tree.nbox;
    const int T = ncoef(p), nd = 4 * nrc;
    const int64_t cnt = (b1 - b0) * nd * T;
    if (cnt > 0)
      k_m2l_prep<<<(unsigned)((cnt + 255) / 256), 256, 0, l.s>>>(T, nd, b0, b1, l.tb->sfac, e.M, e.M32);
    const hipError_t he = hipGetLastError();
    if (he != hipSuccess) return he;
  }
  if (nrc != 1 && nrc != 2 && nrc != 4) return hipErrorInvalidValue;
  // k_m2l_rot takes 64 columns per batch, one per lane, and the four densities
  // of one right-hand side per block, so that its registers leave room for as
  // many waves as the LDS has columns for (15M beads of 20 right-hand sides or
  // fewer, 0.78M of 20, 1M of 1):
  //   FP32 up to order 16: two blocks of 8 waves per CU, 80 KB each;
  //   FP32 17..21, 131 KB: one block of 16 waves (8 before: 64 systems of 16
  //     right-hand sides 35.6 -> 28.8 ms), all densities in one block where
  //     the V lists are too short to fill the batches of one right-hand side
  //     (16 entries).  The line, 54 entries per box, lies between dense clusters
  //     (43: 27 against 31 ms) and the 64 systems (64: 32 against 29).  It is a
  //     rough one: over fourteen more trees of four right-hand sides one block
  //     for all took 0.79 to 0.90 of the time at 27 to 43 entries, 0.87 at 53, 0.93
  //     and 0.86 at 74 and 77, 0.96 at 115 to 123 and 1.02 at 137, and on trees of
  //     fewer boxes than would fill the chip up to 3.0 (73 boxes, 42 entries: 0.34
  //     against 0.11 ms) and 1.2 (585 boxes, 97);
  //   FP64 up to 10: two blocks of 8 waves (order 7: 1.27 -> 0.74 ms);
  //   FP64 11..16, 160 KB: 12 waves (8 waves with all densities 78 ms, 12 with
  //     one right-hand side's 61, 16 spill and take 69).
  // Above that 64 columns do not fit and k_m2l_rows takes over, with 32
  // columns in FP64 up to 21 (order 21: 83 ms with the lanes half idle, 53
  // now) and in FP32 above, 16 in FP64 above 21 (5.96 -> 2.5 ms).
  if (rows_cols(p, sizeof(R)) > 0) {
    if constexpr (sizeof(R) == 4) return launch_rows<R, 27, 32, 16, 4>(l, nrc, e, part);
    else if (p > 21) return launch_rows<R, 27, 16, 12, 3>(l, nrc, e, part);
    else return launch_rows<R, 21, 32, 12, 3>(l, nrc, e, part);
  }
  if constexpr (sizeof(R) == 4) {
    if (p <= 16) return launch_nd<R, 4, 16, 8, 4>(l, e, rot, zt, part, nrc);
    const List& V = l.B->lists[LV];
    if (nrc > 1 && V.len < 54 * (int64_t)l.B->tree.nbox)
      return nrc == 2 ? launch_nd<R, 8, 21, 16, 4>(l, e, rot, zt, part, 1)
                      : launch_nd<R, 16, 21, 16, 4>(l, e, rot, zt, part, 1);
    return launch_nd<R, 4, 21, 16, 4>(l, e, rot, zt, part, nrc);
  } else {
    if (p <= 10) return launch_nd<R, 4, 10, 8, 4>(l, e, rot, zt, part, nrc);
    return launch_nd<R, 4, 16, 12, 3>(l, e, rot, zt, part, nrc);
  }
}

// Blocks are dealt to the 8 XCDs round-robin (block i to XCD i mod 8), and
// each XCD has its own L2.  Every XCD gets one contiguous run of target
// boxes, so that neighbouring targets share their V-list sources in one L2,
// and the runs are cut where the modelled work (V entries, plus the part
// batch and the store of L per box) splits evenly: with clustered beads the
// V lists are far from uniform along the box order, and equal box counts
// per XCD left some XCDs with twice the mean work.  Block 8k + x takes the
// k-th box of run x; blocks past the end of a shorter run take none.
// Map of the boxes [r0, r1) appended to map (8 K entries).
static void append_map(const std::vector<int>& off, int r0, int r1, std::vector<int>& map) {
  if (r1 <= r0) return;
  const int nb = r1 - r0;
  std::vector<double> pre(nb + 1, 0.0);
  for (int i = 0; i < nb; ++i) {
    const int v = off[r0 + i + 1] - off[r0 + i];
    pre[i + 1] = pre[i] + v + (v > 0 ? 1.0 : 0.0) + 0.25;
  }
  int cut[9];
  cut[0] = 0;
  cut[8] = nb;
  for (int x = 1; x < 8; ++x) {
    const double goal = pre[nb] * x / 8.0;
    cut[x] = (int)(std::lower_bound(pre.begin(), pre.end(), goal) - pre.begin());
    cut[x] = std::min(std::max(cut[x], cut[x - 1]), nb);
  }
  int K = 0;
  for (int x = 0; x < 8; ++x) K = std::max(K, cut[x + 1] - cut[x]);
  const size_t base = map.size();
  map.resize(base + (size_t)8 * K, -1);
  for (int x = 0; x < 8; ++x)
    for (int k = 0; k < cut[x + 1] - cut[x]; ++k) map[base + (size_t)8 * k + x] = r0 + cut[x] + k;
}

int make_m2l_map(Built* B, hipStream_t s, Error* err) {
  const int nbox = B->tree.nbox;
  if (B->m2l_map) {
    dev_free(B->m2l_map);
    B->m2l_map = nullptr;
  }
  B->m2l_part[0] = B->m2l_part[1] = B->m2l_part[2] = 0;
  if (nbox == 0) return 0;
  std::vector<int> off(nbox + 1);
  RPY_HIP(hipMemcpyAsync(off.data(), B->lists[LV].off, sizeof(int) * (nbox + 1), hipMemcpyDeviceToHost, s));
  RPY_HIP(hipStreamSynchronize(s));
  // boxes are numbered by level: the deepest level is the last range
  const int deep = B->level_start.empty() ? 0 : B->level_start[B->depth];
  std::vector<int> map;
  append_map(off, deep, nbox, map);
  B->m2l_part[1] = (int)map.size();
  append_map(off, 0, deep, map);
  B->m2l_part[2] = (int)map.size();
  if (map.empty()) return 0;
  RPY_HIP(dev_alloc(&B->m2l_map, sizeof(int) * map.size()));
  RPY_HIP(copy_in(B->m2l_map, map.data(), sizeof(int) * map.size(), s));
  B->bytes += (int64_t)sizeof(int) * map.size();
  return 0;
}

// The tables of k_m2l_rows for the plan's order and precision, from the host
// images of the rotation and z-translation matrices.
int make_m2l_tables(const std::vector<double>& rot, const std::vector<double>& zt, int fp32, Tables* tb,
                    TableImage* im) {
  const int p = tb->p, nc = rows_cols(p, fp32 ? 4 : 8);
  tb->rows_nc = nc;
  if (nc == 0) return 0;
  std::vector<double> tr, tz;
  if (nc == 32) rows_tables<32>(p, rot, zt, tr, tz);
  else rows_tables<16>(p, rot, zt, tr, tz);
  const size_t real = fp32 ? 4 : 8, np = (size_t)2 * 343 * (p + 1);
  const std::vector<float> fr(fp32 ? tr.begin() : tr.end(), tr.end()), fz(fp32 ? tz.begin() : tz.end(), tz.end());
  im->add(&tb->rows_rot, fp32 ? (const void*)fr.data() : tr.data(), real * tr.size());
  im->add(&tb->rows_zt, fp32 ? (const void*)fz.data() : tz.data(), real * tz.size());
  im->add(&tb->rows_ph, nullptr, 2 * real * np);
  return 0;
}

int make_m2l_phases(Tables* tb, int fp32, hipStream_t s, Error* err) {
  if (!tb->rows_ph) return 0;
  if (fp32) k_m2l_phases<float><<<dim3(6, 2), 64, 0, s>>>(tb->p, tb->geo, static_cast<float2*>(tb->rows_ph));
  else k_m2l_phases<double><<<dim3(6, 2), 64, 0, s>>>(tb->p, tb->geo, static_cast<double2*>(tb->rows_ph));
  RPY_HIP(hipGetLastError());
  return 0;
}

hipError_t run_m2l_rot(const Launch& l, int nrc, Exp e, int fp32, int part) {
  return fp32 ? launch_rot<float>(l, nrc, e, l.tb->rot32, l.tb->zt32, part)
              : launch_rot<double>(l, nrc, e, l.tb->rot64, l.tb->zt64, part);
}

}  // namespace rpy
