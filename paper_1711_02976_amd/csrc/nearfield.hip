// Near field of the RPY matvec: the exact RPY block (arXiv:1711.02976, Sec. 1,
// the three RPY block equations, kB*T = 1) summed over every bead of the
// U-list leaves of each target leaf (self term included), plus the overlap
// correction (M_overlap - M_far) F for pairs closer than 2a whose leaves are
// not adjacent (the far field treated them with the r >= 2a formula).
//
// One block of P2P_T threads per target tile (a leaf, or a P2P_T-bead slice
// of a large leaf), or per part of a tile's source chunks (NearWork below);
// each lane owns one target and keeps 3 * nrc sums in
// registers; source beads of each U-list leaf are staged through LDS
// (positions and forces, SoA) and read back as wave-wide broadcasts.  With
// 16 right-hand sides (in the FP64 form plus up to 8 more on the vector units
// of the same launch) the P2P runs on the matrix cores instead (k_p2p_mfma, 16 targets
// per wave, the 3x3 pair blocks as product operands).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fmm.h"

namespace rpy {

namespace {
constexpr double PI = 3.14159265358979323846;
constexpr int P2P_T = 128;
inline unsigned nblk(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

}  // namespace

// ---------------------------------------------------------------- tiles ---
__global__ void k_tile_count(const int* leaves, int nleaf, Tree t, int tile, int* cnt) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nleaf) return;
  int b = leaves[i];
  cnt[i] = (t.end[b] - t.begin[b] + tile - 1) / tile;
}

__global__ void k_tile_fill(const int* leaves, int nleaf, Tree t, int tile, const int* off, int4* out) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nleaf) return;
  int b = leaves[i];
  int o = off[i];
  for (int s = t.begin[b]; s < t.end[b]; s += tile) out[o++] = make_int4(b, s, min(tile, t.end[b] - s), i);
}

// Bounding box of each tile's beads: lo xyz, hi xyz.  One wave per tile (a
// thread per tile read its 128 beads one after another: 56 us for 2,048
// tiles).
__global__ void __launch_bounds__(64) k_tile_box(const int4* tiles, const double* sx, const double* sy,
                                                 const double* sz, double* box) {
  const int i = blockIdx.x, lane = threadIdx.x;
  const int4 tl = tiles[i];
  const double* c[3] = {sx + tl.y, sy + tl.y, sz + tl.y};
  for (int k = 0; k < 3; ++k) {
    double lo = c[k][0], hi = lo;
    for (int j = lane; j < tl.z; j += 64) {
      const double v = c[k][j];
      lo = fmin(lo, v);
      hi = fmax(hi, v);
    }
    for (int d = 1; d < 64; d <<= 1) {
      lo = fmin(lo, __shfl_xor(lo, d));
      hi = fmax(hi, __shfl_xor(hi, d));
    }
    if (lane == 0) {
      box[6 * (int64_t)i + k] = lo;
      box[6 * (int64_t)i + 3 + k] = hi;
    }
  }
}

int make_tiles(const Built* B, int tile, Tiles* out, hipStream_t s, Error* err) {
  out->n = 0;
  out->t = nullptr;
  out->box = nullptr;
  if (B->nleaf == 0) return 0;
  int *cnt = nullptr, *off = nullptr, *tmp = nullptr;
  RPY_HIP(dev_alloc(&cnt, sizeof(int) * B->nleaf));
  RPY_HIP(dev_alloc(&off, sizeof(int) * B->nleaf));
  RPY_HIP(dev_alloc(&tmp, sizeof(int) * scan_tmp_ints(B->nleaf)));
  k_tile_count<<<nblk(B->nleaf, 256), 256, 0, s>>>(B->leaf_ids, B->nleaf, B->tree, tile, cnt);
  RPY_PAGE(int, page);
  RPY_HIP(scan_exclusive(cnt, off, B->nleaf, tmp, s, page));
  RPY_HIP(hipStreamSynchronize(s));
  out->n = page[0];
  RPY_HIP(dev_alloc(&out->t, sizeof(int4) * out->n));
  k_tile_fill<<<nblk(B->nleaf, 256), 256, 0, s>>>(B->leaf_ids, B->nleaf, B->tree, tile, off, out->t);
  RPY_HIP(hipGetLastError());
  RPY_HIP(dev_alloc(&out->box, sizeof(double) * 6 * std::max(out->n, 1)));
  for (int64_t q = 0; q < out->n; q += launch_blocks(64)) {
    k_tile_box<<<(unsigned)std::min<int64_t>(out->n - q, launch_blocks(64)), 64, 0, s>>>(out->t + q, B->sx, B->sy, B->sz,
                                                                                      out->box + 6 * q);
    RPY_HIP(hipGetLastError());
  }
  dev_free(cnt); dev_free(off); dev_free(tmp);
  return 0;
}

// ------------------------------------------------------- near-field work --
// One block per tile leaves most of the chip idle when there are few tiles
// (2,000 beads in one leaf are 16 tiles) and lets the longest tile set a
// kernel's time when their source lists differ (two W-list neighbours of
// dense leaves took 13 ms alone on 64 systems).  So a tile's source chunks
// (P2P_T beads of one list entry each) are split over several blocks when it
// has more than cap = max(1, total / NEAR_ITEMS) of them: the parts' FP64
// sums go to slots of P2P_T targets each and are added in part order
// (k_near_reduce), so results do not depend on timing.  With many more than
// NEAR_ITEMS even tiles nothing is split and no table is kept.  Around that
// number the tiles just above the mean are cut in two: of a uniform cube's 8,192
// all interior ones, whose 54 chunks are 1.14 times the mean.  That pays too, since
// the shorter blocks end more evenly and share the chip better with the far field
// (whole tiles up to twice the mean and split ones: 778k beads, 20 right-hand
// sides, P2P 31.0 and 28.4 ms, matvec 100.4 and 98.5; 1M beads, one, matvec
// FP64 at 3 digits 7.60 and 7.33, mixed at 6 digits 6.25 and 6.12), at the price of
// the slots' memory (3 kB per slot and right-hand side, 0.67 GB for the 778k
// beads; without room for it the matvec runs whole tiles).  NEAR_ITEMS blocks fill
// the chip twice over in the lightest kernel (16 blocks of two waves per CU).
constexpr int NEAR_ITEMS = 8192;

// A W-list box of more than wmax beads is evaluated through its multipole.
struct ChunkFilter {
  int kind;  // LU, LW or LO
  int wmax;  // LW
  double four_a2;  // LO
};

// Whether the near field sums list entry C for a tile with bounding box tb
// (lo xyz, hi xyz): W boxes of few beads only; O leaves whose cube comes
// closer than 2a to the tile's beads.  The counting and filling of the parts and
// the kernels that walk them must agree on it to the last bit, so nothing of it is
// left to the compiler's choice of contractions.
__device__ inline bool near_takes(const ChunkFilter& f, const Tree& t, int C, const double* tb) {
#pragma clang fp contract(off)
  if (f.kind == LW) return t.end[C] - t.begin[C] <= f.wmax;
  if (f.kind == LO) {
    const double hc = 0.5 * t.h[C], cc[3] = {t.cx[C], t.cy[C], t.cz[C]};
    double g2 = 0.0;
    for (int q = 0; q < 3; ++q) {
      const double g = fmax(0.0, fmax(cc[q] - hc - tb[3 + q], tb[q] - cc[q] - hc));
      g2 += g * g;
    }
    return g2 < f.four_a2;
  }
  return true;
}

// cnt[i] = source chunks of tile i; stat[0] += their sum, stat[1] = max.
__global__ void __launch_bounds__(256) k_near_count(const int4* tiles, const double* tbox, int nt, Tree t, List l,
                                                    ChunkFilter f, int* cnt, unsigned long long* stat) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  int c = 0;
  if (i < nt) {
    const int b = tiles[i].x;
    for (int e = l.off[b]; e < l.off[b + 1]; ++e) {
      const int C = l.ent[e];
      if (near_takes(f, t, C, tbox + 6 * (int64_t)i)) c += (t.end[C] - t.begin[C] + P2P_T - 1) / P2P_T;
    }
    cnt[i] = c;
  }
  unsigned long long s = c, m = c;
  for (int d = 1; d < 64; d <<= 1) {
    s += __shfl_xor(s, d);
    const unsigned long long o = __shfl_xor(m, d);
    m = o > m ? o : m;
  }
  if ((threadIdx.x & 63) == 0 && m > 0) {
    atomicAdd(&stat[0], s);
    atomicMax(&stat[1], m);
  }
}

// parts[i] = blocks of tile i, held[i] = its slots (0 when it has one part),
// flag[i] = 1 if it has several.
__global__ void k_near_parts(const int* cnt, int nt, int cap, int* parts, int* held, int* flag) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nt) return;
  const int k = (cnt[i] + cap - 1) / cap;
  parts[i] = k;
  held[i] = k > 1 ? k : 0;
  flag[i] = k > 1;
}

// The parts of tile i: (tile, first list entry, first chunk of it, chunks)
// and the slot (-1: the tile has one part), its chunks split evenly.
__global__ void k_near_fill(const int4* tiles, const double* tbox, int nt, Tree t, List l, ChunkFilter f,
                            const int* cnt, const int* off, const int* parts, const int* slot0,
                            const int* order, int4* item, int* slot, int* red) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nt || parts[i] == 0) return;
  const int b = tiles[i].x, k = parts[i], c = cnt[i];
  if (k > 1) red[order[i]] = i;
  int e = l.off[b], ch = 0;  // the next chunk
  for (int q = 0; q < k; ++q) {
    int left = (int)((int64_t)c * (q + 1) / k - (int64_t)c * q / k);
    bool first = true;
    while (e < l.off[b + 1]) {
      const int C = l.ent[e];
      const int nc = near_takes(f, t, C, tbox + 6 * (int64_t)i) ? (t.end[C] - t.begin[C] + P2P_T - 1) / P2P_T : 0;
      if (nc == ch) {  // a refused entry, or past its last chunk
        ++e;
        ch = 0;
        continue;
      }
      if (first) {
        item[off[i] + q] = make_int4(i, e, ch, left);
        slot[off[i] + q] = k > 1 ? slot0[i] + q : -1;
        first = false;
      }
      const int take = min(left, nc - ch);
      ch += take;
      left -= take;
      if (left == 0) break;
    }
  }
}

// u (+)= the slots of a split tile (red[blockIdx.x]), in part order; one block
// per component row.
__global__ void __launch_bounds__(P2P_T) k_near_reduce(const int4* tiles, const int* red, const int* parts,
                                                       const int* slot0, const double* __restrict__ part, int nq,
                                                       int64_t n, int add, double* u) {
  const int i = red[blockIdx.x], k = parts[i], q = blockIdx.y;
  const int4 tl = tiles[i];
  if ((int)threadIdx.x >= tl.z) return;
  const double* p = part + ((int64_t)slot0[i] * nq + q) * P2P_T + threadIdx.x;
  double s = 0.0;
#pragma unroll 8
  for (int j = 0; j < k; ++j) s += p[(int64_t)j * nq * P2P_T];
  double* o = u + (int64_t)q * n + tl.y + threadIdx.x;
  *o = add ? *o + s : s;
}

static int make_near_work(const Built* B, const Tiles& tiles, const ChunkFilter& f, NearWork* out, hipStream_t s,
                          Error* err) {
  *out = NearWork{};
  const List& l = B->lists[f.kind];
  const int nt = tiles.n;
  if (nt == 0 || l.len == 0 || (f.kind == LW && f.wmax < 0)) return 0;
  // scratch: the counts, two statistics, and the tables' scans
  const size_t ntmp = scan_tmp_ints(nt);
  unsigned long long* stat = nullptr;
  RPY_HIP(dev_alloc(&stat, 2 * sizeof(unsigned long long) + sizeof(int) * (4 * (size_t)nt + ntmp)));
  int* cnt = reinterpret_cast<int*>(stat + 2);
  int *held = cnt + nt, *flag = held + nt, *order = flag + nt, *tmp = order + nt;
  RPY_HIP(hipMemsetAsync(stat, 0, 2 * sizeof(unsigned long long), s));
  k_near_count<<<nblk(nt, 256), 256, 0, s>>>(tiles.t, tiles.box, nt, B->tree, l, f, cnt, stat);
  RPY_HIP(hipGetLastError());
  unsigned long long hs[2] = {0, 0};
  RPY_HIP(hipMemcpyAsync(hs, stat, sizeof(hs), hipMemcpyDeviceToHost, s));
  RPY_HIP(hipStreamSynchronize(s));
  const unsigned long long cap = std::max<unsigned long long>(1, (hs[0] + NEAR_ITEMS - 1) / NEAR_ITEMS);
  out->nothing = hs[1] == 0;
  if (hs[1] > cap) {
    // at most total / cap + 1 per tile parts
    const size_t most = (size_t)NEAR_ITEMS + nt;
    RPY_HIP(dev_alloc(&out->item, sizeof(int4) * most + sizeof(int) * (most + 4 * (size_t)nt)));
    out->slot = reinterpret_cast<int*>(out->item + most);
    out->parts = out->slot + most;
    out->slot0 = out->parts + nt;
    out->red = out->slot0 + nt;
    out->off = out->red + nt;
    k_near_parts<<<nblk(nt, 256), 256, 0, s>>>(cnt, nt, (int)std::min<unsigned long long>(cap, 0x7fffffff),
                                               out->parts, held, flag);
    RPY_PAGE(int, page);
    RPY_HIP(scan_exclusive(out->parts, out->off, nt, tmp, s, page));
    RPY_HIP(scan_exclusive(held, out->slot0, nt, tmp, s, page + 1));
    RPY_HIP(scan_exclusive(flag, order, nt, tmp, s, page + 2));
    k_near_fill<<<nblk(nt, 64), 64, 0, s>>>(tiles.t, tiles.box, nt, B->tree, l, f, cnt, out->off, out->parts,
                                            out->slot0, order, out->item, out->slot, out->red);
    RPY_HIP(hipGetLastError());
    RPY_HIP(hipStreamSynchronize(s));
    out->n = page[0];
    out->nslot = page[1];
    out->nred = page[2];
  }
  dev_free(stat);
  return 0;
}

int make_near_plan(const Built* B, const Tiles& tiles, double a, int wd, NearPlan* out, hipStream_t s, Error* err) {
  const double four_a2 = 4.0 * a * a;
  if (int rc = make_near_work(B, tiles, ChunkFilter{LU, 0, four_a2}, &out->u, s, err)) return rc;
  if (int rc = make_near_work(B, tiles, ChunkFilter{LW, wd, four_a2}, &out->w, s, err)) return rc;
  return make_near_work(B, tiles, ChunkFilter{LO, 0, four_a2}, &out->o, s, err);
}

void free_near_plan(NearPlan* p) {
  for (NearWork* w : {&p->u, &p->w, &p->o}) {
    dev_free(w->item);  // the other tables follow it
    *w = NearWork{};
  }
  p->sub = p->direct = 0;
}

// The part of a tile's source chunks that a block sums: from NearWork's
// tables, or (no tables) all of tile blockIdx's list.
struct Part {
  int tile, e, c, left, slot;
  __device__ inline Part(const int4* item, const int* slots, int i, const int4* tiles, const List& l) {
    if (item) {
      const int4 it = item[i];
      tile = it.x;
      e = __builtin_amdgcn_readfirstlane(it.y);
      c = __builtin_amdgcn_readfirstlane(it.z);
      left = __builtin_amdgcn_readfirstlane(it.w);
      slot = __builtin_amdgcn_readfirstlane(slots[i]);
    } else {
      tile = i;
      e = __builtin_amdgcn_readfirstlane(l.off[tiles[i].x]);
      c = 0;
      left = 0x7fffffff;
      slot = -1;
    }
  }
};

// Where the sums of a block's targets go, row q = 3 r + c, target k of the
// tile: its slot, or u (assigned, or added when ADD).
struct Sums {
  double* p;
  int64_t ld;
  __device__ inline Sums(const Part& w, const int4& tl, int nq, int64_t n, double* u, double* part) {
    p = w.slot >= 0 ? part + (int64_t)w.slot * nq * P2P_T : u + tl.y;
    ld = w.slot >= 0 ? P2P_T : n;
  }
  __device__ inline double* at(int q, int k) const { return p + (int64_t)q * ld + k; }
};

// ------------------------------------------------------------ pair math ---

// Pair coefficients of the P2P sum with the far prefactor c1 = 1/(8 pi eta)
// taken out of the sum (applied once per target):
//   far      A' = 1/r + (2a^2/3)/r^3,        B' = (1 - 2a^2/r^2)/r^3,
//   overlap  A' = (c0/c1)(1 - 9r/(32a)),     B' = (c0/c1)(3/(32a))/r,
// c0/c1 = 4/(3a).  The pair kernels work in units scaled by a power of two S
// chosen so that 2aS lies in [1, 2): positions are scaled by S (exactly),
// the constants are those of the radius aS, and the sums come out divided by
// S, which the prefactor c1 S restores.  Apart from overflow and underflow
// this is the same arithmetic rounded the same way, and it keeps every pair
// quantity of order one whatever the length unit.
template <class R>
struct PairK {
  R a3;       // 2a^2/3
  R a2;       // 2a^2
  R four_a2;  // (2a)^2
  R oc;       // c0/c1
  R ock9;     // (c0/c1) 9/(32a)
  R ob;       // (c0/c1) 3/(32a)
  R r2min;    // floor added to r^2 before the reciprocal square root (coincident beads)
  R i2a;      // 1/(2a)
};

// Power of two S with 2aS in [1, 2).
static double pair_scale(double a) { return std::ldexp(1.0, -std::ilogb(2.0 * a)); }

// The FP64 kernels take the scaled positions as twice the distances in units twice
// as long, in which 2a lies in [1/2, 1): with r' = 2r the reciprocal square root's
// Newton step gives 1/r = 2/r' one operation sooner (rinv_of), and r'^2, which
// passes through an FP32 estimate, has the range that r^2 would have.  1/r and A'
// stay as they are; B', which multiplies d' d'^T = 4 d d^T, is a quarter.  All of
// it is exact scaling by powers of two.  With the wave's test for overlaps on FP32
// roundings, the FP64 P2P of one right-hand side takes 28 FP64 operations and roots
// per pair (30 before; 1M beads in leaves of 244: 7.18 ms and 6.96 now, 0.17 vector
// instructions per SIMD cycle of 2.4 GHz; FP64 alone reaches 0.21 to 0.24, roots 0.12).
template <class R>
constexpr double PAIR_ZOOM = std::is_same<R, double>::value ? 2.0 : 1.0;
template <class R>
constexpr R B_ONE = (R)(1.0 / (PAIR_ZOOM<R> * PAIR_ZOOM<R>));

// Constants for the scaled radius as = a S.
template <class R>
static PairK<R> pair_const(double as) {
  const double oc = 4.0 / (3.0 * as), z2 = PAIR_ZOOM<R> * PAIR_ZOOM<R>;
  return PairK<R>{(R)(2.0 * as * as / 3.0), (R)(2.0 * as * as / z2), (R)(4.0 * as * as * z2), (R)oc,
                  (R)(oc * 9.0 / (32.0 * as) / z2), (R)(oc * 3.0 / (32.0 * as) / z2), (R)(1e-30 * z2), (R)(0.5 / as)};
}

// 1/r from (PAIR_ZOOM r)^2.
__device__ inline float rinv_of(float r2) { return __builtin_amdgcn_rsqf(r2); }
// single-precision estimate w of 1/r' refined by one Newton step (relative error
// below 2^-44), 2/r' = w (3 - r'^2 w^2); r2 >= 4e-30 here (a normal FP32 number),
// so the estimate is finite
__device__ inline double rinv_of(double r2) {
  const double w = (double)__builtin_amdgcn_rsqf((float)r2);
  return w * fma(-r2, w * w, 3.0);
}

// --------------------------------------------------------------- P2P -----
// The overlap formula is evaluated only when some lane of the wave has a
// source closer than 2a (a wave-uniform branch), since such pairs are rare
// apart from each target's own bead.  For r = 0 (the bead itself, or a
// coincident bead) r^2 carries a floor of 1e-30 in the scaled units (r2min) (added
// in the first FMA) before the reciprocal square root: the far values are
// then finite and discarded, and the overlap values give the r -> 0 limit
// A' = c0/c1, B' d = 0.  Since 2a >= 1/2 in these units, the floor changes
// r^2 by a relative amount below 1e-29 at every r >= 2a, where the far
// formula applies.
// Positions enter the pair arithmetic relative to the target leaf's centre
// (differences taken in FP64, scaled by S and rounded once); in the mixed
// form the pair arithmetic and per-source-leaf sums run in FP32.
// The FP32 launch of 4 right-hand sides (the rest of 20 after the
// matrix-core group) is held to 96 registers, five waves per SIMD instead of
// four (two registers spill; 192 instead of 196 ms on cube-15M).
// DIRECT: plans without a far field whose near field is this kernel alone and
// takes few blocks (2,000 beads in one leaf), where launches and a block's own
// length are what counts.  Forces come straight from the caller's array sF
// ([n][3] per right-hand side) through perm, every block writes its sums to the
// slot of its own number, and k_direct_out adds them into the caller's array:
// two launches instead of four.  A part is split further over `sub` blocks, each
// taking P2P_T / sub sources of every chunk (FP64 form only: the mixed form's
// FP32 sums stay sums over whole chunks).  2,000 beads, FP64, one right-hand
// side: 22.7 us whole, 12.1 so.
template <int NRC, bool MIXED, bool DIRECT = false>
__global__ void __launch_bounds__(P2P_T, (NRC == 4 && MIXED) ? 5 : 1) k_p2p(const int4* tiles, const int4* item, const int* slots,
                                               Tree t, List U, const double* sx,
                                               const double* sy, const double* sz, const double* sF, int64_t n,
                                               PairK<typename std::conditional<MIXED, float, double>::type> k,
                                               double S, double c1, double* u, double* part,
                                               const int* perm = nullptr, int sub = 1) {
  using R = typename std::conditional<MIXED, float, double>::type;
  using V4 = typename std::conditional<MIXED, float4, double4>::type;
  __shared__ alignas(32) R xs[P2P_T];
  __shared__ alignas(32) R ys[P2P_T];
  __shared__ alignas(32) R zs[P2P_T];
  __shared__ alignas(32) R fs[NRC * 3][P2P_T];
  Part w(item, slots, DIRECT ? blockIdx.x / sub : xcd_run(blockIdx.x, gridDim.x), tiles, U);
  const int take = DIRECT ? P2P_T / sub : P2P_T, skip = DIRECT ? blockIdx.x % sub * take : 0;
  const int4 tl = tiles[w.tile];
  const int b = tl.x;
  const bool valid = (int)threadIdx.x < tl.z;
  const bool wlive = (int)(threadIdx.x & ~63u) < tl.z;  // this wave holds a target of the tile
  const int i = tl.y + (valid ? threadIdx.x : 0);
  const double ox = t.cx[b], oy = t.cy[b], oz = t.cz[b];
  const R xi = (R)((sx[i] - ox) * S), yi = (R)((sy[i] - oy) * S), zi = (R)((sz[i] - oz) * S);
  double acc[NRC][3];
  for (int r = 0; r < NRC; ++r) acc[r][0] = acc[r][1] = acc[r][2] = 0.0;
  const int e1 = __builtin_amdgcn_readfirstlane(U.off[b + 1]);
  for (; w.e < e1 && w.left > 0; ++w.e, w.c = 0) {
    const int C = __builtin_amdgcn_readfirstlane(U.ent[w.e]);
    const int j1 = __builtin_amdgcn_readfirstlane(t.end[C]);
    for (int jc = __builtin_amdgcn_readfirstlane(t.begin[C]) + w.c * P2P_T; jc < j1 && w.left > 0; jc += P2P_T, --w.left) {
      const int ns = min(take, j1 - jc - skip);
      if (DIRECT && ns <= 0) continue;
      // the tile is padded to a multiple of 4 sources with inert ones: zero
      // force at 1e30, where 1/r, A' and B' all evaluate to exactly zero
      const int ns4 = (ns + 3) & ~3;
      __syncthreads();
      if ((int)threadIdx.x < ns) {
        const int j = jc + skip + threadIdx.x;
        xs[threadIdx.x] = (R)((sx[j] - ox) * S); ys[threadIdx.x] = (R)((sy[j] - oy) * S);
        zs[threadIdx.x] = (R)((sz[j] - oz) * S);
        const int64_t pj = DIRECT ? perm[j] : 0;
        for (int q = 0; q < NRC * 3; ++q)
          fs[q][threadIdx.x] = (R)(DIRECT ? sF[((q / 3) * n + pj) * 3 + q % 3] : sF[(int64_t)q * n + j]);
      } else if ((int)threadIdx.x < ns4) {
        xs[threadIdx.x] = (R)1e30; ys[threadIdx.x] = (R)1e30; zs[threadIdx.x] = (R)1e30;
        for (int q = 0; q < NRC * 3; ++q) fs[q][threadIdx.x] = (R)0;
      }
      __syncthreads();
      R ar[NRC][3];
      for (int r = 0; r < NRC; ++r) ar[r][0] = ar[r][1] = ar[r][2] = (R)0;
      // four sources per trip, read as vectors; one wave-wide test for the
      // overlap branch per trip.  A wave with no target of the tile (the
      // second wave of a tile of 64 beads or fewer) stages and syncs only.
      for (int s0 = 0; s0 < (wlive ? ns4 : 0); s0 += 4) {
        const V4 X4 = *reinterpret_cast<const V4*>(xs + s0), Y4 = *reinterpret_cast<const V4*>(ys + s0),
                 Z4 = *reinterpret_cast<const V4*>(zs + s0);
        // padding sources: r^2 overflows to inf in FP32, 1/r = 0, A = B = 0
        const R dx[4] = {xi - X4.x, xi - X4.y, xi - X4.z, xi - X4.w};
        const R dy[4] = {yi - Y4.x, yi - Y4.y, yi - Y4.z, yi - Y4.w};
        const R dz[4] = {zi - Z4.x, zi - Z4.y, zi - Z4.z, zi - Z4.w};
        R r2[4], rinv[4], A[4], B[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          // r^2 + r2min: the floor rides in the first FMA instead of a max
          r2[q] = fma(dx[q], dx[q], fma(dy[q], dy[q], fma(dz[q], dz[q], k.r2min)));
          rinv[q] = rinv_of(r2[q]);
          const R ri2 = rinv[q] * rinv[q], ri3 = ri2 * rinv[q];
          A[q] = fma(k.a3, ri3, rinv[q]);
          B[q] = ri3 * fma(-k.a2, ri2, B_ONE<R>);
        }
        // in FP32 also in the FP64 form: r2 < (2a)^2 implies the same, or
        // equality, of their roundings, and the exact test follows
        const float r2lo = fminf(fminf((float)r2[0], (float)r2[1]), fminf((float)r2[2], (float)r2[3]));
        if (__builtin_expect(__any(MIXED ? r2lo < (float)k.four_a2 : r2lo <= (float)k.four_a2), 0)) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const bool ov = r2[q] < k.four_a2;
            // r from r^2 without the floor: exactly 0 for the bead itself
            const R Ao = fma(-k.ock9, (r2[q] - k.r2min) * rinv[q], k.oc), Bo = k.ob * rinv[q];
            A[q] = ov ? Ao : A[q];
            B[q] = ov ? Bo : B[q];
          }
        }
        // with several right-hand sides, B d is formed once per pair (3
        // multiplies) so that each right-hand side costs 9 operations:
        // t = d.F, u += A F + t (B d)
        R bdx[4], bdy[4], bdz[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bdx[q] = NRC >= 4 ? B[q] * dx[q] : dx[q];
          bdy[q] = NRC >= 4 ? B[q] * dy[q] : dy[q];
          bdz[q] = NRC >= 4 ? B[q] * dz[q] : dz[q];
        }
#pragma unroll
        for (int r = 0; r < NRC; ++r) {
          const V4 FX = *reinterpret_cast<const V4*>(&fs[3 * r][s0]), FY = *reinterpret_cast<const V4*>(&fs[3 * r + 1][s0]),
                   FZ = *reinterpret_cast<const V4*>(&fs[3 * r + 2][s0]);
          const R fx[4] = {FX.x, FX.y, FX.z, FX.w}, fy[4] = {FY.x, FY.y, FY.z, FY.w}, fz[4] = {FZ.x, FZ.y, FZ.z, FZ.w};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const R dF = fma(dx[q], fx[q], fma(dy[q], fy[q], dz[q] * fz[q]));
            const R t = NRC >= 4 ? dF : B[q] * dF;
            ar[r][0] = fma(A[q], fx[q], fma(t, bdx[q], ar[r][0]));
            ar[r][1] = fma(A[q], fy[q], fma(t, bdy[q], ar[r][1]));
            ar[r][2] = fma(A[q], fz[q], fma(t, bdz[q], ar[r][2]));
          }
        }
      }
      for (int r = 0; r < NRC; ++r)
        for (int c = 0; c < 3; ++c) acc[r][c] += (double)ar[r][c];
    }
  }
  if (DIRECT) w.slot = blockIdx.x;
  const Sums o(w, tl, 3 * NRC, n, u, part);
  if (valid)
    for (int r = 0; r < NRC; ++r)
      for (int c = 0; c < 3; ++c) *o.at(3 * r + c, threadIdx.x) = c1 * acc[r][c];
}

// The direct sums into the caller's array: the slots of tile i's parts (cnt[i]
// from off[i] on; without tables, part i), sub of each, in order.  One block per
// tile and component row: DO_G waves' worth of slots side by side, then their sum.
constexpr int DO_G = 4;
__global__ void __launch_bounds__(P2P_T * DO_G) k_direct_out(const int4* tiles, const int* off, const int* cnt, int sub,
                                                             const double* __restrict__ part, int nq, int64_t n,
                                                             const int* perm, double* out) {
  const int i = blockIdx.x, q = blockIdx.y, x = threadIdx.x % P2P_T, g = threadIdx.x / P2P_T;
  const int4 tl = tiles[i];
  const int s0 = (off ? off[i] : i) * sub, k = (off ? cnt[i] : 1) * sub;
  const double* p = part + ((int64_t)s0 * nq + q) * P2P_T + x;
  __shared__ double sum[DO_G][P2P_T];
  double s = 0.0;
  if (x < tl.z)
#pragma unroll 8
    for (int j = g; j < k; j += DO_G) s += p[(int64_t)j * nq * P2P_T];
  sum[g][x] = s;
  __syncthreads();
  if (g == 0 && x < tl.z)
    out[((q / 3) * n + perm[tl.y + x]) * 3 + q % 3] = (sum[0][x] + sum[1][x]) + (sum[2][x] + sum[3][x]);
}

// ------------------------------------------- P2P on the matrix cores ----
// With 16 right-hand sides the P2P of a target tile is a product
//   U[3 x targets][16] += M[3 x targets][3 x sources] F[3 x sources][16]
// whose 3x3 blocks M_ij = A_ij I + B_ij d d^T (the RPY block of Sec. 1, with
// the overlap branch for r < 2a) are formed on the fly.  A wave owns 16
// targets; per step of 4 sources each lane forms one pair (target lane % 16,
// source lane / 16) and the six distinct entries of its block, which are
// exactly the A operands of 16x16x4 matrix-core products in that lane:
// D_a += M_ab F_b for a, b in {x, y, z}, nine products per step, with F_b
// (source, right-hand side) as the B operand.  The FP32 form uses
// v_mfma_f32_16x16x4f32 and adds D into FP64 sums after each staged chunk of
// sources (as the vector kernel does); the FP64 form uses
// v_mfma_f64_16x16x4f64 and keeps the sums in D.
// In the FP64 form XR = 1, 2, 4 or 8 further right-hand sides ride in the
// same launch on the vector units: each lane applies its pair block to them
// (nine multiply-adds per right-hand side), so the pair geometry is formed
// once for 16 + XR right-hand sides.  FP32 and FP64 products and vector
// instructions do not overlap on this chip (measured: their times add at one
// to eight waves per SIMD), so the bound is their sum: per step nine products
// (290 cycles of 2.4 GHz in FP32, 687 in FP64, whose load lowers the clock) and
// about 27 (FP64 16 + 4: 80) vector instructions of 2.4 (FP64: 4.2).  Products and
// plain multiply-adds in these numbers alone take 374 (1,020) cycles per step, 423
// ms (1,157) on 15M beads; the launches take 480 (1,202), 88 % (96 %) of it.  The
// forces are staged row by row as they lie in memory, in rows whose padding keeps
// both the stores and the reads free of bank conflicts (with index arithmetic per
// staged force and 16 lanes per bank the FP32 launch took 506).  Their per-lane
// partial sums are added
// over the four source lanes of a target after each staged chunk, and lane
// (t, k) keeps the FP64 sums of the right-hand sides k, k + 4.  (The mixed
// form runs its extra right-hand sides in the vector kernel: there the
// registers they take cost the matrix-core loop more than the shared
// geometry saves.)
namespace {
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef double v4d_t __attribute__((ext_vector_type(4)));
constexpr int MF_W = 8;         // waves per block: 16 targets each, P2P_T per tile
constexpr int MF_R = NEAR_MC_RHS;  // right-hand sides on the matrix cores (the product's N)
__device__ inline v4f_t mfma16(float a, float b, v4f_t c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
__device__ inline v4d_t mfma16(double a, double b, v4d_t c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
// Row (target within the wave's 16) of item v of a 16x16 result in lane l;
// the column (right-hand side) is l % 16 in both forms.
// LDS row length of the staged forces: reads of lane (target t, source k) at
// row 3 t + c, source s + k fall into 64 different banks (FP32: 12 t + k mod 64;
// FP64: 30 t + k mod 32 per half wave); with 8 vector-unit right-hand sides a
// shorter row, two lanes per bank, keeps two blocks per CU.
constexpr int mf_ld(bool mixed, int xr) { return mixed ? 132 : (xr < 8 ? 138 : 131); }
__device__ inline int mf_row(float, int l, int v) { return 4 * (l >> 4) + v; }
__device__ inline int mf_row(double, int l, int v) { return 4 * v + (l >> 4); }
}  // namespace

template <bool MIXED, int XR>
__global__ void __launch_bounds__(64 * MF_W) k_p2p_mfma(const int4* tiles, const int4* item, const int* slots,
                                                       Tree t, List U, const double* sx,
                                                       const double* sy, const double* sz, const double* sF,
                                                       int64_t n,
                                                       PairK<typename std::conditional<MIXED, float, double>::type> k,
                                                       double S, double c1, double* u, double* part) {
  using R = typename std::conditional<MIXED, float, double>::type;
  using R4 = typename std::conditional<MIXED, float4, double4>::type;
  using VD = typename std::conditional<MIXED, v4f_t, v4d_t>::type;
  constexpr int XS = XR > 0 ? XR : 1, XH = (XR + 3) / 4 > 0 ? (XR + 3) / 4 : 1;
  constexpr int ROWS = 3 * (MF_R + XR), LD = mf_ld(MIXED, XR);
  __shared__ R4 ps[P2P_T];      // positions (x, y, z, -)
  // forces along the sources: row 3 x + c of the vector-unit right-hand side x,
  // then row 3 r + c of the others (both within reach of a load's offset)
  __shared__ R fs[ROWS][LD];
  Part w(item, slots, xcd_run(blockIdx.x, gridDim.x), tiles, U);
  const int4 tl = tiles[w.tile];
  const int b = tl.x;
  const int tid = threadIdx.x, lane = tid & 63;
  const int t0 = 16 * __builtin_amdgcn_readfirstlane(tid >> 6);  // the wave's first target in the tile
  const bool wlive = t0 < tl.z;
  const int ti = lane & 15, sk = lane >> 4;  // lane's target row and source within a step
  // rows past the tile take its last target (finite values, never stored)
  const int i = tl.y + max(0, min(t0 + ti, tl.z - 1));
  const double ox = t.cx[b], oy = t.cy[b], oz = t.cz[b];
  const R xi = (R)((sx[i] - ox) * S), yi = (R)((sy[i] - oy) * S), zi = (R)((sz[i] - oz) * S);
  VD D[3];
  double acc[3][4];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    D[c] = VD{0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[c][v] = 0.0;
  }
  R xa[XS][3];      // this lane's pair sums of the vector-unit right-hand sides (one chunk)
  double xacc[XH][3];  // FP64 sums of right-hand sides sk + 4 h for target ti
#pragma unroll
  for (int h = 0; h < XH; ++h) xacc[h][0] = xacc[h][1] = xacc[h][2] = 0.0;
  const int e1 = __builtin_amdgcn_readfirstlane(U.off[b + 1]);
  for (; w.e < e1 && w.left > 0; ++w.e, w.c = 0) {
    const int C = __builtin_amdgcn_readfirstlane(U.ent[w.e]);
    const int j1 = __builtin_amdgcn_readfirstlane(t.end[C]);
    for (int jc = __builtin_amdgcn_readfirstlane(t.begin[C]) + w.c * P2P_T; jc < j1 && w.left > 0; jc += P2P_T, --w.left) {
      const int ns = min(P2P_T, j1 - jc);
      // padded to a multiple of 4 sources with inert ones (zero force at 1e30)
      const int ns4 = (ns + 3) & ~3;
      __syncthreads();
      if (tid < ns) {
        const int j = jc + tid;
        ps[tid] = R4{(R)((sx[j] - ox) * S), (R)((sy[j] - oy) * S), (R)((sz[j] - oz) * S), (R)0};
      } else if (tid < ns4) {
        ps[tid] = R4{(R)1e30, (R)1e30, (R)1e30, (R)0};
      }
      // forces: rows of sF, read and stored along the sources; a thread keeps
      // its source and takes every fourth row
      {
        const int sj = tid & (P2P_T - 1), row0 = __builtin_amdgcn_readfirstlane(tid / P2P_T);
        const double* F = sF + (int64_t)row0 * n + jc + min(sj, ns - 1);
        if (sj < ns4)
#pragma unroll
          for (int row = row0, q = 0; q < (ROWS + 3) / 4; ++q, row += 64 * MF_W / P2P_T, F += 64 * MF_W / P2P_T * n)
            if (ROWS % 4 == 0 || row < ROWS) {
              const R v = (R)*F;
              fs[XR == 0 || row < 3 * MF_R ? row + 3 * XR : row - 3 * MF_R][sj] = sj < ns ? v : (R)0;
            }
      }
      __syncthreads();
      if (wlive) {
        R m[6], f[3];
#pragma unroll
        for (int x = 0; x < XS; ++x) xa[x][0] = xa[x][1] = xa[x][2] = (R)0;
        for (int s0 = 0; s0 < ns4; s0 += 4) {
          const int j = s0 + sk;
          const R4 p = ps[j];
          {  // the pair block, as in k_p2p: six distinct entries xx, yy, zz, xy, xz, yz
            const R dx = xi - p.x, dy = yi - p.y, dz = zi - p.z;
            const R r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, k.r2min)));
            const R rinv = rinv_of(r2);
            const R ri2 = rinv * rinv, ri3 = ri2 * rinv;
            R A = fma(k.a3, ri3, rinv);
            R B = ri3 * fma(-k.a2, ri2, B_ONE<R>);
            if (__builtin_expect(__any(r2 < k.four_a2), 0)) {
              const bool ov = r2 < k.four_a2;
              const R Ao = fma(-k.ock9, (r2 - k.r2min) * rinv, k.oc), Bo = k.ob * rinv;
              A = ov ? Ao : A;
              B = ov ? Bo : B;
            }
            const R bx = B * dx, by = B * dy, bz = B * dz;
            m[0] = fma(bx, dx, A);
            m[1] = fma(by, dy, A);
            m[2] = fma(bz, dz, A);
            m[3] = bx * dy;
            m[4] = bx * dz;
            m[5] = by * dz;
          }
          f[0] = fs[3 * XR + 3 * ti][j];
          f[1] = fs[3 * XR + 3 * ti + 1][j];
          f[2] = fs[3 * XR + 3 * ti + 2][j];
          D[0] = mfma16(m[0], f[0], D[0]);
          D[1] = mfma16(m[3], f[0], D[1]);
          D[2] = mfma16(m[4], f[0], D[2]);
          D[0] = mfma16(m[3], f[1], D[0]);
          D[1] = mfma16(m[1], f[1], D[1]);
          D[2] = mfma16(m[5], f[1], D[2]);
          D[0] = mfma16(m[4], f[2], D[0]);
          D[1] = mfma16(m[5], f[2], D[1]);
          D[2] = mfma16(m[2], f[2], D[2]);
#pragma unroll
          for (int x = 0; x < XR; ++x) {
            const R gx = fs[3 * x][j], gy = fs[3 * x + 1][j], gz = fs[3 * x + 2][j];
            xa[x][0] = fma(m[0], gx, fma(m[3], gy, fma(m[4], gz, xa[x][0])));
            xa[x][1] = fma(m[3], gx, fma(m[1], gy, fma(m[5], gz, xa[x][1])));
            xa[x][2] = fma(m[4], gx, fma(m[5], gy, fma(m[2], gz, xa[x][2])));
          }
        }
        if (MIXED) {
#pragma unroll
          for (int c = 0; c < 3; ++c) {
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[c][v] += (double)D[c][v];
            D[c] = VD{0, 0, 0, 0};
          }
        }
        // the chunk's sums over the four source lanes of each target; lane
        // sk keeps right-hand sides sk, sk + 4
#pragma unroll
        for (int x = 0; x < XR; ++x)
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            R v = xa[x][c];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (sk == (x & 3)) xacc[x >> 2][c] += (double)v;
          }
      }
    }
  }
  if (!wlive) return;
  const Sums o(w, tl, 3 * (MF_R + XR), n, u, part);
#pragma unroll
  for (int c = 0; c < 3; ++c)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = mf_row(R(0), lane, v);
      if (t0 + row < tl.z) {
        const double x = MIXED ? acc[c][v] : (double)D[c][v];
        *o.at(3 * ti + c, t0 + row) = c1 * x;
      }
    }
  if (t0 + ti < tl.z)
#pragma unroll
    for (int h = 0; h < XH; ++h) {
      const int x = sk + 4 * h;
      if (x < XR)
#pragma unroll
        for (int c = 0; c < 3; ++c) *o.at(3 * (MF_R + x) + c, t0 + ti) = c1 * xacc[h][c];
    }
}

// ---------------------------------------------------- W list, direct ----
// W-list boxes with few beads: their multipole evaluation at this leaf's
// targets (Theorem 1, order p + 2) costs more than summing their beads, so
// they are summed directly with the far formula, which is what the far field
// stands for (pairs closer than 2a are then corrected by the O list as
// before).  Boxes with more than wmax beads keep the multipole route.
template <int NRC, bool MIXED>
__global__ void __launch_bounds__(P2P_T) k_wdirect(const int4* tiles, const int4* item, const int* slots,
                                                   Tree t, List W, ChunkFilter filter, const double* sx,
                                                   const double* sy, const double* sz, const double* sF, int64_t n,
                                                   PairK<typename std::conditional<MIXED, float, double>::type> k,
                                                   double S, double c1, double* u, double* part) {
  using R = typename std::conditional<MIXED, float, double>::type;
  __shared__ R xs[P2P_T], ys[P2P_T], zs[P2P_T];
  __shared__ R fs[NRC * 3][P2P_T];
  Part w(item, slots, blockIdx.x, tiles, W);
  const int4 tl = tiles[w.tile];
  const int b = tl.x;
  const int e1 = __builtin_amdgcn_readfirstlane(W.off[b + 1]);
  if (w.e == e1) return;
  const bool valid = (int)threadIdx.x < tl.z;
  const bool wlive = (int)(threadIdx.x & ~63u) < tl.z;  // this wave holds a target of the tile
  const int i = tl.y + (valid ? threadIdx.x : 0);
  const double ox = t.cx[b], oy = t.cy[b], oz = t.cz[b];  // positions relative to the target leaf
  const R xi = (R)((sx[i] - ox) * S), yi = (R)((sy[i] - oy) * S), zi = (R)((sz[i] - oz) * S);
  double acc[NRC][3];
  for (int r = 0; r < NRC; ++r) acc[r][0] = acc[r][1] = acc[r][2] = 0.0;
  bool any = false;
  for (; w.e < e1 && w.left > 0; ++w.e, w.c = 0) {
    const int C = __builtin_amdgcn_readfirstlane(W.ent[w.e]);
    const int j0 = __builtin_amdgcn_readfirstlane(t.begin[C]), j1 = __builtin_amdgcn_readfirstlane(t.end[C]);
    if (!near_takes(filter, t, C, nullptr)) continue;
    any = true;
    for (int jc = j0 + w.c * P2P_T; jc < j1 && w.left > 0; jc += P2P_T, --w.left) {
      const int ns = min(P2P_T, j1 - jc);
      const int ns4 = (ns + 3) & ~3;
      __syncthreads();
      if ((int)threadIdx.x < ns) {
        int j = jc + threadIdx.x;
        xs[threadIdx.x] = (R)((sx[j] - ox) * S); ys[threadIdx.x] = (R)((sy[j] - oy) * S);
        zs[threadIdx.x] = (R)((sz[j] - oz) * S);
        for (int q = 0; q < NRC * 3; ++q) fs[q][threadIdx.x] = (R)sF[(int64_t)q * n + j];
      } else if ((int)threadIdx.x < ns4) {
        xs[threadIdx.x] = (R)1e30; ys[threadIdx.x] = (R)1e30; zs[threadIdx.x] = (R)1e30;
        for (int q = 0; q < NRC * 3; ++q) fs[q][threadIdx.x] = (R)0;
      }
      __syncthreads();
      R ar[NRC][3];
      for (int r = 0; r < NRC; ++r) ar[r][0] = ar[r][1] = ar[r][2] = (R)0;
      for (int s0 = 0; s0 < (wlive ? ns4 : 0); s0 += 4)
#pragma unroll
      for (int s = s0; s < s0 + 4; ++s) {
        const R dx = xi - xs[s], dy = yi - ys[s], dz = zi - zs[s];
        const R r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, k.r2min)));
        const R rinv = rinv_of(r2);
        const R ri2 = rinv * rinv, ri3 = ri2 * rinv;
        const R A = fma(k.a3, ri3, rinv), B = ri3 * fma(-k.a2, ri2, B_ONE<R>);
#pragma unroll
        for (int r = 0; r < NRC; ++r) {
          const R fx = fs[3 * r][s], fy = fs[3 * r + 1][s], fz = fs[3 * r + 2][s];
          const R sdf = B * fma(dx, fx, fma(dy, fy, dz * fz));
          ar[r][0] = fma(A, fx, fma(sdf, dx, ar[r][0]));
          ar[r][1] = fma(A, fy, fma(sdf, dy, ar[r][1]));
          ar[r][2] = fma(A, fz, fma(sdf, dz, ar[r][2]));
        }
      }
      for (int r = 0; r < NRC; ++r)
        for (int c = 0; c < 3; ++c) acc[r][c] += (double)ar[r][c];
    }
  }
  const Sums o(w, tl, 3 * NRC, n, u, part);
  if (valid && any)
    for (int r = 0; r < NRC; ++r)
      for (int c = 0; c < 3; ++c) {
        double* x = o.at(3 * r + c, threadIdx.x);
        *x = w.slot >= 0 ? c1 * acc[r][c] : *x + c1 * acc[r][c];
      }
}

// ------------------------------------------------------- overlap (O) -----
// Pairs closer than 2a whose leaves are not adjacent: the far field treated
// them with the r >= 2a formula, so (M_overlap - M_far) F is added.  Same
// tiling as the P2P (padded, unrolled by 4); leaves of the O list are
// separated, so r > 0 and the far values are finite.  Pairs at r >= 2a get a
// zero coefficient (masked, no branch).  With the prefactor taken out and
// rho = r/(2a), the two branches' differences are
//   A' = oc (1 - 9r/(32a)) - 1/r - (2a^2/3)/r^3
//      = -(2a^2/3) (1 - rho)^2 (9 rho^2 + 2 rho + 1) / r^3,
//   B' = ob/r - (1 - 2a^2/r^2)/r^3 = 2a^2 (1 - rho)^2 (1 + rho)^2 / r^5,
// both with a double zero at r = 2a, where the branches meet.  In this
// factored form nothing cancels, so the mixed form evaluates it in FP32
// (rounding errors relative to the difference itself) and, as the P2P, adds
// each staged chunk's FP32 sums into FP64.  The FP64 form subtracts the two
// branches (fewer operations; the cancellation costs digits FP64 can spare).
// Most pairs of two such leaves are farther apart than 2a, so the staged
// sources are cut into groups of OV_G with bounding boxes, and a wave skips a
// group whose box is 2a or more from every one of the wave's targets.  The lanes
// first test all of a chunk's groups at once against the box of the wave's
// targets (4M clustered beads, 4 right-hand sides, of all groups two in five are
// out of reach: 84.7 ms and 79.8; the pairs in reach issue 0.27 vector
// instructions per SIMD cycle of the 0.41 that plain FP32 reaches).
constexpr int OV_G = 4;

template <int NRC, bool MIXED>
__global__ void __launch_bounds__(P2P_T) k_overlap(const int4* tiles, const double* tbox, const int4* item,
                                                   const int* slots, Tree t, List O, ChunkFilter filter,
                                                   const double* sx,
                                                   const double* sy, const double* sz, const double* sF, int64_t n,
                                                   PairK<typename std::conditional<MIXED, float, double>::type> k,
                                                   double S, double c1, double* u, double* part) {
  using R = typename std::conditional<MIXED, float, double>::type;
  constexpr int NG = P2P_T / OV_G;
  __shared__ R xs[P2P_T], ys[P2P_T], zs[P2P_T];
  __shared__ R fs[NRC * 3][P2P_T];
  __shared__ R gbox[NG][6];  // per source group: lo xyz, hi xyz
  Part w(item, slots, blockIdx.x, tiles, O);
  const int4 tl = tiles[w.tile];
  const int b = tl.x;
  const int e1 = __builtin_amdgcn_readfirstlane(O.off[b + 1]);
  if (w.e == e1) return;
  const bool valid = (int)threadIdx.x < tl.z;
  const bool wlive = (int)(threadIdx.x & ~63u) < tl.z;  // this wave holds a target of the tile
  const int i = tl.y + (valid ? threadIdx.x : 0);
  const double ox = t.cx[b], oy = t.cy[b], oz = t.cz[b];  // positions relative to the target leaf
  const R xi = (R)((sx[i] - ox) * S), yi = (R)((sy[i] - oy) * S), zi = (R)((sz[i] - oz) * S);
  // a group is skipped only when its box is clearly 2a away (rounding margin,
  // scaled units); idle lanes repeat the tile's first bead, so they add no
  // extra groups
  const R skip2 = k.four_a2 * (R)(1.0 + 1e-4);
  double acc[NRC][3];
  for (int r = 0; r < NRC; ++r) acc[r][0] = acc[r][1] = acc[r][2] = 0.0;
  R wb[6];  // the wave's targets' bounding box (idle lanes repeat a target)
  {
    const R p[3] = {xi, yi, zi};
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      wb[q] = wb[3 + q] = p[q];
      for (int d = 1; d < 64; d <<= 1) {
        wb[q] = min(wb[q], __shfl_xor(wb[q], d));
        wb[3 + q] = max(wb[3 + q], __shfl_xor(wb[3 + q], d));
      }
    }
  }
  double tb[6];  // the tile's bounding box
  for (int q = 0; q < 6; ++q) tb[q] = tbox[6 * (int64_t)w.tile + q];
  for (; w.e < e1 && w.left > 0; ++w.e, w.c = 0) {
    const int C = __builtin_amdgcn_readfirstlane(O.ent[w.e]);
    // skip source leaves whose cube is 2a or more away from this tile's beads
    if (!near_takes(filter, t, C, tb)) continue;
    const int j1 = __builtin_amdgcn_readfirstlane(t.end[C]);
    for (int jc = __builtin_amdgcn_readfirstlane(t.begin[C]) + w.c * P2P_T; jc < j1 && w.left > 0; jc += P2P_T, --w.left) {
      const int ns = min(P2P_T, j1 - jc);
      const int ns4 = (ns + 3) & ~3;
      __syncthreads();
      if ((int)threadIdx.x < ns) {
        int j = jc + threadIdx.x;
        xs[threadIdx.x] = (R)((sx[j] - ox) * S); ys[threadIdx.x] = (R)((sy[j] - oy) * S);
        zs[threadIdx.x] = (R)((sz[j] - oz) * S);
        for (int q = 0; q < NRC * 3; ++q) fs[q][threadIdx.x] = (R)sF[(int64_t)q * n + j];
      } else if ((int)threadIdx.x < ns4) {
        xs[threadIdx.x] = (R)1e30; ys[threadIdx.x] = (R)1e30; zs[threadIdx.x] = (R)1e30;
        for (int q = 0; q < NRC * 3; ++q) fs[q][threadIdx.x] = (R)0;
      }
      __syncthreads();
      const int ng = (ns + OV_G - 1) / OV_G;
      if ((int)threadIdx.x < 3 * ng) {
        // box of the real sources of group g along one axis
        const int g = threadIdx.x / 3, q = threadIdx.x - 3 * g;
        const R* col = q == 0 ? xs : (q == 1 ? ys : zs);
        const int s1 = min(g * OV_G + OV_G, ns);
        R lo = col[g * OV_G], hi = lo;
        for (int s = g * OV_G + 1; s < s1; ++s) {
          lo = min(lo, col[s]);
          hi = max(hi, col[s]);
        }
        gbox[g][q] = lo;
        gbox[g][3 + q] = hi;
      }
      __syncthreads();
      R ar[NRC][3];
      for (int r = 0; r < NRC; ++r) ar[r][0] = ar[r][1] = ar[r][2] = (R)0;
      // the groups whose boxes come within 2a of the wave's targets' box, one per
      // lane (at most 32 of them)
      unsigned long long near = 0;
      {
        const int g = (threadIdx.x & 63) < (unsigned)ng ? threadIdx.x & 63 : 0;
        const R gx = max((R)0, max(gbox[g][0] - wb[3], wb[0] - gbox[g][3]));
        const R gy = max((R)0, max(gbox[g][1] - wb[4], wb[1] - gbox[g][4]));
        const R gz = max((R)0, max(gbox[g][2] - wb[5], wb[2] - gbox[g][5]));
        near = __ballot((int)(threadIdx.x & 63) < (wlive ? ng : 0) && fma(gx, gx, fma(gy, gy, gz * gz)) < skip2);
      }
      for (; near; near &= near - 1) {
        const int g = __builtin_ctzll(near);
        // distance from this lane's target to the group's box; the wave
        // skips the group when no lane comes within 2a of it
        const R gx = max((R)0, max(gbox[g][0] - xi, xi - gbox[g][3]));
        const R gy = max((R)0, max(gbox[g][1] - yi, yi - gbox[g][4]));
        const R gz = max((R)0, max(gbox[g][2] - zi, zi - gbox[g][5]));
        const R g2 = fma(gx, gx, fma(gy, gy, gz * gz));
        if (!__any(g2 < skip2)) continue;  // wave-uniform
        const int s1 = min(g * OV_G + OV_G, ns4);
        for (int s0 = g * OV_G; s0 < s1; s0 += 4)
#pragma unroll
        for (int s = s0; s < s0 + 4; ++s) {
          const R dx = xi - xs[s], dy = yi - ys[s], dz = zi - zs[s];
          const R r2 = fma(dx, dx, fma(dy, dy, fma(dz, dz, k.r2min)));
          const R rinv = rinv_of(r2);
          const R ri2 = rinv * rinv, ri3 = ri2 * rinv;
          const bool ov = r2 < k.four_a2;
          R A, B;
          if constexpr (MIXED) {  // factored
            const R rho = (r2 - k.r2min) * rinv * k.i2a;
            const R om = (R)1 - rho, op = (R)1 + rho, wt = om * om * ri3;
            A = ov ? -k.a3 * wt * fma(fma((R)9, rho, (R)2), rho, (R)1) : (R)0;
            B = ov ? k.a2 * wt * (op * op) * ri2 : (R)0;
          } else {  // the two branches and their difference (fewer operations)
            const R Af = fma(k.a3, ri3, rinv), Bf = ri3 * fma(-k.a2, ri2, B_ONE<R>);
            const R Ao = fma(-k.ock9, (r2 - k.r2min) * rinv, k.oc), Bo = k.ob * rinv;
            A = ov ? Ao - Af : (R)0;
            B = ov ? Bo - Bf : (R)0;
          }
#pragma unroll
          for (int r = 0; r < NRC; ++r) {
            const R fx = fs[3 * r][s], fy = fs[3 * r + 1][s], fz = fs[3 * r + 2][s];
            const R sdf = B * fma(dx, fx, fma(dy, fy, dz * fz));
            ar[r][0] = fma(A, fx, fma(sdf, dx, ar[r][0]));
            ar[r][1] = fma(A, fy, fma(sdf, dy, ar[r][1]));
            ar[r][2] = fma(A, fz, fma(sdf, dz, ar[r][2]));
          }
        }
      }
      for (int r = 0; r < NRC; ++r)
        for (int c = 0; c < 3; ++c) acc[r][c] += (double)ar[r][c];
    }
  }
  const Sums o(w, tl, 3 * NRC, n, u, part);
  if (valid)
    for (int r = 0; r < NRC; ++r)
      for (int c = 0; c < 3; ++c) {
        double* x = o.at(3 * r + c, threadIdx.x);
        *x = w.slot >= 0 ? c1 * acc[r][c] : *x + c1 * acc[r][c];
      }
}

// Launch arguments shared by the pair kernels: the scale S of the positions (2aS in
// [1, 2)), the constants of the scaled radius in both precisions and the
// prefactors c1 S = S / (8 pi eta) that undo the scaling of the sums (FP64: of S / 2).
struct PairLaunch {
  double S, c1S, c1Sd;
  PairK<float> kf;
  PairK<double> kd;
};

static PairLaunch pair_launch(double a, double eta) {
  PairLaunch q;
  q.S = pair_scale(a);
  q.c1S = q.S / (8.0 * PI * eta);
  q.c1Sd = q.c1S / PAIR_ZOOM<double>;
  q.kf = pair_const<float>(a * q.S);
  q.kd = pair_const<double>(a * q.S / PAIR_ZOOM<double>);
  return q;
}

// A launch's blocks: the parts of NearWork's tables, or one per tile when it
// has none or the caller has no partial-sum slots.
struct NearGrid {
  const int4* item;
  const int* slots;
  int blocks;
  NearGrid(const Tiles& tiles, const NearWork& w, const double* part)
      : item(part ? w.item : nullptr), slots(w.slot), blocks(item ? w.n : tiles.n) {}
};

static hipError_t near_reduce(const Launch& l, const Tiles& tiles, const NearWork& w, const NearGrid& g, int nq,
                              const double* part, double* u, int add) {
  hipError_t he = hipGetLastError();
  if (he != hipSuccess || !g.item) return he;
  k_near_reduce<<<dim3(w.nred, nq), P2P_T, 0, l.s>>>(tiles.t, w.red, w.parts, w.slot0, part, nq, l.B->n, add, u);
  return hipGetLastError();
}

hipError_t run_p2p(const Launch& l, const Tiles& tiles, const NearPlan& np, int nrc, const double* sF, double* u,
                   double* part, int mixed) {
  if (tiles.n == 0) return hipSuccess;
  const Built* B = l.B;
  const PairLaunch q = pair_launch(l.a, l.eta);
  const NearGrid g(tiles, np.u, part);
#define P2P_CASE(NR)                                                                                               \
  case NR:                                                                                                         \
    if (mixed)                                                                                                     \
      k_p2p<NR, true><<<g.blocks, P2P_T, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LU], B->sx, B->sy,    \
                                                   B->sz, sF, B->n, q.kf, q.S, q.c1S, u, part);                    \
    else                                                                                                           \
      k_p2p<NR, false><<<g.blocks, P2P_T, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LU], B->sx, B->sy,   \
                                                    B->sz, sF, B->n, q.kd, q.S, q.c1Sd, u, part);                   \
    break;
  switch (nrc) {
    P2P_CASE(1)
    P2P_CASE(2)
    P2P_CASE(4)
    P2P_CASE(8)
    case MF_R:
      if (mixed)
        k_p2p_mfma<true, 0><<<g.blocks, 64 * MF_W, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LU], B->sx,
                                                             B->sy, B->sz, sF, B->n, q.kf, q.S, q.c1S, u, part);
      else
        k_p2p_mfma<false, 0><<<g.blocks, 64 * MF_W, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LU], B->sx,
                                                              B->sy, B->sz, sF, B->n, q.kd, q.S, q.c1Sd, u, part);
      break;
    // 16 + XR: the FP64 form only
#define MF_CASE(XR)                                                                                                \
  case MF_R + XR:                                                                                                  \
    if (mixed) return hipErrorInvalidValue;                                                                        \
    k_p2p_mfma<false, XR><<<g.blocks, 64 * MF_W, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LU], B->sx,   \
                                                           B->sy, B->sz, sF, B->n, q.kd, q.S, q.c1Sd, u, part);     \
    break;
    MF_CASE(1)
    MF_CASE(2)
    MF_CASE(4)
    MF_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef P2P_CASE
#undef MF_CASE
  return near_reduce(l, tiles, np.u, g, 3 * nrc, part, u, 0);
}

// Blocks of a direct launch: a chip's worth, 16 waves per CU, at most.
constexpr int DIRECT_BLOCKS = 2048;
void plan_direct(const Tiles& tiles, bool alone, bool mixed, NearPlan* np) {
  const int items = np->u.item ? np->u.n : tiles.n;
  np->sub = 0;
  if (!alone || items == 0 || items > DIRECT_BLOCKS) return;
  for (np->sub = mixed ? 1 : 4; np->sub * items > DIRECT_BLOCKS;) np->sub /= 2;
  np->direct = np->sub * items;
}

bool direct_fits(const NearPlan& np, int nrc, const double* part) { return np.sub > 0 && part && nrc <= NEAR_VEC_RHS; }

hipError_t run_direct(const Launch& l, const Tiles& tiles, const NearPlan& np, int nrc, const double* F, double* part,
                      int mixed) {
  const Built* B = l.B;
  const PairLaunch q = pair_launch(l.a, l.eta);
#define DIRECT_CASE(NR)                                                                                              \
  case NR:                                                                                                           \
    if (mixed)                                                                                                       \
      k_p2p<NR, true, true><<<np.direct, P2P_T, 0, l.s>>>(tiles.t, np.u.item, np.u.slot, B->tree, B->lists[LU], B->sx,   \
                                                          B->sy, B->sz, F, B->n, q.kf, q.S, q.c1S, nullptr, part,      \
                                                          B->perm, np.sub);                                            \
    else                                                                                                             \
      k_p2p<NR, false, true><<<np.direct, P2P_T, 0, l.s>>>(tiles.t, np.u.item, np.u.slot, B->tree, B->lists[LU], B->sx,  \
                                                           B->sy, B->sz, F, B->n, q.kd, q.S, q.c1Sd, nullptr, part,     \
                                                           B->perm, np.sub);                                           \
    break;
  switch (nrc) {
    DIRECT_CASE(1)
    DIRECT_CASE(2)
    DIRECT_CASE(4)
    DIRECT_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef DIRECT_CASE
  return hipGetLastError();
}

hipError_t direct_out(const Launch& l, const Tiles& tiles, const NearPlan& np, int nrc, const double* part, double* out) {
  k_direct_out<<<dim3(tiles.n, 3 * nrc), P2P_T * DO_G, 0, l.s>>>(tiles.t, np.u.off, np.u.parts, np.sub, part, 3 * nrc,
                                                                 l.B->n, l.B->perm, out);
  return hipGetLastError();
}

// The overlap correction: FP32 pair arithmetic (the factored differences)
// with FP64 sums per staged chunk in the mixed form, FP64 otherwise.
hipError_t run_overlap(const Launch& l, const Tiles& tiles, const NearPlan& np, int nrc, const double* sF, double* u,
                       double* part, int mixed) {
  const Built* B = l.B;
  if (tiles.n == 0 || B->lists[LO].len == 0 || np.o.nothing) return hipSuccess;
  if (nrc > NEAR_VEC_RHS) {  // launches of 8 right-hand sides, then the rest
    const hipError_t he = run_overlap(l, tiles, np, NEAR_VEC_RHS, sF, u, part, mixed);
    const int64_t off = (int64_t)NEAR_VEC_RHS * 3 * B->n;
    return he != hipSuccess ? he : run_overlap(l, tiles, np, nrc - NEAR_VEC_RHS, sF + off, u + off, part, mixed);
  }
  const PairLaunch q = pair_launch(l.a, l.eta);
  const ChunkFilter f{LO, 0, 4.0 * l.a * l.a};
  const NearGrid g(tiles, np.o, part);
#define OV_CASE(NR)                                                                                                 \
  case NR:                                                                                                          \
    if (mixed)                                                                                                      \
      k_overlap<NR, true><<<g.blocks, P2P_T, 0, l.s>>>(tiles.t, tiles.box, g.item, g.slots, B->tree, B->lists[LO],  \
                                                       f, B->sx, B->sy, B->sz, sF, B->n, q.kf, q.S, q.c1S, u, part); \
    else                                                                                                            \
      k_overlap<NR, false><<<g.blocks, P2P_T, 0, l.s>>>(tiles.t, tiles.box, g.item, g.slots, B->tree, B->lists[LO], \
                                                        f, B->sx, B->sy, B->sz, sF, B->n, q.kd, q.S, q.c1Sd, u, part); \
    break;
  switch (nrc) {
    OV_CASE(1)
    OV_CASE(2)
    OV_CASE(4)
    OV_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef OV_CASE
  return near_reduce(l, tiles, np.o, g, 3 * nrc, part, u, 1);
}

// The direct W sums are far-formula pair sums like the P2P: FP32 in the
// mixed form.
hipError_t run_wdirect(const Launch& l, const Tiles& tiles, const NearPlan& np, int nrc, const double* sF, double* u,
                       double* part, int mixed) {
  const Built* B = l.B;
  if (tiles.n == 0 || B->lists[LW].len == 0 || l.wd < 0 || np.w.nothing) return hipSuccess;
  if (nrc > NEAR_VEC_RHS) {  // launches of 8 right-hand sides, then the rest
    const hipError_t he = run_wdirect(l, tiles, np, NEAR_VEC_RHS, sF, u, part, mixed);
    const int64_t off = (int64_t)NEAR_VEC_RHS * 3 * B->n;
    return he != hipSuccess ? he : run_wdirect(l, tiles, np, nrc - NEAR_VEC_RHS, sF + off, u + off, part, mixed);
  }
  const PairLaunch q = pair_launch(l.a, l.eta);
  const ChunkFilter f{LW, l.wd, 0.0};
  const NearGrid g(tiles, np.w, part);
#define WD_CASE(NR)                                                                                                 \
  case NR:                                                                                                          \
    if (mixed)                                                                                                      \
      k_wdirect<NR, true><<<g.blocks, P2P_T, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LW], f, B->sx,   \
                                                       B->sy, B->sz, sF, B->n, q.kf, q.S, q.c1S, u, part);          \
    else                                                                                                            \
      k_wdirect<NR, false><<<g.blocks, P2P_T, 0, l.s>>>(tiles.t, g.item, g.slots, B->tree, B->lists[LW], f, B->sx,  \
                                                        B->sy, B->sz, sF, B->n, q.kd, q.S, q.c1Sd, u, part);         \
    break;
  switch (nrc) {
    WD_CASE(1)
    WD_CASE(2)
    WD_CASE(4)
    WD_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef WD_CASE
  return near_reduce(l, tiles, np.w, g, 3 * nrc, part, u, 1);
}

// Bytes of the partial-sum slots for near-field groups of nrn right-hand
// sides (0: no tile is split and no direct launch taken).
int64_t near_part_bytes(const NearPlan& np, int nrn) {
  const int64_t vec = std::max(np.w.nslot, np.o.nslot);  // launches of at most NEAR_VEC_RHS
  const int64_t rows = std::max((int64_t)np.u.nslot * nrn,
                                std::max(vec, (int64_t)np.direct) * std::min(nrn, NEAR_VEC_RHS));
  return rows * 3 * P2P_T * (int64_t)sizeof(double);
}

// ------------------------------------------------ sampled direct sums ---
// The exact RPY matvec (Sec. 1, all three blocks) at a few targets, summed
// over every bead of the target's system in FP64: the reference the
// autotuner measures candidate plans against.  One block per sampled
// target (tree order); threads stride over the sources and their partial
// sums are added in a fixed order.  sF is [nrc][3][n] in tree order; out is
// [k][nrc][3].
constexpr int DS_T = 256;
__global__ void __launch_bounds__(DS_T) k_direct_sample(const int* tgt, const int* sys_begin, int nsys,
                                                        const double* sx, const double* sy, const double* sz,
                                                        const double* sF, int64_t n, int nrc, double a, double eta,
                                                        double* out) {
  __shared__ double red[DS_T];
  const int i = tgt[blockIdx.x];
  // the target's system: sys_begin[s] <= i < sys_begin[s + 1] (binary search)
  int lo = 0, hi = nsys;
  while (hi - lo > 1) {
    const int mid = (lo + hi) / 2;
    if (sys_begin[mid] <= i) lo = mid;
    else hi = mid;
  }
  const int sy0 = sys_begin[lo], sy1 = sys_begin[lo + 1];
  const double xi = sx[i], yi = sy[i], zi = sz[i];
  const double c0 = 1.0 / (6.0 * PI * eta * a), c1 = 1.0 / (8.0 * PI * eta), four_a2 = 4.0 * a * a;
  for (int r = 0; r < nrc; ++r) {
    double acc[3] = {0.0, 0.0, 0.0};
    for (int j = sy0 + threadIdx.x; j < sy1; j += DS_T) {
      const double dx = xi - sx[j], dy = yi - sy[j], dz = zi - sz[j];
      const double r2 = dx * dx + dy * dy + dz * dz;
      const double fx = sF[((int64_t)r * 3 + 0) * n + j], fy = sF[((int64_t)r * 3 + 1) * n + j],
                   fz = sF[((int64_t)r * 3 + 2) * n + j];
      double A, B;
      if (r2 == 0.0) {
        A = c0;
        B = 0.0;
      } else if (r2 >= four_a2) {
        const double rr = sqrt(r2), cr = c1 / rr;
        A = cr * (1.0 + 2.0 * a * a / (3.0 * r2));
        B = cr * (1.0 - 2.0 * a * a / r2) / r2;
      } else {
        const double rr = sqrt(r2);
        A = c0 * (1.0 - 9.0 * rr / (32.0 * a));
        B = c0 * (3.0 / (32.0 * a)) / rr;
      }
      const double df = dx * fx + dy * fy + dz * fz;
      acc[0] += A * fx + B * df * dx;
      acc[1] += A * fy + B * df * dy;
      acc[2] += A * fz + B * df * dz;
    }
    for (int c = 0; c < 3; ++c) {
      red[threadIdx.x] = acc[c];
      __syncthreads();
      for (int w = DS_T / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
      }
      if (threadIdx.x == 0) out[((int64_t)blockIdx.x * nrc + r) * 3 + c] = red[0];
      __syncthreads();
    }
  }
}

hipError_t run_direct_sample(const Launch& l, const int* tgt, int k, int nrc, const double* sF, double* out) {
  const Built* B = l.B;
  if (k <= 0) return hipSuccess;
  k_direct_sample<<<k, DS_T, 0, l.s>>>(tgt, B->d_sys_begin, B->nsys, B->sx, B->sy, B->sz, sF, B->n, nrc, l.a,
                                       l.eta, out);
  return hipGetLastError();
}

}  // namespace rpy
