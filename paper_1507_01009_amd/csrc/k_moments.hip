// Monopole and quadrupole moments about each node's centre of mass (the
// multipole expansion of a distant group about its centre of mass).
//
// A leaf sums its particles in sorted order, two passes (mass and first
// moment, then the second moment about the centre of mass) with no
// contraction, so leaf moments equal the plain definition bit for bit.  An
// internal node combines its children with the parallel-axis theorem:
//   M = sum M_c,  com = (sum M_c com_c) / M,
//   S = sum (S_c + M_c d d^T),  d = com_c - com,
// eight lanes to a node, one child each, summed in a fixed tree order.
//
// Two to four launches, whatever the depth.  The particles are cut into
// tiles, and k_moments_tile takes a tile each block: the leaves that start
// in it, then, level by level from the deepest, the internal nodes that lie
// inside it.  At one level at most one node that starts in a tile reaches
// beyond its end.  Those are left to k_moments_span over runs of tiles, a
// block taking the ones inside its run, and what reaches beyond a run to one
// block at the end.  (One launch per level, 21 or 42 of them, cost 4 to 7 us
// each however few nodes a level had: 92 us of leaves and levels at 131072
// stars, 166 at 1M.)
//
// The cell side s = L 2^-level (exact) is stored squared beside the centre
// of mass for the opening-angle test, and as the node's opening size.
//
// Refit (the tree is an earlier build, the particles have moved): the same
// passes also take each node's particle bounding box (exact min / max,
// leaves from their particles, internal nodes from their children) and the
// opening size becomes s' = max(s, 2 e), e the largest distance from the
// cell's geometric centre to the box: the smallest cube about the centre
// that holds the cell and all its particles.
#include "tg_internal.h"

namespace tg {

__global__ void k_mass_gather(const int32_t *__restrict__ gate, const double *__restrict__ mass,
                              const uint32_t *__restrict__ perm, int64_t n,
                              double4 *__restrict__ spart, uint32_t *err) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  bool bad = false;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n;
       r += (int64_t)gridDim.x * blockDim.x) {
    double m = mass[perm[r]];
    bad |= !(m > 0.0) || !isfinite(m);
    spart[r].w = m;
  }
  if (bad) set_err(err, TG_ERR_MASS);
}

// Opening size of node v: the cell side s, or with a refit its refitted
// size from the bounding box [lo, hi] (every operation rounded separately).
__device__ __forceinline__ double open_size(uint32_t v, int l, const uint32_t *first,
                                           const uint32_t *nsys, const uint64_t *skey,
                                           const double *cube, const double lo[3],
                                           const double hi[3], bool refit) {
  double g[3];
  const double s = cell_centre(v, l, first, nsys, skey, cube, g);
  if (!refit) return s;
  double e = 0.0;
  for (int k = 0; k < 3; ++k) e = fmax(fmax(e, dsub(hi[k], g[k])), dsub(g[k], lo[k]));
  return 2.0 * e > s ? 2.0 * e : s;
}

__device__ __forceinline__ void store_moments(uint32_t v, double s, double M, double cx,
                                              double cy, double cz, const double S[6],
                                              double4 *com, double *mom, double *side) {
  com[v] = make_double4(cx, cy, cz, dmul(s, s));
  side[v] = s;
  double *o = mom + 8 * (size_t)v;
  o[0] = M;
  for (int k = 0; k < 6; ++k) o[1 + k] = S[k];
  o[7] = 0.0;
}

struct MomArgs {
  TreeCounters *ctr;
  const double *cube;
  const uint4 *ninfo;            // {first, count, child, nchild}
  const uint32_t *first, *nsys;
  const uint32_t *cnt;           // [levels][tl] nodes of a level before each 256-particle tile
  int64_t tl, ft;                // row length, 256-particle tiles
  int64_t n;
  int levels;
  const double4 *spart;
  const uint64_t *skey;
  const int32_t *refit;
  double4 *com;
  double *mom, *side;
  double4 *bbox;
  uint32_t *err;
};

// One leaf by one thread.  Its first kLeafRegs particles are loaded into
// registers at once, so both passes over them wait for memory once;
// particles beyond (over-full leaves of the deepest level, or leaves of a
// larger leaf size) are read in the passes.  The sums take the particles in
// the same order either way.
constexpr uint32_t kLeafRegs = 8;

template <bool kBox>
__device__ __forceinline__ void leaf_moments(const MomArgs &A, uint32_t v, uint32_t f, uint32_t n,
                                             int lv, bool &bad) {
#pragma clang fp contract(off)
  const double cside = kBox ? 0.0 : A.cube[4 * A.nsys[v] + 3];
  double4 pr[kLeafRegs];
#pragma unroll
  for (uint32_t q = 0; q < kLeafRegs; ++q)
    if (q < n) pr[q] = A.spart[f + q];
  // compensated sums: a leaf may hold any number of coincident particles
  CSum Mc, sxc, syc, szc;
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  auto first_moments = [&](const double4 &p) {
    Mc.add(p.w);
    sxc.add(p.w * p.x);
    syc.add(p.w * p.y);
    szc.add(p.w * p.z);
    if constexpr (kBox) {
      lo[0] = fmin(lo[0], p.x); lo[1] = fmin(lo[1], p.y); lo[2] = fmin(lo[2], p.z);
      hi[0] = fmax(hi[0], p.x); hi[1] = fmax(hi[1], p.y); hi[2] = fmax(hi[2], p.z);
      bad |= !isfinite(p.x) || !isfinite(p.y) || !isfinite(p.z);
    }
  };
#pragma unroll
  for (uint32_t q = 0; q < kLeafRegs; ++q)
    if (q < n) first_moments(pr[q]);
  for (uint32_t j = f + kLeafRegs; j < f + n; ++j) first_moments(A.spart[j]);
  const double M = Mc.get();
  const double cx = sxc.get() / M, cy = syc.get() / M, cz = szc.get() / M;
  CSum Sc[6];
  auto second_moments = [&](const double4 &p) {
    const double dx = p.x - cx, dy = p.y - cy, dz = p.z - cz;
    Sc[0].add(p.w * dx * dx); Sc[1].add(p.w * dy * dy); Sc[2].add(p.w * dz * dz);
    Sc[3].add(p.w * dx * dy); Sc[4].add(p.w * dx * dz); Sc[5].add(p.w * dy * dz);
  };
#pragma unroll
  for (uint32_t q = 0; q < kLeafRegs; ++q)
    if (q < n) second_moments(pr[q]);
  for (uint32_t j = f + kLeafRegs; j < f + n; ++j) second_moments(A.spart[j]);
  double S[6];
  for (int k = 0; k < 6; ++k) S[k] = Sc[k].get();
  double so;
  if constexpr (kBox) {
    A.bbox[2 * (size_t)v] = make_double4(lo[0], lo[1], lo[2], 0.0);
    A.bbox[2 * (size_t)v + 1] = make_double4(hi[0], hi[1], hi[2], 0.0);
    so = open_size(v, lv, A.first, A.nsys, A.skey, A.cube, lo, hi, *A.refit > 0);
  } else {
    so = ldexp(cside, -lv);
  }
  store_moments(v, so, M, cx, cy, cz, S, A.com, A.mom, A.side);
}

// Sum, minimum and maximum over the 8 lanes of an aligned octet, on DPP lane
// moves: neighbours, then pairs, then the two halves (a half's lanes hold
// the same value by then, so its mirror image serves).
template <int kCtrl>
__device__ __forceinline__ double dpp_move(double v) {
  const int2 x = __builtin_bit_cast(int2, v);
  const int2 y = {__builtin_amdgcn_update_dpp(0, x.x, kCtrl, 0xf, 0xf, true),
                  __builtin_amdgcn_update_dpp(0, x.y, kCtrl, 0xf, 0xf, true)};
  return __builtin_bit_cast(double, y);
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141;   // quad_perm 1032, 2301
__device__ __forceinline__ double oct_sum(double v) {
  v += dpp_move<kDppXor1>(v);
  v += dpp_move<kDppXor2>(v);
  return v + dpp_move<kDppHalfMirror>(v);
}
__device__ __forceinline__ double oct_min(double v) {
  v = fmin(v, dpp_move<kDppXor1>(v));
  v = fmin(v, dpp_move<kDppXor2>(v));
  return fmin(v, dpp_move<kDppHalfMirror>(v));
}
__device__ __forceinline__ double oct_max(double v) {
  v = fmax(v, dpp_move<kDppXor1>(v));
  v = fmax(v, dpp_move<kDppXor2>(v));
  return fmax(v, dpp_move<kDppHalfMirror>(v));
}

// One internal node of level l from its nch children from c0 on, by the
// eight lanes of an octet (k: the lane's child); nch = 0: no node.  All
// lanes of the wave are here.
template <bool kBox>
__device__ __forceinline__ void inner_moments(const MomArgs &A, int l, uint32_t v, uint32_t c0,
                                              uint32_t nch, uint32_t k) {
#pragma clang fp contract(off)
  const double cside = (!kBox && nch) ? A.cube[4 * A.nsys[v] + 3] : 0.0;
  const bool mine = k < nch;
  const uint32_t c = mine ? c0 + k : 0u;
  double mc = 0.0, cx_ = 0.0, cy_ = 0.0, cz_ = 0.0;
  double4 cc = make_double4(0.0, 0.0, 0.0, 0.0);
  double o1 = 0.0, o2 = 0.0, o3 = 0.0, o4 = 0.0, o5 = 0.0, o6 = 0.0;
  if (mine) {
    const double *o = A.mom + 8 * (size_t)c;
    cc = A.com[c];
    mc = o[0];
    o1 = o[1]; o2 = o[2]; o3 = o[3]; o4 = o[4]; o5 = o[5]; o6 = o[6];
    cx_ = mc * cc.x; cy_ = mc * cc.y; cz_ = mc * cc.z;
  }
  const double M = oct_sum(mc);
  const double cx = oct_sum(cx_) / M, cy = oct_sum(cy_) / M, cz = oct_sum(cz_) / M;
  const double dx = cc.x - cx, dy = cc.y - cy, dz = cc.z - cz;
  double S[6];
  S[0] = oct_sum(mine ? o1 + mc * dx * dx : 0.0);
  S[1] = oct_sum(mine ? o2 + mc * dy * dy : 0.0);
  S[2] = oct_sum(mine ? o3 + mc * dz * dz : 0.0);
  S[3] = oct_sum(mine ? o4 + mc * dx * dy : 0.0);
  S[4] = oct_sum(mine ? o5 + mc * dx * dz : 0.0);
  S[5] = oct_sum(mine ? o6 + mc * dy * dz : 0.0);
  double lo[3] = {0.0, 0.0, 0.0}, hi[3] = {0.0, 0.0, 0.0};
  if constexpr (kBox) {
    double4 b0 = make_double4(INFINITY, INFINITY, INFINITY, 0.0);
    double4 b1 = make_double4(-INFINITY, -INFINITY, -INFINITY, 0.0);
    if (mine) { b0 = A.bbox[2 * (size_t)c]; b1 = A.bbox[2 * (size_t)c + 1]; }
    lo[0] = oct_min(b0.x); lo[1] = oct_min(b0.y); lo[2] = oct_min(b0.z);
    hi[0] = oct_max(b1.x); hi[1] = oct_max(b1.y); hi[2] = oct_max(b1.z);
  }
  if (nch > 0 && k == 0) {
    double so;
    if constexpr (kBox) {
      A.bbox[2 * (size_t)v] = make_double4(lo[0], lo[1], lo[2], 0.0);
      A.bbox[2 * (size_t)v + 1] = make_double4(hi[0], hi[1], hi[2], 0.0);
      so = open_size(v, l, A.first, A.nsys, A.skey, A.cube, lo, hi, *A.refit > 0);
    } else {
      so = ldexp(cside, -l);
    }
    store_moments(v, so, M, cx, cy, cz, S, A.com, A.mom, A.side);
  }
}

// The level of slot i among ascending level starts: the last one <= i (an
// empty level shares its start with the next).
__device__ __forceinline__ int level_of_slot(const uint32_t *start, int levels, uint32_t i) {
  int lo = 0, hi = levels - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (start[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Tile b: particles [kMT b, kMT (b + 1)).  The nodes that start in it are,
// level by level, runs of ids known from the build's per-tile counts; a slot
// is a place in the concatenation of those runs.  The slots' leaves and the
// internal nodes inside the tile are listed in LDS, in level order; then the
// leaves are summed, a thread each, and the listed nodes level by level.
constexpr int kMT = 512;                  // particles per tile
constexpr int kMTThreads = 256;
constexpr uint32_t kMTList = 1024;        // internal nodes listed (more: read again per level)

template <bool kBox>
__global__ __launch_bounds__(kMTThreads) void k_moments_tile(const int32_t *__restrict__ gate,
                                                             MomArgs A) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  constexpr int kW = kMTThreads / 64;
  __shared__ uint32_t s_a[kLevelsMax + 1], s_start[kLevelsMax + 1], s_inner[kLevelsMax + 1];
  __shared__ uint32_t s_leaf[kMT];        // leaves start at different particles: at most kMT
  __shared__ uint8_t s_leaf_l[kMT];
  __shared__ uint2 s_list[kMTList];       // {node, first child}
  __shared__ uint8_t s_nch[kMTList];
  __shared__ uint32_t s_w[kW][2];
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
  const int64_t b = blockIdx.x;
  const uint32_t t1 = (uint32_t)min(A.n, (b + 1) * (int64_t)kMT);
  const int nl = A.levels;
  if (tid < 64u) {
    uint32_t a = 0, m = 0;
    if ((int)tid < nl) {
      const uint32_t *c = A.cnt + tid * A.tl;
      const int64_t q0 = b * (kMT / 256), q1 = min(A.ft, q0 + kMT / 256);
      a = c[q0];
      m = c[q1] - a;
      a += A.ctr->lvl[tid];
    }
    uint32_t tot;
    const uint32_t st = wave_excl_scan(m, tot);
    if ((int)tid <= nl) { s_a[tid] = a; s_start[tid] = (int)tid < nl ? st : tot; s_inner[tid] = 0u; }
  }
  __syncthreads();
  if (A.ctr->overflow) return;            // no nodes this time
  const uint32_t total = s_start[nl];
  bool bad = false;
  uint32_t n_leaf = 0, n_in = 0;          // the same in every thread
  for (uint32_t i0 = 0; i0 < total; i0 += kMTThreads) {
    const uint32_t i = i0 + tid;
    bool leaf = false, inner = false;
    uint32_t v = 0;
    int l = 0;
    uint4 ni = make_uint4(0u, 0u, 0u, 0u);
    if (i < total) {
      l = level_of_slot(s_start, nl, i);
      v = s_a[l] + (i - s_start[l]);
      ni = A.ninfo[v];
      leaf = ni.w == 0u;
      inner = !leaf && ni.x + ni.y <= t1;
    }
    const unsigned long long lm = __ballot(leaf), im = __ballot(inner);
    if (lane == 0) { s_w[w][0] = (uint32_t)__popcll(lm); s_w[w][1] = (uint32_t)__popcll(im); }
    __syncthreads();
    uint32_t lb = n_leaf, ib = n_in;
    for (int q = 0; q < kW; ++q) {
      const uint32_t x = s_w[q][0], y = s_w[q][1];
      if (q < (int)w) { lb += x; ib += y; }
      n_leaf += x;
      n_in += y;
    }
    if (leaf) {
      const uint32_t at = lb + lanes_below(lm);
      s_leaf[at] = v;
      s_leaf_l[at] = (uint8_t)l;
    }
    if (inner) {
      const uint32_t at = ib + lanes_below(im);
      if (at < kMTList) { s_list[at] = make_uint2(v, ni.z); s_nch[at] = (uint8_t)ni.w; }
      atomicAdd(&s_inner[l], 1u);
    }
    __syncthreads();
  }
  for (uint32_t i = tid; i < n_leaf; i += kMTThreads) {
    const uint32_t v = s_leaf[i];
    const uint4 ni = A.ninfo[v];
    leaf_moments<kBox>(A, v, ni.x, ni.y, (int)s_leaf_l[i], bad);
  }
  if (kBox && bad) set_err(A.err, TG_ERR_NONFINITE);
  const uint32_t k = tid & 7u, oct = tid >> 3;
  constexpr uint32_t kOct = kMTThreads / 8;
  uint32_t end = n_in;                    // listed nodes of levels <= l
  for (int l = nl - 2; l >= 0; --l) {
    const uint32_t m = s_inner[l];
    if (m == 0u) continue;
    __syncthreads();                      // the children are stored
    if (n_in <= kMTList) {
      const uint32_t beg = end - m;
      for (uint32_t j0 = beg; j0 < end; j0 += kOct) {
        const uint32_t j = j0 + oct;
        const bool live = j < end;
        const uint2 e = live ? s_list[j] : make_uint2(0u, 0u);
        inner_moments<kBox>(A, l, e.x, e.y, live ? s_nch[j] : 0u, k);
      }
      end = beg;
    } else {                              // more nodes than listed: all of the level's
      const uint32_t a = s_a[l], e = a + (s_start[l + 1] - s_start[l]);
      for (uint32_t v0 = a; v0 < e; v0 += kOct) {
        const uint32_t v = v0 + oct;
        const uint4 ni = v < e ? A.ninfo[v] : make_uint4(0u, 0u, 0u, 0u);
        inner_moments<kBox>(A, l, v, ni.z, ni.x + ni.y <= t1 ? ni.w : 0u, k);
      }
    }
  }
}

// Internal nodes that reach beyond the unit they start in (unit: `unit`
// particles, a multiple of 256) but not beyond the block's `per` units: at
// each level at most one per unit, the last that starts there.  The
// candidates of every level are looked up first, then taken level by level,
// eight lanes to a node.
constexpr int kSpanMax = 64;              // units per block
constexpr int kSpanThreads = 512;

template <bool kBox>
__global__ __launch_bounds__(kSpanThreads) void k_moments_span(const int32_t *__restrict__ gate,
                                                               MomArgs A, int64_t unit, int per) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  constexpr int kCap = 22 * kSpanMax;     // candidates kept (42 levels: up to 33 units)
  __shared__ uint2 s_cand[kCap];          // {node, first child}
  __shared__ uint8_t s_nch[kCap];
  __shared__ uint32_t s_any[kLevelsMax];
  if (A.ctr->overflow) return;            // no nodes this time
  const uint32_t tid = threadIdx.x;
  const int nl = A.levels - 1;            // the deepest level holds only leaves
  const int64_t units = (A.n + unit - 1) / unit;
  const int64_t u0 = (int64_t)blockIdx.x * per;
  const int nu = (int)min((int64_t)per, units - u0);
  const int64_t end = min(A.n, (u0 + per) * unit);
  // the candidate of level l and unit u0 + q: its children (none: nch = 0)
  auto look = [&](int l, int q, uint32_t &v, uint32_t &c0) -> uint32_t {
    const uint32_t *c = A.cnt + l * A.tl;
    const int64_t b0 = (u0 + q) * (unit / 256), b1 = min(A.ft, b0 + unit / 256);
    const uint32_t e = c[b1];
    if (e == c[b0]) return 0u;
    v = A.ctr->lvl[l] + e - 1u;
    const uint4 ni = A.ninfo[v];
    const int64_t stop = (int64_t)ni.x + ni.y;
    c0 = ni.z;
    return stop > min(A.n, (u0 + q + 1) * unit) && stop <= end ? ni.w : 0u;
  };
  const bool kept = nl * nu <= kCap;
  for (int i = (int)tid; i < nl; i += (int)blockDim.x) s_any[i] = kept ? 0u : 1u;
  __syncthreads();
  if (kept)
    for (int i = (int)tid; i < nl * nu; i += (int)blockDim.x) {
      uint32_t v = 0, c0 = 0;
      const uint32_t nch = look(i / nu, i % nu, v, c0);
      s_cand[i] = make_uint2(v, c0);
      s_nch[i] = (uint8_t)nch;
      if (nch) s_any[i / nu] = 1u;
    }
  __syncthreads();
  const uint32_t k = tid & 7u;
  const int oct = (int)(tid >> 3), n_oct = (int)(blockDim.x >> 3);
  for (int l = nl - 1; l >= 0; --l) {
    if (s_any[l] == 0u) continue;
    for (int q0 = 0; q0 < nu; q0 += n_oct) {
      const int q = q0 + oct;
      uint32_t v = 0, c0 = 0, nch = 0;
      if (q < nu) {
        if (kept) {
          v = s_cand[l * nu + q].x;
          c0 = s_cand[l * nu + q].y;
          nch = s_nch[l * nu + q];
        } else {
          nch = look(l, q, v, c0);
        }
      }
      if (__ballot(nch > 0u) != 0ull) inner_moments<kBox>(A, l, v, c0, nch, k);
    }
    __syncthreads();                      // stored before the level above reads
  }
}

template <bool kBox>
static void launch_moment_passes(tg_ctx *c) {
  Buffers &b = c->b;
  MomArgs A;
  A.ctr = b.ctr; A.cube = b.cube; A.ninfo = b.ninfo;
  A.first = b.first; A.nsys = b.nsys;
  A.cnt = b.fl_cnt; A.tl = c->flat_tiles + 1; A.ft = (c->n + 255) / 256;
  A.n = c->n; A.levels = c->max_level + 1;
  A.spart = b.spart; A.skey = b.key[0]; A.refit = b.refit_flag;
  A.com = b.com; A.mom = b.mom; A.side = b.side; A.bbox = b.bbox; A.err = b.err;
  const int64_t tiles = (c->n + kMT - 1) / kMT;
  hipLaunchKernelGGL(k_moments_tile<kBox>, dim3((unsigned)tiles), dim3(kMTThreads), 0, c->stream,
                     c->gate, A);
  // up to kSpanMax units end in one block, more are taken 32 to a block (a
  // wave per SIMD; with 128 a level's FP64 work on one CU took 2.4 us)
  int64_t unit = kMT, units = tiles;
  while (units > 1) {
    const int per = units <= kSpanMax ? (int)units : 32;
    const int64_t runs = (units + per - 1) / per;
    const int threads = (8 * per + 63) / 64 * 64;
    hipLaunchKernelGGL(k_moments_span<kBox>, dim3((unsigned)runs), dim3(threads), 0, c->stream,
                       c->gate, A, unit, per);
    unit *= per;
    units = runs;
  }
}

hipError_t launch_moments(tg_ctx *c, const double *mass, bool gathered, bool refit) {
  Buffers &b = c->b;
  if (c->n == 0) return hipSuccess;
  int g = (int)std::min<int64_t>((c->n + 255) / 256, 4096);
  if (!gathered)        // else the build's gather brought the masses already
    hipLaunchKernelGGL(k_mass_gather, dim3(g), dim3(256), 0, c->stream, c->gate, mass,
                       b.val[0], c->n, b.spart, b.err);
  if (refit)
    launch_moment_passes<true>(c);
  else
    launch_moment_passes<false>(c);
  return hipGetLastError();
}

}  // namespace tg
