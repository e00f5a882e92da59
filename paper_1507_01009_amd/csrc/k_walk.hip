// Active groups, the group tree walk with the opening-angle
// test, and the softened P2P / quadrupole P2M force sums.
//
// One 64-lane wavefront owns one group of targets at a time, or one part of a
// group's sources where there are few groups (persistent grid, items taken
// from per-XCD queues).  The walk is breadth first: the
// frontier holds the cells opened on the level above as ranges of
// consecutive children, and the wave tests the children of eight of them at
// once (eight lanes each) against the group's box,
//   accept iff side^2 < theta^2 d^2,  d = box-to-centre-of-mass distance,
// evaluated in double precision with no contraction (bit-identical decisions
// to the plain definition).  A second mode replaces it by the relative
// test (G M s^2 / d^4 <= alpha min|a_old|, group box outside the cell cube
// enlarged by 20 %; the paper's "Gadget" criterion, Sec. 3, run set-up, in
// the form of Springel 2005, Sec. 3.1).  Ballot + mbcnt compaction appends accepted
// cells to an LDS P2M list and the particles of refused leaves to an LDS
// P2P queue; a refused internal cell goes onto the next frontier as one
// {first child, child count} record.  Whenever a list holds a full tile it
// is flushed: the sources are staged in LDS once and each lane sums one
// slice of them (every slices-th entry) onto the T (1..3) targets it holds,
// on the vector ALUs.  No MFMA: a P2M pair is a chain of dependent scalar
// operations around one rsqrt, and the bilinear parts that could be cast as
// products have an N dimension of 1-9, which FP32 MFMA (twice the unpacked
// VALU rate) would mostly pad.
//
// Precision modes.  FP64: all sums in double, rsqrt from the hardware
// estimate plus one third-order correction (Householder).  MIXED: the walk
// decisions stay double; targets and sources are taken relative to the
// group's box centre c_g in double and rounded to float, the interaction
// arithmetic is float with the hardware rsqrt, and each tile's float
// partial sums (at most 128 sources per lane slice) are added into per-target
// double accumulators (one conversion and one FP64 add, both full rate).
//
// Flops per interaction as written in p2p_term / p2m_term (FMA = 2; the
// rsqrt and, in FP64, its refinement are not counted):
//   P2P 19: 3 sub, 6 for r^2 + eps^2, 3 for m D1 and m D3, 6 for the three
//          accelerations, 1 for the potential.
//   P2M 54: 3 sub, 6 for r^2 + eps^2, 3 for D2..D5, 15 for Q x, 6 for W,
//          2 for D4 W, 3 for the radial coefficient, 12 for the
//          accelerations, 4 for the potential (Q = 3S - T I, -T eps^2 and M
//          of every node are formed once per evaluation, cell_records).
#include <type_traits>

#include "tg_internal.h"

namespace tg {

// Most targets a lane holds (the per-group choice is 1..this), and the
// occupancy the kernel is compiled for, per precision mode.
#ifndef TG_WALK_MAXT_MIXED
#define TG_WALK_MAXT_MIXED 3
#endif
#ifndef TG_WALK_MAXT_MIXED_SPLINE
#define TG_WALK_MAXT_MIXED_SPLINE 2        // the spline terms need more registers
#endif
#ifndef TG_WALK_MAXT_FP64
#define TG_WALK_MAXT_FP64 3
#endif
#ifndef TG_WALK_WAVES_MIXED
#define TG_WALK_WAVES_MIXED 4
#endif
#ifndef TG_WALK_WAVES_FP64
#define TG_WALK_WAVES_FP64 2
#endif

constexpr uint32_t kAllParts = 1u << 31;    // of an item: all parts, by one wave

constexpr int kTile = 128;                  // source tile entries (a flush uses <= 128)
constexpr int kMCap = 128 + 64;             // P2M cell list (LDS): < one flush + one append
constexpr int kQCap = 128 + 64 * 8;         // P2P particle queue (LDS); overflow goes leaf by leaf

struct WalkArgs {
  const uint4 *ninfo;       // {first, count, child, nchild} per node
  const double4 *com;
  const double4 *rel;       // relative test: per node {lo, P}, {hi, 0} (enlarged cube)
  const double *arel;       // relative test: per group (alpha alpha) min |a_old|^2
  const void *cell;         // walk records per node (float4[2] mixed, double4[2] FP64)
  const double4 *spart;
  const uint32_t *root_of;
  const uint4 *groups;
  const uint32_t *alist;
  const double *abox;
  const uint8_t *sact;        // active flag per sorted particle (null: all active)
  const uint32_t *perm;
  TreeCounters *ctr;
  unsigned long long *wtot;   // force walk: per workgroup {P2P, P2M, targets, groups}
  const uint2 *items;         // force walk: {group, part | (parts - 1) << 5 | first slot << 10 | all}
  uint32_t item_gap;          // extra entries of each queue's range of items
  const uint2 *slots;         // split groups: {group, parts} at the slot of part 0
  double4 *wpart;             // partial results of split groups [slot][kMaxGroup]
  uint32_t starts;            // blocks that start with an item of their own
  uint32_t *err;
  uint32_t *frontier;
  int fcap;
  double th2, eps2, G;
  double *acc, *pot;
  // external point masses (SMBHs) of each system, added in FP64 per target
  const double *ext_pos, *ext_mass, *ext_eps;
  const int32_t *ext_seg;   // [S+1]: externals of system s
  double eps;
  // list mode
  uint32_t *wl_count;
  const uint32_t *wl_off;
  uint32_t *ids;
};

// ---------------------------------------------------------------- helpers
// LDS written by some lanes of a wave, read by others of the same wave: a
// wave's LDS accesses execute in order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Squared distance from the group box to the centre of mass, the same
// operations in the same order as the plain definition: d^2 = sum_k
// max(max(lo_k - c_k, c_k - hi_k), 0)^2.  fmax (one v_max_f64) equals the
// compare-and-select of the definition for the finite inputs the build
// guarantees.
__device__ __forceinline__ double box_d2(const double lo[3], const double hi[3], double4 c) {
#pragma clang fp contract(off)
  double d2 = 0.0;
  {
    double a = dsub(lo[0], c.x), b = dsub(c.x, hi[0]);
    const double m = fmax(fmax(a, b), 0.0);
    d2 = dadd(d2, dmul(m, m));
  }
  {
    double a = dsub(lo[1], c.y), b = dsub(c.y, hi[1]);
    const double m = fmax(fmax(a, b), 0.0);
    d2 = dadd(d2, dmul(m, m));
  }
  {
    double a = dsub(lo[2], c.z), b = dsub(c.z, hi[2]);
    const double m = fmax(fmax(a, b), 0.0);
    d2 = dadd(d2, dmul(m, m));
  }
  return d2;
}

// Opening-angle test: accept iff side^2 < theta^2 d^2 (c.w = side^2).
__device__ __forceinline__ bool mac_accept(const double lo[3], const double hi[3],
                                           double4 c, double th2) {
  return c.w < dmul(th2, box_d2(lo, hi, c));
}

// Relative test: accept iff P P <= A (d^2 d^2)(d^2 d^2), P = (G M) s^2,
// A = (alpha alpha) min |a_old|^2 of the group, and the box misses the
// enlarged cube [r0.xyz, r1.xyz] on some axis (touching counts as a hit).
__device__ __forceinline__ bool mac_rel(const double lo[3], const double hi[3], double4 c,
                                        double4 r0, double4 r1, double A) {
  const double d2 = box_d2(lo, hi, c);
  const double d4 = dmul(d2, d2);
  const bool near = dmul(r0.w, r0.w) <= dmul(A, dmul(d4, d4));
  const bool apart = lo[0] > r1.x || hi[0] < r0.x || lo[1] > r1.y || hi[1] < r0.y ||
                     lo[2] > r1.z || hi[2] < r0.z;
  return near && apart;
}

// ---------------------------------------------------------------- terms
template <class R> struct Vec4;
template <> struct Vec4<float> { using T = float4; };
template <> struct Vec4<double> { using T = double4; };

__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq(double x) { return rsqrt_dp(x); }

// Softened quadrupole term of one cell on one target, x = target - com.
// Cell: a = {com, M}, b = {Qxx, Qyy, Qzz, -T eps^2}, c = {Qxy, Qxz, Qyz, -}
// with the traceless Q = 3S - T I, T = tr S.  With r^2 = |x|^2 + eps^2 and
// D_n = r^-n, the expansion of the softened potential about the centre of
// mass gives
//   W = x.Q.x - T eps^2      (= 3 x.S.x - T r^2)
//   a += -(M D3 + 2.5 D7 W) x + D5 Q x
//   phi -= M D1 + 0.5 D5 W
// (the same as -(M D3 + T D5 + 2.5 D7 W) x + 3 D5 S x, with T x folded
// into Q x).
template <class R>
__device__ __forceinline__ void p2m_term(typename Vec4<R>::T a, typename Vec4<R>::T b,
                                         typename Vec4<R>::T c, R tx, R ty, R tz, R e2,
                                         R &ax, R &ay, R &az, R &ph) {
  const R x = tx - a.x, y = ty - a.y, z = tz - a.z;
  const R r2 = fma(z, z, fma(y, y, fma(x, x, e2)));
  const R D1 = rsq(r2);
  const R u = D1 * D1, D3 = D1 * u, D5 = D3 * u;
  const R Qx = fma(c.y, z, fma(c.x, y, b.x * x));
  const R Qy = fma(c.z, z, fma(b.y, y, c.x * x));
  const R Qz = fma(b.z, z, fma(c.z, y, c.y * x));
  const R W = fma(z, Qz, fma(y, Qy, fma(x, Qx, b.w)));
  const R k = (u * W) * u;                     // D4 W
  const R C = D3 * fma(R(2.5), k, a.w);        // M D3 + 2.5 D7 W
  ax = fma(D5, Qx, fma(-C, x, ax));
  ay = fma(D5, Qy, fma(-C, y, ay));
  az = fma(D5, Qz, fma(-C, z, az));
  ph = fma(-D1, fma(R(0.5), k, a.w), ph);      // M D1 + 0.5 D5 W
}

// Softened particle term, source s = {position, m}; keep = false drops the
// pair (a target and itself).
template <class R>
__device__ __forceinline__ void p2p_term(typename Vec4<R>::T s, R tx, R ty, R tz, R e2,
                                         R &ax, R &ay, R &az, R &ph, bool keep = true) {
  const R dx = tx - s.x, dy = ty - s.y, dz = tz - s.z;
  const R r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, e2)));
  const R D1 = keep ? rsq(r2) : R(0);
  const R mD1 = s.w * D1;
  const R mD3 = mD1 * (D1 * D1);
  ax = fma(-mD3, dx, ax);
  ay = fma(-mD3, dy, ay);
  az = fma(-mD3, dz, az);
  ph -= mD1;
}

// Cubic-spline softening (Monaghan-Lattanzio kernel, support 2h, h = eps):
// with u = r/h, psi is the pair's softened 1/r and psi_k+1 = -(1/r) d psi_k
// / dr; beyond 2h they are 1/r, 1/r^3, 3/r^5, 15/r^7.  The Newtonian values
// come from one rsqrt; the polynomial pieces are evaluated only where some
// lane of the wave has a pair inside 2h.  At r = 0 (a particle and itself,
// coincident ones, or a zero-mass tile pad at the target) u = 0 selects the
// inner piece, which is finite; psi_3 (1/u there) is set to 0, since it
// multiplies x.S.x = 0.
template <class R>
__device__ __forceinline__ void spline_psi01(R r2, R h, R ih, R &p0, R &p1) {
  const R ir = rsq(r2);
  p0 = ir;
  p1 = ir * ir * ir;
  const R u = (r2 > R(0) ? r2 * ir : R(0)) * ih;
  if (u < R(2)) {
    const R u2 = u * u, ih3 = ih * ih * ih, iu = h * ir;
    const R a0 = ih * fma(u2, fma(u2, fma(R(-0.1), u, R(0.3)), R(-2.0 / 3.0)), R(1.4));
    const R a1 = ih3 * fma(u2, fma(R(0.5), u, R(-1.2)), R(4.0 / 3.0));
    const R b0 = ih * fma(R(-1.0 / 15.0), iu,
                          fma(u2, fma(u, fma(u, fma(u, R(1.0 / 30.0), R(-0.3)), R(1)),
                                      R(-4.0 / 3.0)), R(1.6)));
    const R b1 = ih3 * fma(R(-1.0 / 15.0), iu * iu * iu,
                           fma(u, fma(u, fma(u, R(-1.0 / 6.0), R(1.2)), R(-3)), R(8.0 / 3.0)));
    const bool in = u < R(1);
    p0 = in ? a0 : b0;
    p1 = in ? a1 : b1;
  }
}

template <class R>
__device__ __forceinline__ void spline_psi0123(R r2, R h, R ih, R &p0, R &p1, R &p2, R &p3) {
  const R ir = rsq(r2), ir2 = ir * ir;
  p0 = ir;
  p1 = ir * ir2;
  p2 = R(3) * p1 * ir2;
  p3 = R(5) * p2 * ir2;
  const R u = (r2 > R(0) ? r2 * ir : R(0)) * ih;
  if (u < R(2)) {
    const R u2 = u * u, ih2 = ih * ih, ih3 = ih2 * ih, ih5 = ih3 * ih2, ih7 = ih5 * ih2;
    const R iu = h * ir, iu2 = iu * iu, iu3 = iu2 * iu, iu5 = iu3 * iu2;
    const R a0 = ih * fma(u2, fma(u2, fma(R(-0.1), u, R(0.3)), R(-2.0 / 3.0)), R(1.4));
    const R a1 = ih3 * fma(u2, fma(R(0.5), u, R(-1.2)), R(4.0 / 3.0));
    const R a2 = ih5 * fma(R(-1.5), u, R(2.4));
    const R a3 = r2 > R(0) ? ih7 * (R(1.5) * iu) : R(0);   // multiplies V = 0 at r = 0
    const R b0 = ih * fma(R(-1.0 / 15.0), iu,
                          fma(u2, fma(u, fma(u, fma(u, R(1.0 / 30.0), R(-0.3)), R(1)),
                                      R(-4.0 / 3.0)), R(1.6)));
    const R b1 = ih3 * fma(R(-1.0 / 15.0), iu3,
                           fma(u, fma(u, fma(u, R(-1.0 / 6.0), R(1.2)), R(-3)), R(8.0 / 3.0)));
    const R b2 = ih5 * fma(R(-0.2), iu5, fma(R(3), iu, fma(R(0.5), u, R(-2.4))));
    const R b3 = ih7 * fma(R(-1), iu5 * iu2, fma(R(3), iu3, R(-0.5) * iu));
    const bool in = u < R(1);
    p0 = in ? a0 : b0;
    p1 = in ? a1 : b1;
    p2 = in ? a2 : b2;
    p3 = in ? a3 : b3;
  }
}

// Spline-softened cell term, x = target - com, cell as for p2m_term but
// b.w = T.  The second-order expansion of the kernel about the centre of
// mass, with V = x.Q.x + T |x|^2 (= 3 x.S.x):
//   a  += -(M psi_1 - 5/6 psi_2 T + psi_3 V / 6) x + (psi_2 / 3) Q x
//   phi -= M psi + psi_2 V / 6 - psi_1 T / 2
template <class R>
__device__ __forceinline__ void p2m_spline(typename Vec4<R>::T a, typename Vec4<R>::T b,
                                           typename Vec4<R>::T c, R tx, R ty, R tz, R h, R ih,
                                           R &ax, R &ay, R &az, R &ph) {
  const R x = tx - a.x, y = ty - a.y, z = tz - a.z;
  const R r2 = fma(z, z, fma(y, y, x * x));
  R p0, p1, p2, p3;
  spline_psi0123<R>(r2, h, ih, p0, p1, p2, p3);
  const R Qx = fma(c.y, z, fma(c.x, y, b.x * x));
  const R Qy = fma(c.z, z, fma(b.y, y, c.x * x));
  const R Qz = fma(b.z, z, fma(c.z, y, c.y * x));
  const R V = fma(b.w, r2, fma(z, Qz, fma(y, Qy, x * Qx)));
  const R V6 = V * R(1.0 / 6.0);
  const R C = fma(p3, V6, fma(R(-5.0 / 6.0) * p2, b.w, a.w * p1));
  const R q = p2 * R(1.0 / 3.0);
  ax = fma(q, Qx, fma(-C, x, ax));
  ay = fma(q, Qy, fma(-C, y, ay));
  az = fma(q, Qz, fma(-C, z, az));
  ph -= fma(p2, V6, fma(R(-0.5) * p1, b.w, a.w * p0));
}

// Spline-softened particle term, source s = {position, m}; keep = false
// drops the pair (a target and itself: x = 0, only the potential term).
template <class R>
__device__ __forceinline__ void p2p_spline(typename Vec4<R>::T s, R tx, R ty, R tz, R h, R ih,
                                           R &ax, R &ay, R &az, R &ph, bool keep = true) {
  const R dx = tx - s.x, dy = ty - s.y, dz = tz - s.z;
  const R r2 = fma(dz, dz, fma(dy, dy, dx * dx));
  R p0, p1;
  spline_psi01<R>(r2, h, ih, p0, p1);
  const R mp1 = s.w * p1;
  ax = fma(-mp1, dx, ax);
  ay = fma(-mp1, dy, ay);
  az = fma(-mp1, dz, az);
  ph -= keep ? s.w * p0 : R(0);
}

// ---------------------------------------------------------------- tiles
struct P2MTileD { double4 a, b, c; };
struct P2MTileF { float4 a, b, c; };

// Targets per lane: a group of nt targets is spread over the 64 lanes as
// lt = ceil(nt / T) lane-targets (each lane holding up to T targets) times
// slices = floor(64 / lt) source slices; T is chosen per group to minimise
// the evaluations per source, T / slices.
template <bool kMixed, bool kSpline> struct Shape {
  static constexpr int kMaxT =
      kMixed ? (kSpline ? TG_WALK_MAXT_MIXED_SPLINE : TG_WALK_MAXT_MIXED) : TG_WALK_MAXT_FP64;
  static_assert(kMaxT >= 1 && kMaxT <= 3, "1..3 targets per lane");
};
template <bool kMixed>
constexpr int kRedT = Shape<kMixed, false>::kMaxT > Shape<kMixed, true>::kMaxT
                          ? Shape<kMixed, false>::kMaxT : Shape<kMixed, true>::kMaxT;

// Source tiles in LDS.  A flush of k sources fills entries [0, slices *
// trips) with trips = ceil(k / slices), the entries past k with zero mass;
// slice s evaluates the entries s, s + slices, s + 2 slices, ... (trips of
// them), so every lane runs the same trip count with no masking, and the
// slices of one trip read neighbouring entries (interleaving them measured
// 0.8% faster than contiguous runs per slice).  Full flushes take exactly
// slices * floor(128 / slices) (65..128) sources, so the fixed cost of a
// flush (two barriers, the staging set-up, the FP64 accumulation) is shared
// by as many sources as the tile holds.  `red` holds the per-lane sums of
// the final slice reduction.
template <bool kMixed> union TileMem;
template <> union __align__(16) TileMem<true> {
  P2MTileF m[kTile];
  float4 p[kTile];
  double red[kRedT<true> * 256];
};
template <> union __align__(16) TileMem<false> {
  P2MTileD m[kTile];
  double4 p[kTile];
  double red[kRedT<false> * 256];
};

// ------------------------------------------- one wave's tiles and targets
// (kWhole only keeps the functions of that form's kernels apart from the
// others', whose inlining they would change)
template <bool kMixed, bool kSpline, bool kWhole>
struct Eval {
  using R = typename std::conditional<kMixed, float, double>::type;
  using R4 = typename Vec4<R>::T;
  static constexpr int kMaxT = Shape<kMixed, kSpline>::kMaxT;
  TileMem<kMixed> *tile;
  int T, lt, slices, tfull, F, my_s;
  double cgx, cgy, cgz;              // coordinate origin of the group (0 in FP64)
  R e2;
  R h, ih;                           // spline softening length and its inverse
  R tx[kMaxT], ty[kMaxT], tz[kMaxT];
  const uint32_t *s_tgt;             // sorted indices of the nt targets (LDS)
  int nt;
  // The group's own particles [g0, g0 + gn) met in refused leaves are not
  // queued: bit b of own (own0 | own1 << 64) marks particle g0 + b, and
  // they are evaluated last, each target without its own pair.
  uint32_t g0, gn;
  unsigned long long own0, own1;     // wave-uniform
  // per-target totals in FP64 (mixed: each tile's FP32 partial sums are
  // added here, so rounding accumulates only within a tile)
  double hax[kMaxT], hay[kMaxT], haz[kMaxT], hph[kMaxT];

  // The lane shape and targets of a group (box lo, hi) whose active targets
  // are listed in tgt[0, n): T targets per lane (at least ceil(n / 64)), lt
  // lane-targets, slices source slices; minimise T / slices.  Ties go to the
  // larger T (fewer tile reads per pair), except that in mixed precision
  // three targets to a lane are taken only where they evaluate strictly
  // fewer pairs: measured on the 1M cusp, ties between two and three ran
  // slower with three.
  __device__ __forceinline__ void init(const WalkArgs &A, uint4 gr, const double lo[3],
                                       const double hi[3], const uint32_t *tgt, int n) {
    const unsigned lane = lane_id();
    T = (n + 63) / 64;
    lt = (n + T - 1) / T;
    slices = 64 / lt;
#pragma unroll
    for (int t = 2; t <= kMaxT; ++t) {
      if (t <= T) continue;
      const int l2 = (n + t - 1) / t, s2 = 64 / l2;
      const bool better = (kMixed && t >= 3) ? t * slices < T * s2 : t * slices <= T * s2;
      if (better) { T = t; lt = l2; slices = s2; }
    }
    g0 = gr.x; gn = gr.y; own0 = own1 = 0ull;
    s_tgt = tgt; nt = n;
    tfull = 128 / slices;
    F = slices * tfull;
    const int j = (int)lane % lt;
    const int sl = (int)lane / lt;
    my_s = sl < slices ? sl : 0;             // idle lanes shadow slice 0 (discarded)
    if constexpr (kMixed) {
      cgx = 0.5 * (lo[0] + hi[0]);
      cgy = 0.5 * (lo[1] + hi[1]);
      cgz = 0.5 * (lo[2] + hi[2]);
    } else {
      cgx = cgy = cgz = 0.0;
    }
    e2 = (R)A.eps2;
    h = (R)A.eps;
    ih = (R)(1.0 / A.eps);
#pragma unroll
    for (int k = 0; k < kMaxT; ++k) {
      // lane-target j holds targets j, j + lt, ...; missing ones repeat j
      const int i = j + k * lt;
      const double4 p = A.spart[tgt[i < n ? i : j]];
      tx[k] = (R)(p.x - cgx); ty[k] = (R)(p.y - cgy); tz[k] = (R)(p.z - cgz);
      hax[k] = hay[k] = haz[k] = hph[k] = 0.0;
    }
  }

  __device__ void add(int k, R ax, R ay, R az, R ph) {
    hax[k] += (double)ax; hay[k] += (double)ay; haz[k] += (double)az; hph[k] += (double)ph;
  }

  template <int kT>
  __device__ void eval_m(int base, int trips_in, int st) {
    const int trips = __builtin_amdgcn_readfirstlane(trips_in);
    R ax[kT], ay[kT], az[kT], ph[kT];
#pragma unroll
    for (int k = 0; k < kT; ++k) ax[k] = ay[k] = az[k] = ph[k] = R(0);
    const auto *e = &tile->m[base];
    if constexpr (kSpline) {
      for (int it = 0; it < trips; ++it) {
        const R4 a = e[it * st].a, b = e[it * st].b, c = e[it * st].c;
#pragma unroll
        for (int k = 0; k < kT; ++k)
          p2m_spline<R>(a, b, c, tx[k], ty[k], tz[k], h, ih, ax[k], ay[k], az[k], ph[k]);
      }
    } else if constexpr (kT == 1) {
#pragma unroll 2
      for (int it = 0; it < trips; ++it)
        p2m_term<R>(e[it * st].a, e[it * st].b, e[it * st].c, tx[0], ty[0], tz[0], e2, ax[0], ay[0], az[0], ph[0]);
    } else {
      for (int it = 0; it < trips; ++it) {
        const R4 a = e[it * st].a, b = e[it * st].b, c = e[it * st].c;
#pragma unroll
        for (int k = 0; k < kT; ++k)
          p2m_term<R>(a, b, c, tx[k], ty[k], tz[k], e2, ax[k], ay[k], az[k], ph[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < kT; ++k) add(k, ax[k], ay[k], az[k], ph[k]);
  }

  // kOwn: entry et[k] of the tile is target k itself, its pair dropped
  template <int kT, bool kOwn = false>
  __device__ void eval_p(int base, int trips_in, int st, const uint32_t *et = nullptr) {
    const int trips = __builtin_amdgcn_readfirstlane(trips_in);
    R ax[kT], ay[kT], az[kT], ph[kT];
#pragma unroll
    for (int k = 0; k < kT; ++k) ax[k] = ay[k] = az[k] = ph[k] = R(0);
    const R4 *e = &tile->p[base];
    if constexpr (kOwn) {
      for (int it = 0; it < trips; ++it) {
        const R4 s = e[it * st];
        const uint32_t en = (uint32_t)(base + it * st);
#pragma unroll
        for (int k = 0; k < kT; ++k) {
          if constexpr (kSpline)
            p2p_spline<R>(s, tx[k], ty[k], tz[k], h, ih, ax[k], ay[k], az[k], ph[k], en != et[k]);
          else
            p2p_term<R>(s, tx[k], ty[k], tz[k], e2, ax[k], ay[k], az[k], ph[k], en != et[k]);
        }
      }
    } else if constexpr (kSpline) {
      for (int it = 0; it < trips; ++it) {
        const R4 s = e[it * st];
#pragma unroll
        for (int k = 0; k < kT; ++k)
          p2p_spline<R>(s, tx[k], ty[k], tz[k], h, ih, ax[k], ay[k], az[k], ph[k]);
      }
    } else if constexpr (kT == 1) {
#pragma unroll 4
      for (int it = 0; it < trips; ++it)
        p2p_term<R>(e[it * st], tx[0], ty[0], tz[0], e2, ax[0], ay[0], az[0], ph[0]);
    } else {
#pragma unroll 2
      for (int it = 0; it < trips; ++it) {
        const R4 s = e[it * st];
#pragma unroll
        for (int k = 0; k < kT; ++k)
          p2p_term<R>(s, tx[k], ty[k], tz[k], e2, ax[k], ay[k], az[k], ph[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < kT; ++k) add(k, ax[k], ay[k], az[k], ph[k]);
  }

  __device__ int trips_for(int k) const {
    return k == F ? tfull : (k + slices - 1) / slices;
  }

  // P2M tile entry of cell v, relative to the group origin
  __device__ void stage_cell(const WalkArgs &A, int e, bool live, uint32_t v) {
    if (live) {
      const double4 cm = A.com[v];
      const R4 *r = reinterpret_cast<const R4 *>(A.cell) + 2 * (size_t)v;
      const R4 q0 = r[0], q1 = r[1];
      tile->m[e].a = R4{(R)(cm.x - cgx), (R)(cm.y - cgy), (R)(cm.z - cgz), q1.w};
      tile->m[e].b = q0;
      tile->m[e].c = q1;
    } else {
      tile->m[e].a = tile->m[e].b = tile->m[e].c = R4{R(0), R(0), R(0), R(0)};
    }
  }

  // k cells, lane l holding the ids of entries l and l + 64
  __device__ void tile_p2m(const WalkArgs &A, uint32_t v0, uint32_t v1, int k) {
    const int lane = (int)lane_id();
    const int trips = trips_for(k);
    const int ne = slices * trips;
    const int e0 = lane, e1 = lane + 64;
    if (e0 < ne) stage_cell(A, e0, e0 < k, v0);
    if (e1 < ne) stage_cell(A, e1, e1 < k, v1);
    wave_sync();
    const int base = my_s;
    if (T == 1) eval_m<1>(base, trips, slices);
    else if constexpr (kMaxT >= 2) {
      if (T == 2) eval_m<2>(base, trips, slices);
      else if constexpr (kMaxT >= 3) eval_m<3>(base, trips, slices);
    }
    wave_sync();
  }

  __device__ void flush_p2m(const WalkArgs &A, const uint32_t *list, int k) {
    const int e0 = (int)lane_id(), e1 = e0 + 64;
    tile_p2m(A, e0 < k ? list[e0] : 0u, e1 < k ? list[e1] : 0u, k);
  }

  __device__ void stage_part(const WalkArgs &A, int e, bool live, uint32_t j) {
    R4 v = R4{R(0), R(0), R(0), R(0)};
    if (live) {
      const double4 p = A.spart[j];
      v = R4{(R)(p.x - cgx), (R)(p.y - cgy), (R)(p.z - cgz), (R)p.w};
    }
    tile->p[e] = v;
  }

  // k particles, lane l holding the indices of entries l and l + 64
  __device__ void tile_p2p(const WalkArgs &A, uint32_t j0, uint32_t j1, int k) {
    const int lane = (int)lane_id();
    const int trips = trips_for(k);
    const int ne = slices * trips;
    const int e0 = lane, e1 = lane + 64;
    if (e0 < ne) stage_part(A, e0, e0 < k, j0);
    if (e1 < ne) stage_part(A, e1, e1 < k, j1);
    wave_sync();
    const int base = my_s;
    if (T == 1) eval_p<1>(base, trips, slices);
    else if constexpr (kMaxT >= 2) {
      if (T == 2) eval_p<2>(base, trips, slices);
      else if constexpr (kMaxT >= 3) eval_p<3>(base, trips, slices);
    }
    wave_sync();
  }

  __device__ void flush_p2p(const WalkArgs &A, const uint32_t *list, int k) {
    const int e0 = (int)lane_id(), e1 = e0 + 64;
    tile_p2p(A, e0 < k ? list[e0] : 0u, e1 < k ? list[e1] : 0u, k);
  }

  // rank among the own particles of bit b (b < 128)
  __device__ uint32_t own_rank(uint32_t b) const {
    return b < 64u ? (uint32_t)__popcll(own0 & ((1ull << b) - 1ull))
                   : (uint32_t)__popcll(own0) +
                         (uint32_t)__popcll(own1 & ((1ull << (b - 64u)) - 1ull));
  }

  __device__ bool own_bit(uint32_t b) const {
    return b < 64u ? ((own0 >> b) & 1ull) != 0ull : ((own1 >> (b - 64u)) & 1ull) != 0ull;
  }

  // One tile of the kq queued particles s_q[0, kq) followed by the own
  // particles of ranks [o, o + k) at entries kq + rank - o, each target
  // without itself.
  __device__ void flush_own(const WalkArgs &A, const uint32_t *s_q, int kq, uint32_t o, int k) {
    const uint32_t lane = lane_id();
    const int trips = trips_for(kq + k);
    const int ne = slices * trips;
    for (int e = (int)lane; e < kq; e += 64) stage_part(A, e, true, s_q[e]);
    for (uint32_t b = lane; b < 128u; b += 64u) {
      if (b < gn && own_bit(b)) {
        const int e = (int)(own_rank(b) - o);
        if (e >= 0 && e < k) stage_part(A, kq + e, true, g0 + b);
      }
    }
    for (int e = kq + k + (int)lane; e < ne; e += 64) stage_part(A, e, false, 0u);
    // the lane's targets as placed at the start (missing ones repeat j)
    const int j = (int)lane % lt;
    uint32_t et[kMaxT];
#pragma unroll
    for (int q = 0; q < kMaxT; ++q) {
      const int i = j + q * lt;
      const uint32_t b = s_tgt[i < nt ? i : j] - g0;   // < gn: targets lie in the group
      et[q] = own_bit(b) ? own_rank(b) - o + (uint32_t)kq : 0xffffffffu;
    }
    wave_sync();
    const int base = my_s;
    if (T == 1) eval_p<1, true>(base, trips, slices, et);
    else if constexpr (kMaxT >= 2) {
      if (T == 2) eval_p<2, true>(base, trips, slices, et);
      else if constexpr (kMaxT >= 3) eval_p<3, true>(base, trips, slices, et);
    }
    wave_sync();
  }

  // Marks of the group's own particles in the leaf [f, f + c) of the lanes
  // of `omask` (own part [oa, ob)); rare, one leaf after another.
  __device__ void mark_own(unsigned long long omask, uint32_t oa, uint32_t ob) {
    while (omask) {
      const int L = __ffsll((long long)omask) - 1;
      omask &= omask - 1ull;
      const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)oa, L) - g0;
      const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)ob, L) - g0;
      own0 |= bits_below(b) & ~bits_below(a);                 // b <= gn <= 128
      own1 |= bits_below(b - min(b, 64u)) & ~bits_below(a - min(a, 64u));
    }
  }

  // the lowest n bits (all of them from 64 on)
  __device__ static unsigned long long bits_below(uint32_t n) {
    return n >= 64u ? ~0ull : (1ull << n) - 1ull;
  }

  __device__ uint32_t own_count() const {
    return (uint32_t)(__popcll(own0) + __popcll(own1));
  }

  // per-lane totals -> LDS, [k][lane][4]
  __device__ void store_red() {
    double *red = tile->red;
    const int lane = (int)lane_id();
#pragma unroll
    for (int k = 0; k < kMaxT; ++k) {
      double *o = red + 4 * (64 * k + lane);
      o[0] = hax[k]; o[1] = hay[k]; o[2] = haz[k]; o[3] = hph[k];
    }
  }
};

// ------------------------------------------------------- force-mode sink
// The lists of a group; an item that is one of several parts of a group
// evaluates every parts-th tile.  With kWhole an item may also be a split
// group as a whole (all): its tiles go to the parts' sums in turn, so that
// each sum is the one that the part alone would form.
template <bool kMixed, bool kSpline, bool kWhole>
struct ForceSink : Eval<kMixed, kSpline, kWhole> {
  using E = Eval<kMixed, kSpline, kWhole>;
  using E::F; using E::g0; using E::gn; using E::own0; using E::own1;
  using E::flush_p2m; using E::flush_p2p; using E::flush_own;
  uint32_t *s_m;
  uint32_t *s_q;
  uint32_t nm, nq;
  unsigned long long cells, parts;   // wave-uniform totals
  int turn, parts_;                  // tiles until this item's next one; the group's parts
  bool all;                          // kWhole: turn is the next tile's part
  double (*sum)[E::kMaxT][4];        // kWhole: [part], in an array of its own (scratch memory)

  __device__ bool my_turn() {
    if constexpr (kWhole)
      if (all) return true;
    const bool mine = turn == 0;
    turn = mine ? parts_ - 1 : turn - 1;
    return mine;
  }

  // kWhole: no sums yet; a tile's sums (the only ones in hax ..) to its part's;
  // part p's sums to hax ..
  __device__ void start_parts() {
    for (int p = 0; p < parts_; ++p)
#pragma unroll
      for (int k = 0; k < E::kMaxT; ++k) sum[p][k][0] = sum[p][k][1] = sum[p][k][2] = sum[p][k][3] = 0.0;
  }
  __device__ void tile_done() {
    if constexpr (kWhole) {
      if (!all) return;
#pragma unroll
      for (int k = 0; k < E::kMaxT; ++k) {
        double *o = sum[turn][k];
        o[0] += this->hax[k]; o[1] += this->hay[k]; o[2] += this->haz[k]; o[3] += this->hph[k];
        this->hax[k] = this->hay[k] = this->haz[k] = this->hph[k] = 0.0;
      }
      turn = turn + 1 == parts_ ? 0 : turn + 1;
    }
  }
  __device__ void take_part(int p) {
#pragma unroll
    for (int k = 0; k < E::kMaxT; ++k) {
      const double *o = sum[p][k];
      this->hax[k] = o[0]; this->hay[k] = o[1]; this->haz[k] = o[2]; this->hph[k] = o[3];
    }
  }

  // Queue the particles [lf, lf + lc), flushing whenever a tile is full.
  __device__ void append_run(const WalkArgs &A, uint32_t lf, uint32_t lc) {
    uint32_t o = 0;
    while (o < lc) {
      const uint32_t take = min(lc - o, (uint32_t)kQCap - nq);
      for (uint32_t j = lane_id(); j < take; j += 64u) s_q[nq + j] = lf + o + j;
      nq += take;
      o += take;
      wave_sync();
      drain_q(A);
    }
  }

  __device__ void p2m(const WalkArgs &A, bool pred, uint32_t node) {
    const unsigned long long mask = __ballot(pred);
    if (mask == 0ull) return;
    if (pred) s_m[nm + lanes_below(mask)] = node;
    const uint32_t c = (uint32_t)__popcll(mask);
    nm += c;
    cells += c;
    wave_sync();
    if (nm >= (uint32_t)F) {          // nm < F + 64 <= 2 F: one flush
      if (my_turn()) { flush_p2m(A, s_m + (nm - F), F); tile_done(); }
      nm -= F;
    }
  }

  __device__ void drain_q(const WalkArgs &A) {
    while (nq >= (uint32_t)F) {
      if (my_turn()) { flush_p2p(A, s_q + (nq - F), F); tile_done(); }
      nq -= F;
    }
  }

  // pred: this lane's leaf is refused; c = its particle count (0 if not
  // pred), pre / tot = exclusive prefix and wave total of c
  __device__ void p2p(const WalkArgs &A, bool pred, uint32_t node, uint32_t f,
                      uint32_t c, uint32_t pre, uint32_t tot) {
    (void)node;
    const unsigned long long mask = __ballot(pred);
    if (mask == 0ull) return;
    parts += tot;
    // the leaf minus the group's own particles: [f, oa) and [ob, f + c)
    uint32_t oa = f + c, ob = f + c;
    if (pred) {
      oa = min(max(f, g0), f + c);
      ob = min(max(f, g0 + gn), f + c);
    }
    const unsigned long long omask = __ballot(ob > oa);
    if (omask != 0ull) {
      // rare (the group's own leaves): mark them, queue the rest
      this->mark_own(omask, oa, ob);
      pre = wave_excl_scan(c - (ob - oa), tot);
    }
    const uint32_t left = oa - f, right = f + c - ob;
    if (nq + tot <= (uint32_t)kQCap) {
      for (uint32_t k = 0; k < left; ++k) s_q[nq + pre + k] = f + k;
      for (uint32_t k = 0; k < right; ++k) s_q[nq + pre + left + k] = ob + k;
      nq += tot;
      wave_sync();
      drain_q(A);
      return;
    }
    // rare: many large leaves at once; one run at a time
    unsigned long long m = mask;
    while (m) {
      const int L = __ffsll((long long)m) - 1;
      m &= m - 1ull;
      append_run(A, (uint32_t)__shfl((int)f, L, 64), (uint32_t)__shfl((int)left, L, 64));
      append_run(A, (uint32_t)__shfl((int)ob, L, 64), (uint32_t)__shfl((int)right, L, 64));
    }
  }

  __device__ void finish(const WalkArgs &A) {
    if (nm > 0 && my_turn()) { flush_p2m(A, s_m, (int)nm); tile_done(); }
    nm = 0;
    // the queue's rest (nq < F) and the own particles share the last tiles
    const uint32_t no = this->own_count();
    uint32_t o = 0;
    while (nq + (no - o) > 0u) {
      const uint32_t k = min(no - o, (uint32_t)F - nq);
      if (my_turn()) { flush_own(A, s_q, (int)nq, o, (int)k); tile_done(); }
      nq = 0;
      o += k;
    }
    own0 = own1 = 0ull;
  }
};

// -------------------------------------------------------- list-mode sinks
struct CountSink {
  uint32_t nm = 0, np = 0;
  __device__ void p2m(const WalkArgs &, bool pred, uint32_t) {
    nm += (uint32_t)__popcll(__ballot(pred));
  }
  __device__ void p2p(const WalkArgs &, bool pred, uint32_t, uint32_t, uint32_t, uint32_t,
                      uint32_t) {
    np += (uint32_t)__popcll(__ballot(pred));
  }
  __device__ void finish(const WalkArgs &) {}
};

struct FillSink {
  uint32_t nm = 0, np = 0;
  uint32_t base_m = 0, base_p = 0;
  __device__ void p2m(const WalkArgs &A, bool pred, uint32_t node) {
    const unsigned long long mask = __ballot(pred);
    if (pred) A.ids[base_m + nm + lanes_below(mask)] = node;
    nm += (uint32_t)__popcll(mask);
  }
  __device__ void p2p(const WalkArgs &A, bool pred, uint32_t node, uint32_t, uint32_t,
                      uint32_t, uint32_t) {
    const unsigned long long mask = __ballot(pred);
    if (pred) A.ids[base_p + np + lanes_below(mask)] = node;
    np += (uint32_t)__popcll(mask);
  }
  __device__ void finish(const WalkArgs &) {}
};

// ---------------------------------------------------------- traversal
// Breadth-first walk of the group's system tree.  The frontier holds the
// cells opened on the level above as {first child, child count} (children
// have consecutive ids); a pass takes eight of them, lane 8 j + k testing
// child k of cell j, so an opened cell is pushed with one store and no
// per-child loop.  The walk starts from the range {root, 1}.  Returns false
// if the frontier overflowed (the group's results are then invalid).
// wave: its number in the grid (its part of the frontier's memory).
template <bool kRel, class Sink>
__device__ bool traverse(const WalkArgs &A, Sink &sink, uint32_t wave, uint32_t root,
                         const double lo[3], const double hi[3], double arel) {
  const unsigned lane = lane_id();
  const uint32_t cap = (uint32_t)A.fcap >> 1;     // ranges per half (two words each)
  uint2 *cur = reinterpret_cast<uint2 *>(A.frontier + (size_t)wave * 2 * A.fcap);
  uint2 *nxt = cur + cap;
  if (lane == 0) cur[0] = make_uint2(root, 1u);
  __threadfence_block();
  wave_sync();
  uint32_t fsize = 1;
  const uint32_t kk = lane & 7u;
  while (fsize > 0) {
    uint32_t nf = 0;
    for (uint32_t base = 0; base < fsize; base += 8) {
      // Lanes with no child to test take the first child of their range
      // (lanes past the frontier the first range) and are masked off after
      // the test: the wave runs one path, with no branch around the loads
      // and the test.
      const uint32_t i = base + (lane >> 3);
      const uint2 r = cur[i < fsize ? i : 0u];
      const bool valid = (i < fsize) & (kk < r.y);
      const uint32_t node = r.x + (valid ? kk : 0u);
      const double4 c = A.com[node];
      const uint4 ni = A.ninfo[node];
      const uint32_t f = ni.x, cnt = ni.y, ch = ni.z, nch = ni.w;
      bool acc;
      if constexpr (kRel)
        acc = mac_rel(lo, hi, c, A.rel[2 * (size_t)node], A.rel[2 * (size_t)node + 1], arel);
      else
        acc = mac_accept(lo, hi, c, A.th2);
      acc = acc & valid;
      const bool refused = valid & !acc;
      const bool leaf = refused & (nch == 0u);
      const bool open = refused & (nch > 0u);
      // prefix sum of the particles of refused leaves (most passes have none)
      const uint32_t pc = leaf ? cnt : 0u;
      uint32_t ptot = 0, ppre = 0;
      if (__ballot(leaf) != 0ull) ppre = wave_excl_scan(pc, ptot);
      sink.p2m(A, acc, node);
      sink.p2p(A, leaf, node, f, pc, ppre, ptot);
      const unsigned long long om = __ballot(open);
      const uint32_t no = (uint32_t)__popcll(om);
      if (nf + no > cap) {
        if (lane == 0) set_err(A.err, TG_ERR_FRONTIER);
        return false;
      }
      if (open) nxt[nf + lanes_below(om)] = make_uint2(ch, nch);
      nf += no;
    }
    __threadfence_block();
    wave_sync();
    uint2 *tmp = cur;
    cur = nxt;
    nxt = tmp;
    fsize = nf;
  }
  sink.finish(A);
  return true;
}

// Work distribution aware of the 8 XCDs (each with its own L2): queue q
// holds the contiguous, hence spatially coherent, active groups
// [q G / 8, (q + 1) G / 8); workgroups are dispatched to the XCDs round
// robin, so block b drains queue b mod 8 first and then helps the others.
struct GroupQueue {
  uint32_t q, tried;
  __device__ explicit GroupQueue(uint32_t home) : q(home & 7u), tried(0) {}
  __device__ uint32_t next(TreeCounters *ctr, uint32_t G) {
    while (tried < 8u) {
      const uint32_t lo = (uint32_t)(((uint64_t)q * G) >> 3);
      const uint32_t hi = (uint32_t)(((uint64_t)(q + 1u) * G) >> 3);
      uint32_t g = 0;
      if (lane_id() == 0) g = atomicAdd(&ctr->xq[kQueueStride * q], 1u);
      // every lane is active here: the first lane is lane 0, and the group
      // index (with all that is loaded from it) is known to be uniform
      g = (uint32_t)__builtin_amdgcn_readfirstlane((int)g);
      if (lo + g < hi) return lo + g;
      q = (q + 1u) & 7u;
      ++tried;
    }
    return G;
  }
};

// The force walk's queues: range q of the items starts at q G / 8 plus q
// gaps (G active groups; the gap is room for the parts of split groups) and
// holds n[q] items.  Workgroups are dispatched to the XCDs round robin:
// block b < starts begins with item b / 8 of queue b mod 8, then drains that
// queue through its counter (which counts from the last start) and helps
// the others.  A queue that the starts exhaust is never asked: with few
// items, thousands of waves asking eight counters each had delayed the ones
// with work.
struct ItemQueue {
  uint32_t q, tried;
  bool started;
  __device__ explicit ItemQueue(uint32_t starts)
      : q(blockIdx.x & 7u), tried(0), started(blockIdx.x >= starts) {}
  __device__ bool next(const WalkArgs &A, uint32_t G, uint32_t &at) {
    TreeCounters *ctr = A.ctr;
    while (tried < 8u) {
      const uint32_t n = ctr->q_items[q], starts = (A.starts - q + 7u) >> 3;
      uint32_t i = blockIdx.x >> 3;
      if (started) {
        i = n;
        if (n > starts) {
          if (lane_id() == 0) i = starts + atomicAdd(&ctr->xq[kQueueStride * q], 1u);
          // every lane is active here: the first lane is lane 0, and the item
          // (with all that is loaded from it) is known to be uniform
          i = (uint32_t)__builtin_amdgcn_readfirstlane((int)i);
        }
      }
      started = true;
      if (i < n) {
        at = (uint32_t)(((uint64_t)q * G) >> 3) + q * A.item_gap + i;
        return true;
      }
      if (n <= starts || i >= n) {
        q = (q + 1u) & 7u;
        ++tried;
      }
    }
    return false;
  }
};

// ------------------------------------------------------------ force kernel
// The active targets of a group, compacted into s_tgt in order by one wave.
__device__ __forceinline__ int active_targets(const WalkArgs &A, uint4 gr, uint32_t *s_tgt) {
  const uint32_t lane = lane_id();
  int nt = 0;
  for (uint32_t c0 = 0; c0 < gr.y; c0 += 64u) {
    const bool act = c0 + lane < gr.y && (!A.sact || A.sact[gr.x + c0 + lane]);
    const unsigned long long amask = __ballot(act);
    if (act) s_tgt[nt + lanes_below(amask)] = gr.x + c0 + lane;
    nt += __popcll(amask);
  }
  return nt;
}

// Adds the term of external point mass (SMBH) e on a target at p, in FP64 in
// both precision modes.
template <bool kSpline>
__device__ __forceinline__ void external_term(const WalkArgs &A, double4 p, int32_t e, double &ex,
                                              double &ey, double &ez, double &ep) {
  const double es = fmax(A.eps, A.ext_eps[e]);
  const double dx = p.x - A.ext_pos[3 * e], dy = p.y - A.ext_pos[3 * e + 1],
               dz = p.z - A.ext_pos[3 * e + 2];
  double mD1, mD3;
  if constexpr (kSpline) {
    double p0, p1;
    spline_pair_dp(sqrt(dx * dx + dy * dy + dz * dz), es, p0, p1);
    mD1 = A.ext_mass[e] * p0;
    mD3 = A.ext_mass[e] * p1;
  } else {
    const double r2 = dx * dx + dy * dy + dz * dz + es * es;
    const double D1 = 1.0 / sqrt(r2);
    mD1 = A.ext_mass[e] * D1;
    mD3 = mD1 * D1 * D1;
  }
  ex -= mD3 * dx; ey -= mD3 * dy; ez -= mD3 * dz; ep -= mD1;
}

// The result of sorted target r_t of system sys: the tree's sums (NaN after
// a failed walk) and the external point masses' terms.
template <bool kSpline>
__device__ __forceinline__ void store_target(const WalkArgs &A, uint32_t sys, uint32_t r_t,
                                             double ax, double ay, double az, double ph) {
  const double4 p = A.spart[r_t];
  const uint32_t orig = A.perm[r_t];
  double ex = 0.0, ey = 0.0, ez = 0.0, ep = 0.0;
  if (A.ext_seg)
    for (int32_t e = A.ext_seg[sys]; e < A.ext_seg[sys + 1]; ++e)
      external_term<kSpline>(A, p, e, ex, ey, ez, ep);
  A.acc[3 * (size_t)orig + 0] = A.G * (ax + ex);
  A.acc[3 * (size_t)orig + 1] = A.G * (ay + ey);
  A.acc[3 * (size_t)orig + 2] = A.G * (az + ez);
  if (A.pot) A.pot[orig] = A.G * (ph + ep);
}

// One wave takes one item at a time: a group, or one of the parts of a group
// that was split to give every wave an item of about the same work.
// Each part makes the whole walk and evaluates every parts-th tile, so
// lists, tiles and the sums inside a tile are those of the unsplit group;
// the parts' FP64 totals are added in order by k_walk_finish.
//
// kFormEven (FP64, Plummer): at most two waves on a SIMD.  The kernel needs
// 167 registers, so a SIMD takes three of its waves: of the eight that a CU is
// given three can fall to one SIMD and one to another, and a walk of few groups
// ends with those.  With 169 registers or more they are two to each, so this
// form names a higher one as overwritten.  (Asked for by the attribute, two
// waves at most change the schedule as well, and small walks take up to 20%
// longer.)  A walk in us without and with it: 1000 stars 51 and 51, 24000 245
// and 241, 50000 444 and 376, 65536 554 and 486, 80000 634 and 557, 100000 720
// and 662, 131072 867 and 837, 160000 1024 and 1029.
//
// kFormWhole: for contexts that ask for at most four waves per CU.  Where
// these have several groups each, nothing is gained by parts, and what they
// repeat is lost; but results may not depend on the waves, so one wave walks a
// split group once and keeps the parts' sums apart (in scratch memory, of which
// a tile reads and writes one part's).  A walk in us before groups were split,
// with parts alone and with this, mixed precision: 20000 stars on one wave per
// CU 519, 867 and 537, on two 376, 486 and 374; 50000 on one 1280, 1572 and
// 1302, on four 423, 487 and 440; 100000 on one 2647, 2780 and 2622.
constexpr int kFormFull = 0, kFormEven = 1, kFormWhole = 2;
template <bool kMixed, bool kRel, bool kSpline, int kForm>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kMixed ? TG_WALK_WAVES_MIXED : TG_WALK_WAVES_FP64)))
void k_walk_forces(const int32_t *__restrict__ gate, WalkArgs A) {
  static_assert(kForm != kFormEven || (!kMixed && !kSpline), "the others fill a SIMD evenly");
  if constexpr (kForm == kFormEven) asm volatile("" ::: "v170");
  if (gate && *gate <= 0) return;   // nothing active: skipped
  __shared__ uint32_t s_tgt[kMaxGroup];
  __shared__ uint32_t s_m[kMCap];
  __shared__ uint32_t s_q[kQCap];
  __shared__ TileMem<kMixed> tile;
  using Sink = ForceSink<kMixed, kSpline, kForm == kFormWhole>;
  const unsigned lane = lane_id();
  const uint32_t n_groups = A.ctr->n_active_groups;
  unsigned long long tot_p2p = 0, tot_p2m = 0, tot_t = 0, tot_g = 0;
  ItemQueue Q(A.starts);
  uint32_t at;
  while (Q.next(A, n_groups, at)) {
    const uint2 item = A.items[at];
    const uint32_t g = item.x;
    const uint32_t part = item.y & 31u, parts = ((item.y >> 5) & 31u) + 1u;
    const uint4 gr = A.groups[g];
    double lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) { lo[k] = A.abox[6 * (size_t)g + k]; hi[k] = A.abox[6 * (size_t)g + 3 + k]; }
    const int nt = active_targets(A, gr, s_tgt);
    __syncthreads();
    if (nt == 0) continue;   // cannot happen for a listed group; keeps s_tgt reads defined
    Sink S;
    S.s_m = s_m; S.s_q = s_q; S.tile = &tile;
    S.nm = 0; S.nq = 0; S.cells = 0; S.parts = 0;
    S.turn = (int)part; S.parts_ = (int)parts;
    [[maybe_unused]] double sums[kForm == kFormWhole ? kMaxParts : 1][Sink::E::kMaxT][4];
    if constexpr (kForm == kFormWhole) {
      S.all = (item.y & kAllParts) != 0u;
      S.sum = sums;
      if (S.all) S.start_parts();
    }
    S.init(A, gr, lo, hi, s_tgt, nt);
    const bool ok = traverse<kRel>(A, S, blockIdx.x, A.root_of[gr.w], lo, hi,
                                   kRel ? A.arel[g] : 0.0);
    // rows of kMaxGroup, not of the context's group size: a captured walk is
    // replayed on trees built with another one
    const uint32_t slot0 = (kForm == kFormWhole ? item.y & ~kAllParts : item.y) >> 10;
    double4 *out = A.wpart + (size_t)(slot0 + part) * kMaxGroup;
    const uint32_t rows = kForm == kFormWhole && S.all ? parts : 1u;
    for (uint32_t r = 0; r < rows; ++r, out += kMaxGroup) {
      if constexpr (kForm == kFormWhole) {
        if (S.all) S.take_part((int)r);
        if (r > 0u) __syncthreads();   // the row before has been summed
      }
      S.store_red();
      const double *red = tile.red;
      __syncthreads();
      for (int i = (int)lane; i < nt; i += 64) {
        // target i sits at k = i / lt, lane-target i % lt of every slice; sum
        // the slices in slice order (deterministic)
        const int k = i / S.lt, jj = i % S.lt;
        double ax = 0.0, ay = 0.0, az = 0.0, ph = 0.0;
        for (int q = 0; q < S.slices; ++q) {
          const double *o = red + 4 * (64 * k + q * S.lt + jj);
          ax += o[0]; ay += o[1]; az += o[2]; ph += o[3];
        }
        if (!ok) ax = ay = az = ph = __longlong_as_double(0x7ff8000000000000ll);
        if (parts > 1u) out[i] = make_double4(ax, ay, az, ph);
        else store_target<kSpline>(A, gr.w, s_tgt[i], ax, ay, az, ph);
      }
    }
    if (part == 0u) {
      tot_p2m += S.cells * (unsigned long long)nt;
      tot_p2p += S.parts * (unsigned long long)nt - (unsigned long long)nt;
      tot_t += (unsigned long long)nt;
      tot_g += 1;
    }
    __syncthreads();
  }
  // each workgroup stores its own totals (k_walk_finish adds them up): eight
  // atomics per wave on one line, most of them issued as the queues ran
  // dry, had kept the last waves waiting (the walk took 8% longer)
  if (lane == 0) {
    unsigned long long *w = A.wtot + 4 * (size_t)blockIdx.x;
    w[0] = tot_p2p;
    w[1] = tot_p2m;
    w[2] = tot_t;
    w[3] = tot_g;
  }
}

// After the walk.  Block 0: the counts, the sums of the nb workgroups'
// totals, into the last walk's counts and added to the running ones.  The
// other blocks: the results of the split groups, a wave to a group, its
// parts' totals added in order.
constexpr int kFinishThreads = 256;
constexpr int kFinishBlocks = 1 + 512;

template <bool kSpline>
__global__ __launch_bounds__(kFinishThreads) void k_walk_finish(const int32_t *__restrict__ gate,
                                                                WalkArgs A, int nb) {
  if (gate && *gate <= 0) {         // nothing active: no walk, its counts are zero
    if (blockIdx.x == 0 && threadIdx.x < 4) (&A.ctr->n_p2p)[threadIdx.x] = 0;
    return;
  }
  constexpr int kWaves = kFinishThreads / 64;
  __shared__ unsigned long long part[kWaves][4];
  __shared__ uint32_t s_tgt[kWaves][kMaxGroup];
  const unsigned lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (blockIdx.x > 0) {
    const uint32_t ns = A.ctr->n_slots;
    for (uint32_t s = (blockIdx.x - 1u) * kWaves + w; s < ns; s += (gridDim.x - 1u) * kWaves) {
      const uint2 sl = A.slots[s];
      if (sl.y == 0u) continue;           // a later part
      const uint4 gr = A.groups[sl.x];
      const int nt = active_targets(A, gr, s_tgt[w]);
      wave_sync();
      for (int i = (int)lane; i < nt; i += 64) {
        const double4 *o = A.wpart + (size_t)s * kMaxGroup + i;
        double4 v = o[0];
        for (uint32_t k = 1; k < sl.y; ++k) {
          const double4 u = o[(size_t)k * kMaxGroup];
          v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
        }
        store_target<kSpline>(A, gr.w, s_tgt[w][i], v.x, v.y, v.z, v.w);
      }
      wave_sync();
    }
    return;
  }
  unsigned long long v[4] = {0, 0, 0, 0};
#pragma unroll 4
  for (int b = threadIdx.x; b < nb; b += kFinishThreads)
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] += A.wtot[4 * (size_t)b + k];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v[k] += __shfl_xor(v[k], o, 64);
  if (lane == 0)
#pragma unroll
    for (int k = 0; k < 4; ++k) part[w][k] = v[k];
  __syncthreads();
  if (threadIdx.x < 4) {
    const unsigned k = threadIdx.x;
    unsigned long long t = 0;
    for (int q = 0; q < kWaves; ++q) t += part[q][k];
    (&A.ctr->n_p2p)[k] = t;
    (&A.ctr->cum_p2p)[k] += t;
  }
}

// The external point masses' terms of every active target, added to its
// result, where a system has more of them than kExternalsInWalk.  64 targets to
// a block, each wave a quarter of the masses.  In store_target they are one
// chain for each group, 0.28 us a mass, and two of them come one after the
// other: the walk ends with those of its small groups, and k_walk_finish takes
// those of the split ones.  1024 masses on 4096 stars in mixed precision: 715
// us an evaluation, 136 with this kernel (541 before groups were split); on 1M
// stars 10.5 and 5.4 ms.  It costs a launch: 16 masses on 1021 stars 53.4 and
// 54.9 us, 32 57.3 and 55.7.
constexpr int kExternalsInWalk = 16;

template <bool kSpline>
__global__ __launch_bounds__(256) void k_externals(const int32_t *__restrict__ gate, WalkArgs A,
                                                   int64_t n, const int64_t *__restrict__ sysoff,
                                                   int S) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  if (A.ctr->n_active_groups == 0u) return;   // no tree this time: no results either
  constexpr int kW = 4;
  __shared__ double4 s_f[kW - 1][64];
  const unsigned lane = lane_id();
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int64_t r0 = blockIdx.x * (int64_t)64; r0 < n; r0 += gridDim.x * (int64_t)64) {
    const int64_t r = r0 + lane;
    const bool live = r < n && (!A.sact || A.sact[r]);
    double ex = 0.0, ey = 0.0, ez = 0.0, ep = 0.0;
    if (live) {
      const double4 p = A.spart[r];
      int s = 0, hi = S - 1;          // last s with sysoff[s] <= r
      while (s < hi) {
        const int mid = (s + hi + 1) >> 1;
        if (sysoff[mid] <= r) s = mid; else hi = mid - 1;
      }
      for (int32_t e = A.ext_seg[s] + w; e < A.ext_seg[s + 1]; e += kW)
        external_term<kSpline>(A, p, e, ex, ey, ez, ep);
    }
    if (w > 0) s_f[w - 1][lane] = make_double4(ex, ey, ez, ep);
    __syncthreads();
    if (w == 0 && live) {
#pragma unroll
      for (int q = 0; q < kW - 1; ++q) {
        const double4 f = s_f[q][lane];
        ex += f.x; ey += f.y; ez += f.z; ep += f.w;
      }
      const uint32_t orig = A.perm[r];
      A.acc[3 * (size_t)orig + 0] += A.G * ex;
      A.acc[3 * (size_t)orig + 1] += A.G * ey;
      A.acc[3 * (size_t)orig + 2] += A.G * ez;
      if (A.pot) A.pot[orig] += A.G * ep;
    }
    __syncthreads();                  // the sums have been read
  }
}

// -------------------------------------------------------- list kernels
// pass 0: sizes per active group into wl_count[2 gi + {0,1}];
// pass 1: ids at the offsets wl_off (exclusive scan of wl_count).
template <int kPass, bool kRel>
__global__ __launch_bounds__(64) void k_walk_lists(WalkArgs A) {
  const uint32_t n_groups = A.ctr->n_active_groups;
  GroupQueue Q(blockIdx.x);
  for (;;) {
    const uint32_t gi = Q.next(A.ctr, n_groups);
    if (gi >= n_groups) break;
    const uint32_t g = A.alist[gi];
    const uint4 gr = A.groups[g];
    double lo[3], hi[3];
    for (int k = 0; k < 3; ++k) { lo[k] = A.abox[6 * (size_t)g + k]; hi[k] = A.abox[6 * (size_t)g + 3 + k]; }
    const double arel = kRel ? A.arel[g] : 0.0;
    if constexpr (kPass == 0) {
      // the fill pass repeats this walk exactly (also up to a frontier
      // overflow), so these counts bound what it writes
      CountSink S;
      traverse<kRel>(A, S, blockIdx.x, A.root_of[gr.w], lo, hi, arel);
      if (lane_id() == 0) {
        A.wl_count[2 * (size_t)gi] = S.nm;
        A.wl_count[2 * (size_t)gi + 1] = S.np;
      }
    } else {
      FillSink S;
      S.base_m = A.wl_off[2 * (size_t)gi];
      S.base_p = A.wl_off[2 * (size_t)gi + 1];
      traverse<kRel>(A, S, blockIdx.x, A.root_of[gr.w], lo, hi, arel);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------ active groups
__global__ void k_mark_active(const int32_t *__restrict__ gate, const int32_t *__restrict__ idx,
                              const int32_t *__restrict__ n_act, int64_t n,
                              const uint32_t *__restrict__ rank,
                              uint8_t *__restrict__ sact) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  const int64_t m = min((int64_t)n_act[0], n);
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < m;
       k += (int64_t)gridDim.x * blockDim.x) {
    const int32_t i = idx[k];
    if (i >= 0 && i < n) sact[rank[i]] = 1;
  }
}

// Min / max over the 16 lanes of a quarter wave.
__device__ __forceinline__ double qmin(double v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double qmax(double v) {
#pragma unroll
  for (int o = 8; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Sixteen lanes per group (a group holds at most kMaxGroup particles):
// flag groups with an active particle and store the box of their active
// particles.  With old accelerations (caller order, reached through perm)
// also the relative test's group threshold (alpha alpha) min |a_old|^2,
// |a|^2 = (ax ax + ay ay) + az az unfused.  Without active flags (sact null)
// every particle is active, every group is in the list in its own place, and
// there is nothing to compact.
__global__ __launch_bounds__(256) void k_group_active(const int32_t *__restrict__ gate, TreeCounters *ctr,
                                                      const uint4 *__restrict__ groups,
                                                      const uint8_t *__restrict__ sact,
                                                      const double4 *__restrict__ spart,
                                                      const double *__restrict__ acc_old,
                                                      const uint32_t *__restrict__ perm,
                                                      double alpha2,
                                                      uint32_t *__restrict__ aflag,
                                                      uint32_t *__restrict__ acnt,
                                                      uint32_t *__restrict__ alist,
                                                      double *__restrict__ abox,
                                                      double *__restrict__ arel) {
#pragma clang fp contract(off)
  if (gate && *gate <= 0) return;   // nothing active: skipped
  const uint32_t ng = ctr->n_groups;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctr->n_slots = 0;               // counted by the ordering
    if (!sact) ctr->n_active_groups = ng;
  }
  const unsigned q = threadIdx.x & 15u;
  const uint32_t qpb = blockDim.x >> 4;
  for (uint32_t g0 = blockIdx.x * qpb; g0 < ng; g0 += gridDim.x * qpb) {
    const uint32_t g = g0 + (threadIdx.x >> 4);     // quarter-waves stay in step
    const bool live = g < ng;
    const uint4 gr = live ? groups[g] : make_uint4(0, 0, 0, 0);
    double lx = INFINITY, ly = INFINITY, lz = INFINITY;
    double hx = -INFINITY, hy = -INFINITY, hz = -INFINITY;
    double a2min = INFINITY;
    bool any = false;
    uint32_t nact = 0;      // active targets of the quarter-wave's group
#pragma unroll
    for (int r = 0; r < kMaxGroup / 16; ++r) {
      const uint32_t j = q + 16u * r;
      const bool a = j < gr.y && (!sact || sact[gr.x + j]);
      nact += (uint32_t)__popcll((__ballot(a) >> (threadIdx.x & 48u)) & 0xffffull);
      if (a) {
        const double4 p = spart[gr.x + j];
        lx = fmin(lx, p.x); ly = fmin(ly, p.y); lz = fmin(lz, p.z);
        hx = fmax(hx, p.x); hy = fmax(hy, p.y); hz = fmax(hz, p.z);
        any = true;
        if (acc_old) {
          const double *ao = acc_old + 3 * (size_t)perm[gr.x + j];
          const double a2 = dadd(dadd(dmul(ao[0], ao[0]), dmul(ao[1], ao[1])),
                                      dmul(ao[2], ao[2]));
          a2min = fmin(a2min, a2);
        }
      }
    }
    lx = qmin(lx); ly = qmin(ly); lz = qmin(lz);
    hx = qmax(hx); hy = qmax(hy); hz = qmax(hz);
    if (acc_old) a2min = qmin(a2min);
    const unsigned long long m = __ballot(any);
    const unsigned long long mine = (m >> (threadIdx.x & 48u)) & 0xffffull;
    if (live && q == 0) {
      if (sact) aflag[g] = mine ? 1u : 0u;
      else alist[g] = g;
      acnt[g] = nact;
      double *b = abox + 6 * (size_t)g;
      b[0] = lx; b[1] = ly; b[2] = lz; b[3] = hx; b[4] = hy; b[5] = hz;
      if (acc_old) arel[g] = mine ? dmul(alpha2, a2min) : 0.0;
    }
  }
}

__global__ void k_compact_groups(const int32_t *__restrict__ gate, const TreeCounters *ctr,
                                 const uint32_t *__restrict__ aflag,
                                 const uint32_t *__restrict__ aidx,
                                 uint32_t *__restrict__ alist) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  const uint32_t ng = ctr->n_groups;
  for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < ng;
       g += gridDim.x * blockDim.x)
    if (aflag[g]) alist[aidx[g]] = g;
}

// The force walk's items and their order.  A group with nt targets becomes
// ceil(nt / per) items of about equal work, per = max(kMinPart, targets /
// want): the walk's wall time ends with its longest items, and a group of 64
// targets is three to five times the work of an average one, more than a
// wave's share when there are few groups.  What a part repeats of its group
// (the traversal, a tenth to a sixth of an unsplit group's time) is the
// price; with many groups per wave nothing is split.
// Each XCD's queue range [q G / 8, (q + 1) G / 8) of the compacted list keeps
// its groups (and so its part of the tree), taken by size class, largest
// class first (thresholds on the active targets), and in tree order
// within a class: ending on the small ones shortens the tail in which few
// waves are left, and keeping tree order inside a class keeps neighbouring
// groups, which share most of their cells, close in time for the XCD's L2.
// One block per range: a first sweep counts the classes' items, then the
// range is taken in chunks staged in LDS, each thread placing a contiguous
// run of the chunk at offsets from one block scan of its counts.  Stable,
// so deterministic.  No result depends on the order in which items are
// walked.
constexpr int kSizeClasses = 4;
__device__ __forceinline__ uint32_t size_class(uint32_t nt) {
  return nt >= 48u ? 0u : nt >= 32u ? 1u : nt >= 16u ? 2u : 3u;
}

constexpr int kOrderThreads = 1024;
constexpr uint32_t kOrderItems = 8;                                // groups per thread and chunk
constexpr uint32_t kOrderChunk = kOrderThreads * kOrderItems;

// Exclusive block prefix of a 64-bit value (four 16-bit fields; no carries
// between fields since every field's total stays below 2^16).
__device__ __forceinline__ uint64_t block_exclusive_scan64(uint64_t v, uint64_t *sh,
                                                          uint64_t &total) {
  const unsigned lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  uint64_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= (unsigned)o) x += y;
  }
  if (lane == 63u) sh[w] = x;
  __syncthreads();
  uint64_t base = 0, tot = 0;
  for (unsigned q = 0; q < blockDim.x / 64u; ++q) {
    const uint64_t t = sh[q];
    base += q < w ? t : 0ull;
    tot += t;
  }
  __syncthreads();
  total = tot;
  return base + x - v;
}

template <bool kWhole>
__device__ __forceinline__ void order_items(TreeCounters *ctr, const uint32_t *__restrict__ alist,
                                            const uint32_t *__restrict__ acnt,
                                            const int32_t *__restrict__ n_act, int64_t n,
                                            uint32_t want, uint32_t gap, uint32_t whole,
                                            uint2 *__restrict__ items, uint2 *__restrict__ slots) {
  __shared__ uint64_t scan_sh[kOrderThreads / 64];
  __shared__ uint32_t s_g[kOrderChunk];
  __shared__ uint8_t s_n[kOrderChunk];
  __shared__ uint32_t s_sum[kOrderThreads / 64][kSizeClasses + 1], s_tot[kSizeClasses + 1];
  __shared__ uint32_t s_slot0;
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  const uint32_t G = ctr->n_active_groups;
  const uint32_t lo = (uint32_t)(((uint64_t)blockIdx.x * G) >> 3);
  const uint32_t hi = (uint32_t)(((uint64_t)(blockIdx.x + 1) * G) >> 3);
  const uint32_t targets = (uint32_t)(n_act ? min((int64_t)n_act[0], n) : n);
  const uint32_t per = max((uint32_t)kMinPart, (targets + want - 1u) / want);
  auto parts_of = [&](uint32_t nt) { return min((uint32_t)kMaxParts, (nt + per - 1u) / per); };
  const uint32_t most = kWhole && G >= whole ? 1u : (uint32_t)kMaxParts;   // items of a group
  // the range's items of each class and slots
  uint32_t cnt[kSizeClasses + 1] = {};
  for (uint32_t p0 = lo + tid; p0 < hi; p0 += kOrderChunk) {
    uint32_t nt[kOrderItems];       // the loads of kOrderItems groups in flight at once
#pragma unroll
    for (uint32_t j = 0; j < kOrderItems; ++j) {
      const uint32_t p = p0 + j * kOrderThreads;
      nt[j] = p < hi ? acnt[alist[p]] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < kOrderItems; ++j) {
      if (p0 + j * kOrderThreads >= hi) continue;
      const uint32_t k = size_class(nt[j]), np = parts_of(nt[j]);
#pragma unroll
      for (uint32_t q = 0; q < kSizeClasses; ++q) cnt[q] += k == q ? min(np, most) : 0u;
      cnt[kSizeClasses] += np > 1u ? np : 0u;
    }
  }
#pragma unroll
  for (int k = 0; k <= kSizeClasses; ++k) {
    uint32_t v = cnt[k], t;
    (void)wave_excl_scan(v, t);
    if ((tid & 63u) == 0u) s_sum[w][k] = t;
  }
  __syncthreads();
  if (tid <= (uint32_t)kSizeClasses) {
    uint32_t t = 0;
    for (int q = 0; q < kOrderThreads / 64; ++q) t += s_sum[q][tid];
    s_tot[tid] = t;
    if (tid == (uint32_t)kSizeClasses) s_slot0 = t ? atomicAdd(&ctr->n_slots, t) : 0u;
  }
  __syncthreads();
  uint32_t next[kSizeClasses];      // next free place of each class
  next[0] = lo + blockIdx.x * gap;
#pragma unroll
  for (int k = 1; k < kSizeClasses; ++k) next[k] = next[k - 1] + s_tot[k - 1];
  uint32_t slot = s_slot0;
  const bool split = s_tot[kSizeClasses] > 0u;     // uniform
  if (tid == 0) {
    ctr->q_items[blockIdx.x] = s_tot[0] + s_tot[1] + s_tot[2] + s_tot[3];
    ctr->xq[kQueueStride * blockIdx.x] = 0;        // the walk's queue starts over
  }
  for (uint32_t c0 = lo; c0 < hi; c0 += kOrderChunk) {
    const uint32_t m = min(kOrderChunk, hi - c0);
    uint32_t gg[kOrderItems];
#pragma unroll
    for (uint32_t j = 0; j < kOrderItems; ++j) {
      const uint32_t i = tid + j * kOrderThreads;
      gg[j] = i < m ? alist[c0 + i] : 0u;
    }
#pragma unroll
    for (uint32_t j = 0; j < kOrderItems; ++j) {
      const uint32_t i = tid + j * kOrderThreads;
      if (i < m) {
        s_g[i] = gg[j];
        s_n[i] = (uint8_t)acnt[gg[j]];
      }
    }
    __syncthreads();
    // this thread's run [kOrderItems tid, kOrderItems (tid + 1)) of the
    // chunk; a chunk has at most kOrderChunk + 2 want items (split groups
    // have more than `per` targets each)
    const uint32_t r0 = kOrderItems * tid;
    uint64_t mine = 0;
    uint32_t my_slots = 0;
#pragma unroll
    for (uint32_t j = 0; j < kOrderItems; ++j) {
      if (r0 + j >= m) break;
      const uint32_t nt = s_n[r0 + j], np = parts_of(nt);
      mine += (uint64_t)min(np, most) << (16u * size_class(nt));
      my_slots += np > 1u ? np : 0u;
    }
    uint64_t tot;
    const uint64_t ex = block_exclusive_scan64(mine, scan_sh, tot);
    uint32_t slot_tot = 0, s0 = slot;
    if (split) s0 += block_exclusive_scan(my_slots, reinterpret_cast<uint32_t *>(scan_sh), slot_tot);
    uint32_t at[kSizeClasses];
#pragma unroll
    for (uint32_t q = 0; q < kSizeClasses; ++q) at[q] = next[q] + (uint32_t)((ex >> (16u * q)) & 0xffffu);
#pragma unroll
    for (uint32_t j = 0; j < kOrderItems; ++j) {
      if (r0 + j >= m) break;
      const uint32_t nt = s_n[r0 + j], k = size_class(nt), np = parts_of(nt), g = s_g[r0 + j];
      uint32_t dst = at[0];
#pragma unroll
      for (uint32_t q = 1; q < kSizeClasses; ++q) dst = k == q ? at[q] : dst;
#pragma unroll
      for (uint32_t q = 0; q < kSizeClasses; ++q) at[q] += k == q ? min(np, most) : 0u;
      if (np == 1u) {
        items[dst] = make_uint2(g, 0u);
      } else {
        for (uint32_t e = 0; e < np; ++e) {
          const uint32_t all = kWhole && most == 1u ? kAllParts : 0u;
          if (!kWhole || e < most) items[dst + e] = make_uint2(g, e | (np - 1u) << 5 | s0 << 10 | all);
          slots[s0 + e] = make_uint2(g, e == 0u ? np : 0u);
        }
        s0 += np;
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < kSizeClasses; ++q) next[q] += (uint32_t)((tot >> (16u * q)) & 0xffffu);
    slot += slot_tot;
    __syncthreads();                // the chunk's LDS is read before the next is staged
  }
}

// Walk records of every node: Q = 3S - T I, -T eps^2 (spline: T) and M, in
// the walk's precision, formed once per evaluation instead of once per
// staged cell.
template <class R>
__device__ __forceinline__ void cell_records(uint32_t v0, uint32_t stride, uint32_t nn,
                                             const double *__restrict__ mom, double eps2,
                                             int spline, void *cell) {
  using R4 = typename Vec4<R>::T;
  R4 *out = reinterpret_cast<R4 *>(cell);
  for (uint32_t v = v0; v < nn; v += stride) {
    const double4 m0 = reinterpret_cast<const double4 *>(mom)[2 * (size_t)v];
    const double4 m1 = reinterpret_cast<const double4 *>(mom)[2 * (size_t)v + 1];
    // m0 = {M, Sxx, Syy, Szz}, m1 = {Sxy, Sxz, Syz, -}
    const double T = m0.y + m0.z + m0.w;
    out[2 * (size_t)v] = R4{(R)(3.0 * m0.y - T), (R)(3.0 * m0.z - T), (R)(3.0 * m0.w - T),
                            spline ? (R)T : (R)(-(T * eps2))};
    out[2 * (size_t)v + 1] = R4{(R)(3.0 * m1.x), (R)(3.0 * m1.y), (R)(3.0 * m1.z), (R)m0.x};
  }
}

// Relative-test records of every node: the cell cube enlarged by 20 %
// about its geometric centre and P = (G M) s^2, s the node's opening size
// (the cell side, or its refitted size), every operation rounded separately.
struct RelArgs {
  const uint8_t *level;
  const uint32_t *first, *nsys;
  const uint64_t *skey;
  const double *cube, *mom, *side;
  double G;
  double4 *rel;                  // null: no relative test
};
__device__ __forceinline__ void rel_records(uint32_t v0, uint32_t stride, uint32_t nn,
                                            const RelArgs &A) {
#pragma clang fp contract(off)
  for (uint32_t v = v0; v < nn; v += stride) {
    double g[3];
    cell_centre(v, A.level[v], A.first, A.nsys, A.skey, A.cube, g);
    const double s = A.side[v];
    const double h = dmul(0.6, s);
    double lo[3], hi[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lo[k] = dsub(g[k], h);
      hi[k] = dadd(g[k], h);
    }
    const double P = dmul(dmul(A.G, A.mom[8 * (size_t)v]), dmul(s, s));
    A.rel[2 * (size_t)v] = make_double4(lo[0], lo[1], lo[2], P);
    A.rel[2 * (size_t)v + 1] = make_double4(hi[0], hi[1], hi[2], 0.0);
  }
}

__global__ __launch_bounds__(256) void k_rel_records(const int32_t *__restrict__ gate,
                                                     const TreeCounters *ctr, RelArgs A) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  rel_records(blockIdx.x * blockDim.x + threadIdx.x, gridDim.x * blockDim.x, ctr->n_nodes, A);
}

// What the force walk needs besides the boxes, in one launch: eight blocks
// order its items while the others form the nodes' records (the ordering
// keeps eight CUs busy for 10 to 30 us, most of it waiting; the records take
// 4 to 26).  With the marking, scan and compaction that a walk without an
// active list no longer launches: 1021 stars 187 -> 173 us a force
// evaluation, 131072 stars 748 -> 731 us a step.
constexpr int kRecordBlocks = 504;

template <class R, bool kWhole>
__global__ __launch_bounds__(kOrderThreads) void k_walk_prepare(
    const int32_t *__restrict__ gate, TreeCounters *ctr, const uint32_t *__restrict__ alist,
    const uint32_t *__restrict__ acnt, const int32_t *__restrict__ n_act, int64_t n, uint32_t want,
    uint32_t gap, uint32_t whole, uint2 *__restrict__ items, uint2 *__restrict__ slots,
    const double *__restrict__ mom, double eps2, int spline, void *cell, RelArgs rel) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  if (blockIdx.x < 8u) {
    order_items<kWhole>(ctr, alist, acnt, n_act, n, want, gap, whole, items, slots);
    return;
  }
  const uint32_t v0 = (blockIdx.x - 8u) * kOrderThreads + threadIdx.x;
  constexpr uint32_t kStride = kRecordBlocks * kOrderThreads;
  cell_records<R>(v0, kStride, ctr->n_nodes, mom, eps2, spline, cell);
  if (rel.rel) rel_records(v0, kStride, ctr->n_nodes, rel);
}

__global__ void k_counts_reset(TreeCounters *ctr) {
  if (threadIdx.x == 0) {
    ctr->cum_p2p = 0;
    ctr->cum_p2m = 0;
    ctr->cum_targets = 0;
    ctr->cum_walked = 0;
  }
}

hipError_t launch_counts_reset(tg_ctx *c) {
  hipLaunchKernelGGL(k_counts_reset, dim3(1), dim3(64), 0, c->stream, c->b.ctr);
  return hipGetLastError();
}

__global__ void k_walk_reset(TreeCounters *ctr) {
  if (threadIdx.x < 8) ctr->xq[kQueueStride * threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    ctr->n_p2p = 0;
    ctr->n_p2m = 0;
    ctr->n_targets = 0;
    ctr->n_walked = 0;
  }
}

// As many waves as asked for (the list kernels' launch).
static int walk_grid(const tg_ctx *c) {
  return std::max(1, c->n_cu * c->waves_per_cu);
}

// The force walk's waves that are sure to be resident: as asked for, up to
// what the kernel is compiled for.  Each of them starts with an item of its
// own, the largest first (one that started only when others end would leave
// a longest item to the end: the FP64 walk of the 1M cusp took 8% longer
// with 16 such waves per CU).
static int walk_per_cu(const tg_ctx *c) {
  return 4 * (c->cfg.precision == TG_MIXED ? TG_WALK_WAVES_MIXED : TG_WALK_WAVES_FP64);
}
static int walk_waves(const tg_ctx *c) {
  return std::max(1, c->n_cu * std::min(c->waves_per_cu, walk_per_cu(c)));
}

// Its launch.  The FP64 kernel fits a ninth wave into a CU (three by its 167
// registers into a SIMD, nine by 16 KB of LDS each).  An evaluation with eight
// and with as many as fit, in us: 200000 stars 1427 and 1412, 350000 2424 and
// 2380, 524287 3607 and 3528, 1M 7201 and 7032.  The rule goes by the
// particles, since only the device knows the active ones: with 30% of 300000
// active 996 and 1013 us, of 1M 2956 and 2907; with 10% 604 and 598, 1362 and
// 1364; with 0.3% 342 and 339, 556 and 551.  Above the line none of these is
// slower, below it either may be by 1 or 2%.
static int walk_blocks(const tg_ctx *c) {
  return c->n >= (1 << 19) ? walk_grid(c) : walk_waves(c);
}
// Particles below which an FP64 walk has its waves two to each SIMD: between
// 131072, where that is 3% faster, and 160000, where it is alike.
constexpr int64_t kEvenBelow = 9 << 14;
// Whether split groups are taken as a whole where there are enough groups for
// the context's waves, and from how many on: 5/4 of the waves with one wave per
// CU, twice as many with four.  A walk in us by parts and as a whole, mixed
// precision: with one wave 4096 stars (300 groups) 223 and 226, 6000 311 and
// 261; with two (512 waves) 10000 273 and 280, 14000 356 and 338; with four
// 30000 357 and 396, 40000 (2000) 428 and 414; with six the parts are faster or
// alike (50000 stars 411 unsplit and 372, 100000 587 and 600).
static bool walk_whole(const tg_ctx *c) { return c->waves_per_cu <= 4; }
static uint32_t whole_from(const tg_ctx *c, uint32_t waves) {
  return waves + waves / 4u * (uint32_t)c->waves_per_cu;
}

hipError_t launch_active_groups(tg_ctx *c, const int32_t *idx,
                                const int32_t *n_act, const double *acc_old,
                                double alpha) {
  Buffers &b = c->b;
  if (c->n == 0) return fill_u32(&b.ctr->n_active_groups, 0u, 1, c->stream);
  hipError_t e = hipSuccess;
  if (idx) {
    e = fill_u8(b.sact, 0, c->n, c->stream, c->gate);
    if (e != hipSuccess) return e;
    const int g = (int)std::min<int64_t>((c->n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_mark_active, dim3(g), dim3(256), 0, c->stream, c->gate, idx,
                       n_act, c->n, b.rank, b.sact);
  }
  hipLaunchKernelGGL(k_group_active, dim3(2048), dim3(256), 0, c->stream, c->gate,
                     b.ctr, b.groups, idx ? b.sact : nullptr, b.spart, acc_old, b.val[0],
                     alpha * alpha, b.aflag, b.acnt, b.alist, b.abox, b.arel);
  if (!idx) return hipGetLastError();
  // the group-start scan buffer is free after the build: reuse it
  e = scan_u32(b.aflag, b.gflag, 0u, &b.ctr->n_groups, &b.ctr->n_active_groups,
               b.scan_part, c->stream, c->gate);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_compact_groups, dim3(1024), dim3(256), 0, c->stream, c->gate,
                     b.ctr, b.aflag, b.gflag, b.alist);
  return hipGetLastError();
}

// n_act: the active list's device count (null: every particle is active)
static WalkArgs make_args(tg_ctx *c, double theta, const int32_t *n_act = nullptr) {
  Buffers &b = c->b;
  WalkArgs A;
  A.ninfo = b.ninfo; A.com = b.com; A.cell = b.cell;
  A.rel = b.rel; A.arel = b.arel;
  A.spart = b.spart; A.root_of = b.root_of;
  A.groups = b.groups; A.alist = b.alist; A.abox = b.abox;
  A.sact = n_act ? b.sact : nullptr;
  A.perm = b.val[0]; A.ctr = b.ctr; A.wtot = b.wtot; A.err = b.err; A.frontier = b.frontier;
  A.fcap = c->cfg.frontier_cap;
  A.th2 = theta * theta;
  A.eps2 = 0.0; A.G = c->cfg.G;
  A.acc = nullptr; A.pot = nullptr;
  A.ext_pos = c->ext_pos; A.ext_mass = c->ext_mass; A.ext_eps = c->ext_eps;
  A.ext_seg = c->n_ext > 0 ? c->b.ext_seg : nullptr;
  A.eps = 0.0;
  A.items = nullptr; A.item_gap = 0; A.slots = nullptr; A.wpart = nullptr; A.starts = 0;
  A.wl_count = b.wl_count; A.wl_off = b.wl_off; A.ids = nullptr;
  return A;
}

static RelArgs rel_args(tg_ctx *c, bool rel) {
  Buffers &b = c->b;
  return RelArgs{b.level, b.first, b.nsys, b.key[0], b.cube, b.mom, b.side, c->cfg.G,
                 rel ? b.rel : nullptr};
}

template <bool kRel, bool kSpline>
static void launch_force_kernel(tg_ctx *c, const WalkArgs &A, bool whole) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(walk_blocks(c)), dim3(64), 0, c->stream, c->gate, A);
  };
  const bool mixed = c->cfg.precision == TG_MIXED;
  if (whole)
    return mixed ? go(k_walk_forces<true, kRel, kSpline, kFormWhole>)
                 : go(k_walk_forces<false, kRel, kSpline, kFormWhole>);
  if (mixed) return go(k_walk_forces<true, kRel, kSpline, kFormFull>);
  if constexpr (!kSpline)              // (with the spline two waves fill a SIMD anyway)
    if (c->n < kEvenBelow) return go(k_walk_forces<false, kRel, false, kFormEven>);
  go(k_walk_forces<false, kRel, kSpline, kFormFull>);
}

hipError_t launch_walk_forces(tg_ctx *c, double eps, double theta, const int32_t *n_act,
                              double *acc, double *pot, hipEvent_t before,
                              hipEvent_t after, bool rel) {
  Buffers &b = c->b;
  WalkArgs A = make_args(c, theta, n_act);
  A.items = b.items; A.item_gap = (uint32_t)c->split_cap;
  A.slots = b.slots; A.wpart = b.wpart;
  A.starts = (uint32_t)walk_waves(c);
  A.eps2 = eps * eps;
  A.eps = eps;
  A.acc = acc;
  A.pot = pot;
  const int spline = c->soft == TG_SOFT_SPLINE ? 1 : 0;
  // many external masses: a kernel of their own after the walk
  WalkArgs X = A;
  int32_t most = 0;
  if (A.ext_seg)
    for (size_t k = 1; k < c->ext_seg_host.size(); ++k)
      most = std::max(most, c->ext_seg_host[k] - c->ext_seg_host[k - 1]);
  if (most > kExternalsInWalk) A.ext_seg = nullptr;
  // the split is for the waves that fit, whatever the launch: results do
  // not depend on waves_per_cu
  const uint32_t want = (uint32_t)(kItemsPerWave * c->n_cu * walk_per_cu(c));
  const bool mixed = c->cfg.precision == TG_MIXED;
  const bool whole = walk_whole(c);
  auto prepare = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(8 + kRecordBlocks), dim3(kOrderThreads), 0, c->stream, c->gate,
                       b.ctr, b.alist, b.acnt, n_act, c->n, want, (uint32_t)c->split_cap,
                       whole_from(c, A.starts), b.items, b.slots, b.mom, A.eps2, spline,
                       (void *)b.cell, rel_args(c, rel));
  };
  if (mixed) whole ? prepare(k_walk_prepare<float, true>) : prepare(k_walk_prepare<float, false>);
  else whole ? prepare(k_walk_prepare<double, true>) : prepare(k_walk_prepare<double, false>);
  if (before) {
    hipError_t e = hipEventRecord(before, c->stream);
    if (e != hipSuccess) return e;
  }
  if (spline) {
    if (rel) launch_force_kernel<true, true>(c, A, whole);
    else launch_force_kernel<false, true>(c, A, whole);
  } else {
    if (rel) launch_force_kernel<true, false>(c, A, whole);
    else launch_force_kernel<false, false>(c, A, whole);
  }
  if (spline)
    hipLaunchKernelGGL(k_walk_finish<true>, dim3(kFinishBlocks), dim3(kFinishThreads), 0, c->stream,
                       c->gate, A, walk_blocks(c));
  else
    hipLaunchKernelGGL(k_walk_finish<false>, dim3(kFinishBlocks), dim3(kFinishThreads), 0, c->stream,
                       c->gate, A, walk_blocks(c));
  if (most > kExternalsInWalk) {
    const dim3 grid((unsigned)std::min<int64_t>((c->n + 63) / 64, 16384));
    hipLaunchKernelGGL((spline ? k_externals<true> : k_externals<false>), grid, dim3(256), 0,
                       c->stream, c->gate, X, c->n, b.sysoff, c->S);
  }
  if (after) {                     // the walk's results are whole
    hipError_t e = hipEventRecord(after, c->stream);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t launch_walk_lists(tg_ctx *c, double theta, int pass, int64_t *info,
                             int64_t cap_groups, uint32_t *ids, int64_t cap_ids,
                             bool rel) {
  (void)info; (void)cap_groups; (void)cap_ids;
  WalkArgs A = make_args(c, theta);
  A.ids = ids;
  if (rel && pass == 0)
    hipLaunchKernelGGL(k_rel_records, dim3(1024), dim3(256), 0, c->stream, c->gate, c->b.ctr,
                       rel_args(c, true));
  hipLaunchKernelGGL(k_walk_reset, dim3(1), dim3(64), 0, c->stream, c->b.ctr);
  const dim3 grid(walk_grid(c));
  if (pass == 0 && !rel)
    hipLaunchKernelGGL((k_walk_lists<0, false>), grid, dim3(64), 0, c->stream, A);
  else if (pass == 0)
    hipLaunchKernelGGL((k_walk_lists<0, true>), grid, dim3(64), 0, c->stream, A);
  else if (!rel)
    hipLaunchKernelGGL((k_walk_lists<1, false>), grid, dim3(64), 0, c->stream, A);
  else
    hipLaunchKernelGGL((k_walk_lists<1, true>), grid, dim3(64), 0, c->stream, A);
  return hipGetLastError();
}

}  // namespace tg
