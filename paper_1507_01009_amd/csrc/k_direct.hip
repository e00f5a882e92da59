// Double-precision direct forces between a source set and a target set
// (SMBH <-> stars; perturber <-> chain-member corrections), softening
// max(eps_i, eps_j) per pair: Plummer, or the cubic spline with that h.
//
// Many targets of one segment (checks of the tree's forces, perturbers on
// perturbers): blocks of 64 or 128 targets over source tiles in LDS.  Few
// targets (SMBHs feeling a million stars): one 256-thread block per (target,
// range of few_span sources), threads striding through the range with
// coalesced loads, the block's sums combined in a fixed tree order and the
// per-block partials summed in a second ordered pass.  Anything else
// (more targets of several segments, a handful of pairs): one thread per
// target and source chunk.  direct_plan.h holds the rules.  Every sum is compensated
// (error-free TwoSum with a running correction), so the result does not
// depend on the split beyond the last bit and is deterministic.  Every
// operation is rounded on its own (no FMA contraction): the TwoSum steps
// need it, and so does the fused drift-and-sum kernel, whose sums must equal
// the unfused ones bit for bit.
#include <type_traits>

#include "direct_plan.h"
#include "tg_internal.h"

namespace tg {

__device__ __forceinline__ int seg_of(const int64_t *off, int nseg, int64_t i) {
  int lo = 0, hi = nseg - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// 1 / sqrt(x) to about one unit in the last place: rsqrt_dp.  A rounded square
// root and division (1 / sqrt(x), also about one unit) cost some 25
// instructions more per pair; they stay for everything but positive normal
// numbers (x = 0 of unsoftened coincident pairs, subnormals, infinities, NaN).
__device__ __forceinline__ double inv_sqrt(double x) {
  constexpr int kPositiveNormal = 0x100;
  if (__builtin_expect(!__builtin_amdgcn_class(x, kPositiveNormal), 0)) return 1.0 / sqrt(x);
  return rsqrt_dp(x);
}

// m/r and m/r^3 with the pair's softening ep (soft: cubic spline, h = ep).
__device__ __forceinline__ void pair_terms(double dx, double dy, double dz, double ep, double m,
                                           int soft, double &mD1, double &mD3) {
#pragma clang fp contract(off)
  if (soft) {
    double p0, p1;
    spline_pair_dp(sqrt(dx * dx + dy * dy + dz * dz), ep, p0, p1);
    mD1 = m * p0;
    mD3 = m * p1;
  } else {
    const double D1 = inv_sqrt(dx * dx + dy * dy + dz * dz + ep * ep);
    mD1 = m * D1;
    mD3 = mD1 * D1 * D1;
  }
}

// One thread per target and source chunk.  Bound by the latency of a thread's
// pairs one after another; the next source is read before a pair is summed,
// since no load moves ahead of the branch in inv_sqrt by itself (256 targets
// on 4000 sources each 174 us without, 153 with; one on 8191 101 -> 78; 5000
// targets of 100 segments of 10000 sources 478 -> 272).
__global__ void k_direct(const double *__restrict__ spos, const double *__restrict__ sm,
                         const double *__restrict__ seps, double seps_all,
                         const double *__restrict__ tpos,
                         const double *__restrict__ teps, int64_t nt,
                         const int64_t *__restrict__ sseg, const int64_t *__restrict__ tseg,
                         int nseg, int64_t chunk, int nchunks, int self_pairs,
                         int accumulate, int soft, double *__restrict__ acc,
                         double *__restrict__ pot, double *__restrict__ part) {
#pragma clang fp contract(off)
  const int64_t total = nt * (int64_t)nchunks;
  for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < total;
       w += (int64_t)gridDim.x * blockDim.x) {
    const int64_t i = w % nt;
    const int c = (int)(w / nt);
    const int s = seg_of(tseg, nseg, i);
    const int64_t j0 = sseg[s] + (int64_t)c * chunk;
    const int64_t j1 = min(sseg[s + 1], j0 + chunk);
    const double xi = tpos[3 * i], yi = tpos[3 * i + 1], zi = tpos[3 * i + 2];
    const double ei = teps[i];
    CSum ax, ay, az, ph;
    double nx = 0.0, ny = 0.0, nz = 0.0, nm = 0.0, ne = seps_all;
    auto load = [&](int64_t j) {
      nx = spos[3 * j]; ny = spos[3 * j + 1]; nz = spos[3 * j + 2]; nm = sm[j];
      if (seps) ne = seps[j];
    };
    if (j0 < j1) load(j0);
    for (int64_t j = j0; j < j1; ++j) {
      const double dx = xi - nx, dy = yi - ny, dz = zi - nz, m = nm, ep = fmax(ne, ei);
      if (j + 1 < j1) load(j + 1);
      if (self_pairs && j == i) continue;
      double mD1, mD3;
      pair_terms(dx, dy, dz, ep, m, soft, mD1, mD3);
      ax.add(-mD3 * dx);
      ay.add(-mD3 * dy);
      az.add(-mD3 * dz);
      ph.add(-mD1);
    }
    if (nchunks == 1) {
      double a0 = ax.get(), a1 = ay.get(), a2 = az.get(), p = ph.get();
      if (accumulate) {
        acc[3 * i] += a0; acc[3 * i + 1] += a1; acc[3 * i + 2] += a2;
        if (pot) pot[i] += p;
      } else {
        acc[3 * i] = a0; acc[3 * i + 1] = a1; acc[3 * i + 2] = a2;
        if (pot) pot[i] = p;
      }
    } else {
      double *o = part + 8 * (size_t)w;
      o[0] = ax.s; o[1] = ax.c; o[2] = ay.s; o[3] = ay.c;
      o[4] = az.s; o[5] = az.c; o[6] = ph.s; o[7] = ph.c;
    }
  }
}

// Many targets of one segment: a block of four waves takes 64 kT targets
// (kT to a lane) and one chunk of the sources, staged kTileSrc at a time in
// LDS; each wave sums its quarter of a tile onto all the block's targets,
// and the four waves' sums are combined in order at the end.  A source is
// read from memory once per block and from LDS as a broadcast; the next
// tile's loads are in flight while a tile is summed.  Bound by FP64 issue:
// about 50 instructions per pair, 28 of them the compensated sums.  Two
// targets to a lane: with one the LDS reads set the rate (3.7e11 pairs/s on
// 65536 x 65536), with three and four the lanes' sums leave too few waves
// (5.0e11, 5.2e11); two reach 6.1e11 (2.0e11 with one thread per target and
// every source read from memory by every thread).  8191 targets on 262144
// sources: 13.9 -> 3.7 ms.
template <int kT, bool kSelf, bool kSoft>
__global__ __launch_bounds__(256) void k_direct_tile(
    const double *__restrict__ spos, const double *__restrict__ sm,
    const double *__restrict__ seps, double seps_all, int64_t ns,
    const double *__restrict__ tpos, const double *__restrict__ teps, int64_t nt,
    int64_t chunk, int accumulate, double *__restrict__ acc, double *__restrict__ pot,
    double *__restrict__ part) {
#pragma clang fp contract(off)
  constexpr int kW = kTileSrc / 64;
  __shared__ double4 s_xm[kTileSrc];
  __shared__ double s_e[kTileSrc];
  __shared__ double2 s_sum[kW - 1][4 * kT][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t i0 = (int64_t)blockIdx.x * (64 * kT) + lane;
  const int64_t j0 = (int64_t)blockIdx.y * chunk, j1 = min(ns, j0 + chunk);
  double xi[kT], yi[kT], zi[kT], ei[kT];
#pragma unroll
  for (int k = 0; k < kT; ++k) {
    const int64_t i = min(i0 + 64 * k, nt - 1);     // lanes past the end repeat the last target
    xi[k] = tpos[3 * i]; yi[k] = tpos[3 * i + 1]; zi[k] = tpos[3 * i + 2];
    ei[k] = teps[i];
  }
  CSum r[kT][4];
  double4 nx = make_double4(0.0, 0.0, 0.0, 0.0);
  double ne = 0.0;
  auto load = [&](int64_t j) {
    if (j < j1) {
      nx = make_double4(spos[3 * j], spos[3 * j + 1], spos[3 * j + 2], sm[j]);
      ne = seps ? seps[j] : seps_all;
    }
  };
  load(j0 + tid);
  for (int64_t t0 = j0; t0 < j1; t0 += kTileSrc) {
    s_xm[tid] = nx;
    s_e[tid] = ne;
    __syncthreads();
    load(t0 + kTileSrc + tid);
    const int m = __builtin_amdgcn_readfirstlane((int)min<int64_t>(64, j1 - t0 - 64 * w));
#pragma unroll 2
    for (int q = 0; q < m; ++q) {
      const double4 s = s_xm[64 * w + q];
      const double es = s_e[64 * w + q];
#pragma unroll
      for (int k = 0; k < kT; ++k) {
        const double dx = xi[k] - s.x, dy = yi[k] - s.y, dz = zi[k] - s.z;
        double mD1, mD3;
        pair_terms(dx, dy, dz, fmax(es, ei[k]), s.w, kSoft, mD1, mD3);
        if constexpr (kSelf) {
          const bool own = t0 + 64 * w + q == i0 + 64 * k;   // its own pair adds zeros
          mD1 = own ? 0.0 : mD1;
          mD3 = own ? 0.0 : mD3;
        }
        r[k][0].add(-mD3 * dx);
        r[k][1].add(-mD3 * dy);
        r[k][2].add(-mD3 * dz);
        r[k][3].add(-mD1);
      }
    }
    __syncthreads();
  }
  if (w > 0) {
#pragma unroll
    for (int k = 0; k < kT; ++k)
#pragma unroll
      for (int c = 0; c < 4; ++c) s_sum[w - 1][4 * k + c][lane] = make_double2(r[k][c].s, r[k][c].c);
  }
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int k = 0; k < kT; ++k) {
    const int64_t i = i0 + 64 * k;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
      for (int q = 0; q < kW - 1; ++q) {
        const double2 o = s_sum[q][4 * k + c][lane];
        r[k][c].add(o.x);
        r[k][c].c += o.y;
      }
    }
    if (i >= nt) continue;
    if (gridDim.y == 1) {
      const double a0 = r[k][0].get(), a1 = r[k][1].get(), a2 = r[k][2].get(), p = r[k][3].get();
      if (accumulate) {
        acc[3 * i] += a0; acc[3 * i + 1] += a1; acc[3 * i + 2] += a2;
        if (pot) pot[i] += p;
      } else {
        acc[3 * i] = a0; acc[3 * i + 1] = a1; acc[3 * i + 2] = a2;
        if (pot) pot[i] = p;
      }
    } else {
      double *o = part + 8 * (size_t)(blockIdx.y * nt + i);
#pragma unroll
      for (int c = 0; c < 4; ++c) { o[2 * c] = r[k][c].s; o[2 * c + 1] = r[k][c].c; }
    }
  }
}

// The chunks' partial sums of a target added in order by one thread (few
// chunks, many targets).
__global__ __launch_bounds__(64) void k_direct_chunks(int64_t nt, int nchunks, int accumulate,
                                                      const double *__restrict__ part,
                                                      double *__restrict__ acc,
                                                      double *__restrict__ pot) {
#pragma clang fp contract(off)
  const int64_t i = blockIdx.x * (int64_t)64 + threadIdx.x;
  if (i >= nt) return;
  CSum r[4];
  for (int c = 0; c < nchunks; ++c) {
    const double *o = part + 8 * (size_t)(c * nt + i);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      r[k].add(o[2 * k]);
      r[k].c += o[2 * k + 1];
    }
  }
  const double v0 = r[0].get(), v1 = r[1].get(), v2 = r[2].get(), v3 = r[3].get();
  if (accumulate) {
    acc[3 * i] += v0; acc[3 * i + 1] += v1; acc[3 * i + 2] += v2;
    if (pot) pot[i] += v3;
  } else {
    acc[3 * i] = v0; acc[3 * i + 1] = v1; acc[3 * i + 2] = v2;
    if (pot) pot[i] = v3;
  }
}

// Compensated sums of 256 threads (t: the number among them) combined in a
// fixed tree order; thread 0 returns with the totals in ss[k][0] + sc[k][0].
// Every thread of the block is here.
__device__ __forceinline__ void block_csum4(CSum r[4], double (*ss)[256], double (*sc)[256],
                                            int t = threadIdx.x) {
  for (int k = 0; k < 4; ++k) { ss[k][t] = r[k].s; sc[k][t] = r[k].c; }
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (t < h) {
      for (int k = 0; k < 4; ++k) {
        CSum x;
        x.s = ss[k][t];
        x.c = sc[k][t] + sc[k][t + h];
        x.add(ss[k][t + h]);
        ss[k][t] = x.s;
        sc[k][t] = x.c;
      }
    }
    __syncthreads();
  }
}

// grid (blocks per target, targets): block b of target i sums sources
// [b span, (b + 1) span) of i's segment into part[b nt + i].
__global__ __launch_bounds__(256) void k_direct_few(
    const double *__restrict__ spos, const double *__restrict__ sm,
    const double *__restrict__ seps, double seps_all, const double *__restrict__ tpos,
    const double *__restrict__ teps, int64_t nt, const int64_t *__restrict__ sseg,
    const int64_t *__restrict__ tseg, int nseg, int self_pairs, int soft, int span,
    double *__restrict__ part) {
#pragma clang fp contract(off)
  __shared__ double ss[4][256], sc[4][256];
  const int64_t i = blockIdx.y;
  const int s = seg_of(tseg, nseg, i);
  const int64_t j0 = sseg[s] + (int64_t)blockIdx.x * span;
  const int64_t j1 = min(sseg[s + 1], j0 + span);
  const double xi = tpos[3 * i], yi = tpos[3 * i + 1], zi = tpos[3 * i + 2];
  const double ei = teps[i];
  CSum r[4];
  for (int64_t j = j0 + threadIdx.x; j < j1; j += 256) {
    if (self_pairs && j == i) continue;
    const double ep = fmax(seps ? seps[j] : seps_all, ei);
    const double dx = xi - spos[3 * j], dy = yi - spos[3 * j + 1], dz = zi - spos[3 * j + 2];
    double mD1, mD3;
    pair_terms(dx, dy, dz, ep, sm[j], soft, mD1, mD3);
    r[0].add(-mD3 * dx);
    r[1].add(-mD3 * dy);
    r[2].add(-mD3 * dz);
    r[3].add(-mD1);
  }
  block_csum4(r, ss, sc);
  if (threadIdx.x == 0) {
    double *o = part + 8 * (size_t)(blockIdx.x * nt + i);
    for (int k = 0; k < 4; ++k) { o[2 * k] = ss[k][0]; o[2 * k + 1] = sc[k][0]; }
  }
}

// One block per target: each thread sums a strided subset of the chunks,
// then the block combines the compensated pairs in a fixed tree order.
__global__ __launch_bounds__(256) void k_direct_reduce(int64_t nt, int nchunks,
                                                       int accumulate,
                                                       const double *__restrict__ part,
                                                       double *__restrict__ acc,
                                                       double *__restrict__ pot) {
  __shared__ double ss[4][256], sc[4][256];
  for (int64_t i = blockIdx.x; i < nt; i += gridDim.x) {
    CSum r[4];
    for (int c = threadIdx.x; c < nchunks; c += 256) {
      const double *o = part + 8 * (size_t)(c * nt + i);
      for (int k = 0; k < 4; ++k) {
        r[k].add(o[2 * k]);
        r[k].add(o[2 * k + 1]);
      }
    }
    block_csum4(r, ss, sc);
    if (threadIdx.x == 0) {
      const double v0 = ss[0][0] + sc[0][0], v1 = ss[1][0] + sc[1][0];
      const double v2 = ss[2][0] + sc[2][0], v3 = ss[3][0] + sc[3][0];
      if (accumulate) {
        acc[3 * i] += v0; acc[3 * i + 1] += v1; acc[3 * i + 2] += v2;
        if (pot) pot[i] += v3;
      } else {
        acc[3 * i] = v0; acc[3 * i + 1] = v1; acc[3 * i + 2] = v2;
        if (pot) pot[i] = v3;
      }
    }
    __syncthreads();
  }
}

// The stars' drift fused with the SMBH <- star sums of a block substep
// (one system, at most kDriftSmbhMax SMBHs): block b drifts the stars
// [b span, (b + 1) span) (x <- x + v dt with the operations of k_drift;
// frozen stars stay) and sums their pull on every SMBH at the drifted
// positions with the ranges, thread order and block reduction of
// k_direct_few, so k_smbh_finish turns the partials into the same totals.
// The stars' positions are read once instead of twice.  Bound by memory (4.2M
// stars and two SMBHs 55.7 us, 6.1 TB/s).  The waves per SIMD are asked for:
// 4.2M stars are 1025 blocks, and with two SMBHs the compiler took two
// registers too many for five of them to a CU, so that the last one ran alone
// (63.4 us).
constexpr int kDriftSmbhMax = 4;

template <int kNB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kNB == 1 ? 7 : kNB == 2 ? 5 : 3)))
void k_drift_smbh(
    double *__restrict__ pos, const double *__restrict__ vel, const uint8_t *__restrict__ frozen,
    int64_t n, double dt, const double *__restrict__ sm, double seps,
    const double *__restrict__ bpos, const double *__restrict__ beps, int soft, int span,
    double *__restrict__ part) {
#pragma clang fp contract(off)
  constexpr int nb = kNB;
  __shared__ double ss[4][256], sc[4][256];
  const int64_t j0 = (int64_t)blockIdx.x * span;
  const int64_t j1 = min(n, j0 + span);
  double bx[nb], by[nb], bz[nb], be[nb];
#pragma unroll
  for (int i = 0; i < nb; ++i) {
    bx[i] = bpos[3 * i]; by[i] = bpos[3 * i + 1]; bz[i] = bpos[3 * i + 2]; be[i] = beps[i];
  }
  CSum r[nb][4];
  for (int64_t j = j0 + threadIdx.x; j < j1; j += 256) {
    double x = pos[3 * j], y = pos[3 * j + 1], z = pos[3 * j + 2];
    if (!(frozen && frozen[j])) {
      x = x + vel[3 * j] * dt;
      y = y + vel[3 * j + 1] * dt;
      z = z + vel[3 * j + 2] * dt;
      pos[3 * j] = x; pos[3 * j + 1] = y; pos[3 * j + 2] = z;
    }
    const double m = sm[j];
#pragma unroll
    for (int i = 0; i < nb; ++i) {
      const double ep = fmax(seps, be[i]);
      const double dx = bx[i] - x, dy = by[i] - y, dz = bz[i] - z;
      double mD1, mD3;
      pair_terms(dx, dy, dz, ep, m, soft, mD1, mD3);
      r[i][0].add(-mD3 * dx);
      r[i][1].add(-mD3 * dy);
      r[i][2].add(-mD3 * dz);
      r[i][3].add(-mD1);
    }
  }
  // static indices keep the sums in registers
#pragma unroll
  for (int i = 0; i < nb; ++i) {
    block_csum4(r[i], ss, sc);
    if (threadIdx.x == 0) {
      double *o = part + 8 * (size_t)(blockIdx.x * nb + i);
      for (int k = 0; k < 4; ++k) { o[2 * k] = ss[k][0]; o[2 * k + 1] = sc[k][0]; }
    }
    __syncthreads();
  }
}

// The totals of the stars' partial sums on an SMBH (as k_direct_reduce) plus
// the pull of the other SMBHs of its segment (as k_direct; formed by another
// wave meanwhile), 256 threads per SMBH: one launch of 4.6 us where two took 9.
// A block takes kG SMBHs.  With kStep (one segment, all kG of its SMBHs in one
// block) the next idle substep's kicks and drift of the SMBHs follow, as
// k_bh_substep does them (another launch of 4.7 us).  Bound by latency: the
// partial sums' loads and eight steps of the sums' tree, so the SMBHs of a
// block are taken side by side (one after another, four SMBHs took 17.1 us,
// now 8.8; idle substeps of 20000 stars with four 29.4 -> 23.0 us).
template <int kG, bool kStep>
__global__ __launch_bounds__(256 * kG) void k_smbh_finish(
    int nb, int nchunks, const double *__restrict__ part, double *bpos,
    const double *__restrict__ bmass, const double *__restrict__ beps,
    const int64_t *__restrict__ bseg, int nseg, int soft, double *__restrict__ acc,
    double *__restrict__ pot, double *__restrict__ vel, double dt, int64_t *__restrict__ kctr) {
#pragma clang fp contract(off)
  __shared__ double ss[kG][4][256], sc[kG][4][256], pair[kG][4], a_new[3 * kG];
  const int g = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 8));
  const int t = threadIdx.x & 255;
  const int i = blockIdx.x * kG + g;      // < nb: the grid has nb / kG blocks
  CSum r[4];
  for (int c = t; c < nchunks; c += 256) {
    const double *o = part + 8 * ((size_t)c * nb + i);
    for (int k = 0; k < 4; ++k) {
      r[k].add(o[2 * k]);
      r[k].add(o[2 * k + 1]);
    }
  }
  if (t == 192) {
    int64_t j0 = 0, j1 = nb;
    if (bseg) {
      const int s = seg_of(bseg, nseg, i);
      j0 = bseg[s];
      j1 = bseg[s + 1];
    }
    CSum q[4];
    for (int64_t j = j0; j < j1; ++j) {
      if (j == i) continue;
      const double ep = fmax(beps[j], beps[i]);
      const double dx = bpos[3 * i] - bpos[3 * j], dy = bpos[3 * i + 1] - bpos[3 * j + 1];
      const double dz = bpos[3 * i + 2] - bpos[3 * j + 2];
      double mD1, mD3;
      pair_terms(dx, dy, dz, ep, bmass[j], soft, mD1, mD3);
      q[0].add(-mD3 * dx);
      q[1].add(-mD3 * dy);
      q[2].add(-mD3 * dz);
      q[3].add(-mD1);
    }
    for (int k = 0; k < 4; ++k) pair[g][k] = q[k].get();
  }
  block_csum4(r, ss[g], sc[g], t);
  if (t == 0) {
    for (int k = 0; k < 3; ++k) {
      const double a = (ss[g][k][0] + sc[g][k][0]) + pair[g][k];
      acc[3 * i + k] = a;
      if constexpr (kStep) a_new[3 * g + k] = a;
    }
    if (pot) pot[i] = (ss[g][3][0] + sc[g][3][0]) + pair[g][3];
  }
  if constexpr (kStep) {
    __syncthreads();                      // the positions have been read
    const int64_t k = kctr[0];
    const double h = dt * 0.5;
    const int e = threadIdx.x;
    if (e < 3 * kG) {
      double v = vel[e];
      if (k != 0) v = v + a_new[e] * h;
      v = v + a_new[e] * h;
      vel[e] = v;
      bpos[e] = bpos[e] + v * dt;
    }
    __syncthreads();
    if (e == 0) kctr[0] = k + 1;
  }
}

bool drift_smbh_fits(const tg_ctx *c, int64_t n, int32_t nb) {
  return nb >= 1 && nb <= kDriftSmbhMax && few_path(c->b.dpart_cap, n, nb, 1);
}

hipError_t launch_drift_smbh(tg_ctx *c, const tg_system *y, double dt, int64_t *next_k) {
  const int64_t n = y->n;
  const int32_t nb = y->n_bh;
  const int span = few_span(c->b.dpart_cap, n, nb);
  const int64_t bpt = (n + span - 1) / span;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)bpt), dim3(256), 0, c->stream, y->pos, y->vel,
                       y->frozen, n, dt, y->mass, y->eps, y->bh_pos, y->bh_eps, c->soft, span,
                       c->b.dpart);
  };
  switch (nb) {
    case 1: go(k_drift_smbh<1>); break;
    case 2: go(k_drift_smbh<2>); break;
    case 3: go(k_drift_smbh<3>); break;
    default: go(k_drift_smbh<4>); break;
  }
  auto finish = [&](auto kernel, int per) {
    hipLaunchKernelGGL(kernel, dim3(nb / per), dim3(256 * per), 0, c->stream, nb, (int)bpt,
                       c->b.dpart, y->bh_pos, y->bh_mass, y->bh_eps, nullptr, 1, c->soft,
                       y->bh_acc, y->bh_pot, y->bh_vel, dt, next_k);
  };
  if (!next_k) finish(k_smbh_finish<1, false>, 1);
  else if (nb == 1) finish(k_smbh_finish<1, true>, 1);
  else if (nb == 2) finish(k_smbh_finish<2, true>, 2);
  else if (nb == 3) finish(k_smbh_finish<3, true>, 3);
  else finish(k_smbh_finish<4, true>, 4);
  return hipGetLastError();
}

// From 64 SMBHs on their mutual pull has a kernel of its own (tiles).
bool smbh_sums_fit(const tg_ctx *c, int64_t max_stars, int32_t nb, int nseg) {
  return nb >= 1 && nb < 64 && few_path(c->b.dpart_cap, max_stars, nb, nseg);
}

hipError_t launch_smbh_sums(tg_ctx *c, const int64_t *dseg, const tg_system *y, int nseg,
                            int64_t max_stars) {
  const int32_t nb = y->n_bh;
  const int span = few_span(c->b.dpart_cap, max_stars, nb);
  const int64_t bpt = (max_stars + span - 1) / span;
  hipLaunchKernelGGL(k_direct_few, dim3((unsigned)bpt, (unsigned)nb), dim3(256), 0, c->stream,
                     y->pos, y->mass, nullptr, y->eps, y->bh_pos, y->bh_eps, (int64_t)nb, dseg,
                     dseg + (nseg + 1), nseg, 0, c->soft, span, c->b.dpart);
  hipLaunchKernelGGL((k_smbh_finish<1, false>), dim3(nb), dim3(256), 0, c->stream, nb, (int)bpt,
                     c->b.dpart, y->bh_pos, y->bh_mass, y->bh_eps, dseg + (nseg + 1), nseg,
                     c->soft, y->bh_acc, y->bh_pot, nullptr, 0.0, nullptr);
  return hipGetLastError();
}

template <int kT, bool kSelf, bool kSoft>
static void launch_tile_kernel(const DirectEnv &e, const double *spos, const double *sm,
                               const double *seps, double seps_all, int64_t ns,
                               const double *tpos, const double *teps, int64_t nt, int64_t nchunks,
                               int64_t chunk, int accumulate, double *acc, double *pot) {
  const dim3 grid((unsigned)((nt + 64 * kT - 1) / (64 * kT)), (unsigned)nchunks);
  hipLaunchKernelGGL((k_direct_tile<kT, kSelf, kSoft>), grid, dim3(256), 0, e.stream, spos, sm,
                     seps, seps_all, ns, tpos, teps, nt, chunk, accumulate, acc, pot, e.part);
}

static void launch_reduce(const DirectEnv &e, int64_t nt, int64_t nchunks, int accumulate,
                          double *acc, double *pot) {
  hipLaunchKernelGGL(k_direct_reduce, dim3((unsigned)std::min<int64_t>(nt, 4096)), dim3(256), 0,
                     e.stream, nt, (int)nchunks, accumulate, e.part, acc, pot);
}

static hipError_t launch_tiles(const DirectEnv &e, const DirectPlan &p, const double *spos,
                               const double *sm, const double *seps, double seps_all, int64_t ns,
                               const double *tpos, const double *teps, int64_t nt,
                               int self_pairs, int accumulate, double *acc, double *pot) {
  auto go = [&](auto self, auto soft) {
    constexpr bool kSelf = decltype(self)::value, kSoft = decltype(soft)::value;
    (p.lane_targets == 2 ? launch_tile_kernel<2, kSelf, kSoft>
                         : launch_tile_kernel<1, kSelf, kSoft>)(
        e, spos, sm, seps, seps_all, ns, tpos, teps, nt, p.nchunks, p.chunk, accumulate, acc, pot);
  };
  const std::true_type yes;
  const std::false_type no;
  if (self_pairs && e.soft) go(yes, yes);
  else if (self_pairs) go(yes, no);
  else if (e.soft) go(no, yes);
  else go(no, no);
  if (p.nchunks > 1 && p.block_reduce)
    launch_reduce(e, nt, p.nchunks, accumulate, acc, pot);
  else if (p.nchunks > 1)
    hipLaunchKernelGGL(k_direct_chunks, dim3((unsigned)((nt + 63) / 64)), dim3(64), 0, e.stream,
                       nt, (int)p.nchunks, accumulate, e.part, acc, pot);
  return hipGetLastError();
}

hipError_t launch_direct_env(const DirectEnv &e, const int64_t *dseg, const double *spos,
                             const double *sm, const double *seps, double seps_all,
                             const double *tpos, const double *teps, int64_t nt, int nseg,
                             int64_t max_seg_src, int self_pairs, int accumulate,
                             double *acc, double *pot) {
  if (nt == 0) return hipSuccess;
  const DirectPlan p = direct_plan(e.part_cap, max_seg_src, nt, nseg);
  if (p.path == DirectPath::kTile)
    return launch_tiles(e, p, spos, sm, seps, seps_all, max_seg_src, tpos, teps, nt, self_pairs,
                        accumulate, acc, pot);
  if (p.path == DirectPath::kFew) {
    hipLaunchKernelGGL(k_direct_few, dim3((unsigned)p.nchunks, (unsigned)nt), dim3(256), 0,
                       e.stream, spos, sm, seps, seps_all, tpos, teps, nt, dseg,
                       dseg + (nseg + 1), nseg, self_pairs, e.soft, (int)p.chunk, e.part);
    launch_reduce(e, nt, p.nchunks, accumulate, acc, pot);
    return hipGetLastError();
  }
  const int64_t total = nt * p.nchunks;
  const int g = (int)std::min<int64_t>((total + 255) / 256, 8192);
  hipLaunchKernelGGL(k_direct, dim3(g), dim3(256), 0, e.stream, spos, sm, seps,
                     seps_all, tpos, teps, nt, dseg, dseg + (nseg + 1), nseg,
                     p.chunk, (int)p.nchunks, self_pairs, accumulate, e.soft, acc, pot,
                     e.part);
  if (p.nchunks > 1) launch_reduce(e, nt, p.nchunks, accumulate, acc, pot);
  return hipGetLastError();
}

hipError_t launch_direct(tg_ctx *c, const int64_t *dseg, const double *spos,
                         const double *sm, const double *seps, double seps_all,
                         int64_t ns, const double *tpos,
                         const double *teps, int64_t nt, int nseg,
                         int64_t max_seg_src, int self_pairs, int accumulate,
                         double *acc, double *pot) {
  (void)ns;
  const DirectEnv e{c->stream, c->soft, c->b.dpart, c->b.dpart_cap};
  return launch_direct_env(e, dseg, spos, sm, seps, seps_all, tpos, teps, nt, nseg,
                           max_seg_src, self_pairs, accumulate, acc, pot);
}

}  // namespace tg
