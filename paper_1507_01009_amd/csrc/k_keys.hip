// Bounding cube per system, 21-bit Morton keys (or 42-bit, as two words),
// stable sort of (key, index), and the gather of positions into sorted
// order.  The sort takes one of three paths with the same result: systems of
// one tile at most are sorted by one block each, up to 1.5M particles (4M
// with two key words) sorted runs are merged, and larger sets take the radix
// passes described here.
//
// Work is cut into tiles of kSortTile consecutive particles that never cross
// a system boundary, so one launch handles every system of a batch.  One
// kernel counts each system's digits for all passes; in each pass a tile
// ranks its keys, publishes its per-digit counts and adds those of the
// earlier tiles of its own system (a look-back that ends at the system's
// first tile).  A key's place is the system's first index + the system's
// keys of smaller digits + the earlier tiles' keys of its digit + its rank
// in the tile, so the sort is segmented by system.
//
// Bit-exactness: the quantisation is t = x - lo, u = t * (2^21 / L), floor,
// clamp, with no contraction possible (one subtract, one multiply), and the
// division 2^21 / L is IEEE-rounded; keys and the stable permutation are
// therefore identical to any correct implementation of the same definition.
#include "tg_internal.h"

namespace tg {

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}

// Per-tile min/max of each coordinate; flags non-finite positions.
__global__ __launch_bounds__(256) void k_cube_part(const int32_t *__restrict__ gate, const double *__restrict__ pos,
                                                   const Tile *__restrict__ tiles,
                                                   double *__restrict__ part,
                                                   uint32_t *err) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  __shared__ double sh[4][6];
  const Tile t = tiles[blockIdx.x];
  double lo[3] = {INFINITY, INFINITY, INFINITY};
  double hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false;
#pragma unroll 4
  for (uint32_t i = t.start + threadIdx.x; i < t.end; i += 256u) {   // unrolled: loads in flight together
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double x = pos[3 * (size_t)i + k];
      bad |= !isfinite(x);
      lo[k] = fmin(lo[k], x);
      hi[k] = fmax(hi[k], x);
    }
  }
  if (bad) set_err(err, TG_ERR_NONFINITE);
  const unsigned lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lo[k] = wave_min(lo[k]);
    hi[k] = wave_max(hi[k]);
  }
  if (lane == 0)
    for (int k = 0; k < 3; ++k) { sh[w][k] = lo[k]; sh[w][3 + k] = hi[k]; }
  __syncthreads();
  if (threadIdx.x < 6) {
    double v = sh[0][threadIdx.x];
    for (int i = 1; i < 4; ++i)
      v = threadIdx.x < 3 ? fmin(v, sh[i][threadIdx.x]) : fmax(v, sh[i][threadIdx.x]);
    part[6 * (size_t)blockIdx.x + threadIdx.x] = v;
  }
}

// One block per system: lo = coordinate minimum, L = largest extent (1 if
// every particle coincides or the system is empty).
__global__ __launch_bounds__(256) void k_cube_final(const int32_t *__restrict__ gate, const double *__restrict__ part,
                                                    const uint32_t *__restrict__ sys_tile0,
                                                    double *__restrict__ cube) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  __shared__ double sh[4][6];
  const int s = blockIdx.x;
  const uint32_t a = sys_tile0[s], b = sys_tile0[s + 1];
  double lo[3] = {INFINITY, INFINITY, INFINITY};
  double hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (uint32_t t = a + threadIdx.x; t < b; t += 256u)
    for (int k = 0; k < 3; ++k) {
      lo[k] = fmin(lo[k], part[6 * (size_t)t + k]);
      hi[k] = fmax(hi[k], part[6 * (size_t)t + 3 + k]);
    }
  const unsigned lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  for (int k = 0; k < 3; ++k) { lo[k] = wave_min(lo[k]); hi[k] = wave_max(hi[k]); }
  if (lane == 0)
    for (int k = 0; k < 3; ++k) { sh[w][k] = lo[k]; sh[w][3 + k] = hi[k]; }
  __syncthreads();
  if (threadIdx.x == 0) {
    double L = 1.0, l3[3] = {0.0, 0.0, 0.0};
    if (b > a) {
      double h3[3];
      for (int k = 0; k < 3; ++k) {
        l3[k] = fmin(fmin(sh[0][k], sh[1][k]), fmin(sh[2][k], sh[3][k]));
        h3[k] = fmax(fmax(sh[0][3 + k], sh[1][3 + k]), fmax(sh[2][3 + k], sh[3][3 + k]));
      }
      L = 0.0;
      for (int k = 0; k < 3; ++k) L = fmax(L, h3[k] - l3[k]);
      if (L == 0.0) L = 1.0;
    }
    cube[4 * s + 0] = l3[0]; cube[4 * s + 1] = l3[1]; cube[4 * s + 2] = l3[2];
    cube[4 * s + 3] = L;
  }
}

// Spread the low 21 bits of v so that bit j lands on bit 3j.
__device__ __forceinline__ uint64_t spread3(uint64_t v) {
  v &= 0x1FFFFFull;
  v = (v | (v << 32)) & 0x1F00000000FFFFull;
  v = (v | (v << 16)) & 0x1F0000FF0000FFull;
  v = (v | (v << 8)) & 0x100F00F00F00F00Full;
  v = (v | (v << 4)) & 0x10C30C30C30C30C3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

// q = min(floor((x - lo) sigma), qmax), sigma = 2^bits / L.
__device__ __forceinline__ uint64_t quantise(double x, double lo, double sigma, uint64_t qmax) {
  double t = dsub(x, lo);
  double u = dmul(t, sigma);
  double f = floor(u);
  uint64_t q = f <= 0.0 ? 0ull : (uint64_t)f;
  return q > qmax ? qmax : q;
}

// Interleave the low 21 bits of three coordinates (x above y above z).
__device__ __forceinline__ uint64_t morton21(uint64_t qx, uint64_t qy, uint64_t qz) {
  return (spread3(qx) << 2) | (spread3(qy) << 1) | spread3(qz);
}

// 42 levels: 2^42 / L is 2^21 / L scaled by a power of two, so the top 21
// bits of each 42-bit coordinate are the 21-bit coordinate and the first
// key word is the 21-level key; the second word holds the last 21 digits.
__device__ __forceinline__ void keys42(const double *p, const double *c, double sigma,
                                       uint64_t &hi, uint64_t &lo) {
  const uint64_t m = (1ull << 42) - 1ull;
  const uint64_t qx = quantise(p[0], c[0], sigma, m), qy = quantise(p[1], c[1], sigma, m),
                 qz = quantise(p[2], c[2], sigma, m);
  hi = morton21(qx >> 21, qy >> 21, qz >> 21);
  lo = morton21(qx, qy, qz);
}

__device__ __forceinline__ int system_of_tile(const uint32_t *sys_tile0, int S, uint32_t t) {
  int lo_s = 0, hi_s = S - 1;     // last s with sys_tile0[s] <= t
  while (lo_s < hi_s) {
    int mid = (lo_s + hi_s + 1) >> 1;
    if (sys_tile0[mid] <= t) lo_s = mid; else hi_s = mid - 1;
  }
  return lo_s;
}

// Keys (x bit above y above z at every level) and the identity values;
// with kDeep the 42-level key's first word goes to key and its second to
// klo.
template <bool kDeep>
__global__ __launch_bounds__(256) void k_keys(const int32_t *__restrict__ gate, const double *__restrict__ pos,
                                              const Tile *__restrict__ tiles,
                                              const uint32_t *__restrict__ sys_tile0,
                                              int S, const double *__restrict__ cube,
                                              uint64_t *__restrict__ key,
                                              uint64_t *__restrict__ klo,
                                              uint32_t *__restrict__ val,
                                              uint32_t *__restrict__ zero, int64_t nzero) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  // the sort's counters and tile status, cleared for the sort that follows
  for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < nzero;
       w += (int64_t)gridDim.x * blockDim.x)
    zero[w] = 0u;
  const Tile t = tiles[blockIdx.x];
  const double *c = cube + 4 * system_of_tile(sys_tile0, S, blockIdx.x);
  const double sigma = (kDeep ? 4398046511104.0 : 2097152.0) / c[3];
#pragma unroll 4
  for (uint32_t i = t.start + threadIdx.x; i < t.end; i += 256u) {   // unrolled: loads in flight together
    if constexpr (kDeep) {
      uint64_t hi, lo;
      keys42(pos + 3 * (size_t)i, c, sigma, hi, lo);
      key[i] = hi;
      klo[i] = lo;
    } else {
      const uint64_t m = 0x1FFFFFull;
      key[i] = morton21(quantise(pos[3 * (size_t)i + 0], c[0], sigma, m),
                        quantise(pos[3 * (size_t)i + 1], c[1], sigma, m),
                        quantise(pos[3 * (size_t)i + 2], c[2], sigma, m));
    }
    val[i] = i;
  }
}

// 42 levels, after the sort: the second key words in sorted order, from
// the positions of the sorted particles (slo[r] for perm[r]).
__global__ void k_keys_lo_sorted(const int32_t *__restrict__ gate, const double *__restrict__ pos,
                                 const uint32_t *__restrict__ perm, int64_t n,
                                 const int64_t *__restrict__ sysoff, int S,
                                 const double *__restrict__ cube, uint64_t *__restrict__ slo) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n;
       r += (int64_t)gridDim.x * blockDim.x) {
    int a = 0, b = S - 1;          // last s with sysoff[s] <= r
    while (a < b) {
      const int mid = (a + b + 1) >> 1;
      if (sysoff[mid] <= r) a = mid; else b = mid - 1;
    }
    const double *c = cube + 4 * a;
    uint64_t hi, lo;
    keys42(pos + 3 * (size_t)perm[r], c, 4398046511104.0 / c[3], hi, lo);
    slo[r] = lo;
  }
}

// ---- radix sort, 9-bit digits ----------------------------------------
// Stable LSD sort of (key, index), 7 passes of 9 bits (the 63 bits of a key
// word), each system sorted on its own (tiles never straddle systems).  One
// counting kernel gives the digit totals of all passes per system; then one
// kernel per pass: a tile (taken in dispatch order from a ticket) ranks its
// keys in LDS, publishes its per-digit counts, adds up the counts of the
// earlier tiles of its system by looking back through their published words
// (each a flag and a count in one 32-bit word, written and read with
// agent-scope atomics), and scatters.  The lowest waiting tile never waits
// on a later one, so every wait ends; a wait is still bounded and reports
// TG_ERR_SORT if exceeded.
constexpr uint32_t kSortMask = kSortDigits - 1;
static_assert(kSortBits * kSortPasses == 63, "a key word holds 63 bits");
static_assert(kSortDigits == kSortThreads, "each thread owns one digit");
constexpr uint32_t kStAgg = 1u << 30, kStIncl = 2u << 30, kStVal = (1u << 30) - 1u;

__device__ __forceinline__ int tile_system(const uint32_t *sys_tile0, int S, uint32_t t) {
  int lo = 0, hi = S - 1;      // last s with sys_tile0[s] <= t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (sys_tile0[mid] <= t) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// cnt[s][p][d]: keys of system s with digit d in pass p (cleared beforehand)
__global__ __launch_bounds__(256) void k_sort_count(const int32_t *__restrict__ gate, const uint64_t *__restrict__ key,
                                                    const Tile *__restrict__ tiles,
                                                    const uint32_t *__restrict__ sys_tile0,
                                                    int S, uint32_t *__restrict__ cnt) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  __shared__ uint32_t c[kSortPasses][kSortDigits];
  const Tile t = tiles[blockIdx.x];
  const int s = tile_system(sys_tile0, S, blockIdx.x);
#pragma unroll
  for (int p = 0; p < kSortPasses; ++p) {
    c[p][threadIdx.x] = 0;
    c[p][threadIdx.x + 256] = 0;
  }
  __syncthreads();
  for (uint32_t i = t.start + threadIdx.x; i < t.end; i += 256u) {
    const uint64_t k = key[i];
#pragma unroll
    for (int p = 0; p < kSortPasses; ++p)
      atomicAdd(&c[p][(uint32_t)(k >> (kSortBits * p)) & kSortMask], 1u);
  }
  __syncthreads();
#pragma unroll
  for (int p = 0; p < kSortPasses; ++p) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t d = threadIdx.x + 256u * h;
      const uint32_t v = c[p][d];
      if (v) atomicAdd(&cnt[(size_t)(s * kSortPasses + p) * kSortDigits + d], v);
    }
  }
}

// Exclusive prefix sums over the block of two values per thread at once
// (one barrier).  The wave totals stay in sh; the caller's next barrier
// comes before sh is written again.
__device__ __forceinline__ void block_exclusive_scan2(uint32_t a, uint32_t b, uint2 *sh,
                                                      uint32_t &ea, uint32_t &eb) {
  const unsigned lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  uint32_t x = a, y = b;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t xo = __shfl_up(x, o, 64), yo = __shfl_up(y, o, 64);
    if (lane >= (unsigned)o) { x += xo; y += yo; }
  }
  if (lane == 63u) sh[w] = make_uint2(x, y);
  __syncthreads();
  uint32_t ba = 0, bb = 0;
  for (unsigned q = 0; q < w; ++q) { ba += sh[q].x; bb += sh[q].y; }
  ea = ba + x - a;
  eb = bb + y - b;
}

__global__ __launch_bounds__(kSortThreads) void k_sort_pass(const int32_t *__restrict__ gate, 
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout,
    const Tile *__restrict__ tiles, const uint32_t *__restrict__ sys_tile0, int S,
    const int64_t *__restrict__ sysoff, int pass, const uint32_t *__restrict__ cnt,
    uint32_t *status, uint32_t *ticket, uint32_t *err, uint32_t *__restrict__ rank) {
  constexpr int kWaves = kSortThreads / 64;
  if (gate && *gate <= 0) return;   // nothing active: skipped
  __shared__ uint64_t sk[kSortTile];
  __shared__ uint32_t sv[kSortTile];
  __shared__ uint32_t wcnt[kWaves][kSortDigits];
  __shared__ uint32_t loc_off[kSortDigits];
  __shared__ uint32_t glob_off[kSortDigits];
  __shared__ uint2 scan_sh[kWaves];
  __shared__ uint32_t s_tile;
  const unsigned tid = threadIdx.x, w = tid >> 6, lane = tid & 63u;
  const int shift = kSortBits * pass;
  if (tid == 0) s_tile = atomicAdd(ticket, 1u);
#pragma unroll
  for (int q = 0; q < kWaves; ++q) wcnt[q][tid] = 0;
  __syncthreads();
  const uint32_t tb = s_tile;
  const Tile t = tiles[tb];
  const int s = tile_system(sys_tile0, S, tb);
  const uint32_t first_tile = sys_tile0[s];
  const uint32_t n_in = t.end - t.start;
  // the system's count of digit tid (all tiles) and its first index
  const uint32_t gcnt = cnt[(size_t)(s * kSortPasses + pass) * kSortDigits + tid];
  const int64_t soff = sysoff[s];

  // wave w holds the tile's keys [64 kSortItems w, 64 kSortItems (w + 1)) in index order
  uint64_t k[kSortItems];
  uint32_t v[kSortItems], rk[kSortItems];
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t idx = 64u * kSortItems * w + 64u * r + lane;
    k[r] = idx < n_in ? kin[t.start + idx] : 0ull;
    v[r] = idx < n_in ? vin[t.start + idx] : 0u;
  }
  // stable ranks inside each wave: rounds of 64 keys in index order, peers
  // of equal digit found with ballots, counts kept in the wave's own LDS row
  // (one wave's LDS accesses execute in order: no barrier between rounds)
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t idx = 64u * kSortItems * w + 64u * r + lane;
    const bool valid = idx < n_in;
    const uint32_t d = (uint32_t)(k[r] >> shift) & kSortMask;
    unsigned long long peers = __ballot(valid);
#pragma unroll
    for (int bit = 0; bit < kSortBits; ++bit) {
      const unsigned long long bb = __ballot((d >> bit) & 1u);
      peers &= ((d >> bit) & 1u) ? bb : ~bb;
    }
    const uint32_t lr = lanes_below(peers);
    const uint32_t base = valid ? wcnt[w][d] : 0u;
    rk[r] = base + lr;
    if (valid && lr == 0) wcnt[w][d] = base + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  // digit tid: counts of the waves -> their exclusive offsets in place
  uint32_t mine = 0;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) {
    const uint32_t cq = wcnt[q][tid];
    wcnt[q][tid] = mine;
    mine += cq;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t d = (uint32_t)(k[r] >> shift) & kSortMask;
    rk[r] += wcnt[w][d];
  }
  // publish this tile's count of digit tid
  uint32_t *st = status + (size_t)tb * kSortDigits + tid;
  __hip_atomic_store(st, (tb == first_tile ? kStIncl : kStAgg) | mine, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
  // before waiting on the predecessors: the digit starts inside the system
  // (counts of smaller digits) and inside the tile, and the tile's keys
  // placed in LDS in digit order
  uint32_t dbase, lbase;
  block_exclusive_scan2(gcnt, mine, scan_sh, dbase, lbase);
  loc_off[tid] = lbase;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t idx = 64u * kSortItems * w + 64u * r + lane;
    if (idx < n_in) {
      const uint32_t d = (uint32_t)(k[r] >> shift) & kSortMask;
      const uint32_t p = loc_off[d] + rk[r];
      sk[p] = k[r];
      sv[p] = v[r];
    }
  }
  // look back for the prefix of digit tid over the earlier tiles
  uint32_t prefix = 0;
  if (tb != first_tile) {
    // windows of up to 16 predecessors read at once; walk down from the
    // nearest, adding counts, until a tile that holds its inclusive prefix
    uint32_t q = tb;                 // tiles [first_tile, q) remain
    uint32_t spin = 0;
    for (;;) {
      constexpr int kW = 16;
      const uint32_t avail = min(q - first_tile, (uint32_t)kW);
      uint32_t x[kW];
#pragma unroll
      for (int j = 0; j < kW; ++j)
        x[j] = (uint32_t)j < avail
                   ? __hip_atomic_load(status + (size_t)(q - 1 - j) * kSortDigits + tid,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   : 0u;
      uint32_t used = 0;
      bool done = false;
#pragma unroll
      for (int j = 0; j < kW; ++j) {
        if (done || (uint32_t)j != used || used >= avail) continue;
        if ((x[j] >> 30) == 0u) continue;          // not published yet: poll again
        prefix += x[j] & kStVal;
        ++used;
        done = (x[j] & kStIncl) != 0u;
      }
      if (done) break;
      q -= used;                                   // q > first_tile: the first tile is inclusive
      if (used == 0) {
        if (++spin >= (1u << 18)) {
          set_err(err, TG_ERR_SORT);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __hip_atomic_store(st, kStIncl | (prefix + mine), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
  glob_off[tid] = (uint32_t)soff + dbase + prefix;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kSortItems; ++r) {
    const uint32_t idx = r * (uint32_t)kSortThreads + tid;
    if (idx < n_in) {
      const uint64_t kk = sk[idx];
      const uint32_t d = (uint32_t)(kk >> shift) & kSortMask;
      const uint32_t dst = glob_off[d] + (idx - loc_off[d]);
      kout[dst] = kk;
      vout[dst] = sv[idx];
      if (rank) rank[sv[idx]] = dst;   // last pass: caller index -> sorted position
    }
  }
}

// Sorted particles {x, y, z, m}; the masses come with them when the caller
// has them at build time (else the moments pass fills them in).
__global__ void k_gather(const int32_t *__restrict__ gate, const double *__restrict__ pos,
                         const double *__restrict__ mass, const uint32_t *__restrict__ rank,
                         int64_t n, double4 *__restrict__ spart, uint32_t *err) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  bool bad = false;
  // caller order in, sorted order out: the reads are coalesced, each
  // particle is one 32-byte write (reading the caller's arrays in sorted
  // order would fetch a cache line per 24-byte position and 8-byte mass)
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double m = 0.0;
    if (mass) {
      m = mass[i];
      bad |= !(m > 0.0) || !isfinite(m);
    }
    spart[rank[i]] = make_double4(pos[3 * (size_t)i], pos[3 * (size_t)i + 1],
                                  pos[3 * (size_t)i + 2], m);
  }
  if (bad) set_err(err, TG_ERR_MASS);
}

hipError_t launch_cube_keys(tg_ctx *c, const double *pos) {
  Buffers &b = c->b;
  const int nt = (int)c->n_tiles;
  if (nt > 0)
    hipLaunchKernelGGL(k_cube_part, dim3(nt), dim3(256), 0, c->stream, c->gate, pos,
                       b.tiles, b.cube_part, b.err);
  hipLaunchKernelGGL(k_cube_final, dim3(c->S), dim3(256), 0, c->stream, c->gate,
                     b.cube_part, b.sys_tile0, b.cube);
  // the sort takes its input from the second buffers (an odd number of
  // passes leaves the result in the first)
  if (nt > 0 && c->max_level > kMaxLevel)
    // first words in caller order to key[0], second words to klo[1] (sorted first)
    hipLaunchKernelGGL(k_keys<true>, dim3(nt), dim3(256), 0, c->stream, c->gate, pos, b.tiles,
                       b.sys_tile0, c->S, b.cube, b.key[0], b.klo[1], b.val[1], b.hist,
                       sort_hist_words(c->S, nt));
  else if (nt > 0)
    hipLaunchKernelGGL(k_keys<false>, dim3(nt), dim3(256), 0, c->stream, c->gate, pos, b.tiles,
                       b.sys_tile0, c->S, b.cube, b.key[1], nullptr, b.val[1], b.hist,
                       sort_hist_words(c->S, nt));
  return hipGetLastError();
}

// The passes of a sort whose input is in (kb, vb): passes alternate
// between the two buffer pairs and the result ends in (ka, va).
// rank (may be null): the last pass also writes each caller index's sorted
// position.
static hipError_t sort_passes(tg_ctx *c, uint64_t *ka, uint32_t *va, uint64_t *kb, uint32_t *vb,
                              uint32_t *rank) {
  static_assert(kSortPasses % 2 == 1, "the input starts in the second buffers");
  Buffers &b = c->b;
  const int nt = (int)c->n_tiles;
  // [tickets | pad | counts [S][passes][digits] | status [passes][nt][digits]],
  // all zero: cleared by the kernel before the sort (k_keys, k_gather_hi)
  uint32_t *tickets = b.hist, *cnt = b.hist + kSortStatusBase;
  uint32_t *status = cnt + (size_t)c->S * kSortPasses * kSortDigits;
  hipLaunchKernelGGL(k_sort_count, dim3(nt), dim3(256), 0, c->stream, c->gate, kb, b.tiles,
                     b.sys_tile0, c->S, cnt);
  uint64_t *k2[2] = {ka, kb};
  uint32_t *v2[2] = {va, vb};
  for (int pass = 0; pass < kSortPasses; ++pass) {
    const int dst = pass & 1, src = dst ^ 1;
    hipLaunchKernelGGL(k_sort_pass, dim3(nt), dim3(kSortThreads), 0, c->stream, c->gate, k2[src],
                       v2[src], k2[dst], v2[dst], b.tiles, b.sys_tile0, c->S, b.sysoff, pass,
                       cnt, status + (size_t)pass * kSortDigits * nt, tickets + pass,
                       b.err, pass == kSortPasses - 1 ? rank : nullptr);
  }
  return hipGetLastError();
}

// 42 levels, between the two sort phases: first words in the order of the
// first phase (sorted by the second word) and that order itself, both into
// the second buffers where the next phase starts.
__global__ void k_gather_hi(const int32_t *__restrict__ gate, const uint64_t *__restrict__ hi,
                            const uint32_t *__restrict__ perm, int64_t n,
                            uint64_t *__restrict__ kout, uint32_t *__restrict__ vout,
                            uint32_t *__restrict__ zero, int64_t nzero) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  // the sort's counters and tile status, cleared for the second sort
  for (int64_t w = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; w < nzero;
       w += (int64_t)gridDim.x * blockDim.x)
    zero[w] = 0u;
  for (int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; r < n;
       r += (int64_t)gridDim.x * blockDim.x) {
    const uint32_t p = perm[r];
    kout[r] = hi[p];
    vout[r] = p;
  }
}

hipError_t launch_sort(tg_ctx *c) {
  Buffers &b = c->b;
  const int nt = (int)c->n_tiles;
  if (nt == 0) return hipSuccess;
  if (c->max_level <= kMaxLevel)      // key[1] / val[1] -> key[0] / val[0]
    return sort_passes(c, b.key[0], b.val[0], b.key[1], b.val[1], b.rank);
  // 42 levels, least significant word first: sort by the second words,
  // carry the first words into that order, sort them (stable), then the
  // second words of the final order from the positions
  hipError_t e = sort_passes(c, b.klo[0], b.val[0], b.klo[1], b.val[1], nullptr);
  if (e != hipSuccess) return e;
  const int g = (int)std::min<int64_t>((c->n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_gather_hi, dim3(g), dim3(256), 0, c->stream, c->gate, b.key[0],
                     b.val[0], c->n, b.key[1], b.val[1], b.hist, sort_hist_words(c->S, nt));
  return sort_passes(c, b.key[0], b.val[0], b.key[1], b.val[1], b.rank);
}

// 42 levels: the second key words of the sorted particles (klo[0]).
hipError_t launch_keys_lo(tg_ctx *c, const double *pos) {
  Buffers &b = c->b;
  if (c->max_level <= kMaxLevel || c->n == 0) return hipSuccess;
  const int g = (int)std::min<int64_t>((c->n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_keys_lo_sorted, dim3(g), dim3(256), 0, c->stream, c->gate, pos,
                     b.val[0], c->n, b.sysoff, c->S, b.cube, b.klo[0]);
  return hipGetLastError();
}

hipError_t launch_gather(tg_ctx *c, const double *pos, const double *mass) {
  if (c->n == 0) return hipSuccess;
  int g = (int)std::min<int64_t>((c->n + 255) / 256, 4096);
  hipLaunchKernelGGL(k_gather, dim3(g), dim3(256), 0, c->stream, c->gate, pos, mass,
                     c->b.rank, c->n, c->b.spart, c->b.err);
  return hipGetLastError();
}

// ---- systems of at most one tile each --------------------------------
// Everything up to the sorted particles in one launch, one block per system:
// bounding cube, keys, stable sort, gather and common digits.  The general
// path needs 12 launches for this (17 with 42 levels), and at a few thousand
// particles each of them is 2 to 6 us of launch gaps and memory latency with
// next to no work.  Here positions stay in registers and the keys in LDS,
// where a pass moves only 16-bit indices: each wave ranks its own run of
// indices with ballots as k_sort_pass does, 256 threads turn the waves' counts
// of two digits each into offsets (16-bit halves: no count exceeds 4096), and
// the indices are placed; three barriers a pass.  Bound by the latency of
// these steps: 18 us for 1021 particles and 40 for 4096, where the launches
// it replaces took 64 and 82 of an evaluation's 173 and 228 us (now 126, 185).
constexpr int kSysThreads = 1024, kSysWaves = kSysThreads / 64;
typedef uint16_t __attribute__((may_alias)) Half;   // also accessed as words

// Stable sort of the indices perm[0, n) (identity on entry) by the keys hi
// (and lo) in LDS; the block meets at a barrier before and after.
template <int kItems, bool kDeep>
__device__ __forceinline__ void lds_sort(const uint64_t *hi, const uint64_t *lo, uint16_t *perm,
                                         Half (*cnt)[kSortDigits], Half *base, uint32_t *wtot,
                                         uint32_t ns) {
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = tid & 63u;
  // wave w holds the indices [64 kItems w, 64 kItems (w + 1)) in order
  uint32_t *const cnt2 = reinterpret_cast<uint32_t *>(cnt[0]);
  for (int pass = kDeep ? -kSortPasses : 0; pass < kSortPasses; ++pass) {
    const uint64_t *word = kDeep && pass < 0 ? lo : hi;
    const int shift = kSortBits * (pass < 0 ? pass + kSortPasses : pass);
    uint32_t p[kItems], dg[kItems], rk[kItems];
    reinterpret_cast<uint4 *>(cnt[w])[lane] = make_uint4(0, 0, 0, 0);   // the wave's own row
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const uint32_t j = 64u * kItems * w + 64u * r + lane;
      p[r] = j < ns ? perm[j] : 0u;
      dg[r] = j < ns ? (uint32_t)(word[p[r]] >> shift) & kSortMask : 0u;
    }
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const bool valid = 64u * kItems * w + 64u * r + lane < ns;
      unsigned long long peers = __ballot(valid);
#pragma unroll
      for (int bit = 0; bit < kSortBits; ++bit) {
        const unsigned long long bb = __ballot((dg[r] >> bit) & 1u);
        peers &= ((dg[r] >> bit) & 1u) ? bb : ~bb;
      }
      const uint32_t lr = lanes_below(peers);
      const uint32_t b0 = valid ? cnt[w][dg[r]] : 0u;
      rk[r] = b0 + lr;
      if (valid && lr == 0) cnt[w][dg[r]] = (Half)(b0 + (uint32_t)__popcll(peers));
    }
    __syncthreads();
    if (w < kSortDigits / 128) {         // digits 2 tid and 2 tid + 1
      uint32_t run = 0;
#pragma unroll
      for (int q = 0; q < kSysWaves; ++q) {
        const uint32_t v = cnt2[q * (kSortDigits / 2) + tid];
        cnt2[q * (kSortDigits / 2) + tid] = run;
        run += v;
      }
      const uint32_t even = run & 0xffffu;
      uint32_t tot;
      const uint32_t e = wave_excl_scan(even + (run >> 16), tot);
      reinterpret_cast<uint32_t *>(base)[tid] = e | (e + even) << 16;
      if (lane == 0) wtot[w] = tot;
    }
    __syncthreads();
    uint32_t wb[kSortDigits / 128];      // digits before each 128
    wb[0] = 0;
#pragma unroll
    for (int q = 1; q < kSortDigits / 128; ++q) wb[q] = wb[q - 1] + wtot[q - 1];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
      const uint32_t g = dg[r] >> 7;
      const uint32_t lead = g == 0u ? wb[0] : g == 1u ? wb[1] : g == 2u ? wb[2] : wb[3];
      if (64u * kItems * w + 64u * r + lane < ns)
        perm[lead + base[dg[r]] + cnt[w][dg[r]] + rk[r]] = (uint16_t)p[r];
    }
    __syncthreads();
  }
}

template <int kItems, bool kDeep>
__global__ __launch_bounds__(kSysThreads) void k_sort_systems(
    const int32_t *__restrict__ gate, const double *__restrict__ pos,
    const double *__restrict__ mass, const int64_t *__restrict__ sysoff, int64_t n,
    double *__restrict__ cube, uint64_t *__restrict__ key, uint64_t *__restrict__ klo,
    uint32_t *__restrict__ val, uint32_t *__restrict__ rank, double4 *__restrict__ spart,
    uint8_t *__restrict__ d, uint32_t *__restrict__ gflag, uint32_t *err) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  constexpr int kN = kSysThreads * kItems;
  __shared__ uint64_t hi[kN];
  __shared__ uint64_t lo[kDeep ? kN : 1];
  __shared__ uint16_t perm[kN];
  // the waves' digit counts; after the last pass the inverse of perm
  __shared__ __align__(16) Half cnt[kSysWaves][kSortDigits];
  __shared__ __align__(16) Half base[kSortDigits];
  __shared__ uint32_t wtot[kSortDigits / 128];
  __shared__ double sh[kSysWaves][6];
  __shared__ double box[6];
  static_assert(kN <= kSysWaves * kSortDigits, "the inverse fits the counts");
  const uint32_t tid = threadIdx.x, w = tid >> 6, lane = tid & 63u;
  const int s = blockIdx.x;
  const uint32_t a = (uint32_t)sysoff[s], ns = (uint32_t)(sysoff[s + 1] - sysoff[s]);
  if (s == 0 && tid < 64u) d[n + tid] = 0;
  if (gflag && s == 0 && tid == 64u) gflag[n] = 0u;

  // positions and masses (thread: particles tid, tid + 1024, ...), bounding cube
  double x[kItems][3], m[kItems];
  double l3[3] = {INFINITY, INFINITY, INFINITY}, h3[3] = {-INFINITY, -INFINITY, -INFINITY};
  bool bad = false, bad_mass = false;
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t i = (uint32_t)(kSysThreads * r) + tid;
    const bool in = i < ns;
    const size_t g = (size_t)a + i;
#pragma unroll
    for (int k = 0; k < 3; ++k) x[r][k] = in ? pos[3 * g + k] : 0.0;
    m[r] = in && mass ? mass[g] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    if ((uint32_t)(kSysThreads * r) + tid >= ns) continue;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      bad |= !isfinite(x[r][k]);
      l3[k] = fmin(l3[k], x[r][k]);
      h3[k] = fmax(h3[k], x[r][k]);
    }
    if (mass) bad_mass |= !(m[r] > 0.0) || !isfinite(m[r]);
  }
  if (bad) set_err(err, TG_ERR_NONFINITE);
  if (bad_mass) set_err(err, TG_ERR_MASS);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    l3[k] = wave_min(l3[k]);
    h3[k] = wave_max(h3[k]);
  }
  if (lane == 0)
    for (int k = 0; k < 3; ++k) { sh[w][k] = l3[k]; sh[w][3 + k] = h3[k]; }
  __syncthreads();
  if (tid < 6u) {
    double v = sh[0][tid];
    for (int q = 1; q < kSysWaves; ++q) v = tid < 3u ? fmin(v, sh[q][tid]) : fmax(v, sh[q][tid]);
    box[tid] = v;
  }
  __syncthreads();
  double c[4] = {0.0, 0.0, 0.0, 1.0};
  if (ns > 0) {
    double L = 0.0;
    for (int k = 0; k < 3; ++k) {
      c[k] = box[k];
      L = fmax(L, box[3 + k] - box[k]);
    }
    c[3] = L == 0.0 ? 1.0 : L;
  }
  if (tid == 0)
    for (int k = 0; k < 4; ++k) cube[4 * s + k] = c[k];
  const double sigma = (kDeep ? 4398046511104.0 : 2097152.0) / c[3];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t i = (uint32_t)(kSysThreads * r) + tid;
    if (i >= ns) continue;
    if constexpr (kDeep) {
      keys42(x[r], c, sigma, hi[i], lo[i]);
    } else {
      const uint64_t q = 0x1FFFFFull;
      hi[i] = morton21(quantise(x[r][0], c[0], sigma, q), quantise(x[r][1], c[1], sigma, q),
                       quantise(x[r][2], c[2], sigma, q));
    }
    perm[i] = (uint16_t)i;
  }
  __syncthreads();

  lds_sort<kItems, kDeep>(hi, lo, perm, &cnt[0], base, wtot, ns);

  Half *const inv = &cnt[0][0];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t j = (uint32_t)(kSysThreads * r) + tid;
    if (j >= ns) continue;
    const uint32_t p = perm[j], g = a + j;
    const uint64_t k = hi[p];
    key[g] = k;
    val[g] = a + p;
    if (gflag) gflag[g] = 0u;
    uint32_t eq = 0;
    if (j > 0u) {
      const uint32_t q = perm[j - 1u];
      eq = common_digits(hi[q], k);
      if constexpr (kDeep)
        if (eq == 21u) eq += common_digits(lo[q], lo[p]);
    }
    d[g] = (uint8_t)eq;
    if constexpr (kDeep) klo[g] = lo[p];
    inv[p] = (Half)j;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t i = (uint32_t)(kSysThreads * r) + tid;
    if (i >= ns) continue;
    const uint32_t g = a + inv[i];
    rank[a + i] = g;
    spart[g] = make_double4(x[r][0], x[r][1], x[r][2], m[r]);
  }
}

// Taken when no system exceeds a sort tile (4096): the positions and keys of
// one system have to fit one block.  Largest systems of up to 1024 particles
// take the kernel with one particle per thread, whose passes have a quarter
// of the ranking rounds.
hipError_t launch_sort_systems(tg_ctx *c, const double *pos, const double *mass) {
  Buffers &b = c->b;
  const bool deep = c->max_level > kMaxLevel;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(c->S), dim3(kSysThreads), 0, c->stream, c->gate, pos, mass,
                       b.sysoff, c->n, b.cube, b.key[0], b.klo[0], b.val[0], b.rank, b.spart,
                       b.lcp, flat_groups(c) ? nullptr : b.gflag, b.err);
  };
  if (c->max_sys <= kSysThreads)
    deep ? go(k_sort_systems<1, true>) : go(k_sort_systems<1, false>);
  else
    deep ? go(k_sort_systems<4, true>) : go(k_sort_systems<4, false>);
  return hipGetLastError();
}

// ---- larger systems: sorted runs, then merges ---------------------------
// k_sort_runs forms the keys of kRun particles and sorts them in LDS;
// each round of k_merge_runs then merges groups of kWays runs of a system.
// A block of the merge moves kMergeChunk consecutive keys of one run: where
// its first and last key fall in the other runs is found by one wave each
// (64 probes a step), the keys between are staged in LDS, and every thread
// counts the ones before its own key.  Own index + counts is the place, and
// ties go to the earlier run, so the order is that of the stable sort.  A
// chunk that spans more than kMergeKeys keys of the other runs (a run that
// lies inside a gap of another) searches them in memory.
//
// One radix pass costs 10 to 12 us however few tiles it has (ticket, ranks,
// look-back, scatter), seven of them and the count 100 us at 131072
// particles, the runs and three rounds 51.  A round's cost grows with the
// keys read (each chunk reads its part of kWays runs) and reaches 30 us at
// 1048576, where five rounds equal the radix passes.  Eight ways were 5% and
// 16 ways 40% slower at that size and no faster below (more searches per
// key); runs of 4096 save no round at 131072 and cost 13 us more.
constexpr int kRun = 2048, kWays = 4, kMergeChunk = 512, kMergeKeys = 6 * kMergeChunk;
static_assert(kSortTile % kRun == 0 && kRun % kMergeChunk == 0, "chunks never cross runs or tiles");

// Cube of the system with tiles [t0, t1) from their coordinate ranges, in
// every thread (one barrier).
template <int kBlock>
__device__ __forceinline__ void cube_of(const double *__restrict__ part, uint32_t t0, uint32_t t1,
                                        double (*sh)[6], double *c) {
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (uint32_t t = t0 + threadIdx.x; t < t1; t += kBlock)
    for (int k = 0; k < 3; ++k) {
      lo[k] = fmin(lo[k], part[6 * (size_t)t + k]);
      hi[k] = fmax(hi[k], part[6 * (size_t)t + 3 + k]);
    }
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  const uint32_t nw = min((uint32_t)(kBlock / 64), (t1 - t0 + 63u) / 64u);
  if (w < nw) {
    for (int k = 0; k < 3; ++k) { lo[k] = wave_min(lo[k]); hi[k] = wave_max(hi[k]); }
    if (lane == 0)
      for (int k = 0; k < 3; ++k) { sh[w][k] = lo[k]; sh[w][3 + k] = hi[k]; }
  }
  __syncthreads();
  double L = 0.0;
  for (int k = 0; k < 3; ++k) {
    double a = sh[0][k], b = sh[0][3 + k];
    for (uint32_t q = 1; q < nw; ++q) { a = fmin(a, sh[q][k]); b = fmax(b, sh[q][3 + k]); }
    c[k] = a;
    L = fmax(L, b - a);
  }
  c[3] = L == 0.0 ? 1.0 : L;
}

// Half-tiles of keys in sorted order; also writes the cubes.
template <bool kDeep>
__global__ __launch_bounds__(kSysThreads) void k_sort_runs(
    const int32_t *__restrict__ gate, const double *__restrict__ pos,
    const Tile *__restrict__ tiles, const uint32_t *__restrict__ sys_tile0, int S,
    const double *__restrict__ part, double *__restrict__ cube, uint64_t *__restrict__ key,
    uint64_t *__restrict__ klo, uint32_t *__restrict__ val) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  constexpr int kItems = kRun / kSysThreads;
  __shared__ uint64_t hi[kRun];
  __shared__ uint64_t lo[kDeep ? kRun : 1];
  __shared__ uint16_t perm[kRun];
  __shared__ __align__(16) Half cnt[kSysWaves][kSortDigits];
  __shared__ __align__(16) Half base[kSortDigits];
  __shared__ uint32_t wtot[kSortDigits / 128];
  __shared__ double sh[kSysWaves][6];
  constexpr uint32_t kPer = kSortTile / kRun;
  const uint32_t tid = threadIdx.x, tb = blockIdx.x / kPer;
  const Tile t = tiles[tb];
  const uint32_t a = t.start + (blockIdx.x % kPer) * kRun;
  if (blockIdx.x == 0)                 // empty systems
    for (int s = tid; s < S; s += kSysThreads)
      if (sys_tile0[s] == sys_tile0[s + 1])
        for (int k = 0; k < 4; ++k) cube[4 * s + k] = k == 3 ? 1.0 : 0.0;
  if (a >= t.end) return;
  const uint32_t ns = min((uint32_t)kRun, t.end - a);
  double x[kItems][3];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t i = (uint32_t)(kSysThreads * r) + tid;
#pragma unroll
    for (int k = 0; k < 3; ++k) x[r][k] = i < ns ? pos[3 * ((size_t)a + i) + k] : 0.0;
  }
  const int s = tile_system(sys_tile0, S, tb);
  const uint32_t t0 = sys_tile0[s];
  double c[4];
  cube_of<kSysThreads>(part, t0, sys_tile0[s + 1], sh, c);
  if (a == tiles[t0].start && tid < 4u)
    cube[4 * s + tid] = tid == 0u ? c[0] : tid == 1u ? c[1] : tid == 2u ? c[2] : c[3];
  const double sigma = (kDeep ? 4398046511104.0 : 2097152.0) / c[3];
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t i = (uint32_t)(kSysThreads * r) + tid;
    if (i >= ns) continue;
    if constexpr (kDeep) {
      keys42(x[r], c, sigma, hi[i], lo[i]);
    } else {
      const uint64_t q = 0x1FFFFFull;
      hi[i] = morton21(quantise(x[r][0], c[0], sigma, q), quantise(x[r][1], c[1], sigma, q),
                       quantise(x[r][2], c[2], sigma, q));
    }
    perm[i] = (uint16_t)i;
  }
  __syncthreads();
  lds_sort<kItems, kDeep>(hi, lo, perm, cnt, base, wtot, ns);
#pragma unroll
  for (int r = 0; r < kItems; ++r) {
    const uint32_t j = (uint32_t)(kSysThreads * r) + tid;
    if (j >= ns) continue;
    const uint32_t p = perm[j], g = a + j;
    key[g] = hi[p];
    if constexpr (kDeep) klo[g] = lo[p];
    val[g] = a + p;
  }
}

// key k before e, or (or_equal) not after it
template <bool kDeep>
__device__ __forceinline__ bool key_before(uint64_t kh, uint64_t kl, uint64_t eh, uint64_t el,
                                           bool or_equal) {
  if constexpr (kDeep) {
    if (kh != eh) return kh < eh;
    return or_equal ? kl <= el : kl < el;
  } else {
    return or_equal ? kh <= eh : kh < eh;
  }
}

// Number of keys of run [r0, r0 + m) before e, found by one wave: 64 probes a round.
template <bool kDeep>
__device__ __forceinline__ uint32_t wave_bound(const uint64_t *__restrict__ kin,
                                               const uint64_t *__restrict__ lin, uint32_t r0,
                                               uint32_t m, uint64_t eh, uint64_t el,
                                               bool or_equal) {
  const uint32_t lane = threadIdx.x & 63u;
  uint32_t lo = 0;
  while (m > 0) {
    const uint32_t step = (m + 63u) / 64u;
    const uint32_t q = r0 + lo + min(step * (lane + 1u), m) - 1u;
    const bool p = key_before<kDeep>(kin[q], kDeep ? lin[q] : 0ull, eh, el, or_equal);
    const uint32_t c = (uint32_t)__popcll(__ballot(p));
    if (c == 64u) return lo + m;
    lo += c * step;
    m = min(step, m - c * step) - 1u;
  }
  return lo;
}

// One round: groups of kWays runs of `run` keys (the last of a system shorter).
template <bool kDeep>
__global__ __launch_bounds__(kMergeChunk) void k_merge_runs(
    const int32_t *__restrict__ gate, const Tile *__restrict__ tiles,
    const uint32_t *__restrict__ sys_tile0, int S, const int64_t *__restrict__ sysoff,
    uint32_t run, const uint64_t *__restrict__ kin, const uint64_t *__restrict__ lin,
    const uint32_t *__restrict__ vin, uint64_t *__restrict__ kout, uint64_t *__restrict__ lout,
    uint32_t *__restrict__ vout, uint32_t *__restrict__ rank) {
  if (gate && *gate <= 0) return;   // nothing active: skipped
  __shared__ uint64_t sk[kMergeKeys];
  __shared__ uint64_t sl[kDeep ? kMergeKeys : 1];
  __shared__ uint32_t lo_sh[kWays], hi_sh[kWays];
  constexpr uint32_t kPer = kSortTile / kMergeChunk, kWaves = kMergeChunk / 64;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, tb = blockIdx.x / kPer;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const Tile t = tiles[tb];
  const uint32_t a = t.start + (blockIdx.x % kPer) * kMergeChunk;
  if (a >= t.end) return;
  const uint32_t m = min((uint32_t)kMergeChunk, t.end - a);
  const int s = tile_system(sys_tile0, S, tb);
  const uint32_t so = (uint32_t)sysoff[s], se = (uint32_t)sysoff[s + 1];
  const uint32_t mine = (a - so) / run;              // run of the system, of its group of kWays
  const uint32_t g0 = mine - mine % kWays, own = mine - g0;
  const uint32_t gs = so + g0 * run;
  const uint32_t ge = (uint32_t)min<uint64_t>(se, gs + (uint64_t)kWays * run);   // end of the group
  // the own key, and where the chunk's first and last keys fall in the other runs
  const uint32_t i = a + min(tid, m - 1u);
  const uint64_t eh = kin[i], el = kDeep ? lin[i] : 0ull;
  const uint32_t v = vin[i];
  const uint64_t fh = kin[a], fl = kDeep ? lin[a] : 0ull;
  const uint64_t zh = kin[a + m - 1u], zl = kDeep ? lin[a + m - 1u] : 0ull;
  for (uint32_t q = w; q < 2u * kWays; q += kWaves) {   // a wave per run and end
    const uint32_t r = q % kWays;
    const bool last = q >= kWays;
    const uint32_t r0 = (uint32_t)min<uint64_t>(ge, gs + (uint64_t)r * run), len = min(ge - r0, run);
    uint32_t x = 0;
    if (r != own && len > 0u)
      x = wave_bound<kDeep>(kin, lin, r0, len, last ? zh : fh, last ? zl : fl, r < own);
    if (lane == 0) (last ? hi_sh : lo_sh)[r] = x;
  }
  __syncthreads();
  uint32_t lo[kWays], len[kWays], off[kWays], tot = 0, longest = 0, dst = i - mine * run - so;
#pragma unroll
  for (int r = 0; r < kWays; ++r) {
    lo[r] = (uint32_t)__builtin_amdgcn_readfirstlane((int)lo_sh[r]);
    len[r] = (uint32_t)__builtin_amdgcn_readfirstlane((int)hi_sh[r]) - lo[r];
    off[r] = tot;
    tot += len[r];
    longest = max(longest, len[r]);
    dst += lo[r];
  }
  const bool fits = tot <= (uint32_t)kMergeKeys;
  if (fits) {
#pragma unroll
    for (int r = 0; r < kWays; ++r) {
      const uint32_t g = gs + (uint32_t)r * run + lo[r];
      for (uint32_t q = tid; q < len[r]; q += kMergeChunk) {
        sk[off[r] + q] = kin[g + q];
        if constexpr (kDeep) sl[off[r] + q] = lin[g + q];
      }
    }
    __syncthreads();
  }
  if (longest > 0u) {
    uint32_t p[kWays];
#pragma unroll
    for (int r = 0; r < kWays; ++r) p[r] = 0;
    // the searches of all runs step by step together
    for (uint32_t step = 1u << (31 - __clz((int)longest)); step > 0u; step >>= 1) {
#pragma unroll
      for (int r = 0; r < kWays; ++r) {
        const uint32_t q = p[r] + step;
        if (q <= len[r]) {
          uint64_t kh, kl = 0ull;
          if (fits) {
            kh = sk[off[r] + q - 1u];
            if constexpr (kDeep) kl = sl[off[r] + q - 1u];
          } else {
            const uint32_t g = gs + (uint32_t)r * run + lo[r] + q - 1u;
            kh = kin[g];
            if constexpr (kDeep) kl = lin[g];
          }
          if (key_before<kDeep>(kh, kl, eh, el, (uint32_t)r < own)) p[r] = q;
        }
      }
    }
#pragma unroll
    for (int r = 0; r < kWays; ++r) dst += p[r];
  }
  if (tid < m) {
    dst += gs;
    kout[dst] = eh;
    if constexpr (kDeep) lout[dst] = el;
    vout[dst] = v;
    if (rank) rank[v] = dst;   // last round: caller index -> sorted position
  }
}

// Whether the sort merges runs (else radix passes): the runs and rounds took
// as long as the radix passes at 1.5M particles with one key word (a step of
// 131072 stars 740 -> 686 us, 1.5M 5670 -> 5660, 3M 11210 -> 11330) and at
// 4M with two, where the radix sort runs twice (500000 stars 2605 -> 2428 us,
// 1.5M 8190 -> 8003, 4M 22.6 ms both).
bool sort_merges(const tg_ctx *c) {
  return c->n > 0 && c->n <= (c->max_level > kMaxLevel ? 1 << 22 : 3 << 19);
}

hipError_t launch_sort_merge(tg_ctx *c, const double *pos) {
  Buffers &b = c->b;
  const bool deep = c->max_level > kMaxLevel;
  const int nt = (int)c->n_tiles;
  hipLaunchKernelGGL(k_cube_part, dim3(nt), dim3(256), 0, c->stream, c->gate, pos,
                     b.tiles, b.cube_part, b.err);
  int rounds = 0;
  for (int64_t len = kRun; len < c->max_sys; len *= kWays) ++rounds;
  int at = rounds & 1;                 // the last round ends in the first buffers
  auto runs = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nt * (kSortTile / kRun)), dim3(kSysThreads), 0, c->stream,
                       c->gate, pos, b.tiles, b.sys_tile0, c->S, b.cube_part, b.cube, b.key[at],
                       b.klo[at], b.val[at]);
  };
  deep ? runs(k_sort_runs<true>) : runs(k_sort_runs<false>);
  int64_t len = kRun;
  for (int q = 0; q < rounds; ++q, at ^= 1, len *= kWays) {
    auto merge = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(nt * (kSortTile / kMergeChunk)), dim3(kMergeChunk), 0,
                         c->stream, c->gate, b.tiles, b.sys_tile0, c->S, b.sysoff, (uint32_t)len,
                         b.key[at], b.klo[at], b.val[at], b.key[at ^ 1], b.klo[at ^ 1],
                         b.val[at ^ 1], q == rounds - 1 ? b.rank : nullptr);
    };
    deep ? merge(k_merge_runs<true>) : merge(k_merge_runs<false>);
  }
  return hipGetLastError();
}

}  // namespace tg
