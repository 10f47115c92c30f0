// 3D traveltime tiles (eq 31 over the 3D forward star, class-pair edge costs
// of eqs 27-30) for gfx950: the tile relaxation of trace.hip carried to 3D.
//
// Every grid of the batch is cut into TX x TX x TZ tiles.  A workgroup (one
// thread per tile node) owns one (problem, tile) per round: it stages the
// tile plus an R-wide halo of traveltimes and class ids in LDS, pulls the
// strips facing the neighbour tiles whose halo part changed (all nodes when
// asked), then pushes over a frontier of improved nodes (64-bit LDS atomic
// min and marks, wavefront ballot compaction) until the tile is locally
// converged.  The weights of the class pairs that the box holds are staged
// in LDS (a box rarely holds more than three classes, whatever K is).
//
// Nearly every node of an 8 x 8 x 8 tile lies within R = 3 of a face, so a
// visit is its pull: 512 nodes x 290 offsets, bound by LDS reads and their
// latency (weights by a sum of class codes, eight edges' reads in flight,
// three workgroups per compute unit).  121 x 121 x 61 nodes, 6 classes, 4
// fields: 15.0 -> 6.2 ms (0.65 -> 0.93 T edges/s, ordered tiles making 43
// instead of 68 thousand visits).
// Changed nodes within R of a face, edge or corner wake the neighbour tile
// across it (26 neighbours, the side travels with the flag); rounds repeat
// until one wakes nothing.  Every value written is the left-to-right FP64
// sum along some path and values only decrease, so the fixed point is the
// minimum over paths, bitwise what Dijkstra computes from the same weights.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <vector>

#include "chert.h"
#include "chert_internal.h"
#include "class_codes.h"
#include "grid_sync.h"

#pragma clang fp contract(off)

namespace chert {

namespace {

constexpr int kT3Threads = 1024;        // tiles of at most 1024 nodes
constexpr int kT3IterCap = 4096;        // push levels per visit before a full re-visit
constexpr int kT3Active = 1, kT3Full = 2, kT3Seed = 4;
constexpr int kT3SideShift = 3;         // bits 3 + s, s = (dz+1)*9 + (dy+1)*3 + (dx+1)
constexpr int kT3Self = 13;             // s of (0, 0, 0)
// LDS for the weights of a box's class pairs: three classes at radius 3
// (seven rows of 290 offsets), which with the 8 x 8 x 8 tile's 32 KiB leaves
// three workgroups per compute unit
constexpr size_t kT3WLdsBytes = 16 * 1024;
// Width of the tile ordering in tile sides (times the typical edge weight).
// Ordered rounds visit a tile fewer times (43,061 instead of 67,762 visits on
// a 121 x 121 x 61 grid, 4 fields), but a round holds fewer tiles, so only
// batches of more than twice the resident workgroups -- rounds that fill the
// device several times over -- take it: there 9.0 -> 6.9 ms, while 800 tiles
// (every visit of a round at once) went from 1.80 to 1.98 ms.  A quarter side:
// 6.94 ms, 32 rounds; this: 6.93, 30; half: 6.98, 29; one: 7.78, 29.
constexpr double kT3OrderSides = 0.35;
// Rounds that the ordering may take, some four times what it takes on layered
// models: whatever the weights' contrast, the rounds after these visit every
// active tile, no more of them than an unordered relaxation needs.
inline int order_cap(int span) { return 64 + 2 * span; }
constexpr int kT3PminStride = 16;  // one 128-byte line per shard
constexpr unsigned long long kT3Inf = 0x7ff0000000000000ull;

struct T3JobDev {
  int nx, ny, nz, K;
  int ntx, nty, ntz, pad;
  const int32_t* cls;
  const double* W;  // [2][K][K][n_off]
};

struct T3ProbDev {
  double* tau;
  int64_t src;
  int job, field, tile_base, pad;
};

struct T3Args {
  int tx, tz, R, n_off;
  int lx, lz;          // LDS box: lx x lx x lz (tile + 2R per axis)
  int n_prob, n_tiles;
  int w_classes;       // classes of a box whose pairs' weights fit in LDS
  uint32_t lx_magic, lxx_magic;  // q / lx = umulhi(q, lx_magic), q / lx^2 likewise
  const T3JobDev* jobs;
  const T3ProbDev* probs;
  const int32_t* off;  // [n_off] star offsets in cells of the LDS box
  int32_t* flags;    // [2][n_tiles] by round parity
  int32_t* list;     // [2][n_tiles] tiles active in a round
  int32_t* tile_prob;  // [n_tiles] problem of each tile
  int32_t* counter;  // [counter_words(max_rounds)]: list lengths, then tickets
  uint32_t* tick;    // [2][kTickWords] tickets of the per-round list walk, by round parity
  int32_t* err;
  unsigned long long* stats;  // [kStatSlots][16] shards of: [0] visits, [1] edges examined
  // Tile ordering: a tile woken with key k (the smallest changed border value
  // that woke it) is visited in a round before order_rounds only if k is within
  // `width` times its job's and field's typical edge weight of its problem's
  // smallest pending key; otherwise it stays active for a later round.
  // width 0: every active tile.
  double width;
  int order_rounds;
  double* typ;               // [n_jobs][2] typical edge weights (k_tile3_typ)
  unsigned long long* key;   // [2][n_tiles] keys (double bits) by round parity
  unsigned long long* pmin;  // [3][n_prob][shards][kT3PminStride] smallest key, by round mod 3
  int pmin_shards;
  // the caller's abort word (device view of pinned host memory, nullable)
  // and the device word recording that it was seen (persistent launch)
  const int32_t* abort_host;
  int32_t* abort_seen;
};

__device__ __forceinline__ unsigned long long dbits3(double x) {
  return (unsigned long long)__double_as_longlong(x);
}

__device__ __forceinline__ void frontier_add3(bool flag, int node, uint16_t* list, int* count) {
  const unsigned long long b = __ballot(flag);
  if (b == 0ull) return;
  const int lane = __lane_id();
  const int leader = __ffsll((long long)b) - 1;
  int base = 0;
  if (lane == leader) base = atomicAdd(count, __popcll(b));
  base = __shfl(base, leader);
  if (flag) list[base + __popcll(b & ((1ull << lane) - 1ull))] = (uint16_t)node;
}

// which neighbour tiles see interior node (x, y, z) in their halo
__device__ __forceinline__ int border_bits3(int x, int y, int z, int tx, int tz, int R) {
  int m = 0;
  for (int dz = -1; dz <= 1; ++dz) {
    const bool okz = dz == 0 || (dz < 0 && z < R) || (dz > 0 && z >= tz - R);
    if (!okz) continue;
    for (int dy = -1; dy <= 1; ++dy) {
      const bool oky = dy == 0 || (dy < 0 && y < R) || (dy > 0 && y >= tx - R);
      if (!oky) continue;
      for (int dx = -1; dx <= 1; ++dx) {
        if (dx == 0 && dy == 0 && dz == 0) continue;
        const bool okx = dx == 0 || (dx < 0 && x < R) || (dx > 0 && x >= tx - R);
        if (okx) m |= 1 << ((dz + 1) * 9 + (dy + 1) * 3 + (dx + 1));
      }
    }
  }
  return m;
}

// Does this visit pull interior node (x, y, z)?  The strips facing the
// neighbours whose halo part changed, or every node on a full visit.
__device__ __forceinline__ bool pulls3(int flag, int x, int y, int z, int tx, int tz, int R) {
  if (flag & kT3Full) return true;
  const int sides = (flag >> kT3SideShift) & 0x7ffffff;
  if (!sides) return false;
  const bool nx[3] = {x < R, true, x >= tx - R};
  const bool ny[3] = {y < R, true, y >= tx - R};
  const bool nz[3] = {z < R, true, z >= tz - R};
  for (int s = 0; s < 27; ++s)
    if (((sides >> s) & 1) && nx[s % 3] && ny[(s / 3) % 3] && nz[s / 9]) return true;
  return false;
}

__global__ void k_tile3_clear(int32_t* flags, int64_t n_flags, int32_t* counter, int n_counter,
                              int32_t* err, unsigned long long* stats, const T3ProbDev* probs,
                              int n_prob, int32_t* tile_prob, unsigned long long* key,
                              unsigned long long* pmin, int64_t n_pmin, int32_t* off,
                              const int32_t* ox, const int32_t* oy, const int32_t* oz, int n_off,
                              int lx) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  for (int64_t o = tid; o < n_off; o += (int64_t)gridDim.x * blockDim.x)
    off[o] = ox[o] + lx * (oy[o] + lx * oz[o]);
  for (int64_t t = tid; t < n_flags; t += (int64_t)gridDim.x * blockDim.x) key[t] = kT3Inf;
  // (round 0 visits the source tiles whatever its minimum: their key is 0)
  for (int64_t t = tid; t < n_pmin; t += (int64_t)gridDim.x * blockDim.x) pmin[t] = kT3Inf;
  for (int64_t t = tid; t < n_flags / 2; t += (int64_t)gridDim.x * blockDim.x) {
    int lo = 0, hi = n_prob - 1;  // the last problem whose first tile is not after t
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (probs[mid].tile_base <= t) lo = mid;
      else hi = mid - 1;
    }
    tile_prob[t] = lo;
  }
  for (int64_t t = tid; t < n_flags; t += (int64_t)gridDim.x * blockDim.x) flags[t] = 0;
  for (int64_t t = tid; t < n_counter; t += (int64_t)gridDim.x * blockDim.x) counter[t] = 0;
  if (tid < 64) err[tid] = 0;  // error word, barrier words, result, abort record
  for (int64_t t = tid; t < kStatSlots * kStatSlotU64; t += (int64_t)gridDim.x * blockDim.x)
    stats[t] = 0ull;
}

// The typical edge weight of (job blockIdx.x, field blockIdx.y): the mean of its
// classes' own positive finite weights, summed in a fixed order; +inf (no
// ordering) where there is none.  A mean, not the smallest weight: one nearly
// lossless class or one fine axis makes the smallest arbitrarily small against
// the keys, and every round then holds a tile or two.
constexpr int kTypThreads = 256;
__global__ void __launch_bounds__(kTypThreads) k_tile3_typ(T3Args a) {
  __shared__ double s_sum[kTypThreads];
  __shared__ int s_n[kTypThreads];
  const T3JobDev J = a.jobs[blockIdx.x];
  const int f = blockIdx.y, tid = threadIdx.x;
  double sum = 0.0;
  int n = 0;
  for (int64_t q = tid; q < (int64_t)J.K * a.n_off; q += kTypThreads) {
    const int64_t k = q / a.n_off, o = q - k * a.n_off;
    const double w = J.W[(((int64_t)f * J.K + k) * J.K + k) * a.n_off + o];
    if (w > 0.0 && w < INFINITY) {
      sum += w;
      ++n;
    }
  }
  s_sum[tid] = sum;
  s_n[tid] = n;
  for (int d = kTypThreads / 2; d >= 1; d >>= 1) {
    __syncthreads();
    if (tid < d) {
      s_sum[tid] += s_sum[tid + d];
      s_n[tid] += s_n[tid + d];
    }
  }
  if (tid == 0) a.typ[2 * blockIdx.x + f] = s_n[0] ? s_sum[0] / s_n[0] : INFINITY;
}

// activate the source tile of every problem
__global__ void k_tile3_seed(T3Args a) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.n_prob) return;
  const T3ProbDev P = a.probs[p];
  const T3JobDev J = a.jobs[P.job];
  const int sx = (int)(P.src % J.nx), sy = (int)((P.src / J.nx) % J.ny),
            sz = (int)(P.src / ((int64_t)J.nx * J.ny));
  const int T = P.tile_base + ((sz / a.tz) * J.nty + sy / a.tx) * J.ntx + sx / a.tx;
  a.flags[T] = kT3Active | kT3Seed;
  a.key[T] = 0ull;
  a.list[atomicAdd(&a.counter[0], 1)] = T;
}

struct T3Smem {
  double* val;     // [lx*lx*lz]
  double* W;       // [code_rows][n_off]
  uint16_t* cls;   // [lx*lx*lz] class of a cell: its code (kT3Lds) or its id
  uint16_t* list;  // frontier (interior LDS indices)
  uint8_t* mark;   // [lx*lx*lz] lowered at this level
};

__device__ __forceinline__ T3Smem carve3(const T3Args& a, double* base, int nbox) {
  T3Smem s;
  s.val = base;
  s.W = s.val + nbox;
  s.cls = (uint16_t*)(s.W + (a.w_classes ? (size_t)code_rows(a.w_classes) * a.n_off : 0));
  s.list = s.cls + nbox;
  s.mark = (uint8_t*)(s.list + a.tx * a.tx * a.tz);
  return s;
}

// Where a visit's edge weights come from (uniform over the workgroup): one
// class in the box, few enough to stage their pairs, or the global table.
enum { kT3Uniform = 0, kT3Lds = 1, kT3Global = 2 };

template <int SRC>
__device__ __forceinline__ double w3(const T3Smem& s, const double* Wf, int K, int n_off, int ki,
                                     int kj, int o) {
  if constexpr (SRC == kT3Uniform) return s.W[o];
  if constexpr (SRC == kT3Lds) return s.W[ki + kj + o];
  return Wf[((int64_t)ki * K + kj) * n_off + o];
}

// read-only memory of the launch, read with scalar loads where the index is
// uniform over the wavefront
typedef const __attribute__((address_space(4))) int32_t* const_i32;

// B in-edges of node ml from offset o on: all the values and classes first,
// then all the weights, so that one LDS latency serves the B of them.
template <int SRC, int B>
__device__ __forceinline__ double pull_block3(const T3Smem& s, const double* Wf, int K, int n_off,
                                              const const_i32 off, int ml, int kj, int o,
                                              double best) {
  double v[B], w[B];
  int k[B];
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const int ii = ml - off[o + u];
    k[u] = SRC == kT3Uniform ? 0 : s.cls[ii];
    v[u] = s.val[ii];
  }
#pragma unroll
  for (int u = 0; u < B; ++u) w[u] = w3<SRC>(s, Wf, K, n_off, k[u], kj, o + u);
#pragma unroll
  for (int u = 0; u < B; ++u) {
    const double cand = __dadd_rn(v[u], w[u]);
    if (cand < best) best = cand;
  }
  return best;
}

// The pull of one node over its whole star (cells outside the grid hold
// +inf).  The offsets are uniform over the workgroup (scalar loads).
template <int SRC>
__device__ __forceinline__ double pull3(const T3Args& a, const T3Smem& s, const double* Wf, int K,
                                        int ml) {
  const const_i32 off = (const_i32)(uintptr_t)a.off;
  const int n_off = a.n_off;
  double best = s.val[ml];
  const int kj = SRC == kT3Uniform ? 0 : s.cls[ml];
  int o = 0;
  for (; o + 8 <= n_off; o += 8)
    best = pull_block3<SRC, 8>(s, Wf, K, n_off, off, ml, kj, o, best);
  for (; o < n_off; ++o) best = pull_block3<SRC, 1>(s, Wf, K, n_off, off, ml, kj, o, best);
  return best;
}

// The push levels of a visit: items (frontier node, G offsets) lower their
// heads with LDS atomic mins and mark them without waiting for an answer;
// after a barrier each thread looks at its own node's mark and the marked
// nodes become the next frontier.  Each thread keeps one offset group for the
// whole visit; cells that must not be lowered hold -inf.
template <int G, int SRC>
__device__ __forceinline__ int push3(const T3Args& a, const T3Smem& s, const double* Wf, int K,
                                     int ml, int nf, int* s_cnt, long long* raw, bool* capped) {
  const int n_off = a.n_off, nt = blockDim.x;
  const int ngroups = (n_off + G - 1) / G;
  const int per = nt / ngroups;  // frontier nodes a sweep serves (0: the groups rotate)
  int g = (int)threadIdx.x % ngroups;
  const int f0 = (int)threadIdx.x / ngroups;
  const bool idle = per > 0 && f0 >= per;
  int offr[G], orow[G];
  double wr[G];
  auto load_group = [&]() {
#pragma unroll
    for (int u = 0; u < G; ++u) {
      const int o = g * G + u;
      orow[u] = min(o, n_off - 1);
      offr[u] = a.off[orow[u]];
      if constexpr (SRC == kT3Uniform) wr[u] = o < n_off ? s.W[o] : INFINITY;
    }
  };
  load_group();
  int it = 1;
  while (nf > 0 && it <= kT3IterCap) {
    *raw += (long long)nf * n_off;
    int f = f0;
    if (per == 0) {
      g = (int)threadIdx.x % ngroups;
      load_group();
    }
    while (!idle && f < nf) {
      const int i = s.list[f];
      const double vi = s.val[i];
      const int ki = SRC == kT3Uniform ? 0 : s.cls[i];
      double vj[G], wn[G];
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const int j = i + offr[u];
        vj[u] = s.val[j];
        if constexpr (SRC == kT3Uniform) {
          wn[u] = wr[u];
        } else {
          wn[u] = w3<SRC>(s, Wf, K, n_off, ki, s.cls[j], orow[u]);
          if (G > 1 && g * G + u >= n_off) wn[u] = INFINITY;
        }
      }
#pragma unroll
      for (int u = 0; u < G; ++u) {
        const double cand = __dadd_rn(vi, wn[u]);
        if (cand < vj[u]) {
          atomicMin((unsigned long long*)&s.val[i + offr[u]], dbits3(cand));
          s.mark[i + offr[u]] = 1;
        }
      }
      f += per > 0 ? per : nt / ngroups;
      if (per == 0) {
        g += nt % ngroups;
        if (g >= ngroups) {
          g -= ngroups;
          ++f;
        }
        load_group();
      }
    }
    __syncthreads();
    const bool on = ml >= 0 && s.mark[ml];
    if (on) s.mark[ml] = 0;
    if (threadIdx.x == 0) s_cnt[(it + 1) & 1] = 0;  // read before this level's first barrier
    frontier_add3(on, ml, s.list, &s_cnt[it & 1]);
    __syncthreads();
    nf = s_cnt[it & 1];
    ++it;
  }
  *capped = nf > 0;
  return it - 1;
}

__device__ __forceinline__ unsigned long long* pmin3(const T3Args& a, int round, int p) {
  return a.pmin + ((int64_t)(round % 3) * a.n_prob + p) * a.pmin_shards * kT3PminStride;
}

// One thread: does tile T of problem p wait for a later round?  If so it
// stays active, with its flag bits and key.
__device__ __forceinline__ bool defer3(const T3Args& a, int round, int T, int p, int32_t f) {
  unsigned long long* kin = a.key + (int64_t)(round & 1) * a.n_tiles;
  const unsigned long long k = kin[T];
  kin[T] = kT3Inf;
  const unsigned long long* pm = pmin3(a, round, p);
  unsigned long long lo = kT3Inf;
  for (int q = 0; q < a.pmin_shards; ++q) lo = min(lo, pm[q * kT3PminStride]);
  if (k <= lo) return false;
  const double lim =
      __longlong_as_double((long long)lo) + a.width * a.typ[2 * a.probs[p].job + a.probs[p].field];
  if (__longlong_as_double((long long)k) <= lim) return false;
  const int64_t out = (int64_t)((round + 1) & 1) * a.n_tiles;
  if (atomicOr(&a.flags[out + T], f) == 0)
    a.list[out + atomicAdd(&a.counter[round + 1], 1)] = T;
  atomicMin(&a.key[out + T], k);
  atomicMin(&pmin3(a, round + 1, p)[(T & (a.pmin_shards - 1)) * kT3PminStride], k);
  return true;
}

// The minima of round + 2 start over (round round + 1 fills them; they were
// last read in round - 1).  Workgroup 0 of a round.
__device__ __forceinline__ void reset_pmin3(const T3Args& a, int round) {
  if (!(a.width > 0.0)) return;
  unsigned long long* pm = pmin3(a, round + 2, 0);
  for (int q = threadIdx.x; q < a.n_prob * a.pmin_shards; q += blockDim.x)
    pm[(int64_t)q * kT3PminStride] = kT3Inf;
}

template <int G>
__device__ void visit3(const T3Args& a, int round, int T) {
  extern __shared__ double smem3[];
  __shared__ int s_flag, s_prob, s_mask, s_cnt[2], s_npull;
  __shared__ unsigned long long s_present, s_key;
  if (threadIdx.x == 0) {
    int32_t* fin = a.flags + (int64_t)(round & 1) * a.n_tiles;
    int32_t f = fin[T];
    const int p = a.tile_prob[T];  // in flight with the flag
    if (f) {
      fin[T] = 0;
      if (a.width > 0.0 && round < a.order_rounds && defer3(a, round, T, p, f)) f = 0;
    }
    s_prob = p;
    s_flag = f;
    s_key = kT3Inf;
    s_mask = 0;
    s_npull = 0;
    s_cnt[0] = s_cnt[1] = 0;
    s_present = 0ull;
  }
  __syncthreads();
  const int flag = s_flag;
  if (!flag) return;  // block-uniform
  const T3ProbDev P = a.probs[s_prob];
  const T3JobDev J = a.jobs[P.job];
  const int R = a.R, lx = a.lx, lz = a.lz, n_off = a.n_off, tx = a.tx, tz = a.tz, K = J.K;
  const int t = T - P.tile_base;
  const int ttx = t % J.ntx, tty = (t / J.ntx) % J.nty, ttz = t / (J.ntx * J.nty);
  const int x0 = ttx * tx, y0 = tty * tx, z0 = ttz * tz;
  const int txe = min(tx, J.nx - x0), tye = min(tx, J.ny - y0), tze = min(tz, J.nz - z0);
  const int nbox = lx * lx * lz;
  const T3Smem s = carve3(a, smem3, nbox);
  auto cell = [&](int q, int* qx, int* qy, int* qz) {
    *qz = (int)__umulhi((uint32_t)q, a.lxx_magic);
    const int r = q - *qz * lx * lx;
    *qy = (int)__umulhi((uint32_t)r, a.lx_magic);
    *qx = r - *qy * lx;
  };

  unsigned long long present = 0ull;
  for (int q = threadIdx.x; q < nbox; q += blockDim.x) {
    int qx, qy, qz;
    cell(q, &qx, &qy, &qz);
    const int gx = x0 + qx - R, gy = y0 + qy - R, gz = z0 + qz - R;
    int32_t k = 0;  // outside the grid: any class, the value decides
    double v = INFINITY;
    if (gx >= 0 && gx < J.nx && gy >= 0 && gy < J.ny && gz >= 0 && gz < J.nz) {
      const int64_t g = gx + (int64_t)J.nx * (gy + (int64_t)J.ny * gz);
      k = J.cls[g];
      v = P.tau[g];
      if (k < 0 || k >= K) {
        atomicAdd(a.err, 1);
        k = 0;
        v = INFINITY;
      }
      if (k < kCodeMaskIds) present |= 1ull << k;
    }
    s.val[q] = v;
    s.cls[q] = (uint16_t)k;
    s.mark[q] = 0;
  }
  const double* Wf = J.W + (int64_t)P.field * K * K * n_off;
  for (int d = 32; d >= 1; d >>= 1) present |= __shfl_xor(present, d);
  if (__lane_id() == 0 && present) atomicOr(&s_present, present);
  __syncthreads();
  present = s_present;
  const int nk = __popcll(present);
  const bool staged = K <= kCodeMaskIds && nk <= a.w_classes;
  const int src = !staged ? kT3Global : (nk == 1 ? kT3Uniform : kT3Lds);
  if (staged) {  // codes in place of ids, and the weights of their pairs
    if (nk > 1)
      for (int q = threadIdx.x; q < nbox; q += blockDim.x)
        s.cls[q] = (uint16_t)class_code(present, nk, s.cls[q], n_off);
    stage_codes(s.W, Wf, K, n_off, present, nk);
    __syncthreads();
  }

  // this thread's interior node
  int ml = -1, ix = 0, iy = 0, iz = 0;
  if ((int)threadIdx.x < tx * tx * tz) {
    ix = threadIdx.x % tx;
    iy = (threadIdx.x / tx) % tx;
    iz = threadIdx.x / (tx * tx);
    if (ix < txe && iy < tye && iz < tze) ml = (ix + R) + lx * ((iy + R) + lx * (iz + R));
  }
  const double orig = ml >= 0 ? s.val[ml] : 0.0;
  const bool pl = ml >= 0 && pulls3(flag, ix, iy, iz, tx, tz, R);
  const unsigned long long pb = __ballot(pl);
  if (pb && __lane_id() == 0) atomicAdd(&s_npull, __popcll(pb));
  double best = orig;
  if (pl) {
    if (src == kT3Uniform) best = pull3<kT3Uniform>(a, s, Wf, K, ml);
    else if (src == kT3Lds) best = pull3<kT3Lds>(a, s, Wf, K, ml);
    else best = pull3<kT3Global>(a, s, Wf, K, ml);
  }
  const bool improved = best < orig;
  __syncthreads();  // the pulls' reads are done
  if (improved) s.val[ml] = best;
  frontier_add3(improved, ml, s.list, &s_cnt[0]);
  if (threadIdx.x == 0 && (flag & kT3Seed)) {
    const int sx = (int)(P.src % J.nx) - x0, sy = (int)((P.src / J.nx) % J.ny) - y0,
              sz = (int)(P.src / ((int64_t)J.nx * J.ny)) - z0;
    // (the source's value is 0: it never improves, so it is listed once)
    if (sx >= 0 && sx < txe && sy >= 0 && sy < tye && sz >= 0 && sz < tze)
      s.list[atomicAdd(&s_cnt[0], 1)] = (uint16_t)((sx + R) + lx * ((sy + R) + lx * (sz + R)));
  }
  for (int q = threadIdx.x; q < nbox; q += blockDim.x) {  // not to be lowered by pushes
    int qx, qy, qz;
    cell(q, &qx, &qy, &qz);
    if (qx < R || qx >= R + txe || qy < R || qy >= R + tye || qz < R || qz >= R + tze)
      s.val[q] = -INFINITY;
  }
  __syncthreads();

  long long raw = 0;
  bool capped;
  const int nf = s_cnt[0];
  if (src == kT3Uniform) push3<G, kT3Uniform>(a, s, Wf, K, ml, nf, s_cnt, &raw, &capped);
  else if (src == kT3Lds) push3<G, kT3Lds>(a, s, Wf, K, ml, nf, s_cnt, &raw, &capped);
  else push3<G, kT3Global>(a, s, Wf, K, ml, nf, s_cnt, &raw, &capped);

  int mask = capped ? (1 << kT3Self) : 0;  // iteration cap: this tile again, in full
  unsigned long long key = capped ? 0ull : kT3Inf;
  if (ml >= 0 && s.val[ml] < orig) {
    P.tau[(x0 + ix) + (int64_t)J.nx * ((y0 + iy) + (int64_t)J.ny * (z0 + iz))] = s.val[ml];
    const int bb = border_bits3(ix, iy, iz, tx, tz, R);
    mask |= bb;
    if (bb && !capped) key = dbits3(s.val[ml]);
  }
  if (mask) atomicOr(&s_mask, mask);
  if (a.width > 0.0) {
    for (int d = 32; d >= 1; d >>= 1) key = min(key, __shfl_xor(key, d));
    if (__lane_id() == 0 && key != kT3Inf) atomicMin(&s_key, key);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long* st = stat_slot(a.stats);
    atomicAdd(&st[0], 1ull);
    atomicAdd(&st[1], (unsigned long long)(raw + (long long)s_npull * n_off));
  }
  const int m = s_mask;
  if (m && threadIdx.x < 64) {
    // lane n wakes neighbour n: the flags' device-wide round trips overlap
    // (one lane walking up to 26 neighbours waited for each in turn)
    const int n = threadIdx.x;
    const int64_t out = (int64_t)((round + 1) & 1) * a.n_tiles;
    const int nx_ = ttx + n % 3 - 1, ny_ = tty + (n / 3) % 3 - 1, nz_ = ttz + n / 9 - 1;
    const bool on = n < 27 && ((m >> n) & 1) && nx_ >= 0 && nx_ < J.ntx && ny_ >= 0 &&
                    ny_ < J.nty && nz_ >= 0 && nz_ < J.ntz;
    const int TN = P.tile_base + (nz_ * J.nty + ny_) * J.ntx + nx_;
    bool fresh = false;
    if (a.width > 0.0 && round + 1 < a.order_rounds) {
      const unsigned long long k = s_key;
      if (on) atomicMin(&a.key[out + TN], k);
      if (n == 27)
        atomicMin(&pmin3(a, round + 1, s_prob)[(T & (a.pmin_shards - 1)) * kT3PminStride], k);
    }
    if (on) {
      // the neighbour's halo part facing us (its side -d) changed
      const int32_t bits = (n == kT3Self) ? (kT3Active | kT3Full)
                                          : (kT3Active | (1 << (kT3SideShift + 26 - n)));
      fresh = atomicOr(&a.flags[out + TN], bits) == 0;
    }
    // one reservation for the newly activated tiles (the counter is one
    // address for the whole chip)
    const unsigned long long fm = __ballot(fresh);
    if (fm) {
      int slot = 0;
      if (n == 0) slot = atomicAdd(&a.counter[round + 1], __popcll(fm));
      slot = __shfl(slot, 0);
      if (fresh) a.list[out + slot + __popcll(fm & ((1ull << n) - 1ull))] = TN;
    }
  }
}

// One launch per round: one workgroup per tile (affinity), or a smaller grid
// walking the round's active list on large batches.
template <int G>
__global__ void __launch_bounds__(kT3Threads) __attribute__((amdgpu_waves_per_eu(6)))
k_tile3_tau(T3Args a, int round) {
  if (blockIdx.x == 0) reset_pmin3(a, round);
  if ((int)gridDim.x == a.n_tiles) {
    visit3<G>(a, round, blockIdx.x);
    return;
  }
  const int n_act = a.counter[round];
  const int32_t* lst = a.list + (int64_t)(round & 1) * a.n_tiles;
  // tiles by ticket as workgroups free up; the next round's ticket lines
  // (last used a round ago) start from zero
  if (blockIdx.x == 0)
    for (int q = threadIdx.x; q < kTickWords; q += blockDim.x)
      a.tick[((round + 1) & 1) * kTickWords + q] = 0u;
  uint32_t* tick = a.tick + (round & 1) * kTickWords;
  const Shard sh = shard_of();
  for (int i = first_item(sh, n_act); i >= 0;) {
    const uint32_t t = draw_ticket(tick, sh, n_act);  // the next entry's, in flight meanwhile
    visit3<G>(a, round, lst[i]);
    __syncthreads();  // LDS is reused by the next tile
    i = ticket_item(sh, 0u, n_act, t);
  }
}

// All rounds in one launch: an occupancy-sized grid walks each round's
// active list; rounds are separated by the bounded device-wide barrier.
// The caller's abort word is polled once per round by workgroup 0 and
// published by the barrier, so every workgroup leaves together.  Result:
// rounds to convergence, -1 cap reached, -2 barrier timed out, -3 aborted.
template <int G>
__global__ void __launch_bounds__(kT3Threads) k_tile3_persist(T3Args a, PersistArgs p) {
  const Shard sh = shard_of();
  uint32_t base = 0;  // tickets of this workgroup's shard issued before this round
  for (int round = 0; round < p.max_rounds; ++round) {
    if (blockIdx.x == 0) reset_pmin3(a, round);
    const int n_act =
        __hip_atomic_load(&a.counter[round], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int32_t* lst = a.list + (int64_t)(round & 1) * a.n_tiles;
    for (int i = first_item(sh, n_act); i >= 0;) {
      const uint32_t t = draw_ticket(p.tick, sh, n_act);  // the next entry's, in flight meanwhile
      visit3<G>(a, round, lst[i]);
      __syncthreads();  // LDS is reused by the next tile
      i = ticket_item(sh, base, n_act, t);
    }
    base += round_tickets(sh, n_act);
    if (a.abort_host && blockIdx.x == 0 && threadIdx.x == 0 &&
        __hip_atomic_load(a.abort_host, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) != 0)
      __hip_atomic_store(a.abort_seen, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!grid_barrier(p)) {
      if (threadIdx.x == 0) p.result[0] = -2;
      return;
    }
    if (a.abort_host &&
        __hip_atomic_load(a.abort_seen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
      if (blockIdx.x == 0 && threadIdx.x == 0) p.result[0] = -3;
      return;
    }
    if (__hip_atomic_load(&a.counter[round + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
        0) {
      if (blockIdx.x == 0 && threadIdx.x == 0) p.result[0] = round + 1;
      return;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) p.result[0] = -1;
}

size_t align256_t3(size_t x) { return (x + 255) & ~(size_t)255; }

struct T3Plan {
  int tx = 0, tz = 0, lx = 0, lz = 0, n_tiles = 0, w_classes = 0, pmin_shards = 1;
  int span = 0;  // most tiles along the three axes together
  size_t off_typ = 0, off_jobs = 0, off_probs = 0, off_flags = 0, off_list = 0, off_tprob = 0, off_soff = 0, off_counter = 0, off_key = 0, off_pmin = 0, off_err = 0,
         off_stats = 0, total = 0;
  size_t lds = 0;
};

int plan_t3(const Tile3Job* jobs, int n_jobs, const Tile3Prob* probs, int n_prob, int R,
            int n_off, int tile_x, int tile_z, int max_rounds, T3Plan* P) {
  P->tx = tile_x > 0 ? tile_x : 8;
  P->tz = tile_z > 0 ? tile_z : 8;
  if (P->tx < R || P->tz < R || P->tx * P->tx * P->tz > kT3Threads)
    return fail(CHERT_ERR_INVALID_ARG, "3D tile must be >= radius per side and <= 1024 nodes");
  P->lx = P->tx + 2 * R;
  P->lz = P->tz + 2 * R;
  int64_t tiles = 0;
  int maxK = 0;
  for (int q = 0; q < n_prob; ++q) {
    const Tile3Job& J = jobs[probs[q].job];
    tiles += (int64_t)((J.nx + P->tx - 1) / P->tx) * ((J.ny + P->tx - 1) / P->tx) *
             ((J.nz + P->tz - 1) / P->tz);
  }
  for (int j = 0; j < n_jobs; ++j) {
    const Tile3Job& J = jobs[j];
    maxK = J.K > maxK ? J.K : maxK;
    const int span = (J.nx + P->tx - 1) / P->tx + (J.ny + P->tx - 1) / P->tx +
                     (J.nz + P->tz - 1) / P->tz;
    P->span = span > P->span ? span : P->span;
  }
  if (tiles >= 0x7fffffffLL) return fail(CHERT_ERR_UNSUPPORTED, "batch too large for one launch");
  P->n_tiles = (int)tiles;
  P->w_classes = code_classes(maxK, n_off, kT3WLdsBytes);
  const size_t nbox = (size_t)P->lx * P->lx * P->lz;
  P->lds = (nbox + (P->w_classes ? (size_t)code_rows(P->w_classes) * n_off : 0)) * sizeof(double) +
           (nbox + (size_t)P->tx * P->tx * P->tz) * sizeof(uint16_t) + nbox;
  size_t off = 0;
  P->off_jobs = off;
  off += align256_t3((size_t)n_jobs * sizeof(T3JobDev));
  P->off_probs = off;
  off += align256_t3((size_t)n_prob * sizeof(T3ProbDev));
  P->off_flags = off;
  off += align256_t3((size_t)2 * P->n_tiles * sizeof(int32_t));
  P->off_list = off;
  off += align256_t3((size_t)2 * P->n_tiles * sizeof(int32_t));
  P->off_soff = off;
  off += align256_t3((size_t)n_off * sizeof(int32_t));
  P->off_tprob = off;
  off += align256_t3((size_t)P->n_tiles * sizeof(int32_t));
  P->off_counter = off;
  off += align256_t3(counter_words(max_rounds) * sizeof(int32_t));  // counts, tickets
  P->off_key = off;
  off += align256_t3((size_t)2 * P->n_tiles * sizeof(uint64_t));
  // a problem's visits of a round all lower its minimum: several lines when
  // there are few problems (atomics on one address serialise)
  P->pmin_shards = n_prob <= 8 ? 8 : (n_prob <= 32 ? 2 : 1);
  P->off_pmin = off;
  off += align256_t3((size_t)3 * n_prob * P->pmin_shards * kT3PminStride * sizeof(uint64_t));
  P->off_typ = off;
  off += align256_t3((size_t)2 * n_jobs * sizeof(double));
  P->off_err = off;
  off += 256;
  P->off_stats = off;
  off += align256_t3(kStatBytes);
  P->total = off;
  return CHERT_OK;
}

int threads_of(const T3Plan& P) { return (P.tx * P.tx * P.tz + 63) / 64 * 64; }

// Error word and the sharded statistics, after the relaxation (synchronous).
int read_back(const T3Args& a, hipStream_t s, int32_t* herr, int64_t* visits, int64_t* edges) {
  unsigned long long hs[2] = {0, 0};
  std::vector<unsigned long long> slots((size_t)kStatSlots * kStatSlotU64);
  hipError_t e = hipMemcpyAsync(herr, a.err, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipMemcpyAsync(slots.data(), a.stats, kStatBytes, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return fail(CHERT_ERR_HIP, hipGetErrorString(e));
  stats_reduce(slots.data(), 2, 0u, hs);
  *visits = (int64_t)hs[0];
  *edges = (int64_t)hs[1];
  return CHERT_OK;
}

// Switch the tile ordering on (the jobs' tables are on the device).
void order_tiles(const T3Plan& P, int n_jobs, hipStream_t s, T3Args* a) {
  a->width = kT3OrderSides * P.tx;
  a->order_rounds = order_cap(P.span);
  CHERT_LAUNCH("k_tile3_typ", k_tile3_typ, dim3((unsigned)n_jobs, 2), dim3(kTypThreads), 0, s, *a);
}

// Every round in one launch of an occupancy-sized grid (all of its
// workgroups resident, which the device-wide barrier needs).
int run_persistent(const T3Plan& P, T3Args a, int n_jobs, bool ordered, const int32_t* ox_dev,
                   const int32_t* oy_dev, const int32_t* oz_dev, int push_group, int max_rounds,
                   int threads, hipStream_t s, int* rounds, int64_t* visits, int64_t* edges) {
  void (*kern)(T3Args, PersistArgs) =
      push_group == 1 ? k_tile3_persist<1> : (push_group == 4 ? k_tile3_persist<4>
                                                              : k_tile3_persist<2>);
  int per_cu = 0, cus = 0, dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = resident_per_cu(&per_cu, kern, threads, P.lds);
  if (e != hipSuccess) return fail(CHERT_ERR_HIP, hipGetErrorString(e));
  if (per_cu < 1) return fail(CHERT_ERR_UNSUPPORTED, "3D tile does not fit on a compute unit");
  const int64_t resident = (int64_t)per_cu * cus;
  const int grid = (int)(P.n_tiles < resident ? P.n_tiles : resident);
  if (ordered && P.n_tiles > 2 * resident) order_tiles(P, n_jobs, s, &a);
  PersistArgs pa{};
  pa.max_rounds = max_rounds;
  pa.bar = (uint32_t*)(a.err + 48);  // [0] arrivals, [1] generation, [2] abort
  pa.result = a.err + 52;
  pa.tick = (uint32_t*)a.counter + tick_offset(max_rounds);
  CHERT_LAUNCH("k_tile3_clear", k_tile3_clear, dim3(256), dim3(256), 0, s, a.flags,
               (int64_t)2 * P.n_tiles, a.counter, (int)counter_words(max_rounds), a.err, a.stats, a.probs, a.n_prob,
               a.tile_prob, a.key, a.pmin,
               (int64_t)3 * a.n_prob * a.pmin_shards * kT3PminStride, (int32_t*)a.off, ox_dev, oy_dev,
               oz_dev, a.n_off, a.lx);
  CHERT_LAUNCH("k_tile3_seed", k_tile3_seed, dim3((a.n_prob + 63) / 64), dim3(64), 0, s, a);
  CHERT_LAUNCH("k_tile3_persist", kern, dim3((unsigned)grid), dim3((unsigned)threads), P.lds, s,
               a, pa);
  int32_t res = 0, herr = 0;
  e = hipMemcpyAsync(&res, pa.result, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return fail(CHERT_ERR_HIP, hipGetErrorString(e));
  int rc = read_back(a, s, &herr, visits, edges);
  if (rc) return rc;
  *rounds = res > 0 ? res : max_rounds;
  if (res == -3) return fail(CHERT_ERR_ABORTED, "aborted by the caller");
  if (res == -2) return fail(CHERT_ERR_HIP, "device-wide barrier timed out");
  if (res <= 0) return fail(CHERT_ERR_NO_CONVERGENCE, "relaxation round cap reached");
  if (herr) return fail(CHERT_ERR_INVALID_ARG, "class id out of range");
  return CHERT_OK;
}

}  // namespace

int tiles3d_bytes(const Tile3Job* jobs, int n_jobs, const Tile3Prob* probs, int n_prob, int R,
                  int n_off, int tile_x, int tile_z, int max_rounds, size_t* bytes) {
  T3Plan P;
  const int rc = plan_t3(jobs, n_jobs, probs, n_prob, R, n_off, tile_x, tile_z, max_rounds, &P);
  *bytes = rc ? 0 : P.total;
  return rc;
}

int relax_tiles_3d(const Tile3Job* jobs, int n_jobs, const Tile3Prob* probs, int n_prob,
                   const int32_t* ox_dev, const int32_t* oy_dev, const int32_t* oz_dev, int n_off,
                   int R, int tile_x, int tile_z, int push_group, int max_rounds, void* ws,
                   size_t ws_bytes, hipStream_t s, const volatile int32_t* abort_flag,
                   bool persistent, bool ordered, int* rounds, int64_t* visits,
                   int64_t* edges) {
  T3Plan P;
  int rc = plan_t3(jobs, n_jobs, probs, n_prob, R, n_off, tile_x, tile_z, max_rounds, &P);
  if (rc) return rc;
  if (!ws || ws_bytes < P.total) return fail(CHERT_ERR_INVALID_ARG, "workspace too small");
  uint8_t* w = (uint8_t*)ws;
  std::vector<T3JobDev> jd(n_jobs);
  for (int j = 0; j < n_jobs; ++j) {
    jd[j].nx = jobs[j].nx;
    jd[j].ny = jobs[j].ny;
    jd[j].nz = jobs[j].nz;
    jd[j].K = jobs[j].K;
    jd[j].ntx = (jobs[j].nx + P.tx - 1) / P.tx;
    jd[j].nty = (jobs[j].ny + P.tx - 1) / P.tx;
    jd[j].ntz = (jobs[j].nz + P.tz - 1) / P.tz;
    jd[j].cls = jobs[j].cls;
    jd[j].W = jobs[j].W;
  }
  std::vector<T3ProbDev> pd(n_prob);
  int base = 0;
  for (int q = 0; q < n_prob; ++q) {
    pd[q].tau = probs[q].tau;
    pd[q].src = probs[q].src;
    pd[q].job = probs[q].job;
    pd[q].field = probs[q].field;
    pd[q].tile_base = base;
    const T3JobDev& J = jd[probs[q].job];
    base += J.ntx * J.nty * J.ntz;
  }
  hipError_t e = hipMemcpyAsync(w + P.off_jobs, jd.data(), jd.size() * sizeof(T3JobDev),
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(w + P.off_probs, pd.data(), pd.size() * sizeof(T3ProbDev),
                       hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);  // host buffers are locals
  if (e != hipSuccess) return fail(CHERT_ERR_HIP, hipGetErrorString(e));
  T3Args a{};
  a.tx = P.tx;
  a.tz = P.tz;
  a.R = R;
  a.n_off = n_off;
  a.lx = P.lx;
  a.lz = P.lz;
  a.n_prob = n_prob;
  a.n_tiles = P.n_tiles;
  a.w_classes = P.w_classes;
  a.width = 0.0;  // order_tiles sets it
  a.order_rounds = 0;
  a.typ = (double*)(w + P.off_typ);
  a.key = (unsigned long long*)(w + P.off_key);
  a.pmin = (unsigned long long*)(w + P.off_pmin);
  a.pmin_shards = P.pmin_shards;
  a.lx_magic = (uint32_t)((0x100000000ull + P.lx - 1) / P.lx);
  a.lxx_magic = (uint32_t)((0x100000000ull + P.lx * P.lx - 1) / (P.lx * P.lx));
  a.jobs = (const T3JobDev*)(w + P.off_jobs);
  a.probs = (const T3ProbDev*)(w + P.off_probs);
  a.off = (const int32_t*)(w + P.off_soff);
  a.flags = (int32_t*)(w + P.off_flags);
  a.list = (int32_t*)(w + P.off_list);
  a.tile_prob = (int32_t*)(w + P.off_tprob);
  a.counter = (int32_t*)(w + P.off_counter);
  a.err = (int32_t*)(w + P.off_err);
  a.stats = (unsigned long long*)(w + P.off_stats);
  a.tick = (uint32_t*)a.counter + tick_offset(max_rounds);
  a.abort_seen = a.err + 56;
  a.abort_host = nullptr;
  if (persistent && abort_flag) {
    // the persistent grid polls the word itself: page-locked host memory only
    hipPointerAttribute_t at{};
    const hipError_t pe = hipPointerGetAttributes(&at, (const void*)abort_flag);
    if (pe != hipSuccess || at.type != hipMemoryTypeHost || !at.devicePointer) {
      (void)hipGetLastError();
      return fail(CHERT_ERR_INVALID_ARG, "abort_flag_host must be pinned host memory");
    }
    a.abort_host = (const int32_t*)at.devicePointer;
  }
  if (persistent)
    return run_persistent(P, a, n_jobs, ordered, ox_dev, oy_dev, oz_dev, push_group, max_rounds,
                          threads_of(P), s, rounds, visits, edges);
  void (*kern)(T3Args, int) = push_group == 1 ? k_tile3_tau<1> : (push_group == 4 ? k_tile3_tau<4>
                                                                                   : k_tile3_tau<2>);
  const int threads = threads_of(P);
  int per_cu = 0, cus = 0, dev = 0;
  e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess)
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, P.lds);
  if (e != hipSuccess) return fail(CHERT_ERR_HIP, hipGetErrorString(e));
  if (per_cu < 1) return fail(CHERT_ERR_UNSUPPORTED, "3D tile does not fit on a compute unit");
  const int64_t resident = (int64_t)per_cu * cus;
  // one workgroup per tile up to twice the resident workgroups, else twice
  // the resident walking each round's list by ticket (twice measured 5 %
  // faster than four times on the 3D layered batch)
  const int grid = (int)(P.n_tiles <= 2 * resident ? P.n_tiles : 2 * resident);
  if (ordered && P.n_tiles > 2 * resident) order_tiles(P, n_jobs, s, &a);
  CHERT_LAUNCH("k_tile3_clear", k_tile3_clear, dim3(256), dim3(256), 0, s, a.flags,
               (int64_t)2 * P.n_tiles, a.counter, (int)counter_words(max_rounds), a.err, a.stats, a.probs, a.n_prob,
               a.tile_prob, a.key, a.pmin,
               (int64_t)3 * a.n_prob * a.pmin_shards * kT3PminStride, (int32_t*)a.off, ox_dev, oy_dev,
               oz_dev, a.n_off, a.lx);
  CHERT_LAUNCH("k_tile3_seed", k_tile3_seed, dim3((n_prob + 63) / 64), dim3(64), 0, s, a);
  const int batch = 8;
  int32_t counts[batch];
  int done = -1;
  for (int r = 0; r < max_rounds && done < 0; r += batch) {
    const int nb = r + batch > max_rounds ? max_rounds - r : batch;
    for (int q = 0; q < nb; ++q)
      CHERT_LAUNCH("k_tile3_tau", kern, dim3((unsigned)grid), dim3((unsigned)threads), P.lds, s, a,
                   r + q);
    e = hipMemcpyAsync(counts, a.counter + r + 1, sizeof(int32_t) * nb, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(CHERT_ERR_HIP, hipGetErrorString(e));
    for (int q = 0; q < nb && done < 0; ++q)
      if (counts[q] == 0) done = r + q + 1;
    if (done < 0 && abort_flag && *abort_flag) {
      *rounds = r + nb;
      return fail(CHERT_ERR_ABORTED, "aborted by the caller");
    }
  }
  int32_t herr = 0;
  rc = read_back(a, s, &herr, visits, edges);
  if (rc) return rc;
  *rounds = done < 0 ? max_rounds : done;
  if (done < 0) return fail(CHERT_ERR_NO_CONVERGENCE, "relaxation round cap reached");
  if (herr) return fail(CHERT_ERR_INVALID_ARG, "class id out of range");
  return CHERT_OK;
}

}  // namespace chert
