// k_window.hip -- profile of a time window for any subset of ranks (Sec. II:
// a calling context tree for a trace interval).  Each event's interval
// [t_k, t_{k+1}) (a rank's last event lasts 0) is clipped to [t0, t1) and added
// to its context node; inclusive costs are subtree sums of the result.
#include "ta_internal.h"
#include "ta_select.h"

namespace ta {
namespace {

constexpr int WT = 256;   // threads of the small kernels
constexpr int WWT = 512;  // threads of a window workgroup

typedef long long v2ll __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));

// Visits events k in [lo, hi) of a rank whose events end at e, four
// consecutive events per thread per step from a 4-aligned index (16-byte loads
// of timestamps and contexts; scalar loads within 4 events of the array's end
// E), DEPTH steps' loads in flight before any is visited.  f(k, t_k, t_{k+1}
// (t_k for the rank's last event), ctx_k).
struct EvQuad {
  int64_t t[5];
  int32_t c[4];
};

__device__ inline EvQuad load_quad(const int64_t *__restrict__ ts, const int32_t *__restrict__ ctx,
                                   int64_t E, int64_t k0, int64_t e) {
  EvQuad q;
  if (k0 + 4 <= E) {
    const v2ll a = *reinterpret_cast<const v2ll *>(ts + k0);
    const v2ll b = *reinterpret_cast<const v2ll *>(ts + k0 + 2);
    const v4i c = *reinterpret_cast<const v4i *>(ctx + k0);
    q.t[0] = a.x;
    q.t[1] = a.y;
    q.t[2] = b.x;
    q.t[3] = b.y;
    q.c[0] = c.x;
    q.c[1] = c.y;
    q.c[2] = c.z;
    q.c[3] = c.w;
  } else {
#pragma unroll
    for (int u = 0; u < 4; u++) {
      q.t[u] = k0 + u < E ? ts[k0 + u] : 0;
      q.c[u] = k0 + u < E ? ctx[k0 + u] : 0;
    }
  }
  q.t[4] = k0 + 4 < e ? ts[k0 + 4] : 0;
  return q;
}

// The same, four events at a time: f(k0, quad of events k0..k0+3); those
// outside [lo, hi) are f's to skip.
// Thread t of nt.
template <int DEPTH, class F>
__device__ __forceinline__ void visit_quads(const int64_t *__restrict__ ts, const int32_t *__restrict__ ctx,
                                            int64_t E, int64_t lo, int64_t hi, int64_t e, int t, int nt, F &&f) {
  const int64_t STEP = 4 * (int64_t)nt;
  for (int64_t k0 = (lo & ~(int64_t)3) + 4 * (int64_t)t; k0 < hi; k0 += DEPTH * STEP) {
    // every load is in bounds of the arrays (load_quad guards E); a later
    // step that starts at or past hi loads nothing (f skips its events)
    EvQuad q[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; d++) {
      q[d] = EvQuad{};
      if (d == 0 || k0 + d * STEP < hi) q[d] = load_quad(ts, ctx, E, k0 + d * STEP, e);
    }
#pragma unroll
    for (int d = 0; d < DEPTH; d++) f(k0 + d * STEP, q[d]);
  }
}

template <int DEPTH, class F>
__device__ __forceinline__ void visit_events(const int64_t *__restrict__ ts, const int32_t *__restrict__ ctx,
                                             int64_t E, int64_t lo, int64_t hi, int64_t e, int t, int nt, F &&f) {
  visit_quads<DEPTH>(ts, ctx, E, lo, hi, e, t, nt, [&](int64_t k0, const EvQuad &q) {
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int64_t k = k0 + u;
      if (k < lo || k >= hi) continue;
      f(k, q.t[u], k + 1 < e ? q.t[u + 1] : q.t[u], q.c[u]);
    }
  });
}

// What window_bounds adds up over the selected ranks' events in the window.
struct WinCounts {
  unsigned long long total, longest, ranks;  // ranks: that have any
};

__global__ void zero_i64(int64_t *p, int64_t n, WinCounts *wc) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0;
  if (wc && blockIdx.x == 0 && threadIdx.x == 0) *wc = WinCounts{0, 0, 0};
}

// First index in [a, z) whose timestamp satisfies a monotone predicate (false
// then true), or z: binary search by one thread.
template <class P>
__device__ inline int64_t first_true(const int64_t *__restrict__ ts, int64_t a, int64_t z, P pred) {
  while (a < z) {
    const int64_t m = a + ((z - a) >> 1);
    if (pred(ts[m])) z = m;
    else a = m + 1;
  }
  return a;
}

// The events of each selected rank that overlap the window, one thread per
// rank (so the searches' round trips overlap one another): before the event
// preceding the first timestamp above t0 every interval ends by t0; from the
// first timestamp at or above t1 every interval starts at or after t1.
// bounds[i] = {lo, hi, e (the rank's end), 0}; an invalid rank gets an empty
// range and sets the offsets error bit.
__global__ __launch_bounds__(WT) void window_bounds(const int64_t *__restrict__ off,
                                                   const int64_t *__restrict__ ts, int64_t R, int64_t E,
                                                   const int32_t *__restrict__ ids, int64_t n_sel,
                                                   int64_t t0, int64_t t1, v2ll *__restrict__ bounds,
                                                   WinCounts *wc, uint32_t *err) {
  __shared__ uint64_t sum[WT / 64], top[WT / 64];
  __shared__ int some[WT / 64];
  const int64_t i = (int64_t)blockIdx.x * WT + threadIdx.x;
  const int64_t r = i >= n_sel ? 0 : (ids ? (int64_t)ids[i] : i);
  int64_t lo = 0, hi = 0, e = 0;
  if (i >= n_sel) {
  } else if (r < 0 || r >= R || off[r] < 0 || off[r + 1] < off[r] || off[r + 1] > E) {
    atomicOr(err, ERRBIT_OFFSETS);
  } else {
    const int64_t b = off[r];
    e = off[r + 1];
    const int64_t a = first_true(ts, b, e, [&](int64_t v) { return v > t0; });
    lo = a > b ? a - 1 : b;
    hi = first_true(ts, b, e, [&](int64_t v) { return v >= t1; });
  }
  if (i < n_sel) {
    bounds[2 * i] = v2ll{lo, hi};
    bounds[2 * i + 1] = v2ll{e, 0};
  }
  if (!wc) return;
  const uint64_t own = hi > lo ? (uint64_t)(hi - lo) : 0;
  uint64_t n = wave_sum(own), m = wave_max(own);
  int have = (int)__popcll(__ballot(own > 0));
  if ((threadIdx.x & 63) == 0) {
    sum[threadIdx.x >> 6] = n;
    top[threadIdx.x >> 6] = m;
    some[threadIdx.x >> 6] = have;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < WT / 64; w++) {
      n += sum[w];
      m = top[w] > m ? top[w] : m;
      have += some[w];
    }
    if (n) {
      atomicAdd(&wc->total, (unsigned long long)n);
      atomicMax(&wc->longest, (unsigned long long)m);
      atomicAdd(&wc->ranks, (unsigned long long)have);
    }
  }
}

// Sums by node id in LDS for trees too large for a bin per node: buckets of
// four ids, read at once, at most PROBES of them tried.  (Single slots at a
// third full: the longest of 64 lanes' searches takes seven dependent reads.)
constexpr int HSLOTS = 4096;  // 48 KB: three workgroups per CU beside 160 KB
struct NodeSums {
  static constexpr int PROBES = 16;
  alignas(16) int32_t key[HSLOTS];  // -1: free; buckets are read as 16-byte words
  uint64_t sum[HSLOTS];

  __device__ void clear(int t, int nt) {
    for (int i = t; i < HSLOTS; i += nt) {
      key[i] = -1;
      sum[i] = 0;
    }
  }
  static __device__ uint32_t home(int32_t c) { return (((uint32_t)c * 2654435761u) >> 20) & ~3u; }
  __device__ v4i bucket(uint32_t at) const { return *reinterpret_cast<const volatile v4i *>(&key[at]); }
  static __device__ int which(v4i k, int32_t c) {
    return k.x == c ? 0 : (k.y == c ? 1 : (k.z == c ? 2 : (k.w == c ? 3 : -1)));
  }
  // Adds d[u] to node c[u] where d[u] is not 0; none(c, d) where no slot was found
  // in `probes` buckets.  Nodes already in their home bucket, the most, are
  // added at once; one loop over what is left keeps the code short.
  template <class G>
  __device__ __forceinline__ void add4(const int32_t (&c)[4], uint64_t (&d)[4], int probes, G &&none) {
    v4i k[4];
#pragma unroll
    for (int u = 0; u < 4; u++) k[u] = bucket(home(c[u]));
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int w = which(k[u], c[u]);
      if (d[u] && w >= 0) {
        atomicAdd((unsigned long long *)&sum[home(c[u]) + w], (unsigned long long)d[u]);
        d[u] = 0;
      }
    }
    // the pending ones move up to the front
    int32_t c0 = c[0], c1 = c[1], c2 = c[2], c3 = c[3];
    uint64_t d0 = d[0], d1 = d[1], d2 = d[2], d3 = d[3];
    uint32_t at = home(c0);
    int tries = probes;
    while ((d0 | d1 | d2 | d3) != 0) {
      if (d0 == 0) {
        c0 = c1, c1 = c2, c2 = c3;
        d0 = d1, d1 = d2, d2 = d3, d3 = 0;
        at = home(c0);
        tries = probes;
      }
      if (d0 != 0) {
        const v4i b = bucket(at);
        int w = which(b, c0);
        if (w < 0) {
          const int f = which(b, -1);
          if (f >= 0) {  // taken by another node meanwhile: the bucket again
            const int32_t x = atomicCAS(&key[at + f], -1, c0);
            if (x == -1 || x == c0) w = f;
          } else {
            at = (at + 4) & (HSLOTS - 1);
            if (--tries == 0) {
              none(c0, d0);
              d0 = 0;
            }
          }
        }
        if (w >= 0) {
          atomicAdd((unsigned long long *)&sum[at + w], (unsigned long long)d0);
          d0 = 0;
        }
      }
    }
  }
};
static_assert(HSLOTS == 1 << (32 - 20), "the hash is the product's upper bits");

// How the events of a window are divided over the workgroups and added up;
// `total` and `longest` (window_bounds) count the selected ranks' events in it
// (not for traces of fewer than COUNT_MIN events: a workgroup per rank, atomics).
//   table   trees above 8,192 nodes, sums by node id in LDS: from 2,048 events per
//           rank and 524,288 in all.  Below, a 64-bit atomic on the output per
//           event costs less than clearing, searching and flushing the table
//           (97,833 nodes; atomics, table: 200 ranks of 2,400 events 49, 64 us; of
//           4,800 72, 58; 2,000 ranks of 1,200 136, 139; of 2,400 239, 186).
//   split   an equal share of events, consecutive ones, per workgroup: with the
//           table (neighbouring ranks share nodes), and when the longest rank
//           is more than twice an equal share (3,000 ranks, lognormal lengths, over
//           5,000 nodes: by rank 431 us, split 267; 200 ranks of 9,600 events
//           alike: 38 and 46).  A rank counts as RANK_W events more, which is what a
//           workgroup takes to go on to the next one.  Up to BAL_SEL ranks: each
//           workgroup adds up the ranks' counts.
//   by wave below 512 events per rank, a wave takes a rank: most windows are short
//           (8,192 ranks with two events each split into equal shares: 3,821 us, as one
//           workgroup went from rank to rank).
// The same value in every lane, to a scalar register.
__device__ __forceinline__ int64_t uniform(int64_t x) {
  return ((int64_t)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) |
         (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

constexpr int BAL_SEL = 16 * WWT;
constexpr int RANK_W = 1024;
constexpr int64_t TABLE_MEAN = 2048, TABLE_MIN = 1 << 19, WAVE_MEAN = 512, COUNT_MIN = 1 << 16;

// The events window_bounds found.  LDSH: an LDS histogram over the N nodes
// (N <= 8192) flushed once; otherwise sums by node id in LDS (the table), also
// flushed once (a node that finds no slot: a 64-bit atomic on the output; after
// the first one a node is looked for in its home bucket alone), or 64-bit
// atomics on the output.  Integer sums: the order of the atomics does not matter.
// `fit`: workgroups with a table that fit on the chip.
//
// Bound by the atomics: with one on the output per event, 97,833 nodes, the
// 3,000 ranks' events in a twentieth of the longest one's time took 629 us, all
// events of 429 ranks (20,000 at the median, 200,000 at most) 1,001; now both
// together take 214.
template <bool LDSH>
__global__ __launch_bounds__(WWT) void window_excl(const int64_t *__restrict__ ts,
                                                 const int32_t *__restrict__ ctx, int64_t E,
                                                 const v2ll *__restrict__ bounds, int64_t n_sel, int N,
                                                 int64_t t0, int64_t t1, const WinCounts *__restrict__ wc,
                                                 int fit, int64_t *__restrict__ excl, uint32_t *err) {
  extern __shared__ __align__(16) uint64_t hist[];  // [N] when LDSH, else one NodeSums
  __shared__ int64_t wtot[WWT / 64], cut[4];
  __shared__ int full;  // a node found no slot
  NodeSums &sums = *reinterpret_cast<NodeSums *>(hist);
  const int t = threadIdx.x;
  // uniform over the grid
  constexpr int64_t MIN_SHARE = LDSH ? 32768 : 4096;  // a histogram's flush costs more
  const WinCounts n = wc ? *wc : WinCounts{0, 0, 0};
  const int64_t total = (int64_t)n.total, longest = (int64_t)n.longest, have = (int64_t)n.ranks;
  const bool table = !LDSH && total >= TABLE_MIN && total >= have * TABLE_MEAN;
  const int64_t wgs = table && fit < (int)gridDim.x ? fit : gridDim.x;
  const bool split = n_sel <= BAL_SEL && (table || (longest > 2 * MIN_SHARE && longest * wgs > 2 * total));
  const bool by_wave = !table && !split && total < have * WAVE_MEAN;
  // this workgroup's ranks i, i + next, ... below `last`; split: of rank i from its
  // event cut[1] on, of rank last - 1 up to its event cut[3]
  int64_t i = blockIdx.x, last = n_sel, next = gridDim.x;
  if (split) {
    const int64_t all = total + n_sel * RANK_W;
    int64_t parts = all / MIN_SHARE + 1;
    parts = parts < wgs ? parts : wgs;
    // quads of a rank stay together where its events start at a multiple of 4
    const int64_t share = (((all + parts - 1) / parts) + 3) & ~(int64_t)3;
    const int64_t from = share * blockIdx.x, to = from + share < all ? from + share : all;
    if (from >= all) return;
    const int per = (int)((n_sel + WWT - 1) / WWT), lane = t & 63, wid = t >> 6;
    int64_t own = 0;
    for (int j = 0; j < per; j++) {
      const int64_t r = (int64_t)t * per + j;
      if (r >= n_sel) break;
      const v2ll b = bounds[2 * r];
      own += RANK_W + (b.y > b.x ? b.y - b.x : 0);
    }
    int64_t in = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int64_t y = __shfl_up(in, d, 64);
      if (lane >= d) in += y;
    }
    if (lane == 63) wtot[wid] = in;
    __syncthreads();
    for (int w = 0; w < WWT / 64; w++) in += w < wid ? wtot[w] : 0;
    // the ranks that hold places `from` and `to - 1`: one thread each
    auto find = [&](int64_t x, int64_t *c) {
      if (in - own > x || x >= in) return;
      int64_t at = in - own;
      for (int64_t r = (int64_t)t * per;; r++) {
        const v2ll b = bounds[2 * r];
        const int64_t n = RANK_W + (b.y > b.x ? b.y - b.x : 0);
        if (x < at + n) {
          c[0] = r;
          c[1] = x - at;
          break;
        }
        at += n;
      }
    };
    find(from, cut);
    find(to - 1, cut + 2);
    __syncthreads();
    i = uniform(cut[0]);
    last = uniform(cut[2]) + 1;
    next = 1;
  } else if (table) {  // many ranks: neighbouring ones
    if ((int64_t)blockIdx.x >= wgs) return;
    i = n_sel * blockIdx.x / wgs;
    last = n_sel * (blockIdx.x + 1) / wgs;
    next = 1;
  } else if (by_wave) {
    if (i * (WWT / 64) >= n_sel) return;
    i = i * (WWT / 64) + __builtin_amdgcn_readfirstlane(t >> 6);
    next *= WWT / 64;
  }
  if (!by_wave && i >= last) return;  // uniform
  if (LDSH) {
    for (int v = t; v < N; v += WWT) hist[v] = 0;
  } else if (table) {
    sums.clear(t, WWT);
    if (t == 0) full = 0;
  }
  if (LDSH || table) __syncthreads();
  // visit(lo, hi, e) for the events of each rank
  auto ranks = [&](auto &&visit) {
    for (; i < last; i += next) {
      const v2ll b0 = bounds[2 * i], b1 = bounds[2 * i + 1];
      int64_t lo = b0.x, hi = b0.y;
      if (split) {
        if (i == uniform(cut[0])) lo += uniform(cut[1]);
        const int64_t end = b0.x + uniform(cut[3]) + 1;
        if (i == last - 1 && hi > end) hi = end;
      }
      visit(lo, hi, b1.x);
    }
  };
  auto part = [&](int64_t s, int64_t f, int32_t c) -> uint64_t {  // of an event, in the window
    if (f < s) atomicOr(err, ERRBIT_UNSORTED);
    const int64_t a = s > t0 ? s : t0;
    const int64_t z = f < t1 ? f : t1;
    if (z <= a) return 0;
    if (c >= 0 && c < N) return (uint64_t)(z - a);
    atomicOr(err, ERRBIT_CTX);
    return 0;
  };
  if (table) {
    ranks([&](int64_t lo, int64_t hi, int64_t e) {
      visit_quads<2>(ts, ctx, E, lo, hi, e, t, WWT, [&](int64_t k0, const EvQuad &q) {
        uint64_t d[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
          const int64_t k = k0 + u;
          d[u] = k >= lo && k < hi ? part(q.t[u], k + 1 < e ? q.t[u + 1] : q.t[u], q.c[u]) : 0;
        }
        sums.add4(q.c, d, *(volatile int *)&full ? 1 : NodeSums::PROBES, [&](int32_t c, uint64_t v) {
          full = 1;
          atomicAdd((unsigned long long *)&excl[c], (unsigned long long)v);
        });
      });
    });
  } else {
    auto add = [&](int64_t, int64_t s, int64_t f, int32_t c) {
      const uint64_t d = part(s, f, c);
      if (d) atomicAdd((unsigned long long *)(LDSH ? &hist[c] : (uint64_t *)&excl[c]), (unsigned long long)d);
    };
    if (by_wave)
      ranks([&](int64_t lo, int64_t hi, int64_t e) { visit_events<1>(ts, ctx, E, lo, hi, e, t & 63, 64, add); });
    else
      ranks([&](int64_t lo, int64_t hi, int64_t e) { visit_events<2>(ts, ctx, E, lo, hi, e, t, WWT, add); });
  }
  if (!LDSH && !table) return;
  __syncthreads();
  if (LDSH) {
    for (int v = t; v < N; v += WWT)
      if (hist[v]) atomicAdd((unsigned long long *)&excl[v], (unsigned long long)hist[v]);
  } else {
    for (int k = t; k < HSLOTS; k += WWT)
      if (sums.key[k] >= 0)
        atomicAdd((unsigned long long *)&excl[sums.key[k]], (unsigned long long)sums.sum[k]);
  }
}

// ---- sparse per-rank profiles --------------------------------------------------

constexpr int SPT = 1024;               // threads per rank workgroup
constexpr int SPC = 8192;               // node ids per chunk (64 KB LDS histogram)
constexpr int SPE = SPC / SPT;          // bins per thread in the compaction
constexpr int SPW = MAX_NODES / SPC / 32;  // words of the touched-chunk mask
constexpr int SPBW = 4096;              // node-mask words: trees of up to 131,072 nodes take one pass
constexpr int SPBT = SPBW / SPT;        // mask words per thread
constexpr int SPACC = 4096;             // distinct nodes a rank may reach on the one-pass path

// Exclusive scan of per-thread counts over the workgroup; *total = the sum.
__device__ inline int block_excl_scan_i32(int v, int *wsum, int *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d, 64);
    if (lane >= d) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll
  for (int i = 0; i < SPT / 64; i++) {
    const int s = wsum[i];
    base += i < w ? s : 0;
    all += s;
  }
  __syncthreads();
  *total = all;
  return base + x - v;
}

// One workgroup per rank (grid-stride).  Trees of more than SPC nodes and at
// most SPBW * 32: a pass over the events' contexts (4 bytes per event) marks
// the nodes they reach in an LDS bit mask; a workgroup scan of the mask's word
// counts gives each reached node an accumulator index (ascending id); a
// second pass adds the durations into the LDS accumulator at those indices
// (exact 64-bit atomics), and the nodes with a positive total are written in
// ascending id (a second scan of the per-thread counts of those).  Otherwise,
// or when a rank reaches more than SPACC nodes:
// for each chunk of SPC node ids that the events reach, an LDS histogram of
// the chunk, then its non-zero bins in ascending id, compacted by a workgroup
// scan and appended after the previous chunks'.  Output goes to the rank's own
// event range.
__global__ __launch_bounds__(SPT) void sparse_profiles_kernel(const int64_t *__restrict__ off,
                                                             const int64_t *__restrict__ ts,
                                                             const int32_t *__restrict__ ctx,
                                                             int64_t R, int64_t E, int N,
                                                             int64_t *__restrict__ counts,
                                                             int32_t *__restrict__ ids,
                                                             int64_t *__restrict__ vals,
                                                             uint32_t *err) {
  __shared__ uint64_t pool[SPC];  // chunk histogram, or mask | word prefixes | accumulator
  __shared__ uint32_t touched[SPW];
  __shared__ int wsum[SPT / 64];
  uint64_t *hist = pool;
  uint32_t *bm = reinterpret_cast<uint32_t *>(pool);
  uint32_t *pre = bm + SPBW;
  uint64_t *acc = pool + SPBW;
  const int n_chunks = (N + SPC - 1) / SPC;
  const bool one_pass = n_chunks > 1 && N <= SPBW * 32;
  const int nw = (N + 31) / 32;
  const int t = threadIdx.x;
  for (int64_t r = blockIdx.x; r < R; r += gridDim.x) {
    // a rank's range, clamped to [0, E] (inconsistent offsets are an error)
    const int64_t o0 = off[r], o1 = off[r + 1];
    const bool bad = o0 < 0 || o1 < o0 || o1 > E;
    const int64_t b = bad ? 0 : o0, e = bad ? 0 : o1;
    if (bad && t == 0) atomicOr(err, ERRBIT_OFFSETS);
    auto dur = [&](int64_t k) -> int64_t { return k + 1 < e ? ts[k + 1] - ts[k] : 0; };
    int64_t base = 0;
    bool done = false;
    if (one_pass) {
      for (int i = t; i < nw; i += SPT) bm[i] = 0;
      __syncthreads();
      // the nodes the rank's events reach, from the contexts alone (4 bytes
      // per event; the durations are read once, by the accumulating pass)
      for (int64_t k0 = (b & ~(int64_t)3) + 4 * (int64_t)t; k0 < e; k0 += 4 * (int64_t)SPT) {
        int32_t c4[4];
        if (k0 + 4 <= E) {
          const v4i q = *reinterpret_cast<const v4i *>(ctx + k0);
          c4[0] = q.x;
          c4[1] = q.y;
          c4[2] = q.z;
          c4[3] = q.w;
        } else {
#pragma unroll
          for (int u = 0; u < 4; u++) c4[u] = k0 + u < E ? ctx[k0 + u] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; u++) {
          if (k0 + u < b || k0 + u >= e) continue;
          const int32_t c = c4[u];
          if (c < 0 || c >= N) atomicOr(err, ERRBIT_CTX);
          else atomicOr(&bm[c >> 5], 1u << (c & 31));
        }
      }
      __syncthreads();
      uint32_t wv[SPBT];
      int own = 0;
#pragma unroll
      for (int u = 0; u < SPBT; u++) {
        const int w = t * SPBT + u;
        wv[u] = w < nw ? bm[w] : 0u;
        own += __popc(wv[u]);
      }
      int total;
      int pos = block_excl_scan_i32(own, wsum, &total);
#pragma unroll
      for (int u = 0; u < SPBT; u++) {
        const int w = t * SPBT + u;
        if (w < nw) pre[w] = (uint32_t)pos;
        pos += __popc(wv[u]);
      }
      if (total <= SPACC) {  // uniform
        for (int i = t; i < total; i += SPT) acc[i] = 0;
        __syncthreads();
        visit_events<1>(ts, ctx, E, b, e, e, t, SPT, [&](int64_t, int64_t s, int64_t f, int32_t c) {
          const int64_t d = f - s;
          if (d < 0) atomicOr(err, ERRBIT_UNSORTED);
          if (c >= 0 && c < N && d > 0) {
            const int w = c >> 5;
            const int idx = (int)pre[w] + __popc(bm[w] & ((1u << (c & 31)) - 1u));
            atomicAdd((unsigned long long *)&acc[idx], (unsigned long long)d);
          }
        });
        __syncthreads();
        // the reached nodes with a positive total, in ascending id: a node
        // reached only by zero durations is marked but not written
        int nz = 0;
#pragma unroll
        for (int u = 0; u < SPBT; u++) {
          const int w = t * SPBT + u;
          if (w >= nw) continue;
          const int p0 = (int)pre[w];
          for (int q = 0; q < __popc(wv[u]); q++) nz += acc[p0 + q] != 0 ? 1 : 0;
        }
        int nz_total;
        int o = block_excl_scan_i32(nz, wsum, &nz_total);
#pragma unroll
        for (int u = 0; u < SPBT; u++) {
          const int w = t * SPBT + u;
          if (w >= nw) continue;
          uint32_t m = wv[u];
          int p = (int)pre[w];
          while (m) {
            const int j = __ffs(m) - 1;
            m &= m - 1u;
            if (acc[p] != 0) {
              ids[b + o] = w * 32 + j;
              vals[b + o] = (int64_t)acc[p];
              o++;
            }
            p++;
          }
        }
        base = nz_total;
        done = true;
      }
      __syncthreads();
    }
    if (!done) {
      if (n_chunks > 1) {
        for (int i = t; i < SPW; i += SPT) touched[i] = 0;
        __syncthreads();
        for (int64_t k = b + t; k < e; k += SPT) {
          const int32_t c = ctx[k];
          if (c >= 0 && c < N && dur(k) > 0) atomicOr(&touched[(c / SPC) >> 5], 1u << ((c / SPC) & 31));
        }
        __syncthreads();
      }
      for (int ch = 0; ch < n_chunks; ch++) {
        if (n_chunks > 1 && !((touched[ch >> 5] >> (ch & 31)) & 1u)) continue;  // uniform
        const int lo = ch * SPC;
        for (int i = t; i < SPC; i += SPT) hist[i] = 0;
        __syncthreads();
        visit_events<1>(ts, ctx, E, b, e, e, t, SPT, [&](int64_t, int64_t s, int64_t f, int32_t c) {
          const int64_t d = f - s;
          if (d < 0) atomicOr(err, ERRBIT_UNSORTED);
          if (c < 0 || c >= N) {
            if (ch == 0) atomicOr(err, ERRBIT_CTX);
          } else if (c >= lo && c < lo + SPC && d != 0) {
            atomicAdd((unsigned long long *)&hist[c - lo], (unsigned long long)d);
          }
        });
        __syncthreads();
        uint64_t v[SPE];
        int nz = 0;
#pragma unroll
        for (int u = 0; u < SPE; u++) {
          v[u] = hist[t * SPE + u];
          nz += v[u] != 0 ? 1 : 0;
        }
        int total;
        int pos = block_excl_scan_i32(nz, wsum, &total);
#pragma unroll
        for (int u = 0; u < SPE; u++)
          if (v[u] != 0) {
            const int64_t o = b + base + pos++;
            ids[o] = lo + t * SPE + u;
            vals[o] = (int64_t)v[u];
          }
        base += total;
        __syncthreads();
      }
    }
    if (t == 0) counts[r] = base;
    __syncthreads();
  }
}

int grid_w(int64_t n, int cus, int per_cu) {
  int64_t g = n < (int64_t)cus * per_cu ? n : (int64_t)cus * per_cu;
  return g < 1 ? 1 : (int)g;
}

}  // namespace

// The subtree-sum workspace, then the window's counts and 32 bytes of event
// bounds per selected rank.
size_t window_ws_bytes(int N, int64_t n_sel) {
  return ((subtree_sums_ws_bytes(N) + 255) & ~(size_t)255) + 32 + (size_t)(n_sel > 0 ? n_sel : 0) * 32;
}

hipError_t launch_window_profile(const int64_t *off, const int64_t *ts, const int32_t *ctx, int64_t R,
                                 int64_t E, const int32_t *ids, int64_t n_sel, int N, const int2 *tin_tout,
                                 int64_t t0, int64_t t1, int64_t *excl, int64_t *incl, void *ws,
                                 uint32_t *err, int cus, hipStream_t s) {
  WinCounts *wc = reinterpret_cast<WinCounts *>(static_cast<char *>(ws) +
                                                ((subtree_sums_ws_bytes(N) + 255) & ~(size_t)255));
  v2ll *bounds = reinterpret_cast<v2ll *>(reinterpret_cast<char *>(wc) + 32);
  if (E < COUNT_MIN) wc = nullptr;
  zero_i64<<<grid_w((N + WT - 1) / WT, cus, 4), WT, 0, s>>>(excl, N, n_sel > 0 ? wc : nullptr);
  if (n_sel > 0) {
    window_bounds<<<(unsigned)((n_sel + WT - 1) / WT), WT, 0, s>>>(off, ts, R, E, ids, n_sel, t0, t1,
                                                                   bounds, wc, err);
    // a workgroup per rank, or more where few ranks may hold many events
    const int grid = grid_w(n_sel > E / 4096 ? n_sel : E / 4096, cus, 4);
    if (N <= MAX_NODES_ATTR) {
      static bool attr = false;
      if (!attr) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&window_excl<true>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);
        attr = true;
      }
      window_excl<true><<<grid, WWT, (size_t)N * 8, s>>>(ts, ctx, E, bounds, n_sel, N, t0, t1, wc, 3 * cus,
                                                         excl, err);
    } else {
      window_excl<false><<<grid, WWT, sizeof(NodeSums), s>>>(ts, ctx, E, bounds, n_sel, N, t0, t1, wc,
                                                             3 * cus, excl, err);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !incl) return e;
  return launch_subtree_sums(excl, N, tin_tout, incl, ws, cus, s);
}

hipError_t launch_sparse_profiles(const int64_t *off, const int64_t *ts, const int32_t *ctx, int64_t R,
                                  int64_t E, int N, int64_t *counts, int32_t *ids, int64_t *vals, uint32_t *err,
                                  int cus, hipStream_t s) {
  if (R <= 0) return hipSuccess;
  // Ranks that take more than a step of the workgroup on average differ in how
  // many: a workgroup per rank, placed as others end (3,000 ranks of 20,000 events
  // at the median, lognormal, over 97,833 nodes: 420 us, two workgroups per CU in
  // turns 474; all of 20,000 events: 218 and 209).  Shorter ranks: in turns, which
  // saves the launch of a workgroup (100,000 ranks of 20 events over 5,000 nodes: 1,329
  // and 1,270 us).
  const int per_cu = E / R >= 4 * SPT ? 64 : 2;
  sparse_profiles_kernel<<<grid_w(R, cus, per_cu), SPT, 0, s>>>(off, ts, ctx, R, E, N, counts, ids, vals, err);
  return hipGetLastError();
}

}  // namespace ta
