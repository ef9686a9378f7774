// k_colscan.hip -- the robust FULL scan's first stage for at most COL_REG_MAX
// ranks: per column (iteration, region) the median and the median absolute
// deviation over the ranks, and the ranks' mean scores.
//
//   up to COL_DIRECT_MAX ranks   col_select_direct reads the row-major tensor
//                 (a workgroup's columns side by side, tiles of rows through
//                 LDS into the registers of the wave that owns a column), and
//                 score_rank (up to 256 regions; else score_tensor) reads it again
//   more ranks    col_copy writes a column-major copy in 32-bit offsets,
//                 col_select reads a column of it into the registers of a
//                 workgroup, score_copy reads it again; the columns whose cells
//                 do not fit in 32 bits are listed there, copied in two 32-bit
//                 halves by col_copy_wide and selected by col_select_wide
// Everything between the count of a column and its MAD happens on registers
// (ta_select.h), but for the few that the compiler keeps in scratch (sel_waves).  The row-major passes of longer columns (k_outliers.hip) took
// 10.0 ms for 32,000 columns of 40,000 ranks where this takes 7.1.
#include <algorithm>
#include <type_traits>

#include "ta_device.h"
#include "ta_scan.h"
#include "ta_select.h"

namespace ta {
namespace {

typedef long long v2ll __attribute__((ext_vector_type(2)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

constexpr int64_t COL_DIRECT_MAX = 1024;

// Key words.  64 bits: cell + HALF64.  32 bits: cell - base + HALF32, base the
// cell of rank 0 in that column (whatever it holds), or a mark when that does
// not fit: FAR_LOW below every key, FAR_HIGH above.  NONE: a cell that the rank
// does not have.
constexpr int64_t HALF64 = (int64_t)1 << 62;
constexpr int64_t HALF32 = 0x7fffffffll;
constexpr uint32_t FAR_LOW = 0, FAR_HIGH = 0xfffffffeu;
template <typename K>
constexpr K none() {
  return ~(K)0;
}

constexpr int CT = 128;  // ranks per tile of the copy; its columns are padded to this
__host__ __device__ inline int64_t copy_ranks(int64_t R) { return (R + CT - 1) / CT * CT; }

// Column-major copy cp[IG][copy_ranks(R)] of the tensor in 32-bit key words:
// 64 columns x 128 ranks per workgroup, all 16 loads of a thread in flight, 512-byte pieces of rows in and of columns out.  Bound by
// HBM (12 bytes per cell): 9,600 columns of 10,000 ranks in 229 us, 5.0 TB/s
// (an 8-byte copy, with the statistics, 358 us).  Several tiles
// per workgroup were slower (330 -> 537 us for 16,000 ranks): one tile's loads
// wait for the other's stores.
// STATS: also each column's valid cells as one chunk of the imbalance partials
// per workgroup.  The copy leaves the VALU some room for it (233 -> 267 us), the
// selection does not (206 -> 311 us).
struct ColSum {  // exact, over any cells of one column
  int64_t s1;
  uint64_t lo, hi;  // 128-bit sum of squares
  int64_t mn, mx;
  uint32_t n;
  __device__ void add(const ColSum &o) {
    const u128 q = (((u128)hi << 64) | lo) + (((u128)o.hi << 64) | o.lo);
    n += o.n;
    s1 += o.s1;
    lo = (uint64_t)q;
    hi = (uint64_t)(q >> 64);
    mn = o.mn < mn ? o.mn : mn;
    mx = o.mx > mx ? o.mx : mx;
  }
};

template <bool STATS>
__global__ __launch_bounds__(256, 4) void col_copy(const int64_t *__restrict__ T, int64_t R, int IG, int G,
                                                const int32_t *__restrict__ it, uint32_t *__restrict__ cp,
                                                uint32_t *n_wide, uint8_t *group, ColPartials ps) {
  constexpr int LD = CT + 4;  // 16-byte rows, columns four banks apart
  union Lds {
    uint32_t tile[64 * LD];
    ColSum sum[8][64];
    __device__ Lds() {}
  };
  __shared__ Lds L;
  if (blockIdx.x == 0 && threadIdx.x == 0) {  // col_select adds to them
    group[blockIdx.y] = 0;
    if (blockIdx.y == 0) *n_wide = 0;
  }
  const int c0 = (int)blockIdx.y * 64;
  const int64_t Rp = copy_ranks(R);
  const int p2 = 2 * (threadIdx.x & 31), k0 = threadIdx.x >> 5;
  const int ca = c0 + p2, ia = ca / G, ib = (ca + 1) / G;
  const bool vec = (IG & 1) == 0, ha = ca < IG, hb = ca + 1 < IG;
  const int64_t base[2] = {ha ? T[ca] : 0, hb ? T[ca + 1] : 0};
  ColSum tot[2];
#pragma unroll
  for (int h = 0; h < 2; h++) tot[h] = ColSum{0, 0, 0, INT64_MAX, INT64_MIN, 0};
  constexpr int U = CT / 8;
  const int64_t r0 = (int64_t)blockIdx.x * CT;
  v2ll x[U];
  int nit[U];
#pragma unroll
  for (int k = 0; k < U; k++) {
    const int64_t r = r0 + k0 + 8 * k;
    x[k] = v2ll{0, 0};
    nit[k] = 0;
    if (r < R) {
      nit[k] = it ? it[r] : 0x7fffffff;
      const int64_t *row = T + r * IG + ca;
      if (vec) {
        if (ha) x[k] = __builtin_nontemporal_load(reinterpret_cast<const v2ll *>(row));
      } else {
        if (ha) x[k].x = __builtin_nontemporal_load(row);
        if (hb) x[k].y = __builtin_nontemporal_load(row + 1);
      }
    }
  }
#pragma unroll
  for (int h = 0; h < 2; h++) {
    bool far = false;  // an offset of 2^29 and more
    int64_t sum = 0;
    uint64_t sq = 0;
    int32_t mn = INT32_MAX, mx = INT32_MIN;
    uint32_t n = 0;
#pragma unroll
    for (int k = 0; k < U; k++) {
      const bool in = h == 0 ? ha && ia < nit[k] : hb && ib < nit[k];
      const int64_t d = (int64_t)(h == 0 ? x[k].x : x[k].y) - base[h];
      const uint32_t w = d >= HALF32 ? FAR_HIGH : d <= -HALF32 ? FAR_LOW : (uint32_t)(d + HALF32);
      L.tile[(p2 + h) * LD + k0 + 8 * k] = in ? w : none<uint32_t>();
      if (STATS) {
        far |= in && w - (uint32_t)(HALF32 - (1 << 29)) > 1u << 30;  // marks too
        const int32_t e = in ? (int32_t)d : 0;
        const uint32_t m = (uint32_t)(e < 0 ? -e : e);
        n += in ? 1u : 0u;
        sum += e;
        sq += (uint64_t)m * m;
        mn = in && e < mn ? e : mn;
        mx = in && e > mx ? e : mx;
      }
    }
    if (STATS && !far && n > 0) {
      // sum (base + d)^2 = n base^2 + 2 base sum d + sum d^2, exactly
      const i128 b = base[h];
      const u128 q = (u128)((i128)n * b * b + 2 * b * (i128)sum) + sq;
      tot[h].add(ColSum{(int64_t)n * base[h] + sum, (uint64_t)q, (uint64_t)(q >> 64), base[h] + mn,
                        base[h] + mx, n});
    }
    if (STATS && far) {
#pragma unroll 1
      for (int k = 0; k < U; k++) {
        const int64_t r = r0 + k0 + 8 * k;
        const int c = ca + h;
        if (r >= R || c >= IG || (it && c / G >= it[r])) continue;
        const int64_t v = T[r * IG + c];
        const u128 q = (u128)((i128)v * v);
        tot[h].add(ColSum{v, (uint64_t)q, (uint64_t)(q >> 64), v, v, 1});
      }
    }
  }
  __syncthreads();
  const int q = 4 * (threadIdx.x & 31);
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int c = k0 + 8 * k;
    if (c0 + c < IG)
      *reinterpret_cast<v4u *>(cp + (int64_t)(c0 + c) * Rp + r0 + q) =
          *reinterpret_cast<const v4u *>(&L.tile[c * LD + q]);
  }
  if (STATS) {
    __syncthreads();
    L.sum[k0][p2] = tot[0];
    L.sum[k0][p2 + 1] = tot[1];
    __syncthreads();
    const int c = c0 + (int)threadIdx.x;
    if (threadIdx.x < 64 && c < IG) {
      ColSum s = L.sum[0][threadIdx.x];
      for (int k = 1; k < 8; k++) s.add(L.sum[k][threadIdx.x]);
      const int64_t p = (int64_t)blockIdx.x * IG + c;
      ps.n[p] = s.n;
      ps.s1[p] = s.s1;
      ps.lo[p] = s.lo;
      ps.hi[p] = s.hi;
      ps.mn[p] = s.mn;
      ps.mx[p] = s.mx;
    }
  }
}

// What the waves of a column exchange.
struct ColRed {
  uint64_t mn, mx, a;
  uint32_t n, m, low;
};

struct ColOut {
  ColZ *cz;
  double *mu;      // 32-bit form: the median in doubled key words, as a double; negative where the
                   // column has far cells; NaN for a wide column
  uint32_t *wide;  // 32-bit form: the number of wide columns, then the columns
  uint8_t *group;  // 32-bit form: 1 where any of 64 columns is wide
  ColPartials ps;
};

// From a column's key words in the registers of a group of W waves (u[V] per
// lane) to its coefficients, and with STATS its imbalance statistics.  `off` is
// what a key word of 0 stands for.  32-bit form: cells marked as far count below
// or above the others, which is all that the median needs while it is not one of
// them, and the MAD while it does not exceed their smallest possible deviation
// (so a few stalled ranks cost nothing).  A column of which that does not hold, or
// whose other cells span 2^31 and more, is listed for col_select_wide.
template <typename K, int V, int W, int NB, bool STATS>
__device__ __forceinline__ void select_column(K (&u)[V], SelGroup<W, NB, K> &S, ColRed *red, int64_t off,
                                              int col, bool have, const ColOut &o) {
  constexpr bool NARROW = sizeof(K) == 4;
  static_assert(!STATS || (W == 1 && !NARROW), "statistics: 64-bit words, one wave");
  const int lane = (int)(threadIdx.x & 63), sw = (int)(threadIdx.x >> 6) % W;
  const bool mine = sw == 0 && lane == 0 && have;
  uint32_t n = 0, marks = 0, low = 0;  // marks: cells that are far; low: below
  K mn = none<K>(), mx = 0;  // mx: the largest + 1 (0 for none)
#pragma unroll
  for (int v = 0; v < V; v++) {
    n += u[v] != none<K>() ? 1u : 0u;
    mn = u[v] < mn ? u[v] : mn;
    const K w = u[v] + 1;
    mx = w > mx ? w : mx;
    pace(v);
  }
  mn = wave_min(mn);
  mx = wave_max(mx);
  n = wave_sum(n);
  if (W > 1) {
    if (lane == 0) {
      red[sw].mn = mn;
      red[sw].mx = mx;
      red[sw].n = n;
    }
    __syncthreads();
    n = 0;
#pragma unroll
    for (int q = 0; q < W; q++) {
      mn = (K)red[q].mn < mn ? (K)red[q].mn : mn;
      mx = (K)red[q].mx > mx ? (K)red[q].mx : mx;
      n += red[q].n;
    }
    __syncthreads();
  }
  if (NARROW && (mn == (K)FAR_LOW || mx > (K)FAR_HIGH)) {  // uniform; the same without the marks
    mn = none<K>();
    mx = 0;
#pragma unroll
    for (int v = 0; v < V; v++) {
      const bool lo = u[v] == (K)FAR_LOW, key = u[v] - 1 < (K)FAR_HIGH - 1;
      low += lo ? 1u : 0u;
      marks += lo || u[v] == (K)FAR_HIGH ? 1u : 0u;
      mn = key && u[v] < mn ? u[v] : mn;
      mx = key && u[v] + 1 > mx ? u[v] + 1 : mx;
      pace(v);
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    low = wave_sum(low);
    marks = wave_sum(marks);
    if (W > 1) {
      if (lane == 0) {
        red[sw].mn = mn;
        red[sw].mx = mx;
        red[sw].m = marks;
        red[sw].low = low;
      }
      __syncthreads();
      marks = low = 0;
#pragma unroll
      for (int q = 0; q < W; q++) {
        mn = (K)red[q].mn < mn ? (K)red[q].mn : mn;
        mx = (K)red[q].mx > mx ? (K)red[q].mx : mx;
        marks += red[q].m;
        low += red[q].low;
      }
      __syncthreads();
    }
  }
  const uint32_t keys = n - marks;
  const K range = keys > 0 ? (K)(mx - 1 - mn) : 0;
  const uint32_t k = n > 0 ? (n - 1) / 2 : 0, two = n > 0 && (n & 1) == 0 ? 1u : 0u;
  const bool even = two != 0;
  auto list_wide = [&]() {  // the whole group returns
    if (mine) {
      o.wide[1 + atomicAdd(o.wide, 1u)] = (uint32_t)col;
      o.group[col / 64] = 1;
      o.mu[col] = nan_f64();
    }
  };
  // deviations |2u - med2| of 32-bit offsets need twice the range; with marks,
  // both middle cells and both middle deviations have to be keys
  if (NARROW && n > 0 && (range > (K)0x7ffffffeu || k < low || k - low + two >= keys || k + two >= keys)) {
    list_wide();
    return;
  }

  // offsets from the smallest cell (a word that is no key stays above `range`)
  uint32_t zeros = 0;
  uint64_t su = 0;
  u128 tot = 0;
#pragma unroll
  for (int v = 0; v < V; v++) {
    if (STATS && u[v] != none<K>()) {
      const int64_t x = (int64_t)(u[v] - (K)HALF64);
      su += (uint64_t)x;
      tot += (u128)((i128)x * x);
    }
    u[v] = u[v] - mn;
    zeros += u[v] == 0 ? 1u : 0u;
    pace(v);
  }
  zeros = wave_sum(zeros);
  if (W > 1) {
    if (lane == 0) red[sw].m = zeros;
    __syncthreads();
    zeros = 0;
#pragma unroll
    for (int q = 0; q < W; q++) zeros += red[q].m;
    __syncthreads();
  }
  if (STATS) {
    // 32-bit pieces of the 128-bit totals, summed apart
    const uint64_t p0 = wave_sum((uint64_t)(uint32_t)tot), p1 = wave_sum((uint64_t)(uint32_t)(tot >> 32)),
                   p2 = wave_sum((uint64_t)(tot >> 64));
    tot = (u128)p0 + ((u128)p1 << 32) + ((u128)p2 << 64);
    su = wave_sum(su);
    if (mine) {
      const int64_t lo = off + (int64_t)mn;  // the smallest cell
      o.ps.n[col] = n;
      o.ps.s1[col] = (int64_t)su;
      o.ps.lo[col] = (uint64_t)tot;
      o.ps.hi[col] = (uint64_t)(tot >> 64);
      o.ps.mn[col] = n > 0 ? lo : INT64_MAX;
      o.ps.mx[col] = n > 0 ? lo + (int64_t)range : INT64_MIN;
    }
  }
  if (n == 0) {
    if (mine) {
      o.cz[col] = ColZ{0, 0.0, 1.0, 1.0};
      if (NARROW) o.mu[col] = 0.0;
    }
    return;
  }

  // the median, then the MAD of |2u - med2|
  const uint32_t km = k - low;
  K a = 0, b = 0;
  if (km + two >= zeros)  // else both middle cells are the smallest
    reg_select<true>(S, u, (K)0, zeros, range, nbits64(range), keys, km, even, a, b);
  const K m2 = a + b;
  uint32_t hits = 0;  // deviations equal to med2: the smallest cells', which may be many
#pragma unroll
  for (int v = 0; v < V; v++) {
    const K t = 2 * u[v];
    const K d = t > m2 ? t - m2 : m2 - t;
    u[v] = u[v] <= range ? d : none<K>();
    hits += u[v] == m2 ? 1u : 0u;
    pace(v);
  }
  hits = wave_sum(hits);
  if (W > 1) {
    if (lane == 0) red[sw].m = hits;
    __syncthreads();
    hits = 0;
#pragma unroll
    for (int q = 0; q < W; q++) hits += red[q].m;
  }
  const K far = (K)(2 * range - m2), dmax = far > m2 ? far : m2;
  a = b = 0;
  if (m2 != 0 || k + two >= zeros)  // else both middle deviations are 0
    reg_select<true>(S, u, m2, hits, dmax, nbits64(dmax), keys, k, even, a, b);
  const uint64_t mad4 = (uint64_t)a + (uint64_t)b;
  if (NARROW && marks > 0) {
    // a far cell's deviation is at least that of the mark itself; the mean
    // deviation, wanted when the MAD is 0, needs the cells
    const uint64_t med = 2 * (uint64_t)mn + (uint64_t)m2, hi = 2 * (uint64_t)FAR_HIGH - med;
    if (mad4 == 0 || (uint64_t)b > (med < hi ? med : hi)) {
      list_wide();
      return;
    }
  }
  uint64_t sd = 0;  // the sum of the deviations is wanted when the MAD is 0
  if (mad4 == 0) {
#pragma unroll
    for (int v = 0; v < V; v++) sd += u[v] <= dmax ? (uint64_t)u[v] : 0;
    sd = wave_sum(sd);
    if (W > 1) {
      if (lane == 0) red[sw].a = sd;
      __syncthreads();
      sd = 0;
      for (int q = 0; q < W; q++) sd += red[q].a;
    }
  }
  if (mine) {
    ColZ z;
    z.med2 = 2 * (off + (int64_t)mn) + (int64_t)m2;
    z_coefs((int64_t)mad4, (int64_t)sd, (int64_t)n, z.zc, z.zd);
    z.zy = 1.0 / z.zd;
    o.cz[col] = z;
    const double mu = (double)(2 * (uint64_t)mn + (uint64_t)m2);  // above 0
    if (NARROW) o.mu[col] = marks > 0 ? -mu : mu;
  }
}

template <int W, int V>
constexpr int col_bins() {  // 4 to 16 bins per lane of a single wave, else 2,048
  return W > 1 ? 2048 : (V <= 4 ? 256 : V <= 8 ? 512 : 1024);
}

// Waves per SIMD that V key words and what else a lane needs leave room for (the
// compiler takes up to twice the registers when it is not told; so it keeps 2 to 26
// registers of the rarer branches in scratch).
template <int V>
constexpr int sel_waves() {
  return V <= 32 ? 8 : V <= 48 ? 6 : V <= 64 ? 5 : 4;
}

// Columns of the 32-bit copy: W waves and V key words per lane each; a single
// wave's columns come four to a workgroup.  Radix passes over the column in
// memory took 566 us for 9,600 columns of 10,000 ranks and 1,296 us for 11,520
// of 9,190; this takes 219 and 240 us, bound by its instructions (about 30 per
// key) and the LDS atomics (a quarter of the time).
template <int W, int V>
__global__ __launch_bounds__(W > 1 ? 64 * W : 256, sel_waves<V>()) void col_select(const uint32_t *__restrict__ cp, int64_t R,
                                                                   int IG, const int64_t *__restrict__ T,
                                                                   ColOut o) {
  constexpr int C = W > 1 ? 1 : 4, NB = col_bins<W, V>();
  __shared__ SelGroup<W, NB, uint32_t> L[C];
  __shared__ ColRed red[W];
  const int cl = W > 1 ? 0 : (int)(threadIdx.x >> 6), t = (int)(threadIdx.x % (64 * W));
  const int col = (int)blockIdx.x * C + cl;
  if (col >= IG) return;  // a whole group; single waves meet no workgroup barrier
  const int64_t Rp = copy_ranks(R);
  const uint32_t *p = cp + (int64_t)col * Rp;
  uint32_t u[V];
#pragma unroll
  for (int v = 0; v < V; v += 4) {
    const int64_t r = (int64_t)(v / 4) * 256 * W + 4 * t;
    v4u q = {none<uint32_t>(), none<uint32_t>(), none<uint32_t>(), none<uint32_t>()};
    if (r < Rp) q = *reinterpret_cast<const v4u *>(p + r);
    u[v] = q.x;
    u[v + 1] = q.y;
    u[v + 2] = q.z;
    u[v + 3] = q.w;
  }
  const int64_t off = T[col] - HALF32;
  sel_clear(L[cl]);
  select_column<uint32_t, V, W, NB, false>(u, L[cl], red, off, col, true, o);
}

// The wide columns' keys in two 32-bit halves, the low words in their place of the
// 32-bit copy, the high words in hi[IG][copy_ranks(R)]: a workgroup takes 128
// ranks of every gridDim.y-th group of 64 columns that has a wide one; both halves
// go through the same LDS tile.  Returns at once when there are none.  Bound by HBM
// (16 bytes per cell): 6,400 columns of 16,000 ranks 334 us, 4.9 TB/s.
__global__ __launch_bounds__(256, 4) void col_copy_wide(const int64_t *__restrict__ T, int64_t R, int IG, int G,
                                                        const int32_t *__restrict__ it, uint32_t *__restrict__ cp,
                                                        uint32_t *__restrict__ hi, ColOut o) {
  constexpr int LD = CT + 1, U = CT / 4;
  __shared__ uint32_t tile[64 * LD];
  if (o.wide[0] == 0) return;
  const int64_t Rp = copy_ranks(R), r0 = (int64_t)blockIdx.x * CT;
  const int lane = (int)(threadIdx.x & 63), wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  for (int c0 = (int)blockIdx.y * 64; c0 < IG; c0 += (int)gridDim.y * 64) {
    if (!o.group[c0 / 64]) continue;  // uniform
    const int col = c0 + lane < IG ? c0 + lane : IG - 1, ic = col / G;
    const bool mine = c0 + lane < IG && !(o.mu[col] == o.mu[col]);
    const uint64_t wide = __ballot(mine);  // the same in every wave
    uint64_t x[U];
#pragma unroll
    for (int k = 0; k < U; k++) {
      const int64_t r = r0 + 4 * k + wid;
      x[k] = (uint64_t)T[(r < R ? r : R - 1) * IG + col];
    }
#pragma unroll
    for (int k = 0; k < U; k++) {
      const int64_t r = r0 + 4 * k + wid;
      const bool in = r < R && (!it || ic < it[r]);
      x[k] = in ? x[k] + (uint64_t)HALF64 : none<uint64_t>();
    }
#pragma unroll
    for (int half = 0; half < 2; half++) {
      __syncthreads();  // the previous half is written out
#pragma unroll
      for (int k = 0; k < U; k++) tile[lane * LD + 4 * k + wid] = (uint32_t)(x[k] >> (32 * half));
      __syncthreads();
      uint32_t *to = half ? hi : cp;
      for (int c = (int)threadIdx.x / 32; c < 64; c += 8) {
        if (!(wide >> c & 1)) continue;
        const int q = 4 * ((int)threadIdx.x & 31);
        const uint32_t *l = &tile[c * LD + q];
        *reinterpret_cast<v4u *>(to + (int64_t)(c0 + c) * Rp + r0 + q) = v4u{l[0], l[1], l[2], l[3]};
      }
    }
  }
}

// The wide columns, in 64-bit words: a workgroup per column.  Without high words
// (hi NULL) they are read from the tensor, in 8-byte pieces of rows.
template <int W, int V>
__global__ __launch_bounds__(64 * W) void col_select_wide(const uint32_t *__restrict__ cp, const uint32_t *__restrict__ hi,
                                                          const int64_t *__restrict__ T, int64_t R, int IG,
                                                          int G, const int32_t *__restrict__ it, ColOut o) {
  __shared__ SelGroup<W, 2048, uint64_t> L;
  __shared__ ColRed red[W];
  const int tid = (int)threadIdx.x;
  const uint32_t n = o.wide[0];
  const int64_t Rp = copy_ranks(R);
  for (uint32_t e = blockIdx.x; e < n; e += gridDim.x) {
    const int col = (int)o.wide[1 + e], ic = col / G;
    uint64_t u[V];
    const int own = opaque(tid);  // else V offsets and iteration counts are kept over the columns
    if (hi) {
#pragma unroll
      for (int v = 0; v < V; v += 4) {
        const int64_t r = (int64_t)(v / 4) * 256 * W + 4 * own;
        v4u l = {none<uint32_t>(), none<uint32_t>(), none<uint32_t>(), none<uint32_t>()}, h = l;
        if (r < Rp) {
          l = *reinterpret_cast<const v4u *>(cp + (int64_t)col * Rp + r);
          h = *reinterpret_cast<const v4u *>(hi + (int64_t)col * Rp + r);
        }
        u[v] = (uint64_t)h.x << 32 | l.x;
        u[v + 1] = (uint64_t)h.y << 32 | l.y;
        u[v + 2] = (uint64_t)h.z << 32 | l.z;
        u[v + 3] = (uint64_t)h.w << 32 | l.w;
      }
    } else {
#pragma unroll
      for (int v = 0; v < V; v++) {
        const int r = v * 64 * W + own;
        u[v] = none<uint64_t>();
        if (r < (int)R && (!it || ic < it[r])) u[v] = (uint64_t)(T[(int64_t)r * IG + col] + HALF64);
      }
    }
    __syncthreads();
    sel_clear(L);
    select_column<uint64_t, V, W, 2048, false>(u, L, red, -HALF64, col, true, o);
  }
}

// Short columns in 64-bit words: eight columns of one wave each per workgroup
// (64-byte pieces of rows), tiles of rows through LDS.  Consecutive groups of
// columns go to one XCD (workgroup b runs on XCD b mod 8), so the two halves
// of a line are fetched from HBM once.  6,400 columns of 1,000 ranks: 54 us
// against 96 us of copy and 148 us of radix passes.
template <int V, bool STATS>
__global__ __launch_bounds__(512) void col_select_direct(const int64_t *__restrict__ T, int64_t R, int IG,
                                                         int G, const int32_t *__restrict__ it, ColOut o) {
  constexpr int C = 8, TV = V < 8 ? V : 8, TR = 64 * TV;
  constexpr int LD = TR + 4;  // the half wave's four rows of eight columns hit different banks
  constexpr int NB = col_bins<1, V>();
  union Lds {
    uint64_t tile[C * LD];
    SelGroup<1, NB, uint64_t> sel[C];
    __device__ Lds() {}
  };
  __shared__ Lds L;
  const int tid = (int)threadIdx.x, lane = tid & 63, cl = tid >> 6;
  const int c0 = C * ((int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3));
  if (c0 >= IG) return;
  constexpr int QN = 128, U = TR / QN > 0 ? TR / QN : 1;
  const int p = tid % 4, q0 = tid / 4, ca = c0 + 2 * p;
  const bool vec = (IG & 1) == 0, ha = ca < IG, hb = ca + 1 < IG;
  const int ia = ca / G, ib = (ca + 1) / G;
  v2ll x[U];
  int nit[U];
  auto load = [&](int t) {
#pragma unroll
    for (int k = 0; k < U; k++) {
      const int64_t r = (int64_t)t * TR + q0 + k * QN;
      x[k] = v2ll{0, 0};
      nit[k] = 0;
      if (r < R) {
        nit[k] = it ? it[r] : 0x7fffffff;
        const int64_t *row = T + r * IG + ca;
        if (vec) {
          if (ha) x[k] = *reinterpret_cast<const v2ll *>(row);
        } else {
          if (ha) x[k].x = row[0];
          if (hb) x[k].y = row[1];
        }
      }
    }
  };
  uint64_t u[V];
  load(0);
#pragma unroll
  for (int t = 0; t < V / TV; t++) {
    if ((int64_t)t * TR >= R) {
#pragma unroll
      for (int j = 0; j < TV; j++) u[t * TV + j] = none<uint64_t>();
      continue;
    }
    __syncthreads();  // the previous tile is read
#pragma unroll
    for (int k = 0; k < U; k++) {
      L.tile[2 * p * LD + q0 + k * QN] = ha && ia < nit[k] ? (uint64_t)((int64_t)x[k].x + HALF64) : none<uint64_t>();
      L.tile[(2 * p + 1) * LD + q0 + k * QN] =
          hb && ib < nit[k] ? (uint64_t)((int64_t)x[k].y + HALF64) : none<uint64_t>();
    }
    __syncthreads();
    if (t + 1 < V / TV) load(t + 1);
#pragma unroll
    for (int j = 0; j < TV; j++) u[t * TV + j] = L.tile[cl * LD + j * 64 + lane];
  }
  __syncthreads();
  const int col = c0 + cl;
  sel_clear(L.sel[cl]);
  select_column<uint64_t, V, 1, NB, STATS>(u, L.sel[cl], (ColRed *)nullptr, -HALF64, col, col < IG, o);
}

// a / b rounded to nearest, given y = 1 / b rounded to nearest: two corrections
// of the quotient by its exact remainder.  The first leaves it within an ulp,
// after which the second gives the correctly rounded quotient (Markstein 1990,
// "Computation of elementary functions on the IBM RISC System/6000 processor").
// No step can underflow or overflow here: |a| is 0 or in [1, 2^96], b in
// [1, 2^96].  Five operations instead of the division's full sequence.
__device__ __forceinline__ double div_by(double a, double b, double y) {
  double q = a * y;
  q = fma(fma(-b, q, a), y, q);
  return fma(fma(-b, q, a), y, q);
}

__device__ __forceinline__ int rank_iters(const int32_t *it, int64_t r, int I) {
  const int v = it ? it[r] : I;
  return v > I ? I : (v < 0 ? 0 : v);
}

// m(r,g) = (1/n_r) sum over i < n_r, ascending, of z(r,i,g), from the
// column-major copy: a workgroup owns 256 * RPL consecutive ranks of one
// region.  The region's column numbers are staged in LDS, SI iterations at a
// time, and IU iterations' cells are loaded before the first is scored (read by
// scalar loads, the numbers kept every iteration waiting: 1,741 ranks x 19,200
// columns 127 -> 63 us, 10,000 x 9,600 145 -> 102 us).  Bound by the copy's 4
// bytes per cell for long columns, by the loads' round trips for short ones.
// Staged columns that are all without far cells are scored with no branch (with
// one per column: 10,000 x 9,600 134 us).
template <int RPL, int IU>
__global__ __launch_bounds__(256) void score_copy(const uint32_t *__restrict__ cp, const uint32_t *__restrict__ hi,
                                                  const int64_t *__restrict__ T, int64_t R, int I, int G, const int32_t *__restrict__ it,
                                                  const ColZ *__restrict__ cz, const double *__restrict__ mu,
                                                  double *m_t) {
  constexpr int SI = 256;
  struct alignas(16) Num {
    double mu, zc, zd, zy;
  };
  __shared__ Num num[SI];
  const int tid = (int)threadIdx.x;
  const int64_t rb = (R + 256 * RPL - 1) / (256 * RPL);
  const int g = (int)(blockIdx.x / rb);
  const int64_t Rp = copy_ranks(R), r0 = ((blockIdx.x % rb) * 256 + tid) * RPL;
  const uint32_t *p = cp + (int64_t)g * Rp + (r0 < R ? r0 : 0);
  double acc[RPL];
#pragma unroll
  for (int q = 0; q < RPL; q++) acc[q] = 0.0;
  for (int s0 = 0; s0 < I; s0 += SI) {
    const int ns = I - s0 < SI ? I - s0 : SI;
    __syncthreads();  // the previous numbers are read
    bool near = true;
    if (tid < ns) {
      const int64_t c = (int64_t)(s0 + tid) * G + g;
      const ColZ z = cz[c];
      near = mu[c] >= 0.0;
      num[tid] = Num{mu[c], z.zc, z.zd, z.zy};
    }
    near = __syncthreads_and(near);
    for (int i0 = 0; i0 < ns; i0 += IU) {
      uint32_t w[IU][RPL];
#pragma unroll
      for (int j = 0; j < IU; j++) {
        const int i = i0 + j < ns ? i0 + j : ns - 1;
        const uint32_t *src = p + (int64_t)(s0 + i) * G * Rp;
        if (RPL == 4) {
          const v4u v = *reinterpret_cast<const v4u *>(src);
          w[j][0] = v.x;
          w[j][1 % RPL] = v.y;
          w[j][2 % RPL] = v.z;
          w[j][3 % RPL] = v.w;
        } else {
          w[j][0] = src[0];
        }
      }
      auto score = [&](const Num &z, const uint32_t *x) {  // a column without far cells
#pragma unroll
        for (int q = 0; q < RPL; q++) {
          // 2x - med2 in key words: both terms are integers below 2^34
          const double d = fma(2.0, (double)x[q], -z.mu);
          const double t = acc[q] + div_by(d * z.zc, z.zd, z.zy);
          acc[q] = x[q] != none<uint32_t>() ? t : acc[q];
        }
      };
      if (near && i0 + IU <= ns) {
#pragma unroll
        for (int j = 0; j < IU; j++) score(num[i0 + j], w[j]);
        continue;
      }
#pragma unroll
      for (int j = 0; j < IU; j++) {
        if (i0 + j >= ns) break;
        const Num z = num[i0 + j];
        if (z.mu >= 0.0) {
          score(z, w[j]);
        } else if (z.mu < 0.0) {  // a column with far cells
          const int64_t c = (int64_t)(s0 + i0 + j) * G + g;
#pragma unroll
          for (int q = 0; q < RPL; q++) {
            if (w[j][q] == none<uint32_t>()) continue;
            double d = fma(2.0, (double)w[j][q], z.mu);
            if (w[j][q] == FAR_LOW || w[j][q] == FAR_HIGH)
              d = (double)(2 * T[(r0 + q) * (int64_t)I * G + c] - cz[c].med2);
            acc[q] += div_by(d * z.zc, z.zd, z.zy);
          }
        } else {  // a wide column
          const int64_t c = (int64_t)(s0 + i0 + j) * G + g, med2 = cz[c].med2;
          uint64_t key[RPL];
          if (hi) {
            const uint32_t *src = hi + c * Rp + (r0 < R ? r0 : 0);
            uint32_t h[RPL];
            if (RPL == 4) {
              const v4u v = *reinterpret_cast<const v4u *>(src);
              h[0] = v.x;
              h[1 % RPL] = v.y;
              h[2 % RPL] = v.z;
              h[3 % RPL] = v.w;
            } else {
              h[0] = src[0];
            }
#pragma unroll
            for (int q = 0; q < RPL; q++) key[q] = (uint64_t)h[q] << 32 | w[j][q];
          } else {
#pragma unroll
            for (int q = 0; q < RPL; q++)
              key[q] = r0 + q < R && s0 + i0 + j < rank_iters(it, r0 + q, I)
                           ? (uint64_t)(T[(r0 + q) * (int64_t)I * G + c] + HALF64)
                           : none<uint64_t>();
          }
#pragma unroll
          for (int q = 0; q < RPL; q++) {
            const int64_t x = (int64_t)(key[q] - (uint64_t)HALF64);
            const double t = acc[q] + div_by((double)(2 * x - med2) * z.zc, z.zd, z.zy);
            acc[q] = key[q] != none<uint64_t>() ? t : acc[q];
          }
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < RPL; q++)
    if (r0 + q < R) {
      const int ni = rank_iters(it, r0 + q, I);
      m_t[(int64_t)g * R + r0 + q] = ni > 0 ? acc[q] / (double)ni : 0.0;
    }
}

// The same for few ranks, from the row-major tensor: a workgroup scores NR
// ranks' rows, every cell by a thread of its own, into LDS, and one thread per
// region then adds the scores in ascending iteration.  A chain of additions in
// LDS instead of a chain of loads: 1,600 columns of 64 ranks 33 -> 6 us, 6,400
// of 1,000 ranks 37 -> 26 us.  G <= 256.
constexpr int SC_CELLS = 4096;  // scores in LDS
template <int NR>
__global__ __launch_bounds__(256) void score_rank(const int64_t *__restrict__ T, int64_t R, int I, int G,
                                                  const int32_t *__restrict__ it,
                                                  const ColZ *__restrict__ cz, double *m_t) {
  __shared__ double sc[SC_CELLS];
  const int tid = (int)threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * NR, IG = (int64_t)I * G;
  int ni[NR], nmax = 0;
#pragma unroll
  for (int q = 0; q < NR; q++) {
    ni[q] = r0 + q < R ? rank_iters(it, r0 + q, I) : 0;
    nmax = ni[q] > nmax ? ni[q] : nmax;
  }
  constexpr int CELLS = SC_CELLS / NR, U = CELLS / 256;
  const int ic = CELLS / G;  // iterations per turn
  double acc[NR];
#pragma unroll
  for (int q = 0; q < NR; q++) acc[q] = 0.0;
  for (int i0 = 0; i0 < nmax; i0 += ic) {
    const int in = nmax - i0 < ic ? nmax - i0 : ic, cells = in * G;
    const int64_t c0 = (int64_t)i0 * G;
    __syncthreads();  // the previous scores are added
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int k = u * 256 + tid;
      if (k < cells) {
        const ColZ z = cz[c0 + k];
#pragma unroll
        for (int q = 0; q < NR; q++) {
          const int64_t x = r0 + q < R ? T[(r0 + q) * IG + c0 + k] : 0;
          sc[q * CELLS + k] = div_by((double)(2 * x - z.med2) * z.zc, z.zd, z.zy);
        }
      }
    }
    __syncthreads();
    if (tid < G) {
#pragma unroll
      for (int q = 0; q < NR; q++) {
        const int e = ni[q] - i0 < in ? ni[q] - i0 : in;
        const double *s = sc + q * CELLS + tid;
#pragma unroll 8
        for (int i = 0; i < e; i++) acc[q] += s[i * G];
      }
    }
  }
  if (tid < G)
#pragma unroll
    for (int q = 0; q < NR; q++)
      if (r0 + q < R) m_t[(int64_t)tid * R + r0 + q] = ni[q] > 0 ? acc[q] / (double)ni[q] : 0.0;
}

__device__ __forceinline__ double plain_z(int64_t x, const ColMom &z) {
  const i128 num = (i128)z.n * x - z.s1;
  const int64_t lo = (int64_t)num;
  return div_by(num == (i128)lo ? (double)lo : i128_to_f64(num), z.zd, z.zy);
}

// m(r,g) with plain z scores, from the row-major tensor: a workgroup scores NR
// ranks' rows, every cell by a thread of its own, into LDS, and a thread per
// (rank, region) adds the scores in ascending iteration.  Regions beyond 256 by
// blockIdx.y.  Bound by the row's and the moments' loads: a wave per 64 ranks of
// one region over a column-major copy, one load at a time, took 3,001 ranks of
// 217 x 37 cells 187 us and the copy and the moments from it 205; this takes 74
// and the moments from the tensor 44.
template <int NR>
__global__ __launch_bounds__(256) void score_plain(const int64_t *__restrict__ T, int64_t R, int I, int G,
                                                   const int32_t *__restrict__ it,
                                                   const ColMom *__restrict__ cm, double *m_t) {
  __shared__ double sc[SC_CELLS];
  constexpr int CELLS = SC_CELLS / NR, U = CELLS / 256;
  const int tid = (int)threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * NR, IG = (int64_t)I * G;
  const int g0 = (int)blockIdx.y * 256, gc = G - g0 < 256 ? G - g0 : 256;
  int ni[NR], nmax = 0;
#pragma unroll
  for (int q = 0; q < NR; q++) {
    ni[q] = r0 + q < R ? rank_iters(it, r0 + q, I) : 0;
    nmax = ni[q] > nmax ? ni[q] : nmax;
  }
  // this thread's sums: entries tid, tid + 256, ... of (rank, region)
  int eq[NR], eg[NR], en[NR];
  double acc[NR];
#pragma unroll
  for (int j = 0; j < NR; j++) {
    const int e = tid + 256 * j;
    eq[j] = e / gc;
    eg[j] = e - eq[j] * gc;
    acc[j] = 0.0;
    en[j] = 0;
#pragma unroll
    for (int q = 0; q < NR; q++) en[j] = eq[j] == q ? ni[q] : en[j];
  }
  const int ic = CELLS / gc;  // iterations per turn
  for (int i0 = 0; i0 < nmax; i0 += ic) {
    const int in = nmax - i0 < ic ? nmax - i0 : ic, cells = in * gc;
    __syncthreads();  // the previous scores are added
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int k = u * 256 + tid;
      if (k < cells) {
        const int64_t c = (int64_t)i0 * G + g0 + (gc == G ? k : (k / gc) * G + k % gc);
        const ColMom z = cm[c];
#pragma unroll
        for (int q = 0; q < NR; q++) {
          const int64_t x = r0 + q < R ? T[(r0 + q) * IG + c] : 0;
          sc[q * CELLS + k] = plain_z(x, z);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; j++) {
      const int n = en[j] - i0 < in ? en[j] - i0 : in;
      const double *s = sc + eq[j] * CELLS + eg[j];
#pragma unroll 8
      for (int i = 0; i < n; i++) acc[j] += s[i * gc];
    }
  }
#pragma unroll
  for (int j = 0; j < NR; j++)
    if (eq[j] < NR && r0 + eq[j] < R)
      m_t[(int64_t)(g0 + eg[j]) * R + r0 + eq[j]] = en[j] > 0 ? acc[j] / (double)en[j] : 0.0;
}

// The same for rows of few iterations, a thread per (rank, region).
__global__ __launch_bounds__(256) void score_plain_short(const int64_t *__restrict__ T, int64_t R, int I, int G,
                                                         const int32_t *__restrict__ it,
                                                         const ColMom *__restrict__ cm, double *m_t) {
  constexpr int U = 4;
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= R * G) return;
  const int64_t r = p / G;
  const int g = (int)(p - r * G), ni = rank_iters(it, r, I);
  const int64_t *row = T + r * (int64_t)I * G + g;
  double acc = 0.0;
  for (int i = 0; i < ni; i += U) {
    int64_t x[U];
    ColMom z[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int64_t c = (int64_t)(i + u < ni ? i + u : ni - 1) * G;
      x[u] = row[c];
      z[u] = cm[c + g];
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
      const double v = plain_z(x[u], z[u]);
      acc = i + u < ni ? acc + v : acc;
    }
  }
  m_t[(int64_t)g * R + r] = ni > 0 ? acc / (double)ni : 0.0;
}

// Robust scores from the row-major tensor for many regions or ranks.  A lane owns a
// region of RPL consecutive ranks; with fewer than 64 regions a wave takes 64
// >> lgp ranks' rows side by side.
template <int RPL, int IU>
__global__ __launch_bounds__(256) void score_tensor(const int64_t *__restrict__ T, int64_t R, int I, int G,
                                                    int lgp, const int32_t *__restrict__ it,
                                                    const ColZ *__restrict__ cz, double *m_t) {
  const int lane = (int)(threadIdx.x & 63);
  const int gbn = (G + 63) / 64;
  const int64_t wave = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t r0 = ((wave / gbn) * (64 >> lgp) + (lane >> lgp)) * RPL;
  const int g = (int)(wave % gbn) * 64 + (lane & ((1 << lgp) - 1));
  const bool on = g < G && r0 < R;
  const int gg = on ? g : 0;
  const int64_t rr = on ? r0 : 0, IG = (int64_t)I * G;
  int ni[RPL], nmax = 0;
#pragma unroll
  for (int q = 0; q < RPL; q++) {
    ni[q] = on && rr + q < R ? rank_iters(it, rr + q, I) : 0;
    nmax = ni[q] > nmax ? ni[q] : nmax;
  }
  double acc[RPL];
#pragma unroll
  for (int q = 0; q < RPL; q++) acc[q] = 0.0;
  const int64_t *p = T + rr * IG + gg;
  for (int i0 = 0; i0 < nmax; i0 += IU) {
    int64_t x[IU][RPL];
    ColZ z[IU];
#pragma unroll
    for (int j = 0; j < IU; j++) {
      const int i = i0 + j < nmax ? i0 + j : nmax - 1;
      z[j] = cz[(int64_t)i * G + gg];
#pragma unroll
      for (int q = 0; q < RPL; q++) x[j][q] = i0 + j < ni[q] ? p[q * IG + (int64_t)i * G] : 0;
    }
#pragma unroll
    for (int j = 0; j < IU; j++)
#pragma unroll
      for (int q = 0; q < RPL; q++) {
        const double t = acc[q] + div_by((double)(2 * x[j][q] - z[j].med2) * z[j].zc, z[j].zd, z[j].zy);
        acc[q] = i0 + j < ni[q] ? t : acc[q];
      }
  }
  if (on)
#pragma unroll
    for (int q = 0; q < RPL; q++)
      if (rr + q < R) m_t[(int64_t)g * R + rr + q] = ni[q] > 0 ? acc[q] / (double)ni[q] : 0.0;
}

struct ColWs {
  ColZ *cz;
  double *mu;
  uint32_t *wide;
  uint32_t *cp;
  uint8_t *group;
  uint32_t *hi;
};

// Whether wide columns are copied in two halves: up to 2^33 cells (beside a tensor
// of more than 64 GB the workspace stays at half its size) and from 2^23 on (a
// smaller tensor stays in the caches, and an empty launch is 4 us: 4,000 x 3,200
// cells all spread 365 us from the tensor, 272 with the copy; 12,289 x 128 cells, near,
// 100 and 106).
bool high_words(int64_t R, int IG) {
  const int64_t cells = copy_ranks(R) * IG;
  return cells >= (int64_t)1 << 23 && cells <= (int64_t)1 << 33;
}

ColWs carve(void *ws, int64_t R, int IG, size_t *used) {
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char *p = (char *)ws + off;
    off += (bytes + 255) & ~(size_t)255;
    return (void *)p;
  };
  ColWs w{};
  w.cz = (ColZ *)take((size_t)IG * sizeof(ColZ));
  if (R > COL_DIRECT_MAX) {
    w.mu = (double *)take((size_t)IG * 8);
    w.wide = (uint32_t *)take(((size_t)IG + 1) * 4);
    w.group = (uint8_t *)take((size_t)(IG + 63) / 64);
    w.cp = (uint32_t *)take((size_t)IG * copy_ranks(R) * 4);
    if (high_words(R, IG)) w.hi = (uint32_t *)take((size_t)IG * copy_ranks(R) * 4);
  }
  *used = off;
  return w;
}

}  // namespace

int col_stat_chunks(int64_t R) {
  return R <= COL_DIRECT_MAX ? 1 : (int)(copy_ranks(R) / CT);
}

size_t col_scan_ws_bytes(int64_t R, int IG) {
  size_t used = 0;
  carve((void *)0x100, R, IG, &used);
  return used;
}

hipError_t launch_score_plain(const int64_t *T, int64_t R, int I, int G, const int32_t *it,
                              const ColMom *cm, double *m_t, hipStream_t s) {
  // (for the call: 300,000 ranks of 8 x 5 cells 1,534 us, by ranks' rows 1,788; 40,000
  // of 32 x 16 356 and 384; 2,000 of 64 x 5 61 and 57); also where 64 threads per
  // rank were 2^32 and more
  if (I <= 32 || R >= (int64_t)1 << 26) {
    hipLaunchKernelGGL(score_plain_short, dim3((unsigned)((R * G + 255) / 256)), dim3(256), 0, s, T, R, I, G, it, cm,
                       m_t);
    return hipGetLastError();
  }
  const unsigned gb = (unsigned)((G + 255) / 256);
  // four ranks share a column's moments once they still fill the chip
  if (R >= 2048)
    hipLaunchKernelGGL(score_plain<4>, dim3((unsigned)((R + 3) / 4), gb), dim3(256), 0, s, T, R, I, G, it, cm,
                       m_t);
  else
    hipLaunchKernelGGL(score_plain<1>, dim3((unsigned)R, gb), dim3(256), 0, s, T, R, I, G, it, cm, m_t);
  return hipGetLastError();
}

hipError_t launch_score_tensor(const int64_t *T, int64_t R, int I, int G, const int32_t *it,
                               const ColZ *cz, double *m_t, int cus, hipStream_t s) {
  int lgp = 0;
  while (lgp < 6 && (1 << lgp) < G) lgp++;
  const int64_t side = 64 >> lgp, gbn = (G + 63) / 64;
  // with at least 16 waves per CU left, four ranks per lane share the column
  // numbers; below that the iterations' loads are what there is to overlap
  const bool many = (R + side - 1) / side * gbn / 4 >= 16 * (int64_t)cus;
  const int64_t per = side * (many ? 4 : 1);
  const unsigned grid = (unsigned)(((R + per - 1) / per * gbn + 3) / 4);
  if (many)
    hipLaunchKernelGGL((score_tensor<4, 2>), dim3(grid), dim3(256), 0, s, T, R, I, G, lgp, it, cz, m_t);
  else
    hipLaunchKernelGGL((score_tensor<1, 8>), dim3(grid), dim3(256), 0, s, T, R, I, G, lgp, it, cz, m_t);
  return hipGetLastError();
}

hipError_t launch_col_scan(const int64_t *T, int64_t R, int I, int G, const int32_t *it, ColPartials st,
                           hipEvent_t stats_ready, double *m_t, void *ws, int cus, hipStream_t s) {
  size_t used = 0;
  const int IG = I * G;
  const ColWs w = carve(ws, R, IG, &used);
  const ColOut o{w.cz, w.mu, w.wide, w.group, st};
  const bool stats = st.rc > 0;
  hipError_t e = hipSuccess;
  if (R <= COL_DIRECT_MAX) {
    const unsigned grid = 8u * (unsigned)(((IG + 7) / 8 + 7) / 8);
    auto go = [&](auto kern) { hipLaunchKernelGGL(kern, dim3(grid), dim3(512), 0, s, T, R, IG, G, it, o); };
    if (R <= 256) stats ? go(col_select_direct<4, true>) : go(col_select_direct<4, false>);
    else if (R <= 512) stats ? go(col_select_direct<8, true>) : go(col_select_direct<8, false>);
    else stats ? go(col_select_direct<16, true>) : go(col_select_direct<16, false>);
    e = hipGetLastError();
    if (e == hipSuccess && stats && stats_ready) e = hipEventRecord(stats_ready, s);
    if (e != hipSuccess) return e;
    if (G > 256) return launch_score_tensor(T, R, I, G, it, w.cz, m_t, cus, s);
    // two ranks of a workgroup share the column numbers once that leaves one
    // workgroup per CU
    if (R >= 2 * (int64_t)cus)
      hipLaunchKernelGGL(score_rank<2>, dim3((unsigned)((R + 1) / 2)), dim3(256), 0, s, T, R, I, G, it,
                         (const ColZ *)w.cz, m_t);
    else
      hipLaunchKernelGGL(score_rank<1>, dim3((unsigned)R), dim3(256), 0, s, T, R, I, G, it,
                         (const ColZ *)w.cz, m_t);
    return hipGetLastError();
  }
  const int64_t Rp = copy_ranks(R);
  const dim3 cgrid((unsigned)(Rp / CT), (unsigned)((IG + 63) / 64));
  if (stats)
    hipLaunchKernelGGL(col_copy<true>, cgrid, dim3(256), 0, s, T, R, IG, G, it, w.cp, w.wide, w.group, st);
  else
    hipLaunchKernelGGL(col_copy<false>, cgrid, dim3(256), 0, s, T, R, IG, G, it, w.cp, w.wide, w.group, st);
  e = hipGetLastError();
  if (e == hipSuccess && stats && stats_ready) e = hipEventRecord(stats_ready, s);
  if (e != hipSuccess) return e;
  auto go = [&](auto kern, int nt, int cols) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((IG + cols - 1) / cols)), dim3(nt), 0, s,
                       (const uint32_t *)w.cp, R, IG, T, o);
  };
  // The fewest waves that hold the column in at most 80 words per lane: a column
  // is a chain of barriers and exchanges, so as many columns as possible should
  // be in flight, and beside the column a lane needs 20 to 45 registers.  With
  // 24 or 32 words per lane (twice the waves, half the columns) 10,000 ranks
  // took 311 us instead of 206, 16,000 ranks 354 instead of 261 (before the marks of
  // far cells, which cost 10 us); with 16 waves of 40
  // words 32,000 columns of 40,000 ranks 3.00 ms instead of 2.75 (64 registers a
  // lane, 21 of them in scratch).
  auto shape = [&](auto w, auto v) {
    constexpr int W = decltype(w)::value, V = decltype(v)::value;
    go(col_select<W, V>, W > 1 ? 64 * W : 256, W > 1 ? 1 : 4);
  };
  if (R <= 2048) shape(std::integral_constant<int, 1>(), std::integral_constant<int, 32>());
  else if (R <= 3072) shape(std::integral_constant<int, 1>(), std::integral_constant<int, 48>());
  else if (R <= 4096) shape(std::integral_constant<int, 1>(), std::integral_constant<int, 64>());
  else if (R <= 5120) shape(std::integral_constant<int, 1>(), std::integral_constant<int, 80>());
  else if (R <= 6144) shape(std::integral_constant<int, 2>(), std::integral_constant<int, 48>());
  else if (R <= 8192) shape(std::integral_constant<int, 2>(), std::integral_constant<int, 64>());
  else if (R <= 10240) shape(std::integral_constant<int, 2>(), std::integral_constant<int, 80>());
  else if (R <= 12288) shape(std::integral_constant<int, 4>(), std::integral_constant<int, 48>());
  else if (R <= 16384) shape(std::integral_constant<int, 4>(), std::integral_constant<int, 64>());
  else if (R <= 20480) shape(std::integral_constant<int, 4>(), std::integral_constant<int, 80>());
  else if (R <= 24576) shape(std::integral_constant<int, 8>(), std::integral_constant<int, 48>());
  else if (R <= 32768) shape(std::integral_constant<int, 8>(), std::integral_constant<int, 64>());
  else if (R <= 40960) shape(std::integral_constant<int, 8>(), std::integral_constant<int, 80>());
  else shape(std::integral_constant<int, 16>(), std::integral_constant<int, 48>());
  const uint32_t *cp = w.cp, *hi = w.hi;
  const int64_t tiles = Rp / CT;
  if (w.hi)
    hipLaunchKernelGGL(col_copy_wide,
                       dim3((unsigned)tiles, (unsigned)std::min<int64_t>((IG + 63) / 64, (4 * cus + tiles - 1) / tiles)),
                       dim3(256), 0, s, T, R, IG, G, it, w.cp, w.hi, o);
  auto wide = [&](auto w, auto v) {
    constexpr int W = decltype(w)::value, V = decltype(v)::value;
    hipLaunchKernelGGL((col_select_wide<W, V>), dim3((unsigned)std::min(IG, 16 / W * cus)), dim3(64 * W), 0, s,
                       cp, hi, T, R, IG, G, it, o);
  };
  if (R <= 2048) wide(std::integral_constant<int, 4>(), std::integral_constant<int, 8>());
  else if (R <= 4096) wide(std::integral_constant<int, 8>(), std::integral_constant<int, 8>());
  else if (R <= 12288) wide(std::integral_constant<int, 16>(), std::integral_constant<int, 12>());
  else if (R <= 20480) wide(std::integral_constant<int, 16>(), std::integral_constant<int, 20>());
  else if (R <= 32768) wide(std::integral_constant<int, 16>(), std::integral_constant<int, 32>());
  else if (R <= 40960) wide(std::integral_constant<int, 16>(), std::integral_constant<int, 40>());
  else wide(std::integral_constant<int, 16>(), std::integral_constant<int, (int)(COL_REG_MAX / 1024)>());
  // four ranks per lane (16-byte loads) once that leaves 16 waves per CU
  const int64_t b4 = (R + 1023) / 1024 * G;
  if (b4 >= 4 * (int64_t)cus)
    hipLaunchKernelGGL((score_copy<4, 4>), dim3((unsigned)b4), dim3(256), 0, s, cp, hi, T, R, I, G, it,
                       (const ColZ *)w.cz, (const double *)w.mu, m_t);
  else
    hipLaunchKernelGGL((score_copy<1, 16>), dim3((unsigned)((R + 255) / 256 * G)), dim3(256), 0, s, cp, hi, T, R, I,
                       G, it, (const ColZ *)w.cz, (const double *)w.mu, m_t);
  return hipGetLastError();
}

}  // namespace ta
