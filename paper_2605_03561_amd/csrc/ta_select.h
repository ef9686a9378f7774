// ta_select.h -- exact order statistics of keys held in registers.
//
// A group of W waves holds up to 64 * W * V unsigned keys, V per lane.  The
// k-th smallest is found by most-significant-digit radix passes over the
// registers: a histogram of the digit in LDS (one atomic per key that has the
// prefix found so far), a scan of its bins on the VALU, and the bin of rank k
// becomes the new prefix.  As soon as at most 64 keys share the prefix they are
// gathered into one wave and ranked by comparison, so a spread column takes
// one pass and not one per digit.  Nothing is read twice from memory.  Every
// count is an integer, so the results do not depend on the order of the
// atomics.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace ta {

constexpr int SEL_FEW = 64;  // keys left for the comparison step: one per lane

// LDS of one group: NB bins and the exchange words.
template <int W, int NB, typename K>
struct SelGroup {
  static constexpr int BPT = NB / (64 * W);  // bins per thread of the group
  alignas(16) uint32_t hist[NB];
  K few[SEL_FEW];
  K above, r1, r2;
  uint32_t wsum[W];
  uint32_t bin, below, cnt, nfew;
};

// Orders the LDS accesses of the lanes of a group: a barrier of the workgroup,
// or for groups of one wave (whose LDS operations complete in order) only a
// barrier for the compiler.
template <int W>
__device__ __forceinline__ void group_sync() {
  if (W == 1) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Inclusive scan over the 64 lanes of a wave on the VALU (shifts within
// 16-lane rows, then the row totals).
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t x) {
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return x;
}

// Reductions over the 64 lanes on the VALU (a few cycles per step where an
// exchange through LDS waits for about a hundred); every lane gets the result.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or(uint32_t x, uint32_t none) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)none, (int)x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_or(uint64_t x, uint64_t none) {
  return ((uint64_t)dpp_or<CTRL, ROWS>((uint32_t)(x >> 32), (uint32_t)(none >> 32)) << 32) |
         dpp_or<CTRL, ROWS>((uint32_t)x, (uint32_t)none);
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)x, l);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t x, int l) {
  return ((uint64_t)lane_value((uint32_t)(x >> 32), l) << 32) | lane_value((uint32_t)x, l);
}
template <typename K, class Op>
__device__ __forceinline__ K wave_reduce(K x, K none, Op op) {
  x = op(x, dpp_or<0x111, 0xf>(x, none));  // row_shr:1
  x = op(x, dpp_or<0x112, 0xf>(x, none));
  x = op(x, dpp_or<0x114, 0xf>(x, none));
  x = op(x, dpp_or<0x118, 0xf>(x, none));
  x = op(x, dpp_or<0x142, 0xa>(x, none));  // row_bcast:15
  x = op(x, dpp_or<0x143, 0xc>(x, none));  // row_bcast:31
  return lane_value(x, 63);
}
template <typename K>
__device__ __forceinline__ K wave_min(K x) {
  return wave_reduce(x, ~(K)0, [](K a, K b) { return a < b ? a : b; });
}
template <typename K>
__device__ __forceinline__ K wave_max(K x) {
  return wave_reduce(x, (K)0, [](K a, K b) { return a > b ? a : b; });
}
template <typename K>
__device__ __forceinline__ K wave_sum(K x) {
  return wave_reduce(x, (K)0, [](K a, K b) { return (K)(a + b); });
}

// x, hidden from the compiler: comparisons of all V registers with it in one
// loop are then not kept as V lane masks (spilled scalar registers) for the
// same comparisons in another.
template <typename K>
__device__ __forceinline__ K opaque(K x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Ends a loop body over V registers: the scheduler does not mix the steps of
// more than four of them, which would keep a second set of registers busy.
template <int N = 4>
__device__ __forceinline__ void pace(int v) {
  if (v % N == N - 1) __builtin_amdgcn_sched_barrier(0);
}

// The bins of a group start at zero and are left at zero by reg_select.
template <int W, int NB, typename K>
__device__ __forceinline__ void sel_clear(SelGroup<W, NB, K> &L) {
  for (int j = (int)(threadIdx.x % (64 * W)); j < NB; j += 64 * W) L.hist[j] = 0;
  group_sync<W>();
}

// The k-th smallest (k from 0, k < n) of a group's n keys u[] and, with `next`,
// the (k+1)-th (k + 1 < n).  Keys are at most `last`, which takes `bits` bits; a
// word above `last` is no key (it sorts after every key, so the passes need no
// test for it, and it can not be selected).  HOT: the hot_cnt keys equal to
// `hot`, which many values may share, were counted by the caller and are added
// to their bin once instead of by that many atomics on one address.  The keys
// are plain words in registers: a key computed on the fly is kept in a second
// set of registers by the compiler, across the passes.  A group of more than
// one wave is a whole workgroup; all its threads call this.
template <bool HOT, int V, int W, int NB, typename K>
__device__ __forceinline__ void reg_select(SelGroup<W, NB, K> &L, const K (&u)[V], K hot, uint32_t hot_cnt,
                                           K last, int bits, uint32_t n, uint32_t k, bool next, K &r1,
                                           K &r2) {
  constexpr int T = 64 * W, BPT = NB / T, KB = 8 * (int)sizeof(K);
  constexpr int DB = __builtin_ctz(NB);
  const int t = (int)(threadIdx.x % T), lane = t & 63, sw = t >> 6;
  K pref = 0;
  int lo = bits;
  uint32_t cnt = n;
  auto top = [&](K x, int s) -> K { return s >= KB ? (K)0 : (K)(x >> s); };
  while (lo > 0 && cnt > (uint32_t)SEL_FEW) {
    const int w = lo < DB ? lo : DB, nlo = lo - w;
    const K b0 = (K)(pref << w), nb = (K)1 << w;
    const K h = HOT ? opaque(hot) : hot;
#pragma unroll
    for (int v = 0; v < V; v++) {
      const K b = (K)((u[v] >> nlo) - b0);  // nlo < KB
      if ((!HOT || u[v] != h) && b < nb) atomicAdd(&L.hist[(uint32_t)b], 1u);
      pace(v);
    }
    if (HOT && hot_cnt && t == 0) {
      const K b = (K)((hot >> nlo) - b0);
      if (b < nb) atomicAdd(&L.hist[(uint32_t)b], hot_cnt);
    }
    group_sync<W>();
    uint32_t c[BPT], own = 0;
#pragma unroll
    for (int j = 0; j < BPT; j++) {
      c[j] = L.hist[t * BPT + j];
      own += c[j];
    }
#pragma unroll
    for (int j = 0; j < BPT; j++) L.hist[t * BPT + j] = 0;
    const uint32_t incl = wave_scan_u32(own);
    uint32_t excl = incl - own;
    if (W > 1) {
      if (lane == 63) L.wsum[sw] = incl;
      group_sync<W>();
#pragma unroll
      for (int q = 0; q < W; q++) {
        const uint32_t x = L.wsum[q];
        excl += q < sw ? x : 0u;
      }
    }
    if (excl <= k && k < excl + own) {
      uint32_t cum = excl;
      int j = 0;
      bool go = true;
#pragma unroll
      for (int q = 0; q < BPT; q++) {
        if (go && q + 1 < BPT && cum + c[q] <= k) {
          cum += c[q];
          j = q + 1;
        } else if (go) {
          go = false;
          L.cnt = c[q];
        }
      }
      L.bin = (uint32_t)(t * BPT + j);
      L.below = cum;
    }
    group_sync<W>();
    pref = (K)(b0 + L.bin);
    k -= L.below;
    cnt = L.cnt;
    lo = nlo;
  }
  // At most SEL_FEW keys share the prefix, or it is a whole key (lo == 0).
  const bool few = n > 0 && lo > 0;
  const bool want_above = n > 0 && next && k + 1 >= cnt;
  r1 = r2 = pref;
  if (!few && !want_above) {
    group_sync<W>();  // the exchange words are read
    return;
  }
  if (t == 0) {
    L.nfew = 0;
    L.above = ~(K)0;
  }
  group_sync<W>();
  if (few) {
    const K lim = opaque(last);
#pragma unroll
    for (int v = 0; v < V; v++)
      if (top(u[v], lo) == pref && u[v] <= lim) {
        const uint32_t at = atomicAdd(&L.nfew, 1u);
        if (at < (uint32_t)SEL_FEW) L.few[at] = u[v];
      }
  }
  if (want_above) {
    K m = ~(K)0;
#pragma unroll
    for (int v = 0; v < V; v++) m = top(u[v], lo) > pref && u[v] < m ? u[v] : m;
    m = wave_min(m);
    if (lane == 0) atomicMin(&L.above, m);
  }
  group_sync<W>();
  if (few && sw == 0) {
    // cnt without the words that are no keys
    const int nf = L.nfew < (uint32_t)SEL_FEW ? (int)L.nfew : SEL_FEW;
    const K x = lane < nf ? L.few[lane] : ~(K)0;
    uint32_t rank = 0;
    const int nu = __builtin_amdgcn_readfirstlane(nf);
#pragma unroll 4
    for (int j = 0; j < nu; j++) {
      const K y = lane_value(x, j);
      rank += (y < x || (y == x && j < lane)) ? 1u : 0u;
    }
    if (lane < nf) {
      if (rank == k) L.r1 = x;
      if (rank == k + 1) L.r2 = x;
    }
  }
  group_sync<W>();
  if (few) r1 = L.r1;
  r2 = want_above ? L.above : (few && next ? L.r2 : r1);
  group_sync<W>();  // the exchange words are read
}

}  // namespace ta
