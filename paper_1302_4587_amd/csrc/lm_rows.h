// Rows in lane groups (gfx950, wave64): groups of 2^lg lanes hold one row of a
// CSR, SI consecutive entries a lane, and find its entry of largest key. Used by
// the kernels that take whole rows (lm_solo.hip, lm_first.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "lm_device.h"
#include "lm_internal.h"
#include "lm_key.h"

namespace lm {

typedef int i4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

constexpr unsigned kUnitOrd = 0xBF800000u;  // ordered image of 1.0f

// A value every lane holds, as a scalar.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ unsigned uni(unsigned x) { return (unsigned)__builtin_amdgcn_readfirstlane((int)x); }
__device__ __forceinline__ long long uni(long long x) {
  return (long long)(((unsigned long long)uni((unsigned)((unsigned long long)x >> 32)) << 32) | uni((unsigned)x));
}
__device__ __forceinline__ unsigned long long uni(unsigned long long x) { return (unsigned long long)uni((long long)x); }

// Largest value of the lane's group of 2^lg lanes, on each of its lanes.
__device__ __forceinline__ unsigned group_max(unsigned x, int lg) {
  if (lg >= 1) x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xf, 0xf, true));   // xor 1
  if (lg >= 2) x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xf, 0xf, true));   // xor 2
  if (lg >= 3) x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xf, 0xf, true));  // half row
  if (lg >= 4) x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xf, 0xf, true));  // row
  if (lg >= 6) {
    x = max(x, (unsigned)__shfl_xor((int)x, 16, 64));
    x = max(x, (unsigned)__shfl_xor((int)x, 32, 64));
  }
  return x;
}
__device__ __forceinline__ unsigned long long group_max64(unsigned long long x, int lg) {
  // the high words' maximum, then the low words' among the lanes that reach it
  const unsigned hi = (unsigned)(x >> 32);
  const unsigned mh = group_max(hi, lg);
  const unsigned ml = group_max(hi == mh ? (unsigned)x : 0u, lg);
  return ((unsigned long long)mh << 32) | ml;
}

// SI consecutive entries from offset `at` on (the lane's; nothing past lim
// is read). Lanes with !in get nothing and read nothing.
template <bool W, int SI>
__device__ __forceinline__ void load_row(const int* col, const float* w, int at, int lim, bool in, int (&cv)[SI],
                                         unsigned (&wv)[SI]) {
  if (in) {
    if (at + SI <= lim) {
#pragma unroll
      for (int p = 0; p < SI; p += 4) {
        const i4u x = *reinterpret_cast<const i4u*>(col + at + p);
#pragma unroll
        for (int q = 0; q < 4; ++q) cv[p + q] = x[q];
      }
      if (W) {
#pragma unroll
        for (int p = 0; p < SI; p += 4) {
          const i4u y = *reinterpret_cast<const i4u*>(w + at + p);
#pragma unroll
          for (int q = 0; q < 4; ++q) wv[p + q] = (unsigned)y[q];
        }
      }
    } else {
#pragma unroll
      for (int q = 0; q < SI; ++q) {
        const int k = min(at + q, lim - 1);  // at < lim: the lane has an entry
        cv[q] = col[k];
        if (W) wv[q] = __float_as_uint(w[k]);
      }
    }
  }
}

// What a pass does with a live entry's key.
enum SoloKey : int {
  kKeyNone,    // no candidates are computed
  kKeyWeight,  // the weight, ties by the hash
  kKeyHash,    // an unweighted graph: the hash
  kKeyStored   // an unweighted graph whose entries carry the high word of their hash (never 0), ties by the hash
};
constexpr bool reads_w(SoloKey k) { return k == kKeyWeight || k == kKeyStored; }

// The entries ok[] of a group's row: their winner (largest key) is on the
// lanes that get true, with its neighbour in u (one lane, unless a row lists
// an edge twice); m gets an image of the largest weight that orders as the
// weights do, 0 if the group has no entry. The hash is computed only where it
// can decide; kKeyHash leaves its high word in wv.
template <SoloKey KEY, int SI>
__device__ __forceinline__ bool group_winner(const bool (&ok)[SI], const int (&cv)[SI], unsigned (&wv)[SI], bool in,
                                             int lg, unsigned long long gm, unsigned v, unsigned long long S, int& u,
                                             unsigned& m) {
  if (KEY == kKeyHash) {
    bool mine = false;
    unsigned long long h = 0ull;
#pragma unroll
    for (int q = 0; q < SI; ++q) {
      const unsigned long long x = keep(edge_hash(S, v, (unsigned)cv[q]));
      wv[q] = (unsigned)(x >> 32) | 1u;
      const bool gt = ok[q] && x >= h;
      h = gt ? x : h;
      u = gt ? cv[q] : u;
      mine = mine || ok[q];
    }
    m = (__ballot(mine) & gm) ? kUnitOrd : 0u;
    const unsigned long long hm = group_max64(h, lg);  // (on every lane: not under a condition)
    return mine && h == hm;
  }
  // Positive weights order as their bits do. A step that holds another one
  // orders all of its weights by the general image.
  unsigned ow[SI], x = 0u;
  bool image = false;
  if (KEY == kKeyWeight) {
    int lo = (int)wv[0];
#pragma unroll
    for (int q = 1; q < SI; ++q) lo = min(lo, (int)wv[q]);
    image = __ballot(in && lo <= 0) != 0ull;
  }
  if (image) {
#pragma unroll
    for (int q = 0; q < SI; ++q) ow[q] = ord_weight_bits(wv[q]);
  } else {
#pragma unroll
    for (int q = 0; q < SI; ++q) ow[q] = wv[q];
  }
#pragma unroll
  for (int q = 0; q < SI; ++q) {
    ow[q] = ok[q] ? ow[q] : 0u;
    x = max(x, ow[q]);
  }
  m = group_max(x, lg);
  int hits = 0;  // of the wave; a scalar
#pragma unroll
  for (int q = 0; q < SI; ++q) {
    const bool hit = ow[q] == m && m != 0u;
    hits += (int)__popcll(__ballot(hit));
    u = hit ? cv[q] : u;
  }
  bool mine = x == m && m != 0u;
  const int rows = (int)__popcll(__ballot(m != 0u && (gm & lanemask_lt()) == 0ull));  // the groups' first lanes
  if (hits != rows) {  // a largest weight repeats
    unsigned long long h = 0ull;
#pragma unroll
    for (int q = 0; q < SI; ++q) {
      if (mine && ow[q] == m) {
        const unsigned long long y = edge_hash(S, v, (unsigned)cv[q]);
        if (y >= h) {
          h = y;
          u = cv[q];
        }
      }
    }
    const unsigned long long hm = group_max64(h, lg);
    mine = mine && h == hm;
  }
  if (KEY == kKeyWeight && !image && m != 0u) m |= 0x80000000u;
  return mine;
}

__device__ __forceinline__ unsigned long long group_mask(int lg) {
  const unsigned long long m = lg >= 6 ? ~0ull : ((1ull << (1 << lg)) - 1ull);
  return m << (lane_id() & ~((1 << lg) - 1));
}

// Lanes per row (log2) for E entries in V rows: one step of SI << lg entries
// holds a row one and a half times the average.
template <int SI>
__host__ __device__ __forceinline__ int group_lg(unsigned E, int V) {
  const unsigned long long e3 = 3ull * E, v16 = 2ull * SI * (unsigned)V;
  return e3 <= v16 ? 0 : e3 <= 2 * v16 ? 1 : e3 <= 4 * v16 ? 2 : e3 <= 8 * v16 ? 3 : 4;
}

// (w, u) of v's row becomes the larger of itself and (w2, u2).
__device__ __forceinline__ void best_pair(unsigned& w, int& u, unsigned w2, int u2, unsigned v,
                                          unsigned long long S) {
  if (w2 != 0u && (w2 > w || (w2 == w && edge_hash(S, v, (unsigned)u2) > edge_hash(S, v, (unsigned)u)))) {
    w = w2;
    u = u2;
  }
}

// The best entry of one row read by LANES lanes together (lane `at` of them, a
// multiple of a wave in all): each wave's best on its lanes, w = 0 if it has none.
template <int SI, int LANES>
__device__ __forceinline__ void row_best(const int* col, const float* wt, int off, int len, int at, int lim, int n,
                                         unsigned v, unsigned long long S, unsigned& w, int& u) {
  for (int k0 = uni(at & ~63) * SI; k0 < len; k0 += LANES * SI) {
    const int k = k0 + SI * lane_id();
    int cv[SI];
    unsigned wv[SI];
    load_row<true>(col, wt, off + k, lim, k < len, cv, wv);
    bool ok[SI];
#pragma unroll
    for (int q = 0; q < SI; ++q) ok[q] = k + q < len && (unsigned)cv[q] < (unsigned)n;
    int x = 0;
    unsigned m;
    const unsigned long long win = __ballot(group_winner<kKeyWeight>(ok, cv, wv, k < len, 6, ~0ull, v, S, x, m));
    if (m != 0u) best_pair(w, u, uni(m), __shfl(x, __ffsll((long long)win) - 1, 64), v, S);
  }
}

// ---- ranges of R_1's entries, a wave each (unweighted graphs: lm_first.hip, lm_compact.hip)

// Smallest i in [lo, hi) with pred(i) true (pred monotone), hi if none; every
// lane gets the answer. 64 points per round, one memory access per lane.
template <typename Pred>
__device__ __forceinline__ long long wave_lower_bound(long long lo, long long hi, Pred pred) {
  const int lane = lane_id();
  while (hi > lo) {
    const long long n = hi - lo;
    const long long step = (n + 63) >> 6;
    const long long idx = lo + (long long)lane * step;
    const bool p = idx < hi ? pred(idx) : true;
    const unsigned long long bal = __ballot(p);
    if (bal == 0ull) {  // false at every sampled point: the answer lies past the last one
      lo = lo + 63 * step + 1;
      continue;
    }
    const int f = __ffsll((long long)bal) - 1;
    if (f == 0) return lo;
    // false at lo + (f-1) step, true at lo + f step (or that point is past hi)
    const long long nhi = lo + (long long)f * step < hi ? lo + (long long)f * step : hi;
    lo = lo + (long long)(f - 1) * step + 1;
    hi = nhi;
  }
  return lo;
}

// The entry position of cost c over R_1 read from the CSR (kPieceCostFirst units per row, one
// per entry, as the other first-argmax kernels split it).
__device__ __forceinline__ long long wave_csr_entry_at(const long long* rp, long long n, long long c) {
  constexpr long long K = kPieceCostFirst;
  const long long v1 = wave_lower_bound(0, n + 1, [&](long long v) { return rp[v] + K * v > c; });
  const long long v = v1 - 1;
  const long long u = c - (rp[v] + K * v);
  if (u < K || v >= n) return rp[v];
  const long long deg = rp[v + 1] - rp[v];
  return rp[v] + min(u - K, deg);
}

__device__ __forceinline__ Part unw_part(long long v, int flags, bool any, unsigned long long h,
                                         unsigned long long S) {
  Part p;
  p.v = (int)v;
  p.flags = flags;
  p.kept = 0;
  p.out_row = -1;
  p.w = any ? kUnitOrd : 0u;
  p.hhi = any ? (unsigned)(h >> 32) : 0u;
  p.hlo = any ? (unsigned)h : 0u;
  p.u = any ? hash_neighbour(h, S, (unsigned)v) : -1;
  return p;
}

// The workgroup is one wave: LDS accesses of its lanes are carried out in
// issue order, so lanes exchange data through LDS with no s_barrier and no
// wait for the stores; this only keeps the compiler from moving LDS accesses
// across the point.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One lane to the left across the wave (lane 63 gets ident).
__device__ __forceinline__ unsigned dpp_wave_shl1(unsigned x, unsigned ident) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)ident, (int)x, 0x130, 0xf, 0xf, false);
}

__device__ __forceinline__ long long rdl64(long long x, int l) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)x, l);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)((unsigned long long)x >> 32), l);
  return (long long)(((unsigned long long)hi << 32) | lo);
}

}  // namespace lm
