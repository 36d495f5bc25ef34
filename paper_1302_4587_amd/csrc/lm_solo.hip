// Whole graphs of at most kSoloMaxN vertices, one workgroup each (gfx950,
// wave64): a small graph solved alone, or every graph of a batch.
//
// A phase of a small graph has little work and many dependent steps. Spread
// over the chip, each step ends in a launch or a grid barrier; kept in one
// workgroup it ends in a workgroup barrier, and what the phases look up at
// random (the candidates C[v] as 16-bit local ids, the matched bits) lives in
// LDS. A batch has enough graphs to fill the chip this way, and no phase of
// one graph waits for another's.
//
// Phase t (paper, Section 2, sequential model; synchronous phases):
//   mutual   v with C[C[v]] = v is matched (mate, matched bit);
//   compact  rows of unmatched vertices keep the entries whose neighbour is
//            unmatched, packed densely into the graph's range of the entry
//            buffer not being read, with the candidate of phase t + 1.
// R_1 is the input CSR itself; later live rows are records {v, offset,
// length} in two lists per live set: rows that fit one step of a lane group
// (8 << lg entries) and longer ones, which a wave takes each. Groups of
// 2^lg lanes hold one row, eight consecutive entries a lane (two 16-byte loads
// of col and of w); the group reduces its maximum with DPP. lg follows the
// average row length of the live set.
//
// What bounds it: a small graph, the dependent steps of a phase (about 3 us
// once little is live) and, in its first two passes, the instructions of one
// CU; a batch, HBM: the first argmax of a large graph reads 4.1 TB/s over the
// chip, the first compaction, whose writes and LDS lookups come on top, 3 TB/s.
// Measured against the phase kernels with the grid-wide tail (whole calls):
// ER 300 / 1200 122 -> 47 us, ER 2000 / 16000 203 -> 70 us, 64 unweighted
// graphs of 2^8 to 2^12 vertices 0.79 -> 0.21 ms, 4096 weighted graphs of 2^8
// to 2^16 vertices 12.9 -> 5.2 ms. Entries a lane takes per step and waves per
// SIMD: 8 and 4 for the largest graphs (LDS holds one) and for one graph (4 and
// 8: 98 us of kernel time on ER 4096 against 86), 4 and 8 for the others.
#include <hip/hip_ext.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cstring>
#include <type_traits>
#include <vector>

#include "lm.h"
#include "lm_device.h"
#include "lm_internal.h"
#include "lm_key.h"
#include "lm_rows.h"
#include "lm_runtime.h"

namespace lm {

namespace {


struct SoloCnt {   // counts of one phase
  // low word: entries placed in the destination (long rows reserve their whole
  // length); high word: short rows placed at the front of the next list
  unsigned long long at;
  int nl;           // long rows placed at its back
  unsigned kept;    // live entries of the next live set
  unsigned md;      // entries of the rows dropped as matched
  int mv;           // vertices matched
};

struct SoloSmem {
  SoloCnt cnt[2];
  int nl1;        // long rows of R_1
  int rows1;      // live rows of R_1
  unsigned err;
};

// Dynamic LDS: the counters, then C (16 bits a vertex), the matched bits and
// the bits of R_1's vertices without a candidate, each padded to 64 vertices.
__device__ __forceinline__ unsigned char* solo_dyn() {
  extern __shared__ __align__(16) unsigned char solo_lds_mem[];
  return solo_lds_mem;
}
constexpr int kSoloHead = 64;
static_assert(sizeof(SoloSmem) <= kSoloHead, "counters before the candidates");
__device__ __forceinline__ SoloSmem& solo_sm() { return *reinterpret_cast<SoloSmem*>(solo_dyn()); }
__device__ __forceinline__ unsigned short* cand_of() { return reinterpret_cast<unsigned short*>(solo_dyn() + kSoloHead); }
__device__ __forceinline__ unsigned* words_at(int byte) { return reinterpret_cast<unsigned*>(solo_dyn() + byte); }

// One graph as a workgroup sees it. Offsets are relative to its first entry.
struct SoloGraph {
  int n, E;        // vertices, entries
  int lim;         // entries that may be read from its first one on (to the end of the arrays)
  const long long* rp;  // its row_ptr slice
  long long e0;
  unsigned long long S;  // the seed of the candidates being computed
  int mb, nb;      // LDS byte offsets: matched bits, vertices of R_1 without a candidate
};

__device__ __forceinline__ bool bit_of(int words, int v) { return (words_at(words)[v >> 5] >> (v & 31)) & 1u; }

// A row of R_1 without a valid entry: it names itself, so that nothing it
// could match names it.
__device__ __forceinline__ void no_candidate(const SoloGraph& g, int v) {
  cand_of()[v] = (unsigned short)v;
  atomicOr(&words_at(g.nb)[v >> 5], 1u << (v & 31));
}

// Destination of a compaction (col, list, ci, thr), and of the keys an
// argmax stores (w).
struct SoloOut {
  int* col;
  float* w;
  int4* list;   // n records: short rows from the front, long rows from the back
  int ci;       // its counts (SoloSmem::cnt)
  int thr;      // longest short row of the next live set
};

// Takes room for `tot` entries and ns short rows.
__device__ __forceinline__ void take_room(const SoloOut& o, unsigned tot, int ns, unsigned& base, int& row) {
  unsigned long long x = 0ull;
  if (lane_id() == 0) x = atomicAdd(&solo_sm().cnt[o.ci].at, ((unsigned long long)(unsigned)ns << 32) | tot);
  base = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)x);
  row = __builtin_amdgcn_readfirstlane((int)(x >> 32));
}
__device__ __forceinline__ int take_long(int* count, int nl) {
  int at = 0;
  if (lane_id() == 0) at = atomicAdd(count, nl);
  return __builtin_amdgcn_readfirstlane(at);
}

// How a pass reads its rows.
template <int SI, bool UNW, bool CSR, bool COMPACT, SoloKey KEY>
struct SoloPass {
  // W: the entries' weights (or stored keys) are loaded; OUTW: and written
  static constexpr bool W = reads_w(KEY) || (!UNW && COMPACT);
  static constexpr bool OUTW = COMPACT ? W : (UNW && !CSR);

  // The entries of a step that stay: inside their row, a vertex of the graph
  // (a list holds no others), its neighbour unmatched.
  static __device__ __forceinline__ void filter(const SoloGraph& g, int rem, const int (&cv)[SI], bool (&ok)[SI]) {
#pragma unroll
    for (int q = 0; q < SI; ++q) ok[q] = q < rem && (!CSR || (unsigned)cv[q] < (unsigned)g.n);
    if (COMPACT) {
      unsigned word[SI];
#pragma unroll
      for (int q = 0; q < SI; ++q) word[q] = words_at(g.mb)[ok[q] ? cv[q] >> 5 : 0];
#pragma unroll
      for (int q = 0; q < SI; ++q) ok[q] = ok[q] && !((word[q] >> (cv[q] & 31)) & 1u);
    }
  }

  static __device__ __forceinline__ void write_kept(const SoloOut& o, int at, const bool (&ok)[SI],
                                                    const int (&cv)[SI], const unsigned (&wv)[SI]) {
#pragma unroll
    for (int q = 0; q < SI; ++q) {
      if (ok[q]) {
        o.col[at] = cv[q];
        if (OUTW) o.w[at] = __uint_as_float(wv[q]);
        ++at;
      }
    }
  }

  // One step: every group of 2^lg lanes holds one row (v, len <= SI << lg, its
  // entries at off, already loaded). Compaction writes the entries that stay
  // and appends the row's record.
  static __device__ __forceinline__ unsigned short_step(const SoloGraph& g, const SoloOut& o, int lg,
                                                        unsigned long long gm, int v, int off, int len,
                                                        const int (&cv)[SI], unsigned (&wv)[SI]) {
    const int sub = lane_id() & ((1 << lg) - 1);
    const int rem = len - SI * sub;
    bool ok[SI];
    filter(g, rem, cv, ok);
    if (KEY != kKeyNone) {
      int u = 0;
      unsigned m;
      if (group_winner<KEY>(ok, cv, wv, rem > 0, lg, gm, (unsigned)v, g.S, u, m)) cand_of()[v] = (unsigned short)u;
      if (!COMPACT) {
        if (CSR && len > 0 && sub == 0 && m == 0u) no_candidate(g, v);
        if (OUTW) {
#pragma unroll
          for (int q = 0; q < SI; ++q)
            if (ok[q]) o.w[off + SI * sub + q] = __uint_as_float(wv[q]);
        }
      }
    }
    if (!COMPACT) return 0u;
    // survivors in lane order: a row's are consecutive
    unsigned c = 0;
#pragma unroll
    for (int q = 0; q < SI; ++q) c += ok[q] ? 1u : 0u;
    const unsigned incl = wave_incl_sum_u32(c);
    const unsigned tot = (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    if (tot == 0u) return 0u;
    const unsigned last = lg == 0 ? incl : (unsigned)__shfl((int)incl, lane_id() | ((1 << lg) - 1), 64);
    const int row = sub == 0 ? (int)(last - (incl - c)) : 0;
    const bool es = row > 0 && row <= o.thr, el = row > o.thr;
    const unsigned long long bs = __ballot(es), bl = __ballot(el);
    unsigned base;
    int ps;
    take_room(o, tot, (int)__popcll(bs), base, ps);
    const int first = (int)(base + incl - c);
    write_kept(o, first, ok, cv, wv);
    if (es) o.list[ps + (int)__popcll(bs & lanemask_lt())] = make_int4(v, first, row, 0);
    if (bl) {
      const int pl = take_long(&solo_sm().cnt[o.ci].nl, (int)__popcll(bl));
      if (el) o.list[g.n - 1 - (pl + (int)__popcll(bl & lanemask_lt()))] = make_int4(v, first, row, 0);
    }
    return tot;
  }

  // A row of any length by one wave, 64 SI entries a step.
  static __device__ __forceinline__ unsigned long_row(const SoloGraph& g, const SoloOut& o, const int* col,
                                                      const float* w, int v, int off, int len) {
    const int lane = lane_id();
    unsigned base = 0, kept = 0;
    int ps;
    if (COMPACT) take_room(o, (unsigned)len, 0, base, ps);  // room for all of them
    unsigned bw = 0u;  // the best so far, the same on every lane
    int bu = 0;
    for (int k0 = 0; k0 < len; k0 += 64 * SI) {
      const int k = k0 + SI * lane;
      int cv[SI];
      unsigned wv[SI];
      load_row<W>(col, w, off + k, g.lim, k < len, cv, wv);
      bool ok[SI];
      filter(g, len - k, cv, ok);
      if (KEY != kKeyNone) {
        int u = 0;
        unsigned m;
        const unsigned long long win =
            __ballot(group_winner<KEY>(ok, cv, wv, k < len, 6, ~0ull, (unsigned)v, g.S, u, m));
        if (m != 0u) {
          u = __shfl(u, __ffsll((long long)win) - 1, 64);
          if (m > bw ||
              (m == bw && edge_hash(g.S, (unsigned)v, (unsigned)u) > edge_hash(g.S, (unsigned)v, (unsigned)bu))) {
            bw = m;
            bu = u;
          }
        }
        if (!COMPACT && OUTW) {
#pragma unroll
          for (int q = 0; q < SI; ++q)
            if (ok[q]) o.w[off + k + q] = __uint_as_float(wv[q]);
        }
      }
      if (COMPACT) {
        unsigned c = 0;
#pragma unroll
        for (int q = 0; q < SI; ++q) c += ok[q] ? 1u : 0u;
        const unsigned incl = wave_incl_sum_u32(c);
        write_kept(o, (int)(base + kept + incl - c), ok, cv, wv);
        kept += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
      }
    }
    if (KEY != kKeyNone && lane == 0) {
      if (bw != 0u) cand_of()[v] = (unsigned short)bu;
      else if (CSR && !COMPACT) no_candidate(g, v);
    }
    if (COMPACT && kept > 0u) {
      if ((int)kept <= o.thr) {
        unsigned none;
        take_room(o, 0u, 1, none, ps);
      } else {
        ps = g.n - 1 - take_long(&solo_sm().cnt[o.ci].nl, 1);
      }
      if (lane == 0) o.list[ps] = make_int4(v, (int)base, (int)kept, 0);
    }
    return kept;
  }

  // The rows of one wave block (lane: row v with len entries at off; len = 0:
  // nothing to do), 64 >> lg of them a step. PAIR: two steps' loads in flight.
  template <bool PAIR>
  static __device__ __forceinline__ unsigned block_rows(const SoloGraph& g, const SoloOut& o, const int* col,
                                                        const float* w, int lg, unsigned long long gm, int v, int off,
                                                        int len) {
    const unsigned long long bal = __ballot(len > 0);
    const int na = (int)__popcll(bal);
    if (na == 0) return 0u;
    const int lane = lane_id();
    if (na < 64 && lg > 0) {  // rows with work to the front
      const int rank = (int)__popcll(bal & lanemask_lt());
      const int to = 4 * (len > 0 ? rank : na + lane - rank);
      v = __builtin_amdgcn_ds_permute(to, v);
      off = __builtin_amdgcn_ds_permute(to, off);
      len = __builtin_amdgcn_ds_permute(to, len);
    }
    unsigned kept = 0;
    int ca[SI];
    unsigned wa[SI];
    if (lg == 0) {
      load_row<W>(col, w, off, g.lim, len > 0, ca, wa);
      return short_step(g, o, 0, gm, v, off, len, ca, wa);
    }
    const int sub = lane & ((1 << lg) - 1), grp = lane >> lg, per = 64 >> lg;
    for (int i = 0; i < na; i += PAIR ? 2 * per : per) {
      const int sa = i + grp;  // < 64: per divides 64
      const int va = __shfl(v, sa, 64), oa = __shfl(off, sa, 64), la = __shfl(len, sa, 64);
      load_row<W>(col, w, oa + SI * sub, g.lim, SI * sub < la, ca, wa);
      if (PAIR) {
        const int sb = i + per + grp;  // (per <= 32: below 64 too)
        const int vb = __shfl(v, sb, 64), ob = __shfl(off, sb, 64), lb = __shfl(len, sb, 64);
        int cb[SI];
        unsigned wb[SI];
        load_row<W>(col, w, ob + SI * sub, g.lim, SI * sub < lb, cb, wb);
        kept += short_step(g, o, lg, gm, va, oa, la, ca, wa);
        if (i + per < na) kept += short_step(g, o, lg, gm, vb, ob, lb, cb, wb);
      } else {
        kept += short_step(g, o, lg, gm, va, oa, la, ca, wa);
      }
    }
    return kept;
  }
};

// The solve's final record (t: the first live set without an edge).
__device__ void solo_record(const SoloArgs& a, unsigned err, int t, unsigned long long matched,
                            unsigned long long ticks) {
  PhaseMirror m;
  m.L = 0;
  m.matched = matched;
  m.pieces = 0;
  m.t = t;
  m.gen = a.gen;
  m.err = err;
  m.last_nonempty = t - 1;
  m.pad = 1;  // the live set this kernel started from
  m.ticks = ticks;
  m.tag = 0ull;
  PhaseMirror* slot = a.final_rec;
  *(volatile unsigned long long*)&slot->tag = 0ull;
  __threadfence_system();
  *slot = m;
  __threadfence_system();
  *(volatile unsigned long long*)&slot->tag = mirror_tag(a.gen, t);
}

}  // namespace

// LANES lanes, SI entries per lane and step, WPS waves per SIMD.
template <int LANES, int SI, int WPS, bool UNW>
__global__ __launch_bounds__(LANES, WPS) void k_solo(SoloArgs a) {
  SoloSmem& sm = solo_sm();
  const unsigned long long t0 = wall_clock64();
  constexpr int NW = LANES / 64;
  constexpr bool PAIR = SI == 4 || WPS <= 4;  // registers for two steps' loads
  const int tid = threadIdx.x, lane = lane_id(), wv = uni(wave_id());
  if (a.check_err) {  // the input check found something, or the phase kernels take the batch
    if (tid == 0) sm.err = a.totals->err | (a.order && a.totals->tail_from != kSoloTook ? (unsigned)kErrDeclined : 0u);
    __syncthreads();
    const unsigned e = sm.err;
    __syncthreads();
    if (e) {
      if (!a.order && tid == 0) solo_record(a, e, 1, 0ull, 0ull);
      return;
    }
  }
  int gi = 0;
  long long v0 = 0;
  SoloGraph g;
  unsigned long long S = a.seed;
  g.n = a.n;
  if (a.order) {
    gi = uni(a.order[blockIdx.x]);
    v0 = uni(a.vtx_off[gi]);
    g.n = uni((int)(a.vtx_off[gi + 1] - v0));
    S = uni(a.gseed[gi]);
  }
  const int n = g.n;
  g.rp = a.rp + v0;
  g.e0 = uni(g.rp[0]);
  long long e1 = uni(g.rp[n]);
  const bool bad = g.e0 < 0 || e1 > a.nnz || e1 < g.e0 || (v0 == 0 && g.e0 != 0) ||
                   (v0 + n == a.N && e1 != a.nnz);
  if (bad) e1 = g.e0 = 0;  // every row fails its check below; nothing is read
  g.E = (int)(e1 - g.e0);
  g.lim = (int)(a.nnz - g.e0);
  const int npad = (n + 63) & ~63;
  unsigned short* C = cand_of();
  g.mb = kSoloHead + 2 * npad;
  g.nb = g.mb + npad / 8;
  int* mate = a.mate + v0;
  auto list = [&](int i) -> int4* { return (i ? a.rows[1] : a.rows[0]) + v0; };
  auto bc = [&](int i) -> int* { return (i ? a.ecol[1] : a.ecol[0]) + g.e0; };
  auto bw = [&](int i) -> float* { return (i ? a.ew[1] : a.ew[0]) + g.e0; };
  const int* col = a.col + g.e0;
  const float* w = UNW ? nullptr : a.w + g.e0;
  if (tid == 0) {
    sm.cnt[0] = sm.cnt[1] = SoloCnt{0ull, 0, 0u, 0u, 0};
    sm.nl1 = 0;
    sm.rows1 = 0;
    sm.err = bad ? (unsigned)kErrRowPtr : 0u;
  }
  __syncthreads();
  // Pass t: t = 0 computes the candidates of R_1; t >= 1 is phase t, its
  // mutual check and then the compaction that computes the candidates of
  // phase t + 1. Passes 0 and 1 read R_1 from the CSR (row_ptr; its long rows
  // are listed at the back of list 1 by pass 0), later ones R_t from list cl
  // and entry buffer cl.
  auto pass = [&](auto csr, auto compact, auto key, const SoloOut& o, int lg, unsigned long long gm, int ns, int nl,
                  int cl, unsigned& kept, unsigned& md) {
    constexpr bool COMPACT = decltype(compact)::value, CSR = decltype(csr)::value;
    using P = SoloPass<SI, UNW, CSR, COMPACT, decltype(key)::value>;
    const int thr = SI << lg;
    const int4* li = list(cl);
    const int* ic = CSR ? col : bc(cl);
    const float* iw = CSR ? w : (const float*)bw(cl);
    unsigned err = 0;
    int live = 0;
    const int rows = CSR ? n : ns;
    // rows a wave takes at a time: 64, or fewer so that every wave has some
    // (the bits of R_1's empty rows are written 32 at a time)
    const int rb = min(64, max(CSR ? 32 : 64 >> lg, (rows + NW - 1) / NW));
    const int step = CSR ? (rb > 32 ? 64 : 32) : (rb + (64 >> lg) - 1) & ~((64 >> lg) - 1);
    for (int j0 = wv * step; j0 < rows; j0 += NW * step) {
      int v = j0 + lane, off = 0, len = 0;
      if (CSR) {
        if (v < n && lane < step) {
          const long long r0 = g.rp[v] - g.e0, r1 = g.rp[v + 1] - g.e0;
          if (r0 < 0 || r1 < r0 || r1 > g.E) {
            err = kErrRowPtr;
          } else {
            off = (int)r0;
            len = (int)(r1 - r0);
          }
        }
        if (!COMPACT) {  // R_1's empty and long rows
          const unsigned long long bal = __ballot(len > 0);
          if (lane == 0) {
            words_at(g.nb)[j0 >> 5] = ~(unsigned)bal;
            if (step == 64) words_at(g.nb)[(j0 >> 5) + 1] = ~(unsigned)(bal >> 32);
          }
          if (v < n && lane < step && len == 0) C[v] = (unsigned short)v;
          live += (int)__popcll(bal);
          const bool lng = len > thr;
          const unsigned long long bl = __ballot(lng);
          if (bl) {
            const int at = take_long(&sm.nl1, (int)__popcll(bl));
            if (lng) list(1)[n - 1 - (at + (int)__popcll(bl & lanemask_lt()))] = make_int4(v, off, len, 0);
          }
        }
        if (len > thr) len = 0;  // (below)
      } else if (v < rows && lane < step) {
        const int4 r = li[v];
        v = r.x;
        off = r.y;
        len = r.z;
      }
      if (COMPACT && len > 0 && bit_of(g.mb, v)) {
        md += (unsigned)len;
        len = 0;
      }
      kept += P::template block_rows<PAIR>(g, o, ic, iw, lg, gm, v, off, len);
    }
    if (CSR && !COMPACT) {
      if (lane == 0 && live) atomicAdd(&sm.rows1, live);
      if (err) atomicOr(&sm.err, err);
      __syncthreads();
      nl = uni(sm.err ? 0 : sm.nl1);
    }
    const int4* ll = CSR ? list(1) : li;
    for (int j = wv; j < nl; j += NW) {
      int4 r = ll[n - 1 - j];
      r.x = uni(r.x);
      r.y = uni(r.y);
      r.z = uni(r.z);
      if (COMPACT && bit_of(g.mb, r.x)) {
        md += lane == 0 ? (unsigned)r.z : 0u;
      } else {
        kept += P::long_row(g, o, ic, iw, r.x, r.y, r.z);
      }
    }
  };
  unsigned L = (unsigned)g.E, fail = 0u;
  int V = n, ns = 0, nl = 0, cl = 1;
  int lg = group_lg<SI>(L, max(n, 1));
  int t = 0;
  unsigned long long matched = 0;
  for (;;) {
    const int ci = t & 1;
    const int4* li = list(cl);
    if (t > 0) {  // ---- mutual check
      int mv = 0;
      const int rows = t == 1 ? npad : ns + nl;
      for (int j0 = wv * 64; j0 < rows; j0 += LANES) {
        const int j = j0 + lane;
        int v = j;
        if (t > 1) v = j < rows ? li[j < ns ? j : n - 1 - (j - ns)].x : n;
        bool m = v < n && !(t == 1 && bit_of(g.nb, v));
        const int u = m ? C[v] : 0;
        m = m && C[u] == v;
        const unsigned long long bal = __ballot(m);
        if (t == 1) {
          if (lane == 0) {
            words_at(g.mb)[j0 >> 5] = (unsigned)bal;
            words_at(g.mb)[(j0 >> 5) + 1] = (unsigned)(bal >> 32);
          }
          if (v < n) mate[v] = m ? u : -1;
        } else if (m) {
          mate[v] = u;
          atomicOr(&words_at(g.mb)[v >> 5], 1u << (v & 31));
        }
        mv += (int)__popcll(bal);
      }
      if (lane == 0 && mv) atomicAdd(&sm.cnt[ci].mv, mv);
      __syncthreads();
      if (tid == 0) sm.cnt[ci ^ 1] = SoloCnt{0ull, 0, 0u, 0u, 0};  // every lane has read it
    }
    // ---- first argmax, or the compaction with the next candidates
    const bool compact = t > 0;
    g.S = cand_seed(S, a.renew, t + 1);
    const int lgn = group_lg<SI>(L / 2, max(V, 1));  // lanes per row in the next live set, whose rows are shorter
    const int d = t <= 1 ? 0 : cl ^ 1;
    const SoloOut o{bc(d), bw(d), list(d), ci, SI << lgn};
    const unsigned long long gm = group_mask(lg);
    unsigned kept = 0, md = 0;
    using K0 = std::integral_constant<SoloKey, kKeyNone>;
    using KW = std::integral_constant<SoloKey, kKeyWeight>;
    using KH = std::integral_constant<SoloKey, kKeyHash>;
    using KS = std::integral_constant<SoloKey, kKeyStored>;
    const std::true_type yes{};
    const std::false_type no{};
    // An unweighted graph's hashes cost more than all else, so R_1's are
    // computed once and a later live set's after its compaction (whose lanes
    // mostly hold entries that go), the high words kept for the phases after
    // it; renewed keys are hashed in every phase.
    bool hash = false;
    if (t == 0) {
      if constexpr (UNW) pass(yes, no, KH(), o, lg, gm, ns, nl, cl, kept, md);
      else pass(yes, no, KW(), o, lg, gm, ns, nl, cl, kept, md);
    } else if (t == 1) {
      if constexpr (UNW) pass(yes, yes, K0(), o, lg, gm, ns, nl, cl, kept, md);
      else pass(yes, yes, KW(), o, lg, gm, ns, nl, cl, kept, md);
      hash = UNW;
    } else if constexpr (!UNW) {
      pass(no, yes, KW(), o, lg, gm, ns, nl, cl, kept, md);
    } else if (a.renew) {
      pass(no, yes, K0(), o, lg, gm, ns, nl, cl, kept, md);
      hash = true;
    } else {
      pass(no, yes, KS(), o, lg, gm, ns, nl, cl, kept, md);
    }
    if (t == 0) {
      V = uni(sm.rows1);
      nl = uni(sm.nl1);
      fail = uni(sm.err);
    }
    if (compact) {
      md = (unsigned)__builtin_amdgcn_readlane((int)wave_incl_sum_u32(md), 63);
      if (lane == 0) {
        if (kept) atomicAdd(&sm.cnt[ci].kept, kept);
        if (md) atomicAdd(&sm.cnt[ci].md, md);
      }
    }
    __syncthreads();
    if (compact) {
      SoloCnt c = sm.cnt[ci];
      c.at = uni(c.at);
      c.nl = uni(c.nl);
      c.kept = uni(c.kept);
      c.md = uni(c.md);
      c.mv = uni(c.mv);
      if (tid == 0) {  // the record of phase t
        if (a.acc) {
          const int at = solo_log_slot(t, a.acc_n);
          if (at >= 0) {
            unsigned* rec =
                reinterpret_cast<unsigned*>(t < kSoloHot ? a.hot + (blockIdx.x % kSoloCopies) * kSoloHot + t : a.acc + at);
            atomicAdd(rec + 0, L);
            atomicAdd(rec + 1, (unsigned)V);
            atomicAdd(rec + 2, (unsigned)c.mv / 2u);
            atomicAdd(rec + 3, c.md);
          }
        } else if (t <= a.log_cap) {
          a.log[t - 1] = LogRec{(long long)L, (long long)V, (long long)(c.mv / 2), (long long)c.md};
        }
      }
      matched += (unsigned long long)c.mv;
      L = c.kept;
      ns = (int)(c.at >> 32);
      nl = c.nl;
      V = ns + nl;
      cl = d;
      lg = lgn;
      if (c.mv == 0) fail = kErrStall;  // live edges and no match: the input is not symmetric
      if constexpr (UNW) {
        if (hash && L != 0 && !fail) {
          const SoloOut k{nullptr, bw(cl), nullptr, ci, 0};
          pass(no, no, KH(), k, lgn, group_mask(lgn), ns, nl, cl, kept, md);
          __syncthreads();
        }
      }
    }
    ++t;
    if (fail || L == 0) break;
  }
  if (t == 1) {  // no edge: nothing was matched
    for (int v = tid; v < n; v += LANES) mate[v] = -1;
  }
  // (t - 1 phases ran)
  if (a.order) {
    if (tid == 0) {
      if (fail) atomicOr(&a.totals->err, fail);
      uint4* head = a.hot + (blockIdx.x % kSoloCopies) * kSoloHot;
      atomicAdd(reinterpret_cast<unsigned long long*>(head), matched);
      atomicMax(reinterpret_cast<int*>(head) + 2, t - 1);
      if (a.gphase) a.gphase[gi] = t - 1;
    }
  } else {
    // Every lane's mate is written before the record: a barrier alone does not
    // wait for the other waves' stores, and lane 0's release of the record only
    // for its own wave's.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) {
      if (a.gphase) a.gphase[0] = t - 1;
      solo_record(a, fail, t, matched, wall_clock64() - t0);
    }
  }
}

// Graphs of a batch by size class (class k: at most cls_n[k] vertices), the
// ones with the most entries first; the counters and the phase log cleared.
// One workgroup sorts (a counting sort by four steps per factor of two of
// the entries) and looks for a graph of more than `limit` entries, which leaves
// the batch to the phase kernels; the others clear the log.
constexpr int kSoloBins = 128;
__global__ __launch_bounds__(1024) void k_solo_order(SoloOrder a) {
  if (blockIdx.x > 0) {
    const int stride = ((int)gridDim.x - 1) * 1024;
    for (int i = ((int)blockIdx.x - 1) * 1024 + (int)threadIdx.x; i < a.acc_n; i += stride)
      a.acc[i] = make_uint4(0u, 0u, 0u, 0u);
    for (int i = ((int)blockIdx.x - 1) * 1024 + (int)threadIdx.x; i < kSoloCopies * kSoloHot; i += stride)
      a.hot[i] = make_uint4(0u, 0u, 0u, 0u);
    return;
  }
  __shared__ int hist[kSoloClasses * kSoloBins];
  __shared__ int large;
  const int tid = threadIdx.x;
  if (tid == 0) {
    large = 0;
    if (a.clear) a.totals->err = 0;
  }
  for (int i = tid; i < kSoloClasses * kSoloBins; i += 1024) hist[i] = 0;
  __syncthreads();
  // bin of graph i: class first, then entries descending; -1: no vertices
  auto bin = [&](int i) -> int {
    const long long va = a.vtx_off[i], vb = a.vtx_off[i + 1];
    if (vb == va) return -1;
    int k = 0;
    while (k + 1 < kSoloClasses && vb - va > a.cls_n[k]) ++k;
    const long long e = a.rp[vb] - a.rp[va];
    if (e > a.limit) large = 1;
    int x = 0;
    if (e >= 4) {
      const int lz = __clzll(e);  // entries may be any value in a malformed row_ptr
      x = 4 * (61 - lz) + (int)((e >> (61 - lz)) & 3);
      x = min(max(x, 0), kSoloBins - 1);
    }
    return (kSoloClasses - 1 - k) * kSoloBins + (kSoloBins - 1 - x);
  };
  for (int i = tid; i < a.graphs; i += 1024) {
    const int b = bin(i);
    if (b >= 0) atomicAdd(&hist[b], 1);
    else if (a.gphase) a.gphase[i] = 0;
  }
  __syncthreads();
  if (tid == 0) a.totals->tail_from = large ? 0 : kSoloTook;
  if (tid < 64) {  // exclusive prefix, largest class first
    int carry = 0;
    for (int c = 0; c < kSoloClasses * kSoloBins; c += 64) {
      const int x = hist[c + tid];
      const int incl = (int)wave_incl_sum_u32((unsigned)x);
      hist[c + tid] = carry + incl - x;
      carry += __builtin_amdgcn_readlane(incl, 63);
    }
  }
  __syncthreads();
  for (int i = tid; i < a.graphs; i += 1024) {
    const int b = bin(i);
    if (b >= 0) a.order[atomicAdd(&hist[b], 1)] = i;
  }
}

// The phase log of a batch from its sums, and the final record.
__global__ __launch_bounds__(1024) void k_solo_fin(SoloArgs a) {
  __shared__ unsigned sum[4 * kSoloHot];
  __shared__ unsigned long long matched;
  __shared__ int phases;
  const int tid = threadIdx.x;
  if (tid < 4 * kSoloHot) sum[tid] = 0u;
  if (tid == 0) {
    matched = 0ull;
    phases = 0;
  }
  __syncthreads();
  for (int i = tid; i < kSoloCopies * kSoloHot; i += 1024) {
    const uint4 r = a.hot[i];
    unsigned* rec = sum + 4 * (i % kSoloHot);
    if (i % kSoloHot == 0) {
      atomicAdd(&matched, ((unsigned long long)r.y << 32) | r.x);
      atomicMax(&phases, (int)r.z);
    } else {
      atomicAdd(rec + 0, r.x);
      atomicAdd(rec + 1, r.y);
      atomicAdd(rec + 2, r.z);
      atomicAdd(rec + 3, r.w);
    }
  }
  __syncthreads();
  for (int i = tid; i < phases && i < a.log_cap; i += 1024) {
    const int at = solo_log_slot(i + 1, a.acc_n);
    uint4 r = make_uint4(0u, 0u, 0u, 0u);
    if (at >= 0) {
      if (i + 1 < kSoloHot) r = make_uint4(sum[4 * i + 4], sum[4 * i + 5], sum[4 * i + 6], sum[4 * i + 7]);
      else r = a.acc[at];
    }
    a.log[i] = LogRec{(long long)r.x, (long long)r.y, (long long)r.z, (long long)r.w};
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned declined = a.totals->tail_from != kSoloTook ? (unsigned)kErrDeclined : 0u;
    solo_record(a, a.totals->err | declined, phases + 1, matched, 0ull);
  }
}

// ------------------------------------------------------------------ host

namespace {

template <int LANES, int SI, int WPS, bool UNW>
hipError_t launch_solo(const SoloArgs& a, int grid, size_t lds, hipStream_t s, hipEvent_t* ev) {
  // more dynamic LDS than the default limit: raised per device by solo_setup
  if (ev)
    hipExtLaunchKernelGGL((k_solo<LANES, SI, WPS, UNW>), dim3(grid), dim3(LANES), lds, s, ev[0], ev[1], 0, a);
  else
    hipLaunchKernelGGL((k_solo<LANES, SI, WPS, UNW>), dim3(grid), dim3(LANES), lds, s, a);
  return hipGetLastError();
}

size_t solo_lds(int64_t n) {
  const size_t np = (size_t)((n + 63) & ~(int64_t)63);
  return kSoloHead + np * 2 + np / 4;
}

// Class k of a batch: graphs of at most kSoloClsN[k] vertices.
constexpr int64_t kSoloClsN[kSoloClasses] = {2048, 32768, kSoloMaxN};

hipError_t launch_solo_class(int k, bool unw, const SoloArgs& a, int grid, size_t lds, hipStream_t s,
                             hipEvent_t* ev) {
  if (k == 0)
    return unw ? launch_solo<512, 4, 8, true>(a, grid, lds, s, ev) : launch_solo<512, 4, 8, false>(a, grid, lds, s, ev);
  if (k == 1)
    return unw ? launch_solo<1024, 4, 8, true>(a, grid, lds, s, ev)
               : launch_solo<1024, 4, 8, false>(a, grid, lds, s, ev);
  return unw ? launch_solo<1024, 8, 4, true>(a, grid, lds, s, ev) : launch_solo<1024, 8, 4, false>(a, grid, lds, s, ev);
}

}  // namespace

lm_status solo_setup() {
  const void* f[] = {(const void*)k_solo<512, 4, 8, false>,  (const void*)k_solo<512, 4, 8, true>,
                     (const void*)k_solo<1024, 4, 8, false>, (const void*)k_solo<1024, 4, 8, true>,
                     (const void*)k_solo<1024, 8, 4, false>, (const void*)k_solo<1024, 8, 4, true>};
  for (const void* p : f)
    if (hipFuncSetAttribute(p, hipFuncAttributeMaxDynamicSharedMemorySize, (int)solo_lds(kSoloMaxN)) != hipSuccess) {
      (void)hipGetLastError();
      return LM_EDEVICE;
    }
  return LM_OK;
}

bool Solver::solo_fits(int64_t N, int64_t nnz, int64_t G, const int64_t* vtx_off, const int64_t* row_ptr,
                       bool unweighted, bool async) const {
  if (tun.tail_entries <= 0) return false;  // phase kernels only
  if (G == 1)
    return N <= kSoloMaxN && nnz <= std::min<int64_t>(kSoloEntries, tun.tail_entries);
  if (G > solo_graph_limit(N, async)) return false;
  int64_t mx = 0, me = 0;
  for (int64_t g = 0; g < G; ++g) {
    mx = std::max(mx, vtx_off[g + 1] - vtx_off[g]);
    if (row_ptr) me = std::max(me, row_ptr[vtx_off[g + 1]] - row_ptr[vtx_off[g]]);
  }
  return mx <= kSoloMaxN && me <= solo_entry_limit(N, nnz, unweighted, async);
}

// Runs the solve whose graphs solo_fits accepted. The entries of a batch's graphs
// are on the device: where their number and the graphs' vertices allow one of more
// than the limit, the device looks, and leaves such a batch to the phase kernels
// (*declined; a stream-ordered solve has them queued behind, doing nothing
// otherwise).
lm_status Solver::run_solo(const Problem& p, const Work& wk, const int64_t* vtx_off, uint64_t seed, hipStream_t s,
                           uint32_t flags, lm_stats* st, bool* declined) {
#define HIPCHK(x)                          \
  do {                                     \
    hipError_t _e = (x);                   \
    if (_e != hipSuccess) {                \
      (void)hipGetLastError();             \
      return dev_status(_e);               \
    }                                      \
  } while (0)
  *declined = false;
  if (++gen == 0) gen = 1;
  const bool unw = p.w == nullptr;
  const bool check = (flags & LM_CHECK_GRAPH) != 0;
  const bool prof = (flags & LM_PROFILE) != 0 && (!st || !st->profile_kinds || (st->profile_kinds >> LM_K_TAIL & 1u));
  std::vector<size_t> marks;
  auto timing = [&](hipEvent_t* ev) -> hipEvent_t* {
    if (!prof) return nullptr;
    const size_t i = 2 * marks.size();
    ev[0] = event(i);
    ev[1] = event(i + 1);
    marks.push_back(i);
    return ev;
  };
  SoloArgs a;
  std::memset(&a, 0, sizeof(a));
  a.rp = p.row_ptr;
  a.col = p.col;
  a.w = p.w;
  a.mate = p.mate;
  a.N = p.N;
  a.nnz = p.nnz;
  a.n = (int)p.N;
  a.seed = premix_seed(seed);
  a.renew = (flags & LM_RENEW_KEYS) ? 1 : 0;
  for (int i = 0; i < 2; ++i) {
    a.rows[i] = wk.rows[i];
    a.ecol[i] = wk.ecol[i];
    a.ew[i] = wk.ew[i];
  }
  a.totals = wk.totals;
  a.check_err = check || p.G > 1 ? 1 : 0;
  a.gphase = p.gphase;
  a.log = d_log;
  a.log_cap = kLogCap;
  a.final_rec = d_mir + kMirrorSlots;
  a.gen = gen;
  hipEvent_t ev[2];
  const bool one = p.G == 1 && !check && !prof;  // a single launch
  // Whether a graph of the batch may have too many entries (n (n - 1) at most).
  const long long limit = solo_entry_limit(p.N, p.nnz, unw, (flags & LM_ASYNC) != 0);
  bool ask = false;
  for (int64_t g = 0; p.G > 1 && p.nnz > limit && g < p.G && !ask; ++g) {
    const int64_t n = vtx_off[g + 1] - vtx_off[g];
    ask = n * (n - 1) > limit;
  }
  if (!one) HIPCHK(hipEventRecord(e0, s));
  if (check) {
    HIPCHK(launch_zero(wk.ctl, 0, wk.totals, s, nullptr));
    CheckArgs ca{wk.totals, p.nnz, p.row_ptr, p.col, p.w, (int)p.N, (int)p.G, p.vtx_off};
    HIPCHK(launch_check(ca, (int)std::min<int64_t>(num_cus * 8, (p.N + kBlock - 1) / kBlock + 1), s));
  }
  if (p.G == 1) {
    HIPCHK(launch_solo_class(2, unw, a, 1, solo_lds(p.N), s, timing(ev)));
  } else {
    if (ask && (flags & LM_ASYNC)) HIPCHK(launch_zero(wk.ctl, 2, wk.totals, s, wk.tail));  // (for the phase kernels)
    // With no more graphs than CUs every graph gets the widest workgroup.
    const bool few = p.G <= num_cus;
    int64_t cnt[kSoloClasses] = {}, big[kSoloClasses] = {}, mx = 0;
    for (int64_t g = 0; g < p.G; ++g) {
      const int64_t n = vtx_off[g + 1] - vtx_off[g];
      if (n == 0) continue;
      int k = few ? kSoloClasses - 1 : 0;
      while (k + 1 < kSoloClasses && n > kSoloClsN[k]) ++k;
      ++cnt[k];
      big[k] = std::max(big[k], n);
      mx = std::max(mx, n);
    }
    SoloOrder o;
    o.vtx_off = p.vtx_off;
    o.rp = p.row_ptr;
    o.graphs = (int)p.G;
    for (int k = 0; k < kSoloClasses; ++k) o.cls_n[k] = few ? 0 : kSoloClsN[k];
    o.order = wk.C;  // (candidates stay in LDS here)
    o.acc = reinterpret_cast<uint4*>(wk.parts);
    o.acc_n = (int)solo_log_records(mx);
    o.hot = reinterpret_cast<uint4*>(wk.bstat);
    o.gphase = p.gphase;
    o.totals = wk.totals;
    o.clear = check ? 0 : 1;
    o.limit = ask ? limit : LLONG_MAX;
    hipLaunchKernelGGL(k_solo_order, dim3(1 + (o.acc_n + 8191) / 8192), dim3(1024), 0, s, o);
    HIPCHK(hipGetLastError());
    a.vtx_off = p.vtx_off;
    a.gseed = wk.gseed;
    a.acc = o.acc;
    a.acc_n = o.acc_n;
    a.hot = o.hot;
    // The largest graphs take a CU each and end one by one; the others run
    // beside them on a second stream (the smallest first: their LDS fits next
    // to a large graph's).
    const bool fork = cnt[kSoloClasses - 1] > 0 && cnt[kSoloClasses - 1] < p.G;
    if (fork) {
      if (!side) HIPCHK(hipStreamCreateWithFlags(&side, hipStreamNonBlocking));
      if (!e_fork) HIPCHK(hipEventCreateWithFlags(&e_fork, hipEventDisableTiming));
      HIPCHK(hipEventRecord(e_fork, s));
      HIPCHK(hipStreamWaitEvent(side, e_fork, 0));
    }
    int at[kSoloClasses], sum = 0;
    for (int k = kSoloClasses - 1; k >= 0; --k) {
      at[k] = sum;
      sum += (int)cnt[k];
    }
    for (int i = 0; i < kSoloClasses; ++i) {
      const int k = i == 0 ? kSoloClasses - 1 : i - 1;
      if (cnt[k] == 0) continue;
      a.order = wk.C + at[k];
      HIPCHK(launch_solo_class(k, unw, a, (int)cnt[k], solo_lds(big[k]), i > 0 && fork ? side : s, timing(ev)));
    }
    if (fork) {
      HIPCHK(hipEventRecord(e_fork, side));
      HIPCHK(hipStreamWaitEvent(s, e_fork, 0));
    }
    hipLaunchKernelGGL(k_solo_fin, dim3(1), dim3(1024), 0, s, a);
    HIPCHK(hipGetLastError());
  }
  if (flags & LM_ASYNC) {
    if (ask) {
      Problem q = p;
      q.after_solo = true;
      return run(q, wk, s, flags, st);
    }
    HIPCHK(hipEventRecord(e_async, s));
    async_pending = true;
    return LM_OK;
  }
  if (one) {
    // The record is the kernel's last store: every wave has waited for its
    // stores, and they were released to the system, before it. It is polled, and
    // carries the solve's time. Two events
    // and a wait on one of them cost a short solve half its time (er 300:
    // 52 us a call against 32).
    const volatile PhaseMirror* slot = &h_mir[kMirrorSlots];
    for (unsigned spin = 1; (unsigned)(slot->tag >> 32) != gen; ++spin) {
      if ((spin & 4095u) == 0u) {
        const hipError_t q = hipStreamQuery(s);
        if (q != hipErrorNotReady) {
          HIPCHK(q);
          break;  // ended: the record is there, or never will be
        }
      }
    }
    std::atomic_thread_fence(std::memory_order_acquire);
  } else {
    HIPCHK(hipEventRecord(e1, s));
    HIPCHK(hipEventSynchronize(e1));
  }
  const PhaseMirror fin = h_mir[kMirrorSlots];
  if ((unsigned)(fin.tag >> 32) != gen) return LM_EDEVICE;
  if (fin.err == kErrDeclined) {
    *declined = true;
    return LM_OK;
  }
  if (fin.err) {
    if (fin.err & kErrWeight) return LM_EWEIGHT;
    if (fin.err & (kErrRowPtr | kErrColRange | kErrSelfLoop | kErrStall | kErrAsym)) return LM_EGRAPH;
    return LM_EDEVICE;
  }
  last_phases = fin.last_nonempty;
  if (!st) return LM_OK;
  float ms = (float)((double)fin.ticks / (double)clock_khz);
  if (!one) HIPCHK(hipEventElapsedTime(&ms, e0, e1));
  st->phases = fin.last_nonempty;
  st->matched_edges = (int64_t)(fin.matched / 2);
  st->device_ms = ms;
  for (int k = 0; k < LM_K_KINDS; ++k) {
    st->k_launches[k] = 0;
    st->k_ms[k] = 0.0;
    st->k_bytes[k] = 0.0;
  }
  for (size_t i : marks) {
    float km = 0.f;
    if (!event(i) || !event(i + 1)) return LM_ENOMEM;
    HIPCHK(hipEventElapsedTime(&km, event(i), event(i + 1)));
    st->k_launches[LM_K_TAIL] += 1;
    st->k_ms[LM_K_TAIL] += km;
  }
  const int nrec = std::min(fin.last_nonempty, kLogCap);
  st->log_len = 0;
  if (st->log && st->log_cap > 0) {
    st->log_len = std::min(nrec, st->log_cap);
    std::memcpy(st->log, h_log, sizeof(LogRec) * (size_t)st->log_len);
  }
  // Algorithmic bytes, all of them the one kernel's: row_ptr and the entries
  // read for the first argmax and again (unmatched rows) by the compaction of
  // phase 1, mate written, then the survivors written and read once a phase,
  // with a 16-byte record per live row.
  const double eb = unw ? 4.0 : 8.0;
  double b = 16.0 * ((double)p.N + 1.0) + 4.0 * (double)p.N;
  for (int i = 0; i < nrec; ++i) {
    const double L = (double)h_log[i].live_entries, md = (double)h_log[i].matched_entries;
    const double L2 = i + 1 < nrec ? (double)h_log[i + 1].live_entries : 0.0;
    const double V2 = i + 1 < nrec ? (double)h_log[i + 1].live_rows : 0.0;
    b += (i == 0 ? eb * L : 0.0) + eb * (L - md) + eb * L2 + 48.0 * V2 + 8.0 * (double)h_log[i].matched_edges;
  }
  st->k_bytes[LM_K_TAIL] = b;
  st->bytes_alg = b;
#undef HIPCHK
  return LM_OK;
}

}  // namespace lm
