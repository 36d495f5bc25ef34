// Device-side tail of the phase loop of local-max matching (gfx950, wave64).
//
// Once the live set is small, a phase costs more in launches and host round
// trips than in work (Section 2: the work of a phase is linear in the live
// edges, and Section 3 notes that the GPU code of the paper was weak on small
// inputs for this reason). k_tail takes the live set R_c the phase kernels
// left behind and runs every remaining phase in one persistent launch:
//
//   phase    every live vertex v with C[C[v]] = v is matched (mate); every other
//            live row keeps the entries whose neighbour u is not (C[C[u]] != u),
//            writes them to the same offset of the other entry buffer and
//            computes its new candidate;
//   -------- exchange: the counts of the next list and a grid barrier in one
//   log      the phase record (L_t, V_t, matched_t, matched entries_t).
//
// The candidates of two phases have to be there at once, since a neighbour's
// partner is looked up while the next candidates are written: C holds one
// phase's, mate the next one's (a vertex's own word until its row ends).
//
// Nothing is counted through a shared global counter (atomics on one address
// serialise across the dies): workgroup b owns a segment of the next row list
// and reports its counts in a table (TailCtl::seg) that every workgroup reads
// after the exchange; within a workgroup rows are placed with LDS atomics. The
// row order is irrelevant to the result (the key order is strict, so every
// vertex has one candidate whatever the order of its entries). Once a live
// set is at most kTailSolo entries, workgroup 0 finishes alone and the exchange
// is a workgroup barrier.
//
// Bound by latency: a phase is a chain of four to five dependent loads across
// the dies (3 to 5 us) and an exchange (7 to 9 us, the slowest workgroup's lag
// included). With a mutual check and a compaction of their own, three barriers
// and tables read apart, a phase took 16 to 20 us: RGG with 60 K vertices, all
// phases here, 92 -> 79 us, the tail of R-MAT 20 (renewed keys) 110 -> 89, of
// R-MAT 24 148 -> 115.
#include <hip/hip_ext.h>

#include "lm_device.h"
#include "lm_internal.h"
#include "lm_key.h"

namespace lm {

namespace {

// Live entries workgroup 0 handles alone. A grid phase costs about 12 us down to
// the smallest live set; alone, 14 K entries took 43 us, 2 K take 11 and a
// hundred 4.
constexpr long long kTailSolo = 2048;
constexpr int kTW = kTailBlock / 64;    // waves per workgroup
constexpr int kChunk = 8;               // vertices dealt to a workgroup at a time
constexpr int kLongStep = 4;            // entries per lane and step of a long row
// The first candidate of a longer row is found by the whole grid, behind an exchange
// of its own (8 us; one wave reads 8 K entries in 30). A star of 500 K leaves by one
// wave 1690 us a call, by its workgroup 205, by the grid 89.
constexpr int kHubRow = 8192;
constexpr int kRunCache = kMaxBlocks + 1;

__device__ __forceinline__ unsigned ld_u32(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

struct TailSmem {
  int pre_s[kTailMaxBlocks + 1];  // short rows of the current list before segment b
  int pre_l[kTailMaxBlocks + 1];  // long rows before segment b
  int sbase[kTailMaxBlocks], scap[kTailMaxBlocks];
  long long kept, md;           // the current list: its live entries, the entries matched on the way to it
  unsigned long long mv;        // low word: vertices matched on the way to it; high word: its closed rows
  long long kept_b, md_b;       // the same of this workgroup and the next list
  unsigned long long mv_b;
  int cnt_s, cnt_l;  // rows this workgroup has placed in its segment
  unsigned ok;
  int rp[kRunCache];  // conversion: piece prefix of R_c's runs
  Key hub[kTW];       // each wave's best of a row of the whole grid
};

// Ends a phase: this workgroup's segment of the next list (base, cap, and the
// counts in sm) goes to tab[b], and every workgroup's comes back as the
// prefixes and sums in sm. This is also the barrier of the grid (every
// workgroup is resident: the host sizes the grid from the occupancy of this
// kernel): a workgroup stores the number `g` of the exchange behind its segment
// and its first wave polls the others' numbers, two a lane, until all are
// there. That is one store and one load across the dies, where counters took
// two atomics, a store and a load. The workgroup barrier first waits
// for every lane's stores; lane 0 then makes them visible to the other dies
// (release) before it stores its number; the polls are plain device-scope loads
// (an acquire per poll would invalidate the L2 under the workgroups still
// working), and the caches are invalidated once (acquire) when all have come. A
// wait longer than `limit` ticks of the constant wall clock, or another
// workgroup's abort, makes every workgroup give up (false).
__device__ bool exchange(TailCtl* tc, TailSeg* tab, int base, int cap, int nb, unsigned g, bool alone,
                         unsigned long long limit, Totals* tot, TailSmem& sm) {
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (wave_id() == 0) {
    const int lane = lane_id();
    const int b = (int)blockIdx.x;
    bool ok = true;
    TailSeg s0{}, s1{};
    if (lane == 0) {
      s0.base = base;
      s0.cap = cap;
      s0.ns = sm.cnt_s;
      s0.nl = sm.cnt_l;
      s0.kept = sm.kept_b;
      s0.md = sm.md_b;
      s0.mv = sm.mv_b;
      sm.cnt_s = sm.cnt_l = 0;
      sm.kept_b = sm.md_b = 0;
      sm.mv_b = 0;
    }
    if (!alone) {
      if (lane == 0) {
        tab[b] = s0;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // this die's stores reach the others
        __hip_atomic_store(&tc->tag[b], g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      const unsigned long long t0 = wall_clock64();
      for (;;) {
        const unsigned x0 = lane < nb ? ld_u32(&tc->tag[lane]) : g;
        const unsigned x1 = lane + 64 < nb ? ld_u32(&tc->tag[lane + 64]) : g;
        const unsigned stop = ld_u32(&tc->abort[0]);
        if (__ballot((int)(x0 - g) < 0 || (int)(x1 - g) < 0) == 0ull) break;
        const bool late = __ballot(wall_clock64() - t0 > limit) != 0ull;
        if (late && lane == 0) {
          __hip_atomic_fetch_or(&tc->abort[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          atomicOr(&tot->err, (unsigned)kErrInternal);
        }
        if (late || __ballot(stop != 0u) != 0ull) {
          ok = false;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // drop stale lines before the next step
      s0 = lane < nb ? tab[lane] : TailSeg{};
      s1 = lane + 64 < nb ? tab[lane + 64] : TailSeg{};
    }
    const int n = alone ? 1 : nb;
    const int is0 = (int)wave_incl_sum_u32((unsigned)s0.ns), il0 = (int)wave_incl_sum_u32((unsigned)s0.nl);
    const int is1 = (int)wave_incl_sum_u32((unsigned)s1.ns) + __builtin_amdgcn_readlane(is0, 63);
    const int il1 = (int)wave_incl_sum_u32((unsigned)s1.nl) + __builtin_amdgcn_readlane(il0, 63);
    if (lane < n) {
      sm.pre_s[lane] = is0 - s0.ns;
      sm.pre_l[lane] = il0 - s0.nl;
      sm.sbase[lane] = s0.base;
      sm.scap[lane] = s0.cap;
    }
    if (lane + 64 < n) {
      sm.pre_s[lane + 64] = is1 - s1.ns;
      sm.pre_l[lane + 64] = il1 - s1.nl;
      sm.sbase[lane + 64] = s1.base;
      sm.scap[lane + 64] = s1.cap;
    }
    const long long kept = wave_incl_sum<long long>(s0.kept + s1.kept);
    const long long md = wave_incl_sum<long long>(s0.md + s1.md);
    const long long mv = wave_incl_sum<long long>((long long)(s0.mv + s1.mv));
    if (lane == 63) {
      sm.pre_s[n] = is1;
      sm.pre_l[n] = il1;
      sm.kept = kept;
      sm.md = md;
      sm.mv = (unsigned long long)mv;
      sm.ok = ok ? 1u : 0u;
    }
  }
  __syncthreads();
  return sm.ok != 0u;
}

// Places the rows of the lanes with `es` (short, front of the segment) or `el`
// (long, back of the segment): one LDS atomic per wave and kind.
__device__ __forceinline__ void place_rows(bool es, bool el, int4 rec, int4* out, int base, int cap, TailSmem& sm) {
  const unsigned long long bs = __ballot(es), bl = __ballot(el);
  const unsigned long long lt = lanemask_lt();
  int ps = 0, pl = 0;
  if (lane_id() == 0) {
    if (bs) ps = atomicAdd(&sm.cnt_s, (int)__popcll(bs));
    if (bl) pl = atomicAdd(&sm.cnt_l, (int)__popcll(bl));
  }
  ps = __shfl(ps, 0, 64);
  pl = __shfl(pl, 0, 64);
  if (es) out[base + ps + (int)__popcll(bs & lt)] = rec;
  if (el) out[base + cap - 1 - (pl + (int)__popcll(bl & lt))] = rec;
}

__device__ __forceinline__ void graph_of(const Common& c, int g, int& base, unsigned long long& S) {
  if (c.graphs == 1) {
    base = 0;
    S = c.gseed[0];
  } else {
    base = c.gbase[g];
    S = c.gseed[g];
  }
}

// Row `i` of the short (long) rows of the current list.
__device__ __forceinline__ int4 short_row(const TailSmem& sm, int nseg, const int4* rows, int i) {
  int lo = 0, hi = nseg;  // largest b with pre_s[b] <= i
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sm.pre_s[mid] <= i) lo = mid;
    else hi = mid;
  }
  return rows[sm.sbase[lo] + (i - sm.pre_s[lo])];
}
__device__ __forceinline__ int4 long_row(const TailSmem& sm, int nseg, const int4* rows, int j) {
  int lo = 0, hi = nseg;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (sm.pre_l[mid] <= j) lo = mid;
    else hi = mid;
  }
  return rows[sm.sbase[lo] + sm.scap[lo] - 1 - (j - sm.pre_l[lo])];
}

// The vertex x of the graph at `base` is matched in this phase: its candidate's
// candidate. `a` is x's candidate; cur holds the phase's candidates (ids of the
// graph).
__device__ __forceinline__ int back(const Common& c, const int* cur, int base, int a) {
  return a >= 0 && (unsigned)(base + a) < (unsigned)c.n ? cur[base + a] : -1;
}

// The entry of largest key of the input row r. One lane.
__device__ __forceinline__ void first_lane(const Common& c, int4 r, unsigned long long S, const int* col,
                                           const float* w, Best& best) {
  constexpr int kW = 8;
  for (int k0 = 0; k0 < r.z; k0 += kW) {
    int u[kW];
    float x[kW];
#pragma unroll
    for (int q = 0; q < kW; ++q) {
      const bool in = k0 + q < r.z;
      u[q] = in ? col[r.y + k0 + q] : -1;
      x[q] = in && w ? w[r.y + k0 + q] : 1.0f;
    }
#pragma unroll
    for (int q = 0; q < kW; ++q)
      if ((unsigned)u[q] < (unsigned)c.n)
        best_update(best, ord_weight_bits(__float_as_uint(x[q])), u[q], (unsigned)r.x, S);
  }
}

// The entry of largest key among the entries e0, e0 + step, ... (kStep each) of
// the row r of a graph of n vertices, on every lane of the wave.
constexpr int kStep = 64 * kLongStep;
__device__ __forceinline__ Key best_of_row(int4 r, int e0, int step, const int* col, const float* w, int n,
                                           unsigned long long S) {
  const int lane = lane_id();
  Best best = best_ident();
  for (; e0 < r.z; e0 += step) {
    int u[kLongStep];
    float x[kLongStep];
#pragma unroll
    for (int h = 0; h < kLongStep; ++h) {
      const int e = e0 + 64 * h + lane;
      u[h] = e < r.z ? col[r.y + e] : -1;
      x[h] = e < r.z && w ? w[r.y + e] : 1.0f;
    }
#pragma unroll
    for (int h = 0; h < kLongStep; ++h)
      if ((unsigned)u[h] < (unsigned)n)
        best_update(best, ord_weight_bits(__float_as_uint(x[h])), u[h], (unsigned)r.x, S);
  }
  return wave_max_key(best_key(best, (unsigned)r.x, S));
}

// One phase of the row r (v's) by one lane: -1 if v is matched (with cv);
// otherwise the entries of unmatched neighbours go to the next entry buffer,
// their number is returned and best gets the largest key among them. The loads
// of v's own check go with those of the first entries.
__device__ __forceinline__ int row_lane(const Common& c, int4 r, int base, unsigned vloc, unsigned long long S,
                                        const int* cur, const int* col, const float* w, int* ncol, float* nw, int& cv,
                                        Best& best) {
  constexpr int kW = 8;
  const bool unw = w == nullptr;
  const int off = r.y, len = r.z;
  int kept = 0;
  cv = cur[r.x];
  for (int k0 = 0; k0 < len; k0 += kW) {
    int u[kW], a[kW];
    float x[kW];
    bool ok[kW];
#pragma unroll
    for (int q = 0; q < kW; ++q) {
      ok[q] = k0 + q < len;
      u[q] = ok[q] ? col[off + k0 + q] : -1;
      x[q] = (ok[q] && !unw) ? w[off + k0 + q] : 1.0f;
      ok[q] = ok[q] && u[q] >= 0 && (unsigned)(base + u[q]) < (unsigned)c.n;
    }
    const int own = k0 == 0 ? back(c, cur, base, cv) : -1;
#pragma unroll
    for (int q = 0; q < kW; ++q) a[q] = ok[q] ? cur[base + u[q]] : -1;
    if (own == (int)vloc) return -1;
#pragma unroll
    for (int q = 0; q < kW; ++q) a[q] = back(c, cur, base, a[q]);
#pragma unroll
    for (int q = 0; q < kW; ++q) {
      if (ok[q] && a[q] != u[q]) {
        ncol[off + kept] = u[q];
        if (!unw) nw[off + kept] = x[q];
        ++kept;
        best_update(best, ord_weight_bits(__float_as_uint(x[q])), u[q], vloc, S);
      }
    }
  }
  return kept;
}

}  // namespace

// R_c (the live set the device phase counter names) in the piece layout of
// the phase kernels becomes the tail's first row list: one row per live
// vertex, its entries at the vertex's virtual position. Rows cut into several
// pieces are contiguous there, so for c >= 2 every run is copied to its
// virtual range first. R_1 needs no copy: its entries are the input rows. Where
// the tail is the whole solve of one graph (csr_rp) the list is made from the
// CSR, its offsets checked as k_init does, and the first candidates with it:
// short rows by a lane each, the others, listed first, by a wave each, and up to
// kTailHubs rows of more than kHubRow entries by the whole grid.
__global__ __launch_bounds__(kTailBlock) void k_tail(TailArgs a) {
  __shared__ TailSmem sm;
  Common& c = a.c;
  Totals* tot = c.totals;
  TailCtl* tc = a.tc;
  const int tid = threadIdx.x, lane = lane_id(), wv = wave_id();
  const int b = blockIdx.x;
  // An error found before this launch ends it: every workgroup reads the same
  // word. Where this launch checks the input itself, the word may change under a
  // workgroup that starts late: all go to the first exchange and look behind it.
  if (tid == 0) sm.ok = (a.csr_rp || tot->err == 0u) && !(c.guard && handed_over(c, tot->tail_from)) ? 1u : 0u;
  __syncthreads();
  if (!sm.ok) return;
  const int c0 = tot->t;
  const int si = (c0 - 1) & 1;  // R_c's buffer set
  const Ctl ctl = *a.ctl[si];
  const int nb = (int)gridDim.x;
  const unsigned long long limit = a.spin_ticks;
  const bool unw = a.ew[0] == nullptr;
  const bool csr = c0 == 1 && a.csr_rp != nullptr;
  int4* TA = a.rows[c0 & 1];
  int4* TB = a.rows[(c0 + 1) & 1];
  // ---- conversion: workgroup b takes pieces [P b / nb, P (b + 1) / nb), its
  // segment of the first row list starts at P b / nb. From the CSR it takes
  // every nb-th kChunk vertices (8 offsets are a line; neighbours in a skewed
  // graph's order go to other workgroups).
  const long long P = csr ? a.n : ctl.pieces;
  int k0 = (int)(P * b / nb), kc = (int)(P * (b + 1) / nb) - k0;  // (k0 + kc may be 2^31)
  if (csr) {
    const int chunks = (int)((P + kChunk - 1) / kChunk), q = chunks / nb, r = chunks % nb;
    k0 = kChunk * (q * b + min(b, r));
    kc = kChunk * (q + (b < r ? 1 : 0));
  }
  if (tid == 0) {
    sm.cnt_s = sm.cnt_l = 0;
    sm.kept_b = sm.md_b = 0;
    sm.mv_b = 0;
  }
  if (!csr) {
    for (int i = tid; i <= ctl.nruns && i < kRunCache; i += kTailBlock) sm.rp[i] = a.rpre[si][i];
  }
  __syncthreads();
  const int* cur_col;
  const float* cur_w;
  int ni;  // the entry buffer phase c writes
  if (c0 == 1) {
    cur_col = a.in_col;
    cur_w = unw ? nullptr : a.in_w;
    ni = 1;
  } else {
    cur_col = a.ecol[(c0 + 1) & 1];
    cur_w = unw ? nullptr : a.ew[(c0 + 1) & 1];
    ni = c0 & 1;
  }
  if (csr) {  // rows and first candidates from the input
    const unsigned long long Sd = cand_seed(c.gseed[0], c.renew, 1);
    unsigned err = b == 0 && tid == 0 && (a.csr_rp[0] != 0 || a.csr_rp[c.n] != a.nnz) ? (unsigned)kErrRowPtr : 0u;
    for (int x0 = tid & ~63; x0 < kc; x0 += kTailBlock) {
      const int x = x0 + lane;
      const long long v = ((long long)(x / kChunk) * nb + b) * kChunk + x % kChunk;
      int4 r = make_int4(0, 0, 0, 0);
      bool es = false, el = false;
      if (x < kc && v < P) {
        const long long e0 = a.csr_rp[v], d = a.csr_rp[v + 1] - e0;
        if (d < 0 || e0 < 0 || e0 + d > a.nnz) err |= kErrRowPtr;
        if (d > 0x7fff0000LL) err |= kErrDegree;
        const bool ok = d > 0 && d <= 0x7fff0000LL && e0 >= 0 && e0 + d <= a.nnz;
        r = make_int4((int)v, (int)e0, (int)d, 0);
        es = ok && d <= kTailShort;
        el = ok && !es;
        Best best = best_ident();
        if (es) first_lane(c, r, Sd, cur_col, cur_w, best);
        c.mate[v] = -1;
        if (!el) c.C[v] = best.u;
      }
      place_rows(es, el, r, TA, k0, kc, sm);
    }
    if (err) atomicOr(&tot->err, err);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const int nl = sm.cnt_l;
    for (int j = wv; j < nl; j += kTW) {
      const int4 r = TA[k0 + (kc - 1 - j)];
      if (r.z > kHubRow) {  // left to the grid
        unsigned h = 0;
        if (lane == 0) h = atomicAdd(&tc->hubs, 1u);
        h = __builtin_amdgcn_readfirstlane(h);
        if (h < (unsigned)kTailHubs) {
          if (lane == 0) tc->hub[h] = r.x;
          continue;
        }
      }
      const Key kb = best_of_row(r, 0, kStep, cur_col, cur_w, c.n, Sd);
      if (lane == 0) c.C[r.x] = kb.u;
    }
  } else {
    const Run* runs = a.runs[si];
    const long long* epre = a.epre[si];
    const int4* pin = a.rows[si];
    if (c0 >= 2) {  // runs b, b + nb, ... to their virtual ranges
      const int* sc = a.ecol[c0 & 1];
      const float* sw = unw ? nullptr : a.ew[c0 & 1];
      int* dc = a.ecol[(c0 + 1) & 1];
      float* dw = unw ? nullptr : a.ew[(c0 + 1) & 1];
      for (int rn = b; rn < ctl.nruns; rn += nb) {
        const Run run = runs[rn];
        const long long vb = epre[rn];
        for (int e = tid; e < run.ent_count; e += kTailBlock) {
          dc[vb + e] = sc[run.phys_begin + e];
          if (!unw) dw[vb + e] = sw[run.phys_begin + e];
        }
      }
    }
    for (int x0 = tid & ~63; x0 < kc; x0 += kTailBlock) {
      const int k = k0 + min(x0 + lane, kc - 1);
      int4 r = make_int4(0, 0, 0, 0);
      bool es = false, el = false;
      if (x0 + lane < kc) {
        int lo = 0, hi = ctl.nruns;  // run of piece k: largest lo with rp[lo] <= k
        while (hi - lo > 1) {
          const int mid = (lo + hi) >> 1;
          if (sm.rp[mid] <= k) lo = mid;
          else hi = mid;
        }
        const Run run = runs[lo];
        const int4 rec = pin[run.row_begin + (k - sm.rp[lo])];
        if ((rec.w & kHeadBit) && rec.z > 0) {
          long long total = rec.z;
          // later pieces of the same vertex (its row was cut at a workgroup boundary)
          int j = k - sm.rp[lo] + 1, rr = lo;
          for (;;) {
            while (rr < ctl.nruns && j >= runs[rr].row_count) {
              ++rr;
              j = 0;
            }
            if (rr >= ctl.nruns) break;
            const int4 nx = pin[runs[rr].row_begin + j];
            if (nx.x != rec.x) break;
            total += nx.z;
            ++j;
          }
          r = make_int4(rec.x, (int)(epre[lo] + (rec.y - run.phys_begin)), (int)total, rec.w & kGraphMask);
          es = total <= kTailShort;
          el = !es;
        }
      }
      if (c.graphs != 1 && (es || el)) c.mate[r.x] = c.C[r.x] - c.gbase[r.w];  // (cur below)
      place_rows(es, el, r, TA, k0, kc, sm);
    }
  }
  unsigned g = 1;
  const int cnt_s = sm.cnt_s, cnt_l = sm.cnt_l;
  if (!exchange(tc, tc->seg[g & 1], k0, kc, nb, g, false, limit, tot, sm)) return;
  if (csr && ld_u32(&tot->err)) return;  // (the same word everywhere: nothing is added before the next exchange)
  const int nhub = csr ? min((int)ld_u32(&tc->hubs), kTailHubs) : 0;
  if (nhub > 0) {  // every workgroup a slice of each, then, behind an exchange, the best of the slices
    const unsigned long long Sd = cand_seed(c.gseed[0], c.renew, 1);
    Key* part = reinterpret_cast<Key*>(a.ecol[0]);  // (the buffer that phase 2 writes: more than kHubRow entries)
    for (int h = 0; h < nhub; ++h) {
      const int v = tc->hub[h];
      const int e0 = (int)a.csr_rp[v];
      const long long len = a.csr_rp[v + 1] - e0;
      const int s0 = (int)(len * b / nb), s1 = (int)(len * (b + 1) / nb);
      const Key kb = best_of_row(make_int4(v, e0 + s0, s1 - s0, 0), kStep * wv, kStep * kTW, cur_col, cur_w, c.n, Sd);
      if (lane == 0) sm.hub[wv] = kb;
      __syncthreads();
      if (wv == 0) {
        const Key best = wave_max_key(lane < kTW ? sm.hub[lane] : key_ident());
        if (lane == 0) part[h * kTailMaxBlocks + b] = best;
      }
      __syncthreads();
    }
    if (tid == 0) {
      sm.cnt_s = cnt_s;
      sm.cnt_l = cnt_l;
    }
    ++g;
    if (!exchange(tc, tc->seg[g & 1], k0, kc, nb, g, false, limit, tot, sm)) return;
    for (int h = wv; h < nhub; h += kTW) {  // (every workgroup stores the same)
      const Key* p = part + h * kTailMaxBlocks;
      const Key x0 = lane < nb ? p[lane] : key_ident(), x1 = lane + 64 < nb ? p[lane + 64] : key_ident();
      const Key best = wave_max_key(key_max(x0, x1));
      if (lane == 0) c.C[tc->hub[h]] = best.u;
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
  }
  // ---- phases c, c + 1, ...
  // Candidates, as ids of their graph: one phase's in C, the next one's in
  // mate, which a vertex keeps until its row ends.
  const int* cur = c.graphs == 1 ? c.C : c.mate;
  int* nxt = c.graphs == 1 ? c.mate : c.C;
  const int4* rows = TA;
  int4* out = TB;
  int nseg = nb;  // segments of the current list
  bool solo = false, stall = false;
  int t = c0;
  long long L = csr ? a.nnz : ctl.L, V = 0, prevL = 0, prevV = 0;
  int last_nonempty = 0;
  unsigned long long matched_total = 0;
  if (b == 0 && tid == 0) {
    last_nonempty = tot->last_nonempty;
    matched_total = tot->matched;
  }
  int lo = 0, hi = 0, S = 0, Lg = 0, nwaves = kTW;
  const int gw = b * kTW + wv;
  for (;;) {
    S = sm.pre_s[nseg];
    Lg = sm.pre_l[nseg];
    V = (long long)S + Lg - (long long)(sm.mv >> 32);
    if (t > c0) {
      const unsigned mv = (unsigned)sm.mv;
      L = sm.kept;
      if (b == 0 && tid == 0) {  // the record of phase t - 1
        if (t - 1 >= 1 && t - 1 <= a.log_cap) {
          LogRec rec;
          rec.live_entries = prevL;
          rec.live_rows = prevV;
          rec.matched_edges = mv / 2;
          rec.matched_entries = sm.md;
          a.log[t - 2] = rec;
        }
        last_nonempty = t - 1;
        matched_total += mv;
      }
      stall = mv == 0u;  // nothing matched although edges were live: the input is not symmetric
      if (stall && b == 0 && tid == 0) atomicOr(&tot->err, (unsigned)kErrStall);
    }
    const bool done = stall || L == 0 || V == 0;
    if (!done && !solo && L <= kTailSolo) {
      solo = true;
      if (b != 0) return;  // workgroup 0 finishes alone
    }
    const int nbe = solo ? 1 : nb;
    // this workgroup's short rows [lo, hi); long row j goes to wave j % (nbe * kTW)
    lo = (int)((long long)S * b / nbe);
    hi = (int)((long long)S * (b + 1) / nbe);
    nwaves = nbe * kTW;
    if (done) break;
    const int q = Lg / nwaves, rmd = Lg % nwaves;
    const int longs_mine = kTW * q + min(max(rmd - b * kTW, 0), kTW);
    const int longs_before = b * kTW * q + min(rmd, b * kTW);
    const int obase = lo + longs_before, ocap = (hi - lo) + longs_mine;
    const bool in_mate = cur == c.mate;
    long long kept_b = 0, md_b = 0;
    unsigned long long mv_b = 0;
    int* ncol = a.ecol[ni];
    float* nw = unw ? nullptr : a.ew[ni];
    // What a row's phase leaves behind: its partner, its next candidate, or
    // nothing: mate is then -1 again. Where mate holds the candidates of this
    // phase the others still read it, so the row stays for one more phase, closed
    // (length 0).
    auto close = [&](int4& r, int kept, int cv, int u, bool& es, bool& el) {
      if (kept < 0) {
        if (!in_mate) c.mate[r.x] = cv;
        md_b += r.z;
        ++mv_b;
      } else if (kept > 0) {
        nxt[r.x] = u;
        kept_b += kept;
        es = kept <= kTailShort;
        el = !es;
        r.z = kept;
      } else if (in_mate) {
        mv_b += 1ull << 32;
        es = true;
        r.z = 0;
      } else {
        c.mate[r.x] = -1;
      }
    };
    for (int i0 = lo + (tid & ~63); i0 < hi; i0 += kTailBlock) {
      const int i = i0 + lane;
      int4 r = make_int4(0, 0, 0, 0);
      bool es = false, el = false;
      if (i < hi) {
        r = short_row(sm, nseg, rows, i);
        if (r.z == 0) {
          c.mate[r.x] = -1;
        } else {
          if (c.gphase) atomicMax(&c.gphase[r.w], t);
          int base;
          unsigned long long Sd;
          graph_of(c, r.w, base, Sd);
          Sd = cand_seed(Sd, c.renew, t + 1);  // the candidates of phase t + 1
          Best best = best_ident();
          int cv;
          const int kept = row_lane(c, r, base, (unsigned)(r.x - base), Sd, cur, cur_col, cur_w, ncol, nw, cv, best);
          close(r, kept, cv, best.u, es, el);
        }
      }
      place_rows(es, el, r, out, obase, ocap, sm);
    }
    for (int j = gw; j < Lg; j += nwaves) {  // long rows, a wave each
      int4 r = long_row(sm, nseg, rows, j);
      const int v = r.x, off = r.y, len = r.z;
      if (c.gphase && lane == 0) atomicMax(&c.gphase[r.w], t);
      int base;
      unsigned long long Sd;
      graph_of(c, r.w, base, Sd);
      Sd = cand_seed(Sd, c.renew, t + 1);  // the candidates of phase t + 1
      const unsigned vloc = (unsigned)(v - base);
      const int cv = cur[v];
      Best best = best_ident();
      int kept = back(c, cur, base, cv) == (int)vloc ? -1 : 0;
      const unsigned long long lt = lanemask_lt();
      for (int e0 = 0; kept >= 0 && e0 < len; e0 += 64 * kLongStep) {
        int u[kLongStep], x[kLongStep];
        float w[kLongStep];
        bool ok[kLongStep];
#pragma unroll
        for (int h = 0; h < kLongStep; ++h) {
          const int e = e0 + 64 * h + lane;
          ok[h] = e < len;
          u[h] = ok[h] ? cur_col[off + e] : -1;
          w[h] = (ok[h] && !unw) ? cur_w[off + e] : 1.0f;
          ok[h] = ok[h] && u[h] >= 0 && (unsigned)(base + u[h]) < (unsigned)c.n;
        }
#pragma unroll
        for (int h = 0; h < kLongStep; ++h) x[h] = ok[h] ? cur[base + u[h]] : -1;
#pragma unroll
        for (int h = 0; h < kLongStep; ++h) x[h] = back(c, cur, base, x[h]);
#pragma unroll
        for (int h = 0; h < kLongStep; ++h) {
          const bool keep = ok[h] && x[h] != u[h];
          const unsigned long long bal = __ballot(keep);
          if (keep) {
            const int at = off + kept + (int)__popcll(bal & lt);
            ncol[at] = u[h];
            if (!unw) nw[at] = w[h];
            best_update(best, ord_weight_bits(__float_as_uint(w[h])), u[h], vloc, Sd);
          }
          kept += (int)__popcll(bal);
        }
      }
      const Key kb = wave_max_key(best_key(best, vloc, Sd));
      bool es = false, el = false;
      if (lane == 0) close(r, kept, cv, kb.u, es, el);
      place_rows(es, el, r, out, obase, ocap, sm);
    }
    kept_b = wave_incl_sum<long long>(kept_b);
    md_b = wave_incl_sum<long long>(md_b);
    mv_b = (unsigned long long)wave_incl_sum<long long>((long long)mv_b);
    if (lane == 63) {
      atomicAdd(reinterpret_cast<unsigned long long*>(&sm.kept_b), (unsigned long long)kept_b);
      atomicAdd(reinterpret_cast<unsigned long long*>(&sm.md_b), (unsigned long long)md_b);
      atomicAdd(&sm.mv_b, mv_b);
    }
    ++g;
    if (!exchange(tc, tc->seg[g & 1], obase, ocap, nb, g, solo, limit, tot, sm)) return;
    // next live set
    prevL = L;
    prevV = V;
    nseg = nbe;
    const int4* tmp = rows;
    rows = out;
    out = const_cast<int4*>(tmp);
    cur_col = ncol;
    cur_w = nw;
    ni ^= 1;
    int* held = const_cast<int*>(cur);
    cur = nxt;
    nxt = held;
    ++t;
  }
  // rows that were closed in the last phase, or all of them after a stall
  for (int i = lo + tid; i < hi; i += kTailBlock) {
    const int4 r = short_row(sm, nseg, rows, i);
    if (stall || r.z == 0) c.mate[r.x] = -1;
  }
  if (stall && lane == 0)
    for (int j = gw; j < Lg; j += nwaves) c.mate[long_row(sm, nseg, rows, j).x] = -1;
  if (b == 0 && tid == 0) {
    tot->last_nonempty = last_nonempty;
    tot->matched = matched_total;
    tot->t = t;
    PhaseMirror m;
    m.L = L;
    m.matched = matched_total;
    m.pieces = 0;
    m.t = t;
    m.gen = a.gen;
    m.err = ld_u32(&tot->err);
    m.last_nonempty = last_nonempty;
    m.pad = c0;  // the live set the tail started from
    m.ticks = 0ull;
    m.tag = 0ull;
    PhaseMirror* slot = a.final_rec;
    *(volatile unsigned long long*)&slot->tag = 0ull;
    __threadfence_system();
    *slot = m;
    __threadfence_system();
    *(volatile unsigned long long*)&slot->tag = mirror_tag(a.gen, t);
  }
}

hipError_t launch_tail(const TailArgs& a, int grid, hipStream_t s, hipEvent_t* ev) {
  if (grid < 1 || grid > kTailMaxBlocks) return hipErrorInvalidValue;
  if (ev)
    hipExtLaunchKernelGGL(k_tail, dim3(grid), dim3(kTailBlock), 0, s, ev[0], ev[1], 0, a);
  else
    hipLaunchKernelGGL(k_tail, dim3(grid), dim3(kTailBlock), 0, s, a);
  return hipGetLastError();
}

int tail_blocks_per_cu() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_tail, kTailBlock, 0) != hipSuccess || nb < 1) nb = 1;
  return nb;
}

}  // namespace lm
