// Contraction of a graph by a matching (the coarsening step of multilevel
// partitioning, which contracts maximal matchings: Section 1 of the paper;
// its Section 3.1 runs local max on graph-contraction instances), gfx950.
//
// Result (lm_contract in lm.h): every matched pair {a, b}, a < b, and every
// free vertex a becomes one coarse vertex; coarse ids follow the smaller
// fine id (cmap); coarse row c lists each coarse neighbour once, in the
// order in which its first fine entry appears when a's row and then b's row
// are read; the weight of a coarse edge is the fp32 sum of the fine edges it
// merges (at most four in a simple graph) added in increasing order of the
// fine edge (min end, max end), the same order from both sides.
//
// Work: (1) a scan over the fine vertices numbers the pairs (cmap) and cuts the
// vertices into ranges of equal cost. (2) Coarse rows by their bound deg(a) +
// deg(b): up to kWS entries, several rows at once in a wave's tile; up to kCS,
// a wave each; longer ones, a workgroup each or several (3). All find the
// entries of one coarse neighbour in a hash set in LDS (rows of more than kLTable
// entries in device memory); the first of them in row order keeps it with the sum,
// and the kept entries are written compacted at the start of their fine row part
// (longer rows: in place, the others marked as dropped). (4) A scan over the coarse rows gives their offsets and
// the kept entries are copied out in order. The fine graph's entries are read
// once; cmap is gathered once per entry, which is what bounds the skewed
// graphs (R-MAT scale 24: about 100 G gathers a second).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstring>
#include <mutex>

#include "lm.h"
#include "lm_device.h"
#include "lm_internal.h"
#include "lm_runtime.h"

namespace lm {

namespace {

constexpr int kCV = 16;                 // fine vertices per lane in the numbering scans
constexpr int kCBlockV = kBlock * kCV;  // fine vertices per scan block
constexpr int kCT = 1024;               // entries per workgroup a range is worth at least (twice this)
constexpr int kCS = 512;                // largest coarse-row bound one wave merges
constexpr int kCMaxDup = 4;             // fine edges one coarse edge merges at most in a simple graph
constexpr int kCCost = 4;               // cost of a fine vertex when ranges are split (entries cost 1)
constexpr int kCTopThreads = 1024;
constexpr int kLB = 512;      // average entries of a long row's bucket
constexpr int kLBCap = 1024;  // slots of a bucket's table in LDS (more neighbours: the table path)
constexpr int kLSmall = 4;    // buckets of a long row that a workgroup of kBlock lanes merges
constexpr int kLPart = 8;     // buckets a workgroup of kLBig lanes merges at once
constexpr int kLBig = 1024;
constexpr int kLC = 8192;     // entries of a long row per chunk of the mapping and the output
// A row of more entries than this is merged through a table in device memory: its
// parts would each read all of it, 4 bytes an entry and part, which grows with the
// square of its length. A star of 600 K leaves 423 us (parts) / 339 (table), of 3 M
// 1936 / 1046, of 30 M 100 ms / 9.4.
constexpr int kLTable = 1 << 19;
constexpr int kLDrop = 512;   // chunks of a row whose dropped entries a part counts in LDS

constexpr unsigned kCErrMate = 1u;    // mate is not an involution with -1 for free vertices
constexpr unsigned kCErrRowPtr = 2u;  // row_ptr is not a valid offset array
constexpr unsigned kCErrCol = 4u;     // a neighbour id outside [0, n)
constexpr unsigned kCErrDup = 8u;     // more than four fine edges in one coarse edge: duplicate entries

struct CTot {
  unsigned err;
  unsigned pad;
  long long nc;            // coarse vertices
  long long nnz_c;         // coarse entries
  long long nlong;         // long rows
  long long long_entries;  // the sum of their bounds
  long long tab_entries;   // the same of those merged through device-memory tables
  long long long_slots;    // hash slots these tables take
  long long long_items;    // of the others, low word: rows of at most kLSmall buckets; high word: parts of kLPart buckets
  long long long_chunks;   // row-aligned chunks of kLC entries; from bit 40 on the rows merged through tables
  unsigned overflow;       // a bucket outgrew LDS: the long rows take the table path
  unsigned pad2;
};

struct LongRow {
  int a, b, c, dega;
  int ub;     // deg(a) + deg(b)
  int tbits;  // table of 2^tbits slots
  int nb;     // buckets of the row (about kLB entries each)
  int np;     // parts of kLPart buckets; 0: at most kLSmall buckets; -1: merged through a table
  long long eoff;  // first flat index of the row's entries among those of the rows with a table
  long long toff;  // first slot of its table
  int soff, boff;  // its place among the rows of at most kLSmall buckets; its first part
  long long coff;  // first chunk of the row (kLC entries each)
};

struct CArgs {
  long long n, nnz;
  const long long* rp;
  const int* col;
  const float* w;  // nullptr: every edge weighs 1
  const int* mate;
  const long long* vw;  // nullptr: every vertex weighs 1
  int* cmap;
  int* crep;  // coarse vertex -> its smaller fine vertex
  int* cnt;   // fine vertex -> coarse entries kept from its row part
  long long* cvw;  // nullptr: not wanted
  long long* bsum;
  int* vstart;         // first vertex of each range of the kernels that walk vertices (nullptr: searched for)
  long long per_wg;    // cost units of a range
  int ranges;
  CTot* tot;
  // The merged entries. Rows of bound <= kCS: the kept ones compacted at the
  // start of their fine row part. Long rows: at their own fine entries, -1
  // where dropped. dmap: the coarse neighbour, with kMerged if aux holds the
  // summed weight; without it the weight is the fine entry's own (1 for an
  // unweighted graph), which a compacted entry of a weighted graph has in aux.
  // (While a long row is merged, aux links the fine edges of one coarse edge.)
  int* dmap;
  float* aux;
  int* next;  // per flat entry of the rows with a table: the previous one of its slot's list
  LongRow* lrows;
  long long lrow_cap;
  long long table_from;  // long rows of more entries are merged through tables
  int2* table;  // (key, list head: a flat entry) per slot of the tables
  int* srow;   // long row of each row of at most kLSmall buckets
  int* prow;   // long row of each part
  int* crow;   // long row of each chunk
  int* ccnt;   // kept entries of each chunk
  long long* crp;
  int* ccol;
  float* cw;
  int dup_limit;  // fine edges one coarse edge may merge (4; 1 for the duplicate check)
  int identity;   // every vertex free, cmap the identity (the duplicate check of LM_CHECK_GRAPH)
};

constexpr int kMerged = (int)0x80000000u;  // (coarse ids are below 2^31 - 1, so -1 stays apart)

__device__ __forceinline__ unsigned long long tbl_hash(int d, int bits) {
  return (unsigned long long)(((unsigned)d * 0x9E3779B1u) >> (32 - bits));
}

// Exclusive prefix sum over a workgroup of kCTopThreads lanes.
__device__ __forceinline__ long long top_excl_sum(long long x, long long* sm, long long& total) {
  const long long incl = wave_incl_sum<long long>(x);
  if (lane_id() == 63) sm[wave_id()] = incl;
  __syncthreads();
  long long pre = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kCTopThreads / 64; ++i) {
    const long long v = sm[i];
    pre += (i < wave_id()) ? v : 0ll;
    tot += v;
  }
  __syncthreads();
  total = tot;
  return pre + incl - x;
}

// (1a) Checks mate and row_ptr and counts the pairs' smaller ends per block
// (vertex base + i * kBlock + lane: coalesced). Finds the ranges' starts: the
// first vertex whose cost prefix reaches r per_wg follows the one whose row
// crosses it.
__global__ __launch_bounds__(kBlock) void k_c_count(CArgs a) {
  __shared__ long long sm[kWaves];
  const long long base = (long long)blockIdx.x * kCBlockV;
  unsigned err = 0;
  long long reps = 0;
  constexpr int kI = kCV / 2;  // vertices a lane's loads are in flight for (all of them: 152 registers)
#pragma unroll 1
  for (int i0 = 0; i0 < kCV; i0 += kI) {
    int m[kI], mm[kI];
    long long r0[kI], r1[kI];
    const long long v0 = base + (long long)i0 * kBlock + threadIdx.x;
#pragma unroll
    for (int i = 0; i < kI; ++i) {
      const long long v = v0 + (long long)i * kBlock;
      m[i] = v < a.n && !a.identity ? a.mate[v] : -1;
      r0[i] = v < a.n ? a.rp[v] : 0;
      r1[i] = v < a.n ? a.rp[v + 1] : 0;
    }
#pragma unroll
    for (int i = 0; i < kI; ++i) mm[i] = m[i] >= 0 && m[i] < a.n ? a.mate[m[i]] : -1;
#pragma unroll
    for (int i = 0; i < kI; ++i) {
      const long long v = v0 + (long long)i * kBlock;
      if (v >= a.n) break;
      if (m[i] != -1 && (m[i] < 0 || m[i] >= a.n || m[i] == v || mm[i] != (int)v)) err |= kCErrMate;
      reps += (m[i] == -1 || v < m[i]) ? 1 : 0;
      if (r1[i] < r0[i] || (v == 0 && r0[i] != 0) || (v == a.n - 1 && r1[i] != a.nnz)) err |= kCErrRowPtr;
      if (a.vstart && r0[i] >= 0 && r1[i] >= r0[i] && r1[i] <= a.nnz) {
        const long long c0 = r0[i] + (long long)kCCost * v, c1 = r1[i] + (long long)kCCost * (v + 1);
        for (long long r = c0 / a.per_wg + 1; r * a.per_wg <= c1 && r <= a.ranges; ++r) a.vstart[r] = (int)(v + 1);
        if (v == 0) a.vstart[0] = 0;
      }
    }
  }
  long long total;
  (void)block_excl_sum<long long>(reps, sm, total);
  if (threadIdx.x == 0) a.bsum[blockIdx.x] = total;
  if (err) atomicOr(&a.tot->err, err);
}

// (1b, 4b) Exclusive scan of m block sums in place, one workgroup; the total
// goes to *total.
__global__ __launch_bounds__(kCTopThreads) void k_c_scan_top(long long* v, long long m, long long* total) {
  __shared__ long long sm[kCTopThreads / 64];
  long long carry = 0;
  for (long long base = 0; base < m; base += kCTopThreads) {
    const long long i = base + threadIdx.x;
    const long long x = i < m ? v[i] : 0ll;
    long long t;
    const long long e = top_excl_sum(x, sm, t);
    if (i < m) v[i] = carry + e;
    carry += t;
  }
  if (threadIdx.x == 0) *total = carry;
}

// Exclusive prefix, in index order, of the kCBlockV values a block staged in
// val[] (value of index base + i * kBlock + lane at val[i * kBlock + lane]):
// every lane sums kCV consecutive values, the lanes are scanned, and val[]
// receives the prefixes. Returns the block total.
__device__ __forceinline__ long long block_stage_scan(long long* val, long long start, long long* sm) {
  long long s = 0;
  for (int j = 0; j < kCV; ++j) s += val[threadIdx.x * kCV + j];
  long long total;
  long long run = start + block_excl_sum<long long>(s, sm, total);  // ends after a barrier
  for (int j = 0; j < kCV; ++j) {
    const long long x = val[threadIdx.x * kCV + j];
    val[threadIdx.x * kCV + j] = run;
    run += x;
  }
  __syncthreads();
  return total;
}

// (1c) Numbers the coarse vertices, writes cmap, the coarse vertex weights,
// and clears the per-row-part counts.
__global__ __launch_bounds__(kBlock) void k_c_map(CArgs a) {
  __shared__ long long val[kCBlockV];
  __shared__ long long sm[kWaves];
  if (a.tot->err) return;
  const long long base = (long long)blockIdx.x * kCBlockV;
  int mm[kCV];
#pragma unroll
  for (int i = 0; i < kCV; ++i) {
    const long long v = base + (long long)i * kBlock + threadIdx.x;
    mm[i] = v < a.n ? a.mate[v] : -2;
  }
#pragma unroll
  for (int i = 0; i < kCV; ++i) {
    const long long v = base + (long long)i * kBlock + threadIdx.x;
    if (v < a.n) a.cnt[v] = 0;
    val[i * kBlock + threadIdx.x] = v < a.n && (mm[i] == -1 || v < mm[i]) ? 1 : 0;
  }
  __syncthreads();
  (void)block_stage_scan(val, a.bsum[blockIdx.x], sm);
#pragma unroll
  for (int i = 0; i < kCV; ++i) {
    const long long v = base + (long long)i * kBlock + threadIdx.x;
    const int m = mm[i];
    if (v >= a.n || !(m == -1 || v < m)) continue;
    const int c = (int)val[i * kBlock + threadIdx.x];
    a.cmap[v] = c;
    a.crep[c] = (int)v;
    if (m >= 0) a.cmap[m] = c;
    if (a.cvw) a.cvw[c] = (a.vw ? a.vw[v] : 1ll) + (m >= 0 ? (a.vw ? a.vw[m] : 1ll) : 0ll);
  }
}

// A fine vertex as the head of a coarse row.
struct RowHead {
  bool rep, lng;
  int m, c, dega, ub;
  long long ka, kb;
};
__device__ __forceinline__ RowHead row_head(const CArgs& a, long long v) {
  RowHead h;
  h.m = a.identity ? -1 : a.mate[v];
  h.rep = (h.m == -1 || v < h.m);
  h.c = 0;
  h.dega = h.ub = 0;
  h.ka = h.kb = 0;
  h.lng = false;
  if (h.rep) {
    h.c = a.identity ? (int)v : a.cmap[v];
    h.ka = a.rp[v];
    h.dega = (int)(a.rp[v + 1] - h.ka);
    h.ub = h.dega;
    if (h.m >= 0) {
      h.kb = a.rp[h.m];
      h.ub += (int)(a.rp[h.m + 1] - h.kb);
    }
    h.lng = h.ub > kCS;
  }
  return h;
}

// The range of workgroup b: kCNear neighbouring ranges go to one die (workgroups are
// dealt to the eight dies in turn), which then writes most lines that hold parts of
// rows of two of them (a grid of 16 M vertices paired down its columns 2302 us
// without, 1667; ranges of a workgroup each, as many as are resident, 1771).
constexpr int kCNear = 8;
__device__ __forceinline__ int range_of(int b, int ranges) {
  if (b >= ranges / (8 * kCNear) * (8 * kCNear)) return b;
  const int j = b >> 3;
  return ((j / kCNear) * 8 + (b & 7)) * kCNear + j % kCNear;
}

// The fine vertices [vb, ve) of workgroup blockIdx.x: ranges split by
// entries plus kCCost per vertex (starts past the last crossing: none left).
__device__ __forceinline__ void wg_vertices(const CArgs& a, long long& vb, long long& ve, int* lb) {
  const long long C = a.nnz + (long long)kCCost * a.n;
  const int r = range_of((int)blockIdx.x, a.ranges);
  const long long c0 = (long long)r * a.per_wg;
  const long long c1 = c0 + a.per_wg;
  if (a.vstart) {
    vb = c0 > C ? a.n : a.vstart[r];
    ve = c1 >= C ? a.n : a.vstart[r + 1];
    return;
  }
  vb = c0 >= C ? a.n
               : block_lower_bound(0, a.n + 1, [&](long long v) { return a.rp[v] + (long long)kCCost * v >= c0; },
                                   lb);
  ve = c1 >= C ? a.n
               : block_lower_bound(0, a.n + 1, [&](long long v) { return a.rp[v] + (long long)kCCost * v >= c1; },
                                   lb);
}

// Vertices a wave takes at a time of a range of nv: at least `turns` turns a wave,
// of equal size, so that the range's rows spread over its waves, however few and
// long.
__device__ __forceinline__ int wave_rows(long long nv, int turns) {
  const long long t = max((long long)turns, (nv + 64 * kWaves - 1) / (64 * kWaves));
  return (int)max(4ll, (nv + kWaves * t - 1) / (kWaves * t));
}

// Last row r of the chunk with st[r] <= pos (rows with no tile entries share
// their start with the next row, so r is the row that holds pos).
__device__ __forceinline__ int row_of(const int* st, int pos) {
  int lo = 0, hi = kBlock;  // st[lo] <= pos; answer in [lo, hi)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (st[mid] <= pos)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}
// Sums the n <= 4 fine edges of one group in increasing (min end, max end):
// slots n..3 hold ord = ~0 and sort last; a fixed sorting network keeps every
// index static (no dynamic register indexing).
static_assert(kCMaxDup == 4, "the sorting network below is for four slots");
__device__ __forceinline__ void cswap(unsigned long long& oa, float& wa, unsigned long long& ob, float& wb) {
  if (ob < oa) {
    const unsigned long long t = oa;
    oa = ob;
    ob = t;
    const float u = wa;
    wa = wb;
    wb = u;
  }
}
__device__ __forceinline__ float group_sum(unsigned long long* ord, float* wv, int n) {
  cswap(ord[0], wv[0], ord[1], wv[1]);
  cswap(ord[2], wv[2], ord[3], wv[3]);
  cswap(ord[0], wv[0], ord[2], wv[2]);
  cswap(ord[1], wv[1], ord[3], wv[3]);
  cswap(ord[1], wv[1], ord[2], wv[2]);
  float sum = wv[0];
  if (n > 1) sum += wv[1];
  if (n > 2) sum += wv[2];
  if (n > 3) sum += wv[3];
  return sum;
}

__device__ __forceinline__ unsigned long long edge_order(int s, int x) {
  return ((unsigned long long)(unsigned)min(s, x) << 32) | (unsigned)max(s, x);
}

constexpr int kWT = 256;           // wave tile capacity in entries
constexpr int kWS = 64;            // largest coarse-row bound one wave merges alone
constexpr int kWStep = kWT - kWS;  // wave tiles take the rows that start in a window of this many entries
constexpr int kWTI = kWT / 64;     // tile entries per lane

struct WaveSmem {
  int skey[2 * kWT];   // coarse neighbour of the slot, -1 if free
  int shead[2 * kWT];  // last tile position inserted into the slot's list
  short enext[kWT];
  short eslot[kWT];
  int st[65];  // wave-local start of each lane's row; st[64] = the wave's total
  int ra[64], rb[64], rc[64], rdega[64], rut[64];
  int rrk[64][2];  // kept entries of the tile before the row's a part and b part
  int rka[64], rkb[64];  // the row parts' first entries (nnz < 2^31: five workgroups fit a CU)
};

// Orders the wave's LDS accesses across lanes (a wave's LDS operations are
// performed in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Start of the first of the wave's rows whose start is at least t (the
// wave's total if none).
__device__ __forceinline__ int wstart_at(const int* st, int t) {
  if (st[0] >= t) return st[0];
  int lo = 0, hi = 64;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (st[mid] >= t)
      hi = mid;
    else
      lo = mid;
  }
  return st[hi];
}
__device__ __forceinline__ int wrow_of(const int* st, int pos) {
  int lo = 0, hi = 64;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (st[mid] <= pos)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// (2a) The coarse rows with bound <= kWS, one wave at a time with no
// workgroup barrier: each wave takes 64 fine vertices of every chunk of its
// workgroup's range, lays their rows out back to back and groups them in
// wave tiles of at most kWT entries (equal coarse neighbours meet in a slot of
// the wave's LDS table); ranks in row order come from the tile's ballots.
__global__ __launch_bounds__(kBlock) void k_c_group_wave(CArgs a) {
  __shared__ WaveSmem wsm[kWaves];
  __shared__ int lb[1];
  if (a.tot->err & (kCErrMate | kCErrRowPtr)) return;
  long long vb, ve;
  wg_vertices(a, vb, ve, lb);
  WaveSmem& sm = wsm[wave_id()];
  const int l = lane_id();
  for (int i = l; i < 2 * kWT; i += 64) {
    sm.skey[i] = -1;
    sm.shead[i] = -1;
  }
  wave_sync();
  unsigned err = 0;
  const int step = wave_rows(ve - vb, 2);
  for (long long cb = vb + (long long)wave_id() * step; cb < ve; cb += kWaves * step) {
    const long long v = cb + l;
    RowHead h;
    h.rep = false;
    h.lng = false;
    h.m = -1;
    h.c = h.dega = h.ub = 0;
    h.ka = h.kb = 0;
    if (l < step && v < ve) h = row_head(a, v);
    const int ut = (h.rep && !h.lng && h.ub <= kWS) ? h.ub : 0;
    const int incl = wave_incl_sum<int>(ut);
    const int U = __shfl(incl, 63);
    sm.st[l] = incl - ut;
    if (l == 63) sm.st[64] = U;
    sm.ra[l] = (int)v;
    sm.rb[l] = h.m;
    sm.rc[l] = h.c;
    sm.rdega[l] = h.dega;
    sm.rut[l] = ut;
    sm.rka[l] = (int)h.ka;
    sm.rkb[l] = (int)h.kb;
    wave_sync();
    const int ntile = (U + kWStep - 1) / kWStep;
    for (int j = 0; j < ntile; ++j) {
      const int lo = wstart_at(sm.st, j * kWStep);
      const int hi = wstart_at(sm.st, (j + 1) * kWStep);
      const int len = hi - lo;
      if (len <= 0) continue;
      int Dr[kWTI], xr[kWTI], rr[kWTI];
      float wr[kWTI];
      long long kr[kWTI];
      // 1: load every entry of the lane, then map them all, then insert
#pragma unroll
      for (int i = 0; i < kWTI; ++i) {
        const int q = i * 64 + l;
        rr[i] = 0;
        kr[i] = -1;
        Dr[i] = -1;
        xr[i] = 0;
        wr[i] = 0.f;
        if (q < len) {
          const int pos = lo + q;
          const int r = wrow_of(sm.st, pos);
          const int off = pos - sm.st[r];
          const bool side = off >= sm.rdega[r];
          rr[i] = r;
          kr[i] = side ? sm.rkb[r] + (off - sm.rdega[r]) : sm.rka[r] + off;
        }
      }
#pragma unroll
      for (int i = 0; i < kWTI; ++i) {
        if (kr[i] < 0) continue;
        xr[i] = a.col[kr[i]];
        wr[i] = a.w ? a.w[kr[i]] : 1.0f;
      }
#pragma unroll
      for (int i = 0; i < kWTI; ++i) {
        if (kr[i] < 0) continue;
        if ((unsigned)xr[i] >= (unsigned)a.n)
          err |= kCErrCol;
        else
          Dr[i] = a.identity ? xr[i] : a.cmap[xr[i]];
      }
#pragma unroll
      for (int i = 0; i < kWTI; ++i) {
        const int q = i * 64 + l;
        const int r = rr[i];
        if (kr[i] < 0) continue;
        if (Dr[i] == sm.rc[r]) Dr[i] = -1;
        const int D = Dr[i];
        if (D >= 0) {
          const unsigned sb = 2u * (unsigned)(sm.st[r] - lo);
          const unsigned range = 2u * (unsigned)sm.rut[r];
          unsigned hh = (unsigned)(((unsigned long long)((unsigned)D * 0x9E3779B1u) * range) >> 32);
          for (;;) {
            const int old = atomicCAS(&sm.skey[sb + hh], -1, D);
            if (old == -1 || old == D) break;
            hh = hh + 1 == range ? 0u : hh + 1;
          }
          sm.eslot[q] = (short)(sb + hh);
          sm.enext[q] = (short)atomicExch(&sm.shead[sb + hh], q);
        }
      }
      wave_sync();
      // 2: the first entry of every group keeps it, with the group's sum
      bool keep[kWTI], merged[kWTI];
      float sumr[kWTI];
      unsigned long long bal[kWTI];
#pragma unroll
      for (int i = 0; i < kWTI; ++i) {
        const int q = i * 64 + l;
        keep[i] = false;
        merged[i] = false;
        sumr[i] = 0.f;
        if (q < len && Dr[i] >= 0) {
          int lst[kCMaxDup + 1];
          int nl = 0;
          int p = sm.shead[sm.eslot[q]];
          bool first = true;
#pragma unroll
          for (int t = 0; t <= kCMaxDup; ++t) {  // static indices: at most five nodes matter
            if (p >= 0) {
              lst[t] = p;
              nl = t + 1;
              first = first && p >= q;
              p = sm.enext[p];
            }
          }
          if (nl > a.dup_limit) err |= kCErrDup;
          if (first && nl <= a.dup_limit) {
            keep[i] = true;
            merged[i] = nl > 1;
            const int r = rr[i];
            if (nl == 1) {
              sumr[i] = wr[i];
            } else {
              unsigned long long ord[kCMaxDup];
              float wg[kCMaxDup];
#pragma unroll
              for (int t = 0; t < kCMaxDup; ++t) {
                ord[t] = ~0ull;
                wg[t] = 0.f;
                if (t >= nl) continue;
                const int pp = lst[t];
                const int off = lo + pp - sm.st[r];
                const bool side = off >= sm.rdega[r];
                const int s = side ? sm.rb[r] : sm.ra[r];
                int xp = xr[i];
                float wp = wr[i];
                if (pp != q) {
                  const long long kp = side ? sm.rkb[r] + (off - sm.rdega[r]) : sm.rka[r] + off;
                  xp = a.col[kp];
                  wp = a.w ? a.w[kp] : 1.0f;
                }
                ord[t] = edge_order(s, xp);
                wg[t] = wp;
              }
              sumr[i] = group_sum(ord, wg, nl);
            }
          }
        }
        bal[i] = __ballot(keep[i]);
      }
      // 3: kept entries before a tile position, from the ballots: every row's
      // lane finds its parts' starts, every kept entry its own rank
      int pre[kWTI];
      pre[0] = 0;
#pragma unroll
      for (int i = 1; i < kWTI; ++i) pre[i] = pre[i - 1] + (int)__popcll(bal[i - 1]);
      auto rank_at = [&](int pos) -> int {  // any tile position (row lanes only)
        const int ri = pos >> 6;
        int base = pre[kWTI - 1] + (int)__popcll(bal[kWTI - 1]);
        unsigned long long b = 0ull;
#pragma unroll
        for (int t = 0; t < kWTI; ++t)
          if (t == ri) {
            base = pre[t];
            b = bal[t];
          }
        return base + (int)__popcll(b & ((1ull << (pos & 63)) - 1ull));
      };
      const bool row_here = sm.rut[l] > 0 && sm.st[l] >= lo && sm.st[l] < hi;
      if (row_here) {
        const int s0 = sm.st[l] - lo;
        const int r0 = rank_at(s0), rb_ = rank_at(s0 + sm.rdega[l]);
        sm.rrk[l][0] = r0;
        sm.rrk[l][1] = rb_;
        if (a.cnt) {
          a.cnt[sm.ra[l]] = rb_ - r0;
          if (sm.rb[l] >= 0) a.cnt[sm.rb[l]] = rank_at(s0 + sm.rut[l]) - rb_;
        }
      }
      wave_sync();
      if (a.dmap) {
#pragma unroll
        for (int i = 0; i < kWTI; ++i) {
          const int q = i * 64 + l;
          if (q >= len || !keep[i]) continue;
          const int r = rr[i];
          const int off = lo + q - sm.st[r];
          const bool side = off >= sm.rdega[r];
          const int own = pre[i] + (int)__popcll(bal[i] & lanemask_lt());
          const int at = (side ? sm.rkb[r] : sm.rka[r]) + (own - sm.rrk[r][side ? 1 : 0]);
          const bool sum = a.w != nullptr || merged[i];
          a.dmap[at] = sum ? Dr[i] | kMerged : Dr[i];
          if (sum) a.aux[at] = sumr[i];
        }
      }
      for (int i = l; i < 2 * len; i += 64) {
        sm.skey[i] = -1;
        sm.shead[i] = -1;
      }
      wave_sync();
    }
    wave_sync();
  }
  if (err) atomicOr(&a.tot->err, err);
}

// A slot of an LDS set of coarse neighbours: the neighbour in the low word; in
// the high word the row position of its first entry in with kEnd, or, once
// more entries named it, the position of the last of them (positions link
// back to the one with kEnd). A group that was merged: the summed weight's
// bits, and the first position in row order.
constexpr unsigned long long kFree = ~0ull;
constexpr unsigned kEnd = 0x80000000u;
__device__ __forceinline__ unsigned long long set_slot(int D, unsigned pos) {
  return ((unsigned long long)pos << 32) | (unsigned)D;
}
__device__ __forceinline__ unsigned* slot_pos(unsigned long long* slot) { return reinterpret_cast<unsigned*>(slot) + 1; }

// The coarse edge whose fine edges are the row's entries at positions
// lst[0..nl): the sum of their weights in edge order, and the first position.
// Entry e < dega of the row is fine entry ka + e of vertex va, the others
// kb + (e - dega) of vb.
__device__ __forceinline__ float merge_group(const CArgs& a, const int* lst, int nl, int va, int vb, int dega, int ka,
                                             int kb, int& first) {
  unsigned long long ord[kCMaxDup];
  float wg[kCMaxDup];
  first = lst[0];
#pragma unroll
  for (int t = 0; t < kCMaxDup; ++t) {
    ord[t] = ~0ull;
    wg[t] = 0.f;
    if (t >= nl) continue;
    first = min(first, lst[t]);
    const bool side = lst[t] >= dega;
    const int k = side ? kb + (lst[t] - dega) : ka + lst[t];
    ord[t] = edge_order(side ? vb : va, a.col[k]);
    wg[t] = a.w ? a.w[k] : 1.0f;
  }
  return group_sum(ord, wg, nl);
}

constexpr int kMSlots = 2 * kCS;
constexpr int kMI = kCS / 64;  // entries per lane

struct MidSmem {
  unsigned long long tab[kMSlots];
  unsigned short next[kCS];     // link of a position, with 0x8000 at the end
  unsigned short grp[kCS / 2];  // slots with more than one entry
  int ngrp;
};

// (2b) Merges every medium coarse row (kWS < bound <= kCS), one wave a row: an
// entry enters its coarse neighbour into a set in LDS by one compare-and-swap,
// which also tells whether it is the first; only neighbours named more than
// once (few, in graphs with such rows) are linked, walked and summed. The
// kept entries are compacted at the start of each row part. Queues the long
// rows. What bounds it is the gather of cmap: eight of a lane's are in flight
// at once, and nothing waits on a workgroup barrier.
__global__ __launch_bounds__(kBlock) void k_c_group_mid(CArgs a) {
  __shared__ MidSmem wsm[kWaves];
  __shared__ int lb[1];
  if (a.tot->err & (kCErrMate | kCErrRowPtr)) return;
  long long vb, ve;
  wg_vertices(a, vb, ve, lb);
  MidSmem& sm = wsm[wave_id()];
  const int l = lane_id();
  for (int i = l; i < kMSlots; i += 64) sm.tab[i] = kFree;
  if (l == 0) sm.ngrp = 0;
  wave_sync();
  unsigned err = 0;
  const int step = wave_rows(ve - vb, 4);
  for (long long cb = vb + (long long)wave_id() * step; cb < ve; cb += kWaves * step) {
    const long long v = cb + l;
    RowHead h;
    h.rep = false;
    h.lng = false;
    h.m = -1;
    h.c = h.dega = h.ub = 0;
    h.ka = h.kb = 0;
    if (l < step && v < ve) h = row_head(a, v);
    const unsigned long long lng = __ballot(h.rep && h.lng);
    if (lng) {
      unsigned long long base = 0;
      if (l == 0) base = atomicAdd((unsigned long long*)&a.tot->nlong, (unsigned long long)__popcll(lng));
      base = (unsigned long long)__shfl((long long)base, 0);
      if (h.rep && h.lng) {
        const unsigned long long idx = base + (unsigned long long)__popcll(lng & lanemask_lt());
        if ((long long)idx < a.lrow_cap) {
          LongRow L;
          std::memset(&L, 0, sizeof(L));
          L.a = (int)v;
          L.b = h.m;
          L.c = h.c;
          L.dega = h.dega;
          L.ub = h.ub;
          a.lrows[idx] = L;
        }
      }
    }
    unsigned long long rows = __ballot(h.rep && !h.lng && h.ub > kWS);
    while (rows) {
      const int src = __ffsll((long long)rows) - 1;
      rows &= rows - 1;
      const int va = (int)(cb + src), vbm = __builtin_amdgcn_readlane(h.m, src);
      const int c = __builtin_amdgcn_readlane(h.c, src), dega = __builtin_amdgcn_readlane(h.dega, src);
      const int ub = __builtin_amdgcn_readlane(h.ub, src);
      const int ka = __builtin_amdgcn_readlane((int)h.ka, src), kb = __builtin_amdgcn_readlane((int)h.kb, src);
      int x[kMI], D[kMI], slot[kMI];
      // every entry's neighbour, then its coarse one
#pragma unroll
      for (int i = 0; i < kMI; ++i) {
        x[i] = -1;
        if (i * 64 < ub) {
          const int e = i * 64 + l;
          if (e < ub) x[i] = a.col[e < dega ? ka + e : kb + (e - dega)];
        }
      }
#pragma unroll
      for (int i = 0; i < kMI; ++i) {
        D[i] = -1;
        if (i * 64 < ub) {
          const int e = i * 64 + l;
          if (e < ub) {
            if ((unsigned)x[i] >= (unsigned)a.n)
              err |= kCErrCol;
            else
              D[i] = a.identity ? x[i] : a.cmap[x[i]];
          }
        }
      }
      const int shift = ub <= 256 ? 23 : 22;  // 512 or 1024 slots: at most half of them taken
      const unsigned mask = (1u << (32 - shift)) - 1u;
#pragma unroll
      for (int i = 0; i < kMI; ++i) {
        slot[i] = 0;
        if (D[i] == c) D[i] = -1;
        if (i * 64 < ub && D[i] >= 0) {
          const unsigned e = (unsigned)(i * 64 + l);
          unsigned hh = ((unsigned)D[i] * 0x9E3779B1u) >> shift;
          for (;;) {
            const unsigned long long old = atomicCAS(&sm.tab[hh], kFree, set_slot(D[i], e | kEnd));
            if (old == kFree) break;
            if ((int)(unsigned)old == D[i]) {
              const unsigned prev = atomicExch(slot_pos(&sm.tab[hh]), e);
              sm.next[e] = (unsigned short)((prev & 0x7fffu) | (prev >> 31 << 15));
              if (prev & kEnd) sm.grp[atomicAdd(&sm.ngrp, 1)] = (unsigned short)hh;
              break;
            }
            hh = (hh + 1u) & mask;
          }
          slot[i] = (int)hh;
        }
      }
      wave_sync();
      const int ng = __builtin_amdgcn_readfirstlane(sm.ngrp);
      for (int q = l; q < ng; q += 64) {
        const int hs = sm.grp[q];
        int lst[kCMaxDup];
        int nl = 0;
        unsigned p = (unsigned)(sm.tab[hs] >> 32);
#pragma unroll
        for (int t = 0; t < kCMaxDup; ++t) {  // static indices
          if (p != ~0u) {
            lst[t] = (int)(p & 0x7fffu);
            nl = t + 1;
            p = (p & 0x8000u) ? ~0u : sm.next[p & 0x7fffu];
          }
        }
        if (p != ~0u || nl > a.dup_limit) err |= kCErrDup;
        int first;
        const float sum = merge_group(a, lst, nl, va, vbm, dega, ka, kb, first);
        sm.tab[hs] = ((unsigned long long)(unsigned)first << 32) | __float_as_uint(sum);
      }
      wave_sync();
      // ranks in row order, and the kept entries
      int before = 0, acnt = 0;
#pragma unroll
      for (int i = 0; i < kMI; ++i) {
        if (i * 64 < ub) {
          const int e = i * 64 + l;
          bool keep = D[i] >= 0, sum = false;
          float wk = 1.0f;
          if (keep && ng) {
            const unsigned long long t = sm.tab[slot[i]];
            if (!((unsigned)(t >> 32) & kEnd)) {
              keep = (int)(t >> 32) == e;
              sum = keep;
              wk = __uint_as_float((unsigned)t);
            }
          }
          const unsigned long long bal = __ballot(keep);
          const int own = before + (int)__popcll(bal & lanemask_lt());
          // kept entries of a's part in this round
          const int split = dega - i * 64;
          acnt += split >= 64 ? (int)__popcll(bal) : split > 0 ? (int)__popcll(bal & ((1ull << split) - 1ull)) : 0;
          if (keep && a.dmap) {
            const int at = e < dega ? ka + own : kb + (own - acnt);
            if (a.w && !sum) wk = a.w[e < dega ? ka + e : kb + (e - dega)];
            sum = sum || a.w;
            a.dmap[at] = sum ? D[i] | kMerged : D[i];
            if (sum) a.aux[at] = wk;
          }
          before += (int)__popcll(bal);
        }
      }
      if (l == 0 && a.cnt) {
        a.cnt[va] = acnt;
        if (vbm >= 0) a.cnt[vbm] = before - acnt;
      }
      wave_sync();
#pragma unroll
      for (int i = 0; i < kMI; ++i)
        if (D[i] >= 0) sm.tab[slot[i]] = kFree;
      if (l == 0) sm.ngrp = 0;
      wave_sync();
    }
  }
  if (err) atomicOr(&a.tot->err, err);
}

// (4d) Copies the kept entries of every short coarse row from the starts of
// its two row parts to the output.
__global__ __launch_bounds__(kBlock) void k_c_copy(CArgs a) {
  __shared__ int pre[kBlock + 1];
  __shared__ int sca[kBlock];
  __shared__ long long ska[kBlock], skb[kBlock], sd0[kBlock];
  __shared__ int smi[kWaves];
  __shared__ int lb[1];
  if (a.tot->err) return;
  const int tid = threadIdx.x;
  long long vb, ve;
  wg_vertices(a, vb, ve, lb);
  for (long long cb = vb; cb < ve; cb += kBlock) {
    const long long v = cb + tid;
    int len = 0, ca = 0;
    long long ka = 0, kb = 0, d0 = 0;
    if (v < ve) {
      const RowHead h = row_head(a, v);
      if (h.rep && !h.lng) {
        ca = a.cnt[v];
        len = ca + (h.m >= 0 ? a.cnt[h.m] : 0);
        ka = h.ka;
        kb = h.kb;
        d0 = a.crp[h.c];
      }
    }
    int T;
    const int p = block_excl_sum<int>(len, smi, T);
    pre[tid] = p;
    if (tid == 0) pre[kBlock] = T;
    sca[tid] = ca;
    ska[tid] = ka;
    skb[tid] = kb;
    sd0[tid] = d0;
    __syncthreads();
    for (int q = tid; q < T; q += kBlock) {
      const int r = row_of(pre, q);
      const int off = q - pre[r];
      const long long src = off < sca[r] ? ska[r] + off : skb[r] + (off - sca[r]);
      const int t = a.dmap[src];
      a.ccol[sd0[r] + off] = t & ~kMerged;
      a.cw[sd0[r] + off] = t < 0 ? a.aux[src] : 1.0f;
    }
    __syncthreads();
  }
}

// (3a') Sizes of the long rows: entries (their bound) and table slots (the
// power of two at least twice the bound) of those merged through tables, whether
// one small workgroup merges the row, parts and chunks, and the offsets of each in
// row order. Workgroup
// g sums kLPRows rows (k_c_long_sums), one scan over the workgroup sums per
// quantity gives the totals (k_c_scan_top), and each workgroup writes its
// rows' offsets from its prefix (k_c_long_offs). The grid covers the row
// capacity; workgroups past the long rows counted write zero sums.
constexpr int kLP = 4;                 // long rows per lane in the prep kernels
constexpr int kLPRows = kBlock * kLP;  // long rows per workgroup
constexpr int kLQ = 5;                 // quantities
constexpr long long kLTabBit = 1ll << 40;

__device__ __forceinline__ void long_row_sizes(long long ub, long long table_from, int& bits, int& nb, int& np,
                                               long long v[kLQ]) {
  const bool tab = ub > table_from;
  const long long t = 2 * ub;
  bits = t <= 2 ? 1 : 64 - __clzll((unsigned long long)(t - 1));  // smallest bits >= 1 with 2^bits >= 2 ub
  nb = (int)((ub + kLB - 1) / kLB);
  np = tab ? -1 : nb <= kLSmall ? 0 : (nb + kLPart - 1) / kLPart;
  v[0] = tab ? ub : 0;
  v[1] = tab ? 1ll << bits : 0;
  v[2] = tab ? 0 : np == 0 ? 1 : (long long)np << 32;  // (each sum is below 2^31)
  v[3] = (ub + kLC - 1) / kLC + (tab ? kLTabBit : 0);
  v[4] = ub;
}

__global__ __launch_bounds__(kBlock) void k_c_long_sums(CArgs a, long long* lsum, long long nblk) {
  __shared__ long long sm[kWaves];
  const long long nl = a.tot->err ? 0 : (a.tot->nlong < a.lrow_cap ? a.tot->nlong : a.lrow_cap);
  long long su[kLQ] = {};
  const long long i0 = (long long)blockIdx.x * kLPRows + (long long)threadIdx.x * kLP;
#pragma unroll
  for (int j = 0; j < kLP; ++j) {
    if (i0 + j >= nl) continue;
    int bits, nb, np;
    long long v[kLQ];
    long_row_sizes(a.lrows[i0 + j].ub, a.table_from, bits, nb, np, v);
#pragma unroll
    for (int q = 0; q < kLQ; ++q) su[q] += v[q];
  }
#pragma unroll
  for (int q = 0; q < kLQ; ++q) {
    long long tot;
    (void)block_excl_sum<long long>(su[q], sm, tot);
    if (threadIdx.x == 0) lsum[q * nblk + blockIdx.x] = tot;
  }
}

// Exclusive scans of the kLQ arrays of workgroup sums, one workgroup each.
__global__ __launch_bounds__(kCTopThreads) void k_c_long_top(long long* lsum, long long nblk, CTot* tot) {
  __shared__ long long sm[kCTopThreads / 64];
  long long* v = lsum + (long long)blockIdx.x * nblk;
  long long carry = 0;
  for (long long base = 0; base < nblk; base += kCTopThreads) {
    const long long i = base + threadIdx.x;
    const long long x = i < nblk ? v[i] : 0ll;
    long long t;
    const long long e = top_excl_sum(x, sm, t);
    if (i < nblk) v[i] = carry + e;
    carry += t;
  }
  long long* total[kLQ] = {&tot->tab_entries, &tot->long_slots, &tot->long_items, &tot->long_chunks, &tot->long_entries};
#pragma unroll
  for (int q = 0; q < kLQ; ++q)
    if (threadIdx.x == 0 && blockIdx.x == q) *total[q] = carry;
}

__global__ __launch_bounds__(kBlock) void k_c_long_offs(CArgs a, const long long* lsum, long long nblk) {
  __shared__ long long sm[kWaves];
  if (a.tot->err) return;
  const long long nl = a.tot->nlong < a.lrow_cap ? a.tot->nlong : a.lrow_cap;
  if ((long long)blockIdx.x * kLPRows >= nl) return;  // (uniform)
  const long long i0 = (long long)blockIdx.x * kLPRows + (long long)threadIdx.x * kLP;
  int bits[kLP], nb[kLP], np[kLP];
  long long v[kLP][kLQ];
  long long su[kLQ] = {};
#pragma unroll
  for (int j = 0; j < kLP; ++j) {
    bits[j] = 1;
    nb[j] = np[j] = 0;
#pragma unroll
    for (int q = 0; q < kLQ; ++q) v[j][q] = 0;
    if (i0 + j < nl) long_row_sizes(a.lrows[i0 + j].ub, a.table_from, bits[j], nb[j], np[j], v[j]);
#pragma unroll
    for (int q = 0; q < kLQ; ++q) su[q] += v[j][q];
  }
  long long off[kLQ];
#pragma unroll
  for (int q = 0; q < kLQ; ++q) {
    long long tot;
    off[q] = lsum[q * nblk + blockIdx.x] + block_excl_sum<long long>(su[q], sm, tot);
  }
#pragma unroll
  for (int j = 0; j < kLP; ++j) {
    if (i0 + j < nl) {
      LongRow& L = a.lrows[i0 + j];
      L.eoff = off[0];
      L.toff = off[1];
      L.tbits = bits[j];
      L.nb = nb[j];
      L.np = np[j];
      L.soff = (int)(off[2] & 0x7fffffffll);
      L.boff = (int)(off[2] >> 32);
      L.coff = off[3] & (kLTabBit - 1);
    }
#pragma unroll
    for (int q = 0; q < kLQ; ++q) off[q] += v[j][q];
  }
}

// The long row of every small row, part and chunk; the chunk counts of the rows
// with a table are cleared. A lane a row, a wave the longest ones.
__global__ __launch_bounds__(kBlock) void k_c_long_tables(CArgs a, long long nl) {
  const long long step = (long long)gridDim.x * kBlock;
  for (long long r0 = (long long)blockIdx.x * kBlock + (threadIdx.x & ~63u); r0 < nl; r0 += step) {
    const long long r = r0 + lane_id();
    int np = 0, nc = 0, boff = 0;
    long long coff = 0;
    if (r < nl) {
      const LongRow L = a.lrows[r];
      np = L.np;
      nc = (L.ub + kLC - 1) / kLC;
      boff = L.boff;
      coff = L.coff;
      if (np == 0) a.srow[L.soff] = (int)r;
    }
    auto put = [&](int row, int p, int pe, int bo, int c, int ce, long long co, bool tab, int by) {
      for (; p < pe; p += by) a.prow[bo + p] = row;
      for (; c < ce; c += by) {
        a.crow[co + c] = row;
        if (tab) a.ccnt[co + c] = 0;
      }
    };
    const bool big = nc > 64;
    if (!big) put((int)r, 0, np, boff, 0, nc, coff, np < 0, 1);
    for (unsigned long long m = __ballot(big); m; m &= m - 1) {
      const int src = __ffsll((long long)m) - 1, l = lane_id();
      const int n1 = __shfl(np, src, 64);
      put((int)(r0 + src), l, n1, __shfl(boff, src, 64), l, __shfl(nc, src, 64), __shfl(coff, src, 64), n1 < 0, 64);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_c_fill(int2* t, long long m) {
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < m; i += (long long)gridDim.x * kBlock)
    t[i] = make_int2(-1, -1);
}

// The long row holding flat index i (largest eoff <= i).
__device__ __forceinline__ long long long_row_of(const LongRow* L, long long nl, long long i) {
  long long lo = 0, hi = nl;
  while (hi - lo > 1) {
    const long long mid = (lo + hi) >> 1;
    if (L[mid].eoff <= i)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// The long row of flat index i, searched forward from r0 (the row of the
// chunk's first index), which mostly holds it; rows without a table lie between.
__device__ __forceinline__ long long long_row_from(const LongRow* L, long long nl, long long r0, long long i) {
  if (r0 + 1 >= nl || L[r0 + 1].eoff > i) return r0;
  if (r0 + 2 >= nl || L[r0 + 2].eoff > i) return r0 + 1;
  return long_row_of(L, nl, i);
}

constexpr int kLI = 4;  // long-row entries per lane per round (their loads are in flight together)

// Where flat long-row index i lies: its row, fine entry and side.
struct LongAt {
  long long k;
  int r, off;
  bool side;
};
__device__ __forceinline__ LongAt long_at(const CArgs& a, long long nl, long long r0, long long i) {
  LongAt t;
  t.r = (int)long_row_from(a.lrows, nl, r0, i);
  const LongRow& L = a.lrows[t.r];
  t.off = (int)(i - L.eoff);
  t.side = t.off >= L.dega;
  t.k = t.side ? a.rp[L.b] + (t.off - L.dega) : a.rp[L.a] + t.off;
  return t;
}

// (3b) Inserts every entry of the long rows into its row's table.
__global__ __launch_bounds__(kBlock) void k_c_long_insert(CArgs a, long long nl, long long total) {
  unsigned err = 0;
  const long long step = (long long)gridDim.x * kBlock * kLI;
  for (long long i0 = (long long)blockIdx.x * kBlock * kLI; i0 < total; i0 += step) {
    const long long r0 = long_row_of(a.lrows, nl, i0);
    LongAt at[kLI];
    int x[kLI], D[kLI];
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      const long long i = i0 + (long long)j * kBlock + threadIdx.x;
      at[j].k = -1;
      if (i < total) at[j] = long_at(a, nl, r0, i);
    }
#pragma unroll
    for (int j = 0; j < kLI; ++j) x[j] = at[j].k >= 0 ? a.col[at[j].k] : -1;
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      D[j] = -1;
      if (at[j].k < 0) continue;
      if ((unsigned)x[j] >= (unsigned)a.n)
        err |= kCErrCol;
      else
        D[j] = a.identity ? x[j] : a.cmap[x[j]];
    }
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      if (D[j] < 0) continue;
      const LongRow& L = a.lrows[at[j].r];
      if (D[j] == L.c) continue;
      int2* tb = a.table + L.toff;
      const unsigned long long mask = (1ull << L.tbits) - 1;
      unsigned long long h = tbl_hash(D[j], L.tbits);
      for (;;) {
        const int old = atomicCAS(&tb[h].x, -1, D[j]);
        if (old == -1 || old == D[j]) break;
        h = (h + 1) & mask;
      }
      const int i = (int)(L.eoff + at[j].off);
      a.next[i] = atomicExch(&tb[h].y, i);
    }
  }
  if (err) atomicOr(&a.tot->err, err);
}

// (3c) The first entry of every group of a long row keeps the group's sum
// (written at its own fine entry; the others write -1).
__global__ __launch_bounds__(kBlock) void k_c_long_keep(CArgs a, long long nl, long long total) {
  unsigned err = 0;
  const long long step = (long long)gridDim.x * kBlock * kLI;
  for (long long i0 = (long long)blockIdx.x * kBlock * kLI; i0 < total; i0 += step) {
    const long long r0 = long_row_of(a.lrows, nl, i0);
    LongAt at[kLI];
    int x[kLI], D[kLI];
    float wself[kLI];
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      const long long i = i0 + (long long)j * kBlock + threadIdx.x;
      at[j].k = -1;
      if (i < total) at[j] = long_at(a, nl, r0, i);
    }
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      x[j] = at[j].k >= 0 ? a.col[at[j].k] : -1;
      wself[j] = at[j].k >= 0 && a.w ? a.w[at[j].k] : 1.0f;
    }
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      D[j] = -1;
      if (at[j].k >= 0 && (unsigned)x[j] < (unsigned)a.n) D[j] = a.identity ? x[j] : a.cmap[x[j]];
      if (D[j] >= 0 && D[j] == a.lrows[at[j].r].c) D[j] = -1;
    }
    int2 slot[kLI];
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      slot[j] = make_int2(-1, -1);
      if (D[j] < 0) continue;
      const LongRow& L = a.lrows[at[j].r];
      const int2* tb = a.table + L.toff;
      const unsigned long long mask = (1ull << L.tbits) - 1;
      unsigned long long h = tbl_hash(D[j], L.tbits);
      int2 t = tb[h];
      while (t.x != D[j]) {
        h = (h + 1) & mask;
        t = tb[h];
      }
      slot[j] = t;
    }
    int nxt[kLI];
#pragma unroll
    for (int j = 0; j < kLI; ++j) nxt[j] = D[j] >= 0 ? a.next[slot[j].y] : -1;
    long long ch[kLI];  // the chunk of a kept entry
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      ch[j] = -1;
      if (at[j].k < 0) continue;
      if (D[j] < 0) {
        if (a.dmap) a.dmap[at[j].k] = -1;
        continue;
      }
      const LongRow& L = a.lrows[at[j].r];
      const long long ka = a.rp[L.a];
      const long long kb = L.b >= 0 ? a.rp[L.b] : 0;
      // the row positions of the group's entries
      int lst[kCMaxDup + 1];
      int nlst = 0;
      int p = slot[j].y;
      int pn = nxt[j];
      bool first = true;
#pragma unroll
      for (int t = 0; t <= kCMaxDup; ++t) {  // static indices: at most five nodes matter
        if (p < 0) continue;
        lst[t] = (int)(p - L.eoff);
        nlst = t + 1;
        first = first && lst[t] >= at[j].off;
        p = pn;
        if (p >= 0 && t < kCMaxDup) pn = a.next[p];
      }
      if (nlst > a.dup_limit) err |= kCErrDup;
      if (!a.dmap) continue;
      if (!first || nlst > a.dup_limit) {
        a.dmap[at[j].k] = -1;
        continue;
      }
      float sum = wself[j];
      if (nlst > 1) {
        unsigned long long ord[kCMaxDup];
        float wv[kCMaxDup];
#pragma unroll
        for (int t = 0; t < kCMaxDup; ++t) {
          ord[t] = ~0ull;
          wv[t] = 0.f;
          if (t >= nlst) continue;
          const bool pa = lst[t] < L.dega, self = lst[t] == at[j].off;
          const long long pp = pa ? ka + lst[t] : kb + (lst[t] - L.dega);
          const int xp = self ? x[j] : a.col[pp];
          ord[t] = edge_order(pa ? L.a : L.b, xp);
          wv[t] = self ? wself[j] : (a.w ? a.w[pp] : 1.0f);
        }
        sum = group_sum(ord, wv, nlst);
      }
      a.dmap[at[j].k] = nlst > 1 ? D[j] | kMerged : D[j];
      if (nlst > 1) a.aux[at[j].k] = sum;
      ch[j] = L.coff + at[j].off / kLC;
    }
    // (the lanes of a wave are mostly in one chunk)
#pragma unroll
    for (int j = 0; j < kLI; ++j) {
      const unsigned long long m = __ballot(ch[j] >= 0);
      if (m == 0ull) continue;
      const int lead = __ffsll((long long)m) - 1;
      const long long c0 = __shfl(ch[j], lead, 64);
      const unsigned long long same = __ballot(ch[j] == c0);
      if (lane_id() == lead) atomicAdd(&a.ccnt[c0], (int)__popcll(same));
      else if (ch[j] >= 0 && ch[j] != c0) atomicAdd(&a.ccnt[ch[j]], 1);
    }
  }
  if (err) atomicOr(&a.tot->err, err);
}

// The kept entries of the rows with a table, from their chunks' counts; a wave a
// row.
__global__ __launch_bounds__(kBlock) void k_c_long_cnt(CArgs a, long long nl) {
  for (long long r = (long long)blockIdx.x * kWaves + wave_id(); r < nl; r += (long long)gridDim.x * kWaves) {
    const LongRow L = a.lrows[r];
    if (L.np >= 0) continue;
    int kept = 0;
    const int nc = (L.ub + kLC - 1) / kLC;
    for (int i = lane_id(); i < nc; i += 64) kept += a.ccnt[L.coff + i];
    kept = wave_incl_sum<int>(kept);
    if (lane_id() == 63) a.cnt[L.a] = kept;
  }
}

// ---- long rows: the coarse neighbours of a row are split into buckets by a
// hash, each with a set of kLBCap slots in LDS (a group never spans buckets).
// A row of at most kLSmall buckets is merged by one workgroup of kBlock lanes,
// one of at most kLPart by one of kLBig lanes, in one reading of its entries.
// A longer row is mapped first (its coarse neighbours into dmap, by chunks), and
// each part of kLPart buckets then streams the whole row's dmap, taking its
// own: 4 bytes an entry and part from the caches instead of a sort by bucket.

__device__ __forceinline__ unsigned bucket_of(const LongRow& L, int D) {
  return (unsigned)(((unsigned long long)((unsigned)D * 0x9E3779B1u) * (unsigned)L.nb) >> 32);
}

// Maps the rows of several parts: their coarse neighbours into dmap (-1 for
// the matched edge), the kept counts of their chunks.
__global__ __launch_bounds__(kBlock) void k_c_long_map(CArgs a) {
  __shared__ int smi[kWaves];
  unsigned err = 0;
  const int tid = threadIdx.x;
  const long long c = blockIdx.x;
  const LongRow L = a.lrows[a.crow[c]];
  if (L.np <= 1) return;  // (uniform) mapped while it is merged
  const int e0 = (int)(c - L.coff) * kLC;
  const int ne = min(kLC, L.ub - e0);
  const int ka = (int)a.rp[L.a], kb = L.b >= 0 ? (int)a.rp[L.b] : 0;
  int kept = 0;
  constexpr int kI = 8;
  for (int q0 = 0; q0 < ne; q0 += kBlock * kI) {
    int k[kI], x[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const int q = q0 + j * kBlock + tid, e = e0 + q;
      k[j] = q < ne ? (e < L.dega ? ka + e : kb + (e - L.dega)) : -1;
      x[j] = k[j] >= 0 ? a.col[k[j]] : -1;
    }
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      if (k[j] < 0) continue;
      int D = -1;
      if ((unsigned)x[j] >= (unsigned)a.n)
        err |= kCErrCol;
      else
        D = a.cmap[x[j]];
      x[j] = D == L.c ? -1 : D;
    }
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      if (k[j] < 0) continue;
      a.dmap[k[j]] = x[j];
      kept += x[j] >= 0 ? 1 : 0;
    }
  }
  int tot;
  (void)block_excl_sum<int>(kept, smi, tot);
  if (tid == 0) {
    a.ccnt[c] = tot;
    atomicAdd(&a.cnt[L.a], tot);
  }
  if (err) atomicOr(&a.tot->err, err);
}

// Merges a row (or one part of it), one workgroup each: LANES lanes, NB buckets.
// The entries dropped from each chunk are counted in LDS first: parts on several
// dies that took them off the chunks' counts one by one (95 ns an atomic on one word)
// spent most of their time there where many entries merge: rows of 10 K entries of
// which half merge, 100 M in all, 7.1 -> 3.2 ms, a star of 100 K leaves 560 -> 251 us.
template <int LANES, int NB>
struct LongSmem {
  unsigned long long tab[NB * kLBCap];
  unsigned short grp[NB * kLBCap / 2];  // slots with more than one entry
  int ngrp, kept;
  int drop[LANES == kLBig ? kLDrop : 1];  // entries dropped from each of the row's first chunks
};

template <int LANES, int NB>
__global__ __launch_bounds__(LANES, LANES == kLBig ? 8 : 4) void k_c_long_group(CArgs a, int np) {
  __shared__ LongSmem<LANES, NB> sm;
  constexpr int kI = LANES == kLBig ? 8 : 4;
  constexpr int kGrp = NB * kLBCap / 2;
  const int tid = threadIdx.x;
  unsigned err = 0;
  // (a launch of the wide workgroup may take the small rows too, after the parts)
  const LongRow L = a.lrows[LANES == kLBig && (int)blockIdx.x < np ? a.prow[blockIdx.x] : a.srow[(int)blockIdx.x - np]];
  const unsigned b0 = L.np > 0 ? (unsigned)((int)blockIdx.x - L.boff) * kLPart : 0u;
  const int slots = min(L.nb - (int)b0, NB) * kLBCap;
  for (int i = tid; i < slots; i += LANES) sm.tab[i] = kFree;
  const bool mapped = L.np > 1;
  const int ka = (int)a.rp[L.a], kb = L.b >= 0 ? (int)a.rp[L.b] : 0;
  if (tid == 0) sm.ngrp = sm.kept = 0;
  const int ndrop = LANES == kLBig && mapped ? min((L.ub + kLC - 1) / kLC, kLDrop) : 0;
  for (int i = tid; i < ndrop; i += LANES) sm.drop[i] = 0;
  __syncthreads();
  int kept = 0;
  for (int q0 = 0; q0 < L.ub; q0 += LANES * kI) {
    int k[kI], D[kI];
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const int e = q0 + j * LANES + tid;
      k[j] = e < L.ub ? (e < L.dega ? ka + e : kb + (e - L.dega)) : -1;
      D[j] = k[j] < 0 ? -1 : mapped ? a.dmap[k[j]] : a.col[k[j]];
    }
    if (!mapped) {
#pragma unroll
      for (int j = 0; j < kI; ++j) {
        if (k[j] < 0) continue;
        int d = -1;
        if ((unsigned)D[j] >= (unsigned)a.n)
          err |= kCErrCol;
        else
          d = a.cmap[D[j]];
        D[j] = d == L.c ? -1 : d;
      }
#pragma unroll
      for (int j = 0; j < kI; ++j) {
        if (k[j] < 0) continue;
        a.dmap[k[j]] = D[j];
        kept += D[j] >= 0 ? 1 : 0;
      }
    }
    // Its own entries (another part of the row may have merged its groups by
    // now): every lane enters them one after the other, one probe a step, so a
    // wave takes as many steps as its busiest lane has probes, however few of
    // the entries are this part's.
    unsigned todo = 0u;
#pragma unroll
    for (int j = 0; j < kI; ++j) {
      const bool live = D[j] != -1;
      D[j] &= ~kMerged;
      todo |= live && bucket_of(L, D[j]) - b0 < (unsigned)NB ? 1u << j : 0u;
    }
    int cur = -1, d = 0, probe = 0;
    unsigned tb = 0u, hh = 0u;
    for (;;) {
      if (cur < 0 && todo) {
        cur = __ffs((int)todo) - 1;
        todo &= todo - 1u;
#pragma unroll
        for (int j = 0; j < kI; ++j) d = cur == j ? D[j] : d;
        tb = (bucket_of(L, d) - b0) * kLBCap;
        const unsigned h0 = (unsigned)d * 0x85EBCA77u;
        hh = (h0 ^ (h0 >> 15)) & (kLBCap - 1u);
        probe = 0;
      }
      if (__ballot(cur >= 0) == 0ull) break;
      if (cur >= 0) {
        const int e = q0 + cur * LANES + tid;
        const unsigned long long old = atomicCAS(&sm.tab[tb + hh], kFree, set_slot(d, (unsigned)e | kEnd));
        bool done = old == kFree;
        if (!done && (int)(unsigned)old == d) {
          const unsigned prev = atomicExch(slot_pos(&sm.tab[tb + hh]), (unsigned)e);
          a.aux[e < L.dega ? ka + e : kb + (e - L.dega)] = __uint_as_float(prev);
          if (prev & kEnd) {
            const int g = atomicAdd(&sm.ngrp, 1);
            if (g < kGrp) sm.grp[g] = (unsigned short)(tb + hh);
          }
          done = true;
        }
        if (!done && ++probe == kLBCap) {  // a full bucket
          atomicOr(&a.tot->overflow, 1u);
          done = true;
        }
        cur = done ? -1 : cur;
        hh = (hh + 1u) & (kLBCap - 1u);
      }
    }
  }
  __syncthreads();
  const int ng = min(sm.ngrp, kGrp);
  if (tid == 0 && sm.ngrp > kGrp) atomicOr(&a.tot->overflow, 1u);
  for (int q = tid; q < ng; q += LANES) {
    const unsigned long long t = sm.tab[sm.grp[q]];
    const int d = (int)(unsigned)t;
    int lst[kCMaxDup];
    int nl = 0;
    unsigned p = (unsigned)(t >> 32);
    bool more = true;
#pragma unroll
    for (int i = 0; i < kCMaxDup; ++i) {  // static indices
      if (more) {
        const int e = (int)(p & ~kEnd);
        lst[i] = e;
        nl = i + 1;
        more = !(p & kEnd);
        if (more) p = __float_as_uint(a.aux[e < L.dega ? ka + e : kb + (e - L.dega)]);
      }
    }
    if (more || nl > a.dup_limit) err |= kCErrDup;
    int first;
    const float sum = merge_group(a, lst, nl, L.a, L.b, L.dega, ka, kb, first);
#pragma unroll
    for (int i = 0; i < kCMaxDup; ++i) {
      if (i >= nl) continue;
      const int e = lst[i], k = e < L.dega ? ka + e : kb + (e - L.dega);
      a.dmap[k] = e == first ? d | kMerged : -1;
      if (e == first) a.aux[k] = sum;
      else if (e / kLC < ndrop) atomicAdd(&sm.drop[e / kLC], 1);
      else if (mapped) atomicSub(&a.ccnt[L.coff + e / kLC], 1);
    }
    kept -= nl - 1;
  }
  kept = wave_incl_sum<int>(kept);
  if (lane_id() == 63 && kept) atomicAdd(&sm.kept, kept);
  __syncthreads();
  for (int i = tid; i < ndrop; i += LANES)
    if (sm.drop[i]) atomicSub(&a.ccnt[L.coff + i], sm.drop[i]);
  if (tid == 0) {
    if (sm.kept) atomicAdd(&a.cnt[L.a], sm.kept);
    if (!mapped) a.ccnt[L.coff] = sm.kept;
  }
  if (err) atomicOr(&a.tot->err, err);
}

// Lengths of the coarse rows base + i * kBlock + lane, all loads of a step in
// flight together.
__device__ __forceinline__ void coarse_degs(const CArgs& a, long long base, long long nc, int (&deg)[kCV]) {
  int r[kCV], m[kCV];
#pragma unroll
  for (int i = 0; i < kCV; ++i) {
    const long long c = base + (long long)i * kBlock + threadIdx.x;
    r[i] = c < nc ? a.crep[c] : -1;
  }
#pragma unroll
  for (int i = 0; i < kCV; ++i) {
    m[i] = r[i] >= 0 ? a.mate[r[i]] : -1;
    deg[i] = r[i] >= 0 ? a.cnt[r[i]] : 0;
  }
#pragma unroll
  for (int i = 0; i < kCV; ++i) deg[i] += m[i] >= 0 ? a.cnt[m[i]] : 0;
}

// (4a) Coarse row lengths, summed per block (coalesced).
__global__ __launch_bounds__(kBlock) void k_c_deg_count(CArgs a, long long nc) {
  __shared__ long long sm[kWaves];
  if (a.tot->err) return;
  int deg[kCV];
  coarse_degs(a, (long long)blockIdx.x * kCBlockV, nc, deg);
  long long s = 0;
#pragma unroll
  for (int i = 0; i < kCV; ++i) s += deg[i];
  long long total;
  (void)block_excl_sum<long long>(s, sm, total);
  if (threadIdx.x == 0) a.bsum[blockIdx.x] = total;
}

// (4c) Coarse row offsets.
__global__ __launch_bounds__(kBlock) void k_c_deg_write(CArgs a, long long nc) {
  __shared__ long long val[kCBlockV];
  __shared__ long long sm[kWaves];
  if (a.tot->err) return;
  const long long base = (long long)blockIdx.x * kCBlockV;
  int deg[kCV];
  coarse_degs(a, base, nc, deg);
#pragma unroll
  for (int i = 0; i < kCV; ++i) val[i * kBlock + threadIdx.x] = deg[i];
  __syncthreads();
  (void)block_stage_scan(val, a.bsum[blockIdx.x], sm);
#pragma unroll
  for (int i = 0; i < kCV; ++i) {
    const long long c = base + (long long)i * kBlock + threadIdx.x;
    if (c < nc) a.crp[c] = val[i * kBlock + threadIdx.x];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) a.crp[nc] = a.tot->nnz_c;
}

// (4e) Writes the kept entries of the long rows in order, one workgroup a
// chunk: its place in the output row is the sum of the counts of the chunks
// before it, its entries stay in registers between counting and writing.
__global__ __launch_bounds__(kBlock) void k_c_long_out(CArgs a) {
  __shared__ int smi[kWaves];
  constexpr int kI = kLC / kBlock;  // entries per lane
  if (a.tot->err) return;
  const int tid = threadIdx.x, l = lane_id(), wv = wave_id();
  const long long c = blockIdx.x;
  const LongRow L = a.lrows[a.crow[c]];
  const int e0 = (int)(c - L.coff) * kLC;
  const int ne = min(kLC, L.ub - e0);
  const int ka = (int)a.rp[L.a], kb = L.b >= 0 ? (int)a.rp[L.b] : 0;
  // wave w takes positions [w step, (w + 1) step) of the chunk
  const int step = ((ne + kBlock - 1) / kBlock) * 64;
  int d[kI];
  int mine = 0;
#pragma unroll
  for (int i = 0; i < kI; ++i) {
    d[i] = -1;
    if (i * 64 < step) {
      const int q = wv * step + i * 64 + l, e = e0 + q;
      if (q < ne) d[i] = a.dmap[e < L.dega ? ka + e : kb + (e - L.dega)];
    }
  }
  int before = 0;
  for (int j = tid; j < (int)(c - L.coff); j += kBlock) before += a.ccnt[L.coff + j];
#pragma unroll
  for (int i = 0; i < kI; ++i)
    if (i * 64 < step) mine += (int)__popcll(__ballot(d[i] != -1));
  int pre;
  (void)block_excl_sum<int>(before, smi, pre);
  if (l == 0) smi[wv] = mine;
  __syncthreads();
  long long dest = a.crp[L.c] + pre;
  for (int w = 0; w < wv; ++w) dest += smi[w];
#pragma unroll
  for (int i = 0; i < kI; ++i) {
    if (i * 64 < step) {
      const unsigned long long bal = __ballot(d[i] != -1);
      if (d[i] != -1) {
        const int e = e0 + wv * step + i * 64 + l;
        const int k = e < L.dega ? ka + e : kb + (e - L.dega);
        const long long at = dest + (long long)__popcll(bal & lanemask_lt());
        a.ccol[at] = d[i] & ~kMerged;
        a.cw[at] = d[i] < 0 ? a.aux[k] : (a.w ? a.w[k] : 1.0f);
      }
      dest += (long long)__popcll(bal);
    }
  }
}

size_t a256(size_t b) { return (b + 255) & ~(size_t)255; }

// Ranges of the kernels that walk the fine vertices (wg_vertices). Each
// merges the rows of its own kind only, so a range's work is anything between
// none and its cost: ranges of kCRange units, many more than fit the chip at
// once, even that out (R-MAT scale 24, against one range per resident
// workgroup: short rows 3.75 -> 1.3 ms, medium 6.3 -> 2.4, copy 3.7 -> 1.1).
// k_c_count finds their starts as it reads row_ptr anyway.
constexpr long long kCRange = 8192;

void set_ranges(CArgs& a, Pool& P, DevBuf& buf, int num_cus) {
  const long long cost = a.nnz + (long long)kCCost * a.n;
  // Smaller graphs: 20 ranges a CU, down to 2 kCT units a range. Ranges differ in
  // work by their rows' kind, and are worked off in few rounds (4 a CU: a grid of 4 M
  // vertices paired down its columns, where every other line of vertices has no row of
  // its own, 664 us against 517, R-MAT 18 562 and 415, ER with 400 K vertices 340 and 278).
  const long long want = std::max<long long>((cost + kCRange - 1) / kCRange, (long long)num_cus * 20);
  long long grid = std::max<long long>(1, std::min<long long>(want, (cost + 2 * kCT - 1) / (2 * kCT)));
  a.vstart = nullptr;
  if (P.reserve(buf, a256(sizeof(int) * (size_t)(grid + 2))) == LM_OK)
    a.vstart = (int*)buf.p;
  else  // no room: few ranges, whose starts the workgroups search for
    grid = std::min<long long>(grid, (long long)num_cus * 4);
  a.ranges = (int)grid;
  a.per_wg = (cost + grid - 1) / grid;
}

}  // namespace

// The long rows' sizes and offsets (k_c_long_sums, k_c_long_top, k_c_long_offs)
// over a grid that covers lrow_cap rows; lsum holds kLQ * long_prep_blocks(lrow_cap).
static long long long_prep_blocks(long long lrow_cap) { return std::max<long long>(1, (lrow_cap + kLPRows - 1) / kLPRows); }
static void launch_long_prep(const CArgs& a, long long* lsum, hipStream_t s) {
  const long long nblk = long_prep_blocks(a.lrow_cap);
  hipLaunchKernelGGL(k_c_long_sums, dim3((unsigned)nblk), dim3(kBlock), 0, s, a, lsum, nblk);
  hipLaunchKernelGGL(k_c_long_top, dim3(kLQ), dim3(kCTopThreads), 0, s, lsum, nblk, a.tot);
  hipLaunchKernelGGL(k_c_long_offs, dim3((unsigned)nblk), dim3(kBlock), 0, s, a, (const long long*)lsum, nblk);
}

// Buffers of the contraction, kept in the context between calls.
struct ContractState {
  DevBuf bsum, tot, crep, cnt, scr, next, lrows, table, ltab, lsum, ranges;
  DevBuf in_rp, in_col, in_w, in_mate, in_vw, o_cmap, o_crp, o_ccol, o_cw, o_cvw;
  CTot* h_tot = nullptr;
};

void contract_release(Solver& S) {
  ContractState* cs = S.contract;
  if (!cs) return;
  DevBuf* all[] = {&cs->bsum,  &cs->tot,    &cs->crep,  &cs->cnt,  &cs->scr,     &cs->next,  &cs->lrows,
                   &cs->table, &cs->ltab,   &cs->in_rp, &cs->in_col, &cs->in_w,
                   &cs->in_mate, &cs->in_vw, &cs->o_cmap, &cs->o_crp, &cs->o_ccol, &cs->o_cw, &cs->o_cvw,
                   &cs->lsum, &cs->ranges};
  for (DevBuf* b : all) S.pool.release(*b);
  if (cs->h_tot) (void)hipHostFree(cs->h_tot);
  delete cs;
  S.contract = nullptr;
}

Solver& solver_of(lm_ctx* c);
std::mutex& mutex_of(lm_ctx* c);

// Duplicate entries within rows, for LM_CHECK_GRAPH on device input: the
// grouping kernels of the contraction with every vertex free and a group
// limit of one entry (any neighbour seen twice in a row is an error). Also
// checks row_ptr. Synchronises the stream.
lm_status check_row_duplicates(Solver& S, int64_t n, int64_t nnz, const long long* rp, const int* col,
                               hipStream_t s) {
  if (n == 0) return LM_OK;
  if (!S.contract) S.contract = new ContractState();
  ContractState& cs = *S.contract;
  if (!cs.h_tot && hipHostMalloc((void**)&cs.h_tot, sizeof(CTot), hipHostMallocDefault) != hipSuccess)
    return LM_ENOMEM;
  Pool& P = S.pool;
  const long long nb_v = (n + kCBlockV - 1) / kCBlockV;
  const long long lrow_cap = nnz / (kCS + 1) + 1;
  lm_status rs;
  if ((rs = P.reserve(cs.bsum, a256(sizeof(long long) * (size_t)(nb_v + 1)))) != LM_OK) return rs;
  if ((rs = P.reserve(cs.tot, a256(sizeof(CTot)))) != LM_OK) return rs;
  if ((rs = P.reserve(cs.lrows, a256(sizeof(LongRow) * (size_t)lrow_cap))) != LM_OK) return rs;
  if ((rs = P.reserve(cs.lsum, a256(sizeof(long long) * kLQ * (size_t)long_prep_blocks(lrow_cap)))) != LM_OK) return rs;
  CArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n = n;
  a.nnz = nnz;
  a.rp = rp;
  a.col = col;
  a.bsum = (long long*)cs.bsum.p;
  a.tot = (CTot*)cs.tot.p;
  a.lrows = (LongRow*)cs.lrows.p;
  a.lrow_cap = lrow_cap;
  a.dup_limit = 1;
  a.identity = 1;
  a.table_from = 0;
  if (hipMemsetAsync(a.tot, 0, sizeof(CTot), s) != hipSuccess) return LM_EDEVICE;
  set_ranges(a, P, cs.ranges, S.num_cus);
  hipLaunchKernelGGL(k_c_count, dim3((unsigned)nb_v), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_c_group_wave, dim3((unsigned)a.ranges), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_c_group_mid, dim3((unsigned)a.ranges), dim3(kBlock), 0, s, a);
  launch_long_prep(a, (long long*)cs.lsum.p, s);
  if (hipGetLastError() != hipSuccess) return LM_EDEVICE;
  if (hipMemcpyAsync(cs.h_tot, a.tot, sizeof(CTot), hipMemcpyDeviceToHost, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    return LM_EDEVICE;
  const CTot t1 = *cs.h_tot;
  if (t1.err) return LM_EGRAPH;
  if (t1.nlong > 0) {
    if (t1.nlong > lrow_cap) return LM_EDEVICE;
    if ((rs = P.reserve(cs.next, a256(sizeof(int) * (size_t)t1.tab_entries))) != LM_OK) return rs;
    if ((rs = P.reserve(cs.table, a256(sizeof(int2) * (size_t)t1.long_slots))) != LM_OK) return rs;
    a.next = (int*)cs.next.p;
    a.table = (int2*)cs.table.p;
    const long long fill_grid = std::min<long long>((t1.long_slots + kBlock - 1) / kBlock, 8192);
    hipLaunchKernelGGL(k_c_fill, dim3((unsigned)fill_grid), dim3(kBlock), 0, s, a.table, t1.long_slots);
    const long long lg = std::min<long long>((t1.tab_entries + kBlock * kLI - 1) / (kBlock * kLI), 16384);
    hipLaunchKernelGGL(k_c_long_insert, dim3((unsigned)lg), dim3(kBlock), 0, s, a, t1.nlong, t1.tab_entries);
    hipLaunchKernelGGL(k_c_long_keep, dim3((unsigned)lg), dim3(kBlock), 0, s, a, t1.nlong, t1.tab_entries);
    if (hipGetLastError() != hipSuccess) return LM_EDEVICE;
    if (hipMemcpyAsync(cs.h_tot, a.tot, sizeof(CTot), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
      return LM_EDEVICE;
    if (cs.h_tot->err) return LM_EGRAPH;
  }
  return LM_OK;
}

}  // namespace lm

using namespace lm;

#define LMC_TRY(x)                    \
  do {                                \
    const lm_status st_ = (x);        \
    if (st_ != LM_OK) return st_;     \
  } while (0)
#define LMC_HIP(x)                                \
  do {                                            \
    const hipError_t e_ = (x);                    \
    if (e_ != hipSuccess) return dev_status(e_);  \
  } while (0)

extern "C" {

lm_status lm_contract(lm_ctx* ctx, const lm_csr* g, const int32_t* mate, const int64_t* vwgt, int32_t* cmap,
                      lm_coarse* out, uint32_t flags, void* stream, lm_contract_stats* st) {
  if (!ctx || !g || !out) return LM_EINVAL;
  if (flags & ~(LM_IN_DEVICE | LM_OUT_DEVICE)) return LM_EINVAL;
  const int64_t n = g->n, nnz = g->nnz;
  if (n < 0 || nnz < 0) return LM_EINVAL;
  if (n >= ((int64_t)1 << 31) || nnz >= ((int64_t)1 << 31) - 65536) return LM_ETOOBIG;
  if (!g->row_ptr || !out->row_ptr) return LM_EINVAL;
  if (n > 0 && (!mate || !cmap)) return LM_EINVAL;
  if (nnz > 0 && (!g->col || !out->col || !out->w)) return LM_EINVAL;
  std::lock_guard<std::mutex> lk(mutex_of(ctx));
  Solver& S = solver_of(ctx);
  if (S.busy_server) return LM_EINVAL;
  if (st) std::memset(st, 0, sizeof(*st));
  out->n = 0;
  out->nnz = 0;
  if (hipSetDevice(S.dev) != hipSuccess) return LM_EDEVICE;
  if (S.async_pending) {
    if (hipEventSynchronize(S.e_async) != hipSuccess) return LM_EDEVICE;
    S.async_pending = false;
  }
  hipStream_t s = (hipStream_t)stream;
  const bool din = (flags & LM_IN_DEVICE) != 0, dout = (flags & LM_OUT_DEVICE) != 0;
  if (n == 0) {
    const int64_t zero = 0;
    if (dout) {
      LMC_HIP(hipMemcpyAsync(out->row_ptr, &zero, sizeof(zero), hipMemcpyHostToDevice, s));
      LMC_HIP(hipStreamSynchronize(s));
    } else {
      out->row_ptr[0] = 0;
    }
    return LM_OK;
  }
  if (!S.contract) S.contract = new ContractState();
  ContractState& cs = *S.contract;
  if (!cs.h_tot) LMC_HIP(hipHostMalloc((void**)&cs.h_tot, sizeof(CTot), hipHostMallocDefault));
  Pool& P = S.pool;
  const long long nb_v = (n + kCBlockV - 1) / kCBlockV;
  const long long lrow_cap = nnz / (kCS + 1) + 1;
  LMC_TRY(P.reserve(cs.bsum, a256(sizeof(long long) * (size_t)(nb_v + 1))));
  LMC_TRY(P.reserve(cs.tot, a256(sizeof(CTot))));
  LMC_TRY(P.reserve(cs.crep, a256(sizeof(int) * (size_t)n)));
  LMC_TRY(P.reserve(cs.cnt, a256(sizeof(int) * (size_t)n)));
  LMC_TRY(P.reserve(cs.scr, a256(sizeof(int2) * (size_t)(nnz > 0 ? nnz : 1))));
  LMC_TRY(P.reserve(cs.lrows, a256(sizeof(LongRow) * (size_t)lrow_cap)));
  LMC_TRY(P.reserve(cs.lsum, a256(sizeof(long long) * kLQ * (size_t)long_prep_blocks(lrow_cap))));

  CArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n = n;
  a.nnz = nnz;
  // inputs
  if (din) {
    a.rp = (const long long*)g->row_ptr;
    a.col = g->col;
    a.w = g->w;
    a.mate = mate;
    a.vw = (const long long*)vwgt;
  } else {
    LMC_TRY(P.reserve(cs.in_rp, a256(sizeof(int64_t) * (size_t)(n + 1))));
    LMC_TRY(P.reserve(cs.in_col, a256(sizeof(int32_t) * (size_t)(nnz > 0 ? nnz : 1))));
    LMC_TRY(P.reserve(cs.in_mate, a256(sizeof(int32_t) * (size_t)n)));
    LMC_HIP(hipMemcpyAsync(cs.in_rp.p, g->row_ptr, sizeof(int64_t) * (size_t)(n + 1), hipMemcpyHostToDevice, s));
    if (nnz > 0)
      LMC_HIP(hipMemcpyAsync(cs.in_col.p, g->col, sizeof(int32_t) * (size_t)nnz, hipMemcpyHostToDevice, s));
    LMC_HIP(hipMemcpyAsync(cs.in_mate.p, mate, sizeof(int32_t) * (size_t)n, hipMemcpyHostToDevice, s));
    a.rp = (const long long*)cs.in_rp.p;
    a.col = (const int*)cs.in_col.p;
    a.mate = (const int*)cs.in_mate.p;
    if (g->w) {
      LMC_TRY(P.reserve(cs.in_w, a256(sizeof(float) * (size_t)(nnz > 0 ? nnz : 1))));
      if (nnz > 0) LMC_HIP(hipMemcpyAsync(cs.in_w.p, g->w, sizeof(float) * (size_t)nnz, hipMemcpyHostToDevice, s));
      a.w = (const float*)cs.in_w.p;
    }
    if (vwgt) {
      LMC_TRY(P.reserve(cs.in_vw, a256(sizeof(int64_t) * (size_t)n)));
      LMC_HIP(hipMemcpyAsync(cs.in_vw.p, vwgt, sizeof(int64_t) * (size_t)n, hipMemcpyHostToDevice, s));
      a.vw = (const long long*)cs.in_vw.p;
    }
  }
  // outputs (host outputs go through device buffers of the worst-case size)
  if (dout) {
    a.cmap = cmap;
    a.crp = (long long*)out->row_ptr;
    a.ccol = out->col;
    a.cw = out->w;
    a.cvw = (long long*)out->vwgt;
  } else {
    LMC_TRY(P.reserve(cs.o_cmap, a256(sizeof(int32_t) * (size_t)n)));
    LMC_TRY(P.reserve(cs.o_crp, a256(sizeof(int64_t) * (size_t)(n + 1))));
    LMC_TRY(P.reserve(cs.o_ccol, a256(sizeof(int32_t) * (size_t)(nnz > 0 ? nnz : 1))));
    LMC_TRY(P.reserve(cs.o_cw, a256(sizeof(float) * (size_t)(nnz > 0 ? nnz : 1))));
    a.cmap = (int*)cs.o_cmap.p;
    a.crp = (long long*)cs.o_crp.p;
    a.ccol = (int*)cs.o_ccol.p;
    a.cw = (float*)cs.o_cw.p;
    if (out->vwgt) {
      LMC_TRY(P.reserve(cs.o_cvw, a256(sizeof(int64_t) * (size_t)n)));
      a.cvw = (long long*)cs.o_cvw.p;
    }
  }
  a.crep = (int*)cs.crep.p;
  a.cnt = (int*)cs.cnt.p;
  a.bsum = (long long*)cs.bsum.p;
  a.tot = (CTot*)cs.tot.p;
  a.dmap = (int*)cs.scr.p;
  a.aux = (float*)cs.scr.p + nnz;
  a.lrows = (LongRow*)cs.lrows.p;
  a.lrow_cap = lrow_cap;
  a.dup_limit = kCMaxDup;
  a.identity = 0;
  a.table_from = kLTable;
  set_ranges(a, P, cs.ranges, S.num_cus);

  LMC_HIP(hipEventRecord(S.e0, s));
  LMC_HIP(hipMemsetAsync(a.tot, 0, sizeof(CTot), s));
  hipLaunchKernelGGL(k_c_count, dim3((unsigned)nb_v), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_c_scan_top, dim3(1), dim3(kCTopThreads), 0, s, a.bsum, nb_v, &a.tot->nc);
  hipLaunchKernelGGL(k_c_map, dim3((unsigned)nb_v), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_c_group_wave, dim3((unsigned)a.ranges), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_c_group_mid, dim3((unsigned)a.ranges), dim3(kBlock), 0, s, a);
  launch_long_prep(a, (long long*)cs.lsum.p, s);
  LMC_HIP(hipGetLastError());
  LMC_HIP(hipMemcpyAsync(cs.h_tot, a.tot, sizeof(CTot), hipMemcpyDeviceToHost, s));
  LMC_HIP(hipStreamSynchronize(s));
  CTot t1 = *cs.h_tot;
  if (t1.err & kCErrMate) return LM_EINVAL;
  if (t1.err) return LM_EGRAPH;
  const long long nc = t1.nc;
  const long long nl = t1.nlong;
  if (nl > lrow_cap) return LM_EDEVICE;  // cannot happen: the bounds of the rows sum to nnz
  // sizes and offsets again, with other rows merged through tables
  auto prep_again = [&](long long table_from) -> lm_status {
    a.table_from = table_from;
    launch_long_prep(a, (long long*)cs.lsum.p, s);
    LMC_HIP(hipGetLastError());
    LMC_HIP(hipMemcpyAsync(cs.h_tot, a.tot, sizeof(CTot), hipMemcpyDeviceToHost, s));
    LMC_HIP(hipStreamSynchronize(s));
    t1 = *cs.h_tot;
    return LM_OK;
  };
  auto reserve_tables = [&]() -> lm_status {
    LMC_TRY(P.reserve(cs.next, a256(sizeof(int) * (size_t)t1.tab_entries)));
    LMC_TRY(P.reserve(cs.table, a256(sizeof(int2) * (size_t)t1.long_slots)));
    a.next = (int*)cs.next.p;
    a.table = (int2*)cs.table.p;
    return LM_OK;
  };
  auto launch_tables = [&]() {  // merges the rows with a table
    const long long lg = std::min<long long>((t1.tab_entries + kBlock * kLI - 1) / (kBlock * kLI), 16384);
    const long long fill_grid = std::min<long long>((t1.long_slots + kBlock - 1) / kBlock, 8192);
    hipLaunchKernelGGL(k_c_fill, dim3((unsigned)fill_grid), dim3(kBlock), 0, s, a.table, t1.long_slots);
    hipLaunchKernelGGL(k_c_long_insert, dim3((unsigned)lg), dim3(kBlock), 0, s, a, nl, t1.tab_entries);
    hipLaunchKernelGGL(k_c_long_keep, dim3((unsigned)lg), dim3(kBlock), 0, s, a, nl, t1.tab_entries);
    hipLaunchKernelGGL(k_c_long_cnt, dim3((unsigned)std::min<long long>((nl + kWaves - 1) / kWaves, 4096)), dim3(kBlock),
                       0, s, a, nl);
  };
  auto launch_index = [&]() {
    hipLaunchKernelGGL(k_c_long_tables, dim3((unsigned)std::min<long long>((nl + kBlock - 1) / kBlock, 4096)),
                       dim3(kBlock), 0, s, a, nl);
  };
  if (nl > 0) {
    long long np, nsm, nch;
    auto reserve_index = [&]() -> lm_status {
      np = t1.long_items >> 32;
      nsm = t1.long_items & 0x7fffffffll;
      nch = t1.long_chunks & (kLTabBit - 1);
      return P.reserve(cs.ltab, a256(sizeof(int) * (size_t)(nsm + np + 2 * nch)));
    };
    if (t1.tab_entries > 0 && (reserve_tables() != LM_OK || reserve_index() != LM_OK)) {
      // no room for the tables: the parts need none
      P.release(cs.next);
      P.release(cs.table);
      LMC_TRY(prep_again(LLONG_MAX));
    }
    LMC_TRY(reserve_index());
    a.srow = (int*)cs.ltab.p;
    a.prow = a.srow + nsm;
    a.crow = a.prow + np;
    a.ccnt = a.crow + nch;
    launch_index();
    // a workgroup per chunk, part and row: they differ in work, and are
    // handed out as workgroups end
    if (np > 0) hipLaunchKernelGGL(k_c_long_map, dim3((unsigned)nch), dim3(kBlock), 0, s, a);
    const bool one = np > 0 && np + nsm <= 2 * S.num_cus;  // few of both: one launch
    if (np > 0)
      hipLaunchKernelGGL((k_c_long_group<kLBig, kLPart>), dim3((unsigned)(np + (one ? nsm : 0))), dim3(kLBig), 0, s, a,
                         (int)np);
    if (nsm > 0 && !one)
      hipLaunchKernelGGL((k_c_long_group<kBlock, kLSmall>), dim3((unsigned)nsm), dim3(kBlock), 0, s, a, 0);
    if (t1.tab_entries > 0) launch_tables();
    LMC_HIP(hipGetLastError());
    LMC_HIP(hipMemcpyAsync(cs.h_tot, a.tot, sizeof(CTot), hipMemcpyDeviceToHost, s));
    LMC_HIP(hipStreamSynchronize(s));
    if (cs.h_tot->err & kCErrMate) return LM_EINVAL;
    if (cs.h_tot->err) return LM_EGRAPH;
    if (cs.h_tot->overflow) {  // a bucket outgrew LDS: every long row through per-row tables
      LMC_TRY(prep_again(0));
      LMC_TRY(reserve_tables());
      launch_index();
      launch_tables();
    }
  }
  const long long table_rows = t1.long_chunks / kLTabBit;
  const long long nb_c = (nc + kCBlockV - 1) / kCBlockV;
  if (nb_c > 0) {
    hipLaunchKernelGGL(k_c_deg_count, dim3((unsigned)nb_c), dim3(kBlock), 0, s, a, nc);
    hipLaunchKernelGGL(k_c_scan_top, dim3(1), dim3(kCTopThreads), 0, s, a.bsum, nb_c, &a.tot->nnz_c);
    hipLaunchKernelGGL(k_c_deg_write, dim3((unsigned)nb_c), dim3(kBlock), 0, s, a, nc);
  }
  hipLaunchKernelGGL(k_c_copy, dim3((unsigned)a.ranges), dim3(kBlock), 0, s, a);
  if (nl > 0) hipLaunchKernelGGL(k_c_long_out, dim3((unsigned)(t1.long_chunks & (kLTabBit - 1))), dim3(kBlock), 0, s, a);
  LMC_HIP(hipGetLastError());
  LMC_HIP(hipEventRecord(S.e1, s));
  LMC_HIP(hipMemcpyAsync(cs.h_tot, a.tot, sizeof(CTot), hipMemcpyDeviceToHost, s));
  LMC_HIP(hipStreamSynchronize(s));
  const CTot t2 = *cs.h_tot;
  if (t2.err & kCErrMate) return LM_EINVAL;
  if (t2.err) return LM_EGRAPH;
  const long long nnz_c = t2.nnz_c;
  if (!dout) {
    LMC_HIP(hipMemcpy(cmap, a.cmap, sizeof(int32_t) * (size_t)n, hipMemcpyDeviceToHost));
    LMC_HIP(hipMemcpy(out->row_ptr, a.crp, sizeof(int64_t) * (size_t)(nc + 1), hipMemcpyDeviceToHost));
    if (nnz_c > 0) {
      LMC_HIP(hipMemcpy(out->col, a.ccol, sizeof(int32_t) * (size_t)nnz_c, hipMemcpyDeviceToHost));
      LMC_HIP(hipMemcpy(out->w, a.cw, sizeof(float) * (size_t)nnz_c, hipMemcpyDeviceToHost));
    }
    if (out->vwgt) LMC_HIP(hipMemcpy(out->vwgt, a.cvw, sizeof(int64_t) * (size_t)nc, hipMemcpyDeviceToHost));
  }
  out->n = nc;
  out->nnz = nnz_c;
  if (st) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, S.e0, S.e1) == hipSuccess) st->device_ms = ms;
    const double eb = g->w ? 8.0 : 4.0;
    st->bytes_alg = 8.0 * (n + 1) + 4.0 * n + (eb + 4.0) * nnz + 4.0 * n + 8.0 * (nc + 1) + 8.0 * nnz_c +
                    (vwgt ? 8.0 * n : 0.0) + (out->vwgt ? 8.0 * nc : 0.0);
    st->long_rows = nl;
    st->long_entries = t1.long_entries;
    st->table_rows = table_rows;
  }
  return LM_OK;
}

}  // extern "C"
