// First compaction of one weighted graph by whole rows (R_1 read from its CSR),
// fused with the candidates of phase 2, gfx950.
//
// Workgroup b of the G resident ones takes the vertices [n b / G, n (b + 1) / G)
// (runs G .. P of the live set's P stay empty). A row costs its lane group a step
// whatever its length, so equal vertices are equal work, and no range has to be
// searched for. A wave looks at 64 vertices at a time and queues the rows of the
// unmatched ones in LDS; a step takes up to 64 queued rows, in lane groups
// (lm_rows.h), drops the entries whose neighbour is matched, takes the rows'
// winners and puts the rest, through the wave's LDS, in the next places of the
// workgroup's range of the entry buffer, with one piece record a row. One LDS
// atomic a step hands out both places, so the pieces lie in the order of their
// entries and form one run, as the other phase kernels expect. No row is cut:
// there are no partial results to stitch, and no wave waits for another.
//
// Bound by the dependent gathers of the neighbours' state and, at 2^24 vertices,
// by memory. Against the piece-window kernel (k_stream, a workgroup scan and
// barriers every 2048 entries): RGG with 2^20 vertices 82 -> 29 us, RGG with 2^24
// 583 -> 412 us. Each of these was needed: kept entries stored by the lanes
// directly, 665 us at 2^24; ranges of equal cost, searched for, 74 us at 2^20;
// steps over the rows of 64 vertices without the queue, 606 us; as many ranges as
// k_stream has (5 a CU, where 4 are resident here), 549 us.
#include <hip/hip_ext.h>

#include <algorithm>

#include "lm_device.h"
#include "lm_internal.h"
#include "lm_key.h"
#include "lm_rows.h"

namespace lm {

namespace {

constexpr int kCI = 8;       // entries per lane and step
constexpr int kQueue = 128;  // rows: a step takes up to 64, and a wave adds up to 64 at a time

struct CompactSmem {
  unsigned long long at;  // low word: entries placed; high word: rows placed
  unsigned md, loaded;
  unsigned err;
  int qv[kWaves][kQueue], qo[kWaves][kQueue];  // rows waiting for a step
  unsigned short ql[kWaves][kQueue];
  uint2 stage[kWaves][2 * 64 * kCI];
};

// Places for `tot` entries and `rows` rows of the workgroup's run.
__device__ __forceinline__ void take(CompactSmem& sm, unsigned tot, int rows, int& base, int& row) {
  unsigned long long x = 0ull;
  if (lane_id() == 0) x = atomicAdd(&sm.at, ((unsigned long long)(unsigned)rows << 32) | tot);
  base = uni((int)(unsigned)x);
  row = uni((int)(x >> 32));
}

struct CompactArgs {
  const StreamArgs& a;
  const unsigned* bits;  // matched bits, or nullptr: the state bytes
  int n, lim;
  unsigned long long S;
  int e0, r0;  // the run's first entry and piece
};

// The entries of unmatched neighbours.
__device__ __forceinline__ void filter(const CompactArgs& c, int rem, const int (&cv)[kCI], bool (&ok)[kCI]) {
  unsigned st[kCI];
#pragma unroll
  for (int q = 0; q < kCI; ++q) {
    ok[q] = q < rem && (unsigned)cv[q] < (unsigned)c.n;
    const int u = ok[q] ? cv[q] : 0;
    st[q] = c.bits ? c.bits[u >> 5] >> (u & 31) & 1u : (unsigned)c.a.c.state[u];
  }
#pragma unroll
  for (int q = 0; q < kCI; ++q) ok[q] = ok[q] && st[q] == 0u;
}

__device__ __forceinline__ void write_kept(const CompactArgs& c, int at, const bool (&ok)[kCI], const int (&cv)[kCI],
                                           const unsigned (&wv)[kCI]) {
#pragma unroll
  for (int q = 0; q < kCI; ++q) {
    if (ok[q]) {
      c.a.dst_col[at] = cv[q];
      c.a.dst_w[at] = __uint_as_float(wv[q]);
      ++at;
    }
  }
}

// N steps: every group of 2^lg lanes holds N rows v (len entries each, at most
// kCI << lg; already loaded). What is kept goes through the wave's LDS, so that
// it is written in whole lines.
template <int N>
__device__ __forceinline__ void steps(const CompactArgs& c, CompactSmem& sm, int lg, unsigned long long gm,
                                      const int (&v)[N], const int (&len)[N], const int (&cv)[N][kCI],
                                      unsigned (&wv)[N][kCI]) {
  const int lane = lane_id(), sub = lane & ((1 << lg) - 1);
  uint2* st = sm.stage[wave_id()];
  int at[N], row[N];
  unsigned tot = 0u, nrow = 0u;
#pragma unroll
  for (int p = 0; p < N; ++p) {
    const int rem = len[p] - kCI * sub;
    bool ok[kCI];
    filter(c, rem, cv[p], ok);
    int u = 0;
    unsigned m;
    if (group_winner<kKeyWeight>(ok, cv[p], wv[p], rem > 0, lg, gm, (unsigned)v[p], c.S, u, m)) c.a.c.C[v[p]] = u;
    unsigned k = 0;
#pragma unroll
    for (int q = 0; q < kCI; ++q) k += ok[q] ? 1u : 0u;
    const unsigned incl = wave_incl_sum_u32(k);
    const unsigned last = (unsigned)__shfl((int)incl, lane | ((1 << lg) - 1), 64);
    row[p] = sub == 0 ? (int)(last - (incl - k)) : 0;
    at[p] = (int)(tot + incl - k);
    int x = at[p];
#pragma unroll
    for (int q = 0; q < kCI; ++q)
      if (ok[q]) st[x++] = make_uint2((unsigned)cv[p][q], wv[p][q]);
    tot += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    nrow += (unsigned)__popcll(__ballot(row[p] > 0));
  }
  if (tot == 0u) return;
  int base, ps;
  take(sm, tot, (int)nrow, base, ps);
#pragma unroll
  for (int p = 0; p < N; ++p) {
    const unsigned long long rows = __ballot(row[p] > 0);
    if (row[p] > 0)
      c.a.rows_out[c.r0 + ps + (int)__popcll(rows & lanemask_lt())] =
          make_int4(v[p], c.e0 + base + at[p], row[p], kHeadBit);
    ps += (int)__popcll(rows);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (unsigned k = (unsigned)lane; k < tot; k += 64u) {
    const uint2 e = st[k];
    c.a.dst_col[c.e0 + base + (int)k] = (int)e.x;
    c.a.dst_w[c.e0 + base + (int)k] = __uint_as_float(e.y);
  }
  __builtin_amdgcn_wave_barrier();
}

// A row longer than a step of the wave: counted first, then written.
__device__ __forceinline__ void long_row(const CompactArgs& c, CompactSmem& sm, int v, int off, int len) {
  unsigned bw = 0u, kept = 0u;
  int bu = 0, base = 0, ps = 0;
  for (int pass = 0; pass < 2; ++pass) {
    unsigned done = 0u;
    for (int k0 = 0; k0 < len; k0 += 64 * kCI) {
      const int k = k0 + kCI * lane_id();
      int cv[kCI];
      unsigned wv[kCI];
      load_row<true>(c.a.in.col, c.a.in.w, off + k, c.lim, k < len, cv, wv);
      bool ok[kCI];
      filter(c, len - k, cv, ok);
      unsigned x = 0;
#pragma unroll
      for (int q = 0; q < kCI; ++q) x += ok[q] ? 1u : 0u;
      const unsigned incl = wave_incl_sum_u32(x);
      if (pass == 0) {
        int u = 0;
        unsigned m;
        const unsigned long long win =
            __ballot(group_winner<kKeyWeight>(ok, cv, wv, k < len, 6, ~0ull, (unsigned)v, c.S, u, m));
        if (m != 0u) best_pair(bw, bu, uni(m), __shfl(u, __ffsll((long long)win) - 1, 64), (unsigned)v, c.S);
      } else {
        write_kept(c, c.e0 + base + (int)(done + incl - x), ok, cv, wv);
      }
      done += (unsigned)__builtin_amdgcn_readlane((int)incl, 63);
    }
    if (pass == 0) {
      kept = done;
      if (kept == 0u) return;
      take(sm, kept, 1, base, ps);
    }
  }
  if (lane_id() == 0) {
    if (bw != 0u) c.a.c.C[v] = bu;
    c.a.rows_out[c.r0 + ps] = make_int4(v, c.e0 + base, (int)kept, kHeadBit);
  }
}

__device__ __forceinline__ void put_run(const StreamArgs& a, int b, const Run& r, long long loaded, long long gone) {
  Part none;
  none.v = -1;
  a.parts[2 * b] = none;
  a.parts[2 * b + 1] = none;
  a.runs_out[b] = r;
  BlockStat st;
  st.loaded = loaded;
  st.matched_len = gone;
  st.pieces_out = r.row_count;
  st.pad = 0;
  a.bstat[b] = st;
}

}  // namespace

__global__ __launch_bounds__(kBlock, 4) void k_compact_rows(StreamArgs a, int lg, long long nnz) {
  __shared__ CompactSmem sm;
  if (threadIdx.x == 0) {
    const Totals* t = a.c.totals;
    sm.err = t->err | (handed_over(a.c, t->tail_from) ? 0x80000000u : 0u) | (compact_by_rows(t, a.c.n) ? 0u : 1u);
  }
  __syncthreads();
  if (sm.err) return;
  const int P = uni(a.in.ctl->P);
  CompactArgs c{a, a.c.mbits && bits_on(a.c.totals) ? a.c.mbits : nullptr, a.c.n, (int)nnz,
                cand_seed(a.c.gseed[0], a.c.renew, a.cand_phase), 0, 0};
  const int lane = lane_id(), wv = uni(wave_id());
  const int sub = lane & ((1 << lg) - 1), grp = lane >> lg, per = 64 >> lg, thr = kCI << lg;
  const int cnt = min(2 * per, 64);  // rows a step takes
  const unsigned long long gm = group_mask(lg);
  const int G = min((int)gridDim.x, P), b = blockIdx.x;
  if (b < G) {
    const int vb = (int)((long long)c.n * b / G), ve = (int)((long long)c.n * (b + 1) / G);
    c.e0 = uni((int)a.in.csr_rp[vb]);
    c.r0 = vb;
    if (threadIdx.x == 0) {
      sm.at = 0ull;
      sm.md = sm.loaded = 0u;
    }
    __syncthreads();
    unsigned md = 0u, loaded = 0u;
    auto offs = [&](unsigned v0, int& o0, int& o1, unsigned& st) {
      const unsigned v = v0 + (unsigned)lane;
      const bool in = v < (unsigned)ve;
      o0 = in ? (int)a.in.csr_rp[v] : 0;
      o1 = in ? (int)a.in.csr_rp[v + 1u] : 0;
      st = in ? a.c.state[v] : 1u;
    };
    int n0 = 0, n1 = 0;
    unsigned ns = 1u;
    unsigned v0 = (unsigned)vb + (unsigned)wv * 64u;  // (may pass 2^31)
    if (v0 < (unsigned)ve) offs(v0, n0, n1, ns);
    unsigned head = 0u, tail = 0u;
    for (;;) {
      while (tail - head < (unsigned)cnt && v0 < (unsigned)ve) {
        const int v = (int)(v0 + (unsigned)lane), off = n0;
        int len = n1 - n0;
        const bool matched = ns != 0u;
        v0 += kBlock;
        if (v0 < (unsigned)ve) offs(v0, n0, n1, ns);  // the wave's next rows
        md += matched ? (unsigned)len : 0u;
        loaded += matched ? 0u : (unsigned)len;
        if (matched) len = 0;
        unsigned long long lng = __ballot(len > thr);
        while (lng) {
          const int src = __ffsll((long long)lng) - 1;
          lng &= lng - 1;
          const int rv = __builtin_amdgcn_readlane(v, src), ro = __builtin_amdgcn_readlane(off, src);
          const int rl = __builtin_amdgcn_readlane(len, src);
          long_row(c, sm, rv, ro, rl);
        }
        const bool put = len > 0 && len <= thr;
        const unsigned long long bal = __ballot(put);
        if (put) {
          const unsigned x = (tail + (unsigned)__popcll(bal & lanemask_lt())) & (kQueue - 1);
          sm.qv[wv][x] = v;
          sm.qo[wv][x] = off;
          sm.ql[wv][x] = (unsigned short)len;
        }
        tail += (unsigned)__popcll(bal);
      }
      if (head == tail) break;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int take_n = min(cnt, (int)(tail - head));
      int vv[2], ll[2], cv[2][kCI];
      unsigned wr[2][kCI];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int k = p * per + grp;
        const unsigned x = (head + (unsigned)k) & (kQueue - 1);
        vv[p] = sm.qv[wv][x];
        const int o = sm.qo[wv][x];
        ll[p] = k < take_n ? (int)sm.ql[wv][x] : 0;
        load_row<true>(a.in.col, a.in.w, o + kCI * sub, c.lim, kCI * sub < ll[p], cv[p], wr[p]);
      }
      head += (unsigned)take_n;
      if (take_n > per) steps<2>(c, sm, lg, gm, vv, ll, cv, wr);
      else {
        int v1[1] = {vv[0]}, l1[1] = {ll[0]};
        steps<1>(c, sm, lg, gm, v1, l1, *reinterpret_cast<int(*)[1][kCI]>(&cv), *reinterpret_cast<unsigned(*)[1][kCI]>(&wr));
      }
    }
    md = wave_incl_sum_u32(md);
    loaded = wave_incl_sum_u32(loaded);
    if (lane == 63) {
      atomicAdd(&sm.md, md);
      atomicAdd(&sm.loaded, loaded);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      Run r;
      r.row_begin = c.r0;
      r.row_count = (int)(sm.at >> 32);
      r.phys_begin = c.e0;
      r.ent_count = (int)(unsigned)sm.at;
      put_run(a, b, r, sm.loaded, sm.md);
      for (int e = b + G; e < P; e += G) put_run(a, e, Run{}, 0, 0);
    }
  }
}

int compact_rows_per_cu() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_compact_rows, kBlock, 0) != hipSuccess || nb < 1) nb = 1;
  return nb;
}

hipError_t launch_compact_rows(const StreamArgs& a, int grid, int lg, long long nnz, hipStream_t s, hipEvent_t* ev) {
  if (ev) hipExtLaunchKernelGGL(k_compact_rows, dim3(grid), dim3(kBlock), 0, s, ev[0], ev[1], 0, a, lg, nnz);
  else hipLaunchKernelGGL(k_compact_rows, dim3(grid), dim3(kBlock), 0, s, a, lg, nnz);
  return hipGetLastError();
}

}  // namespace lm
