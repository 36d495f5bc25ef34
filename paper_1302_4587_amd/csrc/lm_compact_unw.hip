// First compaction of one unweighted graph (R_1 read from its CSR), fused with
// the candidates of phase 2, gfx950.
//
// A one-wave workgroup walks its range of R_1 (equal cost: entries plus a fixed
// cost per row) in steps of kCStep consecutive entries, four per lane, as the
// first argmax of these graphs does (lm_first.hip); no workgroup barrier couples
// waves and the output of a range is one run in the order of its entries. A
// window of 64 rows, their ends and whether they are live (unmatched and not
// empty) one per lane, gives the step its rows; a step starts at a live row, so
// matched rows that fill steps are never read. The next step's entries are
// loaded after this step's gathers of the neighbours' state have been issued
// and before they are used. Kept entries go through LDS and are written in whole
// lines; their running count, read back at the row ends, gives the piece records.
// Within a row that spans the step the lanes keep their largest hash in registers;
// rows that end inside a step are combined by LDS 64-bit atomic max. Rows cut at
// range boundaries leave a partial result for the plan kernel.
//
// Bound by the gathers of the matched bits on R-MAT 24: 189 M lines from the L2,
// 96 G a second, the rate any scattered gather reaches here (the VALU is busy a
// third of the time). Against the piece-window kernel (a workgroup scan and
// several barriers per batch, lookups of each entry's row in LDS): R-MAT 20
// 172 -> 116 us, R-MAT 24 2137 -> 1977 us. The entries are read past the caches,
// which leaves the L1 to the bits (whole solves 579 -> 573 and 5712 -> 5660 us;
// the bits read that way: 6980). Eight entries a lane and step: 600 and 5967.
#include <hip/hip_ext.h>

#include "lm_device.h"
#include "lm_internal.h"
#include "lm_key.h"
#include "lm_rows.h"

namespace lm {

namespace {

constexpr int kCIt = 4;  // entries per lane and step
constexpr int kCStep = 64 * kCIt;
constexpr int kCPerCu = 16;  // one-wave ranges per CU

struct UnwCompactSmem {
  unsigned mark[kCStep];             // 1 + window index of the row starting at step position x, 0 none
  unsigned long long slot[64 + 64];  // largest hash of the window's rows combined in LDS (+ a dummy per lane)
  unsigned short kpre[kCStep];       // kept entries of the step before position x
  int stage[kCStep];                 // kept entries of the step
};

// The lane's entries of the step at s; nothing past nnz (>= kCStep) is read.
struct Quad {
  int c[kCIt];
};
__device__ __forceinline__ Quad load_quad(const int* col, int s, int nnz) {
  const int q = s + kCIt * lane_id();
  const int at = min(q, nnz - kCIt);
  int x[kCIt];
#pragma unroll
  for (int j = 0; j < kCIt; j += 4) {
    const i4u y = __builtin_nontemporal_load(reinterpret_cast<const i4u*>(col + at + j));
#pragma unroll
    for (int i = 0; i < 4; ++i) x[j + i] = y[i];
  }
  Quad r;
#pragma unroll
  for (int j = 0; j < kCIt; ++j) r.c[j] = x[j];
  if (s > nnz - kCStep) {  // the entries end inside the step: the last lanes' move down
    const int sh = q - at;
#pragma unroll
    for (int j = 0; j < kCIt; ++j) {
      int y = -1;
#pragma unroll
      for (int i = 0; i < kCIt; ++i) y = j + sh == i ? x[i] : y;
      r.c[j] = y;
    }
  }
  return r;
}

__device__ void compact_unw_range(const StreamArgs& a, const Ctl& ctl, int b, UnwCompactSmem& sm,
                                  unsigned long long S, bool use_bits) {
  const int lane = lane_id();
  const long long* rp = a.in.csr_rp;
  const int* col = a.in.col;
  const int n = a.c.n;
  const int nnz = uni((int)rp[n]);
  const long long cost = ctl.L + (long long)kPieceCostFirst * n;
  const int E0 = uni((int)wave_csr_entry_at(rp, n, cost * b / ctl.P));
  const int E1 = uni((int)wave_csr_entry_at(rp, n, cost * (b + 1) / ctl.P));
  Part pf = unw_part(-1, 0, false, 0ull, S), pl = pf;
  int out = E0, row0 = 0, rows = 0;
  unsigned loaded = 0u;  // the lane's share of the entries of live rows
  if (E0 < E1) {
    const int v0 = uni((int)wave_lower_bound(0, n, [&](long long v) { return rp[v + 1] > E0; }));
    const bool cut_left = uni((int)rp[v0]) < E0;
    row0 = v0 + b;
    int R0 = v0 & ~63;  // the window: lane i holds row R0 + i
    // (of the window i rows on)
    auto end_of = [&](int r, unsigned i) { return (int)rp[row_or_end(r, i + (unsigned)lane + 1u, n)]; };
    auto state_of = [&](int r, unsigned i) {
      const unsigned v = row_or_end(r, i + (unsigned)lane, n);
      return v < (unsigned)n ? (unsigned)a.c.state[v] : 1u;
    };
    int ce = end_of(R0, 0u), cs;
    unsigned st = state_of(R0, 0u);
    unsigned long long live;
    auto enter = [&](int first) {  // (first: where the window's first row starts)
      cs = (int)dpp_wave_shr1((unsigned)ce, (unsigned)first);
      const bool lv = st == 0u && ce > cs;
      live = __ballot(lv);
      loaded += lv ? (unsigned)max(min(ce, E1) - max(cs, E0), 0) : 0u;
    };
    enter(uni((int)rp[R0]));
    int ne = end_of(R0, 64u);  // the next window
    unsigned ns = state_of(R0, 64u);
    int pos = E0;
    // pos to the first entry of a live row from pos on; false: none in the range
    auto seek = [&]() -> bool {
      for (;;) {
        const unsigned long long m = live & __ballot(ce > pos);
        if (m) {
          pos = max(pos, __builtin_amdgcn_readlane(cs, __ffsll((long long)m) - 1));
          return pos < E1;
        }
        const int last = __builtin_amdgcn_readlane(ce, 63);
        if (row_or_end(R0, 64u, n) == (unsigned)n || last >= E1) return false;
        R0 += 64;
        ce = ne;
        st = ns;
        enter(last);
        ne = end_of(R0, 64u);
        ns = state_of(R0, 64u);
      }
    };
    int orow = -1, ostart = E0;   // the row open at the end of the previous step, its first kept entry
    unsigned long long acc = 0ull;  // the lane's largest hash in it
    // a row of the range is finished
    auto finish = [&](bool right) {  // (right: it goes on past the range)
      const int len = out - ostart;
      const bool cl = orow == v0 && cut_left;
      if (len > 0) {
        const unsigned long long h = wave_max_u64(acc);
        const int at = row0 + rows++;
        if (lane == 0) {
          a.rows_out[at] = make_int4(orow, ostart, len, cl || right ? 0 : kHeadBit);
          if (!cl && !right) a.c.C[orow] = hash_neighbour(h, S, (unsigned)orow);
        }
        if (cl || right) {
          Part p = unw_part(orow, cl && right ? kPartSingle : 0, true, h, S);
          p.kept = len;
          p.out_row = at;
          if (cl) pf = p;
          else pl = p;
        }
      } else if (cl || right) {
        const Part p = unw_part(orow, cl && right ? kPartSingle : 0, false, 0ull, S);
        if (cl) pf = p;
        else pl = p;
      }
      acc = 0ull;
      orow = -1;
    };
    // one step over the entries cv holds if it was loaded at pos; two buffers
    // alternate, so a load in flight is never copied
    auto step = [&](Quad& cv, int cvat, Quad& nxt, int& nxat) {
      if (cvat != pos) cv = load_quad(col, pos, nnz);
      const int s = pos;
      const int se = min(min(s + kCStep, E1), __builtin_amdgcn_readlane(ce, 63));
      const int rpos = (int)__popcll(__ballot(ce <= s)), rlast = (int)__popcll(__ballot(ce < se));
      if (orow >= 0 && orow != R0 + rpos) finish(false);
      if (orow < 0) {
        orow = R0 + rpos;
        ostart = out;
      }
      int rr[kCIt];
      bool ok[kCIt];
      if (rpos == rlast) {
#pragma unroll
        for (int j = 0; j < kCIt; ++j) {
          rr[j] = rpos;
          ok[j] = kCIt * lane + j < se - s && (unsigned)cv.c[j] < (unsigned)n;
        }
      } else {  // rows from the boundary markers (all zero between steps)
        const int cn = (int)dpp_wave_shl1((unsigned)ce, 0u);
        // row R0 + lane + 1 starts at ce (the last of several rows starting there: the others are empty)
        if (ce > s && ce < se && (lane == 63 || cn > ce)) sm.mark[ce - s] = (unsigned)(lane + 2);
        wave_lds_sync();
        unsigned m[kCIt];
#pragma unroll
        for (int j = 0; j < kCIt; j += 4) {
          const uint4 mk = *reinterpret_cast<const uint4*>(&sm.mark[kCIt * lane + j]);
          *reinterpret_cast<uint4*>(&sm.mark[kCIt * lane + j]) = make_uint4(0u, 0u, 0u, 0u);
          m[j] = mk.x;
          m[j + 1] = mk.y;
          m[j + 2] = mk.z;
          m[j + 3] = mk.w;
        }
#pragma unroll
        for (int j = 1; j < kCIt; ++j) m[j] = max(m[j], m[j - 1]);
        const unsigned excl = dpp_wave_shr1(wave_incl_max_u32(m[kCIt - 1]), 0u);
#pragma unroll
        for (int j = 0; j < kCIt; ++j) {
          rr[j] = max(rpos, (int)max(excl, m[j]) - 1);
          ok[j] = kCIt * lane + j < se - s && (unsigned)cv.c[j] < (unsigned)n && ((live >> rr[j]) & 1ull) != 0ull;
        }
      }
      unsigned gw[kCIt];
      if (use_bits) {
#pragma unroll
        for (int j = 0; j < kCIt; ++j) gw[j] = a.c.mbits[(ok[j] ? (unsigned)cv.c[j] : 0u) >> 5];
      } else {
#pragma unroll
        for (int j = 0; j < kCIt; ++j) gw[j] = a.c.state[ok[j] ? cv.c[j] : 0];
      }
      {  // the next step's entries: at the first live row from se on
        const unsigned long long m = live & __ballot(ce > se);
        int at = se;
        if (m) {
          at = max(se, __builtin_amdgcn_readlane(cs, __ffsll((long long)m) - 1));
        } else {
          const int ncs = (int)dpp_wave_shr1((unsigned)ne, (unsigned)__builtin_amdgcn_readlane(ce, 63));
          const unsigned long long mn = __ballot(ns == 0u && ne > ncs);
          if (mn) at = __builtin_amdgcn_readlane(ncs, __ffsll((long long)mn) - 1);
        }
        nxat = at;
        nxt = load_quad(col, min(at, nnz - 1), nnz);
      }
      unsigned long long hv[kCIt];
#pragma unroll
      for (int j = 0; j < kCIt; ++j) hv[j] = keep(edge_hash(S, (unsigned)(R0 + rr[j]), (unsigned)cv.c[j]));
      unsigned k = 0u;
#pragma unroll
      for (int j = 0; j < kCIt; ++j) {
        const unsigned g = use_bits ? gw[j] >> ((unsigned)cv.c[j] & 31u) & 1u : gw[j];
        ok[j] = ok[j] && g == 0u;
        hv[j] = ok[j] ? hv[j] : 0ull;
        k += ok[j] ? 1u : 0u;
      }
      const unsigned incl = wave_incl_sum_u32(k), excl = incl - k;
      const int tot = __builtin_amdgcn_readlane((int)incl, 63);
      {
        unsigned x = excl;
#pragma unroll
        for (int j = 0; j < kCIt; ++j)
          if (ok[j]) sm.stage[x++] = cv.c[j];
      }
      if (rpos == rlast) {
#pragma unroll
        for (int j = 0; j < kCIt; ++j) acc = hv[j] > acc ? hv[j] : acc;
        wave_lds_sync();
      } else {
        {
          unsigned x = excl;
#pragma unroll
          for (int j = 0; j < kCIt; ++j) {
            sm.kpre[kCIt * lane + j] = (unsigned short)x;
            x += ok[j] ? 1u : 0u;
          }
        }
        // Runs of one row among the lane's entries (rows never decrease along
        // them), the lane's maximum of the row of pos first. Every run but the
        // one of the step's last row ends in an LDS atomic max on its row's slot,
        // or on the lane's dummy.
        unsigned long long rm = acc;
        int prow = rpos;
#pragma unroll
        for (int j = 0; j < kCIt; ++j) {
          const bool same = rr[j] == prow;
          const bool fl = !same && rm != 0ull;
          if (__ballot(fl)) atomicMax(&sm.slot[fl ? prow : 64 + lane], rm);
          rm = same && rm > hv[j] ? rm : hv[j];
          prow = rr[j];
        }
        const bool open = prow == rlast;
        const bool fl = !open && rm != 0ull;
        if (__ballot(fl)) atomicMax(&sm.slot[fl ? prow : 64 + lane], rm);
        acc = open ? rm : 0ull;
        wave_lds_sync();
        // rows of the window that ended inside the step: rpos .. rlast - 1
        const bool mine = lane >= rpos && lane < rlast;
        const int oe = mine ? out + (int)sm.kpre[ce - s] : out;
        const int before = (int)dpp_wave_shr1((unsigned)oe, 0u);  // (on every lane: not under a condition)
        const int os = lane == rpos ? ostart : before;
        const int len = mine ? oe - os : 0;
        const unsigned long long hh = mine ? sm.slot[lane] : 0ull;
        const unsigned long long put = __ballot(len > 0);
        const int at = row0 + rows + (int)__popcll(put & lanemask_lt());
        const bool fc = mine && cut_left && R0 + lane == v0;
        if (len > 0) {
          a.rows_out[at] = make_int4(R0 + lane, os, len, fc ? 0 : kHeadBit);
          if (!fc) a.c.C[R0 + lane] = hash_neighbour(hh, S, (unsigned)(R0 + lane));
        }
        if (__ballot(fc) != 0ull) {  // v0's part
          const int l0 = v0 - R0;
          const int kl = __builtin_amdgcn_readlane(len, l0);
          const unsigned long long h0 = (unsigned long long)rdl64((long long)hh, l0);
          pf = unw_part(v0, 0, kl > 0, h0, S);
          if (kl > 0) {
            pf.kept = kl;
            pf.out_row = __builtin_amdgcn_readlane(at, l0);
          }
        }
        rows += (int)__popcll(put);
        ostart = __builtin_amdgcn_readlane(oe, rlast - 1);
        sm.slot[mine ? lane : 64 + lane] = 0ull;
        orow = (live >> rlast) & 1ull ? R0 + rlast : -1;
      }
      for (int x = lane; x < tot; x += 64) a.dst_col[out + x] = sm.stage[x];
      wave_lds_sync();  // the staged entries and cleared slots before the next step's
      out += tot;
      pos = se;
    };
    if (seek()) {
      int atA = pos, atB = 0;
      Quad A = load_quad(col, pos, nnz), B;
      for (;;) {
        step(A, atA, B, atB);
        if (!seek()) break;
        step(B, atB, A, atA);
        if (!seek()) break;
      }
      if (orow >= 0) finish(uni((int)rp[orow + 1]) > E1);
    }
  }
  loaded = wave_incl_sum_u32(loaded);
  if (lane == 63) {
    a.parts[2 * b] = pf;
    a.parts[2 * b + 1] = pl;
    Run r;
    r.row_begin = row0;
    r.row_count = rows;
    r.phys_begin = E0;
    r.ent_count = out - E0;
    a.runs_out[b] = r;
    BlockStat bs;
    bs.loaded = loaded;
    bs.matched_len = (long long)(E1 - E0) - loaded;
    bs.pieces_out = rows;
    bs.pad = 0;
    a.bstat[b] = bs;
  }
}

}  // namespace

__global__ __launch_bounds__(64, 4) void k_compact_unw(StreamArgs a) {
  __shared__ UnwCompactSmem sm;
  const Totals* t = a.c.totals;
  if (uni((int)(t->err | (handed_over(a.c, t->tail_from) ? 0x80000000u : 0u))) != 0) return;
  const Ctl ctl = *a.in.ctl;
  const int lane = lane_id();
  const unsigned long long S = cand_seed(a.c.gseed[0], a.c.renew, a.cand_phase);
  const bool use_bits = a.c.mbits && bits_on(t);
  for (int x = lane; x < kCStep; x += 64) sm.mark[x] = 0u;
  for (int x = lane; x < 128; x += 64) sm.slot[x] = 0ull;
  wave_lds_sync();
  for (int b = blockIdx.x; b < ctl.P; b += gridDim.x) compact_unw_range(a, ctl, b, sm, S, use_bits);
}

hipError_t launch_compact_unw(const StreamArgs& a, int grid, hipStream_t s, hipEvent_t* ev) {
  if (ev) hipExtLaunchKernelGGL(k_compact_unw, dim3(grid), dim3(64), 0, s, ev[0], ev[1], 0, a);
  else hipLaunchKernelGGL(k_compact_unw, dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}

int compact_unw_per_cu() { return kCPerCu; }
int compact_unw_min_entries() { return kCStep; }

}  // namespace lm
