// Direction-optimised BFS (Algorithm 1 and Section 7.1 of the paper) with
// one kernel per level.
//
// Each level is f <- A^T f .* not(visited) over the Boolean semiring, run as
// push (SpMSpV from the frontier's out-edges) or pull (masked SpMV over the
// unvisited rows, stopping a row at its first frontier neighbour), chosen on
// the device from the frontier's size and degree sum (the switch rule of the
// descriptor).  The frontier is only a bitmap, and one kernel does all of a
// level, so nothing sits between levels:
// * push gives each wave a run of frontier words and streams the out-edges
//   of its frontier rows as one concatenated list (the same wave-level
//   load-balanced search as pull); rows longer than kPushSplit come from a
//   static list of kPushSplit-edge pieces built by grb_matrix_prepare,
//   spread over all waves, each piece active when its row is in the
//   frontier;
// * a vertex is claimed by the first atomicOr on its visited bit; the
//   claimer writes its level and sets its bit in the next frontier bitmap;
// * the next frontier's size and degree sum are reduced per workgroup and
//   added into kCntStripes striped counters (few atomics per address);
// * bitmaps and counters rotate through three buffers: the level reads
//   buffer d, fills buffer d+1 and clears buffer d+2.
// Pull finds the smallest-id parent directly (ascending adjacency, first
// hit).  A push from a one-vertex frontier writes that vertex as parent.
// Vertices found by a push of several vertices get theirs in the next
// level's kernel, where they are the frontier: the smallest in-neighbour
// one level up, offered edge by edge while that level pushes over the same
// CSR, else found by a pass over their in-edges (first hit in ascending
// order); a standalone pass covers the last level when the level cap stops
// the search.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "grb_device.h"
#include "grb_internal.h"

namespace grb {
namespace {

__device__ __forceinline__ int decide(const BfsArgs &a, int64_t count, int64_t sumdeg) {
  if (a.forced) return a.forced;
  if (!a.can_pull) return GRB_DIR_PUSH;
  const bool pull = a.rule == GRB_SWITCH_EXACT ? (int64_t)a.denom * sumdeg > a.nnz
                                               : (int64_t)a.denom * count > a.n;
  return pull ? GRB_DIR_PULL : GRB_DIR_PUSH;
}

// Finishes the claims won by this lane: level, next-frontier bit, counts.
// dg[s]: out-degree of target c[s], loaded by the caller together with its
// visited word (before the claim is decided, so no load follows it).
// With a one-vertex frontier (`single`) that vertex, par[s], is the only
// parent a target can have, and it is written at once.
// `next_set`: the caller has already set the targets' next-frontier bits.
__device__ __forceinline__ void claim_won(const BfsArgs &a, const int (&c)[kUnroll],
                                          const bool (&won)[kUnroll], const int (&par)[kUnroll],
                                          const int (&dg)[kUnroll], bool single, bool next_set,
                                          int &fc, int &fd, int &fl) {
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    if (won[s]) {
      a.levels[c[s]] = a.d + 1;
      if (single && a.parents) a.parents[c[s]] = par[s];
      if (!next_set)
        atomicOr((unsigned long long *)&a.fnxt[c[s] >> 6], 1ull << (c[s] & 63));
      fc += 1;
      fd += dg[s];
      fl += dg[s] > kPushSplit ? 1 : 0;
    }
  }
}

// Row extents of the targets still unvisited at the filter read (0 for the
// others: a visited target cannot be won), issued beside the claim atomics,
// whose latency covers theirs.
__device__ __forceinline__ void target_degrees(const BfsArgs &a, const int (&c)[kUnroll],
                                               const bool (&open)[kUnroll], int (&d0)[kUnroll],
                                               int (&d1)[kUnroll]) {
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    d0[s] = open[s] ? a.push.rp[c[s]] : 0;
    d1[s] = open[s] ? a.push.rp[c[s] + 1] : 0;
  }
}

// Parents of the frontier while a push expands it (symmetric graphs, whose
// out-edges are the in-edges): an expanded edge (u, v) with v one level
// above u offers v as u's parent, and the smallest offer wins (parents[u]
// is -1 until then, the largest value as unsigned).  lv[s]: level of c[s],
// loaded by the caller together with its visited words.
__device__ __forceinline__ void offer_parents(const BfsArgs &a, const int (&c)[kUnroll],
                                              const int (&par)[kUnroll], const int (&lv)[kUnroll]) {
#pragma unroll
  for (int s = 0; s < kUnroll; ++s)
    if (c[s] >= 0 && lv[s] == a.d - 1)
      atomicMin((unsigned int *)&a.parents[par[s]], (unsigned int)c[s]);
}

// Claims the targets c[0..kUnroll) (-1: none) from a stream that may hold
// one target twice.  The visited words of all of them are read first (a
// plain read is only a filter, the atomic decides) and all atomics are
// issued before any result is used, so their latencies overlap; the row
// extents of the unvisited targets are loaded beside them.
__device__ __forceinline__ void claim_batch(const BfsArgs &a, const int (&c)[kUnroll],
                                            const int (&par)[kUnroll], bool single, bool offer,
                                            int &fc, int &fd, int &fl) {
  uint64_t vw[kUnroll];
  int lv[kUnroll], d0[kUnroll], d1[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    vw[s] = c[s] >= 0 ? a.visited[c[s] >> 6] : ~0ull;
    lv[s] = (offer && c[s] >= 0) ? a.levels[c[s]] : -2;
  }
  if (offer) offer_parents(a, c, par, lv);
  bool open[kUnroll];
  uint64_t old[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    open[s] = c[s] >= 0 && !((vw[s] >> (c[s] & 63)) & 1ull);
    old[s] = ~0ull;
    if (open[s])
      old[s] = atomicOr((unsigned long long *)&a.visited[c[s] >> 6], 1ull << (c[s] & 63));
  }
  target_degrees(a, c, open, d0, d1);
  bool won[kUnroll];
  int dg[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    won[s] = c[s] >= 0 && !((old[s] >> (c[s] & 63)) & 1ull);
    dg[s] = d1[s] - d0[s];
  }
  claim_won(a, c, won, par, dg, single, false, fc, fd, fl);
}

// Claims the targets of one piece of a row: ascending and distinct, so the
// lanes whose targets share a visited word sit side by side and one atomicOr
// per word serves them all (issued by the run's last lane, whose previous
// value of the word every lane of the run then reads).
__device__ __forceinline__ void claim_piece(const BfsArgs &a, const int (&c)[kUnroll],
                                            const int (&par)[kUnroll], bool single, bool offer,
                                            int &fc, int &fd, int &fl) {
  uint64_t vw[kUnroll];
  int lv[kUnroll], d0[kUnroll], d1[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    vw[s] = c[s] >= 0 ? a.visited[c[s] >> 6] : ~0ull;
    lv[s] = (offer && c[s] >= 0) ? a.levels[c[s]] : -2;
  }
  if (offer) offer_parents(a, c, par, lv);
  bool want[kUnroll];
  uint64_t old[kUnroll], run[kUnroll];
  int64_t wd[kUnroll];
  int tail[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    want[s] = c[s] >= 0 && !((vw[s] >> (c[s] & 63)) & 1ull);
    wd[s] = want[s] ? (int64_t)(c[s] >> 6) : -1;
    run[s] = run_tail_or(wd[s], want[s] ? (1ull << (c[s] & 63)) : 0ull, tail[s]);
    old[s] = 0ull;
    if (run[s] && wd[s] >= 0)
      old[s] = atomicOr((unsigned long long *)&a.visited[wd[s]], (unsigned long long)run[s]);
  }
  target_degrees(a, c, want, d0, d1);
  bool won[kUnroll];
  int dg[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    const uint64_t ow = __shfl(old[s], tail[s]);
    won[s] = want[s] && !((ow >> (c[s] & 63)) & 1ull);
    dg[s] = d1[s] - d0[s];
    // the run's tail also sets the won bits of the next frontier at once
    if (run[s] && wd[s] >= 0 && (run[s] & ~old[s]))
      atomicOr((unsigned long long *)&a.fnxt[wd[s]], (unsigned long long)(run[s] & ~old[s]));
  }
  claim_won(a, c, won, par, dg, single, true, fc, fd, fl);
}

// Each wave loads 64 bitmap words at once (one per lane) and compacts their
// set bits into a queue of rows, taken 64 at a time (one row per lane).  The
// edges of rows up to kPushSplit (push) or kHeavyDeg (pull) long are streamed
// as one concatenated list; longer rows come in static pieces spread over
// all waves, so a hub is expanded by hundreds of waves at once.

__device__ __forceinline__ void bfs_push(const BfsArgs &a, int *mark, bool long_rows, bool single,
                                         bool offer, int &fc, int &fd, int &fl) {
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *rp = a.push.rp, *ci = a.push.ci;
  // words dealt out round-robin (wave gw takes words gw, gw + nwaves, ...)
  // so that runs of high-degree rows spread over the waves
  for (int64_t w0 = gw; w0 < a.nw; w0 += 64 * nwaves) {
    const int64_t mw = w0 + (int64_t)ln * nwaves;
    uint64_t mf = 0ull;
    if (mw < a.nw) {
      a.fclr[mw] = 0ull;  // the bitmap two levels ahead
      mf = a.fcur[mw];
    }
    const int cnt = __popcll(mf);
    const int incl = wave_incl_scan(cnt);
    const int total = lane_last(incl);
    for (int b = 0; b < total; b += 64) {
      const int64_t u = queue_slot(mark, mf, cnt, incl, total, b, mw);
      int cur = 0, end = 0;
      if (u >= 0) {
        cur = rp[u];
        end = rp[u + 1];
        if (end - cur > kPushSplit) end = cur;  // long rows: static pieces below
      }
      // the rows' out-edges as one concatenated stream, kUnroll x 64 edges
      // per step
      const int uid = (int)u;
      for (bool more = true; more;) {
        int c[kUnroll], par[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          c[s] = -1;
          par[s] = -1;
          if (!more) continue;
          const int len = end - cur;
          const int incl2 = wave_incl_scan(len);
          const int tot2 = lane_last(incl2);
          if (tot2 == 0) {
            more = false;
            continue;
          }
          const int excl = incl2 - len;
          const bool starts = len > 0 && excl < 64;
          const int r = slot_rows(mark, starts, excl);
          const int rcur = __shfl(cur, r), rexcl = __shfl(excl, r);
          par[s] = __shfl(uid, r);
          if (ln < tot2) c[s] = rcur + (ln - rexcl);
          if (starts) cur += min(incl2, 64) - excl;
        }
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) c[s] = c[s] >= 0 ? ci[c[s]] : -1;
        claim_batch(a, c, par, single, offer, fc, fd, fl);
      }
    }
  }
  // static pieces of long rows, spread over the waves (wave gw owns pieces
  // gw, gw + nwaves, ...), 64 tested per step; a piece whose row is in the
  // frontier is streamed by the whole wave, kUnroll x 64 edges at once
  static_assert(kPushSplit == 64 * kUnroll, "a push piece is one unrolled step");
  if (!long_rows) return;  // no row of the frontier has pieces
  for (int64_t hb = gw; hb < a.push.nsplit; hb += 64 * nwaves) {
    const int64_t h = hb + (int64_t)ln * nwaves;
    int u = -1, b = 0, e = 0;
    if (h < a.push.nsplit) {
      u = a.push.split[2 * h];
      b = a.push.split[2 * h + 1];
      if (bit_of(a.fcur, u)) e = min(b + kPushSplit, rp[u + 1]);
      else u = -1;
    }
    uint64_t act = __ballot(u >= 0);
    while (act) {
      const int k = __ffsll((unsigned long long)act) - 1;
      act &= act - 1;
      const int pb = __shfl(b, k), pe = __shfl(e, k), pu = __shfl(u, k);
      int c[kUnroll], par[kUnroll];
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) {
        const int pos = pb + s * 64 + ln;
        c[s] = pos < pe ? ci[pos] : -1;
        par[s] = pu;
      }
      claim_piece(a, c, par, single, offer, fc, fd, fl);
    }
  }
}

// Records rows found in a pull: rows of one bitmap word sit in consecutive
// lanes (ascending ids), so one atomicOr per word and bitmap serves them.
__device__ __forceinline__ void pull_found(const BfsArgs &a, bool found, int64_t v, int par,
                                           int deg, int &fc, int &fd, int &fl) {
  const int64_t vw = found ? (v >> 6) : -1;
  int tail;
  const uint64_t hb = run_tail_or(vw, found ? (1ull << (v & 63)) : 0ull, tail);
  if (hb && vw >= 0) {
    atomicOr((unsigned long long *)&a.visited[vw], (unsigned long long)hb);
    atomicOr((unsigned long long *)&a.fnxt[vw], (unsigned long long)hb);
  }
  if (found) {
    a.levels[v] = a.d + 1;
    if (a.parents) a.parents[v] = par;
    const int pd = a.same_csr ? deg : a.push.rp[v + 1] - a.push.rp[v];
    fc += 1;
    fd += pd;
    fl += pd > kPushSplit ? 1 : 0;
  }
}

// Pull stream of the unsettled rows (one per lane: `act`, remaining
// positions [rc, re)) as one concatenated list, K steps of 64 positions
// laid out and loaded at once (K > 1 when the probes found the frontier
// sparse, so that rows rarely stop early); the steps are then read in
// order, so a row's first frontier neighbour (its smallest id: columns
// ascend) is its parent.
template <int K>
__device__ __forceinline__ void pull_stream(const BfsArgs &a, int *mark, bool act, int &rc, int re,
                                            bool &found, int &par) {
  const int ln = threadIdx.x & 63;
  const int32_t *ci = a.pull.ci;
  for (bool more = true; more;) {
    int pos[K], sev[K], exv[K];
    bool st[K];
#pragma unroll
    for (int s = 0; s < K; ++s) {
      pos[s] = -1;
      sev[s] = exv[s] = 0;
      st[s] = false;
      if (!more) continue;
      const int len = (act && !found) ? re - rc : 0;
      const int incl = wave_incl_scan(len);
      const int total = lane_last(incl);
      if (total == 0) {
        more = false;
        continue;
      }
      const int excl = incl - len;
      const bool starts = len > 0 && excl < 64;
      const int r = slot_rows(mark, starts, excl);
      const int rcur = __shfl(rc, r), rexcl = __shfl(excl, r);
      if (ln < total) pos[s] = rcur + (ln - rexcl);
      sev[s] = min(incl, 64);
      exv[s] = excl;
      st[s] = starts;
      if (starts) rc += sev[s] - excl;
    }
    int c[K];
#pragma unroll
    for (int s = 0; s < K; ++s) c[s] = pos[s] >= 0 ? ci[pos[s]] : -1;
    uint64_t fw[K];
#pragma unroll
    for (int s = 0; s < K; ++s) fw[s] = c[s] >= 0 ? a.fcur[c[s] >> 6] : 0ull;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const uint64_t hm = __ballot(c[s] >= 0 && ((fw[s] >> (c[s] & 63)) & 1ull));
      const uint64_t seg = st[s] ? (mask_below(sev[s]) & ~mask_below(exv[s])) : 0ull;
      const uint64_t h = hm & seg;
      const int first = h ? (__ffsll((unsigned long long)h) - 1) : 0;
      const int pc = __shfl(c[s], first);
      if (h && !found) {
        found = true;
        par = pc;
      }
    }
  }
}

__device__ __forceinline__ void bfs_pull(const BfsArgs &a, int *mark, int &fc, int &fd, int &fl) {
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *rp = a.pull.rp, *ci = a.pull.ci;
  int64_t lo, hi;
  wave_words(a.nw, gw, nwaves, lo, hi);
  for (int64_t w0 = lo; w0 < hi; w0 += 64) {
    const int64_t mw = w0 + ln;
    uint64_t mc = 0ull;  // candidate rows: not visited
    if (mw < hi) {
      a.fclr[mw] = 0ull;
      mc = ~a.visited[mw];
    }
    const int cnt = __popcll(mc);
    const int incl = wave_incl_scan(cnt);
    const int total = lane_last(incl);
    // kPullRows queued rows per lane: the loads of their first two
    // neighbours are issued together
    for (int b = 0; b < total; b += 64 * kPullRows) {
      int64_t v[kPullRows];
      int cur[kPullRows], end[kPullRows];
      bool act[kPullRows];
#pragma unroll
      for (int q = 0; q < kPullRows; ++q) {
        v[q] = b + q * 64 < total ? queue_slot(mark, mc, cnt, incl, total, b + q * 64, mw) : -1;
        act[q] = v[q] >= 0;
      }
      // row extents and the first two neighbours (a separate array read
      // in row order), all issued together
      int c0[kPullRows], c1[kPullRows];
#pragma unroll
      for (int q = 0; q < kPullRows; ++q) {
        cur[q] = act[q] ? rp[v[q]] : 0;
        end[q] = act[q] ? rp[v[q] + 1] : 0;
        const int2 f = act[q] ? a.pull.first2[v[q]] : make_int2(-1, -1);
        c0[q] = f.x;
        c1[q] = f.y;
      }
#pragma unroll
      for (int q = 0; q < kPullRows; ++q)
        if (end[q] - cur[q] > kHeavyDeg || end[q] == cur[q]) {  // pieces / empty
          act[q] = false;
          c0[q] = c1[q] = -1;
        }
      uint64_t b0[kPullRows], b1[kPullRows];
#pragma unroll
      for (int q = 0; q < kPullRows; ++q) {
        b0[q] = c0[q] >= 0 ? a.fcur[c0[q] >> 6] : 0ull;
        b1[q] = c1[q] >= 0 ? a.fcur[c1[q] >> 6] : 0ull;
      }
      // rows settled by their first two neighbours; the others (with more
      // edges left) are counted per batch for the stream below
      uint64_t rest[kPullRows];
      int nrest = 0, np = 0, nh = 0;
#pragma unroll
      for (int q = 0; q < kPullRows; ++q) {
        bool found = false;
        int par = -1;
        const bool h0 = c0[q] >= 0 && ((b0[q] >> (c0[q] & 63)) & 1ull);
        const bool h1 = c1[q] >= 0 && ((b1[q] >> (c1[q] & 63)) & 1ull);
        np += __popcll(__ballot(c0[q] >= 0)) + __popcll(__ballot(c1[q] >= 0));
        nh += __popcll(__ballot(h0)) + __popcll(__ballot(h1));
        if (h0) {
          found = true;
          par = c0[q];
        } else if (h1) {
          found = true;
          par = c1[q];
        }
        pull_found(a, found, v[q], par, end[q] - cur[q], fc, fd, fl);
        rest[q] = __ballot(act[q] && !found && end[q] - cur[q] > 2);
        nrest += __popcll(rest[q]);
      }
      // the unsettled rows of all batches, compacted 64 at a time, stream
      // their remaining edges as one concatenated list with early exit
      for (int sb = 0; sb < nrest; sb += 64) {
        const int j = sb + ln;  // this lane's place among the unsettled rows
        int64_t rv = -1;
        int rc = 0, re = 0;
        int before = 0;
#pragma unroll
        for (int q = 0; q < kPullRows; ++q) {
          const int cq = __popcll(rest[q]);
          const int li = (j >= before && j < before + cq) ? nth_set_bit(rest[q], j - before) : 0;
          const int64_t sv = __shfl(v[q], li);
          const int sc = __shfl(cur[q], li), se_ = __shfl(end[q], li);
          if (j >= before && j < before + cq) {
            rv = sv;
            rc = sc + 2;
            re = se_;
          }
          before += cq;
        }
        const bool act2 = rv >= 0;
        const int deg2 = re - (rc - 2);
        bool found = false;
        int par = -1;
        // a frontier the probes found below 1/8 dense: four steps at once
        if (8 * nh < np) pull_stream<kUnroll>(a, mark, act2, rc, re, found, par);
        else pull_stream<1>(a, mark, act2, rc, re, found, par);
        pull_found(a, found, rv, par, deg2, fc, fd, fl);
      }
    }
  }
  // pieces of long rows; a row counts as a candidate unless it was reached
  // before this level (its level is then 0..d): a piece's claim must not
  // hide the row from its other pieces, whose first frontier neighbour may
  // have a smaller id.  kUnroll x 64 edges are loaded at once and searched
  // for the first frontier neighbour in order; the parent is the minimum
  // over the pieces.
  // Wave gw owns pieces gw, gw + nwaves, ...: 64 of them are tested at once
  // (one per lane), then the wave streams the live ones.
  for (int64_t hb = gw; hb < a.pull.nheavy; hb += 64 * nwaves) {
    const int64_t hh = hb + (int64_t)ln * nwaves;
    int hr = -1, hbeg = 0, hend = 0;
    if (hh < a.pull.nheavy) {
      hr = a.pull.heavy[2 * hh];
      hbeg = a.pull.heavy[2 * hh + 1];
      const int lr = a.levels[hr];
      if (lr >= 0 && lr <= a.d) hr = -1;
      else hend = min(hbeg + kHeavyChunk, rp[hr + 1]);
    }
    uint64_t live = __ballot(hr >= 0);
    while (live) {
      const int k = __ffsll((unsigned long long)live) - 1;
      live &= live - 1;
      const int r = __shfl(hr, k), b = __shfl(hbeg, k), e = __shfl(hend, k);
      for (int base = b; base < e; base += 64 * kUnroll) {
        int c[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          const int pos = base + s * 64 + ln;
          c[s] = pos < e ? ci[pos] : -1;
        }
        uint64_t fwd[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) fwd[s] = c[s] >= 0 ? a.fcur[c[s] >> 6] : 0ull;
        int pc = -1;
#pragma unroll
        for (int s = kUnroll - 1; s >= 0; --s) {
          const uint64_t hm = __ballot(c[s] >= 0 && ((fwd[s] >> (c[s] & 63)) & 1ull));
          if (hm) pc = __shfl(c[s], __ffsll((unsigned long long)hm) - 1);
        }
        if (pc >= 0) {
          if (ln == 0) {
            const uint64_t bit = 1ull << (r & 63);
            const uint64_t old =
                atomicOr((unsigned long long *)&a.visited[r >> 6], (unsigned long long)bit);
            if (a.parents) atomicMin((unsigned *)&a.parents[r], (unsigned)pc);
            if (!(old & bit)) {
              a.levels[r] = a.d + 1;
              atomicOr((unsigned long long *)&a.fnxt[r >> 6], (unsigned long long)bit);
              const int pd = a.push.rp[r + 1] - a.push.rp[r];
              fc += 1;
              fd += pd;
              fl += pd > kPushSplit ? 1 : 0;
            }
          }
          break;
        }
      }
    }
  }
}

// Smallest-id parent of every vertex reached by a push: the first
// in-neighbour (ascending) whose level is one less.  A wave compacts the
// vertices that need a parent in 8 words of its run into a queue, 64 at a
// time; the first two in-neighbours of every queued row are tested in
// parallel, the rest streamed as one concatenated list.
__device__ __forceinline__ void parents_pass(const BfsArgs &a, int *mark) {
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *rp = a.pull.rp, *ci = a.pull.ci;
  int64_t lo, hi;
  wave_words(a.nw, gw, nwaves, lo, hi);
  for (int64_t w0 = lo; w0 < hi; w0 += 8) {
    // the vertices of 8 words that still need a parent: reached (level > 0)
    // and without one; all 16 loads per lane are issued together
    uint64_t nm[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t v = (w0 + k) * 64 + ln;
      const bool inb = w0 + k < hi && v < a.n;
      const int lv = inb ? a.levels[v] : -1;
      const int pv = inb ? a.parents[v] : 0;
      nm[k] = __ballot(lv > 0 && pv < 0);
    }
    uint64_t mq = 0ull;  // lane k < 8 holds word w0 + k's mask
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (ln == k) mq = nm[k];
    const int cnt = __popcll(mq);
    const int incl = wave_incl_scan(cnt);
    const int total = lane_last(incl);
    for (int b = 0; b < total; b += 64) {
      const int64_t v = queue_slot(mark, mq, cnt, incl, total, b, w0 + ln);
      const bool need = v >= 0;
      int cur = need ? rp[v] : 0;
      const int end = need ? rp[v + 1] : 0;
      const int tgt = need ? a.levels[v] - 1 : -3;
      bool found = false;
      int par = -1;
      if (need) {
        const int2 f = a.pull.first2[v];
        const int c0 = f.x;
        const int c1 = f.y;
        const int l0 = c0 >= 0 ? a.levels[c0] : -2;
        const int l1 = c1 >= 0 ? a.levels[c1] : -2;
        if (l0 == tgt) { found = true; par = c0; }
        else if (l1 == tgt) { found = true; par = c1; }
        cur = min(cur + 2, end);
      }
      for (;;) {
        const int len = (need && !found) ? end - cur : 0;
        const int incl2 = wave_incl_scan(len);
        const int tot2 = lane_last(incl2);
        if (tot2 == 0) break;
        const int excl = incl2 - len;
        const bool starts = len > 0 && excl < 64;
        const int r = slot_rows(mark, starts, excl);
        const int rcur = __shfl(cur, r), rexcl = __shfl(excl, r), rt = __shfl(tgt, r);
        const bool valid = ln < tot2;
        const int c = valid ? ci[rcur + (ln - rexcl)] : -1;
        const uint64_t hm = __ballot(valid && a.levels[c] == rt);
        const int se = min(incl2, 64);
        const uint64_t seg = starts ? (mask_below(se) & ~mask_below(excl)) : 0ull;
        const uint64_t h = hm & seg;
        const int fl = h ? (__ffsll((unsigned long long)h) - 1) : 0;
        const int pc = __shfl(c, fl);
        if (h) { found = true; par = pc; }
        if (starts) cur += se - excl;
      }
      if (found) a.parents[v] = par;
    }
  }
}

// Parents of this level's frontier when a push of more than one vertex
// found it: for each frontier vertex v (queued from the frontier words, dealt
// out round-robin), the first in-neighbour one level up in ascending order.
__device__ __forceinline__ void frontier_parents(const BfsArgs &a, int *mark) {
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *rp = a.pull.rp, *ci = a.pull.ci;
  const int tgt = a.d - 1;
  for (int64_t w0 = gw; w0 < a.nw; w0 += 64 * nwaves) {
    const int64_t mw = w0 + (int64_t)ln * nwaves;
    const uint64_t mf = mw < a.nw ? a.fcur[mw] : 0ull;
    const int cnt = __popcll(mf);
    const int incl = wave_incl_scan(cnt);
    const int total = lane_last(incl);
    for (int b = 0; b < total; b += 64) {
      const int64_t v = queue_slot(mark, mf, cnt, incl, total, b, mw);
      const bool need = v >= 0;
      int cur = need ? rp[v] : 0;
      const int end = need ? rp[v + 1] : 0;
      bool found = false;
      int par = -1;
      if (need) {
        const int2 f = a.pull.first2[v];
        const int c0 = f.x;
        const int c1 = f.y;
        const int l0 = c0 >= 0 ? a.levels[c0] : -2;
        const int l1 = c1 >= 0 ? a.levels[c1] : -2;
        if (l0 == tgt) { found = true; par = c0; }
        else if (l1 == tgt) { found = true; par = c1; }
        cur = min(cur + 2, end);
      }
      for (;;) {
        const int len = (need && !found) ? end - cur : 0;
        const int incl2 = wave_incl_scan(len);
        const int tot2 = lane_last(incl2);
        if (tot2 == 0) break;
        const int excl = incl2 - len;
        const bool starts = len > 0 && excl < 64;
        const int r = slot_rows(mark, starts, excl);
        const int rcur = __shfl(cur, r), rexcl = __shfl(excl, r);
        const bool valid = ln < tot2;
        const int c = valid ? ci[rcur + (ln - rexcl)] : -1;
        const uint64_t hm = __ballot(valid && a.levels[c] == tgt);
        const int se = min(incl2, 64);
        const uint64_t seg = starts ? (mask_below(se) & ~mask_below(excl)) : 0ull;
        const uint64_t h = hm & seg;
        const int fl = h ? (__ffsll((unsigned long long)h) - 1) : 0;
        const int pc = __shfl(c, fl);
        if (h) { found = true; par = pc; }
        if (starts) cur += se - excl;
      }
      if (found) a.parents[v] = par;
    }
  }
}

// Parents of the frontier from the previous one: every vertex at level
// d - 1 offers itself (atomicMin) to its out-neighbours at level d, whose
// parents then hold the smallest such id (the claim's winner is one of
// them).  Chosen over the in-edge pass above when the previous frontier's
// degree sum and a scan of the levels cost less than this frontier's
// in-edges.  Rows of at most kPushSplit edges: 64 vertices per wave step,
// the selected rows' edges as one concatenated stream; longer rows through
// the push CSR's pieces, dealt to the waves with a stride.
__device__ __forceinline__ void prev_offers(const BfsArgs &a, int *mark) {
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *rp = a.push.rp, *ci = a.push.ci;
  const int tgt = a.d - 1;
  for (int64_t b0 = gw * 64; b0 < a.n; b0 += nwaves * 64) {
    const int64_t u = b0 + ln;
    const bool sel = u < a.n && a.levels[u] == tgt;
    int cur = sel ? rp[u] : 0;
    const int end = sel ? rp[u + 1] : 0;
    if (end - cur > kPushSplit) cur = end;  // pieces below
    for (;;) {
      const int len = end - cur;
      const int incl = wave_incl_scan(len);
      const int total = lane_last(incl);
      if (total == 0) break;
      const int excl = incl - len;
      const bool starts = len > 0 && excl < 64;
      const int r = slot_rows(mark, starts, excl);
      const int rcur = __shfl(cur, r), rexcl = __shfl(excl, r);
      if (ln < total) {
        const int v = ci[rcur + (ln - rexcl)];
        if (a.levels[v] == a.d) atomicMin((unsigned *)&a.parents[v], (unsigned)(b0 + r));
      }
      if (starts) cur += min(incl, 64) - excl;
    }
  }
  for (int64_t hb = gw; hb < a.push.nsplit; hb += 64 * nwaves) {
    const int64_t h = hb + (int64_t)ln * nwaves;
    int u = -1, b = 0, e = 0;
    if (h < a.push.nsplit) {
      u = a.push.split[2 * h];
      b = a.push.split[2 * h + 1];
      if (a.levels[u] == tgt) e = min(b + kPushSplit, rp[u + 1]);
      else u = -1;
    }
    for (uint64_t act = __ballot(u >= 0); act; act &= act - 1) {
      const int k = __ffsll((unsigned long long)act) - 1;
      const int pb = __shfl(b, k), pe = __shfl(e, k), pu = __shfl(u, k);
      int v[kUnroll];
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) {
        const int pos = pb + s * 64 + ln;
        v[s] = pos < pe ? ci[pos] : -1;
      }
      int lv[kUnroll];
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) lv[s] = v[s] >= 0 ? a.levels[v[s]] : -1;
#pragma unroll
      for (int s = 0; s < kUnroll; ++s)
        if (lv[s] == a.d) atomicMin((unsigned *)&a.parents[v[s]], (unsigned)pu);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_bfs_parents(BfsArgs a) {
  __shared__ int s_mark[kWavesPerBlock][64];
  parents_pass(a, s_mark[threadIdx.x >> 6]);
}

__global__ __launch_bounds__(kBlock) void k_bfs_level(BfsArgs a) {
  __shared__ int s_mark[kWavesPerBlock][64];
  __shared__ int s_cur[kCntFields];  // count, degree sum, long rows, (unused)
  __shared__ int s_open, s_prev_sd;
  __shared__ int s_red[kWavesPerBlock][3];
  // A lane adds the stripes of one field, and a workgroup ends with one 8-byte
  // add for count and degree sum.  With one thread reading, and clearing, all of
  // them and two adds, single runs from three sources took 75, 60 and 70 us on
  // RMAT-14 (71, 56 and 67 so) and 184, 187 and 217 on RMAT-22 (175, 177 and
  // 210); on other cards the difference lay within that of two runs of one form.
  static_assert(kCntSlots == 128 && 64 % kCntFields == 0, "two stripes a lane");
  if (threadIdx.x < 64) {
    const int ln = threadIdx.x;
    int x = a.cnt_cur[ln] + a.cnt_cur[ln + 64];
    const int open = a.parents ? a.ctrl->pushed[a.d % 3] : 0;
    const int prev_sd = a.parents ? a.ctrl->pushed_sd[a.d % 3] : 0;
#pragma unroll
    for (int off = kCntFields; off < 64; off *= 2) x += __shfl_xor(x, off);
    if (ln < kCntFields) s_cur[ln] = x;
    const int c = __shfl(x, 0), sd = __shfl(x, 1);
    if (ln == 0) {
      s_open = open;
      s_prev_sd = open ? prev_sd : 0;
    }
    if (blockIdx.x == 0) {
      // the buffer two levels ahead is cleared even when this level is
      // empty: it still holds the counts of the previous level
      a.cnt_clr[ln] = a.cnt_clr[ln + 64] = 0;
      if (ln == 0 && c > 0) {
        a.ctrl->nlev = a.d + 1;
        // the next frontier's parents stay open when a push of several
        // vertices finds it
        a.ctrl->pushed[(a.d + 1) % 3] = (decide(a, c, sd) == GRB_DIR_PUSH && c > 1) ? 1 : 0;
        a.ctrl->pushed_sd[(a.d + 1) % 3] = sd;
        if (a.stats && a.d < kStatsCap) {
          a.stats[a.d * kStatFields + 0] = c;
          a.stats[a.d * kStatFields + 1] = sd;
          a.stats[a.d * kStatFields + 2] = decide(a, c, sd);
        }
      }
    }
  }
  __syncthreads();
  const int count = s_cur[0], s_sumdeg = s_cur[1], s_long = s_cur[2];
  if (count == 0) return;
  const int dir = decide(a, count, s_sumdeg);
  int fc = 0, fd = 0, fl = 0;
  // parents of this frontier, when a push of several vertices found it: a
  // push over the same CSR offers them while it expands the frontier;
  // otherwise the previous frontier offers them again when its degree sum
  // and a scan of the levels cost less than this frontier's in-edges, and
  // else a pass over those in-edges finds them first
  const bool offer = s_open && dir == GRB_DIR_PUSH && a.same_csr;
  if (s_open && !offer) {
    if ((int64_t)s_prev_sd + a.n / 16 < (int64_t)s_sumdeg) prev_offers(a, s_mark[threadIdx.x >> 6]);
    else frontier_parents(a, s_mark[threadIdx.x >> 6]);
  }
  if (dir == GRB_DIR_PUSH)
    bfs_push(a, s_mark[threadIdx.x >> 6], s_long > 0, count == 1, offer, fc, fd, fl);
  else
    bfs_pull(a, s_mark[threadIdx.x >> 6], fc, fd, fl);
  if (__ballot(fc != 0)) {
    fc = wave_sum(fc);
    fd = wave_sum(fd);
    fl = wave_sum(fl);
  }
  if ((threadIdx.x & 63) == 0) {
    s_red[threadIdx.x >> 6][0] = fc;
    s_red[threadIdx.x >> 6][1] = fd;
    s_red[threadIdx.x >> 6][2] = fl;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int c = 0, sd = 0, lr = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) {
      c += s_red[i][0];
      sd += s_red[i][1];
      lr += s_red[i][2];
    }
    if (c) {
      const int t = blockIdx.x % kCntStripes;
      // count and degree sum in one: neither carries (both below 2^31)
      atomicAdd((unsigned long long *)&a.cnt_nxt[kCntFields * t],
                ((unsigned long long)(uint32_t)sd << 32) | (uint32_t)c);
      if (lr) atomicAdd(&a.cnt_nxt[kCntFields * t + 2], lr);
    }
  }
}

// The rows of word w that no level can find: without in-edges, or padding.
__device__ __forceinline__ uint64_t never_found(const BfsArgs &a, int64_t w) {
  if (a.can_pull) return a.pull.iso[w];
  const int64_t valid = a.n - w * 64;  // bits past n are padding
  return valid >= 64 ? 0ull : ~mask_below((int)valid);
}

__global__ __launch_bounds__(kBlock) void k_bfs_start(BfsArgs a, int32_t source, uint64_t *f1,
                                                      uint64_t *f2) {
  const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * kBlock;
  // levels and parents: -1 (source: 0 and itself), four vertices per
  // 16-byte store when both arrays allow it
  const bool vec = ((uintptr_t)a.levels % 16 == 0) &&
                   (!a.parents || (uintptr_t)a.parents % 16 == 0);
  const int64_t n4 = vec ? a.n / 4 : 0;
  for (int64_t i = tid; i < n4; i += nt) {
    int4 l = make_int4(-1, -1, -1, -1), p = l;
    if ((source >> 2) == i) {
      const int k = source & 3;
      if (k == 0) { l.x = 0; p.x = source; }
      else if (k == 1) { l.y = 0; p.y = source; }
      else if (k == 2) { l.z = 0; p.z = source; }
      else { l.w = 0; p.w = source; }
    }
    reinterpret_cast<int4 *>(a.levels)[i] = l;
    if (a.parents) reinterpret_cast<int4 *>(a.parents)[i] = p;
  }
  for (int64_t v = n4 * 4 + tid; v < a.n; v += nt) {
    a.levels[v] = (v == source) ? 0 : -1;
    if (a.parents) a.parents[v] = (v == source) ? source : -1;
  }
  // visited = rows a pull can never reach (no in-edges; padding) + source
  const int64_t sw = source >> 6;
  const uint64_t sb = 1ull << (source & 63);
  for (int64_t w = tid; w < a.nw; w += nt) {
    a.visited[w] = never_found(a, w) | (w == sw ? sb : 0ull);
    a.fcur[w] = w == sw ? sb : 0ull;
    f1[w] = 0ull;
    f2[w] = 0ull;
  }
  for (int64_t i = tid; i < a.own.nrec; i += nt) a.own.rec[i] = 0ull;  // no tag
  static_assert(kCntSlots <= kBlock, "a thread per counter");
  if (tid < kCntSlots) {
    const int ds = a.push.rp[source + 1] - a.push.rp[source];
    // level 0 = {source}: count, degree sum, long rows
    a.cnt_cur[tid] = tid == 0 ? 1 : tid == 1 ? ds : tid == 2 && ds > kPushSplit ? 1 : 0;
    a.cnt_nxt[tid] = 0;
    a.cnt_clr[tid] = 0;
  }
  if (tid == 0) {
    a.ctrl->nlev = 0;
    a.ctrl->pushed[0] = a.ctrl->pushed[1] = a.ctrl->pushed[2] = 0;
    a.ctrl->small_levels = INT_MAX;
    a.ctrl->spilled = 0;
  }
}

// ---- multi-workgroup level loop for small frontiers -------------------------
// High-diameter graphs spend thousands of levels on a few thousand vertices
// each, so a level's time is its chain of dependent memory round trips, not
// its work.  Workgroup w of the loop's G owns the vertices [w * chunk, (w + 1)
// * chunk): their visited bits sit in its LDS, it alone claims them (LDS
// atomics), and its share of the frontier is a queue in its LDS.  Level d:
// * the out-edges of its queue (a thread per vertex, four columns at a time):
//   an owned target is claimed at once and queued for level d + 1, another
//   one is sent to its owner;
// * wave 0 exchanges records with the other workgroups, while the other
//   waves write the levels of the newly queued vertices and load their row
//   extents and first columns for the next level;
// * the targets received are claimed and queued.
// On a graph whose ids follow its structure (grids, road networks in
// geographic order) nearly all targets are owned, and a level is the longer
// of the exchange and the two dependent loads beside it.
//
// The exchange needs no barrier and no atomics: workgroup s stores, for every
// owner o, a head (the number of targets sent and the first two of them) and
// a total (entries, queued, sent, full), 8-byte words that each carry the
// level's tag, and o polls the G words written for it.  Further targets go
// to a box in device memory, whose stores complete before the heads are
// written.  The words of level d are overwritten at d + 2, when every
// workgroup has read them (it published level d + 1 afterwards).
//
// All workgroups see the same totals.  The targets sent may be visited
// already or sent twice, so the next frontier holds at most queued + sent
// vertices: while that bound keeps every queue, the loop's edge limit and
// the switch rule's push, the next level starts at once; otherwise a second
// exchange gives the exact sizes, and a frontier that outgrew the loop or
// that the rule would pull is handed to the level kernels.
//
// No wait is unbounded: a workgroup that has polled for wait_ticks leaves the
// loop.  The others cannot pass the next exchange without it, so they leave
// one level later at most; the hand-over continues from the earliest of the
// levels (ctrl->small_levels), whose frontier is complete (every workgroup
// had published the level before it), and drops what was found beyond.
// Every step of a level is a short serial chain in one wave (a dependent
// vector instruction takes 5.5 ns here, an LDS access 25), so the loop keeps
// scans and 64-bit arithmetic off the usual path: slots come from ballots,
// and the totals are judged by ballots against a per-workgroup share of the
// bounds before any sum is taken.
// VIS: vertices whose visited bits it holds.  Beside other streams' kernels a
// workgroup becomes resident the later the more LDS it asks for, so small graphs
// have a form of 45 KB (three PageRanks of 64M entries, 700 x 700 grid, 8
// workgroups: 18 to 97 ms with 135 KB each, 5 to 58 so; alone 2.50 ms both, one
// workgroup's searches on small grids 0 to 1.3 % longer).  A form for 377,000
// vertices made the 3000 x 3000 grid's levels 1.3 % longer.
template <int VIS>
struct OwnShared {
  static constexpr int kVis = VIS;
  static constexpr int kIn = VIS ? 2 : 0;  // targets of each sender in its head
  uint32_t vis[VIS ? VIS / 32 : 1];
  int q[2][kOwnQueue];
  int cnt[2];              // entries found by the expansion into each queue
  int out[kOwnMaxGroups];  // targets sent to each workgroup in this level
  int msg[kOwnMaxGroups][2];   // the first two of each
  int pre[kOwnMaxGroups + 1];  // prefix of the boxes' further targets
  int sent;                // targets sent
  int edges;               // degree sum of the level's entries
  int ovf;                 // a queue or box was full
  int n_new;               // entries of the next level
  int state, nin, nc, ne, any_ovf;
};
enum OwnState { kOwnGo = 0, kOwnDone = 1, kOwnExact = 2, kOwnGaveUp = 3 };

__device__ __forceinline__ int own_sum(int x) { return lane_last(wave_incl_scan(x)); }

// record words (16-bit tag at the top; a tag is never 0, which the start
// kernel leaves)
__device__ __forceinline__ uint32_t own_tag(int64_t level) {  // of level L: 1 + L mod 65535
  return 1u + (uint32_t)level % 65535u;
}
__device__ __forceinline__ uint64_t own_head(uint32_t tag, int cnt, int m0, int m1) {
  return ((uint64_t)((tag << 16) | ((uint32_t)cnt << 8) | ((uint32_t)m0 >> 12)) << 32) |
         (((uint32_t)m0 << 20) | (uint32_t)m1);
}
__device__ __forceinline__ int head_cnt(uint64_t h) { return (int)(h >> 40) & 255; }
__device__ __forceinline__ int head_m0(uint64_t h) { return (int)(h >> 20) & 0xfffff; }
__device__ __forceinline__ int head_m1(uint64_t h) { return (int)h & 0xfffff; }
__device__ __forceinline__ uint64_t own_total(uint32_t tag, int n, int won, int sent, int ovf) {
  return ((uint64_t)((tag << 16) | (uint32_t)n) << 32) |
         (((uint64_t)won << 19) + ((uint64_t)sent << 1)) | (uint64_t)ovf;
}
__device__ __forceinline__ int total_n(uint64_t t) { return (int)(t >> 32) & 8191; }
__device__ __forceinline__ int total_won(uint64_t t) { return (int)((uint32_t)t >> 19); }
__device__ __forceinline__ int total_sent(uint64_t t) { return (int)((uint32_t)t >> 1) & 0x3ffff; }
static_assert(kOwnVertices <= 1 << 20 && kOwnQueue < 1 << 13 && kOwnCapMax < 256 &&
                  kCoopEdges < 1 << 18,  // (a level has at most kCoopEdges edges)
              "fields of the record words");

// Queues the winners among c[0..K) at *cnt of queue q (all 64 lanes call it);
// vertices past its end go straight into the next frontier's bitmap with
// their level.  One LDS atomic per wave: one per lane serialises on the
// counter (1.8 instead of 0.9 us per level).
template <int K, class SH>
__device__ __forceinline__ void own_queue(const BfsArgs &a, SH &sh, int *cnt, int *q,
                                          uint64_t *fn, int level, const int (&c)[K],
                                          const bool (&won)[K]) {
  uint64_t b[K];
  int tot = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    b[k] = __ballot(won[k]);
    tot += __popcll(b[k]);
  }
  if (tot == 0) return;
  int base = 0;
  if ((threadIdx.x & 63) == 0) base = atomicAdd(cnt, tot);
  base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int slot =
        base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b[k] >> 32),
                                              __builtin_amdgcn_mbcnt_lo((uint32_t)b[k], 0));
    base += __popcll(b[k]);
    if (!won[k]) continue;
    if (slot < kOwnQueue) {
      q[slot] = c[k];
    } else {
      a.levels[c[k]] = level;
      atomicOr((unsigned long long *)&fn[c[k] >> 6], 1ull << (c[k] & 63));
      sh.ovf = 1;
    }
  }
}

// Sets the visited bit of the owned vertex l; returns the word as it was.
template <class SH>
__device__ __forceinline__ uint32_t own_claim(const BfsArgs &a, SH &sh, int lo, uint32_t l) {
  if constexpr (SH::kVis != 0) return atomicOr(&sh.vis[l >> 5], 1u << (l & 31));
  else return atomicOr(reinterpret_cast<uint32_t *>(a.visited) + ((lo + l) >> 5), 1u << (l & 31));
}

// Claims the owned targets among c[0..4) (all four atomics are issued
// before a result is used), sends the others to their owners and queues the
// claims won.
template <class SH>
__device__ __forceinline__ void own_expand(const BfsArgs &a, SH &sh, int lo, int nv, int w,
                                           int *cnt, int *q, uint64_t *fn, int32_t *box, int level,
                                           const int (&c)[4]) {
  uint32_t old[4];
  bool far = false;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t l = (uint32_t)(c[k] - lo);  // (no target: beyond nv)
    const bool own = l < (uint32_t)nv;
    far |= c[k] >= 0 && !own;
    old[k] = ~0u;
    if (own) old[k] = own_claim(a, sh, lo, l);
  }
  if (__ballot(far)) {
    const int G = a.own.groups, cap = a.own.cap;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (c[k] < 0 || (uint32_t)(c[k] - lo) < (uint32_t)nv) continue;
      int o = (int)((float)c[k] * a.own.inv_chunk);  // off by one at most
      int m = c[k] - o * a.own.chunk;
      if (m < 0) {
        --o;
        m += a.own.chunk;
      } else if (m >= a.own.chunk) {
        ++o;
        m -= a.own.chunk;
      }
      const int slot = atomicAdd(&sh.out[o], 1);
      atomicAdd(&sh.sent, 1);
      if (slot < SH::kIn) {
        sh.msg[o][slot] = m;
      } else if (slot < cap) {
        st_coherent(&box[((int64_t)w * G + o) * cap + slot], c[k]);
      } else {  // box full: into the bitmap, sorted out by the hand-over
        atomicOr((unsigned long long *)&fn[c[k] >> 6], 1ull << (c[k] & 63));
        sh.ovf = 1;
      }
    }
  }
  bool won[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t l = (uint32_t)(c[k] - lo);
    won[k] = !((old[k] >> (l & 31)) & 1u);
  }
  own_queue(a, sh, cnt, q, fn, level, c, won);
}

// Levels of a low-degree graph back to back: 6,000 dependent levels on the
// 3000 x 3000 grid, bound by each level's chain (the queue, two loads of the
// rows, the exchange).  Every workgroup owns a run of vertices and keeps
// their visited bits and its queue in LDS, so a claim is an LDS atomic and
// only targets of other owners leave the workgroup.  3000 x 3000 grid from a
// corner: 16.3 ms, 2.7 us a level (from inside 2.2); a loop over shared queues
// in device memory (claims by device atomics, a counter barrier) 36.2 ms, 6.0
// us a level.
// R: polled records per lane of wave 0 (G <= 64 R); VIS: as above.  `most`: a frontier of at
// most this many vertices is within the edge limit and one the rule pushes;
// `share`: a level in which no workgroup found and sent more than this keeps
// that bound and every queue.
template <int R, int VIS>
__global__ __launch_bounds__(kOwnThreads) void k_bfs_own(BfsArgs a, int32_t source,
                                                         int max_levels, uint64_t wait_ticks,
                                                         int most, int share, uint64_t *F0,
                                                         uint64_t *F1, uint64_t *F2) {
  __shared__ OwnShared<VIS> sh;
  constexpr int IN = OwnShared<VIS>::kIn;
  constexpr int T = kOwnThreads - 64;  // threads that take queue entries (waves 1, 2, ...)
  const int tid = threadIdx.x, ln = tid & 63;
  const int et = tid - 64;  // this thread's first entry (wave 0 takes none)
  const int w = (int)blockIdx.x, G = a.own.groups, cap = a.own.cap;
  const int32_t *rp = a.push.rp, *ci = a.push.ci;
  const int64_t first = (int64_t)w * a.own.chunk;
  const int lo = (int)(first < a.n ? first : a.n);
  const int nv = (int)(a.n - lo < a.own.chunk ? a.n - lo : a.own.chunk);  // vertices owned
  // visited bits as the start kernel left them (rows nothing reaches, source)
  if constexpr (VIS != 0)
    for (int i = tid; i < (nv + 31) / 32; i += kOwnThreads)
      sh.vis[i] = reinterpret_cast<const uint32_t *>(a.visited)[lo / 32 + i];
  if (tid < kOwnMaxGroups) sh.out[tid] = sh.msg[tid][0] = sh.msg[tid][1] = 0;
  const bool mine = source >= lo && source - lo < nv;
  if (tid == 0) {
    sh.cnt[0] = sh.cnt[1] = 0;
    sh.sent = sh.edges = sh.ovf = 0;
    sh.q[0][0] = source;
  }
  __syncthreads();
  int n = mine ? 1 : 0, npre = 0;  // entries of this level, of them prefetched
  int prs = 0, pdg = 0, pc[4] = {-1, -1, -1, -1};  // this thread's prefetched entry
  // per level parity: boxes, records written and read by this lane, and what
  // rotates with the level, kept in registers (the address and modulo
  // arithmetic would otherwise open every level)
  int32_t *box = a.own.box, *box1 = box + (int64_t)G * G * cap;
  uint64_t *put = a.own.rec + 2 * ((int64_t)ln * G + w);  // + 128 G r: to workgroup 64 r + ln
  uint64_t *get = a.own.rec + 2 * ((int64_t)w * G + ln);  // + 128 r: from workgroup 64 r + ln
  uint64_t *put1 = put + (int64_t)G * G * 2, *get1 = get + (int64_t)G * G * 2;
  uint64_t *fn = F1, *fn1 = F2, *fn2 = F0;
  uint32_t tag = own_tag(0);
  int cur = 0, d = 0, slow = 0;  // queue, level, second exchanges so far
  bool spill = false;
  for (;;) {
    const int nxt = cur ^ 1;
    const bool rec_level = d < kStatsCap;
    if (et >= 0) {
      int esum = 0;
      for (int i0 = et & ~63; i0 < n; i0 += T) {
        const int i = i0 + ln;
        int rs = 0, dg = 0, c[4] = {-1, -1, -1, -1};
        if (i0 < T && i < npre) {
          rs = prs;
          dg = pdg;
#pragma unroll
          for (int q = 0; q < 4; ++q) c[q] = pc[q];
        } else if (i < n) {
          const int v = sh.q[cur][i];
          rs = rp[v];
          dg = rp[v + 1] - rs;
#pragma unroll
          for (int q = 0; q < 4; ++q) c[q] = q < dg ? ci[rs + q] : -1;
        }
        esum += dg;
        own_expand(a, sh, lo, nv, w, &sh.cnt[nxt], sh.q[nxt], fn, box, d + 1, c);
        for (int q0 = 4; __ballot(q0 < dg) != 0ull; q0 += 4) {
#pragma unroll
          for (int q = 0; q < 4; ++q) c[q] = q0 + q < dg ? ci[rs + q0 + q] : -1;
          own_expand(a, sh, lo, nv, w, &sh.cnt[nxt], sh.q[nxt], fn, box, d + 1, c);
        }
      }
      if (rec_level) {
        esum = own_sum(esum);
        if (ln == 0 && esum) atomicAdd(&sh.edges, esum);
      }
      __builtin_amdgcn_s_waitcnt(0);  // box stores are done before the heads go out
    }
    __syncthreads();
    const int nl = min(sh.cnt[nxt], kOwnQueue);
    if (et < 0) {
      int total = nl, nin = 0, state = kOwnGo, nc = n, ne = sh.edges;
      int any_ovf = sh.ovf;
      bool any_n = n > 0;
      if (G == 1) {
        if (nl == 0) state = kOwnDone;
        else if (nl > most || any_ovf) state = kOwnExact;
      } else {
        // lane l: workgroups l, l + 64, ...
        const uint64_t tot = own_total(tag, n, nl, sh.sent, any_ovf);
        uint64_t hd[R], tt[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int o = r * 64 + ln;
          if (o >= G) continue;
          const int x = sh.out[o];
          uint64_t *p = put + (int64_t)128 * G * r;
          store_relaxed_u64(p, own_head(tag, min(x, cap), sh.msg[o][0], sh.msg[o][1]));
          store_relaxed_u64(p + 1, tot);
          if (x) sh.out[o] = 0;
        }
        if (rec_level && ln == 0)
          store_relaxed_u64(&a.own.rec_edges[(d & 1) * G + w],
                            ((uint64_t)tag << 48) | (uint32_t)ne);
        // poll the words written for this workgroup
        uint64_t t0 = 0;
        for (;;) {
          bool ok = true;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int sd = r * 64 + ln;
            hd[r] = tt[r] = 0ull;
            if (sd >= G) continue;
            hd[r] = load_relaxed_u64(get + 128 * r);
            tt[r] = load_relaxed_u64(get + 128 * r + 1);
            ok &= (uint32_t)(hd[r] >> 48) == tag && (uint32_t)(tt[r] >> 48) == tag;
          }
          if (__ballot(!ok) == 0ull) break;
          if (t0 == 0) t0 = wall_clock64();
          if (wall_clock64() - t0 >= (d == 0 ? kCoopFirstWait : 1) * wait_ticks) {
            state = kOwnGaveUp;
            break;
          }
        }
        if (state == kOwnGo) {
          bool found = false, much = false, full = false, more = false, front = false;
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int x = total_won(tt[r]) + total_sent(tt[r]);
            found |= x != 0;
            much |= x > share;
            full |= (tt[r] & 1ull) != 0;
            front |= total_n(tt[r]) != 0;
            const int kc = head_cnt(hd[r]);
            more |= kc > IN;
            if (IN == 0 || __ballot(kc != 0) == 0ull) continue;
            // the first two targets of each sender
            const int m0 = head_m0(hd[r]), m1 = head_m1(hd[r]);
            uint32_t o0 = ~0u, o1 = ~0u;
            if (kc > 0) o0 = atomicOr(&sh.vis[m0 >> 5], 1u << (m0 & 31));
            if (kc > 1) o1 = atomicOr(&sh.vis[m1 >> 5], 1u << (m1 & 31));
            const bool w0 = !((o0 >> (m0 & 31)) & 1u), w1 = !((o1 >> (m1 & 31)) & 1u);
            const uint64_t b0 = __ballot(w0), b1 = __ballot(w1);
            if (b0 | b1) {  // this wave alone appends here
              int slot = total + __popcll(b0 & mask_below(ln)) + __popcll(b1 & mask_below(ln));
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                if (!(q == 0 ? w0 : w1)) continue;
                const int c = lo + (q == 0 ? m0 : m1);
                a.levels[c] = d + 1;
                if (slot < kOwnQueue) {
                  sh.q[nxt][slot] = c;
                } else {
                  atomicOr((unsigned long long *)&fn[c >> 6], 1ull << (c & 63));
                  sh.ovf = 1;
                }
                ++slot;
              }
              total += __popcll(b0) + __popcll(b1);
            }
          }
          any_ovf = __ballot(full) != 0ull;
          any_n = __ballot(front) != 0ull;
          if (__ballot(found) == 0ull) state = kOwnDone;
          else if (any_ovf) state = kOwnExact;
          else if (__ballot(much)) {
            int wsum = 0, ssum = 0, mw = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              wsum += total_won(tt[r]);
              ssum += total_sent(tt[r]);
              mw = max(mw, total_won(tt[r]));
            }
            wsum = own_sum(wsum);
            ssum = own_sum(ssum);
            mw = lane_last(wave_max_scan(mw));
            if (wsum + ssum > most || ssum + mw > kOwnQueue) state = kOwnExact;
          }
          if (__ballot(more)) {  // boxes: prefix of the further targets, lane-major
            int k[R], in = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) in += k[r] = max(head_cnt(hd[r]) - IN, 0);
            const int incl = wave_incl_scan(in);
            int run = incl - in;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              run += k[r];
              sh.pre[ln * R + r + 1] = run;
            }
            if (ln == 0) sh.pre[0] = 0;
            nin = lane_last(incl);
          }
          if (w == 0 && rec_level) {  // the level's record: sizes and degree sums
            nc = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) nc += total_n(tt[r]);
            nc = own_sum(nc);
            ne = 0;
            for (int sd = ln; sd < G; sd += 64) {
              uint64_t x;
              t0 = wall_clock64();
              do {
                x = load_relaxed_u64(&a.own.rec_edges[(d & 1) * G + sd]);
              } while ((uint32_t)(x >> 48) != tag && wall_clock64() - t0 < kCoopWaitTicks);
              ne += (int)(uint32_t)x;
            }
            ne = own_sum(ne);
          }
        }
      }
      if (ln == 0) {
        sh.state = state;
        sh.n_new = total;
        sh.nin = nin;
        sh.any_ovf = any_ovf;
        sh.cnt[cur] = 0;
        sh.sent = 0;
        if (rec_level) sh.edges = 0;
        if (w == 0 && state != kOwnGaveUp && any_n) {
          a.ctrl->nlev = d + 1;
          if (rec_level && a.stats) {
            a.stats[d * kStatFields + 0] = nc;
            a.stats[d * kStatFields + 1] = ne;
            a.stats[d * kStatFields + 2] = GRB_DIR_PUSH;
          }
        }
      }
    } else {
      // beside the exchange: levels, row extents and first columns of what
      // this workgroup queued
      prs = pdg = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) pc[q] = -1;
      if (et < nl) {
        const int v = sh.q[nxt][et];
        prs = rp[v];
        pdg = rp[v + 1] - prs;
#pragma unroll
        for (int q = 0; q < 4; ++q) pc[q] = q < pdg ? ci[prs + q] : -1;
      }
      for (int i = et; i < nl; i += T) a.levels[sh.q[nxt][i]] = d + 1;
    }
    npre = min(nl, T);
    __syncthreads();
    ++d;
    const int state = sh.state;
    if (state == kOwnGaveUp) {
      spill = true;
      break;
    }
    if (state == kOwnDone) break;
    const int nin = sh.nin;
    if (nin > 0) {  // further targets, from the boxes
      for (int i0 = tid & ~63; i0 < nin; i0 += kOwnThreads) {
        const int i = i0 + ln;
        int c[1] = {-1};
        bool wn[1] = {false};
        if (i < nin) {
          int at = 0;  // the last position with pre[at] <= i
#pragma unroll
          for (int step = 32 * R; step > 0; step >>= 1)
            if (sh.pre[at + step] <= i) at += step;
          const int sd = (at % R) * 64 + at / R;
          c[0] = ld_coherent(&box[((int64_t)sd * G + w) * cap + IN + (i - sh.pre[at])]);
          const int l = c[0] - lo;
          wn[0] = !((own_claim(a, sh, lo, (uint32_t)l) >> (l & 31)) & 1u);
          if (wn[0]) a.levels[c[0]] = d;
        }
        own_queue(a, sh, &sh.n_new, sh.q[nxt], fn, d, c, wn);
      }
      __syncthreads();
    }
    n = min(sh.n_new, kOwnQueue);
    cur = nxt;
    {
      int32_t *b = box;
      uint64_t *p = put, *g = get, *f = fn;
      box = box1, box1 = b;
      put = put1, put1 = p;
      get = get1, get1 = g;
      fn = fn1, fn1 = fn2, fn2 = f;
      tag = tag == 65535u ? 1u : tag + 1u;
    }
    if (d >= max_levels) {
      spill = sh.any_ovf != 0;  // targets that found a box full get their level there
      break;
    }
    if (state == kOwnExact || d >= kOwnMaxLevels) {
      // the exact frontier: sizes, degree sums and full queues of every
      // workgroup over a second exchange
      int e = 0;
      for (int i = tid; i < n; i += kOwnThreads) {
        const int v = sh.q[cur][i];
        e += rp[v + 1] - rp[v];
      }
      __syncthreads();
      if (tid == 0) sh.edges = 0;
      __syncthreads();
      e = own_sum(e);
      if (ln == 0 && e) atomicAdd(&sh.edges, e);
      __syncthreads();
      if (tid < 64) {
        int nc = n, ne = sh.edges, gave_up = 0;
        bool ov = sh.ovf != 0 || sh.any_ovf != 0;
        if (G > 1) {
          uint64_t *r2 = a.own.rec2 + (slow & 1) * G;
          const uint32_t tag2 = own_tag(slow);
          if (ln == 0)
            store_relaxed_u64(&r2[w], ((uint64_t)((tag2 << 16) | (uint32_t)n) << 32) |
                                          ((uint32_t)ne << 1) | (ov ? 1u : 0u));
          const uint64_t t0 = wall_clock64();
          for (;;) {
            bool ok = true;
            int c = 0, es = 0, ovs = 0;
            for (int sd = ln; sd < G; sd += 64) {
              const uint64_t x = load_relaxed_u64(&r2[sd]);
              ok &= (uint32_t)(x >> 48) == tag2;
              c += (int)(x >> 32) & 0xffff;
              es += (int)((uint32_t)x >> 1);
              ovs |= (int)x & 1;
            }
            if (__ballot(!ok) == 0ull) {
              nc = own_sum(c);
              ne = own_sum(es);
              ov = __ballot(ovs != 0) != 0ull;
              break;
            }
            if (wall_clock64() - t0 >= wait_ticks) {
              gave_up = 1;
              break;
            }
          }
        }
        if (ln == 0) {
          sh.state = gave_up ? kOwnGaveUp : kOwnGo;
          sh.nc = nc;
          sh.ne = ne;
          sh.any_ovf = ov ? 1 : 0;
          sh.edges = 0;
        }
      }
      ++slow;
      __syncthreads();
      if (sh.state == kOwnGaveUp) {
        spill = true;
        break;
      }
      if (sh.nc == 0 && !sh.any_ovf) break;
      if (sh.any_ovf || sh.ne > kCoopEdges || d >= kOwnMaxLevels ||
          decide(a, sh.nc, sh.ne) == GRB_DIR_PULL) {
        spill = true;
        break;
      }
    }
  }
  if (tid == 0) {
    atomicMin(&a.ctrl->small_levels, d);
    if (spill) atomicOr(&a.ctrl->spilled, 1);
  }
}

// After a loop that spilled at level h = ctrl->small_levels.  What it left:
// the levels of every vertex claimed (the frontier's are h; a workgroup that
// left a level later also claimed some at h + 1), the targets sent in that
// level, which their owners may not have read, and the bits of targets that
// found a box full.  First the targets sent join those bits; then one pass
// over the vertices makes the frontier's bitmap and counters (vertices at
// level h, and unreached ones whose bit is set, which get the level) and the
// visited bitmap of level h for the level kernel, and resets what lies beyond.
__global__ __launch_bounds__(kBlock) void k_bfs_own_boxes(BfsArgs a, uint64_t *F0, uint64_t *F1,
                                                          uint64_t *F2) {
  if (!a.ctrl->spilled) return;
  const int64_t h = a.ctrl->small_levels;
  uint64_t *fh = (h % 3 == 0) ? F0 : ((h % 3 == 1) ? F1 : F2);
  const int G = a.own.groups, cap = a.own.cap, par = (int)((h - 1) & 1);
  const int in = a.own.in_device ? 0 : 2;  // targets in the heads
  const int32_t *box = a.own.box + (int64_t)par * G * G * cap;
  const uint64_t *rec = a.own.rec + (int64_t)par * G * G * 2;
  const uint32_t tag = own_tag(h - 1);
  const int64_t tid = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (G > 1) {
    const int64_t m = (int64_t)G * G * cap, nt = (int64_t)gridDim.x * kBlock;
    for (int64_t t = tid; t < m; t += nt) {
      const int64_t pair = t / cap;
      const int sd = (int)(pair / G), o = (int)(pair % G), j = (int)(t % cap);
      const uint64_t hd = rec[((int64_t)o * G + sd) * 2];
      if ((uint32_t)(hd >> 48) != tag || j >= head_cnt(hd)) continue;
      const int c = j >= in ? box[t] : o * a.own.chunk + (j == 0 ? head_m0(hd) : head_m1(hd));
      atomicOr((unsigned long long *)&fh[c >> 6], 1ull << (c & 63));
    }
  }
  if (tid == 0) {
    for (int i = 0; i < 3 * kCntSlots; ++i) a.ctrl->lists[i] = 0;
    a.ctrl->pushed[0] = a.ctrl->pushed[1] = a.ctrl->pushed[2] = 0;  // parents: final pass
    if (G > 1) {  // the record of level h - 1, where workgroup 0 left before it
      int nc = 0, ne = 0;
      for (int sd = 0; sd < G; ++sd) {
        nc += total_n(rec[(int64_t)sd * 2 + 1]);
        ne += (int)(uint32_t)a.own.rec_edges[par * G + sd];
      }
      if (nc > 0) {
        a.ctrl->nlev = (int)h;
        if (a.stats && h - 1 < kStatsCap) {
          a.stats[(h - 1) * kStatFields + 0] = nc;
          a.stats[(h - 1) * kStatFields + 1] = ne;
          a.stats[(h - 1) * kStatFields + 2] = GRB_DIR_PUSH;
        }
      }
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_bfs_own_handover(BfsArgs a, uint64_t *F0, uint64_t *F1,
                                                             uint64_t *F2) {
  __shared__ int s_red[kWavesPerBlock][2];
  if (!a.ctrl->spilled) return;
  const int64_t h = a.ctrl->small_levels;
  uint64_t *const F[3] = {F0, F1, F2};
  uint64_t *fh = F[h % 3], *f1 = F[(h + 1) % 3], *f2 = F[(h + 2) % 3];
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  int fc = 0, fd = 0;
  for (int64_t w = gw; w < a.nw; w += nwaves) {
    const int64_t v = w * 64 + ln;
    const bool inb = v < a.n;
    int lev = inb ? a.levels[v] : 0;
    const uint64_t bits = fh[w];
    const bool beyond = inb && lev > h;
    if (beyond) a.levels[v] = lev = -1;
    const bool found = inb && lev == -1 && ((bits >> ln) & 1ull);
    const bool front = inb && (lev == h || found);
    if (found) a.levels[v] = (int)h;
    if (front) {
      fc += 1;
      fd += a.push.rp[v + 1] - a.push.rp[v];
    }
    const uint64_t fm = __ballot(front), vm = __ballot(inb && (lev >= 0 || found));
    if (ln == 0) {
      fh[w] = fm;
      f1[w] = 0ull;
      f2[w] = 0ull;
      // (with the visited bits in device memory they hold claims beyond h too)
      a.visited[w] = vm | (a.own.in_device ? never_found(a, w) : a.visited[w]);
    }
  }
  fc = wave_sum(fc);
  fd = wave_sum(fd);
  if (ln == 0) {
    s_red[threadIdx.x >> 6][0] = fc;
    s_red[threadIdx.x >> 6][1] = fd;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int c = 0, sd = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) {
      c += s_red[i][0];
      sd += s_red[i][1];
    }
    if (c) {  // rows are at most kCoopMaxDeg long: none has pieces
      int32_t *cnt = a.ctrl->lists + (h % 3) * kCntSlots + kCntFields * (blockIdx.x % kCntStripes);
      atomicAdd(&cnt[0], c);
      atomicAdd(&cnt[1], sd);
    }
  }
}

}  // namespace

void launch_bfs_own(const BfsArgs &a, int32_t source, int64_t max_levels, uint64_t *const F[3],
                    uint64_t wait_ticks, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const int64_t deg = std::max<int64_t>(a.push.max_deg, 1);
  int64_t m = kCoopEdges / deg;
  if (!a.forced && a.can_pull) {
    const int64_t den = std::max<int64_t>(a.denom, 1);
    m = std::min(m, a.rule == GRB_SWITCH_EXACT ? a.nnz / den / deg : a.n / den);
  }
  const int cap = (int)std::min<int64_t>(max_levels, kOwnMaxLevels + 1);
  const int most = (int)m, share = (int)std::min<int64_t>(m, kOwnQueue) / a.own.groups;
  const auto kernel = a.own.in_device                  ? k_bfs_own<1, 0>
                      : a.own.groups > 64                ? k_bfs_own<4, kOwnVertices>
                      : a.own.chunk <= kOwnVerticesLow ? k_bfs_own<1, kOwnVerticesLow>
                                                       : k_bfs_own<1, kOwnVertices>;
  hipLaunchKernelGGL(kernel, dim3(a.own.groups), dim3(kOwnThreads), 0, s, a, source, cap, wait_ticks,
                     most, share, F[0], F[1], F[2]);
  hipLaunchKernelGGL(k_bfs_own_boxes, dim3(256), dim3(kBlock), 0, s, a, F[0], F[1], F[2]);
  int64_t g = (a.nw + kWavesPerBlock - 1) / kWavesPerBlock;
  g = g < 1 ? 1 : (g > kExpandGrid ? kExpandGrid : g);
  hipLaunchKernelGGL(k_bfs_own_handover, dim3((unsigned)g), dim3(kBlock), 0, s, a, F[0], F[1],
                     F[2]);
}

void launch_bfs_start(const BfsArgs &a, int32_t source, uint64_t *f1, uint64_t *f2,
                      void *stream) {
  int64_t g = (a.n / 4 + kBlock - 1) / kBlock;
  g = g < 1 ? 1 : (g > 4096 ? 4096 : g);
  hipLaunchKernelGGL(k_bfs_start, dim3((unsigned)g), dim3(kBlock), 0, (hipStream_t)stream, a,
                     source, f1, f2);
}

void launch_bfs_level(const BfsArgs &a, void *stream) {
  hipLaunchKernelGGL(k_bfs_level, dim3(kExpandGrid), dim3(kBlock), 0, (hipStream_t)stream, a);
}

void launch_bfs_parents(const BfsArgs &a, void *stream) {
  // one wave per bitmap word
  int64_t g = (a.nw + kWavesPerBlock - 1) / kWavesPerBlock;
  g = g < 1 ? 1 : (g > (1 << 20) ? (1 << 20) : g);
  hipLaunchKernelGGL(k_bfs_parents, dim3((unsigned)g), dim3(kBlock), 0, (hipStream_t)stream, a);
}

}  // namespace grb
