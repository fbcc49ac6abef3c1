// Connected components (Section 7.4 of the paper: the FastSV form of
// Shiloach-Vishkin, hooking and shortcutting in linear algebra).  Vectors
// f (parent), gf (grandparent), mngf (smallest grandparent seen among the
// neighbours); every label is a vertex id and only ever decreases, so the
// fixed point labels each component with its smallest id.  Per iteration:
//   mngf = min(mngf, A (min, second) gf)      the product, pull
//   f[f_old[u]] = min(., mngf[u])             stochastic hooking (scatter)
//   f[u] = min(f[u], mngf[u])                 aggressive hooking
//   f[u] = min(f[u], gf[u])                   shortcutting
//   gf[u] = f[f[u]]; count the u whose gf changed
// until an iteration changes no grandparent.
//
// Two kernels per iteration.  k_cc_sweep takes the product and, as each row's
// minimum is known, its hooking and shortcutting: those three are minima into
// f of values that no step of the iteration changes (gf, f_old) or that only
// this row's wave and pieces lower (mngf), so their order does not matter and
// f_old keeps the iteration's input.  k_cc_grand takes the rest.
//
// The generic product swept every entry in every iteration (RMAT-22: 1.06 ms
// each, 128M random gathers of a presence word and of gf).  The sweep reads
// far fewer, with the same mngf after every iteration:
// * in the first iteration gf(j) = j, so a row's minimum is its first column
//   (columns ascend), read from the prepared first-two array;
// * no label can go below `floor`, the smallest id with an entry, so a row
//   whose minimum has reached it needs no scan, and a scan stops there (the
//   terminal value of the minimum).  On a graph with a giant component that
//   holds the smallest id nearly every row reaches it by its first two
//   neighbours in the second iteration; where no row does, every entry is
//   read, without the presence test of the generic product.
#include <hip/hip_runtime.h>

#include "grb_device.h"
#include "grb_internal.h"

namespace grb {
namespace {

struct OpMinI {
  __device__ __forceinline__ int operator()(int a, int b) const { return a < b ? a : b; }
};

__device__ __forceinline__ int wave_min_i(int x) {
  return lane_last(wave_scan(x, INT_MAX, OpMinI()));
}

__global__ void k_cc_init(CcArgs a, const uint64_t *iso, const uint64_t *iso_t) {
  const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t nt = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = tid; i < a.n; i += nt) {
    a.f[i] = (int32_t)i;
    a.f_old[i] = (int32_t)i;
    a.gf[i] = (int32_t)i;
    a.mngf[i] = (int32_t)i;
  }
  for (int64_t i = tid; i < kStatsCap; i += nt) a.changed[i] = 0;
  // floor: the smallest id with an entry in either orientation (one wave
  // walks the words; the first one with such an id is nearly always first)
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    const int ln = threadIdx.x;
    int32_t lo = INT_MAX;
    for (int64_t w0 = 0; w0 < a.nw; w0 += 64) {
      const int64_t w = w0 + ln;
      const uint64_t any = w < a.nw ? ~(iso[w] & (iso_t ? iso_t[w] : ~0ull)) : 0ull;
      const uint64_t b = __ballot(any != 0ull);
      if (b) {
        const int k = __ffsll((unsigned long long)b) - 1;
        const uint64_t x = __shfl(any, k);
        lo = (int32_t)((w0 + k) * 64 + __ffsll((unsigned long long)x) - 1);
        break;
      }
    }
    if (ln == 0) *a.floor = lo;
  }
}

// Hooks vertex v, whose neighbour minimum is m, parent p and grandparent g.
// Labels only decrease, so a target already at or below the value needs no
// atomic: after the first iteration most vertices share a handful of roots,
// and the reads keep millions of atomics off those few words.
__device__ __forceinline__ void cc_hook(const CcArgs &a, int32_t v, int32_t m, int32_t p,
                                        int32_t g) {
  if (m < a.f[p]) atomicMin(&a.f[p], m);
  const int32_t x = m < g ? m : g;
  if (x < a.f[v]) atomicMin(&a.f[v], x);
}

// The minimum stream of the open rows (one per lane: `own`; positions
// [rc, re)), K steps of 64 positions laid out and loaded at once; a row
// leaves at the floor.  A row takes at most about cmin positions per step
// while enough rows are open, so rows that meet the floor early are not read
// far past it.
template <int K>
__device__ __forceinline__ void min_stream(const CcArgs &a, const int32_t *ci, int *mark, int cmin,
                                           bool own, int32_t floor, int &rc, int re,
                                           int32_t &best) {
  const int ln = threadIdx.x & 63;
  for (bool more = true; more;) {
    int pos[K], row[K], se[K];
    bool st[K];
#pragma unroll
    for (int s = 0; s < K; ++s) {
      pos[s] = -1;
      row[s] = 0;
      se[s] = 0;
      st[s] = false;
      if (!more) continue;
      int len = (own && best != floor) ? re - rc : 0;
      if (cmin < 64) {
        const int nl = __popcll(__ballot(len > 0));
        len = min(len, max(cmin, nl ? (64 + nl - 1) / nl : 64));
      }
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
      row[s] = r;
      se[s] = min(incl, 64);
      st[s] = starts;
      if (starts) rc += se[s] - excl;
    }
    int c[K];
#pragma unroll
    for (int s = 0; s < K; ++s) c[s] = pos[s] >= 0 ? ci[pos[s]] : -1;
    int32_t g[K];
#pragma unroll
    for (int s = 0; s < K; ++s) g[s] = c[s] >= 0 ? a.gf[c[s]] : INT_MAX;
#pragma unroll
    for (int s = 0; s < K; ++s) {
      const int y = wave_seg_scan(g[s], row[s], INT_MAX, OpMinI());
      const int segmin = __shfl(y, st[s] ? se[s] - 1 : 0);
      if (st[s]) best = min(best, segmin);
    }
  }
}

// The rows of up to four words: the loads of all four are issued together.
template <bool FIRST>
__device__ void cc_words(const CcArgs &a, const Csr &g, int32_t floor, const int64_t (&wd)[4],
                         int nq, int *mark, int32_t (*res)[64]) {
  const int ln = threadIdx.x & 63;
  int64_t v[4];
  bool has[4];
  int32_t m[4], p[4], gv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    v[q] = wd[q] * 64 + ln;
    has[q] = q < nq && !((g.iso[wd[q]] >> ln) & 1ull);  // padding rows count as empty
    m[q] = has[q] ? a.mngf[v[q]] : floor;
    p[q] = has[q] ? a.f_old[v[q]] : 0;
    gv[q] = has[q] ? a.gf[v[q]] : 0;
  }
  if constexpr (FIRST) {
    int32_t c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c[q] = has[q] ? g.first2[v[q]].x : INT_MAX;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (has[q]) {
        if (c[q] < m[q]) a.mngf[v[q]] = m[q] = c[q];
        cc_hook(a, (int32_t)v[q], m[q], p[q], gv[q]);
      }
    return;
  }
  bool need[4], lng[4];
  int cur[4], end[4];
  int2 f2[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    need[q] = has[q] && m[q] != floor;
    cur[q] = need[q] ? g.rp[v[q]] : 0;
    end[q] = need[q] ? g.rp[v[q] + 1] : 0;
    f2[q] = need[q] ? g.first2[v[q]] : make_int2(-1, -1);
  }
  int32_t g0[4], g1[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    g0[q] = f2[q].x >= 0 ? a.gf[f2[q].x] : INT_MAX;
    g1[q] = f2[q].y >= 0 ? a.gf[f2[q].y] : INT_MAX;
  }
  uint64_t rest[4];
  int nrest = 0, np = 0, nh = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int32_t best = min(g0[q], g1[q]);
    lng[q] = end[q] - cur[q] > kPushSplit;
    np += __popcll(__ballot(need[q]));
    nh += __popcll(__ballot(need[q] && best == floor));
    res[q][ln] = best;
    cur[q] = min(cur[q] + 2, end[q]);
    rest[q] = __ballot(need[q] && !lng[q] && best != floor && end[q] > cur[q]);
    nrest += __popcll(rest[q]);
  }
  // two probes per row: about np / nh rows' worth of 2 positions per hit
  const int cmin = nh == 0 ? 64 : min(64, max(4, 4 * np / nh));
  for (int sb = 0; sb < nrest; sb += 64) {
    const int j = sb + ln;  // this lane's row among the open rows: word oq, lane li
    int oq = -1, li = 0, rc = 0, re = 0, before = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int cq = __popcll(rest[q]);
      const bool mine = j >= before && j < before + cq;
      const int lq = mine ? nth_set_bit(rest[q], j - before) : 0;
      const int sc = __shfl(cur[q], lq), se = __shfl(end[q], lq);
      if (mine) {
        oq = q;
        li = lq;
        rc = sc;
        re = se;
      }
      before += cq;
    }
    int32_t best = INT_MAX;
    if (cmin == 64) min_stream<kUnroll>(a, g.ci, mark, cmin, oq >= 0, floor, rc, re, best);
    else min_stream<1>(a, g.ci, mark, cmin, oq >= 0, floor, rc, re, best);
    if (oq >= 0) res[oq][li] = min(res[oq][li], best);
  }
  wave_lds_sync();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    if (!has[q]) continue;
    const int32_t b = res[q][ln];
    if (need[q] && b < m[q]) {
      m[q] = b;
      if (lng[q]) atomicMin(&a.mngf[v[q]], b);  // its pieces lower it too
      else a.mngf[v[q]] = b;
    }
    cc_hook(a, (int32_t)v[q], m[q], p[q], gv[q]);
  }
  wave_lds_sync();
}

// FIRST: the first iteration (gf is the identity).  `it` > 0 returns at once
// when the iteration before it changed nothing.
template <bool FIRST>
__global__ __launch_bounds__(kBlock) void k_cc_sweep(CcArgs a, Csr g, const int64_t *prev) {
  __shared__ int s_mark[kWavesPerBlock][64];
  __shared__ int32_t s_res[kWavesPerBlock][4][64];
  if (prev && *prev == 0) return;
  const int wid = threadIdx.x >> 6, ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + wid;
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t floor = *a.floor;
  // up to kWaveParts words: a word per wave (its run would be no longer, and
  // the run bounds would be one more dependent load)
  const bool by_word = a.nw <= kWaveParts;
  const int64_t parts = by_word ? a.nw : kWaveParts;
  for (int64_t part = gw; part < parts; part += nwaves) {
    const int64_t wlo = by_word ? part : g.wpart[part];
    const int64_t whi = by_word ? part + 1 : g.wpart[part + 1];
    for (int64_t w0 = wlo; w0 < whi; w0 += 64) {
      uint64_t todo = __ballot(w0 + ln < whi && ~g.iso[w0 + ln] != 0ull);
      while (todo) {
        int64_t wds[4] = {0, 0, 0, 0};
        int nq = 0;
        while (todo && nq < 4) {
          wds[nq++] = w0 + __ffsll((unsigned long long)todo) - 1;
          todo &= todo - 1;
        }
        cc_words<FIRST>(a, g, floor, wds, nq, s_mark[wid], s_res[wid]);
      }
    }
  }
  if constexpr (FIRST) return;
  // pieces of the long rows not at the floor, dealt to the waves with a
  // stride; each piece hooks with its own minimum
  static_assert(kPushSplit == 64 * kUnroll, "a piece is one unrolled step");
  for (int64_t hb = gw; hb < g.nsplit; hb += 64 * nwaves) {
    const int64_t h = hb + (int64_t)ln * nwaves;
    int r = -1, b = 0, e = 0;
    if (h < g.nsplit) {
      r = g.split[2 * h];
      b = g.split[2 * h + 1];
      if (a.mngf[r] == floor) r = -1;
      else e = min(b + kPushSplit, g.rp[r + 1]);
    }
    for (uint64_t act = __ballot(r >= 0); act; act &= act - 1) {
      const int k = __ffsll((unsigned long long)act) - 1;
      const int pr = __shfl(r, k), pb = __shfl(b, k), pe = __shfl(e, k);
      int c[kUnroll];
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) {
        const int pos = pb + s * 64 + ln;
        c[s] = pos < pe ? g.ci[pos] : -1;
      }
      int32_t x[kUnroll], best = INT_MAX;
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) x[s] = c[s] >= 0 ? a.gf[c[s]] : INT_MAX;
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) best = min(best, x[s]);
      best = wave_min_i(best);
      if (ln == 0) {
        if (best < a.mngf[pr]) atomicMin(&a.mngf[pr], best);
        cc_hook(a, pr, best, a.f_old[pr], best);
      }
    }
  }
}

// gf = f[f]; the vertices whose grandparent changed are counted for this
// iteration (one atomic per workgroup: one per wave on the single counter
// took 0.14 ms of the 0.2 ms pass on RMAT-22); f_old = f for the next hooking
__global__ __launch_bounds__(kBlock) void k_cc_grand(CcArgs a, int64_t *changed,
                                                     const int64_t *prev) {
  __shared__ int s_cnt[kWavesPerBlock];
  if (prev && *prev == 0) return;
  int cnt = 0;
  const int64_t nt = (int64_t)gridDim.x * kBlock;
  for (int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x; i0 < a.n; i0 += nt * kUnroll) {
    int32_t fi[kUnroll], old[kUnroll], g[kUnroll];
#pragma unroll
    for (int s = 0; s < kUnroll; ++s) {
      const int64_t i = i0 + s * nt;
      fi[s] = i < a.n ? a.f[i] : 0;
      old[s] = i < a.n ? a.gf[i] : 0;
    }
#pragma unroll
    for (int s = 0; s < kUnroll; ++s) g[s] = a.f[fi[s]];
#pragma unroll
    for (int s = 0; s < kUnroll; ++s) {
      const int64_t i = i0 + s * nt;
      if (i >= a.n) continue;
      if (g[s] != old[s]) {
        ++cnt;
        a.gf[i] = g[s];
      }
      a.f_old[i] = fi[s];
    }
  }
  cnt = wave_sum(cnt);
  if ((threadIdx.x & 63) == 0) s_cnt[threadIdx.x >> 6] = cnt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int t = 0;
    for (int k = 0; k < kWavesPerBlock; ++k) t += s_cnt[k];
    if (t) atomicAdd((unsigned long long *)changed, (unsigned long long)t);
  }
}

int grid_of(int64_t n, int64_t most) {
  const int64_t g = (n + kBlock - 1) / kBlock;
  return (int)(g < 1 ? 1 : (g > most ? most : g));
}

}  // namespace

void launch_cc_init(const CcArgs &a, const Csr &g, const Csr *gt, void *stream) {
  hipLaunchKernelGGL(k_cc_init, dim3(grid_of(std::max<int64_t>(a.n, kStatsCap), 4096)),
                     dim3(kBlock), 0, (hipStream_t)stream, a, g.iso, gt ? gt->iso : nullptr);
}

void launch_cc_step(const CcArgs &a, const Csr &g, const Csr *gt, int32_t it, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  int64_t *changed = a.changed + it % kStatsCap;
  const int64_t *prev = it > 0 ? a.changed + (it - 1) % kStatsCap : nullptr;
  const int grid = grid_of(a.nw * 64, kSweepGrid);  // a wave per word or run of words
  for (const Csr *c : {&g, gt}) {
    if (!c) continue;
    if (it == 0) hipLaunchKernelGGL(k_cc_sweep<true>, dim3(grid), dim3(kBlock), 0, s, a, *c, prev);
    else hipLaunchKernelGGL(k_cc_sweep<false>, dim3(grid), dim3(kBlock), 0, s, a, *c, prev);
  }
  hipLaunchKernelGGL(k_cc_grand, dim3(grid_of(a.n, 1024)), dim3(kBlock), 0, s, a, changed, prev);
}

}  // namespace grb
