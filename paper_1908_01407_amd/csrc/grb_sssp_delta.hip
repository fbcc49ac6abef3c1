// Bucketed SSSP: the min-plus relaxation of Section 7.2 of the paper
// processed in distance order, a near-far form of delta-stepping.  The
// paper's Bellman-Ford rounds relax every improved vertex at once, which on
// high-diameter graphs (road networks, grids) relaxes each edge over a
// hundred times; here a round relaxes only the pending vertices whose
// distance lies below the current limit, the end of a bucket of width delta,
// and the others wait in the pending set.  Once no vertex is left below the
// limit it moves to the end of the bucket of the smallest pending distance,
// which lies above that distance (grb_bucket.h).  Any order of
// relaxations reaches the same fixed point, so the distances are the exact
// shortest distances, identical to the Bellman-Ford rounds.
//
// One kernel per round, like the BFS levels and the Bellman-Ford rounds:
// * pending sets are bitmaps rotating through three buffers (read d, fill
//   d + 1, clear d + 2); each wave compacts the set bits of its words into a
//   queue of rows;
// * a queued row below the limit is relaxed (push, atomicMin on the float
//   bits) and leaves the set unless it improves again; a row above it is
//   carried into the next set;
// * the first setter of a bit counts the new member: near (below the
//   limit: size, degree sum, rows with pieces) or far (the smallest far
//   distance's bits), plus the pending total, all in striped counters.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "grb_bucket.h"
#include "grb_device.h"
#include "grb_internal.h"

namespace grb {
namespace {

// queue loop of this file: workgroups, queue segments (one per
// wave), segment counts read per lane of one wave
constexpr int kCoopGrid = kCoopGridSssp;
constexpr int kCoopSegs = kCoopGrid * (kCoopThreads / 64);
constexpr int kCoopSegsPerLane = kCoopSegs / 64;
static_assert(kCoopSegs % 64 == 0 && kCoopSegs <= kCoopSegsMax,
              "segment counts are read by one wave");

// far: bits of the smallest far distance (INT_MAX: none)
struct DCount {
  int near = 0, sd = 0, lng = 0, far = INT_MAX, pend = 0;
};

// Counts a new member of the next pending set with distance nd and out-
// degree pd.
__device__ __forceinline__ void count_new(int pd, float nd, float limit, DCount &c) {
  c.pend += 1;
  if (nd < limit) {
    c.near += 1;
    c.sd += pd;
    c.lng += pd > kPushSplit ? 1 : 0;
  } else {
    c.far = min(c.far, __float_as_int(nd));
  }
}

// Relaxes dist[c[s]] with nd[s] (c < 0: none); all reads, then all atomics,
// each beside the loads its success needs (the pending set's word, the
// target's degree), then all marks, then the counts.
__device__ __forceinline__ void relax_near(const SsspArgs &a, const int (&c)[kUnroll],
                                           const float (&nd)[kUnroll], float limit, DCount &cnt) {
  float cd[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) cd[s] = c[s] >= 0 ? a.dist[c[s]] : 0.0f;
  int old[kUnroll], r0[kUnroll], r1[kUnroll];
  uint64_t w[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    old[s] = 0;
    r0[s] = r1[s] = 0;
    w[s] = ~0ull;
    if (c[s] >= 0 && nd[s] < cd[s]) {
      old[s] = atomicMin((int *)&a.dist[c[s]], __float_as_int(nd[s]));
      w[s] = a.fnxt[c[s] >> 6];
      r0[s] = a.push.rp[c[s]];
      r1[s] = a.push.rp[c[s] + 1];
    }
  }
  uint64_t o[kUnroll];
#pragma unroll
  for (int s = 0; s < kUnroll; ++s) {
    o[s] = ~0ull;
    if (c[s] >= 0 && nd[s] < cd[s] && nd[s] < __int_as_float(old[s])) {
      const uint64_t b = 1ull << (c[s] & 63);
      if (!(w[s] & b))
        o[s] = atomicOr((unsigned long long *)&a.fnxt[c[s] >> 6], (unsigned long long)b);
    }
  }
#pragma unroll
  for (int s = 0; s < kUnroll; ++s)
    if (c[s] >= 0 && !(o[s] & (1ull << (c[s] & 63)))) count_new(r1[s] - r0[s], nd[s], limit, cnt);
}

__device__ void delta_push(const SsspArgs &a, int *mark, float limit, bool pieces, DCount &cnt) {
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *rp = a.push.rp, *ci = a.push.ci;
  for (int64_t w0 = gw; w0 < a.nw; w0 += 64 * nwaves) {
    const int64_t mw = w0 + (int64_t)ln * nwaves;
    uint64_t mf = 0ull;
    if (mw < a.nw) {
      a.fclr[mw] = 0ull;  // the set two rounds ahead
      mf = a.fcur[mw];
    }
    const int qc = __popcll(mf);
    const int qincl = wave_incl_scan(qc);
    const int qtotal = lane_last(qincl);
    for (int b = 0; b < qtotal; b += 64) {
      const int64_t u = queue_slot(mark, mf, qc, qincl, qtotal, b, mw);
      const float du = u >= 0 ? a.dist[u] : 0.0f;
      const bool active = u >= 0 && du < limit;
      // rows above the limit stay pending: one atomicOr per word (queued
      // rows are ascending), each lane then learns whether it was first
      const bool carry = u >= 0 && !active;
      const int64_t cw = carry ? (u >> 6) : -1;
      int tail;
      const uint64_t run = run_tail_or(cw, carry ? (1ull << (u & 63)) : 0ull, tail);
      uint64_t oldw = 0ull;
      if (run && cw >= 0) oldw = atomicOr((unsigned long long *)&a.fnxt[cw], (unsigned long long)run);
      oldw = __shfl(oldw, tail);
      if (carry && !((oldw >> (u & 63)) & 1ull)) {
        cnt.pend += 1;
        cnt.far = min(cnt.far, __float_as_int(du));
      }
      int cur = 0, end = 0;
      if (active) {
        cur = rp[u];
        end = rp[u + 1];
        if (end - cur > kPushSplit) end = cur;  // long rows: pieces below
      }
      for (bool more = true; more;) {
        int cc[kUnroll];
        float nd[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          cc[s] = -1;
          nd[s] = 0.0f;
          if (!more) continue;
          const int len = end - cur;
          const int incl = wave_incl_scan(len);
          const int total = lane_last(incl);
          if (total == 0) {
            more = false;
            continue;
          }
          const int excl = incl - len;
          const bool starts = len > 0 && excl < 64;
          const int r = slot_rows(mark, starts, excl);
          const int rcur = __shfl(cur, r), rexcl = __shfl(excl, r);
          const float rdu = __shfl(du, r);
          if (ln < total) {
            cc[s] = rcur + (ln - rexcl);
            nd[s] = rdu;
          }
          if (starts) cur += min(incl, 64) - excl;
        }
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          if (cc[s] >= 0) {
            const int pos = cc[s];
            cc[s] = ci[pos];
            nd[s] += a.wpush[pos];
          }
        }
        relax_near(a, cc, nd, limit, cnt);
      }
    }
  }
  if (!pieces) return;
  // pieces of long rows below the limit, spread over the waves
  static_assert(kPushSplit == 64 * kUnroll, "a piece is one unrolled step");
  for (int64_t hb = gw; hb < a.push.nsplit; hb += 64 * nwaves) {
    const int64_t h = hb + (int64_t)ln * nwaves;
    int u = -1, pbeg = 0, pend = 0;
    float du = 0.0f;
    if (h < a.push.nsplit) {
      u = a.push.split[2 * h];
      pbeg = a.push.split[2 * h + 1];
      if (bit_of(a.fcur, u)) {
        du = a.dist[u];
        if (du < limit) pend = min(pbeg + kPushSplit, rp[u + 1]);
        else u = -1;
      } else {
        u = -1;
      }
    }
    uint64_t act = __ballot(u >= 0);
    while (act) {
      const int k = __ffsll((unsigned long long)act) - 1;
      act &= act - 1;
      const int pb = __shfl(pbeg, k), pe = __shfl(pend, k);
      const float pdu = __shfl(du, k);
      int cc[kUnroll];
      float nd[kUnroll];
#pragma unroll
      for (int s = 0; s < kUnroll; ++s) {
        const int pos = pb + s * 64 + ln;
        cc[s] = pos < pe ? ci[pos] : -1;
        nd[s] = pos < pe ? pdu + a.wpush[pos] : 0.0f;
      }
      relax_near(a, cc, nd, limit, cnt);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_sssp_delta_round(SsspArgs a) {
  __shared__ int s_mark[kWavesPerBlock][64];
  __shared__ int s_pend, s_pieces;
  __shared__ float s_limit;
  __shared__ int s_red[kWavesPerBlock][kDeltaFields];
  if (threadIdx.x == 0) {
    int nr = 0, sd = 0, lg = 0, far = INT_MAX, pend = 0;
    int bucket = a.ctrl->bucket;
    float limit = a.ctrl->limit;
    for (int t = 0; t < kCntStripes; ++t) {
      nr += a.cnt_cur[kDeltaFields * t];
      sd += a.cnt_cur[kDeltaFields * t + 1];
      lg += a.cnt_cur[kDeltaFields * t + 2];
      far = min(far, a.cnt_cur[kDeltaFields * t + 3]);
      pend += a.cnt_cur[kDeltaFields * t + 4];
    }
    // stay in the bucket while it has members, else move to the nearest
    // pending one
    if (nr == 0) {
      bucket = bucket_of(__int_as_float(far), a.delta);
      limit = bucket_end(__int_as_float(far), a.delta);
    }
    s_limit = limit;
    s_pend = pend;
    // a row below the limit may be long although no long row was counted
    // near (its distance can drop after its first insertion), so the pieces
    // are skipped only when the graph has none
    s_pieces = a.push.nsplit > 0 ? 1 : 0;
    if (blockIdx.x == 0) {
      for (int t = 0; t < kCntStripes; ++t) {
        for (int f = 0; f < kDeltaFields; ++f)
          a.cnt_clr[kDeltaFields * t + f] = f == 3 ? INT_MAX : 0;
      }
      if (pend > 0) {
        a.ctrl->nlev = a.d + 1;
        a.ctrl->bucket = bucket;
        a.ctrl->limit = limit;
        if (a.stats && a.d < kStatsCap) {
          a.stats[a.d * kStatFields + 0] = pend;
          a.stats[a.d * kStatFields + 1] = sd;
          a.stats[a.d * kStatFields + 2] = GRB_DIR_PUSH;
          a.stats[a.d * kStatFields + 3] = bucket;
        }
      }
    }
  }
  __syncthreads();
  if (s_pend == 0) return;
  const float limit = s_limit;
  DCount c;
  delta_push(a, s_mark[threadIdx.x >> 6], limit, s_pieces != 0, c);
  c.near = wave_sum(c.near);
  c.sd = wave_sum(c.sd);
  c.lng = wave_sum(c.lng);
  c.pend = wave_sum(c.pend);
  c.far = lane_last(wave_scan(c.far, INT_MAX, [](int x, int y) { return x < y ? x : y; }));
  if ((threadIdx.x & 63) == 0) {
    const int wv = threadIdx.x >> 6;
    s_red[wv][0] = c.near;
    s_red[wv][1] = c.sd;
    s_red[wv][2] = c.lng;
    s_red[wv][3] = c.far;
    s_red[wv][4] = c.pend;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int nr = 0, sd = 0, lg = 0, far = INT_MAX, pend = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) {
      nr += s_red[i][0];
      sd += s_red[i][1];
      lg += s_red[i][2];
      far = min(far, s_red[i][3]);
      pend += s_red[i][4];
    }
    if (pend) {
      const int t = blockIdx.x % kCntStripes;
      if (nr) {
        atomicAdd(&a.cnt_nxt[kDeltaFields * t], nr);
        atomicAdd(&a.cnt_nxt[kDeltaFields * t + 1], sd);
        if (lg) atomicAdd(&a.cnt_nxt[kDeltaFields * t + 2], lg);
      }
      if (far != INT_MAX) atomicMin(&a.cnt_nxt[kDeltaFields * t + 3], far);
      atomicAdd(&a.cnt_nxt[kDeltaFields * t + 4], pend);
    }
  }
}

__global__ __launch_bounds__(kBlock) void k_sssp_delta_start(SsspArgs a, int32_t source,
                                                             uint64_t *f1, uint64_t *f2) {
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int ln = threadIdx.x & 63;
  const float inf = __int_as_float(0x7f800000);
  for (int64_t w = gw; w < a.nw; w += nwaves) {
    const int64_t v = w * 64 + ln;
    if (v < a.n) a.dist[v] = (v == source) ? 0.0f : inf;
    if (ln == 0) {
      a.fcur[w] = (w == (source >> 6)) ? (1ull << (source & 63)) : 0ull;
      f1[w] = 0ull;
      f2[w] = 0ull;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    for (int i = 0; i < kDeltaSlots; ++i) {
      const int v = (i % kDeltaFields) == 3 ? INT_MAX : 0;
      a.cnt_cur[i] = v;
      a.cnt_nxt[i] = v;
      a.cnt_clr[i] = v;
    }
    const int ds = a.push.rp[source + 1] - a.push.rp[source];
    a.cnt_cur[0] = 1;  // the source: near in bucket 0, pending
    a.cnt_cur[1] = ds;
    a.cnt_cur[2] = ds > kPushSplit ? 1 : 0;
    a.cnt_cur[4] = 1;
    a.ctrl->nlev = 0;
    a.ctrl->bucket = 0;
    a.ctrl->limit = bucket_end(0.0f, a.delta);
    a.ctrl->small_levels = INT_MAX;
    a.ctrl->spilled = 0;
    if (a.coop) {  // the multi-workgroup loop's first queue: {source}, near
      a.coop->bar = 0ull;
      for (int i = 0; i < kCoopSegsMax; ++i) {
        a.coop->cnt[0][i] = a.coop->esum[0][i] = a.coop->near[0][i] = 0;
        a.coop->far[0][i] = INT_MAX;
      }
      a.coop->cnt[0][0] = 1;
      a.coop->near[0][0] = 1;
      a.coop->esum[0][0] = ds;
      a.qv[0] = source;
      a.qe[0] = ((uint64_t)(uint32_t)ds << 32) | (uint32_t)a.push.rp[source];
    }
  }
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < a.own.nrec;
       i += (int64_t)gridDim.x * kBlock)
    a.own.rec[i] = 0ull;  // no tag
}

// ---- multi-workgroup bucket rounds while the pending set is small ----------
// The BFS level loop's scheme (grb_bfs.hip, k_bfs_own) for bucket rounds:
// workgroup w owns the vertices [w * chunk, (w + 1) * chunk); its pending
// vertices are two lists in its LDS, near (below the bucket's limit) and far,
// with a membership bit each, and it alone relaxes their distances, which sit
// in its LDS too (up to 64 workgroups of 32,704 vertices).  A round takes every
// near vertex: it relaxes the owned targets of its out-edges, which join the
// next near list or the far one, and sends the others (vertex, distance) to
// their owners.  Wave 0 then exchanges records with the other workgroups (words
// that carry the round's tag; the first message of each pair inside, more in a
// box), while the other waves load the next near vertices' rows and weights.
// Once no workgroup has a near vertex, a second exchange finds the smallest far
// distance, the limit moves past its bucket, and each workgroup splits its far
// list.
//
// A round's near vertices read their distance after leaving the list, so one
// improved again later in the round is queued again.  Messages are path
// lengths: applying one late or twice changes nothing, and a workgroup whose
// list or box is full marks the target in the pending bitmap (relaxed at once
// where it is another owner's) and the loop hands over.  The same goes for an
// exchange given up: each workgroup leaves with its distances and lists
// written back, whatever round it reached, the hand-over applies every message
// still in the boxes, and the round kernels continue from the pending bitmap.
// List entries per workgroup (LDS: 160 KB in all; 16 bits each).  A front that
// lies along a workgroup's rows puts it all there: up to 1,672 near vertices
// and 776 far ones on the 2003 x 1009 grid, more with those queued again.
constexpr int kNearCap = 4096, kFarCap = 3072;
struct DeltaShared {
  float dist[kDeltaOwnLds];
  uint32_t nbit[kDeltaOwnLds / 32], fbit[kDeltaOwnLds / 32];
  uint16_t near[2][kNearCap];
  uint16_t far[kFarCap];
  int cnt[2], nfar, nkeep;
  int out[kDeltaMaxGroups];   // messages to each workgroup in this round
  int midx[kDeltaMaxGroups];  // the first of each: vertex (within its owner) and distance
  float mdist[kDeltaMaxGroups];
  int pre[kDeltaMaxGroups + 1];  // prefix of the boxes' further messages
  int sent_near, edges, ovf, n_new, nin, state, gave_up;
  float limit;
};
enum DeltaState { kDeltaGo = 0, kDeltaAdvance = 1, kDeltaSpill = 2 };

__device__ __forceinline__ uint32_t delta_tag(int round) { return 1u + (uint32_t)round % 8190u; }
__device__ __forceinline__ uint64_t delta_head(uint32_t tag, int idx, float d) {
  return ((uint64_t)((tag << 19) | (uint32_t)idx) << 32) | __float_as_uint(d);
}
__device__ __forceinline__ uint64_t delta_total(uint32_t tag, int cnt, bool near, bool ovf) {
  return ((uint64_t)tag << 51) | ((uint64_t)cnt << 2) | (near ? 2ull : 0ull) | (ovf ? 1ull : 0ull);
}
static_assert(kDeltaOwnLds <= 1 << 16 && kDeltaCapMax < 1 << 13 && kDeltaMaxGroups == 64,
              "fields of the record words; a lane of wave 0 per workgroup");

__device__ __forceinline__ float own_relax(DeltaShared &sh, int l, float nd) {
  return __int_as_float(atomicMin((int *)&sh.dist[l], __float_as_int(nd)));
}

// Appends the wanted ones among local vertices l[0..K) to a list (all 64
// lanes call it; one LDS atomic per wave); past its end a vertex is marked in
// the pending bitmap.
template <int K>
__device__ __forceinline__ void list_add(DeltaShared &sh, uint64_t *pend, int lo, const bool (&want)[K],
                                         const int (&l)[K], int *cnt, uint16_t *list, int cap) {
  uint64_t b[K];
  int tot = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    b[k] = __ballot(want[k]);
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
    if (!want[k]) continue;
    if (slot < cap) {
      list[slot] = (uint16_t)l[k];
    } else {
      const int c = lo + l[k];
      atomicOr((unsigned long long *)&pend[c >> 6], 1ull << (c & 63));
      sh.ovf = 1;
    }
  }
}

// Owned targets whose distance was lowered to nd join the near or the far
// list unless they are there already (all bit atomics before any result).
template <int K>
__device__ __forceinline__ void improved(DeltaShared &sh, uint64_t *pend, int lo, const bool (&imp)[K],
                                         const int (&l)[K], const float (&nd)[K], float limit,
                                         int *cnt, uint16_t *list) {
  uint32_t old[K];
  bool any = false, nr[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    nr[k] = nd[k] < limit;
    any |= imp[k];
    old[k] = ~0u;
    if (imp[k]) old[k] = atomicOr((nr[k] ? sh.nbit : sh.fbit) + (l[k] >> 5), 1u << (l[k] & 31));
  }
  if (__ballot(any) == 0ull) return;
  bool add_n[K], add_f[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const bool fresh = !((old[k] >> (l[k] & 31)) & 1u);
    add_n[k] = fresh && nr[k];
    add_f[k] = fresh && !nr[k];
  }
  list_add<K>(sh, pend, lo, add_n, l, cnt, list, kNearCap);
  list_add<K>(sh, pend, lo, add_f, l, &sh.nfar, sh.far, kFarCap);
}

// Relaxes the targets c[0..4) (none: -1) with distances nd.
__device__ __forceinline__ void delta_expand(const SsspArgs &a, DeltaShared &sh, uint64_t *pend, int lo,
                                             int nv, int w, float limit, int *cnt, uint16_t *list,
                                             uint64_t *box, const int (&c)[4],
                                             const float (&nd)[4]) {
  float old[4];
  bool far = false;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t l = (uint32_t)(c[k] - lo);
    const bool own = l < (uint32_t)nv;
    far |= c[k] >= 0 && !own;
    old[k] = 0.0f;
    if (own) old[k] = own_relax(sh, (int)l, nd[k]);
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
      if (nd[k] < limit) sh.sent_near = 1;
      if (slot == 0) {
        sh.midx[o] = m;
        sh.mdist[o] = nd[k];
      } else if (slot < cap) {
        store_relaxed_u64(&box[((int64_t)w * G + o) * cap + slot],
                          ((uint64_t)(uint32_t)m << 32) | __float_as_uint(nd[k]));
      } else {  // box full: relaxed in device memory; the target stays pending
        atomicMin((int *)&a.dist[c[k]], __float_as_int(nd[k]));
        atomicOr((unsigned long long *)&pend[c[k] >> 6], 1ull << (c[k] & 63));
        sh.ovf = 1;
      }
    }
  }
  bool imp[4];
  int l[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    l[k] = c[k] - lo;
    imp[k] = (uint32_t)l[k] < (uint32_t)nv && nd[k] < old[k];
  }
  improved<4>(sh, pend, lo, imp, l, nd, limit, cnt, list);
}

__device__ __forceinline__ int wave_add(int x) { return lane_last(wave_incl_scan(x)); }

// Bucket rounds back to back, bound by each round's chain as the BFS loop's
// levels are: the owner of a run of vertices keeps their distances in LDS, an
// improvement of another owner's vertex is a message.  2003 x 1009 grid, width
// 512, 62 workgroups, from two sources: 12.5 and 19.4 ms; the queue loop below,
// whose distances are in device memory, 18.9 and 26.4 ms (about 8 us a round;
// one workgroup on graphs that fit it takes 2.6 us).
__global__ __launch_bounds__(kOwnThreads) void k_sssp_delta_own(SsspArgs a, int32_t source,
                                                                int max_rounds,
                                                                uint64_t wait_ticks,
                                                                uint64_t *pend) {
  __shared__ DeltaShared sh;
  constexpr int T = kOwnThreads - 64;  // threads that take near vertices (waves 1, 2, ...)
  const int tid = threadIdx.x, ln = tid & 63;
  const int et = tid - 64;
  const int w = (int)blockIdx.x, G = a.own.groups, cap = a.own.cap;
  const int32_t *rp = a.push.rp, *ci = a.push.ci;
  const float *wt = a.wpush;
  const float inf = __int_as_float(0x7f800000);
  const int64_t first = (int64_t)w * a.own.chunk;
  const int lo = (int)(first < a.n ? first : a.n);
  const int nv = (int)(a.n - lo < a.own.chunk ? a.n - lo : a.own.chunk);  // vertices owned
  for (int i = tid; i < (nv + 31) / 32; i += kOwnThreads) sh.nbit[i] = sh.fbit[i] = 0u;
  for (int i = tid; i < nv; i += kOwnThreads) sh.dist[i] = lo + i == source ? 0.0f : inf;
  for (int i = tid; i < kDeltaMaxGroups; i += kOwnThreads) {
    sh.out[i] = sh.midx[i] = 0;
    sh.mdist[i] = 0.0f;
  }
  const bool mine = source >= lo && source - lo < nv;
  if (tid == 0) {
    sh.cnt[0] = sh.cnt[1] = sh.nfar = 0;
    sh.sent_near = sh.edges = sh.ovf = 0;
    sh.near[0][0] = (uint16_t)(source - lo);
  }
  __syncthreads();
  if (tid == 0 && mine) sh.nbit[(source - lo) >> 5] = 1u << ((source - lo) & 31);
  __syncthreads();
  int n = mine ? 1 : 0, npre = 0;
  int prs = 0, pdg = 0, pc[4] = {-1, -1, -1, -1};
  float pw[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  float limit = bucket_end(0.0f, a.delta);
  int bucket = 0;
  uint64_t *box = a.own.box64, *box1 = box + (int64_t)G * G * cap;
  uint64_t *put = a.own.rec + 2 * ((int64_t)ln * G + w);
  uint64_t *get = a.own.rec + 2 * ((int64_t)w * G + ln);
  uint64_t *put1 = put + (int64_t)G * G * 2, *get1 = get + (int64_t)G * G * 2;
  uint32_t tag = delta_tag(0);
  int cur = 0, d = 0, slow = 0;  // near list, round, second exchanges so far
  bool spill = false, over = false;  // over: this round's near list is not whole
  for (;;) {
    const int nxt = cur ^ 1;
    const bool rec_round = d < kStatsCap;
    if (over) {
      // The messages of the last round left near vertices beyond the list's end:
      // this workgroup's part of the round goes to the hand-over as it is.
      for (int i = tid; i < n; i += kOwnThreads) {
        const int c = lo + sh.near[cur][i];
        atomicOr((unsigned long long *)&pend[c >> 6], 1ull << (c & 63));
      }
    } else if (et >= 0) {
      int esum = 0;
      for (int i0 = et & ~63; i0 < n; i0 += T) {
        const int i = i0 + ln;
        int l = 0, rs = 0, dg = 0, c[4] = {-1, -1, -1, -1};
        float dv = 0.0f, x[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (i < n) {
          l = sh.near[cur][i];
          // off the list before its distance is read
          atomicAnd(&sh.nbit[l >> 5], ~(1u << (l & 31)));
          dv = *(volatile float *)&sh.dist[l];
          if (i0 < T && i < npre) {
            rs = prs;
            dg = pdg;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              c[q] = pc[q];
              x[q] = pw[q];
            }
          } else {
            rs = rp[lo + l];
            dg = rp[lo + l + 1] - rs;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              c[q] = q < dg ? ci[rs + q] : -1;
              x[q] = q < dg ? wt[rs + q] : 0.0f;
            }
          }
        }
        esum += dg;
        float nd[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) nd[q] = dv + x[q];
        delta_expand(a, sh, pend, lo, nv, w, limit, &sh.cnt[nxt], sh.near[nxt], box, c, nd);
        for (int q0 = 4; __ballot(q0 < dg) != 0ull; q0 += 4) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            c[q] = q0 + q < dg ? ci[rs + q0 + q] : -1;
            nd[q] = dv + (q0 + q < dg ? wt[rs + q0 + q] : 0.0f);
          }
          delta_expand(a, sh, pend, lo, nv, w, limit, &sh.cnt[nxt], sh.near[nxt], box, c, nd);
        }
      }
      if (rec_round) {
        esum = wave_add(esum);
        if (ln == 0 && esum) atomicAdd(&sh.edges, esum);
      }
      __builtin_amdgcn_s_waitcnt(0);  // box stores are done before the heads go out
    }
    __syncthreads();
    const int nl = min(sh.cnt[nxt], kNearCap);
    if (et < 0) {
      int nin = 0, state = kDeltaGo, gave_up = 0;
      int np = n + sh.nfar, ne = sh.edges;
      bool any_n = n > 0;
      if (G == 1) {
        if (sh.ovf) state = kDeltaSpill;
        else if (nl == 0) state = kDeltaAdvance;
        if (ln == 0) sh.n_new = nl;
      } else {
        const bool nr = nl > 0 || sh.sent_near != 0, ov = sh.ovf != 0;
        uint64_t hd = 0ull, tt = 0ull;
        if (ln < G) {
          const int k = sh.out[ln];
          store_relaxed_u64(put, delta_head(tag, sh.midx[ln], sh.mdist[ln]));
          store_relaxed_u64(put + 1, delta_total(tag, min(k, cap), nr, ov));
          if (k) sh.out[ln] = 0;
        }
        if (rec_round && ln == 0)
          store_relaxed_u64(&a.own.rec_edges[(d & 1) * G + w],
                            ((uint64_t)tag << 51) | ((uint64_t)(uint32_t)min(np, 0xfffff) << 31) |
                                (uint32_t)ne);
        uint64_t t0 = 0;
        for (;;) {
          bool ok = true;
          if (ln < G) {
            hd = load_relaxed_u64(get);
            tt = load_relaxed_u64(get + 1);
            ok = (uint32_t)(hd >> 51) == tag && (uint32_t)(tt >> 51) == tag;
          }
          if (__ballot(!ok) == 0ull) break;
          if (t0 == 0) t0 = wall_clock64();
          if (wall_clock64() - t0 >= (d == 0 ? kCoopFirstWait : 1) * wait_ticks) {
            gave_up = 1;
            state = kDeltaSpill;
            break;
          }
        }
        if (ln == 0) sh.n_new = nl;  // only this wave appends until the next sync
        if (!gave_up) {
          const int k = (int)(tt >> 2) & 8191;  // messages from workgroup ln
          if (__ballot(k > 0)) {
            const int l[1] = {(int)(hd >> 32) & 0x7ffff};
            const float nd[1] = {__uint_as_float((uint32_t)hd)};
            float old = 0.0f;
            if (k > 0) old = own_relax(sh, l[0], nd[0]);
            const bool imp[1] = {k > 0 && nd[0] < old};
            improved<1>(sh, pend, lo, imp, l, nd, limit, &sh.n_new, sh.near[nxt]);
          }
          if (__ballot((tt & 1ull) != 0)) state = kDeltaSpill;
          else if (__ballot((tt & 2ull) != 0) == 0ull) state = kDeltaAdvance;
          if (__ballot(k > 1)) {  // boxes: prefix of the further messages
            const int in = max(k - 1, 0);
            const int incl = wave_incl_scan(in);
            sh.pre[ln + 1] = incl;
            if (ln == 0) sh.pre[0] = 0;
            nin = lane_last(incl);
          }
          if (w == 0 && rec_round) {
            np = ne = 0;
            for (int sd = ln; sd < G; sd += 64) {
              uint64_t x;
              t0 = wall_clock64();
              do {
                x = load_relaxed_u64(&a.own.rec_edges[(d & 1) * G + sd]);
              } while ((uint32_t)(x >> 51) != tag && wall_clock64() - t0 < kCoopWaitTicks);
              np += (int)(x >> 31) & 0xfffff;
              ne += (int)(x & 0x7fffffffull);
            }
            np = wave_add(np);
            ne = wave_add(ne);
          }
          any_n = true;  // (a round starts only with a near vertex somewhere, or a message)
        }
      }
      if (ln == 0) {
        sh.state = state;
        sh.gave_up = gave_up;
        sh.nin = nin;
        sh.cnt[cur] = 0;
        sh.sent_near = 0;
        if (rec_round) sh.edges = 0;
        if (w == 0 && !gave_up && any_n) {
          a.ctrl->nlev = d + 1;
          if (rec_round && a.stats) {
            a.stats[d * kStatFields + 0] = np;
            a.stats[d * kStatFields + 1] = ne;
            a.stats[d * kStatFields + 2] = GRB_DIR_PUSH;
            a.stats[d * kStatFields + 3] = bucket;
          }
        }
      }
    } else {
      // beside the exchange: rows, first columns and weights of the next round
      prs = pdg = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        pc[q] = -1;
        pw[q] = 0.0f;
      }
      if (et < nl) {
        const int v = lo + sh.near[nxt][et];
        prs = rp[v];
        pdg = rp[v + 1] - prs;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q < pdg) {
            pc[q] = ci[prs + q];
            pw[q] = wt[prs + q];
          }
      }
    }
    npre = min(nl, T);
    __syncthreads();
    ++d;
    const int state = sh.state;
    if (sh.gave_up) {
      n = min(sh.n_new, kNearCap);
      cur = nxt;
      spill = true;
      break;
    }
    const int nin = sh.nin;
    if (nin > 0) {  // further messages, from the boxes
      for (int i0 = tid & ~63; i0 < nin; i0 += kOwnThreads) {
        const int i = i0 + ln;
        int l = 0;
        float nd = 0.0f, old = 0.0f;
        if (i < nin) {
          int sd = 0;  // the sender: the last one with pre[sd] <= i
#pragma unroll
          for (int step = 32; step > 0; step >>= 1)
            if (sh.pre[sd + step] <= i) sd += step;
          const uint64_t x =
              load_relaxed_u64(&box[((int64_t)sd * G + w) * cap + 1 + (i - sh.pre[sd])]);
          l = (int)(x >> 32);
          nd = __uint_as_float((uint32_t)x);
          old = own_relax(sh, l, nd);
        }
        const bool imp[1] = {i < nin && nd < old};
        const int la[1] = {l};
        const float na[1] = {nd};
        improved<1>(sh, pend, lo, imp, la, na, limit, &sh.n_new, sh.near[nxt]);
      }
      __syncthreads();
    }
    n = min(sh.n_new, kNearCap);
    cur = nxt;
    {
      uint64_t *b = box, *p = put, *g = get;
      box = box1, box1 = b;
      put = put1, put1 = p;
      get = get1, get1 = g;
      tag = delta_tag(d);
    }
    if (state == kDeltaSpill || d >= kOwnMaxLevels) {
      spill = true;
      break;
    }
    if (d >= max_rounds) break;
    over = sh.n_new > kNearCap;
    if (state != kDeltaAdvance) continue;
    // No near vertex was left anywhere before the messages of this round,
    // and none of those was below the limit: the next bucket.  A full list
    // since then hands over here.
    const int nf = min(sh.nfar, kFarCap);
    float m = inf;
    for (int i = tid; i < nf; i += kOwnThreads) {
      const float x = sh.dist[sh.far[i]];
      if (x >= limit) m = fminf(m, x);  // (below: relaxed since, from the near list)
    }
    m = wave_min(m);
    __syncthreads();
    if (tid == 0) {
      sh.limit = inf;
      sh.nkeep = 0;
    }
    __syncthreads();
    if (ln == 0) atomicMin((int *)&sh.limit, __float_as_int(m));
    __syncthreads();
    if (et < 0) {
      float mm = sh.limit;
      int gave_up = 0;
      bool ov = sh.ovf != 0;
      if (G > 1) {
        uint64_t *r2 = a.own.rec2 + (slow & 1) * G;
        const uint32_t tag2 = delta_tag(slow);
        if (ln == 0)
          store_relaxed_u64(&r2[w], ((uint64_t)tag2 << 51) | ((uint64_t)(ov ? 1u : 0u) << 32) |
                                        __float_as_uint(mm));
        const uint64_t t0 = wall_clock64();
        for (;;) {
          bool ok = true, o1 = false;
          mm = inf;
          for (int sd = ln; sd < G; sd += 64) {
            const uint64_t x = load_relaxed_u64(&r2[sd]);
            ok &= (uint32_t)(x >> 51) == tag2;
            mm = fminf(mm, __uint_as_float((uint32_t)x));
            o1 |= ((x >> 32) & 1ull) != 0;
          }
          if (__ballot(!ok) == 0ull) {
            mm = wave_min(mm);
            ov = __ballot(o1) != 0ull;
            break;
          }
          if (wall_clock64() - t0 >= wait_ticks) {
            gave_up = 1;
            break;
          }
        }
      }
      if (ln == 0) {
        sh.gave_up = gave_up;
        sh.limit = mm;
        sh.state = ov ? kDeltaSpill : kDeltaGo;
      }
    }
    ++slow;
    __syncthreads();
    const float mm = sh.limit;
    if (sh.gave_up || sh.state == kDeltaSpill) {
      spill = true;
      break;
    }
    if (!(mm < inf)) break;  // nothing pending anywhere: done
    const float was = limit;
    limit = bucket_end(mm, a.delta);
    bucket = bucket_of(mm, a.delta);
    if (w == 0 && tid == 0) {
      a.ctrl->bucket = bucket;
      a.ctrl->limit = limit;
    }
    // split the far list in place, kOwnThreads entries at a time
    if (tid == 0) sh.cnt[cur] = 0;
    for (int b = 0; b < nf; b += kOwnThreads) {
      const int i = b + tid;
      const int l = i < nf ? sh.far[i] : 0;
      const float x = i < nf ? sh.dist[l] : inf;
      __syncthreads();
      // entries below the old limit were relaxed since they joined the list
      bool add = false;
      const bool keep = i < nf && x >= limit;
      if (i < nf && !keep) {
        atomicAnd(&sh.fbit[l >> 5], ~(1u << (l & 31)));
        if (x >= was) add = !((atomicOr(&sh.nbit[l >> 5], 1u << (l & 31)) >> (l & 31)) & 1u);
      }
      const bool an[1] = {add}, kp[1] = {keep};
      const int la[1] = {l};
      list_add<1>(sh, pend, lo, an, la, &sh.cnt[cur], sh.near[cur], kNearCap);
      list_add<1>(sh, pend, lo, kp, la, &sh.nkeep, sh.far, kFarCap);
      __syncthreads();
    }
    __syncthreads();
    n = min(sh.cnt[cur], kNearCap);
    npre = 0;
    if (tid == 0) sh.nfar = sh.nkeep;
    __syncthreads();
  }
  // Distances and, where the loop hands over, the pending vertices.  A message
  // that found its box full lowered the distance in device memory: every
  // workgroup saw its sender's flag and spills, also at the round cap.
  if (!spill) {
    for (int i = tid; i < nv; i += kOwnThreads) a.dist[lo + i] = sh.dist[i];
  } else {
    for (int i = tid; i < nv; i += kOwnThreads)
      atomicMin((int *)&a.dist[lo + i], __float_as_int(sh.dist[i]));
    const int nf = min(sh.nfar, kFarCap);
    for (int i = tid; i < n + nf; i += kOwnThreads) {
      const int c = lo + (i < n ? sh.near[cur][i] : sh.far[i - n]);
      atomicOr((unsigned long long *)&pend[c >> 6], 1ull << (c & 63));
    }
  }
  if (tid == 0) {
    // (a round left to the hand-over is not one of the loop's)
    atomicMin(&a.ctrl->small_levels, over ? d - 1 : d);
    if (spill) atomicOr(&a.ctrl->spilled, 1);
  }
}

// After a loop that spilled: every message still in the boxes is applied
// (most were: then it lowers nothing), its target joining the pending bitmap
// where it does ...
__global__ __launch_bounds__(kBlock) void k_sssp_delta_own_boxes(SsspArgs a, uint64_t *pend) {
  if (!a.ctrl->spilled) return;
  const int G = a.own.groups, cap = a.own.cap;
  if (G > 1) {
    const int64_t m = (int64_t)2 * G * G * cap, nt = (int64_t)gridDim.x * kBlock;
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < m; t += nt) {
      const int64_t pair = t / cap;
      const int j = (int)(t % cap), par = (int)(pair / ((int64_t)G * G));
      const int sd = (int)(pair / G % G), o = (int)(pair % G);
      const uint64_t *rec = a.own.rec + 2 * (((int64_t)par * G + o) * G + sd);
      if (j >= ((int)(rec[1] >> 2) & 8191)) continue;
      const uint64_t x = j == 0 ? rec[0] : a.own.box64[t];
      const int c = o * a.own.chunk + ((int)(x >> 32) & 0x7ffff);
      const float nd = __uint_as_float((uint32_t)x);
      if (nd < __int_as_float(atomicMin((int *)&a.dist[c], __float_as_int(nd))))
        atomicOr((unsigned long long *)&pend[c >> 6], 1ull << (c & 63));
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0)
    for (int i = 0; i < 3 * kDeltaSlots; ++i)
      a.ctrl->lists[i] = (i % kDeltaFields) == 3 ? INT_MAX : 0;
}

// ... then the bitmap (pend = F1) becomes that of round h =
// ctrl->small_levels for the round kernel, with the round's counters.
__global__ __launch_bounds__(kBlock) void k_sssp_delta_own_handover(SsspArgs a, uint64_t *F0,
                                                                     uint64_t *F1, uint64_t *F2) {
  if (!a.ctrl->spilled) return;
  const int h = a.ctrl->small_levels;
  uint64_t *const F[3] = {F0, F1, F2};
  const float limit = a.ctrl->limit;
  const int ln = threadIdx.x & 63;
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  DCount c;
  for (int64_t w0 = gw * 64; w0 < a.nw; w0 += nwaves * 64) {
    const int64_t mw = w0 + ln;
    const uint64_t x = mw < a.nw ? F1[mw] : 0ull;
    if (mw < a.nw) {
      F0[mw] = F1[mw] = F2[mw] = 0ull;
      F[h % 3][mw] = x;
    }
    for (uint64_t any = __ballot(x != 0ull); any; any &= any - 1) {
      const int k = __ffsll((unsigned long long)any) - 1;
      const uint64_t xk = __shfl(x, k);
      const int64_t v = (w0 + k) * 64 + ln;
      if ((xk >> ln) & 1ull) count_new(a.push.rp[v + 1] - a.push.rp[v], a.dist[v], limit, c);
    }
  }
  c.near = wave_sum(c.near);
  c.sd = wave_sum(c.sd);
  c.pend = wave_sum(c.pend);
  c.far = lane_last(wave_scan(c.far, INT_MAX, [](int x, int y) { return x < y ? x : y; }));
  if (ln == 0 && c.pend) {  // rows are at most kCoopMaxDeg long: none has pieces
    int32_t *cnt = a.ctrl->lists + (h % 3) * kDeltaSlots + kDeltaFields * (gw % kCntStripes);
    atomicAdd(&cnt[0], c.near);
    atomicAdd(&cnt[1], c.sd);
    if (c.far != INT_MAX) atomicMin(&cnt[3], c.far);
    atomicAdd(&cnt[4], c.pend);
  }
}

// ---- bucket rounds of larger graphs: a queue in device memory ----------------
// The pending set as a queue in device memory (one segment per wave of the
// loop; entries: vertex, row start | degree << 32) with membership bits in
// F0 / F1 (round d consumes F[d & 1] and fills F[(d + 1) & 1]).  A vertex
// may be queued more than once in a round (each improvement queues it); the
// consumer whose atomicAnd clears its membership bit takes it, and the
// other copies are skipped.  A round: workgroup w takes the entries
// [w n / G, (w + 1) n / G), a thread per entry, which clears the member's
// bit and reads its distance together with its first four out-edges and
// weights; a member below the bucket's limit relaxes its edges (atomicMin
// on the float bits, the target's row extents loaded beside) and queues
// every target it improved, a member above it is queued again (carried).
// Per wave: entries queued, near ones (below the limit), their degree sum,
// the smallest distance of the others.  The limit moves to the end of that
// one's bucket when no near member is left.  A pending set that outgrows
// the segments (or the loop's edge limit) goes to the round kernel.
// Queues in the wave's segment of the next queue (slots counted in wcnt);
// every queued vertex gets its membership bit, also past the segment's end.
__device__ __forceinline__ void coop_queue(bool want, int x, int rs, int dg, float dx, float limit,
                                           uint64_t *fill, int32_t *qv, uint64_t *qe,
                                           int seg, int &wcnt, int &wnear, int &wsd, int &wfar) {
  const int ln = threadIdx.x & 63;
  const uint64_t m = __ballot(want);
  if (m == 0ull) return;
  const bool nr = want && dx < limit;
  wnear += wave_sum(nr ? 1 : 0);
  wsd += wave_sum(nr ? dg : 0);
  const int far = (want && !nr) ? __float_as_int(dx) : INT_MAX;
  wfar = min(wfar, lane_last(wave_scan(far, INT_MAX, [](int p, int q) { return p < q ? p : q; })));
  if (want) {
    const int slot = wcnt + __popcll(m & mask_below(ln));
    atomicOr((unsigned long long *)&fill[x >> 6], 1ull << (x & 63));
    if (slot < seg) {
      st_coherent(qv + slot, x);
      store_relaxed_u64(qe + slot, ((uint64_t)(uint32_t)dg << 32) | (uint32_t)rs);
    }
  }
  wcnt += __popcll(m);
}

__global__ __launch_bounds__(kCoopThreads) void k_sssp_delta_coop(SsspArgs a, int64_t max_rounds,
                                                                  uint64_t wait_ticks,
                                                                  uint64_t *F0, uint64_t *F1) {
  __shared__ int s_pre[kCoopSegs + 1];
  __shared__ int s_n, s_near, s_sd, s_far, s_ovf, s_go;
  const int tid = threadIdx.x, ln = tid & 63;
  const int32_t *rp = a.push.rp, *ci = a.push.ci;
  const float *wt = a.wpush;
  CoopCtl *cc = a.coop;
  const int w = (int)blockIdx.x;
  const int my_seg = w * (kCoopThreads / 64) + (tid >> 6);
  const int seg = a.qseg, qsize = kCoopSegs * seg;
  int bucket = 0;
  float limit = bucket_end(0.0f, a.delta);
  int64_t d = 0;
  bool spill = false;
  for (;;) {
    const int sl = (int)(d & 1);
    if (tid < 64) {  // the round's queue: segment counts and their prefix, totals
      // lane l holds segments kCoopSegsPerLane * l + r
      int c[kCoopSegsPerLane], csum = 0, nr = 0, e = 0, f = INT_MAX;
      bool over = false;
#pragma unroll
      for (int r = 0; r < kCoopSegsPerLane; ++r) {
        const int sg = kCoopSegsPerLane * tid + r;
        c[r] = ld_coherent(&cc->cnt[sl][sg]);
        nr += ld_coherent(&cc->near[sl][sg]);
        e += ld_coherent(&cc->esum[sl][sg]);
        f = min(f, ld_coherent(&cc->far[sl][sg]));
        csum += c[r];
        over |= c[r] > seg;
      }
      const int incl = wave_incl_scan(csum);
      int run = incl - csum;
#pragma unroll
      for (int r = 0; r < kCoopSegsPerLane; ++r) {
        run += c[r];
        s_pre[kCoopSegsPerLane * tid + r + 1] = run;
      }
      const int tot = lane_last(incl), nt = wave_sum(nr), et = wave_sum(e);
      const int ft = lane_last(wave_scan(f, INT_MAX, [](int p, int q) { return p < q ? p : q; }));
      const bool ovf = __ballot(over) != 0ull;
      if (tid == 0) {
        s_pre[0] = 0;
        s_n = tot;
        s_near = nt;
        s_sd = et;
        s_far = ft;
        s_ovf = ovf ? 1 : 0;
      }
    }
    __syncthreads();
    const int n = s_n;
    if (n == 0 || d >= max_rounds) break;
    if (s_ovf || s_sd > kCoopEdges || d >= kCoopMaxLevels) {
      spill = true;
      break;
    }
    if (s_near == 0) {
      bucket = bucket_of(__int_as_float(s_far), a.delta);
      limit = bucket_end(__int_as_float(s_far), a.delta);
    }
    if (w == 0 && tid == 0) {
      a.ctrl->nlev = (int)d + 1;
      a.ctrl->bucket = bucket;
      a.ctrl->limit = limit;
      if (a.stats && d < kStatsCap) {
        a.stats[d * kStatFields + 0] = n;
        a.stats[d * kStatFields + 1] = s_sd;
        a.stats[d * kStatFields + 2] = GRB_DIR_PUSH;
        a.stats[d * kStatFields + 3] = bucket;
      }
    }
    uint64_t *const cons = sl ? F1 : F0, *const fill = sl ? F0 : F1;
    const int qin = sl * qsize, qout = (sl ^ 1) * qsize + my_seg * seg;
    int32_t *const qvo = a.qv + qout;
    uint64_t *const qeo = a.qe + qout;
    const int lo = (int)((int64_t)n * w / kCoopGrid);
    const int hi = (int)((int64_t)n * (w + 1) / kCoopGrid);
    int wcnt = 0, wnear = 0, wsd = 0, wfar = INT_MAX;  // uniform over the wave
    for (int base = lo; base < hi; base += kCoopThreads) {
      const int i = base + tid;
      int v = -1, rs = 0, dg = 0;
      if (i < hi) {
        int s = 0;  // segment holding entry i: the last s with s_pre[s] <= i
#pragma unroll
        for (int step = kCoopSegs / 2; step > 0; step >>= 1)
          if (s_pre[s + step] <= i) s += step;
        const int at = qin + s * seg + (i - s_pre[s]);
        v = ld_coherent(a.qv + at);
        const uint64_t e = load_relaxed_u64(a.qe + at);
        rs = (int)(uint32_t)e;
        dg = (int)(e >> 32);
      }
      bool take = false;
      float dv = 0.0f;
      int c0[4];
      float w0[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c0[q] = -1;
        w0[q] = 0.0f;
      }
      if (v >= 0) {
        const uint64_t bit = 1ull << (v & 63);
        const uint64_t was = atomicAnd((unsigned long long *)&cons[v >> 6], ~bit);
        dv = __int_as_float(ld_coherent((const int32_t *)&a.dist[v]));
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q < dg) {
            c0[q] = ci[rs + q];
            w0[q] = wt[rs + q];
          }
        take = (was & bit) != 0ull;
      }
      const bool relax = take && dv < limit;
      // carried: a member above the limit stays pending
      coop_queue(take && !relax, v, rs, dg, dv, limit, fill, qvo, qeo, seg, wcnt, wnear,
                 wsd, wfar);
      for (int q0 = 0; __ballot(relax && q0 < dg) != 0ull; q0 += 4) {
        int c[4];
        float nd[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bool ok = relax && q0 + q < dg;
          c[q] = !ok ? -1 : (q0 == 0 ? c0[q] : ci[rs + q0 + q]);
          nd[q] = !ok ? 0.0f : dv + (q0 == 0 ? w0[q] : wt[rs + q0 + q]);
        }
        int old[4], r0[4], r1[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          old[q] = 0;
          r0[q] = r1[q] = 0;
          if (c[q] >= 0) {
            old[q] = atomicMin((int *)&a.dist[c[q]], __float_as_int(nd[q]));
            r0[q] = rp[c[q]];
            r1[q] = rp[c[q] + 1];
          }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
          coop_queue(c[q] >= 0 && nd[q] < __int_as_float(old[q]), c[q], r0[q], r1[q] - r0[q],
                     nd[q], limit, fill, qvo, qeo, seg, wcnt, wnear, wsd, wfar);
      }
    }
    // the wave's segment counters go with its entries; the barrier follows
    // once every memory operation of the workgroup is done
    if (ln == 0) {
      st_coherent(&cc->cnt[sl ^ 1][my_seg], wcnt);
      st_coherent(&cc->near[sl ^ 1][my_seg], wnear);
      st_coherent(&cc->esum[sl ^ 1][my_seg], wsd);
      st_coherent(&cc->far[sl ^ 1][my_seg], wfar);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (tid == 0) s_go = coop_barrier(&cc->bar, kCoopGrid, d, wait_ticks);
    __syncthreads();
    ++d;
    if (!s_go) {
      // barrier given up: the pending set of round d (complete: every
      // workgroup finished round d - 1) goes to the round kernel
      spill = true;
      break;
    }
  }
  if (w == 0 && tid == 0) {
    a.ctrl->small_levels = (int)d;
    a.ctrl->spilled = spill ? 1 : 0;
  }
}

// After the loop spilled at round h = ctrl->small_levels: its pending set
// (bitmap F[h & 1] of F0 / F1) becomes the round kernel's F[h % 3] (every
// other buffer is zero), with the counters and bucket of round h.
__global__ __launch_bounds__(kBlock) void k_sssp_delta_coop_handover(SsspArgs a, uint64_t *F0,
                                                                      uint64_t *F1,
                                                                      uint64_t *F2) {
  if (!a.ctrl->spilled) return;
  const int64_t h = a.ctrl->small_levels;
  uint64_t *const F[3] = {F0, F1, F2};
  uint64_t *src = F[h & 1], *dst = F[h % 3];
  if (src != dst)
    for (int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x; w < a.nw;
         w += (int64_t)gridDim.x * kBlock) {
      dst[w] = src[w];
      src[w] = 0ull;
    }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int sl = (int)(h & 1);
    int nq = 0, nr = 0, sd = 0, far = INT_MAX;
    for (int s = 0; s < kCoopSegs; ++s) {
      nq += a.coop->cnt[sl][s];
      nr += a.coop->near[sl][s];
      sd += a.coop->esum[sl][s];
      far = min(far, a.coop->far[sl][s]);
    }
    for (int i = 0; i < 3 * kDeltaSlots; ++i)
      a.ctrl->lists[i] = (i % kDeltaFields) == 3 ? INT_MAX : 0;
    int32_t *cnt = a.ctrl->lists + (h % 3) * kDeltaSlots;
    cnt[0] = nr;
    cnt[1] = sd;
    cnt[2] = 0;  // rows are at most kCoopMaxDeg long
    cnt[3] = far;
    cnt[4] = nq;
  }
}

}  // namespace

void launch_sssp_delta_own(const SsspArgs &a, int32_t source, int64_t max_rounds,
                           uint64_t *const F[3], uint64_t wait_ticks, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const int cap = (int)std::min<int64_t>(max_rounds, kOwnMaxLevels + 1);
  hipLaunchKernelGGL(k_sssp_delta_own, dim3(a.own.groups), dim3(kOwnThreads), 0, s, a, source, cap,
                     wait_ticks, F[1]);
  hipLaunchKernelGGL(k_sssp_delta_own_boxes, dim3(256), dim3(kBlock), 0, s, a, F[1]);
  int64_t gh = (a.nw + kBlock - 1) / kBlock;
  gh = gh < 1 ? 1 : (gh > kExpandGrid ? kExpandGrid : gh);
  hipLaunchKernelGGL(k_sssp_delta_own_handover, dim3((unsigned)gh), dim3(kBlock), 0, s, a, F[0],
                     F[1], F[2]);
}

void launch_sssp_delta_coop(const SsspArgs &a, int64_t max_rounds, uint64_t *const F[3],
                            uint64_t wait_ticks, void *stream) {
  hipLaunchKernelGGL(k_sssp_delta_coop, dim3(kCoopGrid), dim3(kCoopThreads), 0,
                     (hipStream_t)stream, a, max_rounds, wait_ticks, F[0], F[1]);
  int64_t g = (a.nw + kBlock - 1) / kBlock;
  g = g < 1 ? 1 : (g > 4096 ? 4096 : g);
  hipLaunchKernelGGL(k_sssp_delta_coop_handover, dim3((unsigned)g), dim3(kBlock), 0,
                     (hipStream_t)stream, a, F[0], F[1], F[2]);
}

void launch_sssp_delta_start(const SsspArgs &a, int32_t source, uint64_t *f1, uint64_t *f2,
                             void *stream) {
  int64_t g = (a.nw + kWavesPerBlock - 1) / kWavesPerBlock;
  g = g < 1 ? 1 : (g > 4096 ? 4096 : g);
  hipLaunchKernelGGL(k_sssp_delta_start, dim3((unsigned)g), dim3(kBlock), 0, (hipStream_t)stream,
                     a, source, f1, f2);
}

void launch_sssp_delta_round(const SsspArgs &a, void *stream) {
  hipLaunchKernelGGL(k_sssp_delta_round, dim3(kExpandGrid), dim3(kBlock), 0, (hipStream_t)stream,
                     a);
}

}  // namespace grb
