// Masked sparse matrix-matrix product in the dot-product form,
// C = (A B^T) .* M, and triangle counting as its reduction to a scalar
// (Sections 6.3.4 (masked SpGEMM) and 7.5: with L the strict lower triangle
// of a symmetric adjacency, the triangle count is the sum of L L^T .* L).
//
// Only the entries the mask holds are computed: C(i, j) for j in M(i, :) is
// the sum over k of A(i, k) * B(j, k), i.e. the intersection of row i of A
// with row j of B (B is given by its rows, the columns of B^T).  The
// paper's kernel gives one warp a row of the mask and binary-searches the
// column of B for each element of A's row.  Here one wave takes a row i of
// the mask (rows dealt out round-robin), copies row i of A into its own LDS
// segment once, and streams the rows j of B named by the mask row as one
// concatenated list, kUnroll x 64 entries per step (the same wave-level
// load-balanced search as the pull kernels); every entry k is looked up in
// the LDS copy by binary search.  A row of A longer than the LDS segment is
// searched in place in global memory.  With the vertices numbered by
// decreasing degree, a row of L holds only neighbours of at least the
// row's degree, at most sqrt(2 nnz) of them, so the searched rows fit the
// segment and the streamed rows are the short rows of high-degree vertices
// that every wave re-reads from the caches.
//
// Triangle counting fuses the reduction into the structure-only product (the
// kernel fusion the paper names as open work): nothing of C is written, each
// wave counts its hits and adds them to one of the counter's stripes.
#include <hip/hip_runtime.h>

#include "grb_device.h"
#include "grb_internal.h"

namespace grb {
namespace {

// first index in col[0, d) holding a value >= k (ascending list)
template <class P>
__device__ __forceinline__ int lower_pos(P col, int d, int32_t k) {
  int lo = 0, len = d;
  while (len > 0) {
    const int half = len >> 1;
    if (col[lo + half] < k) {
      lo += half + 1;
      len -= half + 1;
    } else {
      len = half;
    }
  }
  return lo;
}

// Writes C(i, j) = sum of the products to c[e] for every mask entry e.
template <class V>
__global__ __launch_bounds__(kBlock) void k_mxm_dot(MxmArgs a) {
  __shared__ int32_t s_col[kWavesPerBlock][kMxmLds];
  __shared__ int s_mark[kWavesPerBlock][64];
  const int wid = threadIdx.x >> 6;
  const int ln = threadIdx.x & 63;
  int32_t *lcol = s_col[wid];
  int *mark = s_mark[wid];
  const int64_t gw = (int64_t)blockIdx.x * kWavesPerBlock + wid;
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  const int32_t *mrp = a.M.rp, *mci = a.M.ci;
  const int32_t *arp = a.A.rp, *aci = a.A.ci;
  const int32_t *brp = a.B.rp, *bci = a.B.ci;
  const V *aval = (const V *)a.A.val, *bval = (const V *)a.B.val;
  V *c = (V *)a.c;
  for (int64_t i = gw; i < a.nrows; i += nwaves) {
    const int mb = mrp[i], me = mrp[i + 1];
    if (mb == me) continue;
    const int ab = arp[i];
    const int da = arp[i + 1] - ab;
    if (da == 0) {  // empty row of A: every entry of the row is zero
      for (int e = mb + ln; e < me; e += 64) c[e] = (V)0;
      continue;
    }
    const bool in_lds = da <= kMxmLds;
    if (in_lds) {
      for (int t = ln; t < da; t += 64) lcol[t] = aci[ab + t];
      wave_lds_sync();
    }
    // the mask row's entries, 64 at a time (one per lane)
    for (int e0 = mb; e0 < me; e0 += 64) {
      const int e = e0 + ln;
      const bool has = e < me;
      int cur = 0, end = 0;
      if (has) {
        const int j = mci[e];
        cur = brp[j];
        end = brp[j + 1];
      }
      V acc = (V)0;
      for (bool more = true; more;) {
        int pos[kUnroll], row[kUnroll], se[kUnroll];
        bool st[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          pos[s] = -1;
          row[s] = 0;
          se[s] = 0;
          st[s] = false;
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
          if (ln < total) pos[s] = rcur + (ln - rexcl);
          row[s] = r;
          st[s] = starts;
          se[s] = min(incl, 64);
          if (starts) cur += se[s] - excl;
        }
        int32_t kk[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) kk[s] = pos[s] >= 0 ? bci[pos[s]] : -1;
        int at[kUnroll];
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          at[s] = -1;
          if (kk[s] >= 0) {
            const int p = in_lds ? lower_pos(lcol, da, kk[s]) : lower_pos(aci + ab, da, kk[s]);
            const int32_t got = p < da ? (in_lds ? lcol[p] : aci[ab + p]) : -1;
            if (got == kk[s]) at[s] = p;
          }
        }
#pragma unroll
        for (int s = 0; s < kUnroll; ++s) {
          const V v = at[s] >= 0 ? aval[ab + at[s]] * bval[pos[s]] : (V)0;
          const V y = seg_sum_scan<V>(v, row[s]);
          const V seg = __shfl(y, st[s] ? se[s] - 1 : 0);
          if (st[s]) acc += seg;
        }
      }
      if (has) c[e] = acc;
    }
    if (in_lds) wave_lds_sync();  // the next row overwrites the segment
  }
}

// Structure-only product (PLUS_PAIR: C(i, j) = |A(i, :) and B(j, :)|) and
// the fused triangle count.  Membership in row i of A is a bit test: each
// wave keeps a bitmap of BITS columns in LDS, sets the bits of row i's
// entries below BITS, and keeps the rest of the row (its tail, the entries at
// or above BITS; rows are sorted, so they come last) as a sorted LDS list
// searched by bisection.  Under the degree numbering the columns of a row are
// the ids of higher-degree vertices, which are small numbers, so nearly every
// probe is a bit test.  Rows of B with at least kPairLong entries are cut into
// units of up to 128 entries (a scan per 64 mask entries), streamed a batch
// of units at a time with the next batch's loads in flight; shorter ones go
// through the load-balanced concatenated stream.
//
// What bounds it: the probes' instructions and the column ids' way from the
// caches (RMAT-20 triangle count, 15.7M mask entries, 4.7G probes: 21 GB into
// the L1s, 11 GB of that past the L2s, in 1.64 ms).  So a step of 64 probes
// is seven vector instructions: the wave is its own workgroup, whose LDS
// addresses are constants; units are padded with copies of their last entry
// and the copies taken back in one product, where predicated lanes or a
// branch per step also kept the loads from being in flight together (26
// instructions and 4.8 ms; straight code per step count 10 and 1.95 ms).
// Before, 64 at a time with a ballot, a population count and a test for the
// tail each: 5.20 ms.
//
// Mask rows of at least kPairSplit entries are shared by kPairGroups
// workgroups, each taking the entries j of one residue: the longest row is
// some 260,000 probes, and an L2 sees half of the long rows' B rows (1.73 ->
// 1.64 ms; eight groups 2.0, since each wave repeats the row's set-up).
template <int BITS>
__device__ __forceinline__ bool pair_hit(const uint32_t *bm, const int32_t *tail, int dt,
                                         bool tail_lds, const int32_t *gtail, int32_t k) {
  if (k < BITS) return (bm[k >> 5] >> (k & 31)) & 1u;
  if (dt == 0) return false;
  const int p = tail_lds ? lower_pos(tail, dt, k) : lower_pos(gtail, dt, k);
  return p < dt && (tail_lds ? tail[p] : gtail[p]) == k;
}

// Mask entry j of a split row if group `grp` computes it, else -1
__device__ __forceinline__ int pair_mine(int j, int grp) {
  return j >= 0 && j % kPairGroups == grp ? j : -1;
}

// The long rows of B of 64 mask entries are cut into units of up to 128
// entries; lane u holds unit u's start, length and mask entry (lane).  A batch
// is kPairUnits units (wave-uniform), lane + 64 s of unit q in k[2 q + s]; the
// lanes past a unit's end hold its last entry again, which the count takes
// back: no step is predicated and no branch stands between the loads.
struct PairBatch {
  uint32_t k[2 * kPairUnits];
  int pad[kPairUnits], l[kPairUnits];
};

__device__ __forceinline__ void pair_load(PairBatch &t, int u0, int pv, int nv, int rv,
                                          const int32_t *bci) {
  const uint32_t ln = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < kPairUnits; ++q) {
    const int32_t *base = bci + __builtin_amdgcn_readlane(pv, u0 + q);
    const int n = __builtin_amdgcn_readlane(nv, u0 + q);  // 0: nothing of this unit counts
    t.pad[q] = 128 - n;
    t.l[q] = __builtin_amdgcn_readlane(rv, u0 + q);
    // byte offsets: one instruction per address
    const uint32_t last = 4u * (uint32_t)max(n - 1, 0);
    t.k[2 * q] = *(const uint32_t *)((const char *)base + min(4u * ln, last));
    t.k[2 * q + 1] = *(const uint32_t *)((const char *)base + min(4u * ln + 256u, last));
  }
}

// Counts the batch's entries that the row of A in `bm` and `tail` holds:
// COUNT into the lanes' cnt, less lane 63's extra, else into acc of the lanes
// of their mask entries.
template <bool COUNT, int BITS>
__device__ __forceinline__ void pair_probe(const PairBatch &t, const uint32_t *bm,
                                           const int32_t *tail, int dt, bool tail_lds,
                                           const int32_t *gtail, int &cnt, int &extra, int &acc) {
  const int ln = threadIdx.x & 63;
  uint32_t top = 0, w[2 * kPairUnits];
#pragma unroll
  for (int s = 0; s < 2 * kPairUnits; ++s) top |= t.k[s];
  if (__ballot(top >= (uint32_t)BITS) == 0ull) {
#pragma unroll
    for (int s = 0; s < 2 * kPairUnits; ++s) w[s] = bm[t.k[s] >> 5];
#pragma unroll
    for (int s = 0; s < 2 * kPairUnits; ++s) w[s] = __builtin_amdgcn_ubfe(w[s], t.k[s], 1u);
  } else {
#pragma unroll
    for (int s = 0; s < 2 * kPairUnits; ++s)
      w[s] = pair_hit<BITS>(bm, tail, dt, tail_lds, gtail, (int32_t)t.k[s]) ? 1u : 0u;
  }
#pragma unroll
  for (int q = 0; q < kPairUnits; ++q) {
    if (COUNT) {
      cnt += (int)(w[2 * q] + w[2 * q + 1]);
      extra += __mul24((int)w[2 * q + 1], t.pad[q]);
    } else {
      const uint64_t hi = __ballot(w[2 * q + 1]);
      const int x = __popcll(__ballot(w[2 * q])) + __popcll(hi) - (int)(hi >> 63) * t.pad[q];
      if (ln == t.l[q]) acc += x;
    }
  }
}

template <bool COUNT, int BITS>
__global__ __launch_bounds__(64, BITS > kPairBits ? 4 : 8) void k_mxm_pair(MxmArgs a) {
  // one wave per workgroup: its LDS addresses are constants
  __shared__ uint32_t bm[BITS / 32];
  __shared__ int32_t tail[kPairTail];
  __shared__ int mark[64];
  const int ln = threadIdx.x;
  const int grp = blockIdx.x % kPairGroups;
  const int64_t gw = blockIdx.x / kPairGroups;
  const int64_t nwaves = gridDim.x / kPairGroups;
  const int32_t *mrp = a.M.rp, *mci = a.M.ci;
  const int32_t *arp = a.A.rp, *aci = a.A.ci;
  const int32_t *brp = a.B.rp, *bci = a.B.ci;
  int *c = (int *)a.c;
  for (int t = ln; t < BITS / 32; t += 64) bm[t] = 0u;
  wave_lds_sync();
  unsigned long long hits = 0;  // COUNT: this lane's
  for (int64_t i0 = gw; i0 < a.nrows; i0 += 64 * nwaves) {
    // the bounds of the wave's next 64 rows, one per lane
    const int64_t il = i0 + (int64_t)ln * nwaves;
    int mbl = 0, mel = 0, abl = 0, dal = 0;
    if (il < a.nrows) {
      mbl = mrp[il];
      mel = mrp[il + 1];
      abl = arp[il];
      dal = arp[il + 1] - abl;
    }
    const bool mine = (ln % kPairGroups) == grp;  // rows that are not split
    if (!COUNT) {
      // an empty row of A: every entry of the mask row is zero
      for (uint64_t z = __ballot(mine && mel > mbl && dal == 0); z; z &= z - 1) {
        const int r = __ffsll((unsigned long long)z) - 1;
        const int ze = __builtin_amdgcn_readlane(mel, r);
        for (int e = __builtin_amdgcn_readlane(mbl, r) + ln; e < ze; e += 64) c[e] = 0;
      }
    }
    const bool cut = mel - mbl >= kPairSplit;
    uint64_t rows = __ballot(mel > mbl && dal > 0 && (cut || mine));
    const uint64_t cuts = __ballot(cut);
    // What the rows need first is loaded ahead: the mask entries two rows
    // ahead, the bounds of their rows of B and the row of A one row ahead
    // (r: current, r1, r2: the next two; 64 when there is none)
    auto take = [&]() {
      if (rows == 0ull) return 64;
      const int r = __ffsll((unsigned long long)rows) - 1;
      rows &= rows - 1;
      return r;
    };
    auto mask_at = [&](int r) {
      // lanes are read before any of them is masked off
      const int e = __builtin_amdgcn_readlane(mbl, r) + ln, me = __builtin_amdgcn_readlane(mel, r);
      const int j = e < me ? mci[e] : -1;
      return (cuts >> r) & 1ull ? pair_mine(j, grp) : j;
    };
    auto row_at = [&](int r) {
      const int f = __builtin_amdgcn_readlane(abl, r) + ln, d = __builtin_amdgcn_readlane(dal, r);
      return ln < d ? aci[f] : INT32_MAX;
    };
    int r = take(), r1 = 64;
    if (r == 64) continue;
    int j1 = mask_at(r), cur1 = 0, end1 = 0, ka1 = row_at(r);
    bool has1 = j1 >= 0;
    if (has1) {
      cur1 = brp[j1];
      end1 = brp[j1 + 1];
    }
    r1 = take();
    if (r1 < 64) j1 = mask_at(r1);
    for (; r < 64; r = r1, r1 = rows ? take() : 64) {
      const int mb = __builtin_amdgcn_readlane(mbl, r), me = __builtin_amdgcn_readlane(mel, r);
      const int ab = __builtin_amdgcn_readlane(abl, r), da = __builtin_amdgcn_readlane(dal, r);
      const bool split = (cuts >> r) & 1ull;
      int cur = cur1, end = end1;
      bool has = has1;
      const int ka = ka1;
      if (r1 < 64) {
        has1 = j1 >= 0;
        cur1 = has1 ? brp[j1] : 0;
        end1 = has1 ? brp[j1 + 1] : 0;
        ka1 = row_at(r1);
        if (rows) j1 = mask_at(__ffsll((unsigned long long)rows) - 1);
      }
      // bits of the entries below BITS (a prefix of the sorted row)
      int t0 = 0;
      for (int t = 0; t < da; t += 64) {
        const int32_t k = t == 0 ? ka : (t + ln < da ? aci[ab + t + ln] : INT32_MAX);
        const bool low = k < BITS;
        if (low) atomicOr(&bm[k >> 5], 1u << (k & 31));
        t0 += __popcll(__ballot(low));
      }
      const int dt = da - t0;
      const bool tail_lds = dt <= kPairTail;
      if (tail_lds)
        for (int t = ln; t < dt; t += 64) tail[t] = aci[ab + t0 + t];
      wave_lds_sync();
      const int32_t *gtail = aci + ab + t0;
      for (int e0 = mb; e0 < me; e0 += 64) {
        const int e = e0 + ln;
        if (e0 != mb) {
          cur = end = 0;
          int j = e < me ? mci[e] : -1;
          if (split) j = pair_mine(j, grp);
          has = j >= 0;
          if (has) {
            cur = brp[j];
            end = brp[j + 1];
          }
        }
        int acc = 0;
        // long rows of B, a batch of units at a time, the next one's loads in
        // flight
        const int nu = end - cur >= kPairLong ? (end - cur + 127) >> 7 : 0;
        const int uincl = wave_incl_scan(nu), units = lane_last(uincl);
        for (int b = 0; b < units; b += 64) {
          const int uex = uincl - nu;
          const bool starts = nu > 0 && uincl > b && uex < b + 64;
          const int rv = slot_rows(mark, starts, max(uex - b, 0));
          int pv = __shfl(cur, rv) + (b + ln - __shfl(uex, rv)) * 128;
          int nv = min(__shfl(end, rv) - pv, 128);
          if (b + ln >= units) pv = nv = 0;
          const int nb = min(units - b, 64);
          int cnt = 0, extra = 0;
          PairBatch x, y;
          pair_load(x, 0, pv, nv, rv, bci);
          for (int u0 = 0;;) {
            u0 += kPairUnits;
            if (u0 < nb) pair_load(y, u0, pv, nv, rv, bci);
            pair_probe<COUNT, BITS>(x, bm, tail, dt, tail_lds, gtail, cnt, extra, acc);
            if (u0 >= nb) break;
            u0 += kPairUnits;
            if (u0 < nb) pair_load(x, u0, pv, nv, rv, bci);
            pair_probe<COUNT, BITS>(y, bm, tail, dt, tail_lds, gtail, cnt, extra, acc);
            if (u0 >= nb) break;
          }
          hits += (unsigned long long)(int64_t)(ln == 63 ? cnt - extra : cnt);
        }
        // short rows as one concatenated stream
        if (end - cur >= kPairLong) end = cur;
        for (bool more = __ballot(end > cur) != 0ull; more;) {
          int pos[kUnroll], row[kUnroll], se[kUnroll];
          bool st[kUnroll];
#pragma unroll
          for (int s = 0; s < kUnroll; ++s) {
            pos[s] = -1;
            row[s] = 0;
            se[s] = 0;
            st[s] = false;
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
            const int rr = slot_rows(mark, starts, excl);
            const int rcur = __shfl(cur, rr), rexcl = __shfl(excl, rr);
            if (ln < total) pos[s] = rcur + (ln - rexcl);
            row[s] = rr;
            st[s] = starts;
            se[s] = min(incl, 64);
            if (starts) cur += se[s] - excl;
          }
          int32_t kk[kUnroll];
#pragma unroll
          for (int s = 0; s < kUnroll; ++s) kk[s] = pos[s] >= 0 ? bci[pos[s]] : -1;
#pragma unroll
          for (int s = 0; s < kUnroll; ++s) {
            const bool hit = kk[s] >= 0 && pair_hit<BITS>(bm, tail, dt, tail_lds, gtail, kk[s]);
            if (COUNT) {
              hits += hit ? 1 : 0;
            } else {
              const int y = seg_sum_scan<int>(hit ? 1 : 0, row[s]);
              const int seg = __shfl(y, st[s] ? se[s] - 1 : 0);
              if (st[s]) acc += seg;
            }
          }
        }
        if (!COUNT && has) c[e] = acc;
      }
      // clear the row's bits for the next row
      wave_lds_sync();
      for (int t = ln; t < t0; t += 64) bm[(t < 64 ? ka : aci[ab + t]) >> 5] = 0u;
      wave_lds_sync();
    }
  }
  if (COUNT) {
    hits = (unsigned long long)wave_sum64((int64_t)hits);
    if (ln == 0 && hits) atomicAdd(a.count + blockIdx.x % kCountStripes, hits);
  }
}

}  // namespace

void launch_mxm_dot(const MxmArgs &a, bool count, void *stream) {
  hipStream_t s = (hipStream_t)stream;
  const dim3 g(kExpandGrid), bp(64), b(kBlock);
  // about 20 rows a wave: a row's work varies by four orders of magnitude, and
  // waves that start as others end level it (RMAT-20 triangle count: 8192
  // workgroups 1.92 ms, 16384 1.88, 32768 1.78, 65536 and 131072 1.73)
  const int64_t want = a.nrows / 20 / kPairGroups * kPairGroups;
  const dim3 gp((unsigned)(want < kPairGridMin ? kPairGridMin
                                               : (want > kPairGridMax ? kPairGridMax : want)));
  if (count || (a.vt != GRB_FP32 && a.vt != GRB_FP64)) {
    // The small bitmap lets 32 waves into a CU where the large one lets 16
    // (RMAT-20 triangle count 1.95 and 2.76 ms).  It is also right where most
    // columns lie beyond both; only matrices of up to 65,536 columns fit the
    // large one and may not fit the small one (R-MAT with 65,536 shuffled ids:
    // 1.24 ms with the small one).
    const bool large = a.B.ncols > kPairBits && a.B.ncols <= 2 * kPairBits;
    if (count && large) hipLaunchKernelGGL((k_mxm_pair<true, 2 * kPairBits>), gp, bp, 0, s, a);
    else if (count) hipLaunchKernelGGL((k_mxm_pair<true, kPairBits>), gp, bp, 0, s, a);
    else if (large) hipLaunchKernelGGL((k_mxm_pair<false, 2 * kPairBits>), gp, bp, 0, s, a);
    else hipLaunchKernelGGL((k_mxm_pair<false, kPairBits>), gp, bp, 0, s, a);
  } else if (a.vt == GRB_FP32) {
    hipLaunchKernelGGL((k_mxm_dot<float>), g, b, 0, s, a);
  } else {
    hipLaunchKernelGGL((k_mxm_dot<double>), g, b, 0, s, a);
  }
}

}  // namespace grb
