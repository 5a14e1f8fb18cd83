// Routing of a small batch by one workgroup, with the router front-end in
// front where the forward starts from logits: used by the plan launch, whose
// workgroups then need no launch before them, and by the routing call.
// (Routing and plan as two launches: 9.6 + 16.7 us for one token of the
// Qwen1.5-shaped block from logits, 21.5 in one.)
#pragma once
#include "mxmoe_internal.h"

namespace mxmoe {
namespace {

// Token t by a group of 8 lanes (E <= 64, k <= 8): lane j of the group holds
// experts j, j + 8, ..., j + 56.  Each lane keeps its best k entries sorted;
// three butterfly steps (partner lane^1, ^2, ^4) merge two sorted lists into
// the best k of their union (a bitonic merge), so that every lane ends with
// the token's k best, sorted.  The maximum and the sum of exp(v - max) take
// the same butterfly, after the lane's own 8 values in expert order.  The
// best k under the strict order are unique, so the ids equal those of the
// wavefront form; the weights differ from it only in the order of the sum.
// the strict order without short-circuit evaluation, so that the compare-
// exchanges below compile to selects rather than branches
__device__ inline bool router_better_sel(float va, int ea, float vb, int eb) {
  return (va > vb) | ((va == vb) & (ea < eb));
}
__device__ inline void router_cmpx(float& va, int& ea, float& vb, int& eb) {  // (a, b) -> (better, worse)
  const bool sw = router_better_sel(vb, eb, va, ea);
  const float xa = sw ? vb : va, xb = sw ? va : vb;
  const int ya = sw ? eb : ea, yb = sw ? ea : eb;
  va = xa;
  vb = xb;
  ea = ya;
  eb = yb;
}

// The ids also go to lds_ids [T, k] (if given); write: ids, weights and gates to
// global memory.
__device__ inline void router_token_group(const RouterArgs& ra, int t, bool live, int E, int j, int32_t* lds_ids,
                                          bool write) {
  constexpr int K = kGroupMaxK;
  const float* row = ra.logits + (int64_t)(live ? t : 0) * E;
  float v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = (live && j + 8 * i < E) ? row[j + 8 * i] : -INFINITY;
  const float shl = (live && ra.shared_logits && j < ra.n_sh) ? ra.shared_logits[(int64_t)t * ra.n_sh + j] : 0.f;
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < 8; ++i) m = fmaxf(m, v[i]);
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
  float se = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (j + 8 * i < E) se += expf(v[i] - m);
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) se += __shfl_xor(se, d, 64);
  // the lane's own list: its 8 entries sorted by a bitonic network, past-E
  // entries and NaNs replaced by the sentinel (-inf, max int), which every
  // real entry beats (a NaN is never chosen)
  float tv[K];
  int te[K];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    const bool ok = (j + 8 * i < E) & (v[i] == v[i]);
    tv[i] = ok ? v[i] : -INFINITY;
    te[i] = ok ? j + 8 * i : 0x7fffffff;
  }
#pragma unroll
  for (int kk = 2; kk <= K; kk <<= 1)
#pragma unroll
    for (int jj = kk >> 1; jj > 0; jj >>= 1)
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const int l = i ^ jj;
        if (l > i) {
          if ((i & kk) == 0)
            router_cmpx(tv[i], te[i], tv[l], te[l]);  // better first
          else
            router_cmpx(tv[l], te[l], tv[i], te[i]);
        }
      }
  // butterfly merges
#pragma unroll
  for (int d = 1; d < 8; d <<= 1) {
    float ov[K];
    int oe[K];
#pragma unroll
    for (int r = 0; r < K; ++r) {
      ov[r] = __shfl_xor(tv[r], d, 64);
      oe[r] = __shfl_xor(te[r], d, 64);
    }
    // the better of tv[r] and ov[K-1-r]: the best K of the union, bitonic
#pragma unroll
    for (int r = 0; r < K; ++r) {
      const bool b = router_better_sel(ov[K - 1 - r], oe[K - 1 - r], tv[r], te[r]);
      tv[r] = b ? ov[K - 1 - r] : tv[r];
      te[r] = b ? oe[K - 1 - r] : te[r];
    }
    // sort the bitonic sequence: half-cleaners of span 4, 2, 1
#pragma unroll
    for (int h = K / 2; h > 0; h >>= 1)
#pragma unroll
      for (int r = 0; r < K; ++r)
        if ((r & h) == 0) router_cmpx(tv[r], te[r], tv[r + h], te[r + h]);
  }
  if (!live) return;
  const int k = ra.k;
  float q = 0.f, den = 0.f;
  int my_e = -1;
#pragma unroll
  for (int r = 0; r < K; ++r) {
    const float qr = (r < k && te[r] != 0x7fffffff) ? expf(tv[r] - m) : 0.f;
    if (r < k) den += qr;
    if (r == j) {
      q = qr;
      my_e = te[r] == 0x7fffffff ? -1 : te[r];
    }
  }
  if (!ra.renorm) den = se;
  if (lds_ids && j < k) lds_ids[t * k + j] = my_e;
  if (!write) return;
  if (j < k) {
    ra.ids[(int64_t)t * k + j] = my_e;
    ra.w[(int64_t)t * k + j] = q / den;
  }
  if (ra.shared_logits)
    for (int s2 = j; s2 < ra.n_sh; s2 += 8)
      ra.shared_w[(int64_t)t * ra.n_sh + s2] =
          1.f / (1.f + expf(-(s2 == j ? shl : ra.shared_logits[(int64_t)t * ra.n_sh + s2])));
}

// Batches of at most kRouteSmall pairs, by a workgroup of 1024 threads: a
// histogram (integer LDS atomics: the counts do not depend on their order), an
// exclusive scan, then the pairs are ranked 1024 at a time, a wavefront by one
// ballot per id bit; positions follow from the expert's base, the counts of
// earlier wavefronts of the step and the rank in the wavefront, so the order
// (expert, then pair id) is the one the chunked launches give.  A thread's
// pairs (up to four) and their gate weights are read once, before the steps:
// read inside them, each step is two memory round trips longer (12.4 us in all
// for 3000 pairs).
constexpr int kSmallThreads = 1024;
constexpr int kSmallPairs = kRouteSmall / kSmallThreads;
template <int EM> struct RouteLds {
  int32_t base[EM];
  int32_t wcnt[kSmallThreads / 64][EM];
  int32_t ids[kRouteSmall];  // the router's choice
  int32_t wsum[kSmallThreads / 64];
  int32_t bad;
};
// Leaves the expert's row count and first sorted row of thread tid < E in
// *count and *first; write: whether the results go to global memory (a second
// workgroup that only needs the counts passes false).  Ends with a barrier.
template <int EM>
__device__ __attribute__((always_inline)) inline void route_block(RouteLds<EM>& L, const RouteJob& J, bool write,
                                                                  int* count, int* first) {
  constexpr int NW = kSmallThreads / 64;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int P = J.P, E = J.E;
  for (int e = tid; e < E; e += kSmallThreads) L.base[e] = 0;
  if (tid == 0) L.bad = 0x7fffffff;
  int ev[kSmallPairs];
  float gw[kSmallPairs];
  if (J.ra.logits) {
    const int T = P / J.ra.k;
    for (int t0 = 0; t0 < T; t0 += kSmallThreads / 8) {  // uniform trip count: every lane shuffles
      const int t = t0 + (tid >> 3);
      router_token_group(J.ra, t, t < T, E, tid & 7, L.ids, write);
    }
    __syncthreads();  // (the weights written above are read back by this workgroup)
#pragma unroll
    for (int i = 0; i < kSmallPairs; ++i) {
      const int p = tid + i * kSmallThreads;
      ev[i] = p < P ? L.ids[p] : -1;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kSmallPairs; ++i) {
      const int p = tid + i * kSmallThreads;
      ev[i] = p < P ? J.ids[p] : -1;
    }
  }
  if (write && J.rm.rtok) {
#pragma unroll
    for (int i = 0; i < kSmallPairs; ++i) {
      const int p = tid + i * kSmallThreads;
      gw[i] = p < P ? J.rm.topk_w[p] : 0.f;
    }
  }
  __syncthreads();
  // 1. histogram
#pragma unroll
  for (int i = 0; i < kSmallPairs; ++i) {
    const int p = tid + i * kSmallThreads;
    if (p < P) {
      if (ev[i] >= 0 && ev[i] < E) atomicAdd(&L.base[ev[i]], 1);
      else {
        atomicMin(&L.bad, p);
        ev[i] = -1;
      }
    }
  }
  __syncthreads();
  // 2. exclusive scan of the counts (E <= 1024: one expert per thread)
  const int mine = tid < E ? L.base[tid] : 0;
  int incl = mine;
  for (int d = 1; d < 64; d <<= 1) {
    const int v = __shfl_up(incl, d, 64);
    if (lane >= d) incl += v;
  }
  if (lane == 63) L.wsum[w] = incl;
  __syncthreads();
  int excl = incl - mine;
  for (int i = 0; i < w; ++i) excl += L.wsum[i];
  *count = mine;
  *first = excl;
  if (!write) return;
  if (tid < E) {
    J.counts[tid] = mine;
    J.offsets[tid] = excl;
    L.base[tid] = excl;  // only this thread read base[tid]
  }
  if (tid == E - 1) J.offsets[E] = excl + mine;
  if (tid == 0) J.status[0] = L.bad == 0x7fffffff ? 0 : L.bad + 1;
  // 3. scatter, 1024 pairs per step
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
  for (int st = 0; st < kSmallPairs; ++st) {
    const int s = st * kSmallThreads;
    if (s >= P) break;
    for (int e = tid; e < E; e += kSmallThreads)
#pragma unroll
      for (int i = 0; i < NW; ++i) L.wcnt[i][e] = 0;
    __syncthreads();
    const int p = s + tid, e = ev[st];  // (-1 past P)
    uint64_t same = __ballot(e >= 0);
    for (int b = 0; b < J.ebits; ++b) {
      const bool bit = e >= 0 && ((e >> b) & 1);
      const uint64_t m = __ballot(bit);
      same &= bit ? m : ~m;
    }
    if (e < 0) same = 0;
    const int rank = __popcll(same & below);
    if (e >= 0 && rank == 0) L.wcnt[w][e] = __popcll(same);
    __syncthreads();
    if (e >= 0) {
      int pos = L.base[e] + rank;
      for (int i = 0; i < w; ++i) pos += L.wcnt[i][e];
      J.sorted_pair[pos] = p;
      J.inv[p] = pos;
      if (J.rm.rtok) {
        const int t = p / J.rm.k, sl = p - t * J.rm.k;
        J.rm.rtok[pos] = t;
        J.rm.rslot[pos] = t * (J.rm.k + J.rm.n_sh) + sl;
        J.rm.rgw[pos] = gw[st];
      }
    } else if (p < P) {
      J.inv[p] = -1;
    }
    __syncthreads();
    for (int ee = tid; ee < E; ee += kSmallThreads) {
      int add = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) add += L.wcnt[i][ee];
      L.base[ee] += add;
    }
    // (no barrier here: thread t alone updates base[t], t + 1024, ... and
    // clears the same columns of wcnt at the next step, whose first barrier
    // orders both before any other thread reads them)
  }
}

}  // namespace
}  // namespace mxmoe
