// k_build.hip -- CAGRA graph construction (Section 2.2 on CAGRA; Section
// 4.2, CAGRA graph construction): an approximate k-NN graph by NN-Descent,
// rank-based edge pruning to the fixed degree, then reverse edges merged in.
//
// Positions 0..n-1 stand for the points being built (pool row ids[p]).
// Every kernel runs one wavefront per node and reads only state that the
// previous kernel finished, so the result does not depend on scheduling:
//
// NN-Descent round (batch-synchronous): sample the first S new and the first
// S old entries of every list (sampled new entries turn old) and record each
// sample at its target; group the records by target; per node v gather
// Bn = its new samples and the S smallest (Dist, u) new reverse samples,
// Bo = the same for old minus Bn; the pairs within Bn and between Bn and Bo
// give proposals (b to a when (Dist, b) is below a's last key at the start
// of the round, and the other way); a range of nodes writes its proposals to
// the record buffers, where they are grouped by target and merged into a copy
// of the lists (the K smallest distinct keys; an existing key keeps its entry
// and flag), then the next range.
//
// Rank-based pruning: per node u, for every neighbour y of rank r, count the
// z of rank rz < r whose list holds y at a rank below r (detourable routes);
// keep the R entries with the fewest routes, by (routes, rank).
// Reverse edges: every pruned edge u -> y at position t is recorded at y
// with key (t, u); y's output is the first R/2 of its pruned list, then its
// reverse neighbours in key order, then the rest of its pruned list,
// skipping ids already taken, up to R.
//
// Distances are exact (uint8) or fp64 sums in dimension order, rounded once
// (fp32): a pair has one distance wherever it is evaluated, as the merges tell
// entries apart by (Dist, position).  Sums in another order are taken again
// where the order could move the rounding (rounds_once).
#include "dispatch.h"

namespace gr {

constexpr uint32_t kNew = 0x80000000u;  // list entry not yet sampled; reverse records: an old sample

__device__ __forceinline__ const uint8_t *row_of(const BuildArgs &a, uint32_t pos) {
  return a.pool.vecs + (size_t)a.ids[pos] * a.pool.stride;
}

static __device__ void build_error(DevScalars *ds, uint32_t id) {
  if (atomicCAS(&ds->err_code, 0u, (uint32_t)kErrInit) == 0u) ds->err_id = id;
}

// Initial lists: K distinct positions other than u, each below n.
__global__ __launch_bounds__(64) void k_nnd_check(BuildArgs a) {
  const uint32_t u = blockIdx.x;
  if (u >= a.n) return;
  const int ln = lane();
  float d[2];
  uint32_t v[2];
  bool bad = false;
#pragma unroll
  for (int r = 0; r < 2; r++) {
    const uint32_t j = r * 64 + ln;
    const uint32_t x = j < a.K ? a.init[(size_t)u * a.K + j] : kInvalid;
    bad |= j < a.K && (x >= a.n || x == u);
    d[r] = j < a.K ? 0.0f : finf();
    v[r] = j < a.K ? x : kInvalid;
  }
  wave_sort<2>(d, v);
  uint64_t dm[2];
  if (ballot(bad) || wave_find_repeats<2>(d, v, dm)) {
    if (ln == 0) build_error(a.ds, u);
  }
}

// Lists from the initial positions, ascending by (Dist, position), all new.
// The rows are gathered by row_dists (one lane a row, 16 bytes at a time, took
// 4.2 ms for 100,000 x 128 rows of 400 bytes; this takes 0.86).
template <int KIND>
__global__ __launch_bounds__(64) void k_nnd_init(BuildArgs a) {
  const uint32_t u = blockIdx.x;
  if (u >= a.n) return;
  __shared__ uint32_t vL[128];
  __shared__ float dL[128];
  const int ln = lane(), K = (int)a.K;
  const uint8_t *ru = row_of(a, u);
  for (int j = ln; j < 128; j += 64) vL[j] = j < K ? a.init[(size_t)u * K + j] : u;
  __syncthreads();
  row_dists<KIND>(ru, a.pool.nch, vL, dL, K, [&](uint32_t x) { return row_of(a, x); });
  __syncthreads();
  float d[2];
  uint32_t v[2];
#pragma unroll
  for (int r = 0; r < 2; r++) {
    const int j = r * 64 + ln;
    v[r] = j < K ? vL[j] : kInvalid;
    d[r] = j < K ? dL[j] : finf();
  }
  wave_sort<2>(d, v);
#pragma unroll
  for (int r = 0; r < 2; r++) {
    const int j = r * 64 + ln;
    if (j < K) {
      a.lid[(size_t)u * K + j] = v[r] | kNew;
      a.ld[(size_t)u * K + j] = d[r];
    }
  }
}

// Samples of node u: the first S new entries (which turn old) and the first
// S old ones, in list order; each sample is also recorded at its target
// (old samples with the source's top bit set).
__global__ __launch_bounds__(64) void k_nnd_sample(BuildArgs a) {
  const uint32_t u = blockIdx.x;
  if (u >= a.n) return;
  const int ln = lane();
  const uint32_t S = a.S;
  uint32_t before_new = 0, before_old = 0;
#pragma unroll
  for (int r = 0; r < 2; r++) {
    const uint32_t j = r * 64 + ln;
    const bool in = j < a.K;
    const uint32_t e = in ? a.lid[(size_t)u * a.K + j] : 0u;
    const float dd = in ? a.ld[(size_t)u * a.K + j] : 0.0f;
    const bool isnew = in && (e & kNew);
    const bool isold = in && !(e & kNew);
    const uint64_t mn = ballot(isnew), mo = ballot(isold);
    const uint32_t kn = before_new + (uint32_t)mbcnt(mn), ko = before_old + (uint32_t)mbcnt(mo);
    const uint32_t v = e & kIdMask;
    if (isnew && kn < S) {
      a.ns[(size_t)u * S + kn] = v;
      const size_t q = (size_t)u * 2 * S + kn;
      a.rec_t[q] = v;
      a.rec_s[q] = u;
      a.rec_d[q] = dd;
      a.lid[(size_t)u * a.K + j] = v;
    }
    if (isold && ko < S) {
      a.os[(size_t)u * S + ko] = v;
      const size_t q = (size_t)u * 2 * S + S + ko;
      a.rec_t[q] = v;
      a.rec_s[q] = u | kNew;
      a.rec_d[q] = dd;
    }
    before_new += (uint32_t)popc(mn);
    before_old += (uint32_t)popc(mo);
  }
  for (uint32_t k = ln; k < S; k += 64) {
    if (k >= before_new) {
      a.ns[(size_t)u * S + k] = kInvalid;
      a.rec_t[(size_t)u * 2 * S + k] = kInvalid;
    }
    if (k >= before_old) {
      a.os[(size_t)u * S + k] = kInvalid;
      a.rec_t[(size_t)u * 2 * S + S + k] = kInvalid;
    }
  }
}

// Bn and Bo of node v (Bn ascending, then Bo ascending) into cand[v][0..4S),
// their sizes into cnb[v] = nb | no << 16.
__global__ __launch_bounds__(64) void k_nnd_cands(BuildArgs a) {
  const uint32_t v = blockIdx.x;
  if (v >= a.n) return;
  __shared__ uint32_t bnL[64];
  const int ln = lane();
  const uint32_t S = a.S;
  // the S smallest (Dist, u) reverse samples of each kind
  float rnd[1] = {finf()}, rod[1] = {finf()};
  uint32_t rni[1] = {kInvalid}, roi[1] = {kInvalid};
  const uint32_t g0 = a.goff[v], g1 = a.goff[v + 1];
  for (uint32_t b = g0; b < g1; b += 64) {
    const bool in = b + ln < g1;
    const uint32_t s = in ? a.gsrc[b + ln] : kInvalid;
    const float dd = in ? a.gd[b + ln] : finf();
    const bool old = in && (s & kNew);
    wave_merge_new<1>(rnd, rni, in && !old ? dd : finf(), in && !old ? s : kInvalid, (int)S);
    wave_merge_new<1>(rod, roi, old ? dd : finf(), old ? (s & kIdMask) : kInvalid, (int)S);
  }
  // Bn: the new samples and the new reverse samples, ascending, distinct
  {
    uint32_t x = kInvalid;
    const uint32_t rv = (uint32_t)__shfl((int)rni[0], (ln - (int)S) & 63, 64);
    if (ln < (int)S) x = a.ns[(size_t)v * S + ln];
    else if (ln < 2 * (int)S) x = rv;
    float kd = kvalid(x) ? 0.0f : finf();
    wave_sort_unique1(kd, x);
    bnL[ln] = x;
  }
  __syncthreads();
  const uint32_t bn = bnL[ln];
  const int nb = popc(ballot(kvalid(bn)));
  // Bo: the old samples and old reverse samples not in Bn
  uint32_t y = kInvalid;
  const uint32_t ro = (uint32_t)__shfl((int)roi[0], (ln - (int)S) & 63, 64);
  if (ln < (int)S) y = a.os[(size_t)v * S + ln];
  else if (ln < 2 * (int)S) y = ro;
  {
    float kd = kvalid(y) ? 0.0f : finf();
    wave_sort_unique1(kd, y);
  }
  bool keep = kvalid(y);
  if (keep) {
    int lo = 0, hi = nb;  // binary search in the ascending Bn
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (bnL[mid] < y) lo = mid + 1;
      else hi = mid;
    }
    keep = !(lo < nb && bnL[lo] == y);
  }
  const uint64_t km = ballot(keep);
  const int no = popc(km);
  uint32_t *c = a.cand + (size_t)v * 4 * S;
  if (ln < nb) c[ln] = bn;
  if (keep) c[nb + mbcnt(km)] = y;
  if (ln == 0) a.cnb[v] = (uint32_t)nb | ((uint32_t)no << 16);
}

// One K step of the joins' 16-row tiles: lane (g, col) holds its part of row
// col as either operand.  fp32: 4 of 16 dimensions, widened to fp64 (squared
// L2: seen from the node's row, so that |x|^2 + |y|^2 - 2 x.y stays close to
// the distances), four fp64 products of 4 dimensions; uint8: 16 of 64 bytes.
template <int KIND> struct Join {
  typedef double v4d __attribute__((ext_vector_type(4)));
  typedef v4d Acc;
  typedef double Sq;
  struct Op { double x[4]; };
  static __device__ __forceinline__ int steps(int nch) { return (nch + 3) >> 2; }
  static __device__ __forceinline__ uint4 load(const uint8_t *row, int k, int g, int nch) {
    const int c = 4 * k + g;
    return ld16(row + (size_t)(c < nch ? c : 0) * 16);
  }
  static __device__ __forceinline__ Op op(uint4 v, uint4 u, int k, int g, int nch) {
    const bool in = 4 * k + g < nch;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w}, c[4] = {u.x, u.y, u.z, u.w};
    Op o;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const double x = (double)__uint_as_float(w[i]) - (KIND == kF32L2 ? (double)__uint_as_float(c[i]) : 0.0);
      o.x[i] = in ? x : 0.0;
    }
    return o;
  }
  static __device__ __forceinline__ Sq square(const Op &o, Sq s) {
#pragma unroll
    for (int i = 0; i < 4; i++) s = __builtin_fma(o.x[i], o.x[i], s);
    return s;
  }
  static __device__ __forceinline__ Acc mul(const Op &a, const Op &b, Acc c) {
#pragma unroll
    for (int i = 0; i < 4; i++) c = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x[i], b.x[i], c, 0, 0, 0);
    return c;
  }
  // the row of element i of a product in lane group g
  static __device__ __forceinline__ int row(int g, int i) { return g + 4 * i; }
};
template <> struct Join<kU8L2> {
  typedef v4i Acc;
  typedef int Sq;
  typedef v4i Op;
  static __device__ __forceinline__ int steps(int nch) { return (nch + 3) >> 2; }
  static __device__ __forceinline__ uint4 load(const uint8_t *row, int k, int g, int nch) {
    const int c = 4 * k + g;
    return ld16(row + (size_t)(c < nch ? c : 0) * 16);
  }
  // chunks past the row are the same in every row, so they add nothing
  static __device__ __forceinline__ Op op(uint4 v, uint4, int k, int g, int nch) {
    return to_i8x16(4 * k + g < nch ? v : make_uint4(0, 0, 0, 0));
  }
  static __device__ __forceinline__ Sq square(const Op &o, Sq s) { return sq_i8x16(o, s); }
  static __device__ __forceinline__ Acc mul(const Op &a, const Op &b, Acc c) { return mfma_i8(a, b, c); }
  static __device__ __forceinline__ int row(int g, int i) { return 4 * g + i; }
};
__device__ __forceinline__ int join_sum(int v) {
  v += (int)xshfl((uint32_t)v, 16);
  return v + (int)xshfl((uint32_t)v, 32);
}
__device__ __forceinline__ double join_sum(double v) {
#pragma unroll
  for (int o = 16; o < 64; o <<= 1) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    v += __longlong_as_double((long long)xshfl64(b, o));
  }
  return v;
}

// Joins at the nodes v0 .. v1: the pairs (i, j), i < nb and i < j < nb + no,
// of a node's candidates, 16 rows i (one block) against all later tiles at a
// time, up to 16 * NT candidates.  A block's proposals take a range of the
// record buffers from the cursor ds->n_prop; a block that finds no room writes
// nothing (what it took below the capacity is filled with empty records) and
// sets its bit of pcnt[v]: the host launches the range again with `retry` for
// those blocks.  Records come in any order: the merge orders by key.
//
// Every distance is evaluated once, on the matrix cores: one pair per lane
// from rows in LDS, counted in one pass and written in a second, took 10 ms a
// round (100,000 x 100 fp32, S = 16; 6 waves per CU for the LDS, three fp64
// instructions per dimension of a pair).  With every row converted once per
// tile product it takes 2.2 ms a round, at two to three waves per SIMD (176
// registers).  Its 63M records would be written in 0.2 ms at the rate of a large
// copy; the cursor weighs more: a second returning atomic of every block on its
// address took 7 ms a round.
template <int KIND, int NT>
__global__ __launch_bounds__(64, NT == 4 ? 3 : 1) void k_nnd_join(BuildArgs a) {
  typedef Join<KIND> J;
  __shared__ uint32_t cL[16 * NT];
  __shared__ float wdL[16 * NT];
  __shared__ uint32_t wiL[16 * NT];
  __shared__ typename J::Sq rsL[16];
  const uint32_t v = a.v0 + blockIdx.x;
  if (v >= a.v1) return;
  const uint32_t todo = a.retry ? a.pcnt[v] : ~0u;
  if (!todo) return;
  const int ln = lane(), g = ln >> 4, col = ln & 15;
  const uint32_t S = a.S, K = a.K;
  const uint32_t cc = a.cnb[v];
  const int nb = (int)(cc & 0xFFFFu), no = (int)(cc >> 16), m = nb + no;
  const uint32_t *c = a.cand + (size_t)v * 4 * S;
  // candidates and their last keys at the start of the round
  for (int i = ln; i < 16 * NT; i += 64) {
    const uint32_t x = i < m ? c[i] : v;
    cL[i] = x;
    wdL[i] = a.ld[(size_t)x * K + K - 1];
    wiL[i] = a.lid[(size_t)x * K + K - 1] & kIdMask;
  }
  __syncthreads();
  const int nch = a.pool.nch, ks = J::steps(nch), nt = (m + 15) >> 4;
  const uint8_t *rv = row_of(a, v);
  uint32_t left = 0;
  for (int ta = 0; 16 * ta < nb; ta++) {
    if (!((todo >> ta) & 1u)) continue;
    // tile t of the block: candidates 16 (ta + t) .. (rows past the last one
    // hold the node's own); tile 0 is also the row operand
    typename J::Acc acc[NT];
    typename J::Sq sq[NT];
    const uint8_t *row[NT];
#pragma unroll
    for (int t = 0; t < NT; t++) {
      const int e = 16 * (ta + t) + col;
      row[t] = row_of(a, e < m ? cL[e] : v);
      acc[t] = typename J::Acc{0, 0, 0, 0};
      sq[t] = 0;
    }
#pragma unroll 1
    for (int k = 0; k < ks; k++) {
      uint4 u = make_uint4(0, 0, 0, 0), w[NT];
      if (KIND == kF32L2) u = J::load(rv, k, g, nch);
#pragma unroll
      for (int t = 0; t < NT; t++)
        if (ta + t < nt) w[t] = J::load(row[t], k, g, nch);
      typename J::Op x0 = J::op(w[0], u, k, g, nch);
#pragma unroll
      for (int t = 0; t < NT; t++) {
        if (ta + t >= nt) continue;
        const typename J::Op x = t ? J::op(w[t], u, k, g, nch) : x0;
        sq[t] = J::square(x, sq[t]);
        acc[t] = J::mul(x0, x, acc[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < NT; t++) sq[t] = join_sum(sq[t]);
    __syncthreads();
    if (g == 0) rsL[col] = sq[0];
    __syncthreads();
    // the distances and which way each is proposed: bit 8t + 2i for j to i,
    // the next one for i to j
    float d[NT][4];
    uint64_t prop = 0;
    uint32_t cnt = 0;
#pragma unroll
    for (int t = 0; t < NT; t++) {
      const int j = 16 * (ta + t) + col;
      const uint32_t pb = cL[j < 16 * NT ? j : 0], wib = wiL[j < 16 * NT ? j : 0];
      const float wdb = wdL[j < 16 * NT ? j : 0];
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int r = J::row(g, i), e = 16 * ta + r;
        const uint32_t pa = cL[e];
        const bool in = e < nb && j > e && j < m;
        if constexpr (KIND == kU8L2) {
          d[t][i] = canon0((float)(rsL[r] + sq[t] - 2 * acc[t][i]));
        } else {
          // the magnitudes of a product's terms add up to at most half of
          // |x|^2 + |y|^2
          const double s = rsL[r] + sq[t];
          const double x = KIND == kF32IP ? -acc[t][i] : __builtin_fma(-2.0, acc[t][i], s);
          d[t][i] = canon0((float)x);
          if (in && !rounds_once(x, s * (KIND == kF32IP ? 0x1p-43 : 0x1p-40)))
            d[t][i] = dist_seq<KIND>(row_of(a, pa), row_of(a, pb), nch);
        }
        const bool pab = in && kless(d[t][i], pb, wdL[e], wiL[e]);
        const bool pba = in && kless(d[t][i], pa, wdb, wib);
        prop |= pab ? 1ull << (8 * t + 2 * i) : 0ull;
        prop |= pba ? 2ull << (8 * t + 2 * i) : 0ull;
        cnt += (uint32_t)(popc(ballot(pab)) + popc(ballot(pba)));
      }
    }
    if (!cnt) continue;
    uint32_t base = 0;
    if (ln == 0) base = atomicAdd(&a.ds->n_prop, cnt);
    base = rdlane(base, 0);
    if ((size_t)base + cnt > a.rcap) {
      for (size_t o = (size_t)base + ln; o < a.rcap; o += 64) a.rec_t[o] = kInvalid;
      left |= 1u << ta;
      continue;
    }
#pragma unroll
    for (int t = 0; t < NT; t++) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const bool pab = (prop >> (8 * t + 2 * i)) & 1ull, pba = (prop >> (8 * t + 2 * i)) & 2ull;
        const uint64_t m1 = ballot(pab), m2 = ballot(pba);
        if (!(m1 | m2)) continue;
        const uint32_t pa = cL[16 * ta + J::row(g, i)];
        const int j = 16 * (ta + t) + col;
        const uint32_t pb = cL[j < 16 * NT ? j : 0];
        if (pab) {
          const size_t o = (size_t)base + (uint32_t)mbcnt(m1);
          a.rec_t[o] = pa;
          a.rec_s[o] = pb;
          a.rec_d[o] = d[t][i];
        }
        base += (uint32_t)popc(m1);
        if (pba) {
          const size_t o = (size_t)base + (uint32_t)mbcnt(m2);
          a.rec_t[o] = pb;
          a.rec_s[o] = pa;
          a.rec_d[o] = d[t][i];
        }
        base += (uint32_t)popc(m2);
      }
    }
  }
  if (ln == 0) a.pcnt[v] = left;
}

// Node u's next list <- the K smallest distinct keys of it and its grouped
// proposals (new entries flagged); one wavefront per node with proposals.
//
// A key is (Dist, position) with the entry's flag below it.  Proposals at or
// behind the list's last key are dropped as they are read and the others
// gathered to 64; those are sorted, freed of repeats and of keys that the
// list holds (a binary search in LDS), and merged in.  Against a sort and a
// merge of pair keys for every 64 proposals read: 35 -> 7.3 ms for a
// construction of 100,000 x 100 (4.9 with fewer ranges).
__device__ __forceinline__ uint64_t nnd_key(float d, uint32_t e) {
  return ((uint64_t)sortable(d) << 32) | ((uint64_t)(e & kIdMask) << 1) | (uint64_t)(e >> 31);
}
__global__ __launch_bounds__(64) void k_nnd_merge(BuildArgs a) {
  __shared__ uint64_t cL[128], pend[128];
  const int ln = lane();
  const int K = (int)a.K;
  const uint32_t nd_total = *a.n_dirty;
  for (uint32_t it = blockIdx.x; it < nd_total; it += gridDim.x) {
    const uint32_t u = a.dirty[it];
    uint64_t c[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
      const int j = r * 64 + ln;
      c[r] = j < K ? nnd_key(a.nd[(size_t)u * K + j], a.nid[(size_t)u * K + j]) : ~0ull;
    }
    uint64_t last = 0;
    auto find_last = [&]() {
#pragma unroll
      for (int r = 0; r < 2; r++)
        if (r == (K - 1) >> 6) last = rdlane64(c[r], (K - 1) & 63);
    };
    find_last();
    const uint32_t g1 = a.goff[u + 1];
    uint32_t b = a.goff[u];
    int np = 0;
    bool changed = false;
    for (;;) {
      while (np < 64 && b < g1) {
        const bool in = b + ln < g1;
        const uint32_t j = in ? b + ln : b;
        const uint64_t x = nnd_key(a.gd[j], a.gsrc[j] | kNew);
        const bool pass = in && x < last;
        const uint64_t pm = ballot(pass);
        if (pass) pend[np + mbcnt(pm)] = x;
        np += popc(pm);
        b += 64;
      }
      if (np == 0) break;
      __syncthreads();
      const int take = np < 64 ? np : 64;
      uint64_t x[1] = {ln < take ? pend[ln] : ~0ull};
      np -= take;
      const uint64_t rest = ln < np ? pend[64 + ln] : 0ull;
      __syncthreads();
      if (ln < np) pend[ln] = rest;
#pragma unroll
      for (int r = 0; r < 2; r++) cL[r * 64 + ln] = c[r];
      wave_sort64<1>(x);
      const uint64_t before = ((uint64_t)shfl_up1((uint32_t)(x[0] >> 32)) << 32) | shfl_up1((uint32_t)x[0]);
      __syncthreads();
      int lo = 0;  // list keys below x (fewer than 128 are below a key below the last one)
#pragma unroll
      for (int s = 64; s > 0; s >>= 1) lo += (cL[lo + s - 1] >> 1) < (x[0] >> 1) ? s : 0;
      const bool keep = x[0] < last && !(ln > 0 && x[0] == before) && (cL[lo & 127] >> 1) != (x[0] >> 1);
      const uint64_t km = ballot(keep);
      if (!km) continue;
      __syncthreads();
      if (keep) cL[mbcnt(km)] = x[0];
      __syncthreads();
      // the kept keys descending from lane 63 - 0 meet the list's upper half
      const int e = 63 - ln;
      const uint64_t y = e < popc(km) ? cL[e] : ~0ull;
      c[1] = y < c[1] ? y : c[1];
      wave_merge_up64<2>(c);
#pragma unroll
      for (int r = 0; r < 2; r++)
        if (r * 64 + ln >= K) c[r] = ~0ull;
      find_last();
      changed = true;
      __syncthreads();
    }
    if (changed) {
#pragma unroll
      for (int r = 0; r < 2; r++) {
        const int j = r * 64 + ln;
        if (j < K) {
          a.nd[(size_t)u * K + j] = unsortable((uint32_t)(c[r] >> 32));
          a.nid[(size_t)u * K + j] = ((uint32_t)c[r] >> 1) | ((uint32_t)c[r] << 31);
        }
      }
    }
    __syncthreads();
  }
}

// Rank-based pruning of node u's list to R entries, and the reverse records
// (P(u)[t], u, t).  Every entry of the K lists that u's list names is looked
// up in it: a table of 1024 (position, rank) words, an eighth full, so that a
// wave's 64 lookups end after one or two reads (with 256 slots and the ranks
// beside them 6.7 ms for 100,000 nodes, K = 128; this 4.3).
constexpr int kRankBits = 10, kRankSlots = 1 << kRankBits;
__global__ __launch_bounds__(64) void k_cagra_rank(BuildArgs a) {
  const uint32_t u = blockIdx.x;
  if (u >= a.n) return;
  __shared__ uint64_t tab[kRankSlots];
  __shared__ uint32_t routes[128];
  __shared__ uint32_t lu[128];
  const int ln = lane();
  const uint32_t K = a.K;
  for (int s = ln; s < kRankSlots; s += 64) tab[s] = ~0ull;
  for (int r = ln; r < 128; r += 64) routes[r] = 0;
  __syncthreads();
  for (uint32_t r = ln; r < K; r += 64) {
    const uint32_t y = a.lid[(size_t)u * K + r] & kIdMask;
    lu[r] = y;
    uint32_t s = (y * 2654435761u) >> (32 - kRankBits);
    const unsigned long long e = ((unsigned long long)y << 32) | r;
    while (atomicCAS(reinterpret_cast<unsigned long long *>(&tab[s]), ~0ull, e) != ~0ull) s = (s + 1) & (kRankSlots - 1);
  }
  __syncthreads();
  auto rank_of = [&](uint32_t y) -> uint32_t {
    uint32_t s = (y * 2654435761u) >> (32 - kRankBits);
    for (;;) {
      const uint64_t e = tab[s];
      if ((uint32_t)(e >> 32) == y) return (uint32_t)e;
      if (e == ~0ull) return kInvalid;
      s = (s + 1) & (kRankSlots - 1);
    }
  };
  for (uint32_t rz = 0; rz < K; rz++) {
    const uint32_t z = lu[rz];
#pragma unroll
    for (int r = 0; r < 2; r++) {
      const uint32_t rzy = r * 64 + ln;
      if (rzy < K) {
        const uint32_t y = a.lid[(size_t)z * K + rzy] & kIdMask;
        const uint32_t ry = rank_of(y);
        if (ry != kInvalid && rz < ry && rzy < ry) atomicAdd(&routes[ry], 1u);
      }
    }
  }
  __syncthreads();
  float kd[2];
  uint32_t ki[2];
#pragma unroll
  for (int r = 0; r < 2; r++) {
    const uint32_t j = r * 64 + ln;
    kd[r] = j < K ? (float)routes[j] : finf();
    ki[r] = j < K ? j : kInvalid;
  }
  wave_sort<2>(kd, ki);
  const uint32_t R = a.R;
  if ((uint32_t)ln < R) {
    const uint32_t y = lu[ki[0]];
    a.prn[(size_t)u * R + ln] = y;
    const size_t q = (size_t)u * R + ln;
    a.rec_t[q] = y;
    a.rec_s[q] = u;
    a.rec_d[q] = (float)ln;
  }
}

// Output list of node y: the first R/2 of its pruned list, its reverse
// neighbours by (position, source), the rest of its pruned list, without
// repeats, up to R; written to the pool row of y.
__global__ __launch_bounds__(64) void k_cagra_out(BuildArgs a) {
  const uint32_t y = blockIdx.x;
  if (y >= a.n) return;
  __shared__ uint32_t outL[64];
  const int ln = lane();
  const uint32_t R = a.R, half = R / 2;
  const uint32_t p = (uint32_t)ln < R ? a.prn[(size_t)y * R + ln] : kInvalid;
  const uint32_t ph = (uint32_t)ln < half ? p : kInvalid;  // the first half
  // the R - half smallest (position, source) reverse neighbours outside the first half
  float rd[1] = {finf()};
  uint32_t ri[1] = {kInvalid};
  const uint32_t g0 = a.goff[y], g1 = a.goff[y + 1];
  for (uint32_t b = g0; b < g1; b += 64) {
    const bool in = b + ln < g1;
    uint32_t s = in ? a.gsrc[b + ln] : kInvalid;
    const float d = in ? a.gd[b + ln] : finf();
    bool dup = false;
    for (uint32_t t = 0; t < half; t++) dup |= s == rdlane(ph, (int)t);
    wave_merge_new<1>(rd, ri, in && !dup ? d : finf(), in && !dup ? s : kInvalid, (int)(R - half));
  }
  const uint32_t nr = (uint32_t)popc(ballot(kvalid(ri[0])));
  if ((uint32_t)ln < half) outL[ln] = p;
  if ((uint32_t)ln < nr) outL[half + ln] = ri[0];
  // the rest of the pruned list, skipping the reverse neighbours taken
  bool take = (uint32_t)ln >= half && (uint32_t)ln < R;
  if (take)
    for (uint32_t t = 0; t < nr; t++) take &= p != rdlane(ri[0], (int)t);
  const uint64_t tm = ballot(take);
  const uint32_t filled = half + nr;
  if (take && filled + (uint32_t)mbcnt(tm) < R) outL[filled + mbcnt(tm)] = p;
  __syncthreads();
  const uint32_t total = min(R, filled + (uint32_t)popc(tm));
  const uint32_t id = a.ids[y];
  if ((uint32_t)ln < R) a.pool.adj[(size_t)id * R + ln] = (uint32_t)ln < total ? a.ids[outL[ln]] : kInvalid;
  if (ln == 0) a.pool.deg[id] = total;
}

// ------------------------------------------------------------------ launches
hipError_t launch_build_check(const BuildArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_nnd_check, dim3(a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_build_init(int kind, const BuildArgs &a, hipStream_t s) {
  if (kind == kU8L2) hipLaunchKernelGGL(k_nnd_init<kU8L2>, dim3(a.n), dim3(64), 0, s, a);
  else if (kind == kF32L2) hipLaunchKernelGGL(k_nnd_init<kF32L2>, dim3(a.n), dim3(64), 0, s, a);
  else hipLaunchKernelGGL(k_nnd_init<kF32IP>, dim3(a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_build_sample(const BuildArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_nnd_sample, dim3(a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_build_cands(const BuildArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_nnd_cands, dim3(a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_build_join(int kind, const BuildArgs &a, hipStream_t s) {
  const uint32_t g = a.v1 - a.v0;
  if (g == 0) return hipSuccess;
  // candidates: at most 4 S, new ones (the row operand) at most 2 S
#define GR_JOIN(K_)                                                                              \
  do {                                                                                           \
    if (a.S <= 16) hipLaunchKernelGGL((k_nnd_join<K_, 4>), dim3(g), dim3(64), 0, s, a);            \
    else hipLaunchKernelGGL((k_nnd_join<K_, 8>), dim3(g), dim3(64), 0, s, a);                     \
  } while (0)
  if (kind == kU8L2) GR_JOIN(kU8L2);
  else if (kind == kF32L2) GR_JOIN(kF32L2);
  else GR_JOIN(kF32IP);
#undef GR_JOIN
  return hipGetLastError();
}
hipError_t launch_build_merge(const BuildArgs &a, uint32_t grid, hipStream_t s) {
  hipLaunchKernelGGL(k_nnd_merge, dim3(grid), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_build_rank(const BuildArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_cagra_rank, dim3(a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_build_out(const BuildArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(k_cagra_out, dim3(a.n), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace gr
