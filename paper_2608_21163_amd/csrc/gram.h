// gram.h -- GrANDRobustPrune (Alg. 4) on the matrix cores, one wavefront per
// node, for rows of any length.
//
// The prune asks one question per pair: does a selected candidate i kill a
// later candidate j, coef * Dist(i, j) <= D[j]?  All pairs of a panel of
// candidates are multiplied at once, the rows read once, a K step at a time.
//
// uint8 rows: Dist(i, j) = |y_i|^2 + |y_j|^2 - 2 y_i.y_j with y = x - 128,
// exact in int32 (int8 products); rounded to fp32 as every distance is, and
// tested as an integer against kill_threshold(coef, D[j]).
//
// fp32 rows: Dist is the fp64 sum rounded once to fp32.  With y = x - x_p (the
// candidates seen from the node p that is pruned) Dist(i, j) = D[i] + D[j] -
// 2 y_i.y_j, and D is known for every candidate before the prune starts.  The
// products run on the bf16 matrix cores, each value split into two bf16
// pieces (hi + lo, three products), and every test comes with a bound on its
// error; a test that the bound leaves open is repeated exactly.  So the
// decisions, and with them the lists, are those of the fp64 arithmetic.
//
// The error of one approximate distance, relative to D[j] (D[i] <= D[j], as
// candidates come in that order, so sum |y_i||y_j| <= sqrt(D[i] D[j]) <=
// D[j]): splitting leaves 3 * 2^-18 of a product (the two residuals of at
// most 2^-18 and lo*lo), the fp32 accumulation of 3 * d products at most
// 2^-23 per addition, and a few more roundings of D, y and the test itself.
// At d = 96 that is 1.0e-4 of D[j], at d = 960 7.1e-4, so few tests are open
// (about one pruned node in ten has one at d = 96).
//
// Measured, fp32, against one lane per candidate summing fp64 (whose
// arithmetic was the bound): rebuilds of a 10,000-point batch on 1M x 96 6.93
// -> 0.88 ms per launch, forward prunes 0.99 -> 0.22 ms; with 2,000-point
// batches on 100K x 960 4.67 -> 0.35 ms and 3.50 -> 0.40 ms.  What bounds it
// now is the issue of the splits and products and the selection around them,
// at three waves per SIMD (the accumulators take 60 registers; four waves
// spill, and loads issued a step ahead cost a wave: both slower).  uint8,
// against blocks of 16 pivots multiplied as they are reached: forward prunes
// on 1M x 128 0.178 -> 0.105 ms.
#pragma once
#include "dispatch.h"

namespace gr {

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Greedy selection inside one block of 16 sorted positions, resolved in
// parallel: kb (lane col) holds the earlier positions that would kill col,
// vb the live positions.  Each round, an undecided position is rejected if
// a selected one kills it, and selected if no undecided earlier position
// can; the lowest undecided position is always decided, so this ends with
// exactly the set the one-by-one walk selects.
__device__ __forceinline__ uint32_t block_greedy(uint32_t kb, uint32_t vb, int col, int g) {
  uint32_t S = 0, U = vb;
  while (U) {
    const bool und = ((U >> col) & 1u) != 0;
    const bool rej = und && (kb & S) != 0u;
    const bool sel = und && !rej && (kb & U) == 0u;
    const uint32_t sm = (uint32_t)ballot(sel && g == 0) & 0xFFFFu;
    const uint32_t rm = (uint32_t)ballot(rej && g == 0) & 0xFFFFu;
    S |= sm;
    U &= ~(sm | rm);
  }
  return S;
}
// The lowest n set bits of m.
__device__ __forceinline__ uint32_t first_bits(uint32_t m, int n) {
  uint32_t r = 0;
  for (int k = 0; k < n && m; k++) {
    r |= m & (0u - m);
    m &= m - 1u;
  }
  return r;
}

// Values of the four 16-lane groups of a wave combined by OR, in every lane.
__device__ __forceinline__ uint32_t or_groups(uint32_t v) {
  const auto a = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  const uint32_t w = a[0] | a[1];
  const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return b[0] | b[1];
}

// x = hi + lo to about 17 significant bits, both pieces rounded to nearest.
// The empty asm keeps the packed conversion as it is: the compiler would
// convert half of the values a second time to widen them again.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  const v2bf h = {(__bf16)a, (__bf16)b};
  uint32_t w = __builtin_bit_cast(uint32_t, h);
  asm("" : "+v"(w));
  return w;
}
__device__ __forceinline__ void split8(const float (&x)[8], v8bf &hi, v8bf &lo) {
  uint4 h, l;
  uint32_t *hw = &h.x, *lw = &l.x;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const uint32_t w = pack_bf16(x[2 * i], x[2 * i + 1]);
    hw[i] = w;
    lw[i] = pack_bf16(x[2 * i] - __uint_as_float(w << 16), x[2 * i + 1] - __uint_as_float(w & 0xFFFF0000u));
  }
  hi = __builtin_bit_cast(v8bf, h);
  lo = __builtin_bit_cast(v8bf, l);
}
__device__ __forceinline__ v4f mfma_split(v8bf ah, v8bf al, v8bf bh, v8bf bl, v4f c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, c, 0, 0, 0);
}

// The largest integer distance d with coef * d <= D (fp64 product, as in the
// prune test), for an integer-valued D >= 0; every d up to it passes, since
// rounding is monotone.
// inv is 1 / coef (rounded): the quotient estimate is off by at most one,
// and the two exact tests correct it.
__device__ __forceinline__ int kill_threshold(double coef, double inv, float D) {
  if (!(coef > 0.0)) return 0x7FFFFFFF;
  const double dd = (double)D;
  if (!(dd < 2147483647.0)) return 0x7FFFFFFF;
  const double q = floor(dd * inv);
  if (!(q < 2147483646.0)) return 0x7FFFFFFF;
  int t = (int)q;
  t = coef * (double)(t + 1) <= dd ? t + 1 : t;
  t = coef * (double)t <= dd ? t : t - 1;
  return t;
}

// Dist of two pool rows (squared L2), by the whole wave: lane l adds chunks
// l, l + 64, ... in fp64.  The result is that of the sum in dimension order.
__device__ __forceinline__ float pair_l2(const PoolView &P, uint32_t a, uint32_t b) {
  const uint8_t *ra = P.vecs + (size_t)a * P.stride, *rb = P.vecs + (size_t)b * P.stride;
  double s = 0.0;
  for (int c = lane(); c < P.nch; c += 64) s = l2_4(ld16(ra + (size_t)c * 16), ld16(rb + (size_t)c * 16), s);
  s = group_sum<64>(s);
  if (!rounds_once(s, s * 0x1p-42)) {
    s = 0.0;
    for (int c = 0; c < P.nch; c++) s = l2_4(ld16(ra + (size_t)c * 16), ld16(rb + (size_t)c * 16), s);
  }
  return canon0((float)s);
}

// The kill test of a column j by the approximate A = D[i] - 2 y_i.y_j
// (Dist = A + D[j]): killed for sure when A <= lo, not killed for sure when
// A > hi, open in between (and whenever A is not a number).
struct KillRange {
  float flo, fhi;  // lo = D[j] * flo, hi = D[j] * fhi
};
__device__ __forceinline__ KillRange kill_range(double coef, int nfl) {
  const double n32 = (double)((nfl + 31) & ~31);
  const double e = 2.0 * (3.0 * 0x1p-18 + 3.0 * n32 * 0x1p-23) + 0x1p-19;
  const double inv = 1.0 / coef;  // alpha = 0: every test passes
  KillRange k;
  k.flo = (float)(inv * (1.0 - 0x1p-20) - 1.0 - e);
  k.fhi = (float)(inv * (1.0 + 0x1p-20) - 1.0 + e);
  return k;
}
// Distances whose products could leave the range of the pieces (tiny ones:
// flushed or denormal terms; huge ones: infinities) are tested exactly.
constexpr float kTinyDist = 1e-25f, kHugeDist = 1e36f;
__device__ __forceinline__ void test_range(const KillRange &k, float dj, float &lo, float &hi) {
  const bool sure = dj >= kTinyDist && dj <= kHugeDist;
  lo = sure ? dj * k.flo : -finf();
  hi = sure ? dj * k.fhi : finf();
}

constexpr int kPanelTiles = 5;               // candidates of one panel: 80
constexpr int kPanel = 16 * kPanelTiles;
constexpr int kPanelPairs = kPanelTiles * (kPanelTiles + 1) / 2;
__host__ __device__ constexpr int pair_at(int b, int c) { return b * kPanelTiles - b * (b - 1) / 2 + (c - b); }

// One K step of the products of 16-row tiles: lane (g, col) holds its part of
// row col -- 8 floats of a 32-dimension step, as two bf16 pieces of their
// difference to the node's row, or 16 bytes of a 64-byte step -- as either
// operand.  The result holds rows 4g .. 4g+3 of column col.
template <int KIND> struct Gram;
template <> struct Gram<kF32L2> {
  typedef v4f Acc;
  struct Raw { uint4 v[2]; };
  struct Op { v8bf hi, lo; };
  static __device__ __forceinline__ int steps(int nch) { return (nch + 7) >> 3; }
  // chunks past the row (nch 16-byte chunks) come from the start of the
  // node's row instead, in `u` as in every tile: their differences are zero
  static __device__ __forceinline__ Raw load(const uint8_t *row, const uint8_t *urow, int k, int g, int nch) {
    const int c = 8 * k + 2 * g;
    Raw r;
    r.v[0] = ld16(c < nch ? row + (size_t)c * 16 : urow);
    r.v[1] = ld16(c + 1 < nch ? row + (size_t)c * 16 + 16 : urow);
    return r;
  }
  static __device__ __forceinline__ Op op(const Raw &v, const Raw &u) {
    float x[8];
#pragma unroll
    for (int h = 0; h < 2; h++) {
      x[4 * h + 0] = __uint_as_float(v.v[h].x) - __uint_as_float(u.v[h].x);
      x[4 * h + 1] = __uint_as_float(v.v[h].y) - __uint_as_float(u.v[h].y);
      x[4 * h + 2] = __uint_as_float(v.v[h].z) - __uint_as_float(u.v[h].z);
      x[4 * h + 3] = __uint_as_float(v.v[h].w) - __uint_as_float(u.v[h].w);
    }
    Op o;
    split8(x, o.hi, o.lo);
    return o;
  }
  static __device__ __forceinline__ Acc mul(const Op &a, const Op &b, Acc c) {
    return mfma_split(a.hi, a.lo, b.hi, b.lo, c);
  }
};
template <> struct Gram<kU8L2> {  // Vamana pool rows are whole 64-byte steps
  typedef v4i Acc;
  struct Raw { uint4 v; };
  typedef v4i Op;
  static __device__ __forceinline__ int steps(int nch) { return nch >> 2; }
  static __device__ __forceinline__ Raw load(const uint8_t *row, const uint8_t *, int k, int g, int) {
    return Raw{ld16(row + (size_t)k * 64 + (size_t)g * 16)};
  }
  static __device__ __forceinline__ Op op(const Raw &v, const Raw &) { return to_i8x16(v.v); }
  static __device__ __forceinline__ Acc mul(const Op &a, const Op &b, Acc c) { return mfma_i8(a, b, c); }
};
__device__ __forceinline__ int sum_groups(int v) {
  const auto a = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
  const uint32_t w = a[0] + a[1];
  const auto b = __builtin_amdgcn_permlane16_swap(w, w, false, false);
  return (int)(b[0] + b[1]);
}

// What a tile column needs for its tests: fp32 the range of A, uint8 the kill
// threshold and |y|^2 (Dist <= thr).
template <int KIND> struct ColTest;
template <> struct ColTest<kF32L2> { float lo, hi; };
template <> struct ColTest<kU8L2> { int thr, sq; };

// The tests of one tile pair's products as words: lane (g, col) holds rows 4g
// .. 4g+3 (`row`: their D, or |y|^2 of uint8 rows; the first n of them exist)
// against column col; every lane gets its column's word, bit i set when row i
// kills the column and bit 16 + i when that test is open.
template <int KIND>
__device__ __forceinline__ uint32_t test_word(typename Gram<KIND>::Acc acc, const float *row, ColTest<KIND> c, int n) {
  const int g = lane() >> 4;
  uint32_t w = 0;
#pragma unroll
  for (int ii = 0; ii < 4; ii++) {
    if constexpr (KIND == kU8L2) {
      const int d = (int)(float)(__float_as_int(row[ii]) + c.sq - 2 * acc[ii]);
      w |= ii < n && d <= c.thr ? 1u << ii : 0u;
    } else {
      const float a = __builtin_fmaf(-2.0f, acc[ii], ii < n ? row[ii] : 0.0f);
      const bool kill = a <= c.lo, safe = a > c.hi;
      w |= ii < n && kill ? 1u << ii : 0u;
      w |= ii < n && !(kill | safe) ? 0x10000u << ii : 0u;
    }
  }
  return or_groups(w << (4 * g));
}

// Open tests of the columns cols[lane] (LDS; their D in cd) against rows whose
// ids are rows[0..16) (LDS): one bit of `open` per row.  Each is repeated
// exactly; returns the rows that kill.  With `first`, a column's remaining
// tests are dropped once a row kills it.
__device__ __forceinline__ uint32_t resolve_open(const PoolView &P, uint32_t open, const uint32_t *rows,
                                                 const uint32_t *cols, const float *cd, double coef, bool first) {
  const int ln = lane();
  uint32_t kills = 0;
  uint64_t any;
  while ((any = ballot(open != 0u)) != 0) {
    const int l = ffs64(any);
    const int i = __ffs(rdlane(open, l)) - 1;
    const float d = pair_l2(P, rows[i], cols[l]);
    const bool kill = coef * (double)d <= (double)cd[l];
    if (ln == l) {
      kills |= kill ? 1u << i : 0u;
      open = kill && first ? 0u : open & (open - 1u);
    }
  }
  return kills;
}

// GrANDRobustPrune of node p over m candidates sorted by (D, id): ids in spos
// and D in dpos (LDS, at least 64 * NR entries; both are overwritten).  The
// selections go to oid / od (LDS, R entries) in order; returns their number.
//
// Panels of up to 80 candidates are taken in order.  A panel's rows are read
// once, one K step at a time, and all pairs of its 16-candidate tiles are
// multiplied (15 tile products, 60 accumulator registers); the tests become
// one word per tile pair and column (16 kill bits, 16 open bits), from which
// the selection is resolved tile by tile without further distances.  The
// candidates behind the panel are then tested against its selections only,
// and the survivors packed for the next panel.
template <int KIND, int NR>
__device__ int prune_gram(const PoolView &P, uint32_t p, int m, uint32_t R, double coef, uint32_t *spos, float *dpos,
                          uint32_t *oid, float *od, uint32_t &ntile) {
  typedef Gram<KIND> G;
  constexpr bool kU8 = KIND == kU8L2;
  __shared__ uint32_t kw[kPanelPairs * 16];                   // test words by (tile pair, column)
  __shared__ __align__(16) float rowL[kU8 ? kPanel : 4];      // |y|^2 of the row tiles (uint8, int32 bits)
  const int ln = lane(), g = ln >> 4, col = ln & 15;
  const int nch = P.nch, ks = G::steps(nch);
  const double inv = 1.0 / coef;
  const KillRange kr = kU8 ? KillRange{} : kill_range(coef, nch * 4);
  const uint8_t *urow = P.vecs + (size_t)p * P.stride;
  auto row_of = [&](uint32_t id) { return P.vecs + (size_t)id * P.stride; };
  auto col_test = [&](float dj, int sq) {
    ColTest<KIND> c;
    if constexpr (kU8) {
      c.thr = kill_threshold(coef, inv, dj);
      c.sq = sq;
    } else {
      test_range(kr, dj, c.lo, c.hi);
    }
    return c;
  };
  int nsel = 0;
  while (m > 0) {
    const int pm = m < kPanel ? m : kPanel;
    const int nt = (pm + 15) >> 4;
    {
      // tiles past the panel hold the node's own row (no branch among the
      // loads, so all of a step's are in flight together)
      const uint8_t *row[kPanelTiles];
      int sq[kPanelTiles];
#pragma unroll
      for (int t = 0; t < kPanelTiles; t++) {
        const int e = 16 * t + col;
        row[t] = row_of(e < pm ? spos[e] : p);
        sq[t] = 0;
      }
      typename G::Acc acc[kPanelPairs];
#pragma unroll
      for (int i = 0; i < kPanelPairs; i++) acc[i] = typename G::Acc{0, 0, 0, 0};
#pragma unroll 1
      for (int k = 0; k < ks; k++) {
        typename G::Raw u{}, v[kPanelTiles];
        if constexpr (!kU8) u = G::load(urow, urow, k, g, nch);
#pragma unroll
        for (int t = 0; t < kPanelTiles; t++) v[t] = G::load(row[t], urow, k, g, nch);
        typename G::Op x[kPanelTiles];
#pragma unroll
        for (int t = 0; t < kPanelTiles; t++) {
          x[t] = G::op(v[t], u);
          if constexpr (kU8) sq[t] = sq_i8x16(x[t], sq[t]);
        }
#pragma unroll
        for (int c = 0; c < kPanelTiles; c++)
#pragma unroll
          for (int b = 0; b <= c; b++) acc[pair_at(b, c)] = G::mul(x[b], x[c], acc[pair_at(b, c)]);
      }
      ntile += (uint32_t)(nt * (nt + 1) / 2);
      if constexpr (kU8) {
#pragma unroll
        for (int t = 0; t < kPanelTiles; t++) {
          sq[t] = sum_groups(sq[t]);
          if (g == 0) rowL[16 * t + col] = __int_as_float(sq[t]);
        }
        __syncthreads();
      }
#pragma unroll
      for (int c = 0; c < kPanelTiles; c++) {
        const int e = 16 * c + col;
        const ColTest<KIND> ct = col_test(e < pm ? dpos[e] : 0.0f, sq[c]);
#pragma unroll
        for (int b = 0; b <= c; b++) {
          const uint32_t w = test_word<KIND>(acc[pair_at(b, c)], (kU8 ? rowL : dpos) + 16 * b + 4 * g, ct, 4);
          if (g == 0) kw[16 * pair_at(b, c) + col] = w;
        }
      }
    }
    __syncthreads();
    // greedy selection: tile b's selections, then their kills in later tiles
    uint64_t live[2] = {pm >= 64 ? ~0ull : (1ull << pm) - 1ull, pm > 64 ? (1ull << (pm - 64)) - 1ull : 0ull};
    const int first = nsel;
    bool done = false;
    for (int b = 0; b < nt && !done; b++) {
      const uint32_t vb = (uint32_t)(live[b >> 2] >> (16 * (b & 3))) & 0xFFFFu;
      if (!vb) continue;
      uint32_t kb = kw[16 * pair_at(b, b) + col];
      const uint32_t before = vb & ((1u << col) - 1u);
      if constexpr (!kU8) {
        const uint32_t open = ((vb >> col) & 1u) && g == 0 ? (kb >> 16) & before : 0u;
        if (ballot(open != 0u)) kb |= resolve_open(P, open, spos + 16 * b, spos + 16 * b, dpos + 16 * b, coef, false);
      }
      kb &= before;
      uint32_t S = block_greedy(kb, vb, col, g);
      int ns = __popc(S);
      const int room = (int)R - nsel;
      if (ns >= room) {  // selection stops at R
        S = first_bits(S, room);
        ns = room;
        done = true;
      }
      if (g == 0 && ((S >> col) & 1u)) {
        const int pos = nsel + __popc(S & ((1u << col) - 1u));
        oid[pos] = spos[16 * b + col];
        od[pos] = dpos[16 * b + col];
      }
      nsel += ns;
      if (done) break;
      // four later tiles at a time, one per lane group
      for (int c0 = b + 1; c0 < nt; c0 += 4) {
        const int c = c0 + g;
        const bool alive = c < nt && ((live[c >> 2] >> (16 * (c & 3) + col)) & 1ull);
        const uint32_t w = alive ? kw[16 * pair_at(b, c) + col] : 0u;
        bool dead = (w & S) != 0u;
        if constexpr (!kU8) {
          const uint32_t o = dead ? 0u : (w >> 16) & S;
          if (ballot(o != 0u))
            dead |= resolve_open(P, o, spos + 16 * b, spos + 16 * c0, dpos + 16 * c0, coef, true) != 0u;
        }
        const uint64_t dm = ballot(dead);
        const int sh = 16 * (c0 & 3);
        live[c0 >> 2] &= ~(dm << sh);
        if (c0 < 4 && sh) live[1] &= ~(dm >> (64 - sh));
      }
    }
    __syncthreads();
    if (done || m <= kPanel) break;
    // the candidates behind the panel against its selections: 64 candidates
    // (4 tiles, one per lane group in the tests) by 32 selections at a time
    const int ns = nsel - first;
    uint64_t keep[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) keep[r] = ballot(r * 64 + ln >= kPanel && r * 64 + ln < m);
    constexpr int NA = 2, NB = 4;
    for (int e0 = kPanel; e0 < m; e0 += 16 * NB) {
      bool alive = e0 + ln < m;
      for (int a0 = 0; a0 < ns && ballot(alive) != 0; a0 += 16 * NA) {
        // tiles past the selections or candidates hold the node's own row
        const uint8_t *row[NA + NB];
        int sq[NA + NB];
#pragma unroll
        for (int t = 0; t < NA + NB; t++) {
          const int e = t < NA ? a0 + 16 * t + col : e0 + 16 * (t - NA) + col;
          row[t] = row_of(t < NA ? (e < ns ? oid[first + e] : p) : (e < m ? spos[e] : p));
          sq[t] = 0;
        }
        typename G::Acc acc[NA][NB];
#pragma unroll
        for (int a = 0; a < NA; a++)
#pragma unroll
          for (int b = 0; b < NB; b++) acc[a][b] = typename G::Acc{0, 0, 0, 0};
#pragma unroll 1
        for (int k = 0; k < ks; k++) {
          typename G::Raw u{}, v[NA + NB];
          if constexpr (!kU8) u = G::load(urow, urow, k, g, nch);
#pragma unroll
          for (int t = 0; t < NA + NB; t++) v[t] = G::load(row[t], urow, k, g, nch);
          typename G::Op x[NA + NB];
#pragma unroll
          for (int t = 0; t < NA + NB; t++) {
            x[t] = G::op(v[t], u);
            if constexpr (kU8) sq[t] = sq_i8x16(x[t], sq[t]);
          }
#pragma unroll
          for (int a = 0; a < NA; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) acc[a][b] = G::mul(x[a], x[NA + b], acc[a][b]);
        }
        ntile += NA * NB;
        if constexpr (kU8) {
#pragma unroll
          for (int t = 0; t < NA + NB; t++) {
            sq[t] = sum_groups(sq[t]);
            if (t < NA && g == 0) rowL[16 * t + col] = __int_as_float(sq[t]);
          }
          __syncthreads();
        }
#pragma unroll
        for (int b = 0; b < NB; b++) {
          const int e = e0 + 16 * b + col;
          const ColTest<KIND> ct = col_test(e < m ? dpos[e] : 0.0f, sq[NA + b]);
#pragma unroll
          for (int a = 0; a < NA; a++) {
            const int i = 16 * a + 4 * g;
            const uint32_t w = test_word<KIND>(acc[a][b], kU8 ? rowL + i : od + first + a0 + i, ct, ns - a0 - i);
            if (g == 0) kw[64 * a + 16 * b + col] = w;
          }
        }
        __syncthreads();
        bool dead = false;
#pragma unroll
        for (int a = 0; a < NA; a++) dead |= alive && (kw[64 * a + ln] & 0xFFFFu) != 0u;
        if constexpr (!kU8) {
          for (int a = 0; a < NA; a++) {
            const uint32_t o = alive && !dead ? kw[64 * a + ln] >> 16 : 0u;
            if (ballot(o != 0u))
              dead |= resolve_open(P, o, oid + first + a0 + 16 * a, spos + e0, dpos + e0, coef, true) != 0u;
          }
        }
        alive = alive && !dead;
        __syncthreads();
      }
      const uint64_t gone = ~ballot(alive);
#pragma unroll
      for (int r = 0; r < NR; r++) {  // where the step's 64 candidates lie in register row r
        const int sh = e0 - 64 * r;
        if (sh >= 0 && sh < 64) keep[r] &= ~(gone << sh);
        if (sh < 0 && sh > -64) keep[r] &= ~(gone >> -sh);
      }
    }
    // survivors to the front, in order
    uint32_t si[NR];
    float sd[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) {
      si[r] = spos[r * 64 + ln];
      sd[r] = dpos[r * 64 + ln];
    }
    __syncthreads();
    int n = 0;
#pragma unroll
    for (int r = 0; r < NR; r++) {
      if ((keep[r] >> ln) & 1ull) {
        spos[n + mbcnt(keep[r])] = si[r];
        dpos[n + mbcnt(keep[r])] = sd[r];
      }
      n += popc(keep[r]);
    }
    m = n;
    __syncthreads();
  }
  __syncthreads();
  return nsel;
}

}  // namespace gr
