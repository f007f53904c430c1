// gram.h -- GrANDRobustPrune (Alg. 4) over fp32 candidates on the matrix
// cores, one wavefront per node.
//
// The prune asks one question per pair: does a selected candidate i kill a
// later candidate j, coef * Dist(i, j) <= D[j], where Dist is the fp64 sum
// rounded once to fp32.  With y = x - x_p (the candidates seen from the node
// p that is pruned) Dist(i, j) = D[i] + D[j] - 2 y_i.y_j, and D is known for
// every candidate before the prune starts.  The products y_i.y_j run on the
// bf16 matrix cores, each value split into two bf16 pieces (hi + lo, three
// products), and every test comes with a bound on its error; a test that the
// bound leaves open is repeated exactly.  So the decisions, and with them the
// lists, are those of the fp64 arithmetic.
//
// The error of one approximate distance, relative to D[j] (D[i] <= D[j], as
// candidates come in that order, so sum |y_i||y_j| <= sqrt(D[i] D[j]) <=
// D[j]): splitting leaves 3 * 2^-18 of a product (the two residuals of at
// most 2^-18 and lo*lo), the fp32 accumulation of 3 * d products at most
// 2^-23 per addition, and a few more roundings of D, y and the test itself.
// At d = 96 that is 1.0e-4 of D[j], at d = 960 7.1e-4, so few tests are open
// (about one pruned node in ten has one at d = 96).
//
// Measured against one lane per candidate summing fp64 (whose arithmetic was
// the bound): rebuilds of a 10,000-point batch on 1M x 96 6.93 -> 0.88 ms per
// launch, forward prunes 0.99 -> 0.21 ms; with 2,000-point batches on 100K x
// 960 4.67 -> 0.35 ms and 3.50 -> 0.40 ms.  What bounds it now is the latency
// of the row gathers at three waves per SIMD (the accumulators take 60
// registers) and the selection around them.
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
__device__ __forceinline__ void split8(const float (&x)[8], v8bf &hi, v8bf &lo) {
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    const v2bf h = {(__bf16)x[i], (__bf16)x[i + 1]};
    const uint32_t w = __builtin_bit_cast(uint32_t, h);
    const v2bf l = {(__bf16)(x[i] - __uint_as_float(w << 16)), (__bf16)(x[i + 1] - __uint_as_float(w & 0xFFFF0000u))};
    hi[i] = h[0];
    hi[i + 1] = h[1];
    lo[i] = l[0];
    lo[i + 1] = l[1];
  }
}
__device__ __forceinline__ v4f mfma_split(v8bf ah, v8bf al, v8bf bh, v8bf bl, v4f c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bl, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(al, bh, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ah, bh, c, 0, 0, 0);
}

// Dist of two pool rows (squared L2), by the whole wave: lane l adds chunks
// l, l + 64, ... in fp64.  The rounded result is that of the sum in dimension
// order: where the two orders (they differ by less than 2^-40 of the sum for
// rows of up to 1024 floats) could round apart, that sum is taken instead.
__device__ __forceinline__ float pair_l2(const PoolView &P, uint32_t a, uint32_t b) {
  const uint8_t *ra = P.vecs + (size_t)a * P.stride, *rb = P.vecs + (size_t)b * P.stride;
  double s = 0.0;
  for (int c = lane(); c < P.nch; c += 64) s = l2_4(ld16(ra + (size_t)c * 16), ld16(rb + (size_t)c * 16), s);
  s = group_sum<64>(s);
  const float f0 = (float)(s * (1.0 - 0x1p-40)), f1 = (float)(s * (1.0 + 0x1p-40));
  if (f0 != f1) {
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

// This lane's 8 floats of one K step (dimensions k0 + 8g ..) of a row;
// dimensions past the row give zeros (rows hold nfl floats, a multiple of 4).
__device__ __forceinline__ void load8(const float *row, int f, int nfl, uint4 (&v)[2]) {
  v[0] = *reinterpret_cast<const uint4 *>(row + (f < nfl ? f : 0));
  v[1] = *reinterpret_cast<const uint4 *>(row + (f + 4 < nfl ? f + 4 : 0));
}
__device__ __forceinline__ void diff8(const uint4 (&v)[2], const uint4 (&u)[2], int f, int nfl, float (&x)[8]) {
  const uint32_t a[8] = {v[0].x, v[0].y, v[0].z, v[0].w, v[1].x, v[1].y, v[1].z, v[1].w};
  const uint32_t b[8] = {u[0].x, u[0].y, u[0].z, u[0].w, u[1].x, u[1].y, u[1].z, u[1].w};
#pragma unroll
  for (int i = 0; i < 8; i++)
    x[i] = f + (i & 4) < nfl ? __uint_as_float(a[i]) - __uint_as_float(b[i]) : 0.0f;
}

// The tests of one tile pair's products as words: lane (g, col) holds rows 4g
// .. 4g+3 (their D in di, the first `n` of them exist) against column col;
// every lane gets its column's word, bit i set when row i kills the column
// and bit 16 + i when that test is open.
__device__ __forceinline__ uint32_t test_word(v4f acc, const float *di, float lo, float hi, int n) {
  const int g = lane() >> 4;
  uint32_t w = 0;
#pragma unroll
  for (int ii = 0; ii < 4; ii++) {
    const float a = __builtin_fmaf(-2.0f, acc[ii], ii < n ? di[ii] : 0.0f);
    const bool kill = a <= lo, safe = a > hi;
    w |= ii < n && kill ? 1u << ii : 0u;
    w |= ii < n && !(kill | safe) ? 0x10000u << ii : 0u;
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
// and D in dpos (LDS, at least m rounded up to 16 entries, at most 256; both
// are overwritten).  The selections go to oid / od (LDS, R entries) in order;
// returns their number.
//
// Panels of up to 80 candidates are taken in order.  A panel's rows are read
// once, 32 dimensions at a time, and all pairs of its 16-candidate tiles are
// multiplied (15 tile products, 60 accumulator registers); the tests become
// one word per tile pair and column (16 kill bits, 16 open bits), from which
// the greedy selection is resolved tile by tile without further distances.
// The candidates behind the panel are then tested against its selections
// only, and the survivors packed for the next panel.
template <int NR>
__device__ int prune_gram(const PoolView &P, uint32_t p, int m, uint32_t R, double coef, uint32_t *spos, float *dpos,
                          uint32_t *oid, float *od, uint32_t &ntile) {
  __shared__ uint32_t kw[kPanelPairs * 16];  // test words by (tile pair, column)
  const int ln = lane(), g = ln >> 4, col = ln & 15;
  const int nfl = P.nch * 4;
  const KillRange kr = kill_range(coef, nfl);
  const float *urow = reinterpret_cast<const float *>(P.vecs + (size_t)p * P.stride);
  int nsel = 0;
  while (m > 0) {
    const int pm = m < kPanel ? m : kPanel;
    const int nt = (pm + 15) >> 4;
    {
      // tiles past the panel hold the node's own row (no branch among the
      // loads, so all of a step's are in flight together)
      const float *row[kPanelTiles];
#pragma unroll
      for (int t = 0; t < kPanelTiles; t++) {
        const int e = 16 * t + col;
        row[t] = reinterpret_cast<const float *>(P.vecs + (size_t)(e < pm ? spos[e] : p) * P.stride);
      }
      v4f acc[kPanelPairs];
#pragma unroll
      for (int i = 0; i < kPanelPairs; i++) acc[i] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
      for (int k0 = 0; k0 < nfl; k0 += 32) {
        const int f = k0 + 8 * g;
        uint4 u[2], v[kPanelTiles][2];
        load8(urow, f, nfl, u);
#pragma unroll
        for (int t = 0; t < kPanelTiles; t++) load8(row[t], f, nfl, v[t]);
        v8bf hi[kPanelTiles], lo[kPanelTiles];
#pragma unroll
        for (int t = 0; t < kPanelTiles; t++) {
          float x[8];
          diff8(v[t], u, f, nfl, x);
          split8(x, hi[t], lo[t]);
        }
#pragma unroll
        for (int c = 0; c < kPanelTiles; c++)
#pragma unroll
          for (int b = 0; b <= c; b++)
            acc[pair_at(b, c)] = mfma_split(hi[b], lo[b], hi[c], lo[c], acc[pair_at(b, c)]);
      }
      ntile += (uint32_t)(nt * (nt + 1) / 2);
#pragma unroll
      for (int c = 0; c < kPanelTiles; c++) {
        const int e = 16 * c + col;
        float lo, hi;
        test_range(kr, e < pm ? dpos[e] : 0.0f, lo, hi);
#pragma unroll
        for (int b = 0; b <= c; b++) {
          const uint32_t w = test_word(acc[pair_at(b, c)], dpos + 16 * b + 4 * g, lo, hi, 4);
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
      const uint32_t open = ((vb >> col) & 1u) && g == 0 ? (kb >> 16) & before : 0u;
      kb &= before;
      if (ballot(open != 0u)) kb |= resolve_open(P, open, spos + 16 * b, spos + 16 * b, dpos + 16 * b, coef, false);
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
        const uint32_t o = dead ? 0u : (w >> 16) & S;
        if (ballot(o != 0u))
          dead |= resolve_open(P, o, spos + 16 * b, spos + 16 * c0, dpos + 16 * c0, coef, true) != 0u;
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
        const float *ra[NA], *rb[NB];
#pragma unroll
        for (int t = 0; t < NA; t++) {
          const int e = a0 + 16 * t + col;
          ra[t] = reinterpret_cast<const float *>(P.vecs + (size_t)(e < ns ? oid[first + e] : p) * P.stride);
        }
#pragma unroll
        for (int t = 0; t < NB; t++) {
          const int e = e0 + 16 * t + col;
          rb[t] = reinterpret_cast<const float *>(P.vecs + (size_t)(e < m ? spos[e] : p) * P.stride);
        }
        v4f acc[NA][NB];
#pragma unroll
        for (int a = 0; a < NA; a++)
#pragma unroll
          for (int b = 0; b < NB; b++) acc[a][b] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
        for (int k0 = 0; k0 < nfl; k0 += 32) {
          const int f = k0 + 8 * g;
          uint4 u[2], v[NA + NB][2];
          load8(urow, f, nfl, u);
#pragma unroll
          for (int t = 0; t < NA + NB; t++) load8(t < NA ? ra[t] : rb[t - NA], f, nfl, v[t]);
          v8bf hi[NA + NB], lo[NA + NB];
#pragma unroll
          for (int t = 0; t < NA + NB; t++) {
            float x[8];
            diff8(v[t], u, f, nfl, x);
            split8(x, hi[t], lo[t]);
          }
#pragma unroll
          for (int a = 0; a < NA; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) acc[a][b] = mfma_split(hi[a], lo[a], hi[NA + b], lo[NA + b], acc[a][b]);
        }
        ntile += NA * NB;
#pragma unroll
        for (int b = 0; b < NB; b++) {
          const int e = e0 + 16 * b + col;
          float lo, hi;
          test_range(kr, e < m ? dpos[e] : 0.0f, lo, hi);
#pragma unroll
          for (int a = 0; a < NA; a++) {
            const int i = a0 + 16 * a + 4 * g;
            const uint32_t w = test_word(acc[a][b], od + first + i, lo, hi, ns - i);
            if (g == 0) kw[64 * a + 16 * b + col] = w;
          }
        }
        __syncthreads();
        bool dead = false;
#pragma unroll
        for (int a = 0; a < NA; a++) dead |= alive && (kw[64 * a + ln] & 0xFFFFu) != 0u;
        for (int a = 0; a < NA; a++) {
          const uint32_t o = alive && !dead ? kw[64 * a + ln] >> 16 : 0u;
          if (ballot(o != 0u))
            dead |= resolve_open(P, o, oid + first + a0 + 16 * a, spos + e0, dpos + e0, coef, true) != 0u;
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
