// k_prune.hip -- the forward prune of new nodes (Alg. 5, second loop) and the
// rebuild of every dirty node (Alg. 5 and Alg. 6, last loops) by
// GrANDRobustPrune (Alg. 4), one wavefront per node.
//
// The rebuild of uint8 rows of 64 or 128 bytes keeps the candidate tiles in
// registers (k_rebuild_mr); forward prunes, every other row length, fp32 rows,
// and scratch capacities above 64 take prune_gram (gram.h).
#include "gram.h"

namespace gr {

// GrANDRobustPrune's greedy selection for uint8 rows of 64*NK bytes, over
// up to 64*NR candidates already sorted by (D_p, id): spos/dpos (LDS) hold
// the sorted ids and distances, valid[] marks positions < m (element
// e = r*64 + lane).  Blocks of 16 sorted positions are taken in order: the
// block's rows are loaded as the MFMA A operand; the diagonal tile's kill
// masks resolve the block's own pivots in order (scalar loop), then every
// later tile that still holds a valid candidate is loaded as the B operand
// and its candidates are invalidated when their mask meets the selected
// pivots.  Distances are exact int32 (x ^ 0x80 operands), and the test
// coef * Dist <= D_p is the integer test Dist <= kill_threshold(coef, D_p).
// Rows are read from global memory (L2) when needed, the later tiles of a
// block kGroup at a time with all their loads in flight; nothing is staged.
// Lane t < nsel returns the t-th selection.
constexpr int kGroup = 4;  // candidate tiles loaded together by greedy_u8

template <int NK, int NR>
__device__ int greedy_u8(const PoolView &P, uint32_t p, int m, uint32_t R, double coef, const uint32_t *spos,
                         const float *dpos, bool (&valid)[NR], uint32_t &sid, float &sdist,
                         unsigned long long &evals) {
  const int ln = lane(), g = ln >> 4, col = ln & 15;
  const double inv = 1.0 / coef;
  const size_t goff = (size_t)g * 16;
  const int nt = (m + 15) >> 4;
  auto load_tile = [&](v4i (&dst)[NK], int t) -> int {
    const int e = 16 * t + col;
    const uint8_t *row = P.vecs + (size_t)(e < m ? spos[e] : p) * P.stride + goff;
    int sq = 0;
#pragma unroll
    for (int kk = 0; kk < NK; kk++) {
      dst[kk] = to_i8x16(ld16(row + (size_t)kk * 64));
      sq = sq_i8x16(dst[kk], sq);
    }
    sq += (int)xshfl((uint32_t)sq, 16);
    sq += (int)xshfl((uint32_t)sq, 32);
    return sq;
  };
  auto tile_valid = [&](int t) -> uint32_t {
    bool v = valid[0];
#pragma unroll
    for (int r = 1; r < NR; r++) v = r == (t >> 2) ? valid[r] : v;
    return (uint32_t)(ballot(v) >> (16 * (t & 3))) & 0xFFFFu;
  };
  sid = kInvalid;
  sdist = finf();
  int nsel = 0;
  bool done = false;
  uint32_t S_blk = 0;
  for (int b = 0; b < nt && !done; b++) {
    const uint32_t vb = tile_valid(b);
    if (!vb) continue;
    v4i A[NK];
    const int na = load_tile(A, b);
    int rn[4];
#pragma unroll
    for (int ii = 0; ii < 4; ii++) rn[ii] = __shfl(na, 4 * g + ii, 64);
    uint32_t kmd = 0;
    {
      const int thr = kill_threshold(coef, inv, dpos[16 * b + col]);
      v4i acc = {0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < NK; kk++) acc = mfma_i8(A[kk], A[kk], acc);
#pragma unroll
      for (int ii = 0; ii < 4; ii++) kmd |= (rn[ii] + na - 2 * acc[ii] <= thr) ? (1u << (4 * g + ii)) : 0u;
      kmd |= xshfl(kmd, 16);
      kmd |= xshfl(kmd, 32);
    }
    evals += 256;
    {
      // kmd (lane col): positions of the block that kill col; only earlier
      // ones matter
      uint32_t S = block_greedy(kmd & ((1u << col) - 1u), vb, col, g);
      int ns = __popc(S);
      if (ns >= (int)R - nsel) {
        ns = (int)R - nsel;
        S = first_bits(S, ns);
        done = true;
      }
      // lane nsel + k takes the k-th selected position of the block
      const int k = ln - nsel;
      if (k >= 0 && k < ns) {
        const int t = __ffs(first_bits(S, k + 1) & ~first_bits(S, k)) - 1;
        sid = spos[16 * b + t];
        sdist = dpos[16 * b + t];
      }
      nsel += ns;
      S_blk = S;
    }
    const uint32_t S = S_blk;
    if (done) break;
    // later tiles that still hold a valid candidate, kGroup at a time: all
    // loads of a group are issued before any is used
    int c = b + 1;
    while (c < nt) {
      int cs[kGroup];
      int ng = 0;
#pragma unroll
      for (int q = 0; q < kGroup; q++) {
        cs[q] = -1;
        while (c < nt && cs[q] < 0) {
          if (tile_valid(c)) cs[q] = c;
          c++;
        }
        ng += cs[q] >= 0 ? 1 : 0;
      }
      if (ng == 0) break;
      v4i Bt[kGroup][NK];
      int nb[kGroup], thr[kGroup];
#pragma unroll
      for (int q = 0; q < kGroup; q++) {
        nb[q] = 0;
        thr[q] = 0;
        if (cs[q] >= 0) {
          const int e = 16 * cs[q] + col;
          const uint8_t *row = P.vecs + (size_t)(e < m ? spos[e] : p) * P.stride + goff;
#pragma unroll
          for (int kk = 0; kk < NK; kk++) Bt[q][kk] = to_i8x16(ld16(row + (size_t)kk * 64));
          thr[q] = kill_threshold(coef, inv, dpos[e]);
        }
      }
#pragma unroll
      for (int q = 0; q < kGroup; q++) {
        if (cs[q] < 0) continue;
        int sq = 0;
        v4i acc = {0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < NK; kk++) {
          sq = sq_i8x16(Bt[q][kk], sq);
          acc = mfma_i8(A[kk], Bt[q][kk], acc);
        }
        sq += (int)xshfl((uint32_t)sq, 16);
        sq += (int)xshfl((uint32_t)sq, 32);
        nb[q] = sq;
        uint32_t km = 0;
#pragma unroll
        for (int ii = 0; ii < 4; ii++) km |= (rn[ii] + nb[q] - 2 * acc[ii] <= thr[q]) ? (1u << (4 * g + ii)) : 0u;
        km |= xshfl(km, 16);
        km |= xshfl(km, 32);
        evals += 256;
        const int cc = cs[q];
        const bool dead = g == (cc & 3) && (km & S) != 0;
#pragma unroll
        for (int r = 0; r < NR; r++)
          if (r == (cc >> 2)) valid[r] = valid[r] && !dead;
      }
    }
  }
  return nsel;
}

// greedy_u8 with every candidate tile resident in registers: the NT tiles
// (16 sorted candidates each, at most 16*NT candidates) are loaded once, all
// loads in flight together.  Live positions are kept as lane masks (bit e of
// vm[e / 64] for sorted position e), and per tile column the kill threshold
// minus the row's norm, so a kill test is one multiply-add and a compare:
// Dist(i, j) <= thr_j  <=>  |y_i|^2 - 2 y_i.y_j <= thr_j - |y_j|^2.  Against
// a later tile the compares of the block's rows are ballots, masked with the
// rows the block selected, and folded to the killed columns.  The selected
// positions go to oid/od (LDS) in order; returns their number.
template <int NK, int NT>
__device__ int greedy_u8_reg(const PoolView &P, uint32_t p, int m, uint32_t R, double coef, const uint32_t *spos,
                             const float *dpos, int *thr, int *nrmL, uint32_t *oid, float *od, uint32_t &ntile) {
  const int ln = lane(), g = ln >> 4, col = ln & 15;
  const double inv = 1.0 / coef;
  const size_t goff = (size_t)g * 16;
  const int nt = (m + 15) >> 4;
  constexpr int NR = (NT + 3) / 4;
  v4i T[NT][NK];
  {
    uint4 raw[NT][NK];
#pragma unroll
    for (int t = 0; t < NT; t++) {
      const int e = 16 * t + col;
      const uint8_t *row = P.vecs + (size_t)(e < m ? spos[e] : p) * P.stride + goff;
#pragma unroll
      for (int kk = 0; kk < NK; kk++) raw[t][kk] = 16 * t < m ? ld16(row + (size_t)kk * 64) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < NT; t++)
#pragma unroll
      for (int kk = 0; kk < NK; kk++) T[t][kk] = to_i8x16(raw[t][kk]);
  }
  // kill thresholds of the sorted positions (LDS), norms of the tile rows
#pragma unroll
  for (int r = 0; r < NR; r++) {
    const int e = r * 64 + ln;
    thr[e] = e < m ? kill_threshold(coef, inv, dpos[e]) : -1;
  }
  __syncthreads();
  int t2[NT];
#pragma unroll
  for (int t = 0; t < NT; t++) {
    int sq = 0;
#pragma unroll
    for (int kk = 0; kk < NK; kk++) sq = sq_i8x16(T[t][kk], sq);
    sq += (int)xshfl((uint32_t)sq, 16);
    sq += (int)xshfl((uint32_t)sq, 32);
    if (g == 0) nrmL[16 * t + col] = sq;
    t2[t] = thr[16 * t + col] - sq;
  }
  __syncthreads();
  uint64_t vm[NR];
#pragma unroll
  for (int r = 0; r < NR; r++) vm[r] = ballot(r * 64 + ln < m);
  int nsel = 0;
  bool done = false;
#pragma unroll
  for (int b = 0; b < NT; b++) {
    if (b >= nt || done) break;
    const uint32_t vb = (uint32_t)(vm[b >> 2] >> (16 * (b & 3))) & 0xFFFFu;
    if (!vb) continue;
    int rn[4];
#pragma unroll
    for (int ii = 0; ii < 4; ii++) rn[ii] = nrmL[16 * b + 4 * g + ii];
    // kb (lane col < 16): the block's earlier positions that would kill col
    uint32_t kb = 0;
    {
      v4i acc = {0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < NK; kk++) acc = mfma_i8(T[b][kk], T[b][kk], acc);
#pragma unroll
      for (int ii = 0; ii < 4; ii++) kb |= (rn[ii] - 2 * acc[ii] <= t2[b]) ? (1u << (4 * g + ii)) : 0u;
      kb |= xshfl(kb, 16);
      kb |= xshfl(kb, 32);
      kb &= (1u << col) - 1u;
    }
    ntile++;
    // the block's pivots in order: a live position is selected unless an
    // earlier selected one kills it
    uint32_t S = block_greedy(kb, vb, col, g);
    int ns = __popc(S);
    const int room = (int)R - nsel;
    if (ns >= room) {  // selection stops at R: keep the first `room`
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
    // whether block row 4g + ii (this lane's rows) was selected
    bool sb[4];
#pragma unroll
    for (int ii = 0; ii < 4; ii++) sb[ii] = ((S >> (4 * g + ii)) & 1u) != 0u;
#pragma unroll
    for (int c = b + 1; c < NT; c++) {
      if (c >= nt) break;
      if (!((vm[c >> 2] >> (16 * (c & 3))) & 0xFFFFull)) continue;
      v4i acc = {0, 0, 0, 0};
#pragma unroll
      for (int kk = 0; kk < NK; kk++) acc = mfma_i8(T[b][kk], T[c][kk], acc);
      // column col of tile c dies when a selected row of the block kills it
      bool k = false;
#pragma unroll
      for (int ii = 0; ii < 4; ii++) k |= sb[ii] && (rn[ii] - 2 * acc[ii] <= t2[c]);
      uint32_t kw = k ? 1u : 0u;
      kw |= xshfl(kw, 16);
      kw |= xshfl(kw, 32);
      const uint64_t d = ballot(kw != 0u && g == 0) & 0xFFFFull;
      vm[c >> 2] &= ~(d << (16 * (c & 3)));
      ntile++;
    }
  }
  __syncthreads();
  return nsel;
}

// ---------------------------------------------------------------------------
// Rebuild of dirty nodes.  For dirty u: scratch_u = the P smallest distinct
// (distance, source) records addressed to u; C = (N_out(u) u scratch_u)
// minus u (and minus the delete batch); if |C| <= R, C is installed (kept
// entries in slot order, then new sources in record order); otherwise
// GrANDRobustPrune(u, C, D_u) is installed.  One owner per dirty node, so
// rows are written without locks.

// C of dirty node u (R <= 64, P <= 64 * NP): the kept entries of N_out(u)
// (minus u and the delete batch) in slot order, then the sources of the P
// smallest distinct records that are not already kept, written to cl (LDS),
// with D_u of each in cdl (LDS): the stored distance of a kept entry, the
// record's distance of a new one.
// Returns |C|; nrec is the number of records addressed to u.
template <int NP>
__device__ int collect_candidates(const RebuildArgs &a, uint32_t u, uint4 *rowL, uint32_t *cl, uint32_t &nrec,
                                  float *cdl) {
  const int ln = lane();
  const PoolView &P = a.pool;
  const uint32_t R = P.R;
  const uint32_t g0 = a.goff[u], g1 = a.goff[u + 1];
  const uint32_t rv = ln < (int)R ? P.adj[(size_t)u * R + ln] : kInvalid;
  const float rdv = ln < (int)R ? P.adjd[(size_t)u * R + ln] : 0.0f;
  nrec = g1 - g0;
  // the first 64 records, loaded beside the row (lanes past the records
  // read a valid one and drop it); then the batch flags of the row's ids and
  // of those records' sources together (index 0 stands in for an id that
  // is not checked)
  const uint32_t j0 = g0 + (uint32_t)ln;
  const uint32_t jc = j0 < g1 ? j0 : (g1 > g0 ? g0 : 0u);
  const uint32_t s0 = a.gsrc[jc];
  const float d0 = a.gd[jc];
  const bool rok = rv != kInvalid && rv != u;
  const bool sok = j0 < g1 && kvalid(s0);
  bool rin = false, sin = false;
  if (a.in_batch) {
    const uint8_t fr = a.in_batch[rok ? rv : 0u];
    const uint8_t fs = a.in_batch[sok ? s0 : 0u];
    rin = rok && fr;
    sin = sok && fs;
  }
  // the merged sources below are all among these records when there are
  // at most 64; then none of them needs its flag loaded again
  const bool recheck = a.in_batch && (g1 - g0 > 64u || ballot(sin) != 0);
  const bool keep = rok && !rin;
  const uint64_t kmask = ballot(keep);
  int m = popc(kmask);
  reinterpret_cast<uint32_t *>(rowL)[ln] = keep ? rv : kInvalid;
  if (keep) {
    cl[mbcnt(kmask)] = rv;
    cdl[mbcnt(kmask)] = rdv;
  }
  __syncthreads();
  // scratch_u: the P smallest distinct (distance, source) records
  float sd[NP];
  uint32_t si[NP];
#pragma unroll
  for (int r = 0; r < NP; r++) {
    sd[r] = finf();
    si[r] = kInvalid;
  }
  for (uint32_t base = g0; base < g1; base += 64) {
    const uint32_t j = base + ln;
    uint32_t sv = j < g1 ? (base == g0 ? s0 : a.gsrc[j]) : kInvalid;
    float dv = j < g1 ? (base == g0 ? d0 : a.gd[j]) : finf();
    if (!kvalid(sv)) { sv = kInvalid; dv = finf(); }
    wave_merge_new_fast<NP>(sd, si, dv, sv, (int)a.P);
  }
#pragma unroll
  for (int r = 0; r < NP; r++) {
    const uint32_t sv = si[r];
    bool isnew = kvalid(sv) && sv != u && !(recheck && a.in_batch[sv]);
#pragma unroll 4
    for (int t = 0; t < 16; t++) {
      const uint4 r4 = rowL[t];
      isnew = isnew & (r4.x != sv) & (r4.y != sv) & (r4.z != sv) & (r4.w != sv);
    }
    const uint64_t nmask = ballot(isnew);
    if (isnew) {
      cl[m + mbcnt(nmask)] = sv;
      cdl[m + mbcnt(nmask)] = sd[r];
    }
    m += popc(nmask);
  }
  __syncthreads();
  return m;
}

// Candidate tiles a rebuild keeps in registers (|C| <= 80: the kept row and
// up to 16 records); larger candidate sets take greedy_u8.
constexpr int kRegTiles = 5;

// Rebuild of dirty nodes for uint8 rows of 64*NK bytes with P <= 64.  When a
// node prunes, its candidates are sorted by (D_u, id) and greedy_u8_reg (or
// greedy_u8, for more than 80 of them) selects.
template <int NK>
__global__ __launch_bounds__(64, 4) void k_rebuild_mr(RebuildArgs a) {
  constexpr int NC = 2;
  __shared__ uint4 rowL[16];
  __shared__ uint32_t cl[64 * NC];
  __shared__ float cdL[64 * NC];  // D_u of the candidates
  __shared__ uint32_t spos[64 * NC];
  __shared__ float dpos[64 * NC];
  __shared__ int thrL[64 * NC];
  __shared__ int nrmL[64 * NC];
  __shared__ uint32_t oid[64];
  __shared__ float od[64];
  const int ln = lane();
  const PoolView &P = a.pool;
  const uint32_t R = P.R;
  const uint32_t nd_total = *a.list_n;
  unsigned long long evals = 0;
  uint32_t prunes = 0, nodes = 0, recs = 0, cand = 0;
  // the next node of this wave is read while the current one is rebuilt
  uint32_t u_next = blockIdx.x < nd_total ? a.list[blockIdx.x] : 0u;
  for (uint32_t it = blockIdx.x; it < nd_total; it += gridDim.x) {
    const uint32_t u = u_next;
    u_next = a.list[it + gridDim.x < nd_total ? it + gridDim.x : it];
    nodes++;
    uint32_t nrec;
    const int m = collect_candidates<1>(a, u, rowL, cl, nrec, cdL);
    recs += nrec;
    if (m <= (int)R) {
      if (ln < (int)R) P.adj[(size_t)u * R + ln] = ln < m ? cl[ln] : kInvalid;
      if (ln < (int)R) P.adjd[(size_t)u * R + ln] = ln < m ? cdL[ln] : 0.0f;
      if (ln == 0) P.deg[u] = (uint32_t)m;
      __syncthreads();
      continue;
    }
    // Candidates by (D_u, id): 32-bit keys D << 7 | list position (uint8
    // distances are integers below 2^23) order them when no two share a
    // distance; a tie, which the id decides, takes the 64-bit key sort.
    uint32_t k32[NC];
#pragma unroll
    for (int r = 0; r < NC; r++) {
      const int e = r * 64 + ln;
      k32[r] = e < m ? ((uint32_t)cdL[e] << 7) | (uint32_t)e : ~0u;
    }
    wave_sort32<NC>(k32);
    bool tie = false;
#pragma unroll
    for (int r = 0; r < NC; r++) {
      // the next element's key (lane 63 of a row: lane 0 of the next row)
      uint32_t nx = __shfl(k32[r], (ln + 1) & 63, 64);
      if (ln == 63) nx = r + 1 < NC ? rdlane(k32[r + 1 < NC ? r + 1 : r], 0) : ~0u;
      tie |= r * 64 + ln + 1 < m && (k32[r] >> 7) == (nx >> 7);
    }
    if (!ballot(tie)) {
      uint32_t sid[NC];
#pragma unroll
      for (int r = 0; r < NC; r++) sid[r] = r * 64 + ln < m ? cl[k32[r] & 127u] : kInvalid;
#pragma unroll
      for (int r = 0; r < NC; r++) {
        spos[r * 64 + ln] = sid[r];
        dpos[r * 64 + ln] = r * 64 + ln < m ? (float)(k32[r] >> 7) : finf();
      }
    } else {
      uint64_t key[NC];
#pragma unroll
      for (int r = 0; r < NC; r++) {
        const int e = r * 64 + ln;
        key[r] = e < m ? key64(cdL[e], cl[e]) : ~0ull;
      }
      wave_sort64<NC>(key);
#pragma unroll
      for (int r = 0; r < NC; r++) {
        spos[r * 64 + ln] = (uint32_t)key[r];
        dpos[r * 64 + ln] = unsortable((uint32_t)(key[r] >> 32));
      }
    }
    __syncthreads();
    int nsel;
    if (m <= 16 * kRegTiles) {  // every candidate tile resident in registers
      uint32_t ntile = 0;
      nsel = greedy_u8_reg<NK, kRegTiles>(P, u, m, R, a.coef, spos, dpos, thrL, nrmL, oid, od, ntile);
      evals += 256ull * ntile;
    } else {  // more candidates (more than 16 records): tiles loaded per block
      bool valid[NC];
#pragma unroll
      for (int r = 0; r < NC; r++) valid[r] = r * 64 + ln < m;
      uint32_t sid;
      float sdist;
      nsel = greedy_u8<NK, NC>(P, u, m, R, a.coef, spos, dpos, valid, sid, sdist, evals);
      if (ln < nsel) {
        oid[ln] = sid;
        od[ln] = sdist;
      }
      __syncthreads();
    }
    if (ln < (int)R) P.adj[(size_t)u * R + ln] = ln < nsel ? oid[ln] : kInvalid;
    if (ln < (int)R) P.adjd[(size_t)u * R + ln] = ln < nsel ? od[ln] : 0.0f;
    if (ln == 0) P.deg[u] = (uint32_t)nsel;
    prunes++;
    cand += (unsigned long long)m;
    __syncthreads();
  }
  if (ln == 0) {
    stat_add(a.ds, kStRbPrunes, prunes);
    stat_add(a.ds, kStRbEvals, evals);
    stat_add(a.ds, kStRbCand, cand);
    if (a.count_nodes) {
      stat_add(a.ds, kStDirty, nodes);
      stat_add(a.ds, kStRbRecs, recs);
    }
  }
}

// Rebuild, fast path (R <= 64, R a multiple of 4): four dirty nodes per
// wavefront, 16 lanes per node, four row slots per lane.  For dirty u the
// records fit when there are at most min(16, P) of them, so scratch_u is all
// of them; C = (N_out(u) u scratch_u) minus u, repeats and the delete batch.
// When C fits in R it is installed here (kept entries in slot order, then
// the new sources); every other node -- more records than that, or |C| > R,
// which needs GrANDRobustPrune -- is flagged in `qflag` and later compacted
// into `queue` for the general kernel.  No distance is needed on this path.
__global__ __launch_bounds__(64) void k_rebuild_fast(RebuildArgs a) {
  __shared__ uint4 rowL[64];
  __shared__ uint32_t srcL[64];
  __shared__ uint32_t outL[4 * 64];
  __shared__ float outD[4 * 64];  // their list distances
  const int ln = lane(), s = ln >> 4, q = ln & 15;
  const PoolView &P = a.pool;
  const uint32_t R = P.R, R4 = R >> 2;
  const uint32_t nd = *a.list_n;
  const uint32_t lim = a.P < 16u ? a.P : 16u;
  unsigned long long nodes = 0, recs = 0;
  for (uint32_t b = blockIdx.x * 4u; b < nd; b += gridDim.x * 4u) {
    const uint32_t idx = b + (uint32_t)s;
    const bool has = idx < nd;
    const uint32_t u = has ? a.list[idx] : 0u;
    uint32_t g0 = 0, g1 = 0;
    uint4 rw = make_uint4(kInvalid, kInvalid, kInvalid, kInvalid);
    float4 rd = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (has) {
      g0 = a.goff[u];
      g1 = a.goff[u + 1];
      if ((uint32_t)q < R4) {
        rw = *reinterpret_cast<const uint4 *>(P.adj + (size_t)u * R + 4 * q);
        rd = *reinterpret_cast<const float4 *>(P.adjd + (size_t)u * R + 4 * q);
      }
    }
    const uint32_t nrec = g1 - g0;
    const bool light = has && nrec <= lim;
    uint32_t src = kInvalid;
    float srd = 0.0f;
    if (light && (uint32_t)q < nrec) {
      src = a.gsrc[g0 + q];
      srd = a.gd[g0 + q];
    }
    const float dk[4] = {rd.x, rd.y, rd.z, rd.w};
    const uint32_t id[4] = {rw.x, rw.y, rw.z, rw.w};
    bool keep[4];
#pragma unroll
    for (int k = 0; k < 4; k++) keep[k] = id[k] != kInvalid && id[k] != u && !(a.in_batch && a.in_batch[id[k]]);
    bool nw = kvalid(src) && src != u && !(a.in_batch && a.in_batch[src]);
    rowL[ln] = make_uint4(keep[0] ? id[0] : kInvalid, keep[1] ? id[1] : kInvalid, keep[2] ? id[2] : kInvalid,
                          keep[3] ? id[3] : kInvalid);
    srcL[ln] = src;
    __syncthreads();
    // a source already in the kept row, or repeated by an earlier record
#pragma unroll 4
    for (int j = 0; j < 16; j++) {
      const uint4 r = rowL[s * 16 + j];
      const uint32_t o = srcL[s * 16 + j];
      nw = nw & (r.x != src) & (r.y != src) & (r.z != src) & (r.w != src) & !((j < q) & (o == src));
    }
    // positions: kept entries in slot order, then the new sources
    const int kc = (int)keep[0] + (int)keep[1] + (int)keep[2] + (int)keep[3];
    int x = kc;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const int y = __shfl_up(x, o, 16);
      if (q >= o) x += y;
    }
    const int kr = __shfl(x, s * 16 + 15, 64);
    const uint32_t gm = (uint32_t)(ballot(nw) >> (16 * s)) & 0xFFFFu;
    const int m = kr + popc((uint64_t)gm);
    const bool install = light && m <= (int)R;
    if (install) {
      int pos = x - kc;
#pragma unroll
      for (int k = 0; k < 4; k++)
        if (keep[k]) {
          outL[s * 64 + pos] = id[k];
          outD[s * 64 + pos] = dk[k];
          pos++;
        }
      if (nw) {
        const int e = kr + popc((uint64_t)(gm & ((1u << q) - 1u)));
        outL[s * 64 + e] = src;
        outD[s * 64 + e] = srd;
      }
    }
    __syncthreads();
    if (install && (uint32_t)q < R4) {
      const int e = 4 * q;
      uint4 o;
      o.x = e + 0 < m ? outL[s * 64 + e + 0] : kInvalid;
      o.y = e + 1 < m ? outL[s * 64 + e + 1] : kInvalid;
      o.z = e + 2 < m ? outL[s * 64 + e + 2] : kInvalid;
      o.w = e + 3 < m ? outL[s * 64 + e + 3] : kInvalid;
      *reinterpret_cast<uint4 *>(P.adj + (size_t)u * R + e) = o;
      float4 d;
      d.x = e + 0 < m ? outD[s * 64 + e + 0] : 0.0f;
      d.y = e + 1 < m ? outD[s * 64 + e + 1] : 0.0f;
      d.z = e + 2 < m ? outD[s * 64 + e + 2] : 0.0f;
      d.w = e + 3 < m ? outD[s * 64 + e + 3] : 0.0f;
      *reinterpret_cast<float4 *>(P.adjd + (size_t)u * R + e) = d;
    }
    if (install && q == 0) P.deg[u] = (uint32_t)m;
    // nodes left for the general kernel are flagged by list position and
    // compacted afterwards (no shared counter on this path)
    if (has && q == 0) {
      a.qflag[idx] = install ? 0u : 1u;
      nodes++;
      recs += nrec;
    }
    __syncthreads();
  }
  // one atomic per wave: the counts live in lanes 0, 16, 32, 48
  unsigned long long tn = nodes, tr = recs;
#pragma unroll
  for (int k = 1; k < 4; k++) {
    tn += __shfl(nodes, 16 * k, 64);
    tr += __shfl(recs, 16 * k, 64);
  }
  if (ln == 0 && tn) {
    stat_add(a.ds, kStDirty, tn);
    stat_add(a.ds, kStRbRecs, tr);
  }
}

// ---------------------------------------------------------------------------
// Rebuild of queued dirty nodes for rows of any length (P <= 64 * NP), one
// wave per node, persistent over twice the resident workgroups: C and its
// distances as in k_rebuild_mr, a 64-bit-key sort, then prune_gram.
template <int KIND, int NP>
__global__ __launch_bounds__(64, 3) void k_rebuild_gram(RebuildArgs a) {
  constexpr int NC = NP == 1 ? 2 : 4;  // 64 + 64 * NP candidates at most, in a power of two of rows
  __shared__ uint4 rowL[16];
  __shared__ uint32_t cl[64 * NC];
  __shared__ __align__(16) float cdL[64 * NC];
  __shared__ uint32_t oid[64];
  __shared__ float od[64];
  const int ln = lane();
  const PoolView &P = a.pool;
  const uint32_t R = P.R;
  const uint32_t nd_total = *a.list_n;
  uint32_t ntile = 0, prunes = 0, nodes = 0, recs = 0, cand = 0;
  for (uint32_t it = blockIdx.x; it < nd_total; it += gridDim.x) {
    const uint32_t u = a.list[it];
    nodes++;
    uint32_t nrec;
    const int m = collect_candidates<NP>(a, u, rowL, cl, nrec, cdL);
    recs += nrec;
    int n = m;
    const uint32_t *ids = cl;
    const float *ds = cdL;
    if (m > (int)R) {
      uint64_t key[NC];
#pragma unroll
      for (int r = 0; r < NC; r++) {
        const int e = r * 64 + ln;
        key[r] = e < m ? key64(cdL[e], cl[e]) : ~0ull;
      }
      __syncthreads();
      wave_sort64<NC>(key);
#pragma unroll
      for (int r = 0; r < NC; r++) {
        cl[r * 64 + ln] = (uint32_t)key[r];
        cdL[r * 64 + ln] = unsortable((uint32_t)(key[r] >> 32));
      }
      __syncthreads();
      n = prune_gram<KIND, NC>(P, u, m, R, a.coef, cl, cdL, oid, od, ntile);
      ids = oid;
      ds = od;
      prunes++;
      cand += (uint32_t)m + 1;
    }
    if (ln < (int)R) {
      P.adj[(size_t)u * R + ln] = ln < n ? ids[ln] : kInvalid;
      P.adjd[(size_t)u * R + ln] = ln < n ? ds[ln] : 0.0f;
    }
    if (ln == 0) P.deg[u] = (uint32_t)n;
    __syncthreads();
  }
  if (ln == 0) {
    stat_add(a.ds, kStRbPrunes, (unsigned long long)prunes);
    stat_add(a.ds, kStRbEvals, 256ull * ntile);
    stat_add(a.ds, kStRbCand, (unsigned long long)cand);
    if (a.count_nodes) {
      stat_add(a.ds, kStDirty, (unsigned long long)nodes);
      stat_add(a.ds, kStRbRecs, (unsigned long long)recs);
    }
  }
}

// Forward GrANDRobustPrune of new points with rows of any length: V_i with the
// search's D, a 64-bit-key sort, then prune_gram.  A search adds fp64 terms in
// the order of its lane layout; the D that goes into the list and the records
// is that of the sum in dimension order (row_dists), so that what a later
// rebuild decides depends on the graph and the vectors alone, not on how an
// entry came into its list or on an import between (10,000 points on 1M x 96:
// 0.22 -> 0.24 ms a launch).
template <int KIND, int NR>
__global__ __launch_bounds__(64, 3) void k_fwd_prune_gram(FwdPruneArgs a) {
  __shared__ uint32_t spos[64 * (NR < 2 ? 2 : NR)];
  __shared__ __align__(16) float dpos[64 * (NR < 2 ? 2 : NR)];
  __shared__ uint32_t oid[64];
  __shared__ float od[64];
  const int ln = lane();
  const uint32_t i = blockIdx.x;
  if (i >= a.n) return;
  const PoolView &P = a.pool;
  const uint32_t p = a.ids[i];
  const uint32_t nv = a.v_n[i];
  const uint32_t R = P.R;
  uint64_t key[NR];
  int m = 0;
#pragma unroll
  for (int r = 0; r < NR; r++) {
    const uint32_t e = r * 64 + ln;
    const uint32_t id = e < nv ? a.v_ids[(size_t)i * a.v_stride + e] : kInvalid;
    const bool ok = kvalid(id) && id != p;
    key[r] = ok ? key64(a.v_d[(size_t)i * a.v_stride + e], id) : ~0ull;
    m += popc(ballot(ok));
  }
  // V_i holds distinct ids: the sort alone gives the candidate order
  wave_sort64<NR>(key);
#pragma unroll
  for (int r = 0; r < NR; r++) {
    spos[r * 64 + ln] = (uint32_t)key[r];
    dpos[r * 64 + ln] = unsortable((uint32_t)(key[r] >> 32));
  }
  __syncthreads();
  uint32_t ntile = 0;
  const int nsel = prune_gram<KIND, NR>(P, p, m, R, a.coef, spos, dpos, oid, od, ntile);
  if constexpr (KIND != kU8L2) {
    if (nsel)
      row_dists<KIND>(P.vecs + (size_t)p * P.stride, P.nch, oid, od, nsel,
                      [&](uint32_t x) { return P.vecs + (size_t)x * P.stride; });
    __syncthreads();
  }
  if (ln < (int)R) {
    const bool in = ln < nsel;
    const uint32_t sid = in ? oid[ln] : kInvalid;
    const float sd = in ? od[ln] : 0.0f;
    P.adj[(size_t)p * R + ln] = sid;
    P.adjd[(size_t)p * R + ln] = sd;
    a.rec_t[(size_t)i * R + ln] = sid;
    a.rec_s[(size_t)i * R + ln] = p;
    a.rec_d[(size_t)i * R + ln] = sd;
  }
  if (ln == 0) {
    P.deg[p] = (uint32_t)nsel;
    stat_add(a.ds, kStFwdPrunes, 1ull);
    stat_add(a.ds, kStFwdEvals, 256ull * ntile);
    stat_add(a.ds, kStRecords, (unsigned long long)nsel);
  }
}

hipError_t launch_fwd_prune(int kind, uint32_t max_iters, const FwdPruneArgs &a, hipStream_t st) {
  if (a.n == 0) return hipSuccess;
  if (a.pool.R > 64 || (kind != kU8L2 && kind != kF32L2)) return hipErrorInvalidValue;
  GR_DISPATCH_N(max_iters, {
    if (kind == kU8L2) hipLaunchKernelGGL((k_fwd_prune_gram<kU8L2, NR>), dim3(a.n), dim3(64), 0, st, a);
    else hipLaunchKernelGGL((k_fwd_prune_gram<kF32L2, NR>), dim3(a.n), dim3(64), 0, st, a);
    return hipGetLastError();
  });
  return hipErrorInvalidValue;
}

// The list distances that an import left unknown, of the nodes that are about
// to be pruned: one wave per node.  (Computing every list's at the import took
// a gather of the whole graph: 0.6 -> 6.9 ms for 50,000 x 960 fp32 rows of
// device memory, 0.9 -> 1.7 for 100,000 x 200 bytes.)
template <int KIND>
__global__ __launch_bounds__(64) void k_fill_dists(PoolView P, const uint32_t *list, const uint32_t *list_n) {
  __shared__ uint32_t ids[64];
  __shared__ float d[64];
  const int ln = lane();
  const uint32_t n = *list_n;
  for (uint32_t it = blockIdx.x; it < n; it += gridDim.x) {
    const uint32_t u = list[it];
    const size_t at = (size_t)u * P.R + ln;
    const uint32_t v = ln < (int)P.R ? P.adj[at] : kInvalid;
    const bool open = kvalid(v) && __float_as_uint(P.adjd[at]) == kUnknownDist;
    const uint64_t m = ballot(open);
    if (!m) continue;
    if (open) ids[mbcnt(m)] = v;
    __syncthreads();
    row_dists<KIND>(P.vecs + (size_t)u * P.stride, P.nch, ids, d, popc(m),
                    [&](uint32_t x) { return P.vecs + (size_t)x * P.stride; });
    __syncthreads();
    if (open) P.adjd[at] = d[mbcnt(m)];
    __syncthreads();
  }
}

// One persistent rebuild kernel over the queue: twice the resident
// workgroups, so that the second half starts as the first ones finish, which
// evens out the work per wave.
#define GR_REBUILD(...)                                                                                 \
  do {                                                                                                  \
    static const uint32_t res = resident_blocks((const void *)__VA_ARGS__);                             \
    hipLaunchKernelGGL((__VA_ARGS__), dim3(clamp_resident(grid, 2 * res)), dim3(64), 0, st, a);         \
  } while (0)

// Dirty nodes are rebuilt by the fast kernel when the row layout allows it
// (R a multiple of 4); the nodes it leaves, and every node otherwise, by the
// pruning kernel of the configuration.
hipError_t launch_rebuild(int kind, uint32_t R, uint32_t P, const RebuildArgs &a0, uint32_t grid, hipStream_t st) {
  if (grid == 0) return hipSuccess;
  if (P > 128 || R > 64 || (kind != kU8L2 && kind != kF32L2)) return hipErrorInvalidValue;
  RebuildArgs a = a0;
  a.list = a0.dirty;
  a.list_n = &a0.ds->n_dirty;
  a.count_nodes = 1;
  if (R % 4 == 0) {
    // grid >= min(records, 8192) >= the blocks needed at four nodes per wave
    hipLaunchKernelGGL(k_rebuild_fast, dim3(grid), dim3(64), 0, st, a);
    hipError_t e = launch_compact_flags(a.qflag, a.list, a.list_n, a0.flag_cap, a.queue, a.queue_n, a.scan_tmp, st);
    if (e != hipSuccess) return e;
    a.list = a0.queue;
    a.list_n = a0.queue_n;
    a.count_nodes = 0;
  }
  if (a.fill) {
    if (kind == kU8L2) hipLaunchKernelGGL(k_fill_dists<kU8L2>, dim3(grid), dim3(64), 0, st, a.pool, a.list, a.list_n);
    else hipLaunchKernelGGL(k_fill_dists<kF32L2>, dim3(grid), dim3(64), 0, st, a.pool, a.list, a.list_n);
  }
  // uint8 rows of 64 and 128 bytes: a node's tiles stay in registers and only
  // the tiles that still hold a live candidate are multiplied (0.42 ms per
  // launch of a 10,000-point batch on 1M x 128, prune_gram 0.54; rebuilds of a
  // 5,000-point batch on 500K x 64 0.34 ms a round, prune_gram 0.48)
  if (kind == kU8L2 && P <= 64 && (a.pool.nch == 8 || a.pool.nch == 4)) {
    if (a.pool.nch == 8) GR_REBUILD(k_rebuild_mr<2>);
    else GR_REBUILD(k_rebuild_mr<1>);
  } else if (kind == kU8L2) {
    if (P <= 64) GR_REBUILD(k_rebuild_gram<kU8L2, 1>);
    else GR_REBUILD(k_rebuild_gram<kU8L2, 2>);
  } else {
    if (P <= 64) GR_REBUILD(k_rebuild_gram<kF32L2, 1>);
    else GR_REBUILD(k_rebuild_gram<kF32L2, 2>);
  }
  return hipGetLastError();
}

}  // namespace gr
