// vec.h -- distance evaluation by a wavefront against gathered pool rows.
//
// Distance (the single Dist used everywhere in the method):
//   L2 : squared Euclidean distance;  IP : negated inner product.
// uint8 rows are summed exactly in 32-bit integers; fp32 rows are summed in
// fp64 (each difference and product is exact in fp64) and rounded once to
// fp32.  A zero result is returned as +0.
//
// Layout: every pool row is padded with zeros to a multiple of 16 bytes
// ("chunks").  A row is handled by LPV consecutive lanes ("a group"); lane
// `sub` of a group owns chunks sub, sub+LPV, ... (at most CPL of them).  The
// query (or the pivot of a prune) is held by every group in registers in the
// same chunk layout, so 64/LPV rows are evaluated per step and a step's
// partial sums are reduced with log2(LPV) shuffles.
#pragma once
#include "wave.h"

namespace gr {

enum { kF32L2 = 0, kF32IP = 1, kU8L2 = 2 };

__device__ __forceinline__ uint4 ld16(const uint8_t* p) { return *reinterpret_cast<const uint4*>(p); }
__device__ __forceinline__ uint32_t udot4(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_udot4(a, b, c, false);
}
__device__ __forceinline__ float canon0(float x) { return x == 0.0f ? 0.0f : x; }

// int8 matrix-core operands: uint8 rows are used as x ^ 0x80 = x - 128
// (signed), which leaves squared Euclidean distances unchanged, so
// Dist(i, j) = |y_i|^2 + |y_j|^2 - 2 y_i.y_j holds exactly in int32.
typedef int v4i __attribute__((ext_vector_type(4)));
__device__ __forceinline__ int sdot4(uint32_t a, uint32_t b, int c) {
  return __builtin_amdgcn_sdot4((int)a, (int)b, c, false);
}
__device__ __forceinline__ v4i to_i8x16(uint4 v) {
  v4i r;
  r[0] = (int)(v.x ^ 0x80808080u);
  r[1] = (int)(v.y ^ 0x80808080u);
  r[2] = (int)(v.z ^ 0x80808080u);
  r[3] = (int)(v.w ^ 0x80808080u);
  return r;
}
__device__ __forceinline__ int sq_i8x16(v4i a, int acc) {
#pragma unroll
  for (int w = 0; w < 4; w++) acc = sdot4((uint32_t)a[w], (uint32_t)a[w], acc);
  return acc;
}
__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

template <int KIND> struct Acc;
template <> struct Acc<kU8L2> { typedef uint32_t T; };
template <> struct Acc<kF32L2> { typedef double T; };
template <> struct Acc<kF32IP> { typedef double T; };

// Whether a sum s known to e rounds to fp32 in one way only.  Two orders of a
// sum of at most 1024 fp64 terms differ by less than 2^-42 of the sum of the
// terms' magnitudes; a kernel that needs the value of the sum in dimension
// order, and adds in another, sums again where this is false.
__device__ __forceinline__ bool rounds_once(double s, double e) { return (float)(s - e) == (float)(s + e); }

template <int KIND, int LPV, int CPL>
struct Slice {
  uint4 q[CPL];
  uint32_t qn;  // uint8 L2: this lane's part of |q|^2
};

template <int KIND, int LPV, int CPL>
__device__ __forceinline__ void load_slice(Slice<KIND, LPV, CPL>& s, const uint8_t* row, int nch) {
  const int sub = lane() % LPV;
  s.qn = 0;
#pragma unroll
  for (int k = 0; k < CPL; k++) {
    const int c = sub + k * LPV;
    s.q[k] = c < nch ? ld16(row + (size_t)c * 16) : make_uint4(0, 0, 0, 0);
    if (KIND == kU8L2) {
      s.qn = udot4(s.q[k].x, s.q[k].x, s.qn);
      s.qn = udot4(s.q[k].y, s.q[k].y, s.qn);
      s.qn = udot4(s.q[k].z, s.q[k].z, s.qn);
      s.qn = udot4(s.q[k].w, s.q[k].w, s.qn);
    }
  }
}

__device__ __forceinline__ double l2_4(uint4 a, uint4 b, double acc) {
  const float* fa = reinterpret_cast<const float*>(&a);
  const float* fb = reinterpret_cast<const float*>(&b);
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const double t = (double)fb[i] - (double)fa[i];
    acc = __builtin_fma(t, t, acc);
  }
  return acc;
}
__device__ __forceinline__ double ip_4(uint4 a, uint4 b, double acc) {
  const float* fa = reinterpret_cast<const float*>(&a);
  const float* fb = reinterpret_cast<const float*>(&b);
#pragma unroll
  for (int i = 0; i < 4; i++) acc = __builtin_fma((double)fa[i], (double)fb[i], acc);
  return acc;
}
__device__ __forceinline__ uint32_t u8l2_4(uint4 a, uint4 b, uint32_t acc) {
  // |b|^2 - 2 a.b over 16 bytes; with the query's |a|^2 added once this is
  // the exact sum of squared differences (modulo 2^32, exact in range)
  acc = udot4(b.x, b.x, acc);
  acc = udot4(b.y, b.y, acc);
  acc = udot4(b.z, b.z, acc);
  acc = udot4(b.w, b.w, acc);
  uint32_t ab = udot4(a.x, b.x, 0u);
  ab = udot4(a.y, b.y, ab);
  ab = udot4(a.z, b.z, ab);
  ab = udot4(a.w, b.w, ab);
  return acc - 2u * ab;
}

template <int KIND, int LPV, int CPL>
__device__ __forceinline__ typename Acc<KIND>::T partial(const Slice<KIND, LPV, CPL>& s, const uint4 (&b)[CPL]) {
  typename Acc<KIND>::T acc;
  if (KIND == kU8L2) acc = s.qn; else acc = 0;
#pragma unroll
  for (int k = 0; k < CPL; k++) {
    if (KIND == kU8L2) acc = u8l2_4(s.q[k], b[k], acc);
    else if (KIND == kF32L2) acc = l2_4(s.q[k], b[k], acc);
    else acc = ip_4(s.q[k], b[k], acc);
  }
  return acc;
}

template <int KIND, int LPV, int CPL>
__device__ __forceinline__ void partial2(const Slice<KIND, LPV, CPL>& s, const uint4 (&a)[CPL], const uint4 (&b)[CPL],
                                         typename Acc<KIND>::T& ta, typename Acc<KIND>::T& tb) {
  if (KIND == kU8L2) ta = tb = s.qn;
#pragma unroll
  for (int k = 0; k < CPL; k++) {
    if constexpr (KIND == kU8L2) {
      ta = u8l2_4(s.q[k], a[k], ta);
      tb = u8l2_4(s.q[k], b[k], tb);
    } else {
      const float *q = reinterpret_cast<const float *>(&s.q[k]), *fa = reinterpret_cast<const float *>(&a[k]),
                  *fb = reinterpret_cast<const float *>(&b[k]);
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const double x = (double)q[i];
        if constexpr (KIND == kF32L2) {
          const double da = (double)fa[i] - x, db = (double)fb[i] - x;
          ta = __builtin_fma(da, da, ta);
          tb = __builtin_fma(db, db, tb);
        } else {
          ta = __builtin_fma(x, (double)fa[i], ta);
          tb = __builtin_fma(x, (double)fb[i], tb);
        }
      }
    }
  }
}

__device__ __forceinline__ uint32_t xshfl_any(uint32_t v, int j) { return xshfl(v, j); }
__device__ __forceinline__ double xshfl_any(double v, int j) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = xshfl((uint32_t)b, j), hi = xshfl((uint32_t)(b >> 32), j);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
template <int LPV>
__device__ __forceinline__ uint32_t group_sum(uint32_t v) {
#pragma unroll
  for (int o = 1; o < LPV; o <<= 1) v += xshfl(v, o);
  return v;
}
template <int LPV>
__device__ __forceinline__ double group_sum(double v) {
#pragma unroll
  for (int o = 1; o < LPV; o <<= 1) v += xshfl_any(v, o);
  return v;
}

// The sums over each group of W lanes of N values (N a power of two below W):
// at every step the lower half of a group passes on one value and the upper
// half the other, so N values cost N - 1 + log2(W / N) exchanges instead of
// N * log2(W).  Returned: in lane l the sum of value fold_index<N, W>().
template <int N, int W, class T>
__device__ __forceinline__ T fold_sum(T (&t)[N]) {
  if constexpr (N == 1) {
    return group_sum<W>(t[0]);
  } else {
    const bool up = (lane() & (W / 2)) != 0;
    T h[N / 2];
#pragma unroll
    for (int i = 0; i < N / 2; i++) {
      const T keep = up ? t[i + N / 2] : t[i], pass = up ? t[i] : t[i + N / 2];
      h[i] = keep + xshfl_any(pass, W / 2);
    }
    return fold_sum<N / 2, W / 2>(h);
  }
}
template <int N, int W>
__device__ __forceinline__ int fold_index() {
  int r = 0;
#pragma unroll
  for (int n = N, w = W; n > 1; n >>= 1, w >>= 1) r += (lane() & (w / 2)) ? n / 2 : 0;
  return r;
}

template <int KIND>
__device__ __forceinline__ float finalize(typename Acc<KIND>::T t) {
  if (KIND == kU8L2) return canon0((float)t);
  if (KIND == kF32L2) return canon0((float)t);
  return canon0((float)(-t));
}

// Dist of two rows of nch 16-byte chunks, one lane, dimensions in order
// (zero padding adds nothing).
template <int KIND>
__device__ __forceinline__ float dist_seq(const uint8_t *a, const uint8_t *b, int nch) {
  if (KIND == kU8L2) {
    uint32_t s = 0;
    for (int c = 0; c < nch; c++) {
      const uint4 x = ld16(a + 16 * c), y = ld16(b + 16 * c);
      const uint32_t xw[4] = {x.x, x.y, x.z, x.w}, yw[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int w = 0; w < 4; w++)
#pragma unroll
        for (int k = 0; k < 4; k++) {
          const int t = (int)((xw[w] >> (8 * k)) & 0xFFu) - (int)((yw[w] >> (8 * k)) & 0xFFu);
          s += (uint32_t)(t * t);
        }
    }
    return canon0((float)s);
  } else {
    double s = 0.0;
    for (int c = 0; c < nch; c++) {
      const float4 x = *reinterpret_cast<const float4 *>(a + 16 * c);
      const float4 y = *reinterpret_cast<const float4 *>(b + 16 * c);
      const float xf[4] = {x.x, x.y, x.z, x.w}, yf[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
      for (int k = 0; k < 4; k++) {
        if (KIND == kF32L2) {
          const double t = (double)xf[k] - (double)yf[k];
          s = __builtin_fma(t, t, s);
        } else {
          s = __builtin_fma((double)xf[k], (double)yf[k], s);
        }
      }
    }
    return canon0(KIND == kF32IP ? (float)(-s) : (float)s);
  }
}

__device__ __forceinline__ uint4 abs_4(uint4 v) {
  return make_uint4(v.x & 0x7FFFFFFFu, v.y & 0x7FFFFFFFu, v.z & 0x7FFFFFFFu, v.w & 0x7FFFFFFFu);
}

// The distances of the row `ru` to n >= 1 rows, row(ids[j]) (ids and out in
// LDS), as the sums in dimension order round: 8 lanes a row, two rows of each
// lane group and four chunks of a lane in flight; a sum whose order could move
// the rounding is taken again, in order (about one in 130,000).
template <int KIND, class Row>
__device__ __forceinline__ void row_dists(const uint8_t *ru, int nch, const uint32_t *ids, float *out, int n, Row row) {
  constexpr int U = 4;
  const int grp = lane() >> 3, sub = lane() & 7;
  for (int j0 = 0; j0 < n; j0 += 16) {
    const uint8_t *r0 = row(ids[min(j0 + grp, n - 1)]), *r1 = row(ids[min(j0 + 8 + grp, n - 1)]);
    typename Acc<KIND>::T s0 = 0, s1 = 0;
    double m0 = 0.0, m1 = 0.0;  // inner products: the terms' magnitudes
    for (int c0 = sub; c0 < nch + sub; c0 += 8 * U) {  // the same steps in every lane
      uint4 q[U], x0[U], x1[U];
#pragma unroll
      for (int k = 0; k < U; k++) {
        const size_t o = (size_t)min(c0 + 8 * k, nch - 1) * 16;
        q[k] = ld16(ru + o);
        x0[k] = ld16(r0 + o);
        x1[k] = ld16(r1 + o);
      }
#pragma unroll
      for (int k = 0; k < U; k++) {
        if (c0 + 8 * k >= nch) q[k] = x0[k] = x1[k] = make_uint4(0, 0, 0, 0);
        if constexpr (KIND == kU8L2) {
          const uint32_t qq =
              udot4(q[k].w, q[k].w, udot4(q[k].z, q[k].z, udot4(q[k].y, q[k].y, udot4(q[k].x, q[k].x, 0u))));
          s0 = u8l2_4(q[k], x0[k], s0 + qq);
          s1 = u8l2_4(q[k], x1[k], s1 + qq);
        } else if constexpr (KIND == kF32L2) {
          s0 = l2_4(q[k], x0[k], s0);
          s1 = l2_4(q[k], x1[k], s1);
        } else {
          s0 = ip_4(q[k], x0[k], s0);
          s1 = ip_4(q[k], x1[k], s1);
          m0 = ip_4(abs_4(q[k]), abs_4(x0[k]), m0);
          m1 = ip_4(abs_4(q[k]), abs_4(x1[k]), m1);
        }
      }
    }
    s0 = group_sum<8>(s0);
    s1 = group_sum<8>(s1);
    float d0 = finalize<KIND>(s0), d1 = finalize<KIND>(s1);
    if constexpr (KIND != kU8L2) {
      const double e0 = KIND == kF32IP ? group_sum<8>(m0) : s0, e1 = KIND == kF32IP ? group_sum<8>(m1) : s1;
      if (!rounds_once(s0, e0 * 0x1p-42)) d0 = dist_seq<KIND>(ru, r0, nch);
      if (!rounds_once(s1, e1 * 0x1p-42)) d1 = dist_seq<KIND>(ru, r1, nch);
    }
    if (sub == 0) {
      if (j0 + grp < n) out[j0 + grp] = d0;
      if (j0 + 8 + grp < n) out[j0 + 8 + grp] = d1;
    }
  }
}

// Distances from the slice to rows ids[0..cnt) (ids in LDS), written to
// out[0..cnt) (LDS).  All gathers of RIF steps are issued before any is
// consumed so that many rows are in flight per wave: 8 chunks per lane for
// rows of 8 lanes (64 rows of one chunk a lane, 16 rows of four), 32 for
// longer rows, whose few sums are folded (fold_sum), and one row's 16 chunks
// per lane for the longest rows of a wave that has its SIMD to itself.  ORDER
// (squared L2; qrow: the slice's row): the distances are those of the sums in
// dimension order, a sum whose order could move its rounding taken again.
template <int KIND, int LPV, int CPL, bool ORDER = false>
__device__ __forceinline__ void wave_dists(const Slice<KIND, LPV, CPL>& s, const uint8_t* __restrict__ vecs,
                                           size_t stride, int nch, const uint32_t* ids, float* out, int cnt,
                                           const uint8_t* qrow = nullptr) {
  static_assert(!ORDER || KIND != kF32IP, "inner products need the magnitude of their terms");
  auto dist = [&](typename Acc<KIND>::T t, int c) {
    if constexpr (ORDER && KIND == kF32L2) {
      if (!rounds_once(t, t * 0x1p-42)) return dist_seq<KIND>(qrow, vecs + (size_t)ids[c] * stride, nch);
    }
    return finalize<KIND>(t);
  };
  constexpr int G = 64 / LPV;
  constexpr bool kFold = LPV >= 16 && CPL <= 4;
  constexpr int RIF = kFold ? 32 / CPL : CPL >= 8 ? 1 : 8 / CPL;
  const int ln = lane(), grp = ln / LPV, sub = ln % LPV;
  for (int base = 0; base < cnt; base += G * RIF) {
    // steps whose rows all lie beyond cnt are skipped (uniform branches)
    const int steps = (cnt - base + G - 1) / G;
    uint4 b[RIF][CPL];
    if constexpr (kFold) {
      // The ids are read together (a read per step waits for LDS before each
      // step's gathers), groups past the rows gather the last one again, and
      // lanes past a row's chunks its last one, cleared afterwards (a branch
      // around each load took ten instructions of a wave that has its SIMD to
      // itself; the first two chunks of a lane always exist).
      uint32_t rid[RIF], off[CPL], mask[CPL];
#pragma unroll
      for (int rr = 0; rr < RIF; rr++) rid[rr] = ids[min(base + rr * G + grp, cnt - 1)];
#pragma unroll
      for (int k = 0; k < CPL; k++) {
        const int ch = sub + k * LPV;
        off[k] = (uint32_t)min(ch, nch - 1) * 16u;
        mask[k] = ch < nch ? ~0u : 0u;
      }
#pragma unroll
      for (int rr = 0; rr < RIF; rr++) {
        if ((rr & ~1) >= steps) break;  // whole pairs, as they are summed below
        const uint32_t id = LPV == 64 ? rdlane(rid[rr], 0) : rid[rr];
        const uint8_t* row = vecs + (size_t)id * stride;
#pragma unroll
        for (int k = 0; k < CPL; k++) b[rr][k] = ld16(row + off[k]);
      }
      typename Acc<KIND>::T t[RIF];
#pragma unroll
      for (int rr = 0; rr < RIF; rr += 2) {  // two rows' chains of sums beside each other
        t[rr] = t[rr + 1] = 0;
        if (rr >= steps) continue;
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
          for (int k = 2; k < CPL; k++) {
            b[rr + h][k].x &= mask[k];
            b[rr + h][k].y &= mask[k];
            b[rr + h][k].z &= mask[k];
            b[rr + h][k].w &= mask[k];
          }
        partial2<KIND, LPV, CPL>(s, b[rr], b[rr + 1], t[rr], t[rr + 1]);
      }
      const typename Acc<KIND>::T v = fold_sum<RIF, LPV>(t);
      const int c = base + fold_index<RIF, LPV>() * G + grp;
      if (ln % (LPV / RIF) == 0 && c < cnt) out[c] = dist(v, c);
    } else {
#pragma unroll
      for (int rr = 0; rr < RIF; rr++) {
        if (rr >= steps) break;
        const int c = base + rr * G + grp;
        const uint8_t* row = vecs + (size_t)(c < cnt ? ids[c] : 0u) * stride;
#pragma unroll
        for (int k = 0; k < CPL; k++) {
          const int ch = sub + k * LPV;
          b[rr][k] = (rr < steps && c < cnt && ch < nch) ? ld16(row + (size_t)ch * 16) : make_uint4(0, 0, 0, 0);
        }
      }
#pragma unroll
      for (int rr = 0; rr < RIF; rr++) {
        if (rr >= steps) break;
        const int c = base + rr * G + grp;
        typename Acc<KIND>::T t = group_sum<LPV>(partial<KIND, LPV, CPL>(s, b[rr]));
        if (sub == 0 && c < cnt) out[c] = dist(t, c);
      }
    }
  }
}

// Distance from the slice to a single row, returned in every lane.
template <int KIND, int LPV, int CPL>
__device__ __forceinline__ float wave_dist1(const Slice<KIND, LPV, CPL>& s, const uint8_t* row, int nch) {
  const int sub = lane() % LPV;
  uint4 b[CPL];
#pragma unroll
  for (int k = 0; k < CPL; k++) {
    const int ch = sub + k * LPV;
    b[k] = ch < nch ? ld16(row + (size_t)ch * 16) : make_uint4(0, 0, 0, 0);
  }
  typename Acc<KIND>::T t = group_sum<LPV>(partial<KIND, LPV, CPL>(s, b));
  return __shfl(finalize<KIND>(t), 0, 64);
}

}  // namespace gr
