// Products of degree 1024..4096 through a polynomial transform (H. J. Nussbaumer, "Fast
// polynomial transform algorithms for digital convolution", IEEE Trans. ASSP 28, 1980),
// the matrix products of Eq. (3) running on its 2k pieces.
//
// Write n = k M with M = 256 and y = x^k.  A polynomial a = sum_{i<k} x^i A_i(y), A_i[j] =
// a[i + k j], has its coefficients in R = Z_q[y]/(y^M + 1), where w = y^(M/k) is a 2k-th
// root of one with w^k = -1: multiplying by a power of w is a signed rotation, no roots in
// Z_q are needed and any odd q will do.  So
//   A^_s = sum_i w^(i s) A_i,   C^_s = A^_s B^_s in R,   P_i = (1/2k) sum_s w^(-i s) C^_s,
//   c = sum_{i<k} x^i (P_i + y P_(i+k))                  (s < 2k; x^k = y folds the top half)
// and one product of degree bound n is 2k negacyclic products of degree bound M: 2k M^2 =
// 2 n M multiply-adds on the matrix units for n^2 (an eighth at n = 4096), and 3 log2(2k)
// additions mod q per coefficient.  With P_i and P_(i+k) the sum and difference of the
// even and odd points' halves, the fold is (1 + y) E_i + w^(-i) (1 - y) O_i: the factors
// 1 +- y are applied to C^_s, where a neighbouring column is at hand.
//
// A workgroup (four waves) takes G = 16 / k products.  A thread owns one column j = ylow +
// 16 yhigh of them, yhigh = lane % 16, ylow = 4 wave + lane / 16, and holds the 32 points
// of both operands in registers: w^e moves yhigh only, so a rotation is a DPP row rotation
// that the butterfly's addition takes as its operand, and the sign is a select on constant
// lane masks.  The 32 sub-products then pass through LDS eight at a time: four points of
// the four threads of a column group are transposed (v_permlane{32,16}_swap) so that each
// thread packs four consecutive coefficients of one point, their digit planes (layout of
// the 16x16-tile kernel: t = 16, r = 16, K = 256) are multiplied by v_mfma_i32_16x16x64_i8,
// two sub-products per wave, and the results return to their columns as words.
//
// Recombination of a sub-product is one Montgomery step: x = lift + sum_s T_s rc_s with
// rc_s = 2^(8s) 2^32 / (2k) mod q, centred.  |T_s| <= P_s M 2^14 and sum_s P_s = L^2, so
// |sum| <= lift = q L^2 M 2^13 <= q 2^25, x is below q 2^32 and hi(x) - hi(m q) lies in
// (-q, q).
//
// Measured against the 32x32-tile kernel on whole products, us per call: n = 4096, 2048
// products 364 -> 92 and 8 products 38.8 -> 18.0; n = 1024, 4095 products 55.5 -> 42.4
// (30-bit moduli).  That kernel was bound by the power its matrix units draw; here they do
// an eighth (n = 4096) or half (n = 1024) of the work and the vector units' additions,
// digit splits and recombinations weigh as much.
//
// 64-bit words (one modulus, 4, 6 or 8 limbs): the same with 64-bit additions and a 64-bit
// Montgomery step, two waves per SIMD.  Sixteen products of n = 65536 with q = 2^64 - 2^32
// + 1, through the outer transform below: 3.03 ms on the streaming kernel, 1.41 ms through
// three Karatsuba levels, 113 us here.
#pragma once
#include "pm_mfma16.h"
#include "pm_stream.h"

namespace pm {

constexpr int kPtM = 256;             // degree bound of the sub-products
constexpr int kPtPoints = 32;         // sub-products per workgroup
constexpr int kPtBatch = 8;           // of them in LDS at a time
constexpr uint32_t kPtAPlane = 272;   // reversed ext positions 0 .. 271: 255 .. -16
constexpr uint32_t kPtBPlane = 31 * 16;  // rows -15 .. 15
constexpr uint32_t kPtRow = 80;       // words between the four result rows of a sub-product
constexpr uint32_t kPtSubWords = 4 * kPtRow;
template <int L>
constexpr uint32_t pt_sub_bytes() { return (uint32_t)L * (kPtAPlane + kPtBPlane); }
template <typename W, int L>
constexpr uint32_t pt_lds_bytes() { return kPtBatch * (pt_sub_bytes<L>() + kPtSubWords * (uint32_t)sizeof(W)); }

struct PtMod32 {
  ModQ32 m;
  uint32_t qinv;   // q^-1 mod 2^32
  uint64_t lift;   // q L^2 M 2^13
  int32_t rc[8];   // 2^(8s) 2^32 / (2k) mod q, centred, s < 2L - 1
};
struct PtMod64 {
  ModQ64 m;
  uint64_t qinv;          // q^-1 mod 2^64
  int64_t lift0, lift1;   // lift0 + 2^32 lift1 = q 2^28
  int32_t w0[15], w1[15]; // w0 + 2^32 w1 = 2^(8s) 2^64 / (2k) mod q
};
template <typename W> struct PtModOf { typedef PtMod32 Mod; static constexpr int kMods = kMaxQ; };
template <> struct PtModOf<uint64_t> { typedef PtMod64 Mod; static constexpr int kMods = 1; };

template <typename W>
struct PtParams {
  const W* a;
  const W* b;
  W* c;
  uint64_t nprod;
  uint32_t n;
  uint32_t lc, nq_total, l0, lrep;  // products and moduli as in Mfma32Params
  uint32_t b_shared;
  typename PtModOf<W>::Mod mods[PtModOf<W>::kMods];
};

__host__ __device__ constexpr int pt_bitrev(int x, int bits) {
  int r = 0;
  for (int i = 0; i < bits; ++i) r |= ((x >> i) & 1) << (bits - 1 - i);
  return r;
}

// Lane yhigh takes the value of lane yhigh - R (mod 16).
template <int R>
__device__ __forceinline__ uint32_t pt_rot(uint32_t v) {
  if constexpr ((R & 15) == 0) return v;
  else return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x120 + (R & 15), 0xf, 0xf, true);
}
template <int R>
__device__ __forceinline__ uint64_t pt_rot(uint64_t v) {
  return ((uint64_t)pt_rot<R>((uint32_t)(v >> 32)) << 32) | pt_rot<R>((uint32_t)v);
}
// y^(16 R) v, R in (-16, 16): the lanes that pass y^M = -1 are negated, then the row rotates.
template <int R, typename W>
__device__ __forceinline__ W pt_shift(W v, W q, uint32_t yhigh) {
  if constexpr (R != 0) {
    const bool wraps = R > 0 ? (int)yhigh >= 16 - R : (int)yhigh < -R;
    v = wraps ? q - v : v;
  }
  return pt_rot<R>(v);
}

// Sum and difference mod q of x, y in [0, q], again in [0, q] (q stands for 0 too);
// 32-bit words: q < 2^31.
__device__ __forceinline__ uint32_t pt_add(uint32_t x, uint32_t y, uint32_t q) {
  const uint32_t s = x + y;
  return min_u32(s, s - q);
}
__device__ __forceinline__ uint32_t pt_sub(uint32_t x, uint32_t y, uint32_t q) {
  const uint32_t d = x - y;
  return min_u32(d, d + q);
}
__device__ __forceinline__ uint64_t pt_add(uint64_t x, uint64_t y, uint64_t q) {
  uint64_t s, t;
  const bool carry = __builtin_add_overflow(x, y, &s);
  const bool below = __builtin_sub_overflow(s, q, &t);
  return carry || !below ? t : s;
}
__device__ __forceinline__ uint64_t pt_sub(uint64_t x, uint64_t y, uint64_t q) {
  uint64_t d;
  const bool below = __builtin_sub_overflow(x, y, &d);
  return below ? d + q : d;
}
// +-(x + y) mod q in [0, q), x, y in [0, q].
template <bool NEG>
__device__ __forceinline__ uint32_t pt_close(uint32_t x, uint32_t y, uint32_t q) {
  const uint32_t u = x + y;
  return NEG ? min_u32(min_u32(0u - u, q - u), 2 * q - u) : min_u32(min_u32(u, u - q), u - 2 * q);
}
template <bool NEG>
__device__ __forceinline__ uint64_t pt_close(uint64_t x, uint64_t y, uint64_t q) {
  const uint64_t s = pt_add(x, y, q);
  const uint64_t r = NEG ? q - s : s;
  return r == q ? 0 : r;
}

// (x, z) <- (x + Y z, Y z - x), Y = y^(16 R).  The difference is taken this way round
// because the rotated operand of an addition or subtraction has to be its first one
// (v_subrev_u32 with a DPP row rotation was measured to rotate the other operand).
template <int R, typename W>
__device__ __forceinline__ void pt_butterfly(W& x, W& z, W q, uint32_t yhigh) {
  const W t = pt_shift<R>(z, q, yhigh);
  z = pt_sub(t, x, q);
  x = pt_add(t, x, q);
}

// Decimation-in-time stages of block size S .. N over v[0 .. N) (bit-reversed order in,
// natural order out); the S-point root of one is y^(16 (32 / S)), DIR -1: its inverse.
// Output i carries the sign (-1)^(bits set in i): the two inputs of a butterfly have the
// same index within their blocks, hence the same sign, and each upper half flips it.  In the
// forward transform the signs of a and b cancel in the products; the inverse's last step
// takes them out.
template <int S, int J, int DIR, int N, typename W>
__device__ __forceinline__ void pt_stage(W* v, W q, uint32_t yhigh) {
  if constexpr (J < S / 2) {
#pragma unroll
    for (int b = 0; b < N; b += S) pt_butterfly<DIR * J * (32 / S)>(v[b + J], v[b + J + S / 2], q, yhigh);
    pt_stage<S, J + 1, DIR, N>(v, q, yhigh);
  }
}
template <int S, int DIR, int N, typename W>
__device__ __forceinline__ void pt_stages(W* v, W q, uint32_t yhigh) {
  if constexpr (S <= N) {
    pt_stage<S, 0, DIR, N>(v, q, yhigh);
    pt_stages<2 * S, DIR, N>(v, q, yhigh);
  }
}

// K input words mod q.  64-bit words are nearly always below q: one test for all of them.
template <int K>
__device__ __forceinline__ void pt_reduce(uint32_t* x, const ModQ32& m) {
#pragma unroll
  for (int i = 0; i < K; ++i) x[i] = reduce_u32(x[i], m);
}
template <int K>
__device__ __forceinline__ void pt_reduce(uint64_t* x, const ModQ64& m) {
  bool over = false;
#pragma unroll
  for (int i = 0; i < K; ++i) over |= x[i] >= m.q;
  if (over) {
#pragma unroll 1
    for (int i = 0; i < K; ++i) {
      uint64_t v = x[0];
#pragma unroll
      for (int k = 1; k < K; ++k) v = i == k ? x[k] : v;  // no dynamic index into registers
      v = mod_u64(v, m);
#pragma unroll
      for (int k = 0; k < K; ++k) x[k] = i == k ? v : x[k];
    }
  }
}

// The 2K points of one operand from its K words: the upper half of the transform's input is
// zero, so its first stage only copies.
template <int LK, typename W, typename M>
__device__ __forceinline__ void pt_forward(W* x, W* v, const M& m, uint32_t yhigh) {
  constexpr int K = 1 << LK;
  pt_reduce<K>(x, m);
#pragma unroll
  for (int p = 0; p < K; ++p) v[2 * p] = v[2 * p + 1] = x[pt_bitrev(p, LK)];
  pt_stages<4, 1, 2 * K>(v, (W)m.q, yhigh);
}

// c_i = +-(E_i + w^(-i) O_i) from the transformed even and odd points, in [0, q).
template <int LK, int I, typename W>
__device__ __forceinline__ void pt_last(const W* e, const W* o, W* c, W q, uint32_t yhigh) {
  if constexpr (I < (1 << LK)) {
    c[I] = pt_close<(__builtin_popcount(I) & 1) != 0>(pt_shift<-I * (16 >> LK)>(o[I], q, yhigh), e[I], q);
    pt_last<LK, I + 1>(e, o, c, q, yhigh);
  }
}

// Transpose the 4x4 block (register, row of 16 lanes): afterwards w[i] of row r holds what
// w[r] of row i held.
__device__ __forceinline__ void pt_transpose(uint32_t (&w)[4]) {
  typedef uint32_t v2 __attribute__((ext_vector_type(2)));
  v2 p = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
  v2 s = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
  v2 x = __builtin_amdgcn_permlane16_swap(p[0], s[0], false, false);
  v2 z = __builtin_amdgcn_permlane16_swap(p[1], s[1], false, false);
  w[0] = x[0]; w[1] = x[1]; w[2] = z[0]; w[3] = z[1];
}
__device__ __forceinline__ void pt_transpose(uint64_t (&w)[4]) {
  uint32_t lo[4], hi[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) { lo[i] = (uint32_t)w[i]; hi[i] = (uint32_t)(w[i] >> 32); }
  pt_transpose(lo);
  pt_transpose(hi);
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = ((uint64_t)hi[i] << 32) | lo[i];
}

// Digit words of x in [0, q] and of -x, and their byte planes.
template <int L>
__device__ __forceinline__ void pt_digits(const uint32_t (&x)[4], const ModQ32& m, uint32_t (&pos)[4], uint32_t (&neg)[4]) {
  digits_pm32<L>(x, m.q, m.thr, pos, neg);
}
template <int L>
__device__ __forceinline__ void pt_digits(const uint64_t (&x)[4], const ModQ64& m, uint64_t (&pos)[4], uint64_t (&neg)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    pos[i] = digits64<L>(x[i], m);
    neg[i] = digits64<L>(m.q - x[i], m);
  }
}
template <int L>
__device__ __forceinline__ void pt_store(uint8_t* base, uint32_t plane, uint32_t off, const uint32_t (&w)[4]) {
  transpose_store<L>(base, plane, off, w);
}
template <int L>
__device__ __forceinline__ void pt_store(uint8_t* base, uint32_t plane, uint32_t off, const uint64_t (&w)[4]) {
  transpose_store64<L>(base, plane, off, w);
}

// Four points of the column group's four columns into the digit planes of sub-product
// `sub` (this row's): the reversed ext of a, or the rows of b.
template <int L, bool IS_B, typename W, typename M>
__device__ __forceinline__ void pt_stage_planes(const W* v, uint8_t* sub, const M& m, uint32_t wave, uint32_t yhigh) {
  W w[4] = {v[0], v[1], v[2], v[3]};
  pt_transpose(w);
  W pos[4], neg[4];
  if constexpr (IS_B) {
    pt_digits<L>(w, m, pos, neg);
    uint8_t* rows = sub + L * kPtAPlane + 4 * wave;
    pt_store<L>(rows, kPtBPlane, (yhigh + 15) * 16, pos);
    if (yhigh > 0) pt_store<L>(rows, kPtBPlane, (yhigh - 1) * 16, neg);
  } else {
    const W rev[4] = {w[3], w[2], w[1], w[0]};
    pt_digits<L>(rev, m, pos, neg);
    const uint32_t off = 252 - 4 * wave - 16 * yhigh;
    pt_store<L>(sub, kPtAPlane, off, pos);
    if (yhigh == 15) pt_store<L>(sub, kPtAPlane, off + 256, neg);
  }
}

// K-step of a sub-product with more than four limbs: the B rows of all limbs are held, the
// A runs are taken limb by limb.
template <int L>
__device__ __forceinline__ void pt_step_wide(v4i_acc (&acc)[2 * L - 1], const uint8_t* aplane, int S,
                                             const uint8_t* bplane, int boff) {
  v4i b[L];
#pragma unroll
  for (int j = 0; j < L; ++j) b[j] = *(const v4i*)(bplane + j * kPtBPlane + boff);
  const uint32_t sh = (uint32_t)(S & 3);
  uint32_t x[2][5];
  load_run(x[0], aplane, S);
#pragma unroll
  for (int i = 0; i < L; ++i) {
    if (i + 1 < L) load_run(x[(i + 1) & 1], aplane + (i + 1) * kPtAPlane, S);
    const v4i a = align_run(x[i & 1], sh);
#pragma unroll
    for (int j = 0; j < L; ++j) acc[i + j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b[j], acc[i + j], 0, 0, 0);
  }
}

// Word e of a lane's results (canonical, scaled by 1/2k).
template <int L>
__device__ __forceinline__ uint32_t pt_recombine(const v4i_acc (&acc)[2 * L - 1], int e, const PtMod32& pm) {
  uint64_t x = pm.lift;
#pragma unroll
  for (int s = 0; s < 2 * L - 1; ++s) x += (uint64_t)((int64_t)acc[s][e] * (int64_t)pm.rc[s]);
  const uint32_t t = (uint32_t)(x >> 32) - mul_hi32((uint32_t)x * pm.qinv, pm.m.q);
  return min_u32(t, t + pm.m.q);
}
// x = lift + sum_s T_s (w0_s + 2^32 w1_s): |sum_s T_s w_s| < L^2 M 2^14 2^31 < 2^60 for
// either half, lift makes x non-negative and below q 2^29, so after the Montgomery step
// hi(x) - hi(m q) is in (-q, q).
template <int L>
__device__ __forceinline__ uint64_t pt_recombine(const v4i_acc (&acc)[2 * L - 1], int e, const PtMod64& pm) {
  int64_t x0 = pm.lift0, x1 = pm.lift1;
#pragma unroll
  for (int s = 0; s < 2 * L - 1; ++s) {
    x0 += (int64_t)acc[s][e] * (int64_t)pm.w0[s];
    x1 += (int64_t)acc[s][e] * (int64_t)pm.w1[s];
  }
  x1 += x0 >> 32;
  const uint64_t lo = ((uint64_t)x1 << 32) | (uint32_t)x0;
  return pt_sub((uint64_t)(x1 >> 32), mulhi64(lo * pm.qinv, pm.m.q), pm.m.q);
}

// One sub-product from its planes to its words: lane (u, g) leaves coefficients 16 u + 4 g + e
// in row e of res.  -c[255] goes to slot 64 of row 3, where column 0 finds y c.
template <int L, typename W, typename PM>
__device__ __forceinline__ void pt_multiply(const uint8_t* sub, W* res, const PM& pm, uint32_t lane) {
  const int zl = (int)(lane & 15), g = (int)(lane >> 4);
  const int S0 = 255 - 16 * g - zl;
  const int B0 = (zl + 15 - g) * 16;
  const uint8_t* bp = sub + L * kPtAPlane;
  v4i_acc acc[2 * L - 1];
#pragma unroll
  for (int s = 0; s < 2 * L - 1; ++s) acc[s] = v4i_acc{0, 0, 0, 0};
#pragma unroll
  for (int st = 0; st < kPtM / 64; ++st) {
    if constexpr (L <= 4) mfma16_step<L>(acc, sub, kPtAPlane, S0 - 64 * st, bp, kPtBPlane, B0 - 64 * st);
    else pt_step_wide<L>(acc, sub, S0 - 64 * st, bp, B0 - 64 * st);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const W r = pt_recombine<L>(acc, e, pm);
    res[e * kPtRow + lane] = r;
    if (e == 3 && lane == 63) res[3 * kPtRow + 64] = (W)pm.m.q - r;
  }
}

// K consecutive words (K words or 16 bytes at a time, whichever is less).
template <int K, typename W>
struct PtVec {
  static constexpr int kN = K * sizeof(W) < 16 ? K : 16 / (int)sizeof(W);
  typedef W vec __attribute__((ext_vector_type(kN)));
};
template <int K, typename W>
__device__ __forceinline__ void pt_load(const W* p, W* x) {
  typedef PtVec<K, W> V;
#pragma unroll
  for (int i = 0; i < K; i += V::kN) {
    const typename V::vec v = *(const typename V::vec*)(p + i);
#pragma unroll
    for (int k = 0; k < V::kN; ++k) x[i + k] = v[k];
  }
}
template <int K, typename W>
__device__ __forceinline__ void pt_put(W* p, const W* x) {
  typedef PtVec<K, W> V;
#pragma unroll
  for (int i = 0; i < K; i += V::kN) {
    typename V::vec v;
#pragma unroll
    for (int k = 0; k < V::kN; ++k) v[k] = x[i + k];
    *(typename V::vec*)(p + i) = v;
  }
}

template <typename W, int L, int LK>
__device__ __forceinline__ void pt_group(const PtParams<W>& P, uint64_t grp, uint8_t* smem) {
  constexpr int K = 1 << LK, G = 16 >> LK, PTS = 2 * K;
  const uint32_t lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const uint32_t yhigh = lane & 15, row = lane >> 4, ylow = 4 * wave + row;
  const uint32_t j = ylow + 16 * yhigh;

  uint64_t off[G], boff[G];
  uint32_t li[G];
  W va[kPtPoints], vb[kPtPoints];
  {
    W xa[16], xb[16];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint64_t p = grp * G + g;
      const uint64_t gp = global_product(P, p < P.nprod ? p : P.nprod - 1, &li[g]);
      off[g] = wave_uniform(gp * P.n);
      boff[g] = wave_uniform(b_product(P, gp, li[g]) * P.n);
      li[g] = wave_uniform(li[g]);
      pt_load<K>(P.a + off[g] + (size_t)K * j, xa + g * K);
      pt_load<K>(P.b + boff[g] + (size_t)K * j, xb + g * K);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      pt_forward<LK>(xa + g * K, va + g * PTS, P.mods[li[g]].m, yhigh);
      pt_forward<LK>(xb + g * K, vb + g * PTS, P.mods[li[g]].m, yhigh);
    }
  }

  W* results = (W*)(smem + kPtBatch * pt_sub_bytes<L>());
  // column j of a sub-product's results, and column j - 1 (times y: -c[255] at j = 0)
  const uint32_t cur = row * kPtRow + 16 * wave + yhigh;
  const uint32_t prev = row > 0 ? cur - kPtRow
                        : wave > 0 ? 3 * kPtRow + 16 * (wave - 1) + yhigh
                        : yhigh > 0 ? 3 * kPtRow + 48 + yhigh - 1 : 3 * kPtRow + 64;
  W ch[kPtPoints];  // C^_s (1 +- y) at column j, the even points of a product first
#pragma unroll
  for (int ph = 0; ph < kPtPoints / kPtBatch; ++ph) {
    const int g = ph * kPtBatch / PTS;  // the batch's product
    const auto& pm = P.mods[li[g]];
#pragma unroll
    for (int h = 0; h < kPtBatch; h += 4) {
      uint8_t* sub = smem + (h + row) * pt_sub_bytes<L>();
      pt_stage_planes<L, false>(va + ph * kPtBatch + h, sub, pm.m, wave, yhigh);
      pt_stage_planes<L, true>(vb + ph * kPtBatch + h, sub, pm.m, wave, yhigh);
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t s = 2 * wave; s < 2 * wave + 2; ++s)
      pt_multiply<L>(smem + s * pt_sub_bytes<L>(), results + s * kPtSubWords, pm, lane);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kPtBatch; ++s) {
      const W x = results[s * kPtSubWords + cur], y = results[s * kPtSubWords + prev];
      const int pt = (ph * kPtBatch + s) % PTS;
      // decimation in time wants the points of each half in bit-reversed order
      const int to = g * PTS + (pt & 1) * K + pt_bitrev(pt >> 1, LK);
      ch[to] = pt & 1 ? pt_sub(x, y, (W)pm.m.q) : pt_add(x, y, (W)pm.m.q);
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const W q = (W)P.mods[li[g]].m.q;
    W* e = ch + g * PTS;
    W c[K];
    pt_stages<2, -1, K>(e, q, yhigh);
    pt_stages<2, -1, K>(e + K, q, yhigh);
    pt_last<LK, 0>(e, e + K, c, q, yhigh);
    if (grp * G + g < P.nprod) pt_put<K>(P.c + off[g] + (size_t)K * j, c);
  }
}

// 32-bit words: three waves per SIMD fit the registers (64 point words per thread); 64-bit
// words: two.
template <typename W, int L, int LK>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(sizeof(W) == 4 ? 3 : 2, sizeof(W) == 4 ? 3 : 2)))
void ptrans_kernel(const PtParams<W> P) {
  extern __shared__ __align__(16) uint8_t smem[];
  pt_group<W, L, LK>(P, blockIdx.x, smem);
}

// ---------------------------------------------------------------------------
// Larger degrees: the same transform once more around it, its points held in a workspace.
// n = k M with M = 4096, k = 2 .. 16: a forward kernel writes the 2k points of a and b as
// polynomials of degree 4096, the kernel above multiplies them (over a's points), an
// inverse kernel puts the products together.  The work on the matrix units stays 2 n 512
// multiply-adds whatever n is.  The forward and inverse kernels move 3 n and 5 n words per operand
// and product (the inverse reads columns j and j - 1, the second from cache) and are bound
// by memory; sixteen columns 256 apart share a row of lanes, so the rotations are again
// row rotations.
// ---------------------------------------------------------------------------
constexpr int kPtOuterM = 4096;

template <typename W> struct PtBase { typedef ModQ32 Mod; };
template <> struct PtBase<uint64_t> { typedef ModQ64 Mod; };

template <typename W>
struct PtOuter {
  const W* a;
  const W* b;
  W* c;
  W* sa;  // [nprod][2k][4096] points of a, then the products of the points
  W* sb;  // points of b
  uint32_t L;  // product p uses mods[p % L]
  typename PtBase<W>::Mod mods[PtModOf<W>::kMods];
};

// Block: product blockIdx.x / 16, 16 columns ylow of it (and their 16 yhigh each);
// blockIdx.y: operand.
template <typename W, int LK>
__global__ __launch_bounds__(256) void pt_outer_forward_kernel(const PtOuter<W> P) {
  constexpr int K = 1 << LK;
  const uint64_t p = blockIdx.x >> 4;
  const uint32_t yhigh = threadIdx.x & 15, j = ((blockIdx.x & 15) << 4) + (threadIdx.x >> 4) + 256 * yhigh;
  const auto& m = P.mods[p % P.L];
  W x[K], v[2 * K];
  pt_load<K>((blockIdx.y ? P.b : P.a) + (p * kPtOuterM + j) * K, x);
  pt_forward<LK>(x, v, m, yhigh);
  W* out = (blockIdx.y ? P.sb : P.sa) + p * 2 * K * kPtOuterM + j;
#pragma unroll
  for (int s = 0; s < 2 * K; ++s) out[s * kPtOuterM] = v[s];
}

template <typename W, int LK>
__global__ __launch_bounds__(256) void pt_outer_inverse_kernel(const PtOuter<W> P) {
  constexpr int K = 1 << LK;
  const uint64_t p = blockIdx.x >> 4;
  const uint32_t yhigh = threadIdx.x & 15, j = ((blockIdx.x & 15) << 4) + (threadIdx.x >> 4) + 256 * yhigh;
  const W q = (W)P.mods[p % P.L].q;
  const W* in = P.sa + p * 2 * K * kPtOuterM;
  const uint32_t prev = j ? j - 1 : kPtOuterM - 1;
  W ch[2 * K], c[K];
#pragma unroll
  for (int s = 0; s < 2 * K; ++s) {
    const W x = in[s * kPtOuterM + j], y0 = in[s * kPtOuterM + prev];
    const W y = j ? y0 : q - y0;
    ch[(s & 1) * K + pt_bitrev(s >> 1, LK)] = s & 1 ? pt_sub(x, y, q) : pt_add(x, y, q);
  }
  pt_stages<2, -1, K>(ch, q, yhigh);
  pt_stages<2, -1, K>(ch + K, q, yhigh);
  pt_last<LK, 0>(ch, ch + K, c, q, yhigh);
  pt_put<K>(P.c + (p * kPtOuterM + j) * K, c);
}

}  // namespace pm
