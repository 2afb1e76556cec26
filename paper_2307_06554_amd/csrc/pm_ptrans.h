// Products of degree 1024..8192 through a polynomial transform (H. J. Nussbaumer, "Fast
// polynomial transform algorithms for digital convolution", IEEE Trans. ASSP 28, 1980),
// the matrix products of Eq. (3) running on its 2k pieces.
//
// Write n = k M with M = 256 (512 at n = 8192) and y = x^k.  A polynomial a = sum_{i<k} x^i
// A_i(y), A_i[j] = a[i + k j], has its coefficients in R = Z_q[y]/(y^M + 1), where w = y^(M/k)
// is a 2k-th root of one with w^k = -1: multiplying by a power of w is a signed rotation, no
// roots in Z_q are needed and any odd q will do.  So
//   A^_s = sum_i w^(i s) A_i,   C^_s = A^_s B^_s in R,   P_i = (1/2k) sum_s w^(-i s) C^_s,
//   c = sum_{i<k} x^i (P_i + y P_(i+k))                  (s < 2k; x^k = y folds the top half)
// and one product of degree bound n is 2k negacyclic products of degree bound M: 2k M^2 =
// 2 n M multiply-adds on the matrix units for n^2 (an eighth at n = 4096 and 8192), and
// 3 log2(2k) additions mod q per coefficient.  With P_i and P_(i+k) the sum and difference of
// the even and odd points' halves, the fold is (1 + y) E_i + w^(-i) (1 - y) O_i: the factors
// 1 +- y are applied to C^_s, where a neighbouring column is at hand.
//
// A workgroup takes G = 16 / k products.  A thread holds 32 points of one column j = ylow +
// (M / 16) yhigh, yhigh = lane % 16: w^e moves yhigh only, so a rotation is a DPP row rotation
// that the butterfly's addition takes as its operand, and the sign is a select on constant lane
// masks.  The 32 sub-products then pass through LDS eight at a time: four points of four
// neighbouring columns are transposed (v_permlane{32,16}_swap) so that each thread packs four
// consecutive coefficients of one point, their digit planes (layout of the 16x16-tile kernel:
// t = 16, r = M / 16, K = M) are multiplied by v_mfma_i32_16x16x64_i8, and the results return to
// their columns as words.
//
// Recombination of a sub-product is one Montgomery step: x = lift + sum_s T_s rc_s with
// rc_s = 2^(8s) 2^32 / (2k) mod q, centred.  |T_s| <= P_s M 2^14 and sum_s P_s = L^2, so
// |sum| <= lift = q L^2 M 2^13 <= q 2^26, x is below q 2^32 and hi(x) - hi(m q) lies in
// (-q, q).
//
// Measured against the 32x32-tile kernel on whole products, us per call (30-bit moduli):
// n = 4096, 2048 products 364 -> 82 and 8 products 38.8 -> 14.2; n = 1024, 4095 products 55.5
// -> 41.5; n = 8192, 512 products, 244 through two Karatsuba levels -> 74.  That kernel was bound
// by the power its matrix units draw.  Here the K loops take half of the time (left out, the
// n = 4096 batch takes 42 us of 82): a step of sixteen MFMAs (256 cycles on each SIMD) reads
// 9 KiB, the A runs five dwords a lane at 128 B a cycle, so four SIMDs' steps keep the LDS busy
// for nearly as long as the matrix units; the rest is the vector units' additions, digit splits
// and recombinations, which overlap with the other waves' products.
//
// 64-bit words (one modulus, 4, 6 or 8 limbs): the same with 64-bit additions and a 64-bit
// Montgomery step.  Sixteen products of n = 65536 with q = 2^64 - 2^32 + 1, through the outer
// transform below: 3.03 ms on the streaming kernel, 1.41 ms through three Karatsuba levels,
// 106 us here.
#pragma once
#include "pm_mfma16.h"
#include "pm_stream.h"

namespace pm {

constexpr int kPtPoints = 32;         // sub-products per workgroup
constexpr int kPtBatch = 8;           // of them in LDS at a time
constexpr uint32_t kPtRow = 80;       // words between the four result rows of a column group

// Sub-products of degree bound M = 256 C: a thread owns C columns.
template <int C>
struct PtGeom {
  static constexpr int kM = 256 * C, kR = 16 * C;             // M = 16 R
  static constexpr uint32_t kAPlane = kM + 16;                // reversed ext positions: M - 1 .. -16
  static constexpr uint32_t kBPlane = (2 * kR - 1) * 16;      // rows -(R - 1) .. R - 1
  static constexpr uint32_t kColWords = 4 * kPtRow + (C > 1 ? 16 : 0);  // results of the c-th columns
  static constexpr uint32_t kResWords = C * kColWords;
  // C = 2: the A planes of sub-product s start 4 (s % 4) bytes in.  A wave's store has the sixteen
  // lanes of a row 16 C bytes apart; the shift puts its four rows, one sub-product each, on
  // different banks (n = 8192, 512 products: 77.3 -> 74.1 us; level at C = 1, which goes without).  The B
  // rows are read 16 bytes at a time and stay aligned.
  static constexpr uint32_t kShift = C > 1 ? 4 : 0;
  template <int L> static constexpr uint32_t b_at() { return (uint32_t)L * kAPlane + 4 * kShift; }
  template <int L> static constexpr uint32_t sub_bytes() { return b_at<L>() + (uint32_t)L * kBPlane; }
};
// LDS: the planes of a batch (in the end the words two halves swap), then its results.
template <typename W, int L, int C, int H>
constexpr uint32_t pt_results_at() {
  const uint32_t planes = kPtBatch * PtGeom<C>::template sub_bytes<L>(), swap = H == 1 ? 0 : 16 * 256 * C * (uint32_t)sizeof(W);
  return planes > swap ? planes : swap;
}
template <typename W, int L, int C, int H>
constexpr uint32_t pt_lds_bytes() {
  return pt_results_at<W, L, C, H>() + kPtBatch * PtGeom<C>::kResWords * (uint32_t)sizeof(W);
}

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
  uint32_t kara;  // plans, n = 4096: product p is sub-product p % 3 of one Karatsuba level on product p / 3
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
// 64-bit words by halves, the carry out of the upper one used as it is: on whole words the compiler
// takes a 64-bit comparison more per addition and subtraction (sixteen products of n = 65536
// 107.8 -> 106.1 us).
__device__ __forceinline__ bool pt_carry_add(uint64_t x, uint64_t y, uint64_t* r) {
  unsigned c;
  const uint32_t lo = __builtin_addc((uint32_t)x, (uint32_t)y, 0u, &c);
  const uint32_t hi = __builtin_addc((uint32_t)(x >> 32), (uint32_t)(y >> 32), c, &c);
  *r = ((uint64_t)hi << 32) | lo;
  return c != 0;
}
__device__ __forceinline__ bool pt_borrow_sub(uint64_t x, uint64_t y, uint64_t* r) {
  unsigned c;
  const uint32_t lo = __builtin_subc((uint32_t)x, (uint32_t)y, 0u, &c);
  const uint32_t hi = __builtin_subc((uint32_t)(x >> 32), (uint32_t)(y >> 32), c, &c);
  *r = ((uint64_t)hi << 32) | lo;
  return c != 0;
}
__device__ __forceinline__ uint64_t pt_add(uint64_t x, uint64_t y, uint64_t q) {
  uint64_t s, t;
  const bool carry = pt_carry_add(x, y, &s);
  const bool below = pt_borrow_sub(s, q, &t);
  return carry || !below ? t : s;
}
__device__ __forceinline__ uint64_t pt_sub(uint64_t x, uint64_t y, uint64_t q) {
  uint64_t d;
  const bool below = pt_borrow_sub(x, y, &d);
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
// because a rotated operand must not be what is subtracted: the compiler makes x - rot(z) one
// v_subrev_u32 with the rotation on z, and on the GPU that gave rot(x) - z in all 64 lanes
// (v_subrev_u32_dpp v1, v2, v1 row_ror:3 with x in v1 and z in v2, encoded as it stands there; ROCm 7.2).
// x + rot(z) and rot(z) - x, v_add_u32 and v_sub_u32, were right in all of them.
// tests/test_machine_code.py looks for reversed forms in the built library.
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

// The 2K points of one operand from its K words in [0, q]: the upper half of the transform's
// input is zero, so its first stage only copies.
template <int LK, typename W>
__device__ __forceinline__ void pt_points(const W* x, W* v, W q, uint32_t yhigh) {
  constexpr int K = 1 << LK;
#pragma unroll
  for (int p = 0; p < K; ++p) v[2 * p] = v[2 * p + 1] = x[pt_bitrev(p, LK)];
  pt_stages<4, 1, 2 * K>(v, q, yhigh);
}
template <int LK, typename W, typename M>
__device__ __forceinline__ void pt_forward(W* x, W* v, const M& m, uint32_t yhigh) {
  pt_reduce<(1 << LK)>(x, m);
  pt_points<LK>(x, v, (W)m.q, yhigh);
}

// O_i <- w^(-i) O_i.
template <int LK, int I, typename W>
__device__ __forceinline__ void pt_twist(W* o, W q, uint32_t yhigh) {
  if constexpr (I < (1 << LK)) {
    o[I] = pt_shift<-I * (16 >> LK)>(o[I], q, yhigh);
    pt_twist<LK, I + 1>(o, q, yhigh);
  }
}
// c_i = +-(E_i + w^(-i) O_i), i in [I, END), in [0, q); e, t and c start at i = I.
template <int I, int END, typename W>
__device__ __forceinline__ void pt_last(const W* e, const W* t, W* c, W q) {
  if constexpr (I < END) {
    c[0] = pt_close<(__builtin_popcount(I) & 1) != 0>(t[0], e[0], q);
    pt_last<I + 1, END>(e + 1, t + 1, c + 1, q);
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
  digits_pm32<L>(x, m.q, L == 4 ? 0xFFFFFFFFu : m.thr, pos, neg);  // four limbs: q is within the window
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
// `sub` (this row's; a: past its shift): the reversed ext of a, or the rows of b.  brow: the columns' index / 16;
// cyclic: the sub-product is one of Z_q[y]/(y^M - 1), what wraps keeps its sign.
template <int L, int C, bool IS_B, typename W, typename M>
__device__ __forceinline__ void pt_stage_planes(const W* v, uint8_t* sub, const M& m, uint32_t wave, uint32_t brow,
                                                bool cyclic = false) {
  typedef PtGeom<C> G;
  W w[4] = {v[0], v[1], v[2], v[3]};
  pt_transpose(w);
  W pos[4], neg[4];
  if constexpr (IS_B) {
    pt_digits<L>(w, m, pos, neg);
    if (cyclic) {
#pragma unroll
      for (int i = 0; i < 4; ++i) neg[i] = pos[i];
    }
    uint8_t* rows = sub + G::template b_at<L>() + 4 * wave;
    pt_store<L>(rows, G::kBPlane, (brow + G::kR - 1) * 16, pos);
    if (brow > 0) pt_store<L>(rows, G::kBPlane, (brow - 1) * 16, neg);
  } else {
    const W rev[4] = {w[3], w[2], w[1], w[0]};
    pt_digits<L>(rev, m, pos, neg);
    if (cyclic) {
#pragma unroll
      for (int i = 0; i < 4; ++i) neg[i] = pos[i];
    }
    const uint32_t off = G::kM - 4 - 4 * wave - 16 * brow;
    pt_store<L>(sub, G::kAPlane, off, pos);
    if (brow == G::kR - 1) pt_store<L>(sub, G::kAPlane, off + G::kM, neg);
  }
}

// K-step of a sub-product with more than four limbs: the B rows of all limbs are held, the
// A runs are taken limb by limb.
template <int L>
__device__ __forceinline__ void pt_step_wide(v4i_acc (&acc)[2 * L - 1], const uint8_t* aplane, uint32_t a_plane, int S,
                                             const uint8_t* bplane, uint32_t b_plane, int boff) {
  v4i b[L];
#pragma unroll
  for (int j = 0; j < L; ++j) b[j] = *(const v4i*)(bplane + j * b_plane + boff);
  const uint32_t sh = (uint32_t)(S & 3);
  uint32_t x[2][5];
  load_run(x[0], aplane, S);
#pragma unroll
  for (int i = 0; i < L; ++i) {
    if (i + 1 < L) load_run(x[(i + 1) & 1], aplane + (i + 1) * a_plane, S);
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

// One 16x16 output tile (columns 16 tile + u) of sub-product s of a batch from its planes to its words:
// lane (u, g) leaves coefficients 16 (16 tile + u) + 4 g + e in row e of the results of columns
// (16 tile + u) % C.  -c[M - 1] goes to slot 64 of the last columns' row 3, where column 0
// finds y c.
template <int L, int C, typename W, typename PM>
__device__ __forceinline__ void pt_multiply(const uint8_t* planes, W* results, uint32_t s, const PM& pm, uint32_t lane, uint32_t tile) {
  typedef PtGeom<C> G;
  const uint8_t* ap = planes + s * G::template sub_bytes<L>() + G::kShift * (s & 3);
  const uint8_t* bp = planes + s * G::template sub_bytes<L>() + G::template b_at<L>();
  W* res = results + s * G::kResWords;
  const int zl = (int)(lane & 15), g = (int)(lane >> 4);
  const int S0 = G::kM - 1 - 16 * g - zl;
  const int B0 = (16 * (int)tile + zl + G::kR - 1 - g) * 16;
  v4i_acc acc[2 * L - 1];
#pragma unroll
  for (int d = 0; d < 2 * L - 1; ++d) acc[d] = v4i_acc{0, 0, 0, 0};
#pragma unroll
  for (int st = 0; st < G::kM / 64; ++st) {
    if constexpr (L <= 4) mfma16_step<L>(acc, ap, G::kAPlane, S0 - 64 * st, bp, G::kBPlane, B0 - 64 * st);
    else pt_step_wide<L>(acc, ap, G::kAPlane, S0 - 64 * st, bp, G::kBPlane, B0 - 64 * st);
  }
  const uint32_t u = 16 * tile + zl;
  W* out = C == 1 ? res + lane : res + (u % C) * G::kColWords + 16 * g + u / C;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const W r = pt_recombine<L>(acc, e, pm);
    out[e * kPtRow] = r;
    if (e == 3 && lane == 63 && tile == C - 1) res[(C - 1) * G::kColWords + 3 * kPtRow + 64] = (W)pm.m.q - r;
  }
}

// Where a thread's column is in a sub-product's results, and the column before it (times y:
// -c[M - 1] before column 0).
template <int C>
__device__ __forceinline__ uint32_t pt_column(uint32_t c, uint32_t w, uint32_t row, uint32_t yhigh) {
  return c * PtGeom<C>::kColWords + row * kPtRow + 16 * w + yhigh;
}
template <int C>
__device__ __forceinline__ uint32_t pt_column_before(uint32_t c, uint32_t w, uint32_t row, uint32_t yhigh) {
  typedef PtGeom<C> G;
  return row > 0 ? pt_column<C>(c, w, row - 1, yhigh)
         : w > 0 ? pt_column<C>(c, w - 1, 3, yhigh)
         : c > 0 ? pt_column<C>(c - 1, 3, 3, yhigh)
                 : (C - 1) * G::kColWords + 3 * kPtRow + (yhigh > 0 ? 48 + yhigh - 1 : 64);
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

// Sub-operand d of one Karatsuba level (pm_karatsuba.h): the even words, the odd ones or their sums.
template <int K>
__device__ __forceinline__ void pt_load_kara(const uint32_t* p, uint32_t d, const ModQ32& m, uint32_t* x) {
#pragma unroll
  for (int i = 0; i < K; i += 2) {
    uint32_t t[4];
    pt_load<4>(p + 2 * i, t);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint32_t e = reduce_u32(t[2 * k], m), o = reduce_u32(t[2 * k + 1], m);
      x[i + k] = d == 0 ? e : d == 1 ? o : pt_add(e, o, m.q);
    }
  }
}

// One workgroup of 4 C H waves: G = 16 / K products of degree bound K 256 C.  Wave: half, c, w
// (w the lowest two bits); a thread owns column 16 c + 4 w + row of the rows of 16 C.  H = 1: it
// holds both operands' points.  H = 2: half 0 transforms a and, in the end, the even points,
// half 1 b and the odd ones; the two swap half of what they have for the last step.
template <typename W, int L, int LK, int C, int H>
__device__ __forceinline__ void pt_group(const PtParams<W>& P, uint64_t grp, uint8_t* smem) {
  typedef PtGeom<C> Geo;
  constexpr int K = 1 << LK, G = 16 >> LK, PTS = 2 * K, OPS = 3 - H;
  constexpr uint32_t kSub = Geo::template sub_bytes<L>();
  const uint32_t lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const uint32_t w = wave & 3, c = (wave >> 2) & (C - 1), half = wave / (4 * C);
  const uint32_t yhigh = lane & 15, row = lane >> 4;
  const uint32_t j = 16 * c + 4 * w + row + Geo::kR * yhigh;

  uint64_t off[G];
  uint32_t li[G];
  W v[OPS][kPtPoints];
  {
    W x[OPS][16];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint64_t p = grp * G + g;
      const uint64_t gp = global_product(P, p < P.nprod ? p : P.nprod - 1, &li[g]);
      off[g] = wave_uniform(gp * P.n);
      const uint64_t boff = wave_uniform(b_product(P, gp, li[g]) * P.n);
      li[g] = wave_uniform(li[g]);
      if constexpr (H == 1 && G == 1 && sizeof(W) == 4) {
        if (P.kara) {
          const uint64_t first = wave_uniform(gp / 3 * 2 * P.n);
          const uint32_t d = wave_uniform((uint32_t)(gp % 3));
          pt_load_kara<K>(P.a + first + (size_t)2 * K * j, d, P.mods[0].m, x[0]);
          pt_load_kara<K>(P.b + first + (size_t)2 * K * j, d, P.mods[0].m, x[OPS - 1]);
          continue;
        }
      }
      if constexpr (H == 1) {
        pt_load<K>(P.a + off[g] + (size_t)K * j, x[0] + g * K);
        pt_load<K>(P.b + boff + (size_t)K * j, x[OPS - 1] + g * K);
      } else {
        pt_load<K>((half ? P.b + boff : P.a + off[g]) + (size_t)K * j, x[0] + g * K);
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int o = 0; o < OPS; ++o) pt_forward<LK>(x[o] + g * K, v[o] + g * PTS, P.mods[li[g]].m, yhigh);
  }

  W* results = (W*)(smem + pt_results_at<W, L, C, H>());
  const uint32_t cur = pt_column<C>(c, w, row, yhigh), prev = pt_column_before<C>(c, w, row, yhigh);
  // C^_s (1 +- y): of a product's points, the even ones first (H = 2: those of this half)
  W ch[kPtPoints / H];
#pragma unroll
  for (int ph = 0; ph < kPtPoints / kPtBatch; ++ph) {
    const int g = ph * kPtBatch / PTS;  // the batch's product
    const auto& pm = P.mods[li[g]];
#pragma unroll
    for (int h = 0; h < kPtBatch; h += 4) {
      uint8_t* sub = smem + (h + row) * kSub;
      if (H == 1 || half == 0)
        pt_stage_planes<L, C, false>(v[0] + ph * kPtBatch + h, sub + Geo::kShift * row, pm.m, w, C * yhigh + c);
      if (H == 1 || half == 1)
        pt_stage_planes<L, C, true>(v[OPS - 1] + ph * kPtBatch + h, sub, pm.m, w, C * yhigh + c);
    }
    __syncthreads();
    constexpr uint32_t kUnits = 2 / H;  // (sub-product, tile) units per wave
#pragma unroll 1
    for (uint32_t i = kUnits * wave; i < kUnits * (wave + 1); ++i)
      pt_multiply<L, C>(smem, results, i / C, pm, lane, i % C);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kPtBatch; s += H) {
      const W* res = results + (s + (H == 1 ? 0 : half)) * Geo::kResWords;
      const int pt = (ph * kPtBatch + s) % PTS;  // H = 2: the even one of the halves' two
      const W x = res[cur], y = res[prev];
      // decimation in time wants the points of each half in bit-reversed order
      const int to = (H == 1 ? g * PTS + (pt & 1) * K : g * K) + pt_bitrev(pt >> 1, LK);
      const W q = (W)pm.m.q;
      if constexpr (H == 1) ch[to] = pt & 1 ? pt_sub(x, y, q) : pt_add(x, y, q);
      else ch[to] = pt_add(x, half ? q - y : y, q);
    }
  }
  if constexpr (H == 1) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const W q = (W)P.mods[li[g]].m.q;
      W* e = ch + g * PTS;
      W o[K];
      pt_stages<2, -1, K>(e, q, yhigh);
      pt_stages<2, -1, K>(e + K, q, yhigh);
      pt_twist<LK, 0>(e + K, q, yhigh);
      pt_last<0, K>(e, e + K, o, q);
      if (grp * G + g < P.nprod) pt_put<K>(P.c + off[g] + (size_t)K * j, o);
    }
  } else {
    // half h keeps the words of i in [h K / 2, (h + 1) K / 2) and hands over the others,
    // through the planes' memory (last read before the last barrier)
    constexpr uint32_t kCols = 256 * C;
    W* give = (W*)smem + half * 8 * kCols + (threadIdx.x & (kCols - 1));
    const W* take = (const W*)smem + (half ^ 1) * 8 * kCols + (threadIdx.x & (kCols - 1));
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const W q = (W)P.mods[li[g]].m.q;
      W* e = ch + g * K;
      pt_stages<2, -1, K>(e, q, yhigh);
      if (half) pt_twist<LK, 0>(e, q, yhigh);
#pragma unroll
      for (int i = 0; i < K / 2; ++i) give[(g * K / 2 + i) * kCols] = half ? e[i] : e[K / 2 + i];
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const W q = (W)P.mods[li[g]].m.q;
      const W* e = ch + g * K;
      W t[K / 2], o[K / 2];
#pragma unroll
      for (int i = 0; i < K / 2; ++i) t[i] = take[(g * K / 2 + i) * kCols];
      if (half) pt_last<K / 2, K>(e + K / 2, t, o, q);
      else pt_last<0, K / 2>(e, t, o, q);
      if (grp * G + g < P.nprod) pt_put<K / 2>(P.c + off[g] + (size_t)K * j + half * (K / 2), o);
    }
  }
}

// Two halves per workgroup.  A thread then holds one operand's 32 points, 32-bit words fit 128
// registers and four waves per SIMD; 64-bit words run at two.  Against one half with both
// operands (three waves per SIMD), us: n = 4096, 8 products 18.0 -> 14.2, 2048 products 83 -> 82;
// n = 16384, 48 products 46.7 -> 43.5 (its outer kernels then as they were); 64-bit n = 4096, one product 50 -> 38, 1024 166 -> 161.
template <typename W, int L, int LK, int C>
__global__ __launch_bounds__(512 * C)
__attribute__((amdgpu_waves_per_eu(sizeof(W) == 4 ? 4 : 2, sizeof(W) == 4 ? 4 : 2)))
void ptrans_kernel(const PtParams<W> P) {
  extern __shared__ __align__(16) uint8_t smem[];
  pt_group<W, L, LK, C, 2>(P, blockIdx.x, smem);
}

// ---------------------------------------------------------------------------
// The ring x^n - 1, n = K M: x^n - 1 = (x^(n/2) + 1)(x^(n/4) + 1) ... (x^M + 1)(x^M - 1).  The
// factor x^(k M) + 1, 2 <= k <= K / 2, goes through the transform above with 2k points, the last
// two are one product of degree M each: 2K - 2 sub-products, in the 2K slots that a product
// of the other ring fills.  With D_k the product in the factor x^(k M) + 1 and D_0 that of
// x^M - 1,
//   c[t] = D_0[t mod M] / K + sum_k +-D_k[t mod k M] k / K, plus where t / M has bit k clear:
// every D_k comes out of its transform scaled by 1/(2k), so 1/(2K) at the recombinations does
// for all of them, D_1 and D_0 taken twice.
// ---------------------------------------------------------------------------
// LDS: both operands' residues (level k at words k M .. 2 k M of a product), or what the halves
// swap and the products D (the same layout).
template <int L, int C>
constexpr uint32_t pt_cyclic_lds() {
  const uint32_t b = pt_lds_bytes<uint32_t, L, C, 2>(), lin = 2 * 16 * 256 * C * 4;
  return b > lin ? b : lin;
}

// Words t + M m of an operand, m < 2k, to its residues (words t + M m, m < k .. 1) in every factor,
// at lin + M k; and back: s[m], m < 2k, from D_0 and the levels up to k.
template <int k, int M>
__device__ __forceinline__ void pt_cyclic_fold(uint32_t* y, uint32_t* lin, uint32_t q) {
  if constexpr (k > 0) {
#pragma unroll
    for (int m = 0; m < k; ++m) {
      lin[(k + m) * M] = pt_sub(y[m], y[m + k], q);
      y[m] = pt_add(y[m], y[m + k], q);
    }
    pt_cyclic_fold<k / 2, M>(y, lin, q);
  } else {
    lin[0] = y[0];
  }
}
template <int k, int M>
__device__ __forceinline__ void pt_cyclic_unfold(uint32_t* s, const uint32_t* d, uint32_t q) {
  if constexpr (k > 0) {
    pt_cyclic_unfold<k / 2, M>(s, d, q);
#pragma unroll
    for (int m = 0; m < k; ++m) {
      const uint32_t x = d[(k + m) * M];
      s[m + k] = pt_sub(s[m], x, q);
      s[m] = pt_add(s[m], x, q);
    }
  } else {
    s[0] = d[0];
  }
}
// Points of the levels k = 2^LK .. 2: 2k slots each, from slot v[0].
template <int LK, int M>
__device__ __forceinline__ void pt_cyclic_points(const uint32_t* lin, uint32_t j, uint32_t* v, uint32_t q, uint32_t yhigh) {
  constexpr int K = 1 << LK;
  if constexpr (LK > 0) {
    uint32_t x[K];
    pt_load<K>(lin + K * M + K * j, x);
    pt_points<LK>(x, v, q, yhigh);
    pt_cyclic_points<LK - 1, M>(lin, j, v + 2 * K, q, yhigh);
  } else {
    v[0] = lin[M + j];  // x^M + 1
    v[1] = lin[j];      // x^M - 1
    v[2] = v[3] = 0;    // no sub-product
  }
}
// Index of even point `pt` within this half's words: the levels one after another, each in
// bit-reversed order.
template <int LK>
__host__ __device__ constexpr int pt_cyclic_to(int pt) {
  if constexpr (LK > 1)
    return pt < (1 << LK) ? pt_bitrev(pt >> 1, LK - 1) : (1 << (LK - 1)) + pt_cyclic_to<LK - 1>(pt - (1 << LK));
  else
    return 0;  // x^M + 1 or x^M - 1
}
// This half's inverse stages of the levels k = 2^LK .. 2: it keeps its words at the start of each
// level's and puts the other half's to `give`.
template <int LK>
__device__ __forceinline__ void pt_cyclic_inverse(uint32_t* e, uint32_t* give, uint32_t cols, uint32_t half, uint32_t q,
                                                  uint32_t yhigh) {
  if constexpr (LK > 0) {
    constexpr int K = 1 << LK;
    pt_stages<2, -1, K>(e, q, yhigh);
    if (half) pt_twist<LK, 0>(e, q, yhigh);
#pragma unroll
    for (int i = 0; i < K / 2; ++i) {
      const uint32_t lo = e[i], hi = e[K / 2 + i];
      give[i * cols] = half ? lo : hi;
      e[i] = half ? hi : lo;
    }
    pt_cyclic_inverse<LK - 1>(e + K, give + K / 2 * cols, cols, half, q, yhigh);
  }
}
template <int LK, int M>
__device__ __forceinline__ void pt_cyclic_last(const uint32_t* e, const uint32_t* take, uint32_t cols, uint32_t* lin, uint32_t j,
                                               uint32_t half, uint32_t q) {
  if constexpr (LK > 0) {
    constexpr int K = 1 << LK;
    uint32_t t[K / 2], o[K / 2];
#pragma unroll
    for (int i = 0; i < K / 2; ++i) t[i] = take[i * cols];
    if (half) pt_last<K / 2, K>(e, t, o, q);
    else pt_last<0, K / 2>(e, t, o, q);
    pt_put<K / 2>(lin + K * M + K * j + half * (K / 2), o);
    pt_cyclic_last<LK - 1, M>(e + K, take + K / 2 * cols, cols, lin, j, half, q);
  }
}

// Workgroup, halves and columns as in pt_group<H = 2>.  The operands are folded, and the levels'
// products put together, with a thread at words t + M m, all m < K: every word of global memory
// is touched once, in whole rows; LDS hands the words over to the columns and back.  Bound as the
// kernel above is.  Against the 32x32-tile kernel, four limbs, us: n = 2048, 1000 products 52.0 ->
// 24.0, one 21.4 -> 13.7; n = 4096, 1024 products 188 -> 43; n = 8192, 512 products 392 -> 67.
template <int L, int LK, int C>
__global__ __launch_bounds__(512 * C) __attribute__((amdgpu_waves_per_eu(4, 4)))
void ptrans_cyclic_kernel(const PtParams<uint32_t> P) {
  extern __shared__ __align__(16) uint8_t smem[];
  typedef PtGeom<C> Geo;
  constexpr int K = 1 << LK, G = 16 >> LK, PTS = 2 * K, M = Geo::kM;
  constexpr uint32_t kSub = Geo::template sub_bytes<L>();
  const uint32_t lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const uint32_t w = wave & 3, c = (wave >> 2) & (C - 1), half = wave / (4 * C);
  const uint32_t yhigh = lane & 15, row = lane >> 4;
  const uint32_t j = 16 * c + 4 * w + row + Geo::kR * yhigh, t = threadIdx.x & (M - 1);

  uint64_t off[G];
  uint32_t li[G];
  uint32_t v[kPtPoints];
  {
    uint32_t* lin = (uint32_t*)smem + half * 16 * M;
    uint32_t x[16];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint64_t p = (uint64_t)blockIdx.x * G + g;
      const uint64_t gp = global_product(P, p < P.nprod ? p : P.nprod - 1, &li[g]);
      off[g] = wave_uniform(gp * P.n);
      li[g] = wave_uniform(li[g]);
      const uint32_t* in = (half ? P.b : P.a) + off[g] + t;
#pragma unroll
      for (int m = 0; m < K; ++m) x[g * K + m] = in[m * M];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const ModQ32& mod = P.mods[li[g]].m;
      uint32_t* y = x + g * K;
      pt_reduce<K>(y, mod);
      pt_cyclic_fold<K / 2, M>(y, lin + g * K * M + t, mod.q);
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < G; ++g)
      pt_cyclic_points<LK - 1, M>(lin + g * K * M, j, v + g * PTS, P.mods[li[g]].m.q, yhigh);
    __syncthreads();
  }

  uint32_t* results = (uint32_t*)(smem + pt_results_at<uint32_t, L, C, 2>());
  const uint32_t cur = pt_column<C>(c, w, row, yhigh), prev = pt_column_before<C>(c, w, row, yhigh);
  uint32_t ch[kPtPoints / 2];
#pragma unroll
  for (int ph = 0; ph < kPtPoints / kPtBatch; ++ph) {
    const int g = ph * kPtBatch / PTS;  // the batch's product
    const auto& pm = P.mods[li[g]];
    const bool last = (ph + 1) * kPtBatch % PTS == 0;  // its end: x^M + 1, x^M - 1 and two idle slots
#pragma unroll
    for (int h = 0; h < kPtBatch; h += 4) {
      uint8_t* sub = smem + (h + row) * kSub;
      const bool cyclic = last && h == kPtBatch - 4 && row == 1;
      if (half == 0) pt_stage_planes<L, C, false>(v + ph * kPtBatch + h, sub + Geo::kShift * row, pm.m, w, C * yhigh + c, cyclic);
      else pt_stage_planes<L, C, true>(v + ph * kPtBatch + h, sub, pm.m, w, C * yhigh + c, cyclic);
    }
    __syncthreads();
    if (!last || wave / C < kPtBatch - 2)
      pt_multiply<L, C>(smem, results, wave / C, pm, lane, wave % C);
    __syncthreads();
    const uint32_t q = pm.m.q;
#pragma unroll
    for (int s = 0; s < kPtBatch; s += 2) {
      const uint32_t* res = results + (s + half) * Geo::kResWords;
      const int pt = (ph * kPtBatch + s) % PTS, to = g * K + pt_cyclic_to<LK>(pt);
      if (pt == PTS - 2) continue;
      const uint32_t x = res[cur];
      if (pt == PTS - 4) {
        ch[to] = pt_add(x, x, q);
      } else {
        const uint32_t y = res[prev];
        ch[to] = pt_add(x, half ? q - y : y, q);
      }
    }
  }

  uint32_t* give = (uint32_t*)smem + half * 8 * M + t;
  const uint32_t* take = (const uint32_t*)smem + (half ^ 1) * 8 * M + t;
  uint32_t* lin = (uint32_t*)smem + 16 * M;
#pragma unroll
  for (int g = 0; g < G; ++g)
    pt_cyclic_inverse<LK - 1>(ch + g * K, give + g * (K / 2) * M, M, half, P.mods[li[g]].m.q, yhigh);
  __syncthreads();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    pt_cyclic_last<LK - 1, M>(ch + g * K, take + g * (K / 2) * M, M, lin + g * K * M, j, half, P.mods[li[g]].m.q);
    lin[(g * K + (half ? 0 : 1)) * M + j] = ch[g * K + K - 2];
  }
  __syncthreads();
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint32_t q = P.mods[li[g]].m.q;
    const uint32_t* d = lin + g * K * M + t;
    uint32_t s[K / 2];
    pt_cyclic_unfold<K / 4, M>(s, d, q);
    if ((uint64_t)blockIdx.x * G + g < P.nprod) {
      uint32_t* out = P.c + off[g] + half * (K / 2) * M + t;
#pragma unroll
      for (int m = 0; m < K / 2; ++m) {
        const uint32_t x = d[(K / 2 + m) * M];
        out[m * M] = pt_close<false>(s[m], half ? q - x : x, q);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Larger degrees: the same transform once more around it, its points held in a workspace.
// n = k M with M = 4096, k = 2 .. 16: a forward kernel writes the 2k points of a and b as
// polynomials of degree 4096, the kernel above multiplies them (over a's points), an
// inverse kernel puts the products together.  The work on the matrix units stays 2 n 512
// multiply-adds whatever n is.  The forward and inverse kernels move 3 n and 5 n words per operand
// and product (the inverse reads columns j and j - 1, the second from cache).
//
// Up to k0 = 4 a thread holds k0 columns j = ylow + (M / k0) h of all 2 k0 points: a power of w is
// then a renaming of registers and a choice between addition and subtraction, and neighbouring lanes
// have neighbouring columns.  k = 8 and 16 are R = k / 4 transforms of k0 = 4 (over i = R i1 + i0 at
// fixed i0) and one step of radix R: with 2 k0 = 8,
//   A^_(s + 8 m) = sum_{i0 < R} w^(8 i0 m) (w^(i0 s) U_i0[s]),  U_i0[s] = sum_i1 w^(R i1 s) A_(R i1 + i0),
// the U's passing through LDS, where w^(i0 s) is an address; w^8 is -1 (R = 2) or y^(M/2) (R = 4).
// The inverse is the same backwards.
//
// With the columns along rows of sixteen lanes instead (rotations by DPP, as above) a wave's access
// was sixteen pieces of four words: forward and inverse took 18.0 and 16.6 us for sixteen products
// of n = 65536 in 64-bit words, 12.2 and 7.5 us for 48 of n = 16384 in 32-bit words; now
// 13.1 and 14.3, 9.3 and 4.3.  64 or 256 threads are no faster within the sequence of three launches.
// ---------------------------------------------------------------------------
constexpr int kPtOuterM = 4096;
constexpr int kPtOuterThreads = 128;

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

template <int LK>
struct PtOuterGeom {
  static constexpr int K = 1 << LK, LK0 = LK < 2 ? LK : 2, K0 = 1 << LK0, R = K / K0, S0 = 2 * K0;
  static constexpr int B = kPtOuterM / K;                 // columns per step of w
  static constexpr int Y = kPtOuterThreads / (R * R);     // of them per workgroup
  static constexpr int kTiles = B / Y;                    // workgroups per product
  static constexpr int kPart = S0 * K * Y + Y;            // words of one U_i0 in LDS (a row of Y more: i0 runs along lanes)
  static constexpr int kHalves = R > 2 ? R / 2 : 1;       // columns M / 2 apart that w^8 joins
  static constexpr int kUnits = S0 * (K / kHalves) / (R * R);  // (s, yhigh) pairs per thread, R > 1
};

// Column h of y^(ROT M / k0) z, as +-z[src].
template <int K0, int ROT>
struct PtTurn {
  static constexpr int src(int h) { return (h - ROT) & (K0 - 1); }
  static constexpr bool neg(int h) { return ((h - ROT) & K0) != 0; }
};
// (x, z) <- (x + Y z, x - Y z), Y = y^(ROT M / k0).
template <int K0, int ROT, typename W>
__device__ __forceinline__ void pt_reg_butterfly(W* x, W* z, W q) {
  W s[K0], d[K0];
#pragma unroll
  for (int h = 0; h < K0; ++h) {
    const W t = z[PtTurn<K0, ROT>::src(h)];
    const W u = pt_add(x[h], t, q), v = pt_sub(x[h], t, q);
    s[h] = PtTurn<K0, ROT>::neg(h) ? v : u;
    d[h] = PtTurn<K0, ROT>::neg(h) ? u : v;
  }
#pragma unroll
  for (int h = 0; h < K0; ++h) { x[h] = s[h]; z[h] = d[h]; }
}
// Decimation in time as in pt_stages, over v[N][K0].
template <int S, int J, int DIR, int N, int K0, typename W>
__device__ __forceinline__ void pt_reg_stage(W* v, W q) {
  if constexpr (J < S / 2) {
#pragma unroll
    for (int b = 0; b < N; b += S)
      pt_reg_butterfly<K0, DIR * J * (2 * K0 / S)>(v + (b + J) * K0, v + (b + J + S / 2) * K0, q);
    pt_reg_stage<S, J + 1, DIR, N, K0>(v, q);
  }
}
template <int S, int DIR, int N, int K0, typename W>
__device__ __forceinline__ void pt_reg_stages(W* v, W q) {
  if constexpr (S <= N) {
    pt_reg_stage<S, 0, DIR, N, K0>(v, q);
    pt_reg_stages<2 * S, DIR, N, K0>(v, q);
  }
}
// c_i[h] = E_i + y^(-i M / k0) O_i in [0, q), into E.
template <int K0, int I, typename W>
__device__ __forceinline__ void pt_reg_last(W* e, const W* o, W q) {
  if constexpr (I < K0) {
#pragma unroll
    for (int h = 0; h < K0; ++h) {
      const W t = o[I * K0 + PtTurn<K0, -I>::src(h)];
      e[I * K0 + h] = pt_close<false>(e[I * K0 + h], PtTurn<K0, -I>::neg(h) ? q - t : t, q);
    }
    pt_reg_last<K0, I + 1>(e, o, q);
  }
}

// One step of radix R on t[R][kHalves] (R = 4: columns j and j + M / 2).  DIR -1: the inverse.
template <int R, int DIR, typename W>
__device__ __forceinline__ void pt_radix(W (&t)[R][R > 2 ? R / 2 : 1], W q) {
  if constexpr (R == 2) {
    const W x = t[0][0], z = t[1][0];
    t[0][0] = pt_add(x, z, q);
    t[1][0] = pt_sub(x, z, q);
  } else {
    W e0[2], e1[2], o0[2], o1[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      e0[h] = pt_add(t[0][h], t[2][h], q);
      e1[h] = pt_sub(t[0][h], t[2][h], q);
      o0[h] = pt_add(t[1][h], t[3][h], q);
      o1[h] = pt_sub(t[1][h], t[3][h], q);
    }
    constexpr int P = DIR > 0 ? 1 : 3, N = 4 - P;  // t[P] = e1 + y^(M/2) o1, t[N] = e1 - y^(M/2) o1
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      t[0][h] = pt_add(e0[h], o0[h], q);
      t[2][h] = pt_sub(e0[h], o0[h], q);
      const W u = pt_add(e1[h], o1[1 - h], q), v = pt_sub(e1[h], o1[1 - h], q);
      t[P][h] = h ? u : v;
      t[N][h] = h ? v : u;
    }
  }
}

// Workgroup: one of kTiles column tiles of product blockIdx.x / kTiles; blockIdx.y: operand.
template <typename W, int LK>
__global__ __launch_bounds__(kPtOuterThreads) void pt_outer_forward_kernel(const PtOuter<W> P) {
  typedef PtOuterGeom<LK> G;
  constexpr int K = G::K, K0 = G::K0, R = G::R, S0 = G::S0, Y = G::Y;
  const uint64_t p = blockIdx.x / G::kTiles;
  const uint32_t tile = blockIdx.x % G::kTiles * Y;
  const uint32_t i0 = threadIdx.x % R, ylow = threadIdx.x / R % Y, b = threadIdx.x / (R * Y);
  const auto& m = P.mods[p % P.L];
  const W q = (W)m.q;
  const W* in = (blockIdx.y ? P.b : P.a) + p * kPtOuterM * K + (size_t)(tile + ylow + G::B * b) * K;
  W* out = (blockIdx.y ? P.sb : P.sa) + p * 2 * K * kPtOuterM + tile;
  W v[S0 * K0];
  {
    W x[K0 * K0];  // [h][i1]
#pragma unroll
    for (int h = 0; h < K0; ++h) {
      if constexpr (R == 1) pt_load<K0>(in + (size_t)h * (kPtOuterM / K0) * K, x + h * K0);
      else
#pragma unroll
        for (int i = 0; i < K0; ++i) x[h * K0 + i] = in[(size_t)h * (kPtOuterM / K0) * K + R * i + i0];
    }
    pt_reduce<K0 * K0>(x, m);
#pragma unroll
    for (int s = 0; s < K0; ++s)
#pragma unroll
      for (int h = 0; h < K0; ++h) v[2 * s * K0 + h] = v[(2 * s + 1) * K0 + h] = x[h * K0 + pt_bitrev(s, G::LK0)];
  }
  pt_reg_stages<4, 1, S0, K0>(v, q);
  if constexpr (R == 1) {
#pragma unroll
    for (int s = 0; s < S0; ++s)
#pragma unroll
      for (int h = 0; h < K0; ++h) out[s * kPtOuterM + h * (kPtOuterM / K0) + ylow] = v[s * K0 + h];
  } else {
    __shared__ W lds[R * G::kPart];
#pragma unroll
    for (int s = 0; s < S0; ++s)
#pragma unroll
      for (int h = 0; h < K0; ++h) lds[i0 * G::kPart + (s * K + b + R * h) * Y + ylow] = v[s * K0 + h];
    __syncthreads();
    const uint32_t yl = threadIdx.x % Y;
#pragma unroll
    for (int u = 0; u < G::kUnits; ++u) {
      const uint32_t unit = threadIdx.x / Y + u * R * R;
      const int yh = (int)(unit % (K / G::kHalves)), s = (int)(unit / (K / G::kHalves));
      W t[R][G::kHalves];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int h = 0; h < G::kHalves; ++h) {
          const int from = yh + h * (K / 2) - i * s;
          const W x = lds[i * G::kPart + (s * K + (from & (K - 1))) * Y + yl];
          t[i][h] = i > 0 && (from & K) ? q - x : x;
        }
      pt_radix<R, 1>(t, q);
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int h = 0; h < G::kHalves; ++h)
          out[(s + S0 * i) * kPtOuterM + G::B * (yh + h * (K / 2)) + yl] = t[i][h];
    }
  }
}

template <typename W, int LK>
__global__ __launch_bounds__(kPtOuterThreads) void pt_outer_inverse_kernel(const PtOuter<W> P) {
  typedef PtOuterGeom<LK> G;
  constexpr int K = G::K, K0 = G::K0, R = G::R, S0 = G::S0, Y = G::Y;
  const uint64_t p = blockIdx.x / G::kTiles;
  const uint32_t tile = blockIdx.x % G::kTiles * Y;
  const uint32_t i0 = threadIdx.x % R, ylow = threadIdx.x / R % Y, b = threadIdx.x / (R * Y);
  const W q = (W)P.mods[p % P.L].q;
  const W* in = P.sa + p * 2 * K * kPtOuterM;
  // C^_s (1 +- y) at column j
  const auto point = [&](int s, uint32_t j) {
    const W x = in[s * kPtOuterM + j], y0 = in[s * kPtOuterM + (j ? j - 1 : kPtOuterM - 1)];
    const W y = (j == 0) != ((s & 1) != 0) ? q - y0 : y0;
    return pt_add(x, y, q);
  };
  W ch[S0 * K0];  // the even points, then the odd ones, in bit-reversed order
  if constexpr (R == 1) {
#pragma unroll
    for (int s = 0; s < S0; ++s)
#pragma unroll
      for (int h = 0; h < K0; ++h)
        ch[((s & 1) * K0 + pt_bitrev(s >> 1, G::LK0)) * K0 + h] = point(s, tile + ylow + h * (kPtOuterM / K0));
  } else {
    __shared__ W lds[R * G::kPart];
    const uint32_t yl = threadIdx.x % Y;
#pragma unroll
    for (int u = 0; u < G::kUnits; ++u) {
      const uint32_t unit = threadIdx.x / Y + u * R * R;
      const int yh = (int)(unit % (K / G::kHalves)), s = (int)(unit / (K / G::kHalves));
      W t[R][G::kHalves];
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int h = 0; h < G::kHalves; ++h) t[i][h] = point(s + S0 * i, tile + yl + G::B * (yh + h * (K / 2)));
      pt_radix<R, -1>(t, q);
#pragma unroll
      for (int i = 0; i < R; ++i)
#pragma unroll
        for (int h = 0; h < G::kHalves; ++h) {
          const int to = yh + h * (K / 2) - i * s;
          lds[i * G::kPart + (s * K + (to & (K - 1))) * Y + yl] = i > 0 && (to & K) ? q - t[i][h] : t[i][h];
        }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < S0; ++s)
#pragma unroll
      for (int h = 0; h < K0; ++h)
        ch[((s & 1) * K0 + pt_bitrev(s >> 1, G::LK0)) * K0 + h] = lds[i0 * G::kPart + (s * K + b + R * h) * Y + ylow];
  }
  pt_reg_stages<2, -1, K0, K0>(ch, q);
  pt_reg_stages<2, -1, K0, K0>(ch + K0 * K0, q);
  pt_reg_last<K0, 0>(ch, ch + K0 * K0, q);
  W* out = P.c + p * kPtOuterM * K + (size_t)(tile + ylow + G::B * b) * K;
#pragma unroll
  for (int h = 0; h < K0; ++h) {
    W c[K0];
#pragma unroll
    for (int i = 0; i < K0; ++i) c[i] = ch[i * K0 + h];
    if constexpr (R == 1) pt_put<K0>(out + (size_t)h * (kPtOuterM / K0) * K, c);
    else
#pragma unroll
      for (int i = 0; i < K0; ++i) out[(size_t)h * (kPtOuterM / K0) * K + R * i + i0] = c[i];
  }
}

}  // namespace pm
