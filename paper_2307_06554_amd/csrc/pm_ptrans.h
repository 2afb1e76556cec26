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
#pragma once
#include "pm_mfma16.h"

namespace pm {

constexpr int kPtM = 256;             // degree bound of the sub-products
constexpr int kPtPoints = 32;         // sub-products per workgroup
constexpr int kPtBatch = 8;           // of them in LDS at a time
constexpr uint32_t kPtAPlane = 272;   // reversed ext positions 0 .. 271: 255 .. -16
constexpr uint32_t kPtBPlane = 31 * 16;  // rows -15 .. 15
constexpr uint32_t kPtRow = 80;       // words between the four result rows of a sub-product
template <int L>
constexpr uint32_t pt_sub_bytes() { return (uint32_t)L * (kPtAPlane + kPtBPlane); }
template <int L>
constexpr uint32_t pt_lds_bytes() { return kPtBatch * (pt_sub_bytes<L>() + 4 * kPtRow * 4); }

struct PtMod {
  ModQ32 m;
  uint32_t qinv;   // q^-1 mod 2^32
  uint64_t lift;   // q L^2 M 2^13
  int32_t rc[8];   // 2^(8s) 2^32 / (2k) mod q, centred, s < 2L - 1
};
struct PtParams {
  const uint32_t* a;
  const uint32_t* b;
  uint32_t* c;
  uint64_t nprod;
  uint32_t n;
  uint32_t lc, nq_total, l0, lrep;  // products and moduli as in Mfma32Params
  uint32_t b_shared;
  PtMod mods[kMaxQ];
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
// y^(16 R) v, R in (-16, 16): the lanes that pass y^M = -1 are negated, then the row rotates.
template <int R>
__device__ __forceinline__ uint32_t pt_shift(uint32_t v, uint32_t q, uint32_t yhigh) {
  if constexpr (R != 0) {
    const bool wraps = R > 0 ? (int)yhigh >= 16 - R : (int)yhigh < -R;
    v = wraps ? q - v : v;
  }
  return pt_rot<R>(v);
}

// Sum and difference mod q of x, y in [0, q], again in [0, q] (q < 2^31; q stands for 0 too).
__device__ __forceinline__ uint32_t pt_add(uint32_t x, uint32_t y, uint32_t q) {
  const uint32_t s = x + y;
  return min_u32(s, s - q);
}
__device__ __forceinline__ uint32_t pt_sub(uint32_t x, uint32_t y, uint32_t q) {
  const uint32_t d = x - y;
  return min_u32(d, d + q);
}

// (x, z) <- (x + Y z, Y z - x), Y = y^(16 R).  The difference is taken this way round
// because the rotated operand of an addition or subtraction has to be its first one
// (v_subrev_u32 with a DPP row rotation was measured to rotate the other operand).
template <int R>
__device__ __forceinline__ void pt_butterfly(uint32_t& x, uint32_t& z, uint32_t q, uint32_t yhigh) {
  const uint32_t t = pt_shift<R>(z, q, yhigh);
  z = pt_sub(t, x, q);
  x = pt_add(t, x, q);
}

// Decimation-in-time stages of block size S .. N over v[0 .. N) (bit-reversed order in,
// natural order out); the S-point root of one is y^(16 (32 / S)), DIR -1: its inverse.
// Output i carries the sign (-1)^(bits set in i): the two inputs of a butterfly have the
// same index within their blocks, hence the same sign, and each upper half flips it.  In the
// forward transform the signs of a and b cancel in the products; the inverse's last step
// takes them out.
template <int S, int J, int DIR, int N>
__device__ __forceinline__ void pt_stage(uint32_t* v, uint32_t q, uint32_t yhigh) {
  if constexpr (J < S / 2) {
#pragma unroll
    for (int b = 0; b < N; b += S) pt_butterfly<DIR * J * (32 / S)>(v[b + J], v[b + J + S / 2], q, yhigh);
    pt_stage<S, J + 1, DIR, N>(v, q, yhigh);
  }
}
template <int S, int DIR, int N>
__device__ __forceinline__ void pt_stages(uint32_t* v, uint32_t q, uint32_t yhigh) {
  if constexpr (S <= N) {
    pt_stage<S, 0, DIR, N>(v, q, yhigh);
    pt_stages<2 * S, DIR, N>(v, q, yhigh);
  }
}

// The 2K points of one operand from its K words (reduced mod q here): the upper half of
// the transform's input is zero, so its first stage only copies.
template <int LK>
__device__ __forceinline__ void pt_forward(const uint32_t* x, uint32_t* v, const ModQ32& m, uint32_t yhigh) {
  constexpr int K = 1 << LK;
#pragma unroll
  for (int p = 0; p < K; ++p) v[2 * p] = v[2 * p + 1] = reduce_u32(x[pt_bitrev(p, LK)], m);
  pt_stages<4, 1, 2 * K>(v, m.q, yhigh);
}

// c_i = +-(E_i + w^(-i) O_i) from the transformed even and odd points, in [0, q).
template <int LK, int I>
__device__ __forceinline__ void pt_last(const uint32_t* e, const uint32_t* o, uint32_t* c, uint32_t q, uint32_t yhigh) {
  if constexpr (I < (1 << LK)) {
    const uint32_t u = pt_shift<-I * (16 >> LK)>(o[I], q, yhigh) + e[I];  // in [0, 2q]
    if constexpr (__builtin_popcount(I) & 1) c[I] = min_u32(min_u32(0u - u, q - u), 2 * q - u);
    else c[I] = min_u32(min_u32(u, u - q), u - 2 * q);
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

// Four points of the column group's four columns into the digit planes of sub-product
// `sub` (this row's): the reversed ext of a, or the rows of b.
template <int L, bool IS_B>
__device__ __forceinline__ void pt_stage_planes(const uint32_t* v, uint8_t* sub, const ModQ32& m, uint32_t wave,
                                                uint32_t yhigh) {
  uint32_t w[4] = {v[0], v[1], v[2], v[3]};
  pt_transpose(w);
  uint32_t pos[4], neg[4];
  if constexpr (IS_B) {
    digits_pm32<L>(w, m.q, m.thr, pos, neg);
    uint8_t* rows = sub + L * kPtAPlane + 4 * wave;
    transpose_store<L>(rows, kPtBPlane, (yhigh + 15) * 16, pos);
    if (yhigh > 0) transpose_store<L>(rows, kPtBPlane, (yhigh - 1) * 16, neg);
  } else {
    const uint32_t rev[4] = {w[3], w[2], w[1], w[0]};
    digits_pm32<L>(rev, m.q, m.thr, pos, neg);
    const uint32_t off = 252 - 4 * wave - 16 * yhigh;
    transpose_store<L>(sub, kPtAPlane, off, pos);
    if (yhigh == 15) transpose_store<L>(sub, kPtAPlane, off + 256, neg);
  }
}

// One sub-product from its planes to its words (canonical, scaled by 1/2k): lane (u, g)
// leaves coefficients 16 u + 4 g + e in row e of res.  -c[255] goes to slot 64 of row 3,
// where column 0 finds y c.
template <int L>
__device__ __forceinline__ void pt_multiply(const uint8_t* sub, uint32_t* res, const PtMod& pm, uint32_t lane) {
  const int zl = (int)(lane & 15), g = (int)(lane >> 4);
  const int S0 = 255 - 16 * g - zl;
  const int B0 = (zl + 15 - g) * 16;
  const uint8_t* bp = sub + L * kPtAPlane;
  v4i_acc acc[2 * L - 1];
#pragma unroll
  for (int s = 0; s < 2 * L - 1; ++s) acc[s] = v4i_acc{0, 0, 0, 0};
#pragma unroll
  for (int st = 0; st < kPtM / 64; ++st) mfma16_step<L>(acc, sub, kPtAPlane, S0 - 64 * st, bp, kPtBPlane, B0 - 64 * st);
  const uint32_t q = pm.m.q;
  uint32_t out[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint64_t x = pm.lift;
#pragma unroll
    for (int s = 0; s < 2 * L - 1; ++s) x += (uint64_t)((int64_t)acc[s][e] * (int64_t)pm.rc[s]);
    const uint32_t t = (uint32_t)(x >> 32) - mul_hi32((uint32_t)x * pm.qinv, q);
    out[e] = min_u32(t, t + q);
    res[e * kPtRow + lane] = out[e];
  }
  if (lane == 63) res[3 * kPtRow + 64] = q - out[3];
}

template <int L, int LK>
__device__ __forceinline__ void pt_group(const PtParams& P, uint64_t grp, uint8_t* smem) {
  constexpr int K = 1 << LK, G = 16 >> LK, PTS = 2 * K;
  const uint32_t lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const uint32_t yhigh = lane & 15, row = lane >> 4, ylow = 4 * wave + row;
  const uint32_t j = ylow + 16 * yhigh;

  uint64_t off[G], boff[G];
  uint32_t li[G];
  uint32_t va[kPtPoints], vb[kPtPoints];
  {
    uint32_t xa[16], xb[16];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint64_t p = grp * G + g;
      const uint64_t gp = global_product(P, p < P.nprod ? p : P.nprod - 1, &li[g]);
      off[g] = wave_uniform(gp * P.n);
      boff[g] = wave_uniform(b_product(P, gp, li[g]) * P.n);
      li[g] = wave_uniform(li[g]);
#pragma unroll
      for (int i = 0; i < K; i += 4) {
        const uint4 x = *(const uint4*)(P.a + off[g] + (size_t)K * j + i);
        const uint4 z = *(const uint4*)(P.b + boff[g] + (size_t)K * j + i);
        xa[g * K + i] = x.x; xa[g * K + i + 1] = x.y; xa[g * K + i + 2] = x.z; xa[g * K + i + 3] = x.w;
        xb[g * K + i] = z.x; xb[g * K + i + 1] = z.y; xb[g * K + i + 2] = z.z; xb[g * K + i + 3] = z.w;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      pt_forward<LK>(xa + g * K, va + g * PTS, P.mods[li[g]].m, yhigh);
      pt_forward<LK>(xb + g * K, vb + g * PTS, P.mods[li[g]].m, yhigh);
    }
  }

  uint32_t* results = (uint32_t*)(smem + kPtBatch * pt_sub_bytes<L>());
  // column j of a sub-product's results, and column j - 1 (times y: -c[255] at j = 0)
  const uint32_t cur = row * kPtRow + 16 * wave + yhigh;
  const uint32_t prev = row > 0 ? cur - kPtRow
                        : wave > 0 ? 3 * kPtRow + 16 * (wave - 1) + yhigh
                        : yhigh > 0 ? 3 * kPtRow + 48 + yhigh - 1 : 3 * kPtRow + 64;
  uint32_t ch[kPtPoints];  // C^_s (1 +- y) at column j, the even points of a product first
#pragma unroll
  for (int ph = 0; ph < kPtPoints / kPtBatch; ++ph) {
    const int g = ph * kPtBatch / PTS;  // the batch's product
    const PtMod& pm = P.mods[li[g]];
#pragma unroll
    for (int h = 0; h < kPtBatch; h += 4) {
      uint8_t* sub = smem + (h + row) * pt_sub_bytes<L>();
      pt_stage_planes<L, false>(va + ph * kPtBatch + h, sub, pm.m, wave, yhigh);
      pt_stage_planes<L, true>(vb + ph * kPtBatch + h, sub, pm.m, wave, yhigh);
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t s = 2 * wave; s < 2 * wave + 2; ++s)
      pt_multiply<L>(smem + s * pt_sub_bytes<L>(), results + s * 4 * kPtRow, pm, lane);
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kPtBatch; ++s) {
      const uint32_t x = results[s * 4 * kPtRow + cur], y = results[s * 4 * kPtRow + prev];
      const int pt = (ph * kPtBatch + s) % PTS;
      // decimation in time wants the points of each half in bit-reversed order
      const int to = g * PTS + (pt & 1) * K + pt_bitrev(pt >> 1, LK);
      ch[to] = pt & 1 ? pt_sub(x, y, pm.m.q) : pt_add(x, y, pm.m.q);
    }
  }
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const uint32_t q = P.mods[li[g]].m.q;
    uint32_t* e = ch + g * PTS;
    uint32_t c[K];
    pt_stages<2, -1, K>(e, q, yhigh);
    pt_stages<2, -1, K>(e + K, q, yhigh);
    pt_last<LK, 0>(e, e + K, c, q, yhigh);
    if (grp * G + g < P.nprod) {
#pragma unroll
      for (int i = 0; i < K; i += 4)
        *(uint4*)(P.c + off[g] + (size_t)K * j + i) = make_uint4(c[i], c[i + 1], c[i + 2], c[i + 3]);
    }
  }
}

template <int L, int LK>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
void ptrans_kernel(const PtParams P) {
  extern __shared__ __align__(16) uint8_t smem[];
  pt_group<L, LK>(P, blockIdx.x, smem);
}

}  // namespace pm
