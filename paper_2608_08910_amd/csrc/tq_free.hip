// Free-scale solver (Sec. 2.1: PTQTP fits W ~ alpha1*T1 + alpha2*T2 per group by
// alternating plane and scale updates with two free scales; the tie alpha = (3s, s) is
// its constrained case). Started from a tied fit, it refines each 256-weight block into
// the free-scale two-plane layout: least-squares scale pairs and best-of-nine plane
// pairs in turn, every decision in a fixed precision and order (stated in tq.h), so the
// result is reproducible bit for bit.
#include "tq_device.hpp"
#include "tq_internal.hpp"

namespace tq {

// A 16-lane group owns one block (four a wave), lane u holding weights u + 16j.
constexpr int kFreeE = 16;

template <int M>
__device__ __forceinline__ double xor_addd(double a) {
  const int lo = __double2loint(a), hi = __double2hiint(a);
  return a + __hiloint2double(lane_xor_i<M>(hi), lane_xor_i<M>(lo));
}
template <int M>
__device__ __forceinline__ int xor_addi(int a) {
  return a + lane_xor_i<M>(a);
}

// Sum over the block in the pairwise-halving order: within the lane for h = 128 .. 16,
// then across the group's lanes for h = 8 .. 1.
__device__ __forceinline__ double block_sum(double (&p)[kFreeE]) {
#pragma unroll
  for (int h = kFreeE / 2; h >= 1; h >>= 1)
#pragma unroll
    for (int j = 0; j < h; ++j) p[j] = p[j] + p[j + h];
  double s = xor_addd<8>(p[0]);
  s = xor_addd<4>(s);
  s = xor_addd<2>(s);
  return xor_addd<1>(s);
}
__device__ __forceinline__ int block_sum(int a) {
  a = xor_addi<8>(a);
  a = xor_addi<4>(a);
  a = xor_addi<2>(a);
  return xor_addi<1>(a);
}

// The plane step: each weight takes the first pair in the order 0, -1, +1 (t1 outer,
// t2 inner) with the least |w - (a1 t1 + a2 t2)| in fp64. The nine candidate values
// are the block's own (a1 t1 exact, one rounding in the sum).
__device__ __forceinline__ void free_plane_step(const float (&w)[kFreeE], float a1, float a2, int (&t1)[kFreeE],
                                                int (&t2)[kFreeE]) {
#pragma clang fp contract(off)
  constexpr int kOrd[3] = {0, -1, 1};
  double cand[9];
#pragma unroll
  for (int x = 0; x < 3; ++x)
#pragma unroll
    for (int y = 0; y < 3; ++y) cand[3 * x + y] = (double)a1 * kOrd[x] + (double)a2 * kOrd[y];
#pragma unroll
  for (int j = 0; j < kFreeE; ++j) {
    const double wd = (double)w[j];
    double best = fabs(wd - cand[0]);
    int bi = 0;
#pragma unroll
    for (int c = 1; c < 9; ++c) {
      const double e = fabs(wd - cand[c]);
      if (e < best) {
        best = e;
        bi = c;
      }
    }
    t1[j] = kOrd[bi / 3];
    t2[j] = kOrd[bi % 3];
  }
}

// f32 -> f16 bits, nearest even, saturating to +-65504.
__device__ __forceinline__ uint16_t f16_sat(float x) {
  const float c = fminf(fmaxf(x, -65504.0f), 65504.0f);
  // values in (65504, 65520) round to 65504 anyway; clamping first keeps 65520 and up
  // from rounding to infinity
  return __builtin_bit_cast(uint16_t, (_Float16)(fabsf(x) >= 65520.0f ? c : x));
}

// Sum over the 16 lanes of a group (whole numbers: any order).
__device__ __forceinline__ int group16_sum(int v) {
  v = group_sum_i32(v);
  return v + __builtin_amdgcn_update_dpp(0, v, kDppRowRor8, 0xf, 0xf, false);
}

// a * b + c in one instruction (24-bit operands; the compiler splits it into a multiply and a
// three-operand add)
__device__ __forceinline__ int mad24(int a, int b, int c) {
  int r;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// A weight's plane pair for |w| (both trits change sign with w) as one word: bits 31:30 t2 and
// 29:28 t1 in two's complement; below them what a sum over the block's weights counts: bit 0
// t1 != 0, bit 6 t2 != 0, bit 12 trits of opposite direction, bit 18 of the same, relative to
// the signs of (a1, a2).
constexpr uint32_t kPairMask = 0xF0000000u;
__device__ __forceinline__ uint32_t trit2(int t) { return (uint32_t)t & 3u; }
// the pair's four top bits for w of either sign
__device__ __forceinline__ uint32_t pair_signed(uint32_t x, float w) {
  return (int)__float_as_uint(w) < 0 ? x ^ ((x & 5u) << 1) : x;
}

// The plane step by thresholds on |w|. With A = |a1| > B = |a2| > 0 the candidates are 0 and
// +- the four levels B, A - B, A, A + B; with every gap at least 2^-16 of the block's largest
// magnitude, all differences w - candidate near a decision are exact in fp64, so the nearest
// candidate changes at the exact middle of two neighbouring levels and a tie goes to the
// pair that comes first in the order 0, -1, +1: the one with the zero trit, whatever the
// signs. T[i] is the smallest fp32 |w| (as bits) that takes level i + 1, K[i] that level's
// pair. (Otherwise `ok` is false, and the wave's blocks take the nine-candidate search.)
struct Levels {
  uint32_t T[4], K[4];
  bool ok;
};

__device__ __forceinline__ Levels make_levels(float a1, float a2, float amax) {
  Levels L;
  const float A = fabsf(a1), B = fabsf(a2);
  const float tol = 0x1p-16f * fmaxf(amax, A + B);
  L.ok = (B >= 0x1p-100f) & (B >= tol) & (A - B >= tol) & (fabsf((A - B) - B) >= tol) & (tol < 0x1p100f);
  const double dA = A, dB = B, dD = dA - dB;
  const bool c = dB < dD;
  const double l2 = c ? dD : dB;
  const double M[4] = {0.5 * (c ? dB : dD), 0.5 * dA, 0.5 * (l2 + dA), dA + 0.5 * dB};
  const bool down[4] = {true, c, !c, true};  // the lower level takes a tie
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float f = (float)M[i];
    L.T[i] = __float_as_uint(f) + (uint32_t)(((double)f < M[i]) | (((double)f == M[i]) & down[i]));
  }
  const int s1 = (int)__float_as_uint(a1) < 0 ? -1 : 1, s2 = (int)__float_as_uint(a2) < 0 ? -1 : 1;
  const uint32_t kA = (trit2(s1) << 28) | 1u, kB = (trit2(s2) << 30) | (1u << 6);
  const uint32_t kD = (trit2(s1) << 28) | (trit2(-s2) << 30) | 1u | (1u << 6) | (1u << 12);
  L.K[0] = c ? kB : kD;
  L.K[1] = c ? kD : kB;
  L.K[2] = kA;
  L.K[3] = (kA | kB) + (1u << 18);
  return L;
}

__device__ __forceinline__ uint32_t level_pair(uint32_t aw, const Levels& L) {
  uint32_t k = aw >= L.T[0] ? L.K[0] : 0u;
  k = aw >= L.T[1] ? L.K[1] : k;
  k = aw >= L.T[2] ? L.K[2] : k;
  return aw >= L.T[3] ? L.K[3] : k;
}

// A block's scale pair at the alternation's end and its plane steps.
struct FreeFit {
  float a1, a2;
  int it;
  float amax;  // the block's largest magnitude (the threshold step's)
};

// The alternation for any block (every lane of the wave): scale sums in the pairwise-halving
// order, the nine-candidate plane step.
__device__ __forceinline__ void free_fit_general(const float (&v)[kFreeE], const uint8_t* cb, float s, int grp, int u,
                                                 int max_iter, FreeFit& F) {
#pragma clang fp contract(off)
  int t1[kFreeE], t2[kFreeE];
  // the tied fit: weight u + 32m in the low nibble of byte 16m + u, u + 32m + 16 in the high
#pragma unroll
  for (int m = 0; m < kFreeE / 2; ++m) {
    const int byte = cb[16 * m + u];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int nib = (byte >> (4 * h)) & 15;
      const int c = nib >= 8 ? nib - 16 : nib;
      const int a = (c + 4) / 3 - 1;  // unfold: balanced-ternary digits of c
      t1[2 * m + h] = a;
      t2[2 * m + h] = c - 3 * a;
    }
  }
  const bool live = s != 0.0f;  // uniform within the group
  float a1 = 3.0f * s, a2 = s;
  int it = 0;
  bool done = !live;  // a group stops at its own stopping point; the wave runs until all do
  while (!__all(done)) {
    // scale step: least squares for (a1, a2) given the planes
    double pu[kFreeE], pv[kFreeE];
    int sa = 0, sb = 0, sc = 0;
#pragma unroll
    for (int j = 0; j < kFreeE; ++j) {
      pu[j] = (double)v[j] * (double)t1[j];
      pv[j] = (double)v[j] * (double)t2[j];
      sa += t1[j] * t1[j];
      sb += t1[j] * t2[j];
      sc += t2[j] * t2[j];
    }
    const double su = block_sum(pu), sv = block_sum(pv);
    sa = block_sum(sa);
    sb = block_sum(sb);
    sc = block_sum(sc);
    const int det = sa * sc - sb * sb;  // |.| <= 256^2: exact in int
    if (!done && det > 0) {
      const double num1 = (double)sc * su - (double)sb * sv;
      const double num2 = (double)sa * sv - (double)sb * su;
      a1 = (float)(num1 / (double)det);
      a2 = (float)(num2 / (double)det);
    }
    // plane step
    int n1[kFreeE], n2[kFreeE];
    free_plane_step(v, a1, a2, n1, n2);
    int diff = 0;
#pragma unroll
    for (int j = 0; j < kFreeE; ++j) {
      diff |= (n1[j] ^ t1[j]) | (n2[j] ^ t2[j]);
      if (!done) {
        t1[j] = n1[j];
        t2[j] = n2[j];
      }
    }
    const uint64_t unchanged = __ballot(diff == 0);
    const bool same = ((unchanged >> (16 * grp)) & 0xFFFFu) == 0xFFFFu;
    if (!done) {
      ++it;
      done = same || it == max_iter;
    }
  }
  F.a1 = a1;
  F.a2 = a2;
  F.it = it;
}

// The same by thresholds, with the same result, where every live block of the wave has well
// separated levels at every step and no tiny weight with a trit in its tied fit (false
// otherwise). Every weight with a trit is then past 2^-17 of the block's largest, so with
// amax < 2^(e+1) it is a multiple of 2^(e-41): |w| = (hi 2^20 + lo) 2^(e-41), and the sums of
// a scale step are exact in whole numbers (as the general path's are in fp64).
__device__ __forceinline__ bool free_fit_levels(const float (&v)[kFreeE], const uint8_t* cb, float s, int grp, int u,
                                                int max_iter, FreeFit& F) {
#pragma clang fp contract(off)
  uint32_t amaxb = 0;
#pragma unroll
  for (int j = 0; j < kFreeE; ++j) amaxb = max(amaxb, __float_as_uint(fabsf(v[j])));
  amaxb = max(amaxb, (uint32_t)lane_xor_i<8>((int)amaxb));
  amaxb = max(amaxb, (uint32_t)lane_xor_i<4>((int)amaxb));
  amaxb = max(amaxb, (uint32_t)lane_xor_i<2>((int)amaxb));
  amaxb = max(amaxb, (uint32_t)lane_xor_i<1>((int)amaxb));
  const float amax = __uint_as_float(amaxb);
  const int e = (int)(amaxb >> 23) - 127;
  const bool live = s != 0.0f;  // uniform within the group
  bool bad = amaxb >= 0x7F800000u;  // infinities and NaN
  int hi[kFreeE], lo[kFreeE];
#pragma unroll
  for (int j = 0; j < kFreeE; ++j) {
    const float x = ldexpf(fabsf(v[j]), 21 - e);
    hi[j] = (int)x;  // below 2^22
    lo[j] = (int)((x - (float)hi[j]) * 0x1p20f);
  }
  // the tied fit's planes (folded onto |w|) and their sums: weight u + 32m in the low nibble of
  // byte 16m + u, u + 32m + 16 in the high
  uint32_t kw[kFreeE];
  int suh = 0, sul = 0, svh = 0, svl = 0, sa = 0, sb = 0, sc = 0;
  const float least = 0x1p-17f * amax;
#pragma unroll
  for (int m = 0; m < kFreeE / 2; ++m) {
    const int byte = cb[16 * m + u];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int j = 2 * m + h;
      int c = (int)((uint32_t)byte << (28 - 4 * h)) >> 28;
      bad |= (c < -4) | (c > 4) | ((c != 0) & (fabsf(v[j]) < least));
      c = (int)__float_as_uint(v[j]) < 0 ? -c : c;
      const int t1 = (c >= 2 ? 1 : 0) - (c <= -2 ? 1 : 0), t2 = c - 3 * t1;  // balanced-ternary digits
      kw[j] = (trit2(t1) << 28) | (trit2(t2) << 30);
      suh = mad24(hi[j], t1, suh);
      sul = mad24(lo[j], t1, sul);
      svh = mad24(hi[j], t2, svh);
      svl = mad24(lo[j], t2, svl);
      sa += t1 * t1;
      sb += t1 * t2;
      sc += t2 * t2;
    }
  }
  if (__any(bad & live)) return false;
  sa = group16_sum(sa);
  sb = group16_sum(sb);
  sc = group16_sum(sc);
  float a1 = 3.0f * s, a2 = s;
  int it = 0;
  bool done = !live;  // a group stops at its own stopping point; the wave runs until all do
  while (!__all(done)) {
    // scale step: least squares for (a1, a2) given the planes
    const double su = ldexp((double)group16_sum(suh) * 0x1p20 + (double)group16_sum(sul), e - 41);
    const double sv = ldexp((double)group16_sum(svh) * 0x1p20 + (double)group16_sum(svl), e - 41);
    const int det = sa * sc - sb * sb;  // |.| <= 256^2: exact in int
    if (!done && det > 0) {
      const double num1 = (double)sc * su - (double)sb * sv;
      const double num2 = (double)sa * sv - (double)sb * su;
      a1 = (float)(num1 / (double)det);
      a2 = (float)(num2 / (double)det);
    }
    // plane step, with the sums and counts of the next scale step
    const Levels L = make_levels(a1, a2, amax);
    if (!__all(L.ok | done)) return false;
    uint32_t diff = 0, cnt = 0;
    suh = sul = svh = svl = 0;
#pragma unroll
    for (int j = 0; j < kFreeE; ++j) {
      const uint32_t k = level_pair(__float_as_uint(fabsf(v[j])), L);
      const int t1 = (int)(k << 2) >> 30, t2 = (int)k >> 30;
      suh = mad24(hi[j], t1, suh);
      sul = mad24(lo[j], t1, sul);
      svh = mad24(hi[j], t2, svh);
      svl = mad24(lo[j], t2, svl);
      cnt += k;  // (fields of 6 bits, at most 16 each)
      diff |= k ^ kw[j];
      kw[j] = k;
    }
    const uint64_t unchanged = __ballot((diff & kPairMask) == 0);
    const bool same = ((unchanged >> (16 * grp)) & 0xFFFFu) == 0xFFFFu;
    if (!done) {
      ++it;
      done = same || it == max_iter;
    }
    const int c02 = group16_sum((int)((cnt & 63u) | ((cnt << 4) & 0x3F0000u)));
    const int c13 = group16_sum((int)(((cnt >> 6) & 63u) | ((cnt >> 2) & 0x3F0000u)));
    sa = c02 & 0xFFFF;
    sc = c13 & 0xFFFF;
    sb = (c13 >> 16) - (c02 >> 16);
    sb = (int)(__float_as_uint(a1) ^ __float_as_uint(a2)) < 0 ? -sb : sb;
  }
  F.a1 = a1;
  F.a2 = a2;
  F.it = it;
  F.amax = amax;
  return true;
}

// Bound by the vector ALU over the iterations of the alternation. Per weight and iteration the
// threshold step is 17 operations (compares and selects of the pair, four whole-number
// multiply-adds, the count, the change test), where the nine-candidate search with its products takes about 60 operations:
// 2048 x 4096 82 us, the search alone 242. (A wave runs until its slowest of four blocks stops:
// 6.9 iterations, 3.5 a block on average.) A wave that falls back in the
// alternation starts the search over and pays for both; where only the rounded scales are too
// close, only the last step is searched (weights of 2^-24, whose scales are an ulp or two of f16's
// least: 112 us, 366 starting over, the search alone 306). All kinds of blocks side by side 131 us
// (171, 198), weights over many orders of magnitude 75 (123, 136), an outlier a block 60 (63, 177).
__global__ __launch_bounds__(256) void k_free_quantize(const float* __restrict__ w, int64_t nblocks, int max_iter,
                                                       const uint8_t* __restrict__ tcodes,
                                                       const uint16_t* __restrict__ tscales,
                                                       uint8_t* __restrict__ codes2, uint32_t* __restrict__ scales2,
                                                       uint8_t* __restrict__ iters) {
#pragma clang fp contract(off)
  __shared__ __attribute__((aligned(16))) uint8_t s_w[16][128];  // per block: the two-plane bytes
  const int lane = threadIdx.x & 63, grp = lane >> 4, u = lane & 15;
  const int lb = (threadIdx.x >> 6) * 4 + grp;
  const int64_t blk0 = (int64_t)blockIdx.x * 16, blk = min(blk0 + lb, nblocks - 1);
  const bool real = blk0 + lb < nblocks;  // a group past the last block repeats it, stores nothing
  const float* wb = w + blk * 256;
  float v[kFreeE];
#pragma unroll
  for (int j = 0; j < kFreeE; ++j) v[j] = wb[u + 16 * j];
  const float s = f16_bits_to_f32(tscales[blk]);
  const uint8_t* cb = tcodes + blk * 128;
  FreeFit F;
  const bool lv = free_fit_levels(v, cb, s, grp, u, max_iter, F);
  if (!lv) free_fit_general(v, cb, s, grp, u, max_iter, F);
  // the planes of the rounded scales: pairs with t1 in bits 1:0, t2 in bits 3:2
  const bool live = s != 0.0f;
  const uint16_t h1 = live ? f16_sat(F.a1) : 0, h2 = live ? f16_sat(F.a2) : 0;
  uint32_t x[kFreeE];
  const Levels L = make_levels(f16_bits_to_f32(h1), f16_bits_to_f32(h2), lv ? F.amax : 0.0f);
  if (lv && __all(L.ok | !live)) {
#pragma unroll
    for (int j = 0; j < kFreeE; ++j) x[j] = pair_signed(level_pair(__float_as_uint(fabsf(v[j])), L) >> 28, v[j]);
  } else {
    int t1[kFreeE], t2[kFreeE];
    free_plane_step(v, f16_bits_to_f32(h1), f16_bits_to_f32(h2), t1, t2);
#pragma unroll
    for (int j = 0; j < kFreeE; ++j) x[j] = trit2(t1[j]) | (trit2(t2[j]) << 2);
  }
#pragma unroll
  for (int j = 0; j < kFreeE; ++j) x[j] = live ? x[j] : 0u;
  // pack: weight u + 16j is column 32 (j / 2) + 16 (j % 2) + 4 (u / 4) + (u % 4) of its
  // block, i.e. plane p's dword 4 (j / 2) + 2p + (j % 2), byte u % 4, bits 2 (u / 4). The four
  // lanes of a byte (u, u ^ 4, u ^ 8, u ^ 12) join their bits (16 bytes a plane, four j to a
  // dword), and each stores the bytes of j = 4i + u / 4.
  const int q4 = u >> 2;
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int i = 0; i < kFreeE / 4; ++i) {
      uint32_t z = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) z |= ((x[4 * i + k] >> (2 * p)) & 3u) << (8 * k);
      z <<= 2 * q4;
      z |= (uint32_t)lane_xor_i<4>((int)z);
      z |= (uint32_t)lane_xor_i<8>((int)z);
      const int j = 4 * i + q4;
      s_w[lb][(4 * (j >> 1) + 2 * p + (j & 1)) * 4 + (u & 3)] = (uint8_t)(z >> (8 * q4));
    }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < 128 && blk0 + (t >> 3) < nblocks)
    reinterpret_cast<uint4*>(codes2 + (blk0 + (t >> 3)) * 128)[t & 7] = reinterpret_cast<const uint4*>(s_w[t >> 3])[t & 7];
  if (u == 0 && real) {
    scales2[blk] = (uint32_t)h1 | ((uint32_t)h2 << 16);
    if (iters) iters[blk] = (uint8_t)F.it;
  }
}

}  // namespace tq

extern "C" tq_status tq_free_quantize(const float* w, int32_t n, int32_t k, int32_t max_iter,
                                      const uint8_t* tied_codes, const uint16_t* tied_scales, uint8_t* codes2,
                                      uint16_t* scales2, uint8_t* iters, void* stream) {
  using namespace tq;
  clear_error();
  if (n < 0 || k <= 0 || k % 256 != 0)
    return fail(TQ_ERR_INVALID, "tq_free_quantize: n = %d, k = %d (need n >= 0, k a positive multiple of 256)", n, k);
  if (max_iter < 1 || max_iter > 255)
    return fail(TQ_ERR_INVALID, "tq_free_quantize: max_iter = %d outside [1, 255]", max_iter);
  if (n == 0) return TQ_OK;
  if (!w || !tied_codes || !tied_scales || !codes2 || !scales2)
    return fail(TQ_ERR_INVALID, "tq_free_quantize: null pointer");
  if (!aligned(w, 4) || !aligned(tied_codes, 128) || !aligned(tied_scales, 2) || !aligned(codes2, 128) ||
      !aligned(scales2, 4))
    return fail(TQ_ERR_ALIGN,
                "tq_free_quantize: w 4-byte, codes 128-byte, tied scales 2-byte and scale pairs 4-byte aligned");
  const int64_t nblocks = (int64_t)n * (k / 256);
  (void)hipGetLastError();
  hipLaunchKernelGGL(k_free_quantize, dim3((unsigned)((nblocks + 15) / 16)), dim3(256), 0, (hipStream_t)stream, w,
                     nblocks, (int)max_iter, tied_codes, tied_scales, codes2, reinterpret_cast<uint32_t*>(scales2),
                     iters);
  return check_launch("tq_free_quantize");
}
