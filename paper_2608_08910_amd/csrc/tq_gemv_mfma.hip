// The dot pass of one matrix on several tokens, on the matrix cores: folded codes, the
// free-scale two-plane format and the MXFP4 bytes (the single-token passes are in
// tq_gemv.hip, tq_gemv2.hip and tq_gemv_mx.hip). On the VALU a token costs eight byte dots
// per 32 weights and a share of the cross-lane butterflies, so two tokens already cost more
// than the weight stream; an int8 MFMA takes 16 tokens for the price of one.
//
// Split: a workgroup is eight waves and owns RT x 16 rows x MTT x 16 tokens; wave w takes
// the 256-blocks b with b mod 8 = w, in ascending order, and the eight partial results meet
// in LDS at the end as ((0+1)+(2+3))+((4+5)+(6+7)). So the waves share nothing until then
// (no barrier in the loop, each streams its own bytes), a small matrix still puts eight
// waves on every row tile, and each sum is taken in exactly the order of the single-token
// kernels (lane group g of those takes the blocks b mod 8 = g, then an xor butterfly), so
// a token's result has the same bits whatever kernel took it (MXFP4 aside, whose block sums
// are taken another way, below). Rows of fewer than five
// blocks use fewer waves per row tile (a power of two >= kb) and more row tiles.
//
// Per block a wave loads its rows' codes and its tokens' activations row-coalesced (a row
// per lane, the MFMA operand order, would fetch 16-byte pieces of 16 rows in one load),
// rearranges both through its own LDS area into operand order, and issues the next block's
// loads as soon as the registers or the area are free.
//
// Bound: a large matrix at up to 16 tokens by its weight stream (32768 x 4096, 16 tokens:
// 16.4 us for 68 MB, where the VALU pass took 41.8; two planes 17.8 against 89.1), more
// tokens by the bytes a compute unit can pull for its tile (2048 x 4096, 509 tokens: 14.2 us
// with 64 x 64 tiles, 16.3 with 64 rows x 32 tokens, VALU pass 142.6).
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>

#include "tq_device.hpp"
#include "tq_decode.hpp"
#include "tq_internal.hpp"

namespace tq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr;

constexpr int kDmWaves = 8;
constexpr uint32_t kDmOob = 0x80000000u;  // past every resource below: reads zero, no memory access

template <int MTT, int RT>
struct DmShape {
  static constexpr int TOK = 16 * MTT, ROWS = 16 * RT;
  // partial results [token][row], rows padded by 4 floats: the four token rows that a wave
  // writes at once then fall in different banks
  static constexpr int PS = ROWS + 4;
  static constexpr int kActs = TOK * 256, kPart = TOK * PS * 4;
  static constexpr int kWave = kActs > kPart ? kActs : kPart;  // the same LDS, one after the other
};

// Order of LDS accesses of one wave (they complete in issue order): only the compiler has
// to keep it.
__device__ __forceinline__ void wave_lds_fence() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_wave_barrier();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// s_waitcnt with only the vector-memory count constrained (gfx9 encoding: vmcnt in bits
// 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt out of range");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// ---------------------------------------------------------------------------------
// MXFP4 on the scaled fp8 x fp4 MFMA. The released bytes are its fp4 operand as they are: a
// lane's 16-byte chunk is 32 codes with their own e8m0 scale. The int8 activations go in as
// two fp8 (e4m3) operands, q = 16 h + l with l = q & 15 and h = q >> 4: both at most four
// significant bits, so exact, as is every product. Each has its own fp32 accumulator: a block's
// low halves add up to at most 256 x 15 x 12 (doubled codes, < 2^15.5) and its high halves to
// 256 x 8 x 12, in units of half the block's least scale; while the row block's scales span at
// most 2^8, every partial sum is below 2^24 of these units, so both come out exact whatever the
// unit's order, and their sum is rounded once. (One accumulator for both would keep that only to
// a span of 2^5.) A row block of a wider span, or of scales outside 2^+-63, goes in groups of
// nine powers of two from its largest scale down, each exact and rounded once: the codes of the
// other chunks as zeros, the scales relative to the group's. A wave that meets such a block goes
// on from it in a second copy of the loop, so that the first keeps its registers (scales within
// 2^8, random over 2^9 and over 2^20, VALU pass: 32768 x 4096, 4 tokens 19.4, 23.1, 25.6 and 35.4
// us; 2048 x 4096, 509 tokens 23.1, 30.8, 35.6 and 150; whole-number sums scaled chunk by chunk,
// in a pass of their own from the first block on, took 36.5 and 47.5). Against 64 bits, in parts
// of the result's norm, 512 x 16384 and 2048 x 4096: 7.2e-8 and 5.6e-8 for scales within 2^8, 7.9e-8
// and 6.4e-8 over 2^20; VALU pass 8.5e-8 and 7.3e-8 (chunk by chunk into one sum, over 2^20: 15e-8
// and 8.7e-8).
// ---------------------------------------------------------------------------------

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t max_u16x2(uint32_t a, uint32_t b) {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}

// Four table entries by the 4-bit index whose low three bits are in the bytes of idx7 (0..7)
// and whose top bit is bit 7 of the bytes of top.
__device__ __forceinline__ int lut16(uint32_t t0, uint32_t t1, uint32_t t2, uint32_t t3, uint32_t idx7, uint32_t top) {
  const uint32_t p = __builtin_amdgcn_perm(t1, t0, idx7), n = __builtin_amdgcn_perm(t3, t2, idx7);
  const uint32_t m = __builtin_amdgcn_perm(top, top << 8, kSignSel);
  return (int)((n & m) | (p & ~m));
}
// Four signed bytes q as fp8: l = q & 15 (0 .. 15; e4m3's bytes 0 .. 15 are the values
// 0 .. 15 times 2^-9 as they are) and h = q >> 4 (-8 .. 7).
constexpr int kLoScale = 127 + 9, kHiScale = 127 + 4;
__device__ __forceinline__ int fp8_lo(uint32_t q) { return (int)(q & 0x0F0F0F0Fu); }
__device__ __forceinline__ int fp8_hi(uint32_t q) {
  return lut16(0x44403800u, 0x4E4C4A48u, 0xCACCCED0u, 0xB8C0C4C8u, (q >> 4) & 0x07070707u, q);
}

// A lane's operand of the tokens for one MFMA of 128 columns (four chunks). The lane (li, g)
// of an fp8 operand holds K positions 16 g .. 16 g + 15 and 64 + 16 g .., so half hf is bytes
// 8 (g & 1) .. + 7 of both 16-byte columns (a: elements 0..15, b: 16..31) of chunk
// 2 hf + (g >> 1), in the order of the chunk's nibbles (element i, then 16 + i).
__device__ __forceinline__ void mx_acts(const uint2 a, const uint2 b, int hf, v8i& lo, v8i& hi) {
  const uint32_t av[2] = {a.x, a.y}, bv[2] = {b.x, b.y};
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const uint32_t e0 = __builtin_amdgcn_perm(bv[m], av[m], 0x05010400u);
    const uint32_t e1 = __builtin_amdgcn_perm(bv[m], av[m], 0x07030602u);
    lo[4 * hf + 2 * m] = fp8_lo(e0);
    lo[4 * hf + 2 * m + 1] = fp8_lo(e1);
    hi[4 * hf + 2 * m] = fp8_hi(e0);
    hi[4 * hf + 2 * m + 1] = fp8_hi(e1);
  }
}

// The partial results of the workgroup's waves -> y. 2^lnw waves share a row tile.
template <int MTT, int RT>
__device__ __forceinline__ void dm_combine(const uint8_t* s_wave, int lnw, int64_t wg_row0, int n, int t0, int t,
                                           float* __restrict__ y) {
  using S = DmShape<MTT, RT>;
  constexpr int OUT = S::TOK * S::ROWS;
  for (int o = threadIdx.x; o < (OUT << (3 - lnw)); o += kDmWaves * 64) {
    const int rg = o / OUT, r = o % S::ROWS, tok = (o % OUT) / S::ROWS;
    const int64_t row = wg_row0 + rg * S::ROWS + r;
    const auto p = [&](int j) {
      return *reinterpret_cast<const float*>(s_wave + ((rg << lnw) + j) * S::kWave + (tok * S::PS + r) * 4);
    };
    float v = p(0);
    if (lnw >= 1) v += p(1);
    if (lnw >= 2) v += p(2) + p(3);
    if (lnw >= 3) v += (p(4) + p(5)) + (p(6) + p(7));
    if (row < n && t0 + tok < t) y[(int64_t)(t0 + tok) * n + row] = v;
  }
}

// FMT 0: folded codes, f16 scales. FMT 1: two planes, f16 scale pairs. FMT 2: MXFP4, e8m0
// scales. DBG: the instance that stores the exact block sums (so that the others carry no store
// addresses). NT: nontemporal weight loads.
template <int FMT, int MTT, int RT, bool DBG, bool NT>
__global__ __launch_bounds__(kDmWaves * 64) __attribute__((amdgpu_waves_per_eu(MTT == 1 && (FMT != 2 || RT == 1) && !DBG ? 4 : 2))) void k_gemv_mfma(
    const uint8_t* __restrict__ codes, const void* __restrict__ scales, int n, int kb, int lnw,
    const int8_t* __restrict__ q, const float* __restrict__ d, int t, float* __restrict__ y,
    int32_t* __restrict__ isum_dbg) {
  using S = DmShape<MTT, RT>;
  constexpr bool MX = FMT == 2;
  constexpr int NP = FMT == 1 ? 2 : 1, SH = FMT == 1 ? 6 : 4, SB = MX ? 8 : (FMT == 1 ? 4 : 2);
  constexpr int AUX = NT ? kBufNT : 0;
  constexpr int NB = MTT <= 2 && RT > 1 ? 2 : 1;  // row tiles in LDS at once
  __shared__ __attribute__((aligned(16))) uint8_t s_wave[kDmWaves * S::kWave];
  // (one variable per area, so that the compiler can tell them from the one being refilled)
  __shared__ __attribute__((aligned(16))) uint8_t s_bt0[kDmWaves * 2048];
  __shared__ __attribute__((aligned(16))) uint8_t s_bt1[NB > 1 ? kDmWaves * 2048 : 16];
  __shared__ __attribute__((aligned(16))) uint32_t s_sd[kDmWaves][128];  // a wave's token scales, row scales
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int kg = wv & ((1 << lnw) - 1);
  const int64_t wg_row0 = (int64_t)blockIdx.x * (S::ROWS << (3 - lnw));
  const int64_t row0 = wg_row0 + (wv >> lnw) * S::ROWS;
  const int64_t rowc = min(row0, (int64_t)n - 1);  // (a row tile past n reads the last row)
  const int nrows = (int)min((int64_t)S::ROWS, n - rowc);
  const __amdgpu_buffer_rsrc_t cr = make_rsrc(codes + rowc * kb * 128, (uint32_t)(nrows * kb * 128));
  const __amdgpu_buffer_rsrc_t sr =
      make_rsrc(reinterpret_cast<const uint8_t*>(scales) + rowc * kb * SB, (uint32_t)(nrows * kb * SB));
  uint8_t* const sa = s_wave + wv * S::kWave;
  uint8_t* const bt0 = s_bt0 + wv * 2048;
  uint8_t* const bt1 = NB > 1 ? s_bt1 + wv * 2048 : bt0;
  uint32_t* const ssd = s_sd[wv];
  // lane offsets of the loads below
  uint32_t vx[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) vx[e] = (uint32_t)(g * kb * 256 + ((li ^ (4 * e + g)) * 16));
  const uint32_t vw = (uint32_t)((lane >> 3) * kb * 128 + (lane & 7) * 16);
  const uint32_t vd = lane < S::TOK ? (uint32_t)(lane * kb * 4) : kDmOob;
  const uint32_t vs = lane < S::ROWS ? (uint32_t)(lane * kb * SB) : kDmOob;
  const uint32_t ve = (uint32_t)(li * kb * 8 + g);

  for (int tt = blockIdx.y; (int64_t)tt * S::TOK < t; tt += gridDim.y) {
    const int t0 = tt * S::TOK, ntok = min(S::TOK, t - t0);
    const __amdgpu_buffer_rsrc_t qr = make_rsrc(q + (int64_t)t0 * kb * 256, (uint32_t)(ntok * kb * 256));
    const __amdgpu_buffer_rsrc_t dr = make_rsrc(d + (int64_t)t0 * kb, (uint32_t)(ntok * kb * 4));
    // Block b. Activations: straight to LDS, 1 KB (token rows 4e .. 4e + 3) a load, 16-byte
    // column c of row r at column c ^ (r & 15). Weights: row 16 rt + 8c + (l >> 3), chunk
    // l & 7. Block scales of token l and row l. Rows past n, tokens past t and blocks past kb lie
    // past their resource and read as zero. Scalar offsets stay below the resource's size (rows
    // and blocks clamped), as its range check subtracts them, so a load that begins past the last
    // row or token reads that one again for its first, whose results are not stored; a block past
    // kb takes kDmOob as the lane's offset.
    constexpr int kAfterX = MX ? 4 * RT + 1 : 2 * RT + 2;  // loads per block issued after the activations'
    uint4 W[RT][2];
    uint32_t E[MX ? RT : 1][2];  // MXFP4: the scales of row 16 rt + li, chunks g and 4 + g (bytes: any alignment)
    uint32_t sc;
    float dd;
    const auto fetch_x = [&](int b) {
#pragma unroll
      for (int e = 0; e < 4 * MTT; ++e)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(qr, (lds_ptr)(sa + e * 1024), 16, b < kb ? vx[e & 3] : kDmOob,
                                                 (min(4 * e, ntok - 1) * kb + min(b, kb - 1)) * 256, 0, 0);
    };
    const auto fetch_sd = [&](int b) {
      const uint32_t so = (uint32_t)min(b, kb - 1);
      dd = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(dr, b < kb ? vd : kDmOob, so * 4u, 0));
      if constexpr (MX) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            E[rt][c] = __builtin_amdgcn_raw_buffer_load_b8(sr, b < kb ? ve + 4 * c : kDmOob,
                                                           (uint32_t)(min(16 * rt, nrows - 1) * kb + min(b, kb - 1)) * 8u, 0);
      } else if constexpr (FMT == 1) sc = __builtin_amdgcn_raw_buffer_load_b32(sr, b < kb ? vs : kDmOob, so * SB, 0);
      else sc = buf_load_u16(sr, b < kb ? vs : kDmOob, so * SB);
    };
    const auto fetch_w = [&](int b, int rt) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
        W[rt][c] = buf_load16(cr, b < kb ? vw : kDmOob,
                              (uint32_t)((min(16 * rt + 8 * c, nrows - 1) * kb + min(b, kb - 1)) * 128), AUX);
    };
    fetch_x(kg);
    __builtin_amdgcn_sched_barrier(0);  // (the wait below counts the loads issued after these)
    fetch_sd(kg);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) fetch_w(kg, rt);
    __builtin_amdgcn_sched_barrier(0);

    float acc[MTT][RT][4];
#pragma unroll
    for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[mt][rt][v] = 0.0f;

    // codes of row tile rt into operand order: chunk x of row r at chunk x ^ ((r >> 1) & 7)
    const auto stage = [&](int b, int rt, uint4 (&w)[2]) {
      uint8_t* const p = rt % NB ? bt1 : bt0;
      const int wr = lane >> 3;
      wave_lds_fence();
#pragma unroll
      for (int c = 0; c < 2; ++c)
        *reinterpret_cast<uint4*>(p + (8 * c + wr) * 128 + (((lane & 7) ^ (((8 * c + wr) >> 1) & 7)) * 16)) = W[rt][c];
      wave_lds_fence();
      const int rs = (li >> 1) & 7;
      w[0] = *reinterpret_cast<const uint4*>(p + li * 128 + ((g ^ rs) * 16));
      w[1] = *reinterpret_cast<const uint4*>(p + li * 128 + (((4 + g) ^ rs) * 16));
      fetch_w(b + kDmWaves, rt);
    };
    if constexpr (MX) {
      // One block, whose loads are issued. FAR: rows of any scales; else false, with nothing taken,
      // where a row's scales are too far apart or too large or small.
      const auto block = [&](int b, auto far_tag) -> bool {
        constexpr bool FAR = decltype(far_tag)::value;
        wait_vmcnt<kAfterX>();  // the block's activations are in LDS (its scales and codes may not be here yet)
        wave_lds_fence();
        uint2 xa[MTT][2][2], xb[MTT][2][2];
#pragma unroll
        for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const uint8_t* const row = sa + (mt * 16 + li) * 256;
              const int col = 2 * (4 * c + 2 * h + (g >> 1));
              xa[mt][c][h] = *reinterpret_cast<const uint2*>(row + ((col ^ li) * 16) + 8 * (g & 1));
              xb[mt][c][h] = *reinterpret_cast<const uint2*>(row + (((col + 1) ^ li) * 16) + 8 * (g & 1));
            }
        ssd[lane] = __float_as_uint(dd);
        wave_lds_fence();
        float4 d4[MTT];
#pragma unroll
        for (int mt = 0; mt < MTT; ++mt) d4[mt] = *reinterpret_cast<const float4*>(&ssd[mt * 16 + 4 * g]);
        wave_lds_fence();
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));  // LDS reads done: the area may be refilled
        wave_lds_fence();
        // The block's scales, and (a bit per row tile) whether those of the lane's row span more
        // than 2^8 (the unit's sums need not be exact then) or any is outside 2^+-63 (they could
        // overflow, or lose bits that d brings back). Halves: E and 255 - E, maxima over the row's
        // eight chunks.
        uint32_t es[RT][2], far = 0;
        uint32_t top[RT];  // the row's largest
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          es[rt][0] = E[rt][0];
          es[rt][1] = E[rt][1];
          const auto halves = [](uint32_t e) { return e * 0xFFFF0001u + 0x00FF0000u; };  // e | (255 - e) << 16
          uint32_t m = max_u16x2(halves(es[rt][0]), halves(es[rt][1]));
          m = max_u16x2(m, (uint32_t)lane_xor_i<16>((int)m));
          m = max_u16x2(m, (uint32_t)lane_xor_i<32>((int)m));
          top[rt] = m & 0xFFFFu;
          const uint32_t low = 255u - (m >> 16);
          far |= (uint32_t)((rt * 16 + li < nrows) & ((top[rt] > 190u) | (low < 64u) | (top[rt] - low > 8u))) << rt;
        }
        if (!FAR && __any(far)) return false;
        fetch_x(b + kDmWaves);
        __builtin_amdgcn_sched_barrier(0);
        fetch_sd(b + kDmWaves);
        uint4 wt[2][2];
        const auto stage_w = [&](int rt) { stage(b, rt, wt[rt & 1]); };
        v8i alo[MTT][2], ahi[MTT][2];
#pragma unroll
        for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
          for (int c = 0; c < 2; ++c) {
#pragma unroll
            for (int h = 0; h < 2; ++h) mx_acts(xa[mt][c][h], xb[mt][c][h], h, alo[mt][c], ahi[mt][c]);
            // (one after the other: all at once they take more registers than this loop has)
            if constexpr (FAR) asm volatile("" : "+v"(alo[mt][c]), "+v"(ahi[mt][c]));
          }
        // one row tile's products with the codes w and the scales s: each sum exact
        const auto products = [&](const uint4 (&w)[2], const uint32_t (&s)[2], v4f (&C)[MTT]) {
          v4f Ch[MTT];
#pragma unroll
          for (int mt = 0; mt < MTT; ++mt) C[mt] = Ch[mt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const v8i bw = {(int)w[c].x, (int)w[c].y, (int)w[c].z, (int)w[c].w, 0, 0, 0, 0};
#pragma unroll
            for (int mt = 0; mt < MTT; ++mt)
              C[mt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(alo[mt][c], bw, C[mt], 0, 4, 0, kLoScale, 0, (int)s[c]);
#pragma unroll
            for (int mt = 0; mt < MTT; ++mt)
              Ch[mt] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(ahi[mt][c], bw, Ch[mt], 0, 4, 0, kHiScale, 0, (int)s[c]);
          }
#pragma unroll
          for (int mt = 0; mt < MTT; ++mt) C[mt] = C[mt] + Ch[mt];
        };
        if constexpr (!FAR) {
          stage_w(0);
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            if (rt + 1 < RT) stage_w(rt + 1);
            v4f C[MTT];
            products(wt[rt & 1], es[rt], C);
#pragma unroll
            for (int mt = 0; mt < MTT; ++mt) {
              const float dv[4] = {d4[mt].x, d4[mt].y, d4[mt].z, d4[mt].w};
#pragma unroll
              for (int v = 0; v < 4; ++v) acc[mt][rt][v] = fmaf(dv[v], C[mt][v], acc[mt][rt][v]);
            }
          }
        } else {
          // A far row takes its chunks in groups: scales 2^0 .. 2^-8 of its largest, 2^-9 .. 2^-17
          // and so on, each group's sum exact and relative to the group; added up, largest first,
          // they meet d once, as a near row's. The other rows take all theirs in the first round,
          // as above: a row's result is its own, whatever its neighbours' scales. (Two independent
          // chains a round: two token tiles or two row tiles.)
          constexpr int RP = RT < 2 || MTT > 1 ? 1 : 2;
#pragma unroll
          for (int r0 = 0; r0 < RT; r0 += RP) {
            uint32_t grp[RP][2];
            v4f sum[RP][MTT];
#pragma unroll
            for (int r = 0; r < RP; ++r) {
              const int rt = r0 + r;
              stage_w(rt);
              if constexpr (DBG) {
                // the chunks' whole-number sums, two chunks (lanes g < 2, g >= 2) at a time, each with
                // the other's codes as zeros: the activations stand in the order of the scaled operand
                const uint8_t* const p = (rt % NB ? bt1 : bt0) + li * 128 + 8 * (g & 1);
#pragma unroll
                for (int c = 0; c < 2; ++c)
#pragma unroll
                  for (int h = 0; h < 2; ++h) {
                    const int j0 = 4 * c + 2 * h;
                    const uint2 x = *reinterpret_cast<const uint2*>(p + (((j0 + (g >> 1)) ^ ((li >> 1) & 7)) * 16));
                    const uint2 wl = {(uint32_t)mx_dec4(x.x & 0x07070707u, x.x << 4), (uint32_t)mx_dec4(x.y & 0x07070707u, x.y << 4)};
                    const uint2 wh = {(uint32_t)mx_dec4((x.x >> 4) & 0x07070707u, x.x), (uint32_t)mx_dec4((x.y >> 4) & 0x07070707u, x.y)};
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                      const bool own = (g >> 1) == j;
                      const long bl = own ? __builtin_bit_cast(long, wl) : 0, bh = own ? __builtin_bit_cast(long, wh) : 0;
#pragma unroll
                      for (int mt = 0; mt < MTT; ++mt) {
                        v4i C = {0, 0, 0, 0};
                        C = __builtin_amdgcn_mfma_i32_16x16x32_i8(__builtin_bit_cast(long, xa[mt][c][h]), bl, C, 0, 0, 0);
                        C = __builtin_amdgcn_mfma_i32_16x16x32_i8(__builtin_bit_cast(long, xb[mt][c][h]), bh, C, 0, 0, 0);
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                          const int tok = mt * 16 + 4 * g + v, r = rt * 16 + li;
                          if (tok < ntok && row0 + r < n)
                            isum_dbg[((int64_t)(t0 + tok) * n + row0 + r) * (kb * 8) + b * 8 + j0 + j] = C[v];
                        }
                      }
                    }
                  }
              }
              const bool fr = (far >> rt) & 1u;
              // (x * 57 >> 9 is x / 9 for a byte x)
              const auto group = [&](uint32_t e) { return (uint32_t)__mul24(fr ? top[rt] - e : 0u, 57) >> 9; };
              grp[r][0] = group(es[rt][0]);
              grp[r][1] = group(es[rt][1]);
#pragma unroll
              for (int mt = 0; mt < MTT; ++mt) sum[r][mt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            }
            uint32_t p = 0;
            do {
#pragma unroll
              for (int r = 0; r < RP; ++r) {
                const int rt = r0 + r;
                const uint32_t unit = (far >> rt) & 1u ? top[rt] - 9 * p - 128 : 0u;
                uint4 w[2];
                uint32_t s[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                  const bool take = grp[r][c] == p;
                  const uint4 z = wt[rt & 1][c];
                  w[c] = make_uint4(take ? z.x : 0u, take ? z.y : 0u, take ? z.z : 0u, take ? z.w : 0u);
                  s[c] = take ? es[rt][c] - unit : 127u;
                }
                v4f C[MTT];
                products(w, s, C);
#pragma unroll
                for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
                  for (int v = 0; v < 4; ++v) sum[r][mt][v] += ldexpf(C[mt][v], -9 * (int)p);
              }
              ++p;
            } while (__any(p <= (RP > 1 ? max(max(grp[0][0], grp[0][1]), max(grp[RP - 1][0], grp[RP - 1][1]))
                                        : max(grp[0][0], grp[0][1]))));
#pragma unroll
            for (int r = 0; r < RP; ++r) {
              const int rt = r0 + r, sh = (far >> rt) & 1u ? (int)top[rt] - 128 : 0;
#pragma unroll
              for (int mt = 0; mt < MTT; ++mt) {
                const float dv[4] = {d4[mt].x, d4[mt].y, d4[mt].z, d4[mt].w};
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[mt][rt][v] = fmaf(ldexpf(dv[v], sh), sum[r][mt][v], acc[mt][rt][v]);
              }
            }
          }
        }
        return true;
      };
      int b = kg;
      if constexpr (!DBG)
        while (b < kb && block(b, std::false_type{})) b += kDmWaves;
      for (; b < kb; b += kDmWaves) block(b, std::true_type{});  // (on from the first such block)
    } else {
      for (int b = kg; b < kb; b += kDmWaves) {
        wait_vmcnt<kAfterX>();  // the block's activations are in LDS (its scales and codes may not be here yet)
        wave_lds_fence();
        v4i aop[MTT][2][2];
#pragma unroll
        for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const uint8_t* const row = sa + (mt * 16 + li) * 256;
              aop[mt][c][h] = *reinterpret_cast<const v4i*>(row + (((2 * (4 * c + g) + h) ^ li) * 16));
            }
        ssd[lane] = __float_as_uint(dd);
        ssd[64 + lane] = sc;
        wave_lds_fence();
        float4 d4[MTT];
#pragma unroll
        for (int mt = 0; mt < MTT; ++mt) d4[mt] = *reinterpret_cast<const float4*>(&ssd[mt * 16 + 4 * g]);
        uint32_t scr[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) scr[rt] = ssd[64 + rt * 16 + li];
        wave_lds_fence();
        __builtin_amdgcn_s_waitcnt(15 | (7 << 4) | (0 << 8) | (3 << 14));  // LDS reads done: the area may be refilled
        wave_lds_fence();
        fetch_x(b + kDmWaves);
        __builtin_amdgcn_sched_barrier(0);
        fetch_sd(b + kDmWaves);
        uint4 wt[2][2];
        const auto stage_w = [&](int rt) { stage(b, rt, wt[rt & 1]); };
        stage_w(0);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          if (rt + 1 < RT) stage_w(rt + 1);  // its LDS round trip runs beside this tile's MFMAs
          v4i bop[NP][2][2];
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            const uint4 w = wt[rt & 1][c];
            int u[8];
            if constexpr (FMT == 1) unpack64t(w.x, w.y, u);
            else unpack16c(w, u);
            bop[0][c][0] = v4i{u[0], u[1], u[2], u[3]};
            bop[0][c][1] = v4i{u[4], u[5], u[6], u[7]};
            if constexpr (FMT == 1) {
              unpack64t(w.z, w.w, u);
              bop[NP - 1][c][0] = v4i{u[0], u[1], u[2], u[3]};
              bop[NP - 1][c][1] = v4i{u[4], u[5], u[6], u[7]};
            }
          }
          const float s1 = f16_bits_to_f32((uint16_t)(scr[rt] & 0xFFFFu));
          const float s2 = FMT == 1 ? f16_bits_to_f32((uint16_t)(scr[rt] >> 16)) : 0.0f;
          v4i C[MTT][NP];
#pragma unroll
          for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
            for (int p = 0; p < NP; ++p) C[mt][p] = v4i{0, 0, 0, 0};
#pragma unroll
          for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
                for (int p = 0; p < NP; ++p)
                  C[mt][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(aop[mt][c][h], bop[p][c][h], C[mt][p], 0, 0, 0);
          // token mt * 16 + 4g + v, row rt * 16 + li: the exact block sums, then one fp32
          // multiply-add per plane
#pragma unroll
          for (int mt = 0; mt < MTT; ++mt) {
            const float dv[4] = {d4[mt].x, d4[mt].y, d4[mt].z, d4[mt].w};
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              acc[mt][rt][v] = fmaf(s1 * dv[v], (float)(C[mt][0][v] >> SH), acc[mt][rt][v]);
              if constexpr (FMT == 1)
                acc[mt][rt][v] = fmaf(s2 * dv[v], (float)(C[mt][NP - 1][v] >> SH), acc[mt][rt][v]);
            }
          }
          if constexpr (DBG) {
#pragma unroll
            for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int tok = mt * 16 + 4 * g + v, r = rt * 16 + li;
                if (tok < ntok && row0 + r < n) {
                  int32_t* o = isum_dbg + (((int64_t)(t0 + tok) * n + row0 + r) * kb + b) * NP;
                  o[0] = C[mt][0][v] >> SH;
                  if constexpr (FMT == 1) o[1] = C[mt][NP - 1][v] >> SH;
                }
              }
          }
        }
      }
    }
    // (the last, empty refills of the activations have landed before the area is reused)
    wait_vmcnt<0>();
    wave_lds_fence();
    float* const pw = reinterpret_cast<float*>(sa);
#pragma unroll
    for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) pw[(mt * 16 + 4 * g + v) * S::PS + rt * 16 + li] = acc[mt][rt][v];
    __syncthreads();
    dm_combine<MTT, RT>(s_wave, lnw, wg_row0, n, t0, t, y);
    __syncthreads();  // the next token tile's activations take the partial results' place
  }
}

template <typename F, typename... A>
static void dm_launch(F k, dim3 grid, hipStream_t st, void* const* events, A... args) {
  if (events)
    hipExtLaunchKernelGGL(k, grid, dim3(kDmWaves * 64), 0, st, (hipEvent_t)events[0], (hipEvent_t)events[1], 0, args...);
  else
    hipLaunchKernelGGL(k, grid, dim3(kDmWaves * 64), 0, st, args...);
}

void launch_gemv_mfma(int fmt, const uint8_t* codes, const void* scales, int n, int kb, const int8_t* q, const float* d,
                      int t, float* y, int32_t* isum_dbg, hipStream_t st, void* const* events) {
  const int lnw = kb >= 5 ? 3 : (kb >= 3 ? 2 : kb - 1);
  // Tiles (16-token tiles x 16-row tiles), largest first: the largest with a workgroup for
  // every compute unit, else the smallest (2048 x 4096, 64 tokens: 6.8 us at 1 x 1 (512
  // workgroups), 5.6 at 2 x 1 (256), 6.2 at 2 x 2 (128), 8.3 at 2 x 4; 8192 x 4096, 128
  // tokens: 37.6 at 1 x 1, 18.3 at 2 x 4, 15.2 at 4 x 4). A larger tile reads fewer bytes per
  // output; one of more 16-token tiles than t fills computes padding. (Two planes: 4 x 4
  // does not fit the registers.)
  struct Tile { int mtt, rt; };
  static constexpr Tile kTiles[] = {{4, 4}, {2, 4}, {2, 2}, {2, 1}, {1, 2}, {1, 1}};
  static constexpr Tile kTilesMx[] = {{2, 4}, {2, 2}, {2, 1}, {1, 4}, {1, 2}, {1, 1}};  // (the last three up to 16 tokens)
  const Tile* tiles = fmt == 2 ? kTilesMx : (fmt == 0 ? kTiles : kTiles + 1);
  const auto wgs = [&](int rt) { return ((((int64_t)n + 16 * rt - 1) / (16 * rt)) + (1 << (3 - lnw)) - 1) >> (3 - lnw); };
  const auto ttiles = [&](int mtt) { return ((int64_t)t + 16 * mtt - 1) / (16 * mtt); };
  while ((tiles->mtt > 1 && t <= 8 * tiles->mtt) || (tiles->mtt * tiles->rt > 1 && wgs(tiles->rt) * ttiles(tiles->mtt) < 256))
    ++tiles;
  // MXFP4 at 16 tokens and fewer: the activations' split into fp8 pairs costs about as much as four
  // row tiles' MFMAs, so a compute unit's share counts, workgroups by the cost of one (1 x 1 5,
  // 1 x 2 10, 1 x 4 17): with 4 tokens 1 x 4 takes 19.5 us at 32768 x 4096 (1 x 2 22.0, 1 x 1 23.3)
  // and 9.8 at 16384 x 4096 (11.1, 12.2), 1 x 2 6.4 at 8192 x 4096 (1 x 4 9.8), and where a few
  // workgroups would begin another round 1 x 1: 8205 x 4096 8.8 (1 x 2 10.0, 1 x 4 9.7, VALU chunks
  // with their own tile for it 8.5), 16610 x 1024 7.1 (8.0, 6.7, 7.2), 33000 x 1024 9.8 (11.2, 12.0, 11.3).
  if (fmt == 2 && t <= 16) {
    const auto cost = [&](int rt) { return (wgs(rt) + 255) / 256 * (rt == 4 ? 17 : 5 * rt); };
    tiles = kTilesMx + (cost(4) <= std::min(cost(2), cost(1)) ? 3 : (cost(2) <= cost(1) ? 4 : 5));
  }
  // The block sums' addresses take registers of their own: their instances go up to the tiles
  // that hold them without spilling (4 x 4 would spill 315).
  const int mtt = isum_dbg ? std::min(tiles->mtt, fmt == 2 ? 1 : 2) : tiles->mtt;
  const int rt = isum_dbg ? std::min(tiles->rt, 2) : tiles->rt;
  const int64_t ntt = ttiles(mtt);
  // several token tiles: a multiple of 8 row tiles, so that a row tile's workgroups share an XCD
  // (520 x 16384, 200 tokens: 16.9 us, 22.1 without; the workgroups past n run their blocks for
  // nothing: returning at once takes 15.8 there, but the wait for n ahead of the first loads 13.7
  // for 13.1 at 2048 x 4096, 509 tokens)
  const int64_t gx = ntt > 1 ? (wgs(rt) + 7) / 8 * 8 : wgs(rt);
  const dim3 grid((unsigned)gx, (unsigned)(ntt < 16384 ? ntt : 16384));
  // 16-token tiles read the weights nontemporally where few tiles read them again (each call
  // another matrix, folded, us so and not: 512 x 16384, 64 tokens 9.6 and 9.9; 2048 x 4096, 24 tokens
  // 4.65 and 4.9; 512 x 4096, 100 tokens 4.6 and 4.2; 256 x 4096, 300 tokens 6.4 and 5.9)
  const bool nt = ntt <= 4;
#define TQ_DM(F, M, R, D) \
  dm_launch(nt && M == 1 && !D ? k_gemv_mfma<F, M, R, D, M == 1 && !D> : k_gemv_mfma<F, M, R, D, false>, grid, st, events, \
            codes, scales, n, kb, lnw, q, d, t, y, isum_dbg)
  switch ((isum_dbg ? 1000 : 0) + fmt * 100 + mtt * 10 + rt) {
    case 11: TQ_DM(0, 1, 1, false); break;
    case 12: TQ_DM(0, 1, 2, false); break;
    case 21: TQ_DM(0, 2, 1, false); break;
    case 22: TQ_DM(0, 2, 2, false); break;
    case 24: TQ_DM(0, 2, 4, false); break;
    case 44: TQ_DM(0, 4, 4, false); break;
    case 111: TQ_DM(1, 1, 1, false); break;
    case 112: TQ_DM(1, 1, 2, false); break;
    case 121: TQ_DM(1, 2, 1, false); break;
    case 122: TQ_DM(1, 2, 2, false); break;
    case 124: TQ_DM(1, 2, 4, false); break;
    case 211: TQ_DM(2, 1, 1, false); break;
    case 212: TQ_DM(2, 1, 2, false); break;
    case 214: TQ_DM(2, 1, 4, false); break;
    case 221: TQ_DM(2, 2, 1, false); break;
    case 222: TQ_DM(2, 2, 2, false); break;
    case 224: TQ_DM(2, 2, 4, false); break;
    case 1011: TQ_DM(0, 1, 1, true); break;
    case 1012: TQ_DM(0, 1, 2, true); break;
    case 1021: TQ_DM(0, 2, 1, true); break;
    case 1022: TQ_DM(0, 2, 2, true); break;
    case 1111: TQ_DM(1, 1, 1, true); break;
    case 1112: TQ_DM(1, 1, 2, true); break;
    case 1121: TQ_DM(1, 2, 1, true); break;
    case 1122: TQ_DM(1, 2, 2, true); break;
    case 1211: TQ_DM(2, 1, 1, true); break;
    default: TQ_DM(2, 1, 2, true); break;
  }
#undef TQ_DM
}

}  // namespace tq
