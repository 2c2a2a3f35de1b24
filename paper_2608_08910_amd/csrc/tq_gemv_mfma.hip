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
// a token's result has the same bits whatever kernel took it. Rows of fewer than five
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

__device__ __forceinline__ float lane_get(float v, int src) {
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src << 2, __float_as_int(v)));
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

// FMT 0: folded codes, f16 scales. FMT 1: two planes, f16 scale pairs. DBG: the instance that
// stores the exact block sums (so that the others carry no store addresses).
template <int FMT, int MTT, int RT, bool DBG>
__global__ __launch_bounds__(kDmWaves * 64) __attribute__((amdgpu_waves_per_eu(MTT == 1 && !DBG ? 4 : 2))) void k_gemv_mfma(
    const uint8_t* __restrict__ codes, const void* __restrict__ scales, int n, int kb, int lnw,
    const int8_t* __restrict__ q, const float* __restrict__ d, int t, float* __restrict__ y,
    int32_t* __restrict__ isum_dbg) {
  using S = DmShape<MTT, RT>;
  constexpr int NP = FMT == 1 ? 2 : 1, SH = FMT == 1 ? 6 : 4, SB = FMT == 1 ? 4 : 2;
  constexpr int AUX = MTT == 1 ? kBufNT : 0;  // up to 16 tokens each weight byte is read once
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

  for (int tt = blockIdx.y; (int64_t)tt * S::TOK < t; tt += gridDim.y) {
    const int t0 = tt * S::TOK, ntok = min(S::TOK, t - t0);
    const __amdgpu_buffer_rsrc_t qr = make_rsrc(q + (int64_t)t0 * kb * 256, (uint32_t)(ntok * kb * 256));
    const __amdgpu_buffer_rsrc_t dr = make_rsrc(d + (int64_t)t0 * kb, (uint32_t)(ntok * kb * 4));
    // Block b. Activations: straight to LDS, 1 KB (token rows 4e .. 4e + 3) a load, 16-byte
    // column c of row r at column c ^ (r & 15). Weights: row 16 rt + 8c + (l >> 3), chunk
    // l & 7. Block scales of token l and row l. Rows past n, tokens past t and blocks past kb
    // read as zero, with no memory access. Scalar offsets stay below the resource's size (rows
    // and blocks clamped), as its range check subtracts them; a block past kb takes kDmOob as
    // the lane's offset.
    uint4 W[RT][2];
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
      if constexpr (FMT == 1) sc = __builtin_amdgcn_raw_buffer_load_b32(sr, b < kb ? vs : kDmOob, so * SB, 0);
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

    for (int b = kg; b < kb; b += kDmWaves) {
      wait_vmcnt<2 * RT + 2>();  // the block's activations are in LDS (its scales and codes may not be here yet)
      wave_lds_fence();
      v4i aop[MTT][2][2];
#pragma unroll
      for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            aop[mt][c][h] = *reinterpret_cast<const v4i*>(sa + (mt * 16 + li) * 256 + (((2 * (4 * c + g) + h) ^ li) * 16));
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
      // codes of row tile rt into operand order: chunk x of row r at chunk x ^ ((r >> 1) & 7)
      uint4 wt[2][2];
      const auto stage_w = [&](int rt) {
        uint8_t* const p = rt % NB ? bt1 : bt0;
        const int wr = lane >> 3;
        wave_lds_fence();
#pragma unroll
        for (int c = 0; c < 2; ++c)
          *reinterpret_cast<uint4*>(p + (8 * c + wr) * 128 + (((lane & 7) ^ (((8 * c + wr) >> 1) & 7)) * 16)) = W[rt][c];
        wave_lds_fence();
        const int rs = (li >> 1) & 7;
        wt[rt & 1][0] = *reinterpret_cast<const uint4*>(p + li * 128 + ((g ^ rs) * 16));
        wt[rt & 1][1] = *reinterpret_cast<const uint4*>(p + li * 128 + (((4 + g) ^ rs) * 16));
        fetch_w(b + kDmWaves, rt);
      };
      stage_w(0);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if (rt + 1 < RT) stage_w(rt + 1);  // its LDS round trip runs beside this tile's MFMAs
        v4i bop[NP][2][2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const uint4 w = wt[rt & 1][c];
          int u[8];
          if constexpr (FMT == 0) unpack16c(w, u);
          else unpack64t(w.x, w.y, u);
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

// MXFP4: a 16-byte chunk is one block of 32 with its own scale, so each 16x16x32 MFMA is
// one block's exact sums, scaled into the chunk's own accumulator (the single-token kernel's
// lane: chunk cp of the blocks b mod 8 = g), the eight of which are summed as
// ((0+1)+(2+3))+((4+5)+(6+7)) after the last block. Lane (li, g) takes dword g of each
// chunk: its low nibbles are columns 4g .. 4g + 3 and its high nibbles columns 16 + 4g ..,
// so the LDS areas hold dword-transposed rows: [row][dword g][chunk].
template <int MTT, int RT, bool DBG>
__global__ __launch_bounds__(kDmWaves * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_gemv_mfma_mx(
    const uint8_t* __restrict__ codes, const uint8_t* __restrict__ scales, int n, int kb, int lnw,
    const int8_t* __restrict__ q, const float* __restrict__ d, int t, float* __restrict__ y,
    int32_t* __restrict__ isum_dbg) {
  using S = DmShape<MTT, RT>;
  constexpr int AUX = MTT == 1 ? kBufNT : 0;
  __shared__ __attribute__((aligned(16))) uint8_t s_wave[kDmWaves * S::kWave];
  __shared__ __attribute__((aligned(16))) uint8_t s_bt[kDmWaves * 2048];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int kg = wv & ((1 << lnw) - 1);
  const int64_t wg_row0 = (int64_t)blockIdx.x * (S::ROWS << (3 - lnw));
  const int64_t row0 = wg_row0 + (wv >> lnw) * S::ROWS;
  const int64_t rowc = min(row0, (int64_t)n - 1);
  const int nrows = (int)min((int64_t)S::ROWS, n - rowc);
  const __amdgpu_buffer_rsrc_t cr = make_rsrc(codes + rowc * kb * 128, (uint32_t)(nrows * kb * 128));
  const __amdgpu_buffer_rsrc_t sr = make_rsrc(scales + rowc * kb * 8, (uint32_t)(nrows * kb * 8));
  uint8_t* const sa = s_wave + wv * S::kWave;
  uint8_t* const bt = s_bt + wv * 2048;
  // lane offsets of the loads below
  const uint32_t vx = (uint32_t)(g * kb * 256 + li * 16), vw = (uint32_t)((lane >> 3) * kb * 128 + (lane & 7) * 16);
  const uint32_t vd = lane < S::TOK ? (uint32_t)(lane * kb * 4) : kDmOob;
  const uint32_t ve = (uint32_t)(li * kb * 8 + 2 * g);

  for (int tt = blockIdx.y; (int64_t)tt * S::TOK < t; tt += gridDim.y) {
    const int t0 = tt * S::TOK, ntok = min(S::TOK, t - t0);
    const __amdgpu_buffer_rsrc_t qr = make_rsrc(q + (int64_t)t0 * kb * 256, (uint32_t)(ntok * kb * 256));
    const __amdgpu_buffer_rsrc_t dr = make_rsrc(d + (int64_t)t0 * kb, (uint32_t)(ntok * kb * 4));
    uint4 X[4 * MTT], W[RT][2];
    uint32_t E[RT][2];  // scale bytes: lane (li, g) loads chunks 2g and 2g + 1 of row li
    float dd;
    // Scalar offsets stay below the resource's size (rows and blocks clamped), as its range
    // check subtracts them; a block past kb takes kDmOob as the lane's offset.
    const auto fetch_x = [&](int b) {
      const uint32_t vo = b < kb ? vx : kDmOob;
#pragma unroll
      for (int e = 0; e < 4 * MTT; ++e)
        X[e] = buf_load16(qr, vo, (uint32_t)((min(4 * e, ntok - 1) * kb + min(b, kb - 1)) * 256), 0);
      dd = __uint_as_float(
          __builtin_amdgcn_raw_buffer_load_b32(dr, b < kb ? vd : kDmOob, (uint32_t)min(b, kb - 1) * 4u, 0));
    };
    const auto fetch_w = [&](int b, int rt) {
      // (bytes: the scales have no alignment)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        E[rt][c] = __builtin_amdgcn_raw_buffer_load_b8(
            sr, b < kb ? ve + c : kDmOob, (uint32_t)((min(16 * rt, nrows - 1) * kb + min(b, kb - 1)) * 8), 0);
#pragma unroll
      for (int c = 0; c < 2; ++c)
        W[rt][c] = buf_load16(cr, b < kb ? vw : kDmOob,
                              (uint32_t)((min(16 * rt + 8 * c, nrows - 1) * kb + min(b, kb - 1)) * 128), AUX);
    };
    fetch_x(kg);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) fetch_w(kg, rt);
    __builtin_amdgcn_sched_barrier(0);

    float acc[8][MTT][RT][4];
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int v = 0; v < 4; ++v) acc[j][mt][rt][v] = 0.0f;

    for (int b = kg; b < kb; b += kDmWaves) {
      // activations: dword u of 16-byte column c of row r at dword
      // 64 r + 16 ((u + r) & 3) + 4 ((c >> 2) ^ ((r >> 2) & 3)) + (c & 3)  (reads and writes
      // both touch every bank once)
      uint32_t* const saw = reinterpret_cast<uint32_t*>(sa);
#pragma unroll
      for (int e = 0; e < 4 * MTT; ++e) {
        const int r = 4 * e + g;
        const uint32_t xs[4] = {X[e].x, X[e].y, X[e].z, X[e].w};
#pragma unroll
        for (int u = 0; u < 4; ++u)
          saw[64 * r + 16 * ((u + r) & 3) + 4 * ((li >> 2) ^ ((r >> 2) & 3)) + (li & 3)] = xs[u];
      }
      wave_lds_fence();
      v4i av[MTT][4];  // dword i of av[mt][m]: column 4m + i's dword g
#pragma unroll
      for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
        for (int m = 0; m < 4; ++m)
          av[mt][m] = *reinterpret_cast<const v4i*>(saw + 64 * (mt * 16 + li) + 16 * ((g + li) & 3) + 4 * (m ^ ((li >> 2) & 3)));
      float d4[MTT][4];
#pragma unroll
      for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
        for (int v = 0; v < 4; ++v) d4[mt][v] = lane_get(dd, mt * 16 + 4 * g + v);
      fetch_x(b + kDmWaves);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        // codes: dword u of chunk x of row r at dword
        // 32 r + 8 ((u + (r >> 1)) & 3) + (x ^ (4 * ((r >> 3) & 1)))
        uint32_t* const btw = reinterpret_cast<uint32_t*>(bt);
        wave_lds_fence();
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int r = 8 * c + (lane >> 3), x = lane & 7;
          const uint32_t ws[4] = {W[rt][c].x, W[rt][c].y, W[rt][c].z, W[rt][c].w};
#pragma unroll
          for (int u = 0; u < 4; ++u) btw[32 * r + 8 * ((u + (r >> 1)) & 3) + (x ^ (4 * c))] = ws[u];
        }
        wave_lds_fence();
        v4i wt[2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
          wt[m] = *reinterpret_cast<const v4i*>(btw + 32 * li + 8 * ((g + (li >> 1)) & 3) + 4 * (m ^ (li >> 3)));
        // the row's eight scale bytes: chunk j's from lane (li, j / 2)
        const int epair = (int)(E[rt][0] | (E[rt][1] << 16));
        int ej[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) ej[m] = __builtin_amdgcn_ds_bpermute((16 * m + li) << 2, epair);
        fetch_w(b + kDmWaves, rt);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t w = (uint32_t)wt[j >> 2][j & 3];
          const int lo = mx_dec4(w & 0x07070707u, w << 4), hi = mx_dec4((w >> 4) & 0x07070707u, w);
          const long bop = (long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
          const int ex = ((j & 1) ? (ej[j >> 1] >> 16) : (ej[j >> 1] & 0xFFFF)) - 128;
#pragma unroll
          for (int mt = 0; mt < MTT; ++mt) {
            const uint32_t a0 = (uint32_t)av[mt][j >> 1][2 * (j & 1)], a1 = (uint32_t)av[mt][j >> 1][2 * (j & 1) + 1];
            const long aop = (long)(((uint64_t)a1 << 32) | a0);
            const v4i C = __builtin_amdgcn_mfma_i32_16x16x32_i8(aop, bop, v4i{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v)
              acc[j][mt][rt][v] = fmaf(ldexpf(d4[mt][v], ex), (float)C[v], acc[j][mt][rt][v]);
            if constexpr (DBG) {
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const int tok = mt * 16 + 4 * g + v, r = rt * 16 + li;
                if (tok < ntok && row0 + r < n) isum_dbg[((int64_t)(t0 + tok) * n + row0 + r) * (kb * 8) + b * 8 + j] = C[v];
              }
            }
          }
        }
      }
    }
    wave_lds_fence();
    float* const pw = reinterpret_cast<float*>(sa);
#pragma unroll
    for (int mt = 0; mt < MTT; ++mt)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const auto a = [&](int j) { return acc[j][mt][rt][v]; };
          pw[(mt * 16 + 4 * g + v) * S::PS + rt * 16 + li] =
              ((a(0) + a(1)) + (a(2) + a(3))) + ((a(4) + a(5)) + (a(6) + a(7)));
        }
    __syncthreads();
    dm_combine<MTT, RT>(s_wave, lnw, wg_row0, n, t0, t, y);
    __syncthreads();
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
  static constexpr Tile kTilesMx[] = {{2, 1}, {1, 2}, {1, 1}};
  const Tile* tiles = fmt == 2 ? kTilesMx : (fmt == 1 ? kTiles + 1 : kTiles);
  const auto wgs = [&](int rt) { return ((((int64_t)n + 16 * rt - 1) / (16 * rt)) + (1 << (3 - lnw)) - 1) >> (3 - lnw); };
  const auto ttiles = [&](int mtt) { return ((int64_t)t + 16 * mtt - 1) / (16 * mtt); };
  while ((tiles->mtt > 1 && t <= 8 * tiles->mtt) || (tiles->mtt * tiles->rt > 1 && wgs(tiles->rt) * ttiles(tiles->mtt) < 256))
    ++tiles;
  const int mtt = tiles->mtt, rt = tiles->rt;
  const int64_t ntt = ttiles(mtt);
  // several token tiles: a multiple of 8 row tiles, so that a row tile's workgroups share an XCD
  const int64_t gx = ntt > 1 ? (wgs(rt) + 7) / 8 * 8 : wgs(rt);
  const dim3 grid((unsigned)gx, (unsigned)(ntt < 16384 ? ntt : 16384));
  const uint8_t* s8 = reinterpret_cast<const uint8_t*>(scales);
#define TQ_DM(F, M, R)                                                                                                  \
  dm_launch(isum_dbg ? k_gemv_mfma<F, M, R, true> : k_gemv_mfma<F, M, R, false>, grid, st, events, codes, scales, n, kb, \
            lnw, q, d, t, y, isum_dbg)
#define TQ_DX(M, R)                                                                                                     \
  dm_launch(isum_dbg ? k_gemv_mfma_mx<M, R, true> : k_gemv_mfma_mx<M, R, false>, grid, st, events, codes, s8, n, kb, lnw, \
            q, d, t, y, isum_dbg)
  switch (fmt * 100 + mtt * 10 + rt) {
    case 11: TQ_DM(0, 1, 1); break;
    case 12: TQ_DM(0, 1, 2); break;
    case 21: TQ_DM(0, 2, 1); break;
    case 22: TQ_DM(0, 2, 2); break;
    case 24: TQ_DM(0, 2, 4); break;
    case 44: TQ_DM(0, 4, 4); break;
    case 111: TQ_DM(1, 1, 1); break;
    case 112: TQ_DM(1, 1, 2); break;
    case 121: TQ_DM(1, 2, 1); break;
    case 122: TQ_DM(1, 2, 2); break;
    case 124: TQ_DM(1, 2, 4); break;
    case 211: TQ_DX(1, 1); break;
    case 212: TQ_DX(1, 2); break;
    default: TQ_DX(2, 1); break;
  }
#undef TQ_DM
#undef TQ_DX
}

}  // namespace tq
