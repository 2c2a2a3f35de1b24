// Per-256 activation quantizer (Sec. 2.2: the codes meet int8 activations that carry one
// scale per block; the block/scale/rounding rule is this library's reading, stated in tq.h).
#include "tq_device.hpp"
#include "tq_internal.hpp"

namespace tq {

__global__ __launch_bounds__(256) void k_quantize(const float* __restrict__ x, int64_t nblocks,
                                                  int8_t* __restrict__ q, float* __restrict__ d,
                                                  int32_t* __restrict__ bsum) {
  quantize_wave_blocks(x, nblocks, (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), q, d, bsum);
}

hipError_t launch_quantize(const float* x, int64_t t, int32_t k, int8_t* q, float* d, int32_t* bsum,
                           hipStream_t st) {
  const int64_t nblocks = t * (k / 256);
  if (nblocks == 0) return hipSuccess;
  const int64_t wgs = (nblocks + 15) / 16;
  hipLaunchKernelGGL(k_quantize, dim3((unsigned)wgs), dim3(256), 0, st, x, nblocks, q, d, bsum);
  return hipSuccess;
}

}  // namespace tq

extern "C" tq_status tq_quantize_act(const float* x, int64_t t, int32_t k, int8_t* q, float* d,
                                     int32_t* bsum, void* stream) {
  using namespace tq;
  clear_error();
  if (t < 0) return fail(TQ_ERR_INVALID, "tq_quantize_act: t = %lld < 0", (long long)t);
  if (k <= 0 || k % 256 != 0 || k > kMaxK)
    return fail(TQ_ERR_INVALID, "tq_quantize_act: k = %d must be a positive multiple of 256 <= %d", k, kMaxK);
  if (t == 0) return TQ_OK;
  if (!x || !q || !d || !bsum) return fail(TQ_ERR_INVALID, "tq_quantize_act: null pointer");
  if (!aligned(x, 16) || !aligned(q, 16) || !aligned(d, 4) || !aligned(bsum, 4))
    return fail(TQ_ERR_ALIGN, "tq_quantize_act: x and q must be 16-byte aligned, d and bsum 4-byte aligned");
  if (t * (int64_t)(k / 256) > (int64_t)INT32_MAX * 32)
    return fail(TQ_ERR_INVALID, "tq_quantize_act: t too large");
  (void)hipGetLastError();
  launch_quantize(x, t, k, q, d, bsum, (hipStream_t)stream);
  return check_launch("tq_quantize_act");
}
