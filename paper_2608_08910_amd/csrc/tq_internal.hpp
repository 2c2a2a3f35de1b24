// Host-side internals shared by the library's translation units (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdarg>
#include <string>

#include "../../include/tq.h"

namespace tq {

// Records a thread-local error message and returns `st`.
tq_status fail(tq_status st, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();
tq_status check_launch(const char* what);

inline bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

constexpr int kMaxK = 16384;

// Internal launchers (arguments already validated).
hipError_t launch_quantize(const float* x, int64_t t, int32_t k, int8_t* q, float* d, int32_t* bsum,
                           hipStream_t st);

// The several-token dot pass of one matrix (fmt 0 folded, 1 two planes, 2 MXFP4); events:
// null or a start and a stop event.
void launch_gemv_mfma(int fmt, const uint8_t* codes, const void* scales, int n, int kb, const int8_t* q, const float* d,
                      int t, float* y, int32_t* isum_dbg, hipStream_t st, void* const* events);

}  // namespace tq
