// Compiles the library's device functions for the host (hipcc -x hip
// --cuda-host-only): functions marked __device__ become callable there, and the
// hardware operations they use get host versions.  v_rcp_f32 and v_rsq_f32 are
// within one ulp of the quotients that stand for them here.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <math.h>

static inline float host_fmed3f(float a, float b, float c) {
    if (a != a || b != b || c != c) return fminf(fminf(a, b), c);
    return fmaxf(fminf(a, b), fminf(fmaxf(a, b), c));
}
#define __builtin_amdgcn_fmed3f host_fmed3f
#define __builtin_amdgcn_rcpf(x) (1.0f / (x))
#define __builtin_amdgcn_rsqf(x) (1.0f / sqrtf(x))
#undef __device__
#define __device__ __attribute__((host)) __attribute__((device))
