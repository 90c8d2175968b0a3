// Shared by the kernels of libsconv.
#pragma once

#include <hip/hip_runtime.h>

#include "sconv_internal.h"

namespace sconv {

typedef int int4v __attribute__((ext_vector_type(4)));

static __device__ __forceinline__ int fdiv(int n, FastDiv f)
{
    return f.magic ? (int)__umulhi((unsigned)n, f.magic) : n / (int)f.d;
}

} // namespace sconv
