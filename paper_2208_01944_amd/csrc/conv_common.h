// Device types and helpers shared by the convolution kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace palq {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr uint32_t kOob = 0x40000000u;  // offset past any tensor these kernels accept (< 2^30 B)

}  // namespace palq
