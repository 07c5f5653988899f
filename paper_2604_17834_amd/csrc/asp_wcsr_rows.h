// What the kernels that walk WCSR entries share (asp_wcsr_rows.hip, asp_wcsr_groups.hip).
#pragma once

#include "asp_internal.h"

namespace asp {

namespace {

typedef __attribute__((address_space(1))) char global_char;

template <typename T, int E>
struct RowVec;
template <int E>
struct RowVec<float, E> {
    typedef float type __attribute__((ext_vector_type(E), aligned(4)));
};
template <int E>
struct RowVec<uint16_t, E> {
    typedef uint16_t type __attribute__((ext_vector_type(E), aligned(2)));
};

__device__ __forceinline__ float widen(float v) { return v; }
__device__ __forceinline__ float widen(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

}  // namespace

}  // namespace asp
