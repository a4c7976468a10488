// Device helpers shared by the kernel files: complex pairs and global-memory
// accesses.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace heom {
namespace {

// --------------------------------------------------------------------------
// Small complex helpers (interleaved re/im, T = float or double).
// --------------------------------------------------------------------------
template <typename T>
struct cpx {
    T re, im;
};

template <typename T>
__device__ __forceinline__ cpx<T> cconj(cpx<T> a) {
    return {a.re, -a.im};
}

// (re, im) pairs as clang vector types: one 8- or 16-byte access per element.
typedef float pair_f __attribute__((ext_vector_type(2)));
typedef double pair_d __attribute__((ext_vector_type(2)));
typedef int pair_i __attribute__((ext_vector_type(2)));
template <typename T>
struct vec2;
template <>
struct vec2<float> {
    using type = pair_f;
};
template <>
struct vec2<double> {
    using type = pair_d;
};

// Global-memory views of pointers held in descriptors.  Without the cast the
// compiler cannot prove these generic pointers are global and emits FLAT
// instructions, whose completion is tracked together with LDS traffic.
template <typename T>
using gcptr = const __attribute__((address_space(1))) T*;
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gcptr<T> G(const T* p) {
    return (gcptr<T>)p;
}
template <typename T>
__device__ __forceinline__ gptr<T> G(T* p) {
    return (gptr<T>)p;
}

template <typename T>
__device__ __forceinline__ cpx<T> ld(const void* base, size_t idx) {
    typename vec2<T>::type v = G(reinterpret_cast<const typename vec2<T>::type*>(base))[idx];
    return {v.x, v.y};
}

template <typename T>
__device__ __forceinline__ void st(void* base, size_t idx, cpx<T> a) {
    typename vec2<T>::type v;
    v.x = a.re;
    v.y = a.im;
    G(reinterpret_cast<typename vec2<T>::type*>(base))[idx] = v;
}

}  // namespace
}  // namespace heom
