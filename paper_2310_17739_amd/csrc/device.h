// Device types and accessors shared by the kernel files.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "launch.h"
#include "swizzle.h"

namespace qk {

template <typename T>
struct alignas(2 * sizeof(T)) Cx {
    T re, im;
};

template <int V>
struct IntC {
    static constexpr int value = V;
};
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (B < E) {
        f(IntC<B>{});
        static_for<B + 1, E>(f);
    }
}

// LDS slot of tile element j (the fold defined with the pass packer).
template <typename T>
__device__ __forceinline__ int sw(int j) {
    return qs::lds_slot(int(sizeof(Cx<T>)), j);
}

// The tile of k_tile sits at LDS byte 0 of its workgroup (the kernel has no
// static LDS, which init_kernels checks), slot i at byte i * sizeof(Cx<T>),
// and is addressed by byte offsets, so that an access costs one XOR; the FP64
// reduction scratch of in-tile measurements follows the tile.
template <typename T>
struct LdsTile {
    static constexpr int LOGE = sizeof(Cx<T>) == 8 ? 3 : 4;
    typedef T V2 __attribute__((ext_vector_type(2)));
    static __device__ __forceinline__ Cx<T> ld(uint32_t byte) {
        const V2 v = *reinterpret_cast<const __attribute__((address_space(3))) V2 *>(uintptr_t(byte));
        return Cx<T>{v.x, v.y};
    }
    static __device__ __forceinline__ void st(uint32_t byte, Cx<T> c) {
        V2 v;
        v.x = c.re;
        v.y = c.im;
        *reinterpret_cast<__attribute__((address_space(3))) V2 *>(uintptr_t(byte)) = v;
    }
    static __device__ __forceinline__ Cx<T> at(int j) { return ld(uint32_t(sw<T>(j)) << LOGE); }
    static __device__ __forceinline__ void set(int j, Cx<T> v) { st(uint32_t(sw<T>(j)) << LOGE, v); }
    static __device__ __forceinline__ __attribute__((address_space(3))) double *red(int t) {
        return reinterpret_cast<__attribute__((address_space(3))) double *>(uintptr_t(uint32_t(sizeof(Cx<T>)) << t));
    }
};

// Tile loads and stores of the state stream past the caches (non-temporal):
// each pass touches every amplitude once, and the operator records and
// coefficients read through the scalar cache then stay resident in L2.
template <typename T>
__device__ __forceinline__ Cx<T> ld_stream(const Cx<T> *p) {
    typedef T V2 __attribute__((ext_vector_type(2)));
    const V2 v = __builtin_nontemporal_load(reinterpret_cast<const V2 *>(p));
    return Cx<T>{v.x, v.y};
}
template <typename T>
__device__ __forceinline__ void st_stream(Cx<T> *p, Cx<T> c) {
    typedef T V2 __attribute__((ext_vector_type(2)));
    V2 v;
    v.x = c.re;
    v.y = c.im;
    __builtin_nontemporal_store(v, reinterpret_cast<V2 *>(p));
}

}  // namespace qk
