// Register-tile arithmetic shared by the radix-2 / radix-4 kernels that hold
// a tile in registers and use LDS only to change which address bits are
// register bits: the tile's address bits split into a thread index and a
// "register field" of consecutive bits (a thread holds the elements that
// differ in the field), and W is applied along the digits inside the field.
#pragma once

#include <type_traits>
#include <utility>

#include "gtt_args.hpp"
#include "gtt_types.hpp"

namespace gtt {

typedef float regf32x4 __attribute__((ext_vector_type(4)));

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// one element with or without the non-temporal hint (the empty asm keeps the
// compiler from merging the two forms of a run-time choice into the plain one)
template <bool NT, typename C>
__device__ __forceinline__ C gload1(const C* p) {
    if constexpr (!NT) {
        return *p;
    } else if constexpr (sizeof(C) == 8) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        return __builtin_bit_cast(C, __builtin_nontemporal_load(reinterpret_cast<const f2*>(p)));
    } else {
        asm volatile("");
        return __builtin_nontemporal_load(p);
    }
}
template <bool NT, typename C>
__device__ __forceinline__ void gstore1(C* p, C v) {
    if constexpr (!NT) {
        *p = v;
    } else if constexpr (sizeof(C) == 8) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        __builtin_nontemporal_store(__builtin_bit_cast(f2, v), reinterpret_cast<f2*>(p));
    } else {
        asm volatile("");
        __builtin_nontemporal_store(v, p);
    }
}

// tile element of thread-index bits t with the field at FS zero
// (a field of FB bits)
template <int FB = 4>
__host__ __device__ constexpr uint32_t reg_insert(uint32_t t, int FS) {
    return (t & ((1u << FS) - 1u)) | ((t >> FS) << (FS + FB));
}

// W (ADJ: W^H) along the digit of stride ST of N register values.
// Radix 2: on the VALU, W in scalar registers.
template <typename C, int B, int N, int ST, bool ADJ>
__device__ __forceinline__ void reg_digit2(C (&v)[N], const C (&w)[B * B]) {
#pragma unroll
    for (int base = 0; base < N; ++base) {
        if ((base / ST) % B != 0) continue;
        C in[B];
#pragma unroll
        for (int q = 0; q < B; ++q) in[q] = v[base + q * ST];
#pragma unroll
        for (int r = 0; r < B; ++r) {
            C acc;
            if constexpr (ADJ) {
                acc = cmac_conj(czero<C>(), in[0], w[r]);
#pragma unroll
                for (int q = 1; q < B; ++q) acc = cmac_conj(acc, in[q], w[q * B + r]);
            } else {
                acc = cmul(w[r * B], in[0]);
#pragma unroll
                for (int q = 1; q < B; ++q) acc = cmac(acc, w[r * B + q], in[q]);
            }
            v[base + r * ST] = acc;
        }
    }
}

// Radix 4: on the 4x4x1 FP32 MFMA, one fibre a lane.  B holds element k of
// every lane's fibre, A column k of W (lane l: row l % 4, the same in every
// group of four lanes), and D's four registers are the lane's four results:
// a rank-1 update per k, the same products and sums in the same order as the
// VALU's FMAs, but 256 of them in two passes.
template <typename C>
struct W4;
template <>
struct W4<float> {
    float w[4];
};
template <>
struct W4<cf> {
    float re[4], im[4], ni[4];
};
__device__ __forceinline__ void w4_load(W4<float>& f, const float* W, bool adj) {
    const uint32_t i = threadIdx.x & 3u;
#pragma unroll
    for (int k = 0; k < 4; ++k) f.w[k] = adj ? W[k * 4 + i] : W[i * 4 + k];
}
__device__ __forceinline__ void w4_load(W4<cf>& f, const cf* W, bool adj) {
    const uint32_t i = threadIdx.x & 3u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const cf x = adj ? cconj(W[k * 4 + i]) : W[i * 4 + k];
        f.re[k] = x.re;
        f.im[k] = x.im;
        f.ni[k] = -x.im;
    }
}
template <int N, int ST>
__device__ __forceinline__ void reg_digit4(float (&v)[N], const W4<float>& w) {
#pragma unroll
    for (int base = 0; base < N; ++base) {
        if ((base / ST) % 4 != 0) continue;
        regf32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) d = __builtin_amdgcn_mfma_f32_4x4x1f32(w.w[k], v[base + k * ST], d, 0, 0, 0);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[base + k * ST] = d[k];
    }
}
template <int N, int ST>
__device__ __forceinline__ void reg_digit4(cf (&v)[N], const W4<cf>& w) {
#pragma unroll
    for (int base = 0; base < N; ++base) {
        if ((base / ST) % 4 != 0) continue;
        regf32x4 dr = {0.f, 0.f, 0.f, 0.f}, di = dr;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const cf x = v[base + k * ST];
            dr = __builtin_amdgcn_mfma_f32_4x4x1f32(w.re[k], x.re, dr, 0, 0, 0);
            di = __builtin_amdgcn_mfma_f32_4x4x1f32(w.re[k], x.im, di, 0, 0, 0);
            dr = __builtin_amdgcn_mfma_f32_4x4x1f32(w.ni[k], x.im, dr, 0, 0, 0);
            di = __builtin_amdgcn_mfma_f32_4x4x1f32(w.im[k], x.re, di, 0, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) v[base + k * ST] = cf{dr[k], di[k]};
    }
}

}  // namespace gtt
