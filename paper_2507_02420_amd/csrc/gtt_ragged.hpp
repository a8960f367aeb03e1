// Ragged batches: instances of different radix and length (each its own GTT,
// Def. 2.4) packed in one buffer.  The host lays out a device work list of
// (descriptor, tile) items, one descriptor per (instance, digit group);
// phase p holds the tiles of digit group p of every instance, sorted by item
// class (VALU radix 2..5, runtime radix, matrix-core radix 16 / 32).
//
// Per-phase mode (the default) launches one kernel per run of one class in a
// phase, specialised to that class: radix 2, 4 (32-bit lanes) and the
// matrix-core classes loop over their items on a resident grid, keeping W while
// consecutive items share it, with the next item's tile in flight (float
// matrix-core items excepted); the other classes take one tile per work-group.
//
// Persistent mode runs every phase in ONE launch of the all-class kernel (a
// work-group takes the items of the current phase round-robin and dispatches
// on the class) and separates the phases by a grid barrier (the next digit
// group of an instance needs all tiles of the previous one).  The barrier
// counts arrivals with a device-scope atomic; the last work-group to arrive
// resets the count and advances a generation word the others wait on, so the
// state returns to zero after every barrier and the launch can be replayed
// from a captured graph.  The grid never exceeds the number of co-resident
// work-groups (occupancy x compute units, not a cooperative launch), and
// every wait is bounded: after `spin_limit` polls a work-group raises the
// failure word; every work-group that sees it leaves the kernel at its next
// barrier (no wave can hang, no phase runs on partial data).  A one-thread
// kernel before every persistent launch zeroes the arrival and generation
// words and moves a raised failure word into a sticky record that the host
// reads and clears with gtt_plan_check.
#pragma once

#include "gtt_args.hpp"
#include "gtt_mfma.hpp"
#include "gtt_pass.hpp"
#include "gtt_types.hpp"

namespace gtt {

struct RaggedDesc {
    PassArgs a;          // tile geometry of this (instance, group)
    int64_t in_off;      // element offset of the group's input
    int64_t out_off;     // element offset of the group's output
    int64_t mid_off_saved;  // offset of this group's output inside `saved`
    int64_t w_off;       // element offset of the instance's W in the W table
    int32_t in_sel;      // 0: x, 1: y, 2: intermediate (saved if given, else y)
    int32_t out_sel;     // 1: y, 2: intermediate
    int32_t in_mid_saved;// 1 when in_sel == 2 (offset in saved is in_off_saved)
    int32_t b;
    int32_t kind;        // kKindValu / kKindGeneric / kKindMfma
    int32_t pad0;
    int64_t in_off_saved;
};

struct RaggedItem {
    int32_t d;           // descriptor index
    int32_t pad0;
    int64_t tile;        // tile index within the descriptor's group
};

constexpr int kMaxPhases = 8;

struct RaggedArgs {
    const RaggedDesc* desc;
    const RaggedItem* items;
    int64_t phase_start[kMaxPhases + 1];
    int32_t nphases;
    int32_t persistent;  // 1: all phases in this launch, grid barriers between
    int32_t phase;       // phase of a per-phase launch
    int32_t adjoint;
    const void* x;
    void* y;
    void* saved;
    const void* W;
    unsigned* bar;       // [0] arrivals, [1] generation, [2] failure of this
                         // launch, [3] sticky failure record
    uint32_t spin_limit; // polls of a barrier wait before it gives up
};

// Returns false when the barrier failed (this or another work-group gave up
// waiting); the caller then leaves the kernel.
__device__ __forceinline__ bool grid_barrier(unsigned* bar, unsigned nblocks, uint32_t spin_limit) {
    __shared__ unsigned failed;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned gen = __hip_atomic_load(&bar[1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT);
        __atomic_thread_fence(__ATOMIC_RELEASE);  // this block's tile stores
        const unsigned arrived =
            __hip_atomic_fetch_add(&bar[0], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        if (arrived == nblocks - 1) {
            __hip_atomic_store(&bar[0], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_fetch_add(&bar[1], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        } else {
            // bounded wait (the default limit, 2^24 polls with s_sleep, is
            // several seconds); a failure raised elsewhere ends it at once
            // (a limit of 0 gives up without polling)
            for (uint32_t spin = 0;; ++spin) {
                if (spin >= spin_limit || __hip_atomic_load(&bar[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    __hip_atomic_store(&bar[2], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
                if (__hip_atomic_load(&bar[1], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != gen) break;
                __builtin_amdgcn_s_sleep(4);
            }
        }
        __atomic_thread_fence(__ATOMIC_ACQUIRE);
        failed = __hip_atomic_load(&bar[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    return failed == 0;
}

template <typename C, int B>
__device__ __forceinline__ void load_w_ptr(C (&w)[B * B], const C* __restrict__ Wg, int adjoint, C* wl) {
    if constexpr (B * B * sizeof(C) <= 128) {
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int q = 0; q < B; ++q) w[r * B + q] = adjoint ? cconj(Wg[q * B + r]) : Wg[r * B + q];
    } else {
        for (int e = threadIdx.x; e < B * B; e += kThreads) {
            const int r = e / B, q = e % B;
            wl[e] = adjoint ? cconj(Wg[q * B + r]) : Wg[e];
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < B * B; ++e) w[e] = wl[e];
    }
}

template <typename T, int B>
__device__ __forceinline__ void ragged_tile_valu(unsigned char* smem, const PassArgs& a, const T* in, T* out,
                                              const typename Tr<T>::C* W, int adjoint, int64_t t) {
    using C = typename Tr<T>::C;
    constexpr int RD = RegDigits<B>::v;
    C* wl = reinterpret_cast<C*>(smem);
    C* lds = wl + 64;  // first 64 elements: staging for W (radix <= 8)
    C w[B * B];
    load_w_ptr<C, B>(w, W, adjoint, wl);
    const uint32_t rows = (uint32_t)a.P * (uint32_t)a.G;
    tile_load<T, C>(lds, a, in, t, rows);
    __syncthreads();
    run_stages<C, B, RD>(lds, a, rows, w);
    tile_store<T, C>(lds, a, out, t, rows);
    __syncthreads();
}

template <typename T>
__device__ __forceinline__ void ragged_tile_generic(unsigned char* smem, const PassArgs& a, const T* in, T* out,
                                                 const typename Tr<T>::C* W, int adjoint, int64_t t) {
    using C = typename Tr<T>::C;
    C* Wl = reinterpret_cast<C*>(smem);
    const uint32_t rows = (uint32_t)a.P * (uint32_t)a.G;
    const uint32_t tileE = rows << a.logC;
    const uint32_t wpad = ((uint32_t)a.wtotal + 15u) & ~15u;
    C* buf0 = Wl + wpad;
    C* buf1 = buf0 + lds_tile_elems(tileE, a.pad_shift);  // only for radices above 16
    for (int j = 0, done = 0; j < a.k; ++j) {
        const int bj = a.rad[j];
        for (int e = threadIdx.x; e < bj * bj; e += kThreads) {
            const int r = e / bj, q = e - r * bj;
            Wl[done + e] = adjoint ? cconj(W[a.wofs[j] + q * bj + r]) : W[a.wofs[j] + e];
        }
        done += bj * bj;
    }
    tile_load<T, C>(buf0, a, in, t, rows);
    __syncthreads();
    const C* res = generic_digits<C>(buf0, buf1, Wl, a, rows);
    tile_store<T, C>(res, a, out, t, rows);
    __syncthreads();
}

// Item classes.  The per-phase launches run the items of one class with a
// kernel specialised to it (its own registers and LDS, hence occupancy);
// the persistent launch dispatches every item at run time.
constexpr int kClsAny = -1;
constexpr int kClsGeneric = 0;  // 2..5: VALU radix; 16, 32: matrix-core radix

__host__ __device__ inline int ragged_class(int kind, int b) {
    if (kind == kKindValu) return (b >= 2 && b <= 5) ? b : kClsGeneric;
    if (kind == kKindMfma) return b;
    return kClsGeneric;
}

// The work list and the descriptors, read by scalar loads: constant for the
// launch, which the compiler cannot know next to the stores to y.  Its vector
// loads of them held the fields in vector registers and, counted in order with
// the stores, waited for the previous tile's stores.
__device__ __forceinline__ const RaggedDesc& ragged_desc(const RaggedArgs& r, int32_t d) {
    typedef const __attribute__((address_space(4))) RaggedDesc* P;
    return *(const RaggedDesc*)((P)(uintptr_t)r.desc + d);
}
__device__ __forceinline__ RaggedItem ragged_item_at(const RaggedArgs& r, int64_t i) {
    typedef const __attribute__((address_space(4))) RaggedItem* P;
    return *(const RaggedItem*)((P)(uintptr_t)r.items + i);
}

// input and output of an item's group (x / y / the saved intermediates)
template <typename T>
__device__ __forceinline__ const T* ragged_in(const RaggedArgs& r, const RaggedDesc& d) {
    if (d.in_sel == 0) return static_cast<const T*>(r.x) + d.in_off;
    if (d.in_sel == 1 || !r.saved) return static_cast<const T*>(r.y) + d.in_off;
    return static_cast<const T*>(r.saved) + d.in_off_saved;
}
template <typename T>
__device__ __forceinline__ T* ragged_out(const RaggedArgs& r, const RaggedDesc& d) {
    if (d.out_sel == 1 || !r.saved) return static_cast<T*>(r.y) + d.out_off;
    return static_cast<T*>(r.saved) + d.mid_off_saved;
}

template <typename T, int CLS>
__device__ __forceinline__ void ragged_item(unsigned char* smem, const RaggedArgs& r, const RaggedItem& it) {
    using C = typename Tr<T>::C;
    const RaggedDesc& d = ragged_desc(r, it.d);
    const T* in = ragged_in<T>(r, d);
    T* out = ragged_out<T>(r, d);
    const C* W = static_cast<const C*>(r.W) + d.w_off;
    if constexpr (CLS == kClsAny) {
        if (d.kind == kKindValu) {
            switch (d.b) {
                case 2: ragged_tile_valu<T, 2>(smem, d.a, in, out, W, r.adjoint, it.tile); break;
                case 3: ragged_tile_valu<T, 3>(smem, d.a, in, out, W, r.adjoint, it.tile); break;
                case 4: ragged_tile_valu<T, 4>(smem, d.a, in, out, W, r.adjoint, it.tile); break;
                case 5: ragged_tile_valu<T, 5>(smem, d.a, in, out, W, r.adjoint, it.tile); break;
                default: ragged_tile_generic<T>(smem, d.a, in, out, W, r.adjoint, it.tile); break;
            }
        } else {
            ragged_tile_generic<T>(smem, d.a, in, out, W, r.adjoint, it.tile);
        }
    } else if constexpr (CLS == kClsGeneric) {
        ragged_tile_generic<T>(smem, d.a, in, out, W, r.adjoint, it.tile);
    } else if constexpr (CLS <= 5) {
        ragged_tile_valu<T, CLS>(smem, d.a, in, out, W, r.adjoint, it.tile);
    } else {
        static_assert(CLS <= 5, "matrix-core classes run ragged_mfma_items");
    }
}

template <typename T, int B>
__device__ __forceinline__ void ragged_tile_mfma_wf(unsigned char* smem, const PassArgs& a, const T* in, T* out,
                                                    const WFrag<T, B>& wf, int64_t t) {
    const uint32_t rows = (uint32_t)a.P * (uint32_t)a.G;
    if constexpr (std::is_same<T, float>::value) {
        float* lds = reinterpret_cast<float*>(smem + 256);
        tile_load<T, float>(lds, a, in, t, rows);
        __syncthreads();
        for (int j = 0; j < a.k; ++j) {
            mfma_stage<T, B>(lds, a, j, rows, wf);
            __syncthreads();
        }
        tile_store<T, float>(lds, a, out, t, rows);
    } else {
        uint16_t* lds = reinterpret_cast<uint16_t*>(smem + 256);
        mfma_tile16<T, B>(lds, a, in, out, t, rows, wf);
    }
    __syncthreads();
}

template <typename T>
__global__ __launch_bounds__(kThreads) void gtt_ragged_kernel(RaggedArgs r) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    constexpr bool kMfma = sizeof(T) == 2 || std::is_same<T, float>::value;
    const int p0 = r.persistent ? 0 : r.phase;
    const int p1 = r.persistent ? r.nphases : r.phase + 1;
    // matrix-core items keep W's fragments while consecutive items share W
    [[maybe_unused]] typename std::conditional<kMfma, WFrag<T, 16>, char>::type wf16;
    [[maybe_unused]] typename std::conditional<kMfma, WFrag<T, 32>, char>::type wf32;
    [[maybe_unused]] int64_t w16 = -1, w32 = -1;
    for (int p = p0; p < p1; ++p) {
        for (int64_t i = r.phase_start[p] + blockIdx.x; i < r.phase_start[p + 1]; i += gridDim.x) {
            const RaggedItem it = ragged_item_at(r, i);
            if constexpr (kMfma) {
                const RaggedDesc& d = ragged_desc(r, it.d);
                if (d.kind == kKindMfma) {
                    PassArgs aw;  // only W / adjoint are read by the fragment loader
                    aw.W = static_cast<const float*>(r.W) + d.w_off;
                    aw.adjoint = r.adjoint;
                    if (d.b == 16) {
                        if (d.w_off != w16) {
                            load_w_frag<T, 16>(wf16, aw);
                            w16 = d.w_off;
                        }
                        ragged_tile_mfma_wf<T, 16>(smem_raw, d.a, ragged_in<T>(r, d), ragged_out<T>(r, d), wf16, it.tile);
                    } else {
                        if (d.w_off != w32) {
                            load_w_frag<T, 32>(wf32, aw);
                            w32 = d.w_off;
                        }
                        ragged_tile_mfma_wf<T, 32>(smem_raw, d.a, ragged_in<T>(r, d), ragged_out<T>(r, d), wf32, it.tile);
                    }
                    continue;
                }
            }
            ragged_item<T, kClsAny>(smem_raw, r, it);
        }
        if (r.persistent && p + 1 < p1 && !grid_barrier(r.bar, gridDim.x, r.spin_limit)) return;
    }
}

// Matrix-core items (one class, one phase): the work-groups loop over the
// items and keep W's fragments while consecutive items share W; 16-bit items
// have the next one's tile in flight meanwhile.
template <typename T, int B>
__device__ __forceinline__ void ragged_mfma_items(unsigned char* smem, const RaggedArgs& r) {
    constexpr bool k16 = sizeof(T) == 2;
    using L = typename std::conditional<k16, uint16_t, float>::type;
    L* lds = reinterpret_cast<L*>(smem + 256);
    WFrag<T, B> wf;
    int64_t wcur = -1;
    int64_t i = r.phase_start[0] + blockIdx.x;
    const int64_t end = r.phase_start[1];
    if (i >= end) return;
    RaggedItem it = ragged_item_at(r, i);
    [[maybe_unused]] typename std::conditional<k16, Prefetch16<T, B>, char>::type next;
    [[maybe_unused]] bool held = false;
    if constexpr (k16) {
        const RaggedDesc& d = ragged_desc(r, it.d);
        held = Prefetch16<T, B>::fits(d.a);
        if (held) next.fetch(d.a, ragged_in<T>(r, d), it.tile);
        else next.clear();
    }
    for (; i < end; i += gridDim.x) {
        const RaggedDesc& d = ragged_desc(r, it.d);
        const PassArgs& a = d.a;
        const int64_t tile = it.tile;
        if (d.w_off != wcur) {
            PassArgs aw;  // only W / adjoint are read by the fragment loader
            aw.W = static_cast<const float*>(r.W) + d.w_off;
            aw.adjoint = r.adjoint;
            load_w_frag<T, B>(wf, aw);
            wcur = d.w_off;
        }
        const uint32_t rows = (uint32_t)a.P * (uint32_t)a.G;
        const bool more = i + gridDim.x < end;
        if (more) it = ragged_item_at(r, i + gridDim.x);
        if constexpr (k16) {
            const bool cur = held;
            if (cur) next.commit(lds, a);
            else mfma_tile16<T, B>(lds, a, ragged_in<T>(r, d), ragged_out<T>(r, d), tile, rows, wf);
            __syncthreads();
            const RaggedDesc& dn = ragged_desc(r, it.d);
            held = more && Prefetch16<T, B>::fits(dn.a);
            if (held) next.fetch(dn.a, ragged_in<T>(r, dn), it.tile);
            else next.clear();
            if (cur) {
                mfma_digits16<T, B>(lds, a, rows, wf);
                tile_store16<T, B>(lds, a, ragged_out<T>(r, d), tile, rows);
            }
        } else {
            tile_load<T, float>(lds, a, ragged_in<T>(r, d), tile, rows);
            __syncthreads();
            for (int j = 0; j < a.k; ++j) {
                mfma_stage<T, B>(lds, a, j, rows, wf);
                __syncthreads();
            }
            tile_store<T, float>(lds, a, ragged_out<T>(r, d), tile, rows);
        }
        __syncthreads();
    }
}

// VALU items of radix B with the next item's tile in flight: vector tiles of up
// to eight 16-byte vectors a thread.  One work-group an item waited for its loads
// each time (MI355X, 46 M and 60 M bf16 elements of radix 2 and 4, two launches
// each: 98 + 73 and 141 + 127 -> 93 + 62 and 99 + 88 us; 34 and 45 at the rate of
// a copy).
template <typename T>
struct RaggedNext {
    static constexpr int V = Vec16<T>::V;
    uint4 r[kPfVec];
    __device__ __forceinline__ static bool fits(const PassArgs& a) {
        const uint32_t tileE = ((uint32_t)a.P * (uint32_t)a.G) << a.logC;
        return (a.mode == kContigVec || a.mode == kRowVec) && a.cut < 0 && tileE / V <= (uint32_t)(kPfVec * kThreads);
    }
    __device__ __forceinline__ void fetch(const PassArgs& a, const T* __restrict__ in, int64_t t) {
        const uint32_t tileE = ((uint32_t)a.P * (uint32_t)a.G) << a.logC;
        const bool contig = a.mode == kContigVec;
        const int64_t hb = contig ? 0 : tile_hb(a, t);
        const int64_t l = contig ? 0 : t - hb * a.L;
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // (offsets not held across the loop)
#pragma unroll
        for (int v = 0; v < kPfVec; ++v) {
            const uint32_t i = tid + v * kThreads;
            uint4 q = make_uint4(0u, 0u, 0u, 0u);
            if (i < tileE / V) q = gload16<true>(in + vec_offset<T>(a, t, i, hb, l, tileE));
            r[v] = q;
        }
    }
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int v = 0; v < kPfVec; ++v) r[v] = make_uint4(0u, 0u, 0u, 0u);
    }
    template <typename C>
    __device__ __forceinline__ void commit(C* lds, const PassArgs& a) const {
        const uint32_t tileE = ((uint32_t)a.P * (uint32_t)a.G) << a.logC;
        uint32_t tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
#pragma unroll
        for (int v = 0; v < kPfVec; ++v) {
            const uint32_t i = tid + v * kThreads;
            if (i < tileE / V) {
                T vals[V];
                *reinterpret_cast<uint4*>(vals) = r[v];
                const uint32_t ph = lds_phys(i * V, a.pad_shift);
#pragma unroll
                for (int e = 0; e < V; ++e) lds[ph + e] = to_c(vals[e]);
            }
        }
    }
};

template <typename T, int B>
__device__ __forceinline__ void ragged_valu_items(unsigned char* smem, const RaggedArgs& r) {
    using C = typename Tr<T>::C;
    C* wl = reinterpret_cast<C*>(smem);
    C* lds = wl + 64;
    C w[B * B];
    int64_t wcur = -1;
    int64_t i = r.phase_start[0] + blockIdx.x;
    const int64_t end = r.phase_start[1];
    if (i >= end) return;
    RaggedItem it = ragged_item_at(r, i);
    RaggedNext<T> next;
    bool held = false;
    {
        const RaggedDesc& d = ragged_desc(r, it.d);
        held = RaggedNext<T>::fits(d.a);
        if (held) next.fetch(d.a, ragged_in<T>(r, d), it.tile);
        else next.clear();
    }
    for (; i < end; i += gridDim.x) {
        const RaggedDesc& d = ragged_desc(r, it.d);
        const PassArgs& a = d.a;
        const int64_t tile = it.tile;
        const uint32_t rows = (uint32_t)a.P * (uint32_t)a.G;
        if (d.w_off != wcur) {
            load_w_ptr<C, B>(w, static_cast<const C*>(r.W) + d.w_off, r.adjoint, wl);
            wcur = d.w_off;
        }
        const bool more = i + gridDim.x < end;
        if (more) it = ragged_item_at(r, i + gridDim.x);
        if (held) next.commit(lds, a);
        else tile_load<T, C>(lds, a, ragged_in<T>(r, d), tile, rows);
        __syncthreads();
        const RaggedDesc& dn = ragged_desc(r, it.d);
        held = more && RaggedNext<T>::fits(dn.a);
        if (held) next.fetch(dn.a, ragged_in<T>(r, dn), it.tile);
        else next.clear();
        run_stages<C, B, RegDigits<B>::v>(lds, a, rows, w);
        tile_store<T, C>(lds, a, ragged_out<T>(r, d), tile, rows);
        __syncthreads();
    }
}

// classes whose kernels loop over their items with the next tile in flight; the
// other radices' vectors mostly start off a 16-byte boundary, where it does not
// apply and one work-group an item is faster
template <typename T, int CLS>
constexpr bool ragged_prefetches() {
    using C = typename Tr<T>::C;
    return CLS >= 16 || ((CLS == 2 || CLS == 4) && pass_prefetches<C, CLS == 4 ? 4 : 2>());
}

// The items [phase_start[0], phase_start[1]) of one class.
// (16-bit storage with a tile in flight: at most 128 registers for the four work-groups a compute unit
// that a 32 KiB tile allows)
template <typename T, int CLS>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 2 && ragged_prefetches<T, CLS>() ? 4 : 1))) void
gtt_ragged_class_kernel(RaggedArgs r) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if constexpr (CLS >= 16) {
        static_assert(sizeof(T) == 2 || std::is_same<T, float>::value,
                      "matrix-core item classes exist for 16-bit and float storage only");
        ragged_mfma_items<T, CLS>(smem_raw, r);
    } else if constexpr (ragged_prefetches<T, CLS>()) {
        ragged_valu_items<T, CLS>(smem_raw, r);
    } else {
        for (int64_t i = r.phase_start[0] + blockIdx.x; i < r.phase_start[1]; i += gridDim.x)
            ragged_item<T, CLS>(smem_raw, r, ragged_item_at(r, i));
    }
}

}  // namespace gtt
