// Forward / inverse pass of one digit group and the natural-order filter's
// middle pass, radix 2 and 4, with a tile of 2^LOGT elements in registers.
//
// A work-group of 256 threads owns a tile (8192 elements of 4 bytes or 4096 of
// 8 bytes, 32 KiB; 32 or 16 elements a thread, FB register bits).  The group's
// digits are taken in blocks of as many digits as fit the FB bits; the blocks
// are worked on one after another, each in the layout whose register field
// holds its digits, and LDS only changes the layout between them.  The first
// block's layout is loaded from global memory and the last one's stored to it
// directly wherever its lanes run along at least four address bits; only a
// layout whose field starts at bit 0 (a thread's elements contiguous) goes
// through LDS in 16-byte vectors.  The digits commute, so the blocks run in
// the order that makes both ends direct: three blocks of a contiguous group as
// 1, 0, 2.  The next tile's loads are in flight from the first exchange on.
//
// FILT: the group is the transform's last one; its coefficients X are split by
// natural index (k < cut to `out`, k >= cut to `out2`, either may be null) and
// the group's inverse runs on each part from the registers that hold X.  One
// read and two writes of the buffers replace the coefficients' write and two
// reads, and two passes' loads and stores.
//
// What bounds it: HBM (the copy rate is reached to 90 % on buffers larger than
// the memory-side cache).  MI355X, before (gtt_pass_kernel: up to four LDS
// sweeps a tile, run-time geometry, 2.5-2.8 waves per SIMD) -> now:
// 64 x 4^10 complex64, groups of 6 and 4 digits 290 + 254 -> 200 + 187 us
// (224 + 215 before the tile order and cache hints of stream_bits);
// 16 x 2^20 int32 45 + 32 -> 26 + 22 us, float 48 + 34 -> 27 + 23 us;
// filter of 64 x 4^10 complex64 1753 -> 961 us (middle pass 400 to 455 us between
// cards, the masked inverse pass alone was 374 us); 32 x 4^5 float 9.4 -> 6.4 us a call.
#pragma once

#include "gtt_args.hpp"
#include "gtt_pass.hpp"
#include "gtt_reg.hpp"
#include "gtt_types.hpp"

namespace gtt {

template <typename C, int B, int K, int LOGT, bool ROW>
struct PassRegGeom {
    static constexpr int FB = sizeof(C) == 4 ? 5 : 4;
    static constexpr int N = 1 << FB;  // elements a thread
    static constexpr int LB = B == 2 ? 1 : 2;
    static constexpr int RD = FB / LB;
    static constexpr int NBLK = (K + RD - 1) / RD;
    static constexpr int LOGC = ROW ? LOGT - K * LB : 0;
    static constexpr int NT = 1 << (LOGT - FB);
    static constexpr uint32_t TE = 1u << LOGT;
    static_assert(LOGC >= 0 && K * LB + LOGC <= LOGT && K >= 1 && NBLK <= 3 && NT == kThreads, "tile bits");
    // LDS position: a pad element after every 16 (and 512) or 32 elements;
    // additive over disjoint bits
    __host__ __device__ static constexpr uint32_t pos(uint32_t x) {
        return FB == 4 ? x + (x >> 4) + (x >> 9) : x + (x >> 5);
    }
    static constexpr uint32_t TP = TE + (FB == 4 ? (TE >> 4) + (TE >> 9) : (TE >> 5));
    static constexpr int digits(int i) { return i < NBLK - 1 ? RD : K - RD * (NBLK - 1); }
    static constexpr int field(int i) {
        const int s = LOGC + LB * RD * i;
        return s > LOGT - FB ? LOGT - FB : s;
    }
    static constexpr int doff(int i) { return LOGC + LB * RD * i - field(i); }
    // the i-th block worked on
    static constexpr int seq(int i) { return NBLK == 3 && !ROW ? (i == 0 ? 1 : i == 1 ? 0 : 2) : i; }
    static constexpr bool kDirectIn = ROW || NBLK == 3;
    static constexpr bool kDirectOut = ROW || NBLK >= 2;
};

// W of a launch (adj: W^H): radix 4 on float data as MFMA operands,
// otherwise in scalar registers
template <typename C, int B>
constexpr bool kPassW4 = B == 4 && (std::is_same<C, float>::value || std::is_same<C, cf>::value);
template <typename C, int B, bool M4 = kPassW4<C, B>>
struct PassW {
    C w[B * B];
    bool h2;
    __device__ __forceinline__ void load(const C* __restrict__ Wg, bool adj) {
#pragma unroll
        for (int r = 0; r < B; ++r)
#pragma unroll
            for (int q = 0; q < B; ++q) w[r * B + q] = adj ? cconj(Wg[q * B + r]) : Wg[r * B + q];
        h2 = false;
        if constexpr (B == 2 && std::is_same<C, uint32_t>::value)
            h2 = w[0] == 1u && w[1] == 1u && w[2] == 1u && w[3] == 0xffffffffu;
    }
    // H2: the integer Hadamard as butterflies
    template <int N, int ST, bool H2>
    __device__ __forceinline__ void digit(C (&v)[N]) const {
        if constexpr (H2) {
#pragma unroll
            for (int m = 0; m < N; ++m) {
                if (m & ST) continue;
                const C x0 = v[m], x1 = v[m + ST];
                v[m] = x0 + x1;
                v[m + ST] = x0 - x1;
            }
        } else {
            reg_digit2<C, B, N, ST, false>(v, w);
        }
    }
};
template <typename C, int B>
struct PassW<C, B, true> {
    W4<C> w;
    __device__ __forceinline__ void load(const C* __restrict__ Wg, bool adj) { w4_load(w, Wg, adj); }
    template <int N, int ST, bool H2>
    __device__ __forceinline__ void digit(C (&v)[N]) const {
        reg_digit4<N, ST>(v, w);
    }
};

// Waves per SIMD to compile for, and whether the next tile's loads are held in
// registers over the tile.  A pass: four waves (the LDS allows four
// work-groups).  The filter holds X besides the part it works on: radix 4 runs
// two waves with the prefetch (64 x 4^10: float 144 against 196 us at three
// waves without it, complex64 399 against 418; at three with it, spilled, 473
// and 736), radix 2 three without (complex64 458 against 460 us, 67 MB float
// 45 against 50).
template <int B, bool FILT>
struct PassRegForm {
    static constexpr int waves = !FILT ? 4 : B == 4 ? 2 : 3;
    static constexpr bool prefetch = !FILT || B == 4;
};

template <typename C, int B, int K, int LOGT, bool ROW, bool FILT>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(PassRegForm<B, FILT>::waves))) void gtt_pass_reg_kernel(
    PassArgs a, C* __restrict__ out2) {
    using Gm = PassRegGeom<C, B, K, LOGT, ROW>;
    constexpr int FB = Gm::FB, N = Gm::N, LB = Gm::LB, NBLK = Gm::NBLK, NT = Gm::NT, LOGC = Gm::LOGC;
    constexpr int V = 16 / (int)sizeof(C), NV = N / V;
    constexpr bool kPrefetch = PassRegForm<B, FILT>::prefetch;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* lds = reinterpret_cast<C*>(smem_raw);
    const C* __restrict__ Wg = static_cast<const C*>(a.W);
    PassW<C, B> w;
    w.load(Wg, !FILT && a.adjoint);
    const uint32_t tid = threadIdx.x;
    auto opaque_tid = [&]() -> uint32_t {  // keeps address sums out of registers across tiles
        uint32_t x = tid;
        asm volatile("" : "+v"(x));
        return x;
    };
    const int64_t total = a.N;  // elements of the buffers (the last contiguous tile may be partial)
    uint32_t S32 = ROW ? (uint32_t)a.S : 0u;
    // byte offset of tile element x from the tile's base (additive over
    // disjoint bits; below 2^31: the planner's rule)
    auto gofs = [&](uint32_t x) -> uint32_t {
        return (ROW ? (x >> LOGC) * S32 + (x & ((1u << LOGC) - 1u)) : x) * (uint32_t)sizeof(C);
    };
    auto tile_base = [&](int64_t t) -> int64_t {
        if constexpr (!ROW) return t << LOGT;
        const int64_t hb = tile_hb(a, t);
        return hb * ((int64_t)a.G * a.S) + ((t - hb * a.L) << LOGC);
    };
    auto tile_left = [&](int64_t t) -> uint32_t {  // elements of the tile inside the buffer
        if constexpr (ROW) return Gm::TE;
        const int64_t l = total - (t << LOGT);
        return l < (int64_t)Gm::TE ? (uint32_t)l : Gm::TE;
    };

    constexpr int I0 = Gm::seq(0), IL = Gm::seq(NBLK - 1);
    C pre[Gm::kDirectIn ? N : 1];
    uint4 pre4[Gm::kDirectIn ? 1 : NV];
    auto fetch = [&](int64_t t) {
        const char* pi = reinterpret_cast<const char*>(static_cast<const C*>(a.in) + tile_base(t));
        const uint32_t left = tile_left(t);
        if constexpr (Gm::kDirectIn) {
            constexpr int FS = Gm::field(I0);
            const uint32_t x0 = reg_insert<FB>(opaque_tid(), FS), lo = gofs(x0);
            if (!FILT && (ROW || left == Gm::TE) && (a.stream & kStreamIn)) {  // uniform
#pragma unroll
                for (int m = 0; m < N; ++m)
                    pre[m] = gload1<true>(reinterpret_cast<const C*>(pi + gofs((uint32_t)m << FS) + lo));
            } else if (ROW || left == Gm::TE) {
#pragma unroll
                for (int m = 0; m < N; ++m)
                    pre[m] = gload1<false>(reinterpret_cast<const C*>(pi + gofs((uint32_t)m << FS) + lo));
            } else {
#pragma unroll
                for (int m = 0; m < N; ++m) {
                    pre[m] = czero<C>();
                    if ((x0 | ((uint32_t)m << FS)) < left)
                        pre[m] = gload1<false>(reinterpret_cast<const C*>(pi + gofs((uint32_t)m << FS) + lo));
                }
            }
        } else {
            const uint32_t e0 = opaque_tid() * V, lo = gofs(e0);
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                pre4[m] = make_uint4(0u, 0u, 0u, 0u);
                if (e0 + (uint32_t)m * NT * V < left) pre4[m] = gload16<true>(pi + gofs((uint32_t)m * NT * V) + lo);
            }
        }
    };
    // layout i <-> LDS
    auto put = [&](auto ic, const C (&v)[N]) {
        constexpr int FS = Gm::field(decltype(ic)::value);
        const uint32_t p = Gm::pos(reg_insert<FB>(tid, FS));
#pragma unroll
        for (int m = 0; m < N; ++m) lds[p + Gm::pos((uint32_t)m << FS)] = v[m];
    };
    auto get = [&](auto ic, C (&v)[N]) {
        constexpr int FS = Gm::field(decltype(ic)::value);
        const uint32_t p = Gm::pos(reg_insert<FB>(tid, FS));
#pragma unroll
        for (int m = 0; m < N; ++m) v[m] = lds[p + Gm::pos((uint32_t)m << FS)];
    };
    auto apply = [&](auto ic, C (&v)[N], const PassW<C, B>& pw, auto h2) {
        constexpr int i = decltype(ic)::value;
        static_for<0, Gm::digits(i)>([&](auto d) {
            pw.template digit<N, (1 << (Gm::doff(i) + decltype(d)::value * LB)), decltype(h2)::value>(v);
        });
    };
    // layout i -> global memory
    auto store = [&](auto ic, const C (&v)[N], C* out, int64_t t) {
        constexpr int FS = Gm::field(decltype(ic)::value);
        char* po = reinterpret_cast<char*>(out + tile_base(t));
        const uint32_t x0 = reg_insert<FB>(opaque_tid(), FS), lo = gofs(x0), left = tile_left(t);
        if ((ROW || left == Gm::TE) && (a.stream & kStreamOut)) {
#pragma unroll
            for (int m = 0; m < N; ++m) gstore1<true>(reinterpret_cast<C*>(po + gofs((uint32_t)m << FS) + lo), v[m]);
        } else if (ROW || left == Gm::TE) {
#pragma unroll
            for (int m = 0; m < N; ++m) gstore1<false>(reinterpret_cast<C*>(po + gofs((uint32_t)m << FS) + lo), v[m]);
        } else {
#pragma unroll
            for (int m = 0; m < N; ++m)
                if ((x0 | ((uint32_t)m << FS)) < left) gstore1<false>(reinterpret_cast<C*>(po + gofs((uint32_t)m << FS) + lo), v[m]);
        }
    };
    // LDS (natural order) -> global memory in vectors
    auto store_lds = [&](C* out, int64_t t) {
        char* po = reinterpret_cast<char*>(out + tile_base(t));
        const uint32_t e0 = opaque_tid() * V, lo = gofs(e0), left = tile_left(t), p0 = Gm::pos(e0);
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            C vals[V];
#pragma unroll
            for (int e = 0; e < V; ++e) vals[e] = lds[p0 + Gm::pos((uint32_t)m * NT * V) + e];
            if (e0 + (uint32_t)m * NT * V < left)
                gstore16<true>(po + gofs((uint32_t)m * NT * V) + lo, *reinterpret_cast<const uint4*>(vals));
        }
    };
    using ci0 = std::integral_constant<int, I0>;
    using ciL = std::integral_constant<int, IL>;

    PassW<C, B> wh;
    if constexpr (FILT) wh.load(Wg, true);

    auto tiles = [&](auto h2) {
        int64_t n = blockIdx.x;
        if (kPrefetch && n < a.ntiles) fetch(tile_at(a, n));
        for (; n < a.ntiles; n += gridDim.x) {
            const int64_t t = tile_at(a, n);
            if constexpr (ROW) asm volatile("" : "+s"(S32));  // the same for the uniform parts
            const bool more = n + gridDim.x < a.ntiles;
            if (!kPrefetch) fetch(t);
            C v[N];
            // the first block's elements
            if constexpr (Gm::kDirectIn) {
#pragma unroll
                for (int m = 0; m < N; ++m) v[m] = pre[m];
                if constexpr (NBLK == 1) {
                    if (kPrefetch && more) fetch(tile_at(a, n + gridDim.x));
                }
            } else {
                const uint32_t p0 = Gm::pos(opaque_tid() * V);
#pragma unroll
                for (int m = 0; m < NV; ++m) {
                    C vals[V];
                    *reinterpret_cast<uint4*>(vals) = pre4[m];
#pragma unroll
                    for (int e = 0; e < V; ++e) lds[p0 + Gm::pos((uint32_t)m * NT * V) + e] = vals[e];
                }
                if (kPrefetch && more) fetch(tile_at(a, n + gridDim.x));
                __syncthreads();
                get(ci0{}, v);
            }
            apply(ci0{}, v, w, h2);
            static_for<1, NBLK>([&](auto s) {
                constexpr int j = decltype(s)::value;
                put(std::integral_constant<int, Gm::seq(j - 1)>{}, v);
                if constexpr (Gm::kDirectIn && j == 1) {
                    if (kPrefetch && more) fetch(tile_at(a, n + gridDim.x));
                }
                __syncthreads();
                get(std::integral_constant<int, Gm::seq(j)>{}, v);
                // (each put after the first writes the positions its own thread
                // read; the barrier after the last get orders the next tile's)
                if constexpr (j == NBLK - 1) __syncthreads();
                apply(std::integral_constant<int, Gm::seq(j)>{}, v, w, h2);
            });
            if constexpr (!FILT) {
                if constexpr (Gm::kDirectOut) {
                    store(ciL{}, v, static_cast<C*>(a.out), t);
                } else {
                    put(ciL{}, v);
                    __syncthreads();
                    store_lds(static_cast<C*>(a.out), t);
                    __syncthreads();
                }
            } else {
                // natural index of an element: its offset inside the instance
                constexpr int FS = Gm::field(IL);
                const int64_t hb = ROW ? tile_hb(a, t) : 0;
                const uint32_t nb = ROW ? (uint32_t)((t - hb * a.L) << LOGC) : 0u;
                const uint32_t nm = ROW ? 0xffffffffu : (1u << (K * LB)) - 1u;
                const uint32_t x0 = reg_insert<FB>(tid, FS);
#pragma unroll 1
                for (int part = 0; part < 2; ++part) {
                    C* out = part == 0 ? static_cast<C*>(a.out) : out2;
                    if (!out) continue;
                    C u[N];
#pragma unroll
                    for (int m = 0; m < N; ++m) {
                        const uint32_t k = (gofs(x0) + gofs((uint32_t)m << FS)) / (uint32_t)sizeof(C) + nb;
                        const bool low = (int64_t)(k & nm) < a.cut;
                        u[m] = low == (part == 0) ? v[m] : czero<C>();
                    }
                    apply(ciL{}, u, wh, h2);
                    static_for<1, NBLK>([&](auto s) {
                        constexpr int j = NBLK - 1 - decltype(s)::value;
                        put(std::integral_constant<int, Gm::seq(j + 1)>{}, u);
                        __syncthreads();
                        get(std::integral_constant<int, Gm::seq(j)>{}, u);
                        if constexpr (j == 0 && Gm::kDirectIn) __syncthreads();
                        apply(std::integral_constant<int, Gm::seq(j)>{}, u, wh, h2);
                    });
                    if constexpr (Gm::kDirectIn) {
                        store(ci0{}, u, out, t);
                    } else {
                        put(ci0{}, u);
                        __syncthreads();
                        store_lds(out, t);
                        __syncthreads();
                    }
                }
            }
        }
    };
    // the integer Hadamard has its own tile loop: a choice inside one loop
    // spilled both forms
    if constexpr (B == 2 && std::is_same<C, uint32_t>::value) {
        if (w.h2) {
            tiles(std::true_type{});
            return;
        }
    }
    tiles(std::false_type{});
}

template <typename C, int B, int K, bool ROW, bool FILT>
inline hipError_t launch_pass_reg_one(const PassArgs& a, C* out2, hipStream_t s) {
    constexpr int LOGT = sizeof(C) == 4 ? 13 : 12;
    using Gm = PassRegGeom<C, B, K, LOGT, ROW>;
    auto kernel = gtt_pass_reg_kernel<C, B, K, LOGT, ROW, FILT>;
    constexpr size_t lds = (size_t)Gm::TP * sizeof(C);
    const unsigned tiles = (unsigned)std::min<int64_t>(a.ntiles, 0x7fffffff);
    hipLaunchKernelGGL(kernel, dim3(resident_grid(kernel, kThreads, lds, tiles)), dim3(kThreads), lds, s, a, out2);
    return hipGetLastError();
}

template <typename C, int B, int K>
inline hipError_t launch_pass_reg_k(const PassArgs& a, bool row, bool filt, C* out2, hipStream_t s) {
    constexpr int LB = B == 2 ? 1 : 2;
    constexpr int LOGT = sizeof(C) == 4 ? 13 : 12;
    constexpr bool kFilt = !std::is_same<C, uint32_t>::value;
    if constexpr (K * LB > LOGT) {
        return hipErrorInvalidValue;
    } else {
        if (a.k > K) return launch_pass_reg_k<C, B, K + 1>(a, row, filt, out2, s);
        if (!row) {
            if constexpr (kFilt) {
                if (filt) return launch_pass_reg_one<C, B, K, false, true>(a, out2, s);
            }
            return launch_pass_reg_one<C, B, K, false, false>(a, out2, s);
        }
        if constexpr (((size_t)1 << (LOGT - K * LB)) * sizeof(C) >= kRegMinRow) {
            if constexpr (kFilt) {
                if (filt) return launch_pass_reg_one<C, B, K, true, true>(a, out2, s);
            }
            return launch_pass_reg_one<C, B, K, true, false>(a, out2, s);
        }
        return hipErrorInvalidValue;
    }
}

}  // namespace gtt

#define GTT_PASS_REG_INSTANTIATE(NAME, C, B)                                                                  \
    namespace gtt {                                                                                          \
    hipError_t launch_pass_reg_##NAME##_b##B(const PassArgs& a, bool row, bool filt, void* out2, hipStream_t s) { \
        return launch_pass_reg_k<C, B, 1>(a, row, filt, static_cast<C*>(out2), s);                            \
    }                                                                                                        \
    }
