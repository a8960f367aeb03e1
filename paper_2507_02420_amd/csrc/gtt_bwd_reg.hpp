// Backward of one digit group with the tile's activations in registers, one W
// for every digit: radix 2 and 4 (float and complex64), radix 16 (float, bf16
// and f16 storage).
//
// A tile of 2^LOGT elements (LOGT address bits: column bits, LB = log2 B bits
// a digit, hi-block bits) belongs to a work-group of 2^(LOGT-4) threads, 16
// elements a thread.  The group's digits are taken in blocks of RD = 4 / LB
// digits (16 positions); while block i is worked on, a thread holds the 16
// elements that differ in four address bits, the "register field" of the
// block, so W (or W^H) along the block's digits is register arithmetic.  LDS
// only changes the layout between blocks:
//   - forward: the activation a_i at the start of block i is read in block
//     i's layout and kept in registers, W applied, the result written back
//     for block i + 1 to read in its own layout;
//   - backward, from the top block down: a_i goes back to LDS, the gradient
//     sums of the block are taken from LDS, W^H is applied to the cotangent
//     in registers, which returns to LDS in place.
//
// Gradient sums: the joint sums of a block,
//     P[m][m'] = sum over the blocks of the tile of c[m] conj(a[m']),
// m, m' < 16 the positions inside a block, are a contraction over blocks and
// run on the matrix cores (16x16x4: lane (p, k) supplies position p of block k
// for both operands; complex data as re re + im im, im re and re im).
// The sums of every digit of the block follow from P alone (Eq. (1), factors
// act digit by digit): with the other digits e of the block carried through W,
//     gW_d[r][q] = sum over m_d = r, m'_d = q of P[m][m'] prod_e conj(W[m_e][m'_e]),
// so no activation inside a block is formed, and that product is taken once
// per work-group, in FP64.  The sums take FP64 matrix instructions, or FP32 ones
// in chains of kRegChain steps that are added into FP64 sums per lane, where that is
// as accurate as before (kRegF64; one chain of 16 steps: error of gW 2.5e-7
// against 1.9e-7 with four, 256 x 4^6 complex64).  A top block of fewer than RD digits has
// its own P, whose remaining field bits only pair with themselves.
//
// A wave takes the sums over exactly the blocks that its own threads hold, so
// sums and in-place cotangent update need no barrier between them: one
// barrier a block.
//
// What bounds it: matrix-core issue and latency at two waves per SIMD
// (complex; the registers and the LDS both allow two), HBM for two-digit
// blocks.  MI355X, 64 x 4^10 complex64, groups of 6 and 4 digits: 539 + 392 us
// against 1753 + 1230 us for the LDS-slot kernel (gtt_bwd_block_kernel: 14 LDS
// phases a tile instead of 5, 2236 VALU instructions a wave and tile of 4
// elements a thread), floor 300 us each at the copy rate; 64 x 2^20 (FP64 sums): 822
// + 541 against 1576 + 1232 us; 64 x 4^10 float 220 + 184 against 561 + 488 us; one
// to a few tiles (32 x 4^5 float) 12-14 against 17.4 us; radix 16 against
// gtt_bwd_mfma_kernel: 256 x 16^4 bf16 59 + 26 against 158 + 59 us, 64 x 16^5 f16
// 209 + 164 against 616 + 693 us.
#pragma once

#include "gtt_bwd.hpp"
#include "gtt_reg.hpp"

namespace gtt {

// LDS position of tile element x: a pad element after every 16 and every 512.
// Additive over numbers with disjoint bits.  The lanes of a wave that walk
// a block field or its complement meet at most one pair on a bank.
__host__ __device__ constexpr uint32_t reg_pos(uint32_t x) { return x + (x >> 4) + (x >> 9); }

template <int B, int K, int LOGT, bool ROW>
struct RegGeom {
    static constexpr int LB = B == 2 ? 1 : B == 4 ? 2 : 4;
    static constexpr int RD = 4 / LB;
    static constexpr int NBLK = (K + RD - 1) / RD;
    static constexpr int LOGC = ROW ? LOGT - K * LB : 0;
    static constexpr int NT = 1 << (LOGT - 4);
    static constexpr uint32_t TE = 1u << LOGT;
    static constexpr uint32_t TP = reg_pos(TE - 1) + 1;  // LDS elements of a tile
    static_assert(LOGC >= 0 && K * LB + LOGC <= LOGT && K >= 1, "tile bits");
    static constexpr int digits(int i) { return i < NBLK - 1 ? RD : K - RD * (NBLK - 1); }
    // lowest bit of block i's register field, and of its digits inside it
    static constexpr int field(int i) {
        const int s = LOGC + LB * RD * i;
        return s > LOGT - 4 ? LOGT - 4 : s;
    }
    static constexpr int doff(int i) { return LOGC + LB * RD * i - field(i); }
    static constexpr bool kFull = NBLK > 1 || K == RD;  // some block has RD digits
    static constexpr bool kPart = K % RD != 0;          // the top block has fewer
};

// orders a wave's own LDS writes before its other lanes' reads, and back
__device__ __forceinline__ void reg_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The thread-index bit (of the low six, a wave's) that lane bit 4 stands for
// in the gradient sums' reads: the one with the fewest bank conflicts among
// 32 lanes (16 field positions x that bit).
template <int FS>
constexpr int reg_pbit() {
    int best = 0, bc = 1 << 20;
    for (int b = 0; b < 6; ++b) {
        int cnt[32] = {0}, worst = 0;
        for (int l = 0; l < 32; ++l) {
            const uint32_t x = ((uint32_t)(l & 15) << FS) | reg_insert((uint32_t)(l >> 4) << b, FS);
            const int k = (int)(reg_pos(x) & 31u);
            ++cnt[k];
        }
        for (int k = 0; k < 32; ++k) worst += cnt[k] * cnt[k];
        if (worst < bc) {
            bc = worst;
            best = b;
        }
    }
    return best;
}

// thread-index bits of a wave's block number i (0..63): the low two bits of i
// are lane bits 4 and 5 (pbit, then the lowest other bit), the rest the step
template <int FS>
__host__ __device__ constexpr uint32_t reg_wave_block(uint32_t i) {
    constexpr int p0 = reg_pbit<FS>();
    constexpr int p1 = p0 == 0 ? 1 : 0;
    uint32_t t = ((i & 1u) << p0) | (((i >> 1) & 1u) << p1);
    uint32_t s = i >> 2;
    for (int b = 0; b < 6; ++b)
        if (b != p0 && b != p1) {
            t |= (s & 1u) << b;
            s >>= 1;
        }
    return t;
}

// The tile elements of a thread in a block's layout: bits of the thread index,
// plus those of register m.  Radix 2 and 4: the thread holds one block, m its
// positions.  Radix 16: the operand (and result) layout of the 16x16x4 MFMA
// with W's rows permuted to match: lane (q, i) holds elements q + 4v (v < 4) of
// four fibres, i plus 16 g within the wave's 64; register m = 4 g + v.
template <int B, int FS>
__device__ __forceinline__ uint32_t reg_lane(uint32_t tid) {
    if constexpr (B == 16)
        return reg_insert((tid & 15u) | (tid & ~63u), FS) | (((tid >> 4) & 3u) << FS);
    else
        return reg_insert(tid, FS);
}
template <int B, int FS>
__host__ __device__ constexpr uint32_t reg_elem(uint32_t m) {
    return B == 16 ? reg_insert((m >> 2) << 4, FS) | ((4u * (m & 3u)) << FS) : m << FS;
}

// W of the whole launch: radix 2 in scalar registers (the adjoint reads it
// transposed and conjugated), radix 4 and 16 as the MFMA operands of W and W^H
template <typename C, int B>
struct RegW {
    C w[4];
    __device__ __forceinline__ void load(const C* __restrict__ Wg) {
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = Wg[e];
    }
};
template <typename C>
struct RegW<C, 4> {
    W4<C> f, h;
    __device__ __forceinline__ void load(const C* __restrict__ Wg) {
        w4_load(f, Wg, false);
        w4_load(h, Wg, true);
    }
};

// radix 16: column q + 4v of row i / 4 + 4 (i % 4) of W and of W^T in lane
// (q, i), step v
template <>
struct RegW<float, 16> {
    float f[4], h[4];
    __device__ __forceinline__ void load(const float* __restrict__ Wg) {
        const uint32_t i = threadIdx.x & 15u, q = (threadIdx.x >> 4) & 3u, r = (i >> 2) + 4u * (i & 3u);
#pragma unroll
        for (uint32_t v = 0; v < 4; ++v) {
            f[v] = Wg[r * 16u + q + 4u * v];
            h[v] = Wg[(q + 4u * v) * 16u + r];
        }
    }
};

template <bool ADJ>
__device__ __forceinline__ void reg_digit16(float (&x)[16], const RegW<float, 16>& w) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 4; ++v)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ADJ ? w.h[v] : w.f[v], x[4 * g + v], acc, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) x[4 * g + v] = acc[v];
    }
}

template <typename C, int B, int LB, int R, int DOFF, bool ADJ>
__device__ __forceinline__ void reg16_block(C (&v)[16], const RegW<C, B>& w) {
    if constexpr (B == 16) {
        reg_digit16<ADJ>(v, w);
    } else {
        static_for<0, R>([&](auto d) {
            // digits in ascending order forward, descending backward
            constexpr int dd = ADJ ? R - 1 - decltype(d)::value : decltype(d)::value;
            if constexpr (B == 4)
                reg_digit4<16, (1 << (DOFF + dd * LB))>(v, ADJ ? w.h : w.f);
            else
                reg_digit2<C, B, 16, (1 << (DOFF + dd * LB)), ADJ>(v, w.w);
        });
    }
}

// FP64 sums of one kind of block: a lane's four entries of the 16x16 blocks
// (real: c a; complex: real and imaginary part of c conj(a)).
template <typename C>
struct RegSums;
template <>
struct RegSums<float> {
    f64x4 re;
    __device__ __forceinline__ void clear() { re = f64x4{0.0, 0.0, 0.0, 0.0}; }
};
template <>
struct RegSums<cf> {
    f64x4 re, im;
    __device__ __forceinline__ void clear() { re = im = f64x4{0.0, 0.0, 0.0, 0.0}; }
};

// kRegF64: products and sums in FP64 (the FP64 MFMA, half the FP32 rate);
// otherwise FP32 chains of kRegChain steps, added into the FP64 sums.  FP64 for
// radix 2 and for float radix 4, and for contiguous groups of few digits (complex
// radix 4 up to three, radix 16 up to two; a strided group has a contiguous one
// below it): there the activations carry so little rounding that the chains
// would set the error of gW.  Mean over six random inputs against 64 bits,
// with FP32 chains -> FP64: 1021 x 2 complex64 6.8e-8 -> 2.2e-8, 1021 x 2^4 1.0e-7
// -> 2.1e-8, 1021 x 4 9.2e-8 -> 2.5e-8, 1021 x 4^3 1.1e-7 -> 6.7e-8, 1021 x 16 float
// 7.8e-8 -> 2.6e-8, 61 x 16^2 1.1e-7 -> 7.9e-8; with more digits the chains stay
// at or below the LDS-slot kernels (which sum radix 2 and real radix 4 in FP64 and
// chain complex radix 4 and radix 16 over a tile): 61 x 4^7 complex64 1.4e-7 both, 256
// x 4^6 1.2e-7 for 1.4e-7, 16 x 16^4 float 1.6e-7 for 2.0e-7.  The FP64 step costs 4-25 % of the
// launch (2097153 x 4 complex64 41 -> 44 us, 4097 x 2^11 100 -> 122).
// The row of entry v of a lane: lane / 16 + 4 v with the FP64 instruction,
// 4 (lane / 16) + v with the FP32 one.
template <typename C, int B, int K, bool ROW>
constexpr bool kRegF64 = B == 2 || (B == 4 && std::is_same<C, float>::value) || (!ROW && K <= (B == 4 ? 3 : 2));
constexpr int kRegChain = 4;

// LDS position of the operand of lane `lane` in step 0 (its field position in
// block reg_wave_block(lane >> 4) of its wave), and the part of step s
template <int FS>
__device__ __forceinline__ uint32_t reg_sum_base(uint32_t lane, uint32_t wave) {
    return reg_pos((lane & 15u) << FS) + reg_pos(reg_insert(reg_wave_block<FS>(lane >> 4), FS)) +
           reg_pos(reg_insert(wave << 6, FS));
}
template <int FS>
__host__ __device__ constexpr uint32_t reg_sum_step(uint32_t s) {
    return reg_pos(reg_insert(reg_wave_block<FS>(s << 2), FS));
}

// The 16 steps run as a loop of 16 / CH chains of CH steps (not unrolled:
// with all operands in flight at once the kernel spills)
template <int FS, int CH, bool F64>
__device__ __forceinline__ void reg_sums(const float* Cb, const float* Ab, uint32_t lane, uint32_t wave,
                                         RegSums<float>& M) {
    const uint32_t p0 = reg_sum_base<FS>(lane, wave);
#pragma unroll 1
    for (uint32_t g = 0; g < 16; g += CH) {
        const uint32_t p = p0 + reg_sum_step<FS>(g);
        [[maybe_unused]] f32x4 D = {0.f, 0.f, 0.f, 0.f};
        static_for<0, CH>([&](auto s) {
            constexpr uint32_t o = reg_sum_step<FS>((uint32_t)decltype(s)::value);
            if constexpr (F64)
                M.re = __builtin_amdgcn_mfma_f64_16x16x4f64((double)Cb[p + o], (double)Ab[p + o], M.re, 0, 0, 0);
            else
                D = __builtin_amdgcn_mfma_f32_16x16x4f32(Cb[p + o], Ab[p + o], D, 0, 0, 0);
        });
        if constexpr (!F64) {
#pragma unroll
            for (int v = 0; v < 4; ++v) M.re[v] += (double)D[v];
        }
    }
}
template <int FS, int CH, bool F64>
__device__ __forceinline__ void reg_sums(const cf* Cb, const cf* Ab, uint32_t lane, uint32_t wave, RegSums<cf>& M) {
    const uint32_t p0 = reg_sum_base<FS>(lane, wave);
#pragma unroll 1
    for (uint32_t g = 0; g < 16; g += CH) {
        const uint32_t p = p0 + reg_sum_step<FS>(g);
        [[maybe_unused]] f32x4 Dr = {0.f, 0.f, 0.f, 0.f}, Di = Dr, Dx = Dr;
        static_for<0, CH>([&](auto s) {
            constexpr uint32_t o = reg_sum_step<FS>((uint32_t)decltype(s)::value);
            const cf c = Cb[p + o], a = Ab[p + o];
            if constexpr (F64) {
                const double cr = (double)c.re, ci = (double)c.im, ar = (double)a.re, ai = (double)a.im;
                M.re = __builtin_amdgcn_mfma_f64_16x16x4f64(cr, ar, M.re, 0, 0, 0);
                M.im = __builtin_amdgcn_mfma_f64_16x16x4f64(ci, ar, M.im, 0, 0, 0);
                M.re = __builtin_amdgcn_mfma_f64_16x16x4f64(ci, ai, M.re, 0, 0, 0);
                M.im = __builtin_amdgcn_mfma_f64_16x16x4f64(-cr, ai, M.im, 0, 0, 0);
                return;
            }
            Dr = __builtin_amdgcn_mfma_f32_16x16x4f32(c.re, a.re, Dr, 0, 0, 0);
            Di = __builtin_amdgcn_mfma_f32_16x16x4f32(c.im, a.re, Di, 0, 0, 0);
            Dx = __builtin_amdgcn_mfma_f32_16x16x4f32(c.re, a.im, Dx, 0, 0, 0);
            Dr = __builtin_amdgcn_mfma_f32_16x16x4f32(c.im, a.im, Dr, 0, 0, 0);
        });
        if constexpr (!F64) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                M.re[v] += (double)Dr[v];
                M.im[v] += (double)Di[v] - (double)Dx[v];
            }
        }
    }
}

__device__ __forceinline__ double reg_acc(const RegSums<float>& M, int v, double) { return M.re[v]; }
__device__ __forceinline__ cd reg_acc(const RegSums<cf>& M, int v, cd) { return cd{M.re[v], M.im[v]}; }
__device__ __forceinline__ double reg_wconj(float w) { return (double)w; }
__device__ __forceinline__ cd reg_wconj(cf w) { return cd{(double)w.re, -(double)w.im}; }

// This work-group's gW entry (thread t < B*B) from one kind of block: the
// waves' P added in wave order, then the contraction with W above.  Thread t <
// 256 takes entry (r, q) = t % B^2 of every digit's gradient and one of the
// 256 / B^2 values of the other field bits of (m, m'); the threads of an entry
// are folded over the lanes of a wave, then over the four waves in order.
// smem: NT / 64 copies of P, W, and the waves' folds.
template <typename C, typename Acc, int B, int LB, int R, int DOFF, int NT, bool F64>
__device__ __forceinline__ Acc reg_finish(const RegSums<C>& M, unsigned char* smem, const C* __restrict__ Wg) {
    constexpr int BB = B * B, OB = 4 - LB, NW = NT / 64;
    static_assert(BB <= 16 || (B == 16 && R == 1 && DOFF == 0), "radix 2, 4 or 16");
    Acc* P = reinterpret_cast<Acc*>(smem);
    Acc* red = P + NW * 256;
    C* Wl = reinterpret_cast<C*>(red + 4 * BB);
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6;
    __syncthreads();
#pragma unroll
    for (int v = 0; v < 4; ++v)
        P[wave * 256u + (F64 ? (lane >> 4) + 4u * (uint32_t)v : 4u * (lane >> 4) + (uint32_t)v) * 16u + (lane & 15u)] =
            reg_acc(M, v, Acc{});
    if (t < BB) Wl[t] = Wg[t];
    __syncthreads();
    if (t < 256) {
        Acc x = P[t];
#pragma unroll
        for (int w = 1; w < NW; ++w) x = acc_add(x, P[w * 256 + t]);
        P[t] = x;  // entries are read and written by this thread alone
    }
    if constexpr (B == 16) {  // one digit a block: P is gW
        return t < 256 ? P[t] : acc_zero(Acc{});
    }
    __syncthreads();
    if (t < 256) {
        constexpr uint32_t used = ((1u << (R * LB)) - 1u) << DOFF;  // field bits that are digits
        const uint32_t o = t % BB, r = o / B, q = o % B, mo = (t / BB) >> OB, no = (t / BB) & ((1u << OB) - 1u);
        Acc s = acc_zero(Acc{});
#pragma unroll
        for (int d = 0; d < R; ++d) {
            constexpr uint32_t dm = B - 1;
            const uint32_t at = DOFF + d * LB, low = (1u << at) - 1u;
            const uint32_t m = ((mo & ~low) << LB) | (r << at) | (mo & low);
            const uint32_t n = ((no & ~low) << LB) | (q << at) | (no & low);
            Acc x = P[m * 16u + n];
#pragma unroll
            for (int f = 0; f < R; ++f)
                if (f != d) x = cmul(reg_wconj(Wl[((m >> (DOFF + f * LB)) & dm) * B + ((n >> (DOFF + f * LB)) & dm)]), x);
            if (((m ^ n) & ~used & 15u) == 0) s = acc_add(s, x);
        }
#pragma unroll
        for (int h = 32; h >= BB; h >>= 1) s = acc_add(s, acc_shfl_down(s, h));
        if (lane < BB) red[wave * BB + lane] = s;
    }
    __syncthreads();
    Acc tot = acc_zero(Acc{});
    if (t < BB) {
        tot = red[t];
#pragma unroll
        for (int w = 1; w < 4; ++w) tot = acc_add(tot, red[w * BB + t]);
    }
    return tot;
}

// waves per SIMD the kernel is compiled for: the two tiles' LDS (68 KiB) leaves
// room for two work-groups a compute unit, of 256 threads for complex data and of
// 512 for float data
template <typename C, int LOGT>
struct RegWaves {
    static constexpr int value = sizeof(C) == 8 ? 2 : 4;
};

template <typename T, int B, int K, int LOGT, bool ROW>
__global__ __launch_bounds__(1 << (LOGT - 4))
__attribute__((amdgpu_waves_per_eu(RegWaves<typename Tr<T>::C, LOGT>::value))) void gtt_bwd_reg_kernel(BwdArgs ba) {
    using C = typename Tr<T>::C;
    using Gm = RegGeom<B, K, LOGT, ROW>;
    using Acc = typename AccOf<C>::type;
    constexpr int LB = Gm::LB, RD = Gm::RD, NBLK = Gm::NBLK, NT = Gm::NT, LOGC = Gm::LOGC;
    constexpr int V = 16 / (int)sizeof(T), NV = 16 / V;
    constexpr bool F64 = kRegF64<C, B, K, ROW>;
    // strided tiles: the last block's result goes straight to global memory
    // where its lanes run along a row
    constexpr bool kDirect = ROW && B != 16;
    const PassArgs& a = ba.p;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    C* Ab = reinterpret_cast<C*>(smem_raw);
    C* Cb = Ab + Gm::TP;
    const C* __restrict__ Wg = static_cast<const C*>(a.W);
    RegW<C, B> w;
    w.load(Wg);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
    RegSums<C> Mf, Mp;
    Mf.clear();
    Mp.clear();

    const int64_t total = a.N;  // elements of the buffers (the last contiguous tile may be partial)
    // Element x of a tile lies at the tile's base plus x (contiguous) or
    // (x >> LOGC) S + x mod C (rows), which is additive over disjoint bits: a
    // uniform 64-bit base per access plus one 32-bit byte offset per lane
    // (G S sizeof(T) < 2^31: the planner's rule)
    const uint32_t S32 = ROW ? (uint32_t)a.S : 0u;
    auto gofs = [&](uint32_t x) -> uint32_t {
        return (ROW ? (x >> LOGC) * S32 + (x & ((1u << LOGC) - 1u)) : x) * (uint32_t)sizeof(T);
    };
    auto tile_base = [&](int64_t t) -> int64_t {
        if constexpr (!ROW) return t << LOGT;
        const int64_t hb = tile_hb(a, t);
        return hb * ((int64_t)a.G * a.S) + ((t - hb * a.L) << LOGC);
    };
    // vector m of this thread: tile element e0 + m NT V.  The lane parts are
    // recomputed for every tile from an opaque thread index: hoisted out of the
    // tile loop, the sums with each m's part would hold a register each.
    auto opaque_tid = [&]() -> uint32_t {
        uint32_t x = tid;
        asm volatile("" : "+v"(x));
        return x;
    };
    uint4 ra[NV], rc[NV];
    auto fetch = [&](int64_t t) {
        const int64_t g0 = tile_base(t);
        const uint32_t e0 = opaque_tid() * V, lo0 = gofs(e0);
        const char* pa = reinterpret_cast<const char*>(static_cast<const T*>(a.in) + g0);
        const char* pc = reinterpret_cast<const char*>(static_cast<const T*>(ba.c_out) + g0);
        if (ROW || ((t + 1) << LOGT) <= total) {  // uniform
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                ra[m] = gload16<true>(pa + gofs((uint32_t)m * NT * V) + lo0);
                rc[m] = gload16<true>(pc + gofs((uint32_t)m * NT * V) + lo0);
            }
        } else {
            const uint32_t left = (uint32_t)(total - g0);
#pragma unroll
            for (int m = 0; m < NV; ++m) {
                ra[m] = rc[m] = make_uint4(0u, 0u, 0u, 0u);
                if (e0 + (uint32_t)m * NT * V < left) {
                    ra[m] = gload16<true>(pa + gofs((uint32_t)m * NT * V) + lo0);
                    rc[m] = gload16<true>(pc + gofs((uint32_t)m * NT * V) + lo0);
                }
            }
        }
    };
    auto put = [&](C* buf, const uint4 (&r)[NV]) {
        const uint32_t p0 = reg_pos(opaque_tid() * V);
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            T vals[V];
            *reinterpret_cast<uint4*>(vals) = r[m];
#pragma unroll
            for (int e = 0; e < V; ++e) buf[p0 + reg_pos((uint32_t)m * NT * V) + e] = to_c(vals[e]);
        }
    };

    int64_t t = blockIdx.x;
    if (t < a.ntiles) fetch(t);
    for (; t < a.ntiles; t += gridDim.x) {
        put(Ab, ra);
        put(Cb, rc);
        __syncthreads();
        C A[NBLK > 1 ? NBLK - 1 : 1][16];
        static_for<0, NBLK - 1>([&](auto ib) {
            constexpr int i = decltype(ib)::value;
            constexpr int FS = Gm::field(i);
            const uint32_t p = reg_pos(reg_lane<B, FS>(tid));
            C v[16];
#pragma unroll
            for (int m = 0; m < 16; ++m) v[m] = A[i][m] = Ab[p + reg_pos(reg_elem<B, FS>((uint32_t)m))];
            reg16_block<C, B, LB, RD, 0, false>(v, w);
#pragma unroll
            for (int m = 0; m < 16; ++m) Ab[p + reg_pos(reg_elem<B, FS>((uint32_t)m))] = v[m];
            __syncthreads();
        });
        static_for<0, NBLK>([&](auto ib) {
            constexpr int i = NBLK - 1 - decltype(ib)::value;
            constexpr int FS = Gm::field(i), R = Gm::digits(i), DOFF = Gm::doff(i);
            const uint32_t p = reg_pos(reg_lane<B, FS>(tid));
            if constexpr (i < NBLK - 1) {
                // the activation at the start of this block, back to the
                // positions it came from (only this wave reads them now)
#pragma unroll
                for (int m = 0; m < 16; ++m) Ab[p + reg_pos(reg_elem<B, FS>((uint32_t)m))] = A[i][m];
            }
            if constexpr (i == 0) {
                if (t + gridDim.x < a.ntiles) fetch(t + gridDim.x);
            }
            reg_wave_sync();
            if constexpr (R == RD)
                reg_sums<FS, kRegChain, F64>(Cb, Ab, lane, wave, Mf);
            else
                reg_sums<FS, kRegChain, F64>(Cb, Ab, lane, wave, Mp);
            reg_wave_sync();
            if (i > 0 || a.out) {
                C v[16];
#pragma unroll
                for (int m = 0; m < 16; ++m) v[m] = Cb[p + reg_pos(reg_elem<B, FS>((uint32_t)m))];
                reg16_block<C, B, LB, R, DOFF, true>(v, w);
                if constexpr (i == 0 && kDirect) {
                    // straight to global memory: lanes run along a row
                    char* po = reinterpret_cast<char*>(static_cast<T*>(a.out) + tile_base(t));
                    const uint32_t lo = gofs(reg_lane<B, FS>(opaque_tid()));
#pragma unroll
                    for (int m = 0; m < 16; ++m) *reinterpret_cast<T*>(po + gofs(reg_elem<B, FS>((uint32_t)m)) + lo) = from_c<T>(v[m]);
                } else {
#pragma unroll
                    for (int m = 0; m < 16; ++m) Cb[p + reg_pos(reg_elem<B, FS>((uint32_t)m))] = v[m];
                }
            }
            __syncthreads();
        });
        if constexpr (!kDirect) {
            if (a.out) {
                const int64_t g0 = tile_base(t);
                char* po = reinterpret_cast<char*>(static_cast<T*>(a.out) + g0);
                const uint32_t left = !ROW && total - g0 < (int64_t)Gm::TE ? (uint32_t)(total - g0) : Gm::TE;
                const uint32_t e0 = opaque_tid() * V, lo0 = gofs(e0), p0 = reg_pos(e0);
#pragma unroll
                for (int m = 0; m < NV; ++m) {
                    T vals[V];
#pragma unroll
                    for (int e = 0; e < V; ++e) vals[e] = from_c<T>(Cb[p0 + reg_pos((uint32_t)m * NT * V) + e]);
                    if (e0 + (uint32_t)m * NT * V < left)
                        gstore16<true>(po + gofs((uint32_t)m * NT * V) + lo0, *reinterpret_cast<const uint4*>(vals));
                }
                __syncthreads();
            }
        }
    }
    Acc tot = acc_zero(Acc{});
    if constexpr (Gm::kFull) tot = reg_finish<C, Acc, B, LB, RD, 0, NT, F64>(Mf, smem_raw, Wg);
    if constexpr (Gm::kPart)
        tot = acc_add(tot, reg_finish<C, Acc, B, LB, Gm::digits(NBLK - 1), Gm::doff(NBLK - 1), NT, F64>(Mp, smem_raw, Wg));
    if (tid < B * B) (static_cast<Acc*>(ba.partials) + (size_t)blockIdx.x * ba.wslot)[tid] = tot;
}

// log2 of the tile of the register backward for compute type C: 4096
// complex, 8192 float elements (32 KiB)
template <typename C>
constexpr int reg_logt() {
    return sizeof(C) == 8 ? 12 : 13;
}

template <typename T, int B, int K, bool ROW>
inline hipError_t launch_bwd_reg_one(const BwdArgs& a, unsigned grid, hipStream_t s) {
    using C = typename Tr<T>::C;
    constexpr int LOGT = reg_logt<C>();
    using Gm = RegGeom<B, K, LOGT, ROW>;
    return bwd_launch_one(gtt_bwd_reg_kernel<T, B, K, LOGT, ROW>, a, grid, Gm::NT, 2 * (size_t)Gm::TP * sizeof(C), s);
}

template <typename T, int B, int K>
inline hipError_t launch_bwd_reg_k(const BwdArgs& a, int k, bool row, unsigned grid, hipStream_t s) {
    constexpr int LB = RegGeom<B, 1, reg_logt<typename Tr<T>::C>(), false>::LB;
    constexpr int LOGT = reg_logt<typename Tr<T>::C>();
    if constexpr (K * LB > LOGT) {
        return hipErrorInvalidValue;
    } else {
        if (k > K) return launch_bwd_reg_k<T, B, K + 1>(a, k, row, grid, s);
        if (!row) return launch_bwd_reg_one<T, B, K, false>(a, grid, s);
        // rows of at least kRegMinRow bytes
        if constexpr (((size_t)1 << (LOGT - K * LB)) * sizeof(T) >= kRegMinRow) return launch_bwd_reg_one<T, B, K, true>(a, grid, s);
        return hipErrorInvalidValue;
    }
}

}  // namespace gtt

#define GTT_BWD_REG_INSTANTIATE(NAME, T, B)                                                               \
    namespace gtt {                                                                                      \
    hipError_t launch_bwd_reg_##NAME##_b##B(const BwdArgs& a, int k, bool row, unsigned grid, hipStream_t s) { \
        return launch_bwd_reg_k<T, B, 1>(a, k, row, grid, s);                                             \
    }                                                                                                    \
    }
