// Device-side building blocks of the FO-SGD codec kernels (gfx950, wave64).
//
// Tile model.  Every kernel works on tiles of 2^15 coordinates held entirely in the registers
// of one 512-thread workgroup: 64 values per thread.  A Walsh-Hadamard stage on index bit k is
// a butterfly between two registers of one thread whenever bit k is mapped to the register
// number; the kernels therefore alternate "register rounds" (six stages each, no data
// movement) with exchanges through LDS that remap which index bits live in registers.
// Stages commute, so each kernel visits the bits in the order that suits its memory layout.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace fo {

constexpr int kTileLog2 = 15;
constexpr uint32_t kTile = 1u << kTileLog2;
constexpr int kThreads = 512;
constexpr int kV = 64;             // values per thread
constexpr uint32_t kXWords = 16896; // exchange buffer: 128 rows of 128 words padded to 132
constexpr uint32_t kEpsWords = 1024;
constexpr uint32_t kLamWords = 512;
constexpr uint32_t kRedWords = 520;
constexpr uint32_t kLdsWords = kXWords + kEpsWords + kLamWords + kRedWords;

// Layout of the int16 intermediate of blocks of 2^26 and 2^27 between the low and the strided stages.  A strided tile is 16
// or 8 columns wide there, pieces of 32 or 16 bytes of every row; row-major they would lie far apart.  Columns go in
// groups of 64, one 128-byte line a row, the rows of a group one after the other: tiles that share lines read one
// contiguous region.  A group is followed by a line of padding, so that groups are not a power of two apart.
// n = 2^27, four workers: server pass 1118 -> 1045 us, low pass 206 -> 216 us.
struct Grouped16 {
    static __device__ __forceinline__ constexpr uint32_t group(uint32_t log_rows) { return (64u << log_rows) + 64u; } // elements
};

constexpr uint32_t kDomainEps = 1u;
constexpr uint32_t kDomainDither = 2u;

// ---------------------------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64 multiplies whose high
// halves are mixed with the neighbouring words and the round key; the key advances by two Weyl
// increments per round.  The key schedule is wave-uniform and lives in scalar registers.
// ---------------------------------------------------------------------------------------------
struct RngKey {
    uint32_t k0, k1; // key: seed low word, seed high word xor round high word
    uint32_t c1;     // domain | k << 8
    uint32_t c2;     // round low word
    uint32_t c3;     // party
};

__device__ __forceinline__ void philox(uint32_t counter, const RngKey &key, uint32_t (&out)[4])
{
    uint32_t x0 = counter, x1 = key.c1, x2 = key.c2, x3 = key.c3;
    uint32_t ka = key.k0, kb = key.k1;
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        // full 64-bit products: one v_mad_u64_u32 each instead of a low and a high multiply
        const uint64_t pa = (uint64_t)x0 * 0xD2511F53u;
        const uint64_t pb = (uint64_t)x2 * 0xCD9E8D57u;
        // three-input xor (truth table 0x96) in one v_bitop3_b32
        x0 = __builtin_amdgcn_bitop3_b32((uint32_t)(pb >> 32), x1, ka, 0x96);
        x2 = __builtin_amdgcn_bitop3_b32((uint32_t)(pa >> 32), x3, kb, 0x96);
        x1 = (uint32_t)pb;
        x3 = (uint32_t)pa;
        ka += 0x9E3779B9u;
        kb += 0xBB67AE85u;
    }
    out[0] = x0; out[1] = x1; out[2] = x2; out[3] = x3;
}

// The round counter enters the generator key (low word as counter word 2, high word xored into key word 1).
// It is either fixed at launch (dev == nullptr: k1_in already holds the xor) or read from device memory when
// the kernel runs, so that a captured graph can be replayed for one round after the other.
__device__ __forceinline__ void resolve_round(uint32_t k1_in, uint32_t lo_in, const unsigned long long *dev, uint32_t &k1,
                                              uint32_t &lo)
{
    k1 = k1_in;
    lo = lo_in;
    if (dev) {
        const unsigned long long r = *dev;
        lo = (uint32_t)r;
        k1 = k1_in ^ (uint32_t)(r >> 32);
    }
}

// ---------------------------------------------------------------------------------------------
// Small helpers
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ void wave_sync()
{
    // Orders LDS traffic between lanes of one wave: the LDS queue of a wave is in order, the
    // fences keep the compiler from moving accesses across this point.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ float flip_if(float x, uint32_t bit) // bit in {0,1}
{
    return __uint_as_float(__float_as_uint(x) ^ (bit << 31));
}
// x with its sign flipped when bit 31 of w is set: x ^ (w & 0x80000000) as one three-input operation
__device__ __forceinline__ float flip_by_bit31(float x, uint32_t w)
{
    return __uint_as_float(__builtin_amdgcn_bitop3_b32(__float_as_uint(x), w, 0x80000000u, 0x78));
}

// Load through a base pointer that is the same in every lane (held in scalar registers: the load takes the
// "scalar base + 32-bit lane offset" addressing form instead of 64-bit vector adds) plus a per-lane byte offset.
template <typename T>
__device__ __forceinline__ T ld_uniform(const void *uniform_base, uint32_t byte_off)
{
    typedef const __attribute__((address_space(1))) char *gptr;
    const uint64_t v = reinterpret_cast<uint64_t>(uniform_base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    const gptr g = (gptr)(((uint64_t)hi << 32) | lo);
    return *(const __attribute__((address_space(1))) T *)(g + byte_off);
}
template <typename T>
__device__ __forceinline__ void st_uniform(void *uniform_base, uint32_t byte_off, T value)
{
    typedef __attribute__((address_space(1))) char *gptr;
    const uint64_t v = reinterpret_cast<uint64_t>(uniform_base);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    const gptr g = (gptr)(((uint64_t)hi << 32) | lo);
    *(__attribute__((address_space(1))) T *)(g + byte_off) = value;
}

// The same by bit 0 of n: 2^31 n added to the bits, one v_lshl_add_u32.  flip_next brings the next bit to bit 0 in a shift of
// its own (v_lshrrev_b32 by a constant issues in half the time of v_lshlrev_b32 or v_bitop3_b32); without the barrier the
// compiler joins the two shifts and needs a mask and an addition more.
__device__ __forceinline__ float flip_by_bit0(float x, uint32_t n) { return __uint_as_float(__float_as_uint(x) + (n << 31)); }
__device__ __forceinline__ uint32_t flip_next(uint32_t n)
{
    n >>= 1;
    asm("" : "+v"(n));
    return n;
}

template <typename T, int BIT, int V = kV>
__device__ __forceinline__ void bfly(T (&v)[V])
{
    static_assert((1 << BIT) < V, "stage bit outside the register index");
#pragma unroll
    for (int r = 0; r < V; ++r)
        if (!(r & (1 << BIT))) {
            const T a = v[r], b = v[r | (1 << BIT)];
            v[r] = a + b;
            v[r | (1 << BIT)] = a - b;
        }
}

// Compile-time loop: f(std::integral_constant<int, 0>{}), ..., f(std::integral_constant<int, N - 1>{})
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// Largest of the M workers' amplitudes of block gb ([M][nblocks]), NaN if any of them is NaN.
__device__ __forceinline__ float largest_scale(const float *scales, uint64_t nblocks, uint32_t M, uint64_t gb)
{
    float m = 0.f;
    bool nan = false;
    for (uint32_t n = 0; n < M; n += 8u) { // eight loads on their way together; the last worker's again where there are fewer
        float l[8];
#pragma unroll
        for (uint32_t i = 0; i < 8u; ++i) l[i] = scales[(uint64_t)(n + i < M ? n + i : M - 1u) * nblocks + gb];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            nan |= (l[i] != l[i]);
            m = fmaxf(m, l[i]);
        }
    }
    return nan ? __builtin_nanf("") : m;
}

// Step K of a butterfly sum: s plus the s of the lane whose number differs in bit K.  Lanes that differ below bit K only hold the
// same sum, so mirroring 8 or 16 lanes reaches the partner as well; bits 4 and 5 are the row swaps.  In registers: a shuffle goes
// through LDS, 100 cycles and more of a chain of six (step of 3 M coordinates in blocks of 2^9, M = 5, K = 4: 53.2 -> 48.9 us; of
// 10^6 in blocks of 2^8, M = 8: 32.3 -> 29.7; d = 1000, M = 2: 14.5 -> 14.2).
template <int K, typename T>
__device__ __forceinline__ T wave_sum_step(T s)
{
    constexpr int words = sizeof(T) / 4;
    struct Words { uint32_t w[words]; };
    const Words x = __builtin_bit_cast(Words, s);
    Words a = x, b;
#pragma unroll
    for (int i = 0; i < words; ++i) {
        if constexpr (K < 4) {
            constexpr int ctrl = K == 0 ? 0xB1 : K == 1 ? 0x4E : K == 2 ? 0x141 : 0x140; // quad_perm 1,0,3,2 | 2,3,0,1, row_half_mirror, row_mirror
            b.w[i] = (uint32_t)__builtin_amdgcn_mov_dpp((int)x.w[i], ctrl, 0xf, 0xf, true);
        } else if constexpr (K == 4) {
            const auto r = __builtin_amdgcn_permlane16_swap(x.w[i], x.w[i], false, false);
            a.w[i] = r[0]; b.w[i] = r[1];
        } else {
            const auto r = __builtin_amdgcn_permlane32_swap(x.w[i], x.w[i], false, false);
            a.w[i] = r[0]; b.w[i] = r[1];
        }
    }
    return __builtin_bit_cast(T, a) + __builtin_bit_cast(T, b);
}

template <typename T>
__device__ __forceinline__ T wave_sum(T s, int steps) // butterfly sum over 2^steps lanes, steps >= 4; every lane takes part
{
    static_for<4>([&](auto k) { s = wave_sum_step<decltype(k)::value>(s); });
    if (steps > 4) s = wave_sum_step<4>(s);
    if (steps > 5) s = wave_sum_step<5>(s);
    return s;
}

// The sum of a block's n partial sums by a workgroup of kThreads: every wave's part, then, behind a barrier, the whole of `part`
// (a double a wave).  Whoever wants an amplitude from partial sums takes it from here: the same one to the bit.
__device__ __forceinline__ void sum_of_partials(double *part, const float *p, uint32_t n, uint32_t t)
{
    double d = 0.0;
    for (uint32_t k = t; k < n; k += kThreads) d += (double)p[k];
    d = wave_sum(d, 6);
    if ((t & 63u) == 0u) part[t >> 6] = d;
}
__device__ __forceinline__ double sum_of_waves(const double *part)
{
    double s = 0.0;
    for (uint32_t k = 0; k < kThreads / 64u; ++k) s += part[k];
    return s;
}

// wave_sum by shuffles, for many independent sums in a kernel whose vector units are busier than its LDS (k_enc_wave; the step of
// 5 M coordinates, M = 4, in blocks of 2^7 65.5 us, 66.8 with the sums in registers).
__device__ __forceinline__ float wave_sum_shuffled(float s, int steps)
{
#pragma unroll
    for (int k = 0; k < 6; ++k)
        if (k < steps) s += __shfl_xor(s, 1 << k, 64);
    return s;
}

// v_writelane_b32 as the compiler's own intrinsic (this toolchain has no clang builtin for it, so the LLVM
// intrinsic is bound by name).  Unlike inline assembly, the compiler sees the instruction and inserts the wait
// states gfx950 needs between a vector compare that writes a scalar register pair and a vector instruction that
// reads it (two; back to back the lane write can pick up the register's previous contents).
extern "C" __device__ int fo_llvm_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// Returns v with lane LANE replaced by the wave-uniform value s (every other lane keeps its own).
template <int LANE>
__device__ __forceinline__ uint32_t write_lane(uint32_t v, uint32_t s)
{
    return (uint32_t)fo_llvm_writelane((int)s, LANE, (int)v);
}

// One Walsh-Hadamard stage on lane bit 5 (partner = lane ^ 32).  v_permlane32_swap trades the
// upper half-wave of its first operand with the lower half-wave of its second, which brings both
// ends of a butterfly into one lane; a second swap restores the layout.
template <typename T, int V>
__device__ __forceinline__ void bfly_lane5(T (&v)[V])
{
#pragma unroll
    for (int k = 0; k < V / 2; ++k) {
        uint32_t a = __builtin_bit_cast(uint32_t, v[k]), b = __builtin_bit_cast(uint32_t, v[k + V / 2]);
        auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        const T x = __builtin_bit_cast(T, (uint32_t)r[0]), y = __builtin_bit_cast(T, (uint32_t)r[1]);
        a = __builtin_bit_cast(uint32_t, (T)(x + y));
        b = __builtin_bit_cast(uint32_t, (T)(x - y));
        r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
        v[k] = __builtin_bit_cast(T, (uint32_t)r[0]);
        v[k + V / 2] = __builtin_bit_cast(T, (uint32_t)r[1]);
    }
}

// Swap register bit 5 with lane bit 5: afterwards v[k] of the upper half-wave and v[k+32] of
// the lower half-wave have traded places.
template <typename T>
__device__ __forceinline__ void swap_reg5_lane5(T (&v)[kV])
{
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        const uint32_t lo = __builtin_bit_cast(uint32_t, v[k]);
        const uint32_t hi = __builtin_bit_cast(uint32_t, v[k + 32]);
        // v_permlane32_swap: lanes 32..63 of the first operand trade with lanes 0..31 of the second
        const auto r = __builtin_amdgcn_permlane32_swap(lo, hi, false, false);
        v[k] = __builtin_bit_cast(T, (uint32_t)r[0]);
        v[k + 32] = __builtin_bit_cast(T, (uint32_t)r[1]);
    }
}

} // namespace fo
