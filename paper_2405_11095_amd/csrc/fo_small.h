// Kernels for short vectors: tiles of 2^12 coordinates, 256 threads with 16 values each.
//
// The kernels of fo_contig.h and fo_strided.h put 2^15 coordinates on one workgroup.  That is the better shape when
// there are enough tiles for every compute unit; a vector of few tiles leaves most of the chip idle and costs the time
// that one compute unit needs for 2^15 values (12 to 20 us a kernel, whatever the vector's length).  Here the same
// vector occupies eight times as many workgroups, each with an eighth of the work.  Everything is fp32: on the decode
// side the values are half integers below 2^23, so every sum is exact (the plan's rule sees to the bound).
// Measured, general kernels before and these after: one encode of 1000 coordinates 12.0 -> 7.3 us (kernel 4.9 us), a step of
// n = 2^16 with four workers 71.7 -> 24.2 us, n = 2^20 with eight 123 -> 53.9 us.  What bounds a kernel here is latency: one
// trip to memory, two exchanges and the generator's chain of ten rounds, 4 to 7 us each with few waves per SIMD.  At n = 2^20
// with eight workers the joined low pass takes 19.6 us with the vector units 49 % busy, at 58 instructions per value (the long
// kernels' encode and decode: 31 and 9).
//
// Transforms of up to 2^12 points (whole or blocked) take one pass, longer ones (up to 2^20 points) two: up to eight
// stages over rows 2^12 apart (k_small_high), twelve inside the contiguous tile (k_small_encode, k_small_decode).
// Since the low stages of the encoder and of the decoder act on the same tile, fo_step runs them in one kernel: the
// tile's signs go out as the message and straight back in as the decoder's input.
//
// k_small_block does both passes of an encode of up to 2^16 points in one launch without the intermediate, for the entry
// point that has no scratch of its own.
//
// Index-bit choreography of the contiguous tile (b0..b11 = bits of the tile-local coordinate):
//   L0 (16-byte loads): regs = (b0,b1,b8,b9)    lanes = (b2..b7)            waves = (b10,b11)
//   L1                : regs = (b2..b5)         lanes = (b0,b1,b8,b9,b6,b7) waves = (b10,b11)
//   L2 (outputs)      : regs = (b6,b7,b10,b11)  lanes = (b0..b5)            waves = (b8,b9)
// Coordinate c sits at LDS word c + 4 (c / 64): few bank conflicts in any of the three layouts (64 cycles per wave and
// transform by the counter, 5 to 9 % of a busy kernel's time), so L1 goes back to where it was
// read and the tile needs one workgroup barrier.
#pragma once
#include "fo_strided.h"

namespace fo {

constexpr int kSmLog2 = 12;
constexpr uint32_t kSmTile = 1u << kSmLog2;
constexpr uint32_t kSmThreads = 256;
constexpr uint32_t kSmXWords = kSmTile + kSmTile / 16; // 4 words of padding per 64, or 16 per 256 (k_small_high)
constexpr uint32_t kSmEpsWords = kSmTile / 32;
constexpr uint32_t kSmPlanes = 8;                      // bit planes of a K-fold message, at most

enum { SMI_GRAD = 0, SMI_MID = 1 };          // k_small_encode: the vector itself (b <= 2^12) | after the high stages
enum { SMS_GIVEN = 0, SMS_MEASURED = 1, SMS_SERVER = 2 }; // amplitude: read | from the measured norm | coef * max of the workers'
enum { SMH_ENC = 0, SMH_SERVER = 1, SMH_DEC = 2 };

struct SmallArgs {
    const float *src;          // encode: gradient or intermediate; high passes: intermediate   [slot]
    uint64_t src_stride;
    const uint64_t *bits_in;   // decode, server: packed signs [slot or worker][W] (or [plane][W])
    uint64_t bits_in_stride;
    uint64_t *bits_out;        // encode, server: packed signs [slot][W] (or [plane][W])
    uint64_t bits_out_stride;
    float *mid;                // fp32 intermediate written by this kernel [slot]
    uint64_t mid_stride;
    float *out;                // decoded vector: fp32 [len_out]
    float *gbar;               // server: optional copy of the mean, fp32 [ntot]
    float *scales;             // [slot][nblocks] amplitudes of the message being written or decoded
    uint64_t scales_stride;
    const float *scales_up;    // SMS_SERVER, server: the workers' amplitudes [M][nblocks]
    float *partials;           // [slot][ntiles] sums of squares of the high pass's tiles
    uint64_t len_in, len_out;  // valid coordinates of the input vector / of out
    uint64_t W, nblocks, ntiles;
    uint32_t S;                // stages inside the tile: min(log2 b, 12)
    uint32_t logb;
    uint32_t use_tab;
    uint32_t scale_mode;       // SMS_*
    uint32_t scales_only;      // encode, SMI_GRAD: write the amplitudes and stop
    uint32_t common;           // encode, SMI_MID: the amplitude is the largest of `common` slots' (0: the slot's own)
    uint32_t dither;
    uint32_t M, count;         // server, decode: workers; count: their signs are added before the transform (shared eps)
    uint32_t K, planes;        // quantiser of the message written
    uint32_t Kin, planes_in;   // of the message read
    uint32_t store_mode;
    uint32_t party0, eps_party0, eps_in; // writer of slot 0, its eps stream; eps stream(s) of the messages read
    uint32_t k0, k1, round_lo;
    const unsigned long long *round_dev;
    float coef;                // SMS_MEASURED: alpha sqrt(ln b / b); SMS_SERVER: factor on the workers' largest
    float sqrtb;
    float in_coef;             // server: value = lambda_n * in_coef * (half integer)
    float out_coef;            // decode: the same for out
    float delta;
    unsigned long long *stat_clipped, *stat_near; // optional diagnostic counters per slot (see ContigArgs)
};

struct SmallLds {
    alignas(16) float x[kSmXWords];
    uint32_t eps[kSmEpsWords];
    float lam[64];             // per block of the tile: the amplitude
    float kq[64];              // and the slope -128 / (lambda' 2^-24) of the integer-domain comparison
    float red[64];
    double red64[4];
    uint64_t words[kSmPlanes * 64];
};

// L0 -> L2 with the stages b0 .. b(S-1), S = 6 .. 12.  Callers pass a barrier between the last read here and the next
// write to x.
__device__ __forceinline__ void small_transform(float (&v)[16], uint32_t S, float *x, uint32_t lane, uint32_t wave)
{
    bfly<float, 0, 16>(v);
    bfly<float, 1, 16>(v);
    if (S > 8u) bfly<float, 2, 16>(v);
    if (S > 9u) bfly<float, 3, 16>(v);
    {
        float *const w = x + wave * 1088u + lane * 4u + 4u * (lane >> 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<float4 *>(w + 272 * q) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    }
    wave_sync();
    {
        float *const p = x + wave * 1088u + (lane & 3u) + (lane >> 4) * 68u + ((lane >> 2) & 3u) * 272u;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = p[4 * r];
        bfly<float, 0, 16>(v);
        bfly<float, 1, 16>(v);
        bfly<float, 2, 16>(v);
        bfly<float, 3, 16>(v);
#pragma unroll
        for (int r = 0; r < 16; ++r) p[4 * r] = v[r];
    }
    __syncthreads();
    {
        const float *const p = x + lane + wave * 272u;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = p[(r & 3) * 68 + (r >> 2) * 1088];
    }
    if (S > 6u) bfly<float, 0, 16>(v);
    if (S > 7u) bfly<float, 1, 16>(v);
    if (S > 10u) bfly<float, 2, 16>(v);
    if (S > 11u) bfly<float, 3, 16>(v);
}

// tile-local coordinate of register r in L2, without the lane
__device__ __forceinline__ uint32_t small_l2(int r, uint32_t wave)
{
    return (uint32_t)(r & 3) * 64u + wave * 256u + (uint32_t)(r >> 2) * 1024u;
}

// eps words of the tile for one stream, by the first 32 threads; the caller's next barrier publishes them
__device__ __forceinline__ void small_eps(uint32_t *eps, const SmallArgs &a, uint32_t rk1, uint32_t rlo, uint32_t party, uint64_t base)
{
    const uint32_t t = threadIdx.x;
    if (t < 32u) {
        const RngKey key = { a.k0, rk1, kDomainEps, rlo, party };
        uint32_t w[4];
        philox((uint32_t)(base >> 7) + t, key, w);
        *reinterpret_cast<uint4 *>(eps + 4u * t) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// The decoder's input in L0: half the values of a message, bit - 1/2, count - K/2 of a K-fold one, or the sum over
// the workers of bit - 1/2.  `word(p, w)` is word w (of the tile's 64) of plane or worker p.
template <typename F>
__device__ __forceinline__ void small_from_bits(float (&v)[16], uint32_t n, bool add, float half, uint32_t lane, uint32_t wave, F &&word)
{
    uint32_t c[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) c[r] = 0u;
    for (uint32_t p = 0; p < n; ++p) {
        const uint32_t sh = add ? 0u : p;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t nib = (uint32_t)(word(p, wave * 16u + (lane >> 4) + 4u * q) >> ((lane & 15u) * 4u));
#pragma unroll
            for (int k = 0; k < 4; ++k) c[4 * q + k] += ((nib >> k) & 1u) << sh;
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = (float)c[r] - half;
}

// The same for a plain sign message, from this lane's four words
__device__ __forceinline__ void small_from_signs(float (&v)[16], const uint64_t (&w)[4], uint32_t lane)
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t nib = (uint32_t)(w[q] >> ((lane & 15u) * 4u));
#pragma unroll
        for (int k = 0; k < 4; ++k) v[4 * q + k] = flip_by_bit31(-0.5f, nib << (31 - k));
    }
}

// Dither, sign and pack (Def. 3.2, Def. 3.7) of the tile in L2; l.lam holds the blocks' amplitudes (published).  The
// words go to memory and, with KEEP, to l.words as well.
template <bool DITHER, bool MULTIK, bool KEEP>
__device__ __forceinline__ void small_pack(const float (&v)[16], const SmallArgs &a, SmallLds &l, uint32_t rk1, uint32_t rlo,
                                           uint32_t party, uint32_t slot, uint64_t tile, uint32_t lane, uint32_t wave)
{
    const uint64_t base = tile << kSmLog2;
    const RngKey key = { a.k0, rk1, kDomainDither, rlo, party };
    const float tscale = a.sqrtb * 5.9604644775390625e-08f; // 2^-24: u = m * 2^-24 with m odd
    const uint32_t at = (lane & 3u) + wave * 4u + ((lane >> 2) & 3u) * 16u; // word of register `lane` of this wave
    const uint64_t gw = tile * 64u + at;
    uint64_t *const dst = a.bits_out + slot * a.bits_out_stride + gw;
    const bool mine = lane < 16u;
    if (a.stat_clipped) {
        uint32_t clipped = 0u, near = 0u;
        static_for<4>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            uint32_t w[4] = { 0u, 0u, 0u, 0u };
            if constexpr (DITHER) philox((uint32_t)((base + small_l2(4 * g, wave)) >> 8) << 6 | lane, key, w);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const float z = v[4 * g + s], lam = l.lam[small_l2(4 * g + s, wave) >> a.S];
                float tv = z;
                if constexpr (DITHER) tv = fmaf(lam * tscale, fmaf((float)(w[s] >> 8), 2.f, -16777215.f), tv);
                clipped += (uint32_t)__popcll(__ballot(fabsf(z) > lam * a.sqrtb));
                near += (uint32_t)__popcll(__ballot(fabsf(tv) < 1e-6f * lam * a.sqrtb));
            }
        });
        // One addition per workgroup and counter, and none of a zero: all of them go to the same two words, where every wave's
        // pair of additions took most of the kernel's time (n = 2^22 in blocks of 2^12: 55 us with them, 9.3 like this).
        uint32_t *const sums = reinterpret_cast<uint32_t *>(l.red); // last read before the transform's barrier
        if (lane == 0u) {
            sums[wave] = clipped;
            sums[4u + wave] = near;
        }
        __syncthreads();
        if (threadIdx.x < 2u) {
            const uint32_t *const p = sums + 4u * threadIdx.x, n = (p[0] + p[1]) + (p[2] + p[3]);
            if (n) atomicAdd((threadIdx.x ? a.stat_near : a.stat_clipped) + slot, (unsigned long long)n);
        }
    }
    if constexpr (!MULTIK) {
        uint32_t lo = 0u, hi = 0u;
        static_for<4>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            uint32_t w[4] = { 0u, 0u, 0u, 0u };
            if constexpr (DITHER) philox((uint32_t)((base + small_l2(4 * g, wave)) >> 8) << 6 | lane, key, w);
            static_for<4>([&](auto sc) {
                constexpr int r = 4 * g + decltype(sc)::value;
                uint64_t word;
                if constexpr (DITHER) {
                    // the integer-domain comparison of fo_contig.h: w >= 2^31 - 128 - 128 z 2^24 / lambda'
                    const float kq = l.kq[small_l2(r, wave) >> a.S];
                    uint32_t thr;
                    asm("v_cvt_u32_f32 %0, %1" : "=v"(thr) : "v"(fmaf(v[r], kq, 2147483520.f)));
                    word = __ballot(w[decltype(sc)::value] >= thr) & __ballot(kq == kq);
                } else {
                    word = __ballot(v[r] >= 0.f);
                }
                lo = write_lane<r>(lo, (uint32_t)word);
                hi = write_lane<r>(hi, (uint32_t)(word >> 32));
            });
        });
        const uint64_t out = ((uint64_t)hi << 32) | lo;
        if (mine && gw < a.W) *dst = out;
        if (KEEP && mine) l.words[at] = out;
    } else {
        uint32_t lo[kSmPlanes], hi[kSmPlanes];
#pragma unroll
        for (int p = 0; p < (int)kSmPlanes; ++p) lo[p] = hi[p] = 0u;
        static_for<4>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            uint32_t cnt[4] = { 0u, 0u, 0u, 0u };
            float thr[4];
#pragma unroll
            for (int s = 0; s < 4; ++s) thr[s] = l.lam[small_l2(4 * g + s, wave) >> a.S] * tscale;
            for (uint32_t k = 0; k < a.K; ++k) {
                uint32_t w[4] = { 0u, 0u, 0u, 0u };
                const RngKey kk = { key.k0, key.k1, kDomainDither | (k << 8), key.c2, key.c3 };
                if constexpr (DITHER) philox((uint32_t)((base + small_l2(4 * g, wave)) >> 8) << 6 | lane, kk, w);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    float z = v[4 * g + s];
                    if constexpr (DITHER) z = fmaf(thr[s], fmaf((float)(w[s] >> 8), 2.f, -16777215.f), z);
                    cnt[s] += (z >= 0.f) ? 1u : 0u;
                }
            }
            static_for<(int)kSmPlanes>([&](auto pc) {
                constexpr int p = decltype(pc)::value;
                if ((uint32_t)p < a.planes)
                    static_for<4>([&](auto sc) {
                        constexpr int s = decltype(sc)::value, r = 4 * g + s;
                        const uint64_t word = __ballot(((cnt[s] >> p) & 1u) != 0u);
                        lo[p] = write_lane<r>(lo[p], (uint32_t)word);
                        hi[p] = write_lane<r>(hi[p], (uint32_t)(word >> 32));
                    });
            });
        });
#pragma unroll
        for (int p = 0; p < (int)kSmPlanes; ++p)
            if ((uint32_t)p < a.planes) {
                const uint64_t out = ((uint64_t)hi[p] << 32) | lo[p];
                if (mine && gw < a.W) dst[(uint64_t)p * a.W] = out;
                if (KEEP && mine) l.words[64 * p + at] = out;
            }
    }
}

// The decoder's input from the message just packed (l.words)
template <bool MULTIK>
__device__ __forceinline__ void small_from_kept(float (&v)[16], const SmallArgs &a, const SmallLds &l, uint32_t lane, uint32_t wave)
{
    if constexpr (MULTIK) {
        small_from_bits(v, a.planes, false, 0.5f * (float)a.K, lane, wave, [&](uint32_t p, uint32_t w) { return l.words[64u * p + w]; });
    } else {
        uint64_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = l.words[wave * 16u + (lane >> 4) + 4u * q];
        small_from_signs(v, w, lane);
    }
}

// Encoder from the vector in L0 (b <= 2^12): block norms where measured, amplitudes into l.lam and memory, eps flip,
// transform.  Leaves the tile in L2 with l.lam published; returns false if only the amplitudes were wanted.
__device__ __forceinline__ bool small_encode_tile(float (&v)[16], const SmallArgs &a, SmallLds &l, uint32_t rk1, uint32_t rlo,
                                                  uint32_t eps_party, uint32_t slot, uint64_t tile, uint32_t lane, uint32_t wave)
{
    const uint32_t t = threadIdx.x, S = a.S;
    const uint64_t base = tile << kSmLog2;
    if (a.scale_mode == SMS_MEASURED) {
        float p[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            p[q] = (v[4 * q] * v[4 * q] + v[4 * q + 1] * v[4 * q + 1]) + (v[4 * q + 2] * v[4 * q + 2] + v[4 * q + 3] * v[4 * q + 3]);
        if (S >= 10u) { // a wave's 1024 coordinates lie in one block
            const float s = wave_sum((p[0] + p[1]) + (p[2] + p[3]), 6);
            if (lane == 0u) l.red[wave] = s;
        } else if (S == 9u) { // two sums instead of one for each half block (3 M coordinates, M = 5, K = 4: 48.9 -> 46.6 us a step)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float s = wave_sum(p[2 * q] + p[2 * q + 1], 6);
                if (lane == 0u) l.red[wave * 2u + q] = s;
            }
        } else {
            const uint32_t ll = S < 8u ? S - 2u : 6u; // log2 of the lanes that share a block's part of 256 coordinates
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float s = wave_sum(p[q], (int)ll);
                if ((lane & ((1u << ll) - 1u)) == 0u) l.red[((wave * 4u + q) << (6u - ll)) + (lane >> ll)] = s;
            }
        }
    }
    small_eps(l.eps, a, rk1, rlo, eps_party, base);
    __syncthreads();
    const uint32_t nblk = kSmTile >> S;
    if (t < nblk) {
        const uint64_t gb = tile * nblk + t;
        float lam = 0.f;
        if (gb < a.nblocks) {
            float *const out = a.scales + slot * a.scales_stride + gb;
            if (a.scale_mode == SMS_MEASURED) {
                const uint32_t per = S >= 10u ? 1u << (S - 10u) : 1u;
                float s = 0.f;
                for (uint32_t k = 0; k < per; ++k) s += l.red[t * per + k];
                *out = lam = a.coef * sqrtf(s);
            } else if (a.scale_mode == SMS_SERVER) {
                *out = lam = a.coef * largest_scale(a.scales_up, a.nblocks, a.M, gb);
            } else {
                lam = *out;
            }
        }
        l.lam[t] = lam;
        l.kq[t] = -128.f / (lam * (a.sqrtb * 5.9604644775390625e-08f));
    }
    if (a.scales_only) return false;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t nib = l.eps[wave * 32u + q * 8u + (lane >> 3)] >> ((lane & 7u) * 4u);
#pragma unroll
        for (int k = 0; k < 4; ++k) v[4 * q + k] = flip_by_bit31(v[4 * q + k], nib << (31 - k));
    }
    small_transform(v, S, l.x, lane, wave); // its barrier publishes l.lam
    return true;
}

// lambda * eps * value of register r in L2 (eps words and amplitudes of the tile in LDS), coefficient included in lam
__device__ __forceinline__ float small_signed_lam(const SmallLds &l, const uint32_t *eps, int r, uint32_t S, uint32_t lane, uint32_t wave)
{
    const uint32_t c = small_l2(r, wave);
    return flip_by_bit0(l.lam[c >> S], eps[(c >> 5) + (lane >> 5)] >> (lane & 31u));
}

// The decoder's result `y` for an element that held `old` (read ahead of the transform; unused by STORE_SET)
__device__ __forceinline__ float small_result(float y, float old, uint32_t mode, float delta)
{
    return mode == STORE_SET ? y : mode == STORE_ACC ? old + y : old - delta * y;
}

// Encoder, low stages: tile blockIdx.x of slot blockIdx.y.  MID: the input has its high stages done (b > 2^12), the
// amplitude comes from the high pass's partial sums.  DEC: the decoder's low stages of the message follow in place.
template <int IN, bool DITHER, bool MULTIK, bool DEC>
__global__ __launch_bounds__(kSmThreads) void k_small_encode(const SmallArgs a, const PtrTab tab)
{
    __shared__ SmallLds l;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, slot = blockIdx.y;
    const uint64_t tile = blockIdx.x, base = tile << kSmLog2;
    uint32_t rk1, rlo;
    resolve_round(a.k1, a.round_lo, a.round_dev, rk1, rlo);
    const uint32_t party = a.party0 == 0xFFFFFFFFu ? a.party0 : a.party0 + slot;
    const uint32_t eps_party = a.eps_party0 >= 0xFFFFFFFEu ? a.eps_party0 : a.eps_party0 + slot;
    const float *const src = a.use_tab ? tab.p[slot] : a.src + slot * a.src_stride;
    float v[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t i = base + wave * 1024u + q * 256u + lane * 4u;
        float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
        if (IN == SMI_MID || i + 3 < a.len_in) {
            x = *reinterpret_cast<const float4 *>(src + i);
        } else {
            if (i < a.len_in) x.x = src[i];
            if (i + 1 < a.len_in) x.y = src[i + 1];
            if (i + 2 < a.len_in) x.z = src[i + 2];
        }
        v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
    }
    if constexpr (IN == SMI_GRAD) {
        if (!small_encode_tile(v, a, l, rk1, rlo, eps_party, slot, tile, lane, wave)) return;
    } else {
        // one block per tile; every workgroup of a block adds the partial sums in the same order
        const uint64_t gb = base >> a.logb;
        const uint32_t nparts = 1u << (a.logb - kSmLog2); // at most 2^8: one per thread
        float lam;
        if (a.scale_mode == SMS_MEASURED) {
            lam = 0.f;
            bool nan = false;
            const uint32_t s0 = a.common ? 0u : slot, s1 = a.common ? a.common : slot + 1u;
            for (uint32_t s = s0; s < s1; ++s) {
                double d = t < nparts ? (double)a.partials[(uint64_t)s * a.ntiles + gb * nparts + t] : 0.0;
                d = wave_sum(d, 6);
                if (s > s0) __syncthreads(); // red64 is free
                if (lane == 0) l.red64[wave] = d;
                __syncthreads();
                const float x = a.coef * (float)sqrt((l.red64[0] + l.red64[1]) + (l.red64[2] + l.red64[3]));
                nan |= (x != x);
                lam = fmaxf(lam, x);
            }
            if (nan) lam = __builtin_nanf("");
        } else if (a.scale_mode == SMS_SERVER) {
            lam = a.coef * largest_scale(a.scales_up, a.nblocks, a.M, gb);
        } else {
            lam = a.scales[slot * a.scales_stride + gb];
        }
        if (t == 0) {
            l.lam[0] = lam;
            l.kq[0] = -128.f / (lam * (a.sqrtb * 5.9604644775390625e-08f));
            if (a.scale_mode != SMS_GIVEN && (base & ((1ull << a.logb) - 1u)) == 0u) a.scales[slot * a.scales_stride + gb] = lam;
        }
        small_transform(v, 12u, l.x, lane, wave); // its barrier publishes l.lam
    }
    small_pack<DITHER, MULTIK, DEC>(v, a, l, rk1, rlo, party, slot, tile, lane, wave);
    if constexpr (DEC) {
        __syncthreads(); // the words are published, l.x is free
        small_from_kept<MULTIK>(v, a, l, lane, wave);
        small_transform(v, a.S, l.x, lane, wave);
        float *const dst = a.mid + slot * a.mid_stride + base + lane;
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[small_l2(r, wave)] = v[r];
    }
}

// Decoder, low stages.  FINAL (b <= 2^12): amplitude, eps flip and store / update; else the fp32 intermediate.
template <bool FINAL>
__global__ __launch_bounds__(kSmThreads) void k_small_decode(const SmallArgs a)
{
    __shared__ SmallLds l;
    const uint32_t t = threadIdx.x, lane = t & 63u, wave = t >> 6, slot = blockIdx.y, S = a.S;
    const uint64_t tile = blockIdx.x, base = tile << kSmLog2;
    const uint64_t *const bits = a.bits_in + slot * a.bits_in_stride;
    auto word = [&](uint32_t p, uint32_t w) { const uint64_t gw = tile * 64u + w; return gw < a.W ? bits[(uint64_t)p * a.W + gw] : 0ull; };
    float v[16];
    if (!a.count && a.Kin == 1u) {
        uint64_t w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) w[q] = word(0u, wave * 16u + (lane >> 4) + 4u * q);
        small_from_signs(v, w, lane);
    } else { // planes of a message, or (count) the workers' messages: both lie W words apart
        small_from_bits(v, a.count ? a.M : a.planes_in, a.count != 0u, 0.5f * (float)(a.count ? a.M : a.Kin), lane, wave, word);
    }
    float old[16];
    if constexpr (FINAL) {
        if (a.store_mode != STORE_SET)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const uint64_t i = base + small_l2(r, wave) + lane;
                old[r] = i < a.len_out ? a.out[i] : 0.f;
            }
        uint32_t rk1, rlo;
        resolve_round(a.k1, a.round_lo, a.round_dev, rk1, rlo);
        small_eps(l.eps, a, rk1, rlo, a.eps_in, base);
        const uint32_t nblk = kSmTile >> S;
        if (t < nblk) {
            const uint64_t gb = tile * nblk + t;
            l.lam[t] = gb < a.nblocks ? a.scales[gb] * a.out_coef : 0.f;
        }
    }
    small_transform(v, S, l.x, lane, wave); // its barrier publishes the tables
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = base + small_l2(r, wave) + lane;
        if constexpr (FINAL) {
            if (i < a.len_out) a.out[i] = small_result(v[r] * small_signed_lam(l, l.eps, r, S, lane, wave), old[r], a.store_mode, a.delta);
        } else {
            a.mid[slot * a.mid_stride + i] = v[r];
        }
    }
}

// G groups of 256 threads share the workers of a tile: in every round each group transforms one worker's message, then every
// group adds up its share of the registers over the round's workers, in the workers' order.  What the groups hand one another
// are the transforms with the eps signs on, which are exact, and the amplitude comes in with the addition, so the mean has
// the roundings, and the bits, of one group that takes one worker after the other.  (Sums of each group's own workers, added
// up at the end, round every group's first product as well: the mean's error against 64-bit sums grew by up to 20 % for
// two to seven workers of like amplitudes.)
template <int G>
struct SmallJoin {
    static constexpr int R = 16 / G; // registers a group adds up: R grp ..
    float4 value[G][4 * kSmThreads]; // registers 4 q .. 4 q + 3 of thread t at 256 q + t
    __device__ __forceinline__ void put(uint32_t grp, uint32_t t, const float (&v)[16])
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) value[grp][q * 256 + t] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    }
    // coef(g, r): amplitude of group g's worker for register r.  A group without a worker in the last round puts any finite
    // values, and its amplitude is zero.  A barrier lies between put and this, and another between this and the next put.
    template <typename F>
    __device__ __forceinline__ void add(float (&part)[R], uint32_t grp, uint32_t t, F &&coef) const
    {
#pragma unroll
        for (uint32_t g = 0; g < (uint32_t)G; ++g)
#pragma unroll
            for (int i = 0; i < R; i += 4) {
                const float4 x = value[g][(grp * R + i) * 64u + t];
                part[i] = fmaf(x.x, coef(g, grp * R + i), part[i]);
                part[i + 1] = fmaf(x.y, coef(g, grp * R + i + 1), part[i + 1]);
                part[i + 2] = fmaf(x.z, coef(g, grp * R + i + 2), part[i + 2]);
                part[i + 3] = fmaf(x.w, coef(g, grp * R + i + 3), part[i + 3]);
            }
    }
    // the groups' shares to the first one, through LDS that nothing else uses any more (16-byte aligned)
    static __device__ __forceinline__ void hand_over(const float (&part)[R], float *x, uint32_t grp, uint32_t t)
    {
        if (grp)
#pragma unroll
            for (int i = 0; i < R; i += 4)
                reinterpret_cast<float4 *>(x)[i * 64 + t] = make_float4(part[i], part[i + 1], part[i + 2], part[i + 3]);
    }
    template <typename F>
    static __device__ __forceinline__ void take_over(float (&acc)[16], const float (&part)[R], F &&x_of, uint32_t t)
    {
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = part[r];
#pragma unroll
        for (int r = R; r < 16; r += 4) {
            const float4 x = reinterpret_cast<const float4 *>(x_of((uint32_t)(r / R)))[(r % R) * 64 + t];
            acc[r] = x.x; acc[r + 1] = x.y; acc[r + 2] = x.z; acc[r + 3] = x.w;
        }
    }
};

// Server for b <= 2^12: the mean of the M messages in registers, its encode, and with UPDATE (fo_step) the decoder of
// the server's own message with the update of x.  G > 1: G groups of 256 threads share the workers (see SmallJoin).  One wave
// on a SIMD waits out every exchange and generator chain of the workers one after the other; the step, us, one group and four:
// d = 10^6 in blocks of 2^12, M = 8 35.9 and 28.7; 2 * 10^5, M = 32 78.6 and 45.6; 5 * 10^4, M = 4 20.6 and 17.5.
// The eps words come eight workers at a time, so that every thread has a generator block to draw (d = 3 * 10^6 in blocks of
// 2^9, M = 5, K = 4: 53.5 us a step with one worker's at a time, 52.9 like this).
template <bool DITHER, bool MULTIK, bool UPDATE, int G>
__global__ __launch_bounds__(kSmThreads * G) void k_small_server(const SmallArgs a)
{
    __shared__ SmallLds l; // of the first group
    __shared__ __attribute__((aligned(16))) uint32_t eps8s[G][8 * kSmEpsWords];
    const uint32_t t = G > 1 ? threadIdx.x & (kSmThreads - 1u) : threadIdx.x, lane = t & 63u, wave = t >> 6, S = a.S;
    const uint32_t grp = G > 1 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kSmThreads)) : 0u;
    uint32_t *const eps8 = eps8s[grp];
    const uint64_t tile = blockIdx.x, base = tile << kSmLog2;
    const uint32_t nblk = kSmTile >> S;
    uint32_t rk1, rlo;
    resolve_round(a.k1, a.round_lo, a.round_dev, rk1, rlo);
    float acc[16], v[16];
    const uint32_t nmsg = a.count ? 1u : a.M;
    auto word = [&](uint32_t p, uint32_t w) { const uint64_t gw = tile * 64u + w; return gw < a.W ? a.bits_in[(uint64_t)p * a.W + gw] : 0ull; };
    // a worker's words and amplitude are asked for one worker ahead
    uint64_t wnext[4] = { 0ull, 0ull, 0ull, 0ull };
    const uint64_t gb_mine = tile * nblk + t;
    const bool lam_mine = t < nblk && gb_mine < a.nblocks;
    float lnext = 0.f;
    auto request = [&](uint32_t m) {
        if (!a.count)
#pragma unroll
            for (int q = 0; q < 4; ++q) wnext[q] = word(m, wave * 16u + (lane >> 4) + 4u * q);
        lnext = lam_mine ? a.scales_up[(uint64_t)m * a.nblocks + gb_mine] : 0.f;
    };
    // the eps words of the group's next eight workers from m on, a generator block for every thread
    auto draw_eps = [&](uint32_t m) {
        const uint32_t w8 = m + (t >> 5) * G;
        if (w8 < nmsg) {
            const RngKey key = { a.k0, rk1, kDomainEps, rlo, a.eps_in >= 0xFFFFFFFEu ? a.eps_in : a.eps_in + w8 };
            uint32_t w[4];
            philox((uint32_t)(base >> 7) + (t & 31u), key, w);
            *reinterpret_cast<uint4 *>(eps8 + 4u * t) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    };
    if (grp < nmsg) request(grp);
    if constexpr (G == 1) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.f;
        for (uint32_t m = 0; m < nmsg; ++m) {
            if (a.count) small_from_bits(v, a.M, true, 0.5f * (float)a.M, lane, wave, word);
            else small_from_signs(v, wnext, lane);
            const float lam = lnext * a.in_coef;
            if (m + 1u < nmsg) request(m + 1u);
            if ((m & 7u) == 0u) draw_eps(m); // the last use was before the barrier
            if (t < nblk) l.lam[t] = lam;
            small_transform(v, S, l.x, lane, wave);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = fmaf(v[r], small_signed_lam(l, eps8 + (m & 7u) * kSmEpsWords, r, S, lane, wave), acc[r]);
            __syncthreads(); // the tables and l.x are free
        }
    } else {
        __shared__ __attribute__((aligned(16))) float xs[G - 1][kSmXWords];
        __shared__ float lams[2][G][64];
        __shared__ SmallJoin<G> join;
        float *const x = grp ? xs[grp - 1u] : l.x;
        float part[16 / G];
#pragma unroll
        for (int i = 0; i < 16 / G; ++i) part[i] = 0.f;
        for (uint32_t m0 = 0, k = 0; m0 < nmsg; m0 += G, ++k) {
            const uint32_t m = m0 + grp;
            small_from_signs(v, wnext, lane);
            if (t < nblk) lams[k & 1u][grp][t] = m < nmsg ? lnext * a.in_coef : 0.f; // last read two rounds ago
            if (m + G < nmsg) request(m + G);
            if ((k & 7u) == 0u) draw_eps(m); // the last use was before the barrier
            small_transform(v, S, x, lane, wave);
#pragma unroll
            for (int r = 0; r < 16; ++r)
                v[r] = flip_by_bit0(v[r], eps8[(k & 7u) * kSmEpsWords + (small_l2(r, wave) >> 5) + (lane >> 5)] >> (lane & 31u));
            join.put(grp, t, v);
            __syncthreads(); // the values are published, eps8 and x are free
            join.add(part, grp, t, [&](uint32_t g, uint32_t r) { return lams[k & 1u][g][small_l2((int)r, wave) >> S]; });
        }
        SmallJoin<G>::hand_over(part, x, grp, t);
        __syncthreads();
        if (grp) { // the barriers of the first group: here, in small_encode_tile and small_transform, in small_pack, with the update
            const uint32_t left = 3u + (a.stat_clipped ? 1u : 0u) + (UPDATE ? 2u : 0u);
            for (uint32_t k = 0; k < left; ++k) __syncthreads();
            return;
        }
        SmallJoin<G>::take_over(acc, part, [&](uint32_t g) { return xs[g - 1u]; }, t);
    }
    {
        float *const p = l.x + lane + wave * 272u;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint64_t i = base + small_l2(r, wave) + lane;
            if (a.gbar && i < 64u * a.W) a.gbar[i] = acc[r];
            p[(r & 3) * 68 + (r >> 2) * 1088] = acc[r];
        }
    }
    __syncthreads();
    {
        const float *const p = l.x + wave * 1088u + lane * 4u + 4u * (lane >> 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(p + 272 * q);
            v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
    }
    small_encode_tile(v, a, l, rk1, rlo, a.eps_party0, 0u, tile, lane, wave); // starts with a barrier before it writes l.x
    small_pack<DITHER, MULTIK, UPDATE>(v, a, l, rk1, rlo, 0xFFFFFFFFu, 0u, tile, lane, wave);
    if constexpr (UPDATE) {
        __syncthreads(); // the words are published; l.x and l.lam are free, l.eps is the server's own stream still
        float old[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint64_t i = base + small_l2(r, wave) + lane;
            old[r] = i < a.len_out ? a.out[i] : 0.f;
        }
        if (t < nblk) l.lam[t] *= a.out_coef;
        small_from_kept<MULTIK>(v, a, l, lane, wave);
        small_transform(v, S, l.x, lane, wave);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const uint64_t i = base + small_l2(r, wave) + lane;
            if (i < a.len_out) a.out[i] = small_result(v[r] * small_signed_lam(l, l.eps, r, S, lane, wave), old[r], a.store_mode, a.delta);
        }
    }
}

// A thread's sum of squares of a strided tile, spelled out: a block's amplitude is the same to the bit whichever kernel forms it
__device__ __forceinline__ float small_sumsq(const float (&v)[16])
{
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 4)
        s += fmaf(v[r], v[r], v[r + 1] * v[r + 1]) + fmaf(v[r + 2], v[r + 2], v[r + 3] * v[r + 3]);
    return s;
}

// The HB = 1 .. 8 stages above the contiguous tile: 2^HB rows, 2^12 apart, by 2^(12-HB) columns.  Tile coordinate
// u = row << cb | column:
//   A (loads): regs = (u8..u11), threads = (u0..u7)        B: regs = (u4..u7), threads = (u0..u3, u8..u11)
// B is reached through LDS (word u + 16 (u / 256)) where some row bit lies below u8 (HB > 4).
// G > 1 (SMH_SERVER): G groups of 256 threads share the workers (SmallJoin), and the first goes on alone with the mean.  A vector
// of 2^20 has one tile for every compute unit, and one wave on a SIMD waits out every exchange and every generator chain of the M
// workers one after the other.  The step, us, one group and four: n = 2^16, M = 4 25.9 and 24.9; 2^17, M = 8 32.6 and 30.4;
// 2^18, M = 32 71.9 and 59.8; 2^20, M = 32 164.6 and 157.8.
template <int MODE, int HB, int G = 1>
__global__ __launch_bounds__(kSmThreads * G) void k_small_high(const SmallArgs a, const PtrTab tab)
{
    static_assert(G == 1 || MODE == SMH_SERVER, "groups share the workers");
    constexpr uint32_t cb = kSmLog2 - HB;
    constexpr bool X = HB > 4;
    __shared__ __attribute__((aligned(16))) float xbs[G][kSmXWords];
    __shared__ __attribute__((aligned(16))) uint32_t epss[G][2][kSmEpsWords];
    __shared__ float red[4];
    const uint32_t t = G > 1 ? threadIdx.x & (kSmThreads - 1u) : threadIdx.x, lane = t & 63u, wave = t >> 6, slot = blockIdx.y;
    const uint32_t grp = G > 1 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kSmThreads)) : 0u;
    float *const xb = xbs[grp];
    uint32_t (&eps)[2][kSmEpsWords] = epss[grp];
    // Rows of 64 bytes (HB = 8), half a line: the two tiles that share lines are given block indices that land on the same XCD
    // (blocks are dealt round-robin over 8 XCDs).  n = 2^20, M = 8, us: encoder 18.8 -> 14.7, server 15.6 -> 13.0, decoder 10.0 -> 7.3.
    const uint32_t i0 = blockIdx.x;
    const uint64_t tile = HB == 8 ? (i0 & ~15u) | ((i0 & 7u) << 1) | ((i0 >> 3) & 1u) : i0;
    const uint64_t origin = ((tile >> HB) << (kSmLog2 + HB)) + ((tile & ((1u << HB) - 1u)) << cb);
    const uint64_t gb = origin >> a.logb;
    uint32_t rk1, rlo;
    resolve_round(a.k1, a.round_lo, a.round_dev, rk1, rlo);
    auto off = [](uint32_t u) -> uint32_t { return ((u >> cb) << kSmLog2) + (u & ((1u << cb) - 1u)); };
    auto ua = [&](int r) -> uint32_t { return t | (uint32_t)r << 8; };
    auto uo = [&](int r) -> uint32_t { return X ? ((t & 15u) | (uint32_t)r << 4 | (t >> 4) << 8) : ua(r); };
    // eps bits of the tile, bit u & 31 of word u >> 5: one generator call per 128 columns of a row, or per row
    auto fill = [&](uint32_t *e, uint32_t party) {
        constexpr uint32_t calls = cb >= 7u ? 32u : 1u << HB;
        if (t >= calls) return;
        const uint32_t u = cb >= 7u ? t << 7 : t << cb;
        const uint64_t i = origin + off(u);
        const RngKey key = { a.k0, rk1, kDomainEps, rlo, party };
        uint32_t w[4];
        philox((uint32_t)(i >> 7), key, w);
        const uint32_t sel = (uint32_t)(i >> 5) & 3u;
        const uint32_t ws = sel == 0 ? w[0] : sel == 1 ? w[1] : sel == 2 ? w[2] : w[3];
        if constexpr (cb >= 7u) {
            *reinterpret_cast<uint4 *>(e + 4u * t) = make_uint4(w[0], w[1], w[2], w[3]);
        } else if constexpr (cb == 6u) {
            e[2u * t] = ws;
            e[2u * t + 1u] = sel ? w[3] : w[1];
        } else if constexpr (cb == 5u) {
            e[t] = ws;
        } else {
            static_assert(cb >= 4u, "rows of 16 columns at least");
            reinterpret_cast<uint16_t *>(e)[t] = (uint16_t)(ws >> ((uint32_t)i & 16u));
        }
    };
    auto flip = [&](float x, const uint32_t *e, uint32_t u) -> float { return flip_if(x, (e[u >> 5] >> (u & 31u)) & 1u); };
    auto stages_hi = [&](float (&v)[16]) { // u8 .. u11, in A
        if constexpr (cb <= 8u) bfly<float, 0, 16>(v);
        if constexpr (cb <= 9u) bfly<float, 1, 16>(v);
        if constexpr (cb <= 10u) bfly<float, 2, 16>(v);
        bfly<float, 3, 16>(v);
    };
    auto stages_lo = [&](float (&v)[16]) { // u4 .. u7, in B
        if constexpr (cb <= 4u) bfly<float, 0, 16>(v);
        if constexpr (cb <= 5u) bfly<float, 1, 16>(v);
        if constexpr (cb <= 6u) bfly<float, 2, 16>(v);
        if constexpr (cb <= 7u) bfly<float, 3, 16>(v);
    };
    float *const pa = xb + t, *const pb = xb + (t & 15u) + (t >> 4) * 272u;
    auto a_to_b = [&](float (&v)[16]) {
#pragma unroll
        for (int r = 0; r < 16; ++r) pa[r * 272] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = pb[r * 16];
    };
    auto tile_sumsq = [&](const float (&v)[16]) { // -> partials[slot][tile]; two barriers
        const float s = wave_sum(small_sumsq(v), 6);
        if (lane == 0) red[wave] = s;
        __syncthreads();
        if (t == 0) a.partials[(uint64_t)slot * a.ntiles + tile] = (red[0] + red[1]) + (red[2] + red[3]);
    };

    float v[16];
    if constexpr (MODE == SMH_ENC) {
        const float *const src = (a.use_tab ? tab.p[slot] : a.src + slot * a.src_stride) + origin;
        const uint64_t room = a.len_in > origin ? a.len_in - origin : 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = off(ua(r)) < room ? src[off(ua(r))] : 0.f;
        fill(eps[0], a.eps_party0 >= 0xFFFFFFFEu ? a.eps_party0 : a.eps_party0 + slot);
        tile_sumsq(v); // its barrier publishes the eps table
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = flip(v[r], eps[0], ua(r));
        stages_hi(v);
        if constexpr (X) {
            a_to_b(v);
            stages_lo(v);
        }
        float *const dst = a.mid + slot * a.mid_stride + origin;
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[off(uo(r))] = v[r];
    } else if constexpr (MODE == SMH_DEC) {
        const float *const src = a.src + origin;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = src[off(ua(r))];
        const uint64_t room = a.len_out > origin ? a.len_out - origin : 0;
        float *const dst = a.out + origin;
        float old[16];
        if (a.store_mode != STORE_SET)
#pragma unroll
            for (int r = 0; r < 16; ++r) old[r] = off(uo(r)) < room ? dst[off(uo(r))] : 0.f;
        fill(eps[0], a.eps_in);
        const float c = a.scales[gb] * a.out_coef;
        stages_hi(v);
        if constexpr (X) {
            a_to_b(v); // its barrier publishes the eps table
            stages_lo(v);
        } else {
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (off(uo(r)) < room) dst[off(uo(r))] = small_result(flip(c * v[r], eps[0], uo(r)), old[r], a.store_mode, a.delta);
    } else {
        float acc[16], next[16];
        const uint32_t nmsg = a.count ? 1u : a.M;
        const float *src = a.src + origin;
        auto request = [&](uint32_t m) {
#pragma unroll
            for (int r = 0; r < 16; ++r) next[r] = src[m * a.src_stride + off(ua(r))];
        };
        // worker m (v in layout A on entry) transformed in layout `uo`, its eps words in e; one barrier
        auto transform = [&](uint32_t *e, uint32_t m) {
            fill(e, a.eps_in >= 0xFFFFFFFEu ? a.eps_in : a.eps_in + m);
            stages_hi(v);
            if constexpr (X) {
                a_to_b(v); // its barrier publishes the eps table
                stages_lo(v);
            } else {
                __syncthreads();
            }
        };
        auto coef_of = [&](uint32_t m) -> float { return a.scales_up[(uint64_t)m * a.nblocks + gb] * a.in_coef; };
        if constexpr (G == 1) {
            request(0u);
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            for (uint32_t m = 0; m < nmsg; ++m) {
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = next[r];
                if (m + 1u < nmsg) request(m + 1u);
                uint32_t *const e = eps[m & 1u]; // last read one worker ago, before that worker's closing barrier
                const float c = coef_of(m);
                transform(e, m);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = fmaf(v[r], flip(c, e, uo(r)), acc[r]);
                __syncthreads(); // xb is free
            }
        } else {
            __shared__ SmallJoin<G> join;
            float part[16 / G], c[G];
#pragma unroll
            for (int i = 0; i < 16 / G; ++i) part[i] = 0.f;
            request(grp < nmsg ? grp : 0u);
            for (uint32_t m0 = 0; m0 < nmsg; m0 += G) {
                const uint32_t m = m0 + grp;
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = next[r];
                if (m + G < nmsg) request(m + G);
#pragma unroll
                for (int g = 0; g < G; ++g) c[g] = coef_of(m0 + g < nmsg ? m0 + g : m0);
#pragma unroll
                for (int g = 0; g < G; ++g) c[g] = m0 + g < nmsg ? c[g] : 0.f;
                transform(eps[0], m); // the last read of eps was before the barrier
#pragma unroll
                for (int r = 0; r < 16; ++r) v[r] = flip(v[r], eps[0], uo(r));
                join.put(grp, t, v);
                __syncthreads(); // the values are published, xb and eps are free
                join.add(part, grp, t, [&](uint32_t g, uint32_t) { return c[g]; });
            }
            SmallJoin<G>::hand_over(part, xb, grp, t);
            __syncthreads();
            if (grp) { // the barriers of the first group
                if (a.partials) __syncthreads();
                __syncthreads();
                if constexpr (X) __syncthreads();
                return;
            }
            SmallJoin<G>::take_over(acc, part, [&](uint32_t g) { return xbs[g]; }, t);
        }
        if (a.gbar)
#pragma unroll
            for (int r = 0; r < 16; ++r) a.gbar[origin + off(uo(r))] = acc[r];
        fill(eps[0], a.eps_party0);
        if (a.partials) tile_sumsq(acc);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = flip(acc[r], eps[0], uo(r));
        if constexpr (X) {
            stages_lo(acc);
#pragma unroll
            for (int r = 0; r < 16; ++r) pb[r * 16] = acc[r];
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = pa[r * 272];
        }
        stages_hi(acc);
        float *const dst = a.mid + origin;
#pragma unroll
        for (int r = 0; r < 16; ++r) dst[off(ua(r))] = acc[r];
    }
}

// Encoder of a block of 2^(12+HB) coordinates, HB = 1 .. 4, in one launch and without scratch memory: the workgroup of a
// contiguous tile, row R of the block's 2^HB rows, reads the whole block in the strided tiles of k_small_high, adds up
// their squares as it does and keeps the one output of the high stages that falls into its row, then goes on like
// k_small_encode<SMI_MID>.  Every sum has the operands and the order it has in those two kernels, so the message and the
// amplitude are theirs to the bit.  It reads a block 2^HB times (from the caches but once) to save the trip through memory
// and the second launch: n = 2^13 7.1 us, n = 2^16 9.2, the two kernels 10.1 and 10.2; 2^21 coordinates in blocks of 2^16, where
// the repeated reads are 128 MiB of cache traffic, 18.5 and 13.4 (the kernels for long vectors 42).
// The strided tiles are dealt to up to four groups of 256 threads, whose loads are in flight together; the first group does
// the contiguous tile.  No diagnostic counters (their barrier would be the first group's alone).
constexpr uint32_t small_block_groups(int hb) { return hb == 1 ? 2u : 4u; }
template <int HB, bool DITHER, bool MULTIK>
__global__ __launch_bounds__(kSmThreads * small_block_groups(HB)) void k_small_block(const SmallArgs a)
{
    constexpr uint32_t G = small_block_groups(HB);
    static_assert(HB >= 1 && HB <= 4, "the strided tiles' rows have 256 columns at least, so a thread's columns are t mod 256");
    constexpr uint32_t cb = kSmLog2 - HB, C = 4 - HB; // C: register bits of a strided tile that are column bits
    __shared__ SmallLds l;
    __shared__ __attribute__((aligned(16))) uint32_t eps[kSmEpsWords << HB]; // of the whole block
    const uint32_t t = threadIdx.x & 255u, grp = threadIdx.x >> 8, lane = t & 63u, wave = t >> 6;
    const uint64_t tile = blockIdx.x, gb = tile >> HB, origin = gb << (kSmLog2 + HB);
    const uint32_t row = (uint32_t)tile & ((1u << HB) - 1u);
    uint32_t rk1, rlo;
    resolve_round(a.k1, a.round_lo, a.round_dev, rk1, rlo);
    const char *const src = reinterpret_cast<const char *>(a.src + origin);
    constexpr uint32_t b = kSmTile << HB;
    const uint32_t room = a.len_in >= origin + b ? b : a.len_in > origin ? (uint32_t)(a.len_in - origin) : 0u;
    // coordinate, inside the block, of register r of strided tile j: the register's part (the same in every lane) + the lane's
    auto part = [](int r) -> uint32_t { return ((uint32_t)r >> C << kSmLog2) + (((uint32_t)r & ((1u << C) - 1u)) << 8); };
    float v[16], next[16];
    auto load = [&](uint32_t j) {
        const uint32_t mine = (j << cb) + t;
#pragma unroll
        for (int r = 0; r < 16; ++r) next[r] = mine + part(r) < room ? ld_uniform<float>(src + part(r) * 4u, mine * 4u) : 0.f;
    };
    load(grp);
    {
        const RngKey key = { a.k0, rk1, kDomainEps, rlo, a.eps_party0 };
        for (uint32_t c = threadIdx.x; c < (kSmEpsWords << HB) / 4u; c += kSmThreads * G) {
            uint32_t w[4];
            philox((uint32_t)(origin >> 7) + c, key, w);
            *reinterpret_cast<uint4 *>(eps + 4u * c) = make_uint4(w[0], w[1], w[2], w[3]);
        }
    }
    __syncthreads();
#pragma unroll 1
    for (uint32_t j = grp; j < (1u << HB); j += G) {
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = next[r];
        if (j + G < (1u << HB)) load(j + G);
        const float s = wave_sum(small_sumsq(v), 6);
        if (lane == 0u) l.red[4u * j + wave] = s;
#pragma unroll
        for (int r = 0; r < 16; ++r) v[r] = flip_if(v[r], (eps[(part(r) >> 5) + (((j << cb) + t) >> 5)] >> (t & 31u)) & 1u);
        // of every butterfly the output that this row keeps: a + b or a - b (the product by one is exact)
        static_for<HB>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            const float sgn = (row >> k) & 1u ? -1.f : 1.f;
#pragma unroll
            for (int h = 0; h < (1 << (HB - 1 - k)); ++h)
#pragma unroll
                for (int c = 0; c < (1 << C); ++c) v[(h << C) | c] = fmaf(v[((2 * h + 1) << C) | c], sgn, v[((2 * h) << C) | c]);
        });
#pragma unroll
        for (int c = 0; c < (1 << C); ++c) {
            const uint32_t col = (j << cb) + t + 256u * (uint32_t)c;
            l.x[col + 4u * (col >> 6)] = v[c];
        }
    }
    __syncthreads();
    if (grp != 0u) {
        __syncthreads(); // the one in small_transform
        return;
    }
    float lam;
    if (a.scale_mode == SMS_MEASURED) {
        double d = 0.0;
        if (lane < (1u << HB)) d = (double)((l.red[4u * lane] + l.red[4u * lane + 1u]) + (l.red[4u * lane + 2u] + l.red[4u * lane + 3u]));
        d = wave_sum(d, 6);
        lam = a.coef * (float)sqrt(d);
    } else {
        lam = a.scales[gb];
    }
    if (t == 0) {
        l.lam[0] = lam;
        l.kq[0] = -128.f / (lam * (a.sqrtb * 5.9604644775390625e-08f));
        if (a.scale_mode != SMS_GIVEN && row == 0u) a.scales[gb] = lam;
    }
    {
        const float *const p = l.x + wave * 1088u + lane * 4u + 4u * (lane >> 4);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 x = *reinterpret_cast<const float4 *>(p + 272 * q);
            v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
        }
    }
    small_transform(v, 12u, l.x, lane, wave); // its barrier publishes l.lam
    small_pack<DITHER, MULTIK, false>(v, a, l, rk1, rlo, a.party0, 0u, tile, lane, wave);
}

} // namespace fo
