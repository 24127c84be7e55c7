// Encoder (Def. 3.7) for blocks of 2^6 .. 2^12 coordinates, plain messages (K = 1) with dither: every wave takes 4096
// coordinates through the whole path by itself.  A workgroup is one wave with 8.25 KiB of LDS (8.75 as it is dealt out),
// eighteen to a compute unit.
//
// Layouts of a wave's 4096 coordinates (b0..b11):
//   L0 (global loads, 16 B per lane): regs = (b0,b1,b8,b9,b10,b11)  lanes = (b2..b7)               stages b0,b1,b8..b11
//   L1 (after the exchange):          regs = (b2,b3,b4,b5,b6,b7)    lanes = (b0,b1,b8,b9,b10,b11)  stages b2..b7
// The values are quantised where they are, in L1, instead of going through a second exchange into a layout whose lanes are a
// packed word's bits: a lane holds the four coordinates (b6, b7) of a generator block for each of its 16 (b2..b5), all in
// one block of the transform (from 2^8 on), and it collects its 64 signs as nibbles, bit 4 (b2..b5) + (b6,b7).  A quad of lanes
// differs in (b0, b1), and a word's bit is 4 (b2..b5) + (b0,b1): transposing the 4 x 4 bits of every nibble across the quad, a
// dozen instructions for 64 values, leaves each lane with the packed word of its own number.
//
// What bounds it, by the instructions and the rates at which each was measured to issue (additions and shifts twice as fast as
// the rest): 115 to 125 cycles of a SIMD for a value of its 64 lanes (Philox 48, butterflies 31, the eps flips 12, the quantiser
// 17, the lane swaps 4) of the 140 it takes; the counters give 32.4 vector instructions a value.  And the exchange: LDS takes a
// wave's dword in 3.1 cycles of the compute unit (ds_write2_b32) and gives it back in 2.4, 22 cycles of each of the four SIMDs for a
// value through write and read, which the vector units overlap only in part.  A second exchange, packing through lane writes
// and workgroup barriers cost a third more.  2^27 coordinates, eight workers and the server, us, k_contig before and this:
// blocks of 2^6 1670 -> 1030, 2^8 1630 -> 1080, 2^10 1260 -> 1045, 2^12 1290 -> 1110; read and write of its 4.99 GB take 970.
// Workgroups of one wave (no wave waits for another's LDS to be free): 2 to 4 % better than of four with 36 KiB.
#pragma once
#include "fo_contig.h"

namespace fo {

constexpr uint32_t kWvThreads = 64u;
constexpr uint32_t kWvLds = 2112u; // exchange: two half waves of 32 rows of 33 words.  Before it: 128 eps words, 64 sums, then slopes

// (w[k] >= t[k]) for k = 3, 2, 1, 0, shifted into acc from below.  A vector instruction may read a scalar register as carry two
// wait states after a vector compare has written it; four compares before the four additions keep them apart.
__device__ __forceinline__ void wv_collect(uint32_t &acc, const uint32_t (&w)[4], const uint32_t (&t)[4])
{
    uint64_t c0, c1, c2, c3;
    asm("v_cmp_ge_u32_e64 %4, %8, %12\n\t"
        "v_cmp_ge_u32_e64 %3, %7, %11\n\t"
        "v_cmp_ge_u32_e64 %2, %6, %10\n\t"
        "v_cmp_ge_u32_e64 %1, %5, %9\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %4\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %3\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %2\n\t"
        "v_addc_co_u32_e64 %0, vcc, %0, %0, %1"
        : "+v"(acc), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
        : "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]), "v"(t[0]), "v"(t[1]), "v"(t[2]), "v"(t[3])
        : "vcc");
}

// SC = log2 of the block.
template <int SC>
__global__ __launch_bounds__(kWvThreads, 4) void k_enc_wave(const ContigArgs a, const PtrTab tab)
{
    static_assert(SC >= 6 && SC <= 12, "blocks inside a wave's 4096 coordinates");
    __shared__ __attribute__((aligned(16))) uint32_t lds[kWvLds];
    const uint32_t lane = threadIdx.x, slot = blockIdx.y, part = blockIdx.x; // which 4096 coordinates
    const uint64_t base = (uint64_t)part << 12;
    uint32_t *const epsw = lds;
    float *const blk = reinterpret_cast<float *>(lds + 128);
    const uint32_t party = (a.party0 == 0xFFFFFFFFu) ? a.party0 : a.party0 + slot;
    const uint32_t eps_party = (a.eps_party0 >= 0xFFFFFFFEu) ? a.eps_party0 : a.eps_party0 + slot;
    uint32_t rk1, rlo;
    resolve_round(a.k1, a.round_lo, a.round_dev, rk1, rlo);
    const RngKey key_eps = { a.k0, rk1, kDomainEps, rlo, eps_party };
    const RngKey key_dit = { a.k0, rk1, kDomainDither, rlo, party };

    float v[kV];
    const float *const src = (a.use_tab ? tab.p[slot] : static_cast<const float *>(a.src) + slot * a.src_stride);
    if (base + 4096u <= a.len_in) {
        static_for<16>([&](auto cc) { load_chunk(v, src + base, lane, cc); });
    } else {
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const uint64_t i = base + c * 256u + lane * 4u;
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i + 3 < a.len_in) {
                x = *reinterpret_cast<const float4 *>(src + i);
            } else {
                if (i < a.len_in) x.x = src[i];
                if (i + 1 < a.len_in) x.y = src[i + 1];
                if (i + 2 < a.len_in) x.z = src[i + 2];
            }
            v[4 * c + 0] = x.x; v[4 * c + 1] = x.y; v[4 * c + 2] = x.z; v[4 * c + 3] = x.w;
        }
    }
    // eps words, while the loads are on their way: lane q < 32 draws the generator block of coordinates 128 q ..
    if (lane < 32u) {
        uint32_t w[4];
        philox((uint32_t)(base >> 7) + lane, key_eps, w);
        *reinterpret_cast<uint4 *>(epsw + lane * 4u) = make_uint4(w[0], w[1], w[2], w[3]);
    }

    constexpr uint32_t nseg = 4096u >> SC;
    const uint64_t gb = (base >> SC) + lane; // block of lane l < nseg
    if (a.compute_scale) {
        // sums of squares of the blocks (sign flips do not change them), spelled out as in contig_tile, whose kernels measure
        // the same blocks for a K-fold message, without dither and with counters: the same amplitude to the bit
        float acc = 0.f;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float p = fmaf(v[4 * c], v[4 * c], v[4 * c + 1] * v[4 * c + 1]) + fmaf(v[4 * c + 2], v[4 * c + 2], v[4 * c + 3] * v[4 * c + 3]);
            if constexpr (SC >= 8) {
                acc += p;
                if (((c + 1) & ((1 << (SC - 8)) - 1)) == 0) {
                    const float s = wave_sum_shuffled(acc, 6);
                    if (lane == 0) blk[c >> (SC - 8)] = s;
                    acc = 0.f;
                }
            } else {
                constexpr int ll = SC < 8 ? SC - 2 : 5; // log2 of the lanes of a block: 16 or 32
                const float s = wave_sum_shuffled(p, ll);
                if ((lane & ((1u << ll) - 1u)) == 0u) blk[c * (256 >> SC) + (lane >> ll)] = s;
            }
        }
    }
    wave_sync();
    if (lane < nseg) {
        float l = 0.f;
        if (a.compute_scale) {
            l = a.coef_lambda * sqrtf(blk[lane]);
            if (gb < a.nblocks) a.scales[slot * a.scales_stride + gb] = l;
        } else if (gb < a.nblocks) {
            float *const at = a.scales + slot * a.scales_stride + gb;
            if (a.scales_up) *at = l = a.coef_lambda * largest_scale(a.scales_up, a.nblocks, a.M, gb);
            else l = *at;
        }
        blk[lane] = -128.f / (l * (a.sqrtb * 5.9604644775390625e-08f));
    }
    if (a.scales_only) return;
    wave_sync();
    // Slope of the quantiser for the lane's coordinates with (b6, b7) = s after the exchange
    float kq[4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
        kq[s] = SC >= 8 ? (s ? kq[0] : blk[(lane >> 2) >> (SC >= 8 ? SC - 8 : 0)])
              : SC == 7 ? ((s & 1) ? kq[s & 2] : blk[(lane >> 2) * 2u + (s >> 1)]) : blk[(lane >> 2) * 4u + s];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
        uint32_t n = epsw[c * 8 + (lane >> 3)] >> ((lane & 7u) * 4u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[4 * c + k] = flip_by_bit0(v[4 * c + k], n);
            n = flip_next(n);
        }
    }

    wave_sync(); // the exchange writes over the tables

    bfly<float, 0>(v);
    bfly<float, 1>(v);
    if constexpr (SC > 8) bfly<float, 2>(v);
    if constexpr (SC > 9) bfly<float, 3>(v);
    if constexpr (SC > 10) bfly<float, 4>(v);
    if constexpr (SC > 11) bfly<float, 5>(v);
    {
        uint32_t *const wb = lds + (lane >> 5) * 1056u;
        const uint32_t col = lane & 31u;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
            for (int r = 0; r < 32; ++r) wb[r * 33 + col] = __float_as_uint(v[sub * 32 + r]);
            wave_sync();
#pragma unroll
            for (int r = 0; r < 32; ++r) v[sub * 32 + r] = __uint_as_float(wb[col * 33 + r]);
            wave_sync();
        }
        swap_reg5_lane5(v);
    }
    bfly<float, 0>(v);
    bfly<float, 1>(v);
    bfly<float, 2>(v);
    bfly<float, 3>(v);
    if constexpr (SC > 6) bfly<float, 4>(v);
    if constexpr (SC > 7) bfly<float, 5>(v);

    // Def. 3.2, see contig_tile: w >= T, T = 2^31 - 128 + kq z
    const uint32_t ctr = (((uint32_t)(base >> 8) + (lane >> 2)) << 6) | (lane & 3u);
    uint32_t bits[2];
#pragma unroll
    for (int half = 1; half >= 0; --half) {
        uint32_t acc = 0u;
#pragma unroll
        for (int g = 8 * half + 7; g >= 8 * half; --g) { // (b2..b5)
            uint32_t w[4], thr[4];
            philox(ctr + 4u * g, key_dit, w);
#pragma unroll
            for (int s = 0; s < 4; ++s)
                asm("v_cvt_u32_f32 %0, %1" : "=v"(thr[s]) : "v"(fmaf(v[g + 16 * (s & 1) + 32 * (s >> 1)], kq[s], 2147483520.f)));
            wv_collect(acc, w, thr);
        }
        bits[half] = acc;
    }
    // a NaN amplitude gives all bits 0, as NaN comparisons do
    uint32_t dead = 0u;
#pragma unroll
    for (int s = 0; s < 4; ++s) dead |= kq[s] == kq[s] ? 0u : 0x11111111u << s;
    // bit s of the nibbles of lane j of a quad -> bit j of lane s
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        uint32_t x = bits[half] & ~dead;
        const uint32_t y = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xf, 0xf, true); // quad_perm 1,0,3,2
        x = (lane & 1u) ? (x & 0xAAAAAAAAu) | ((y >> 1) & 0x55555555u) : (x & 0x55555555u) | ((y << 1) & 0xAAAAAAAAu);
        const uint32_t z = (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xf, 0xf, true); // quad_perm 2,3,0,1
        bits[half] = (lane & 2u) ? (x & 0xCCCCCCCCu) | ((z >> 2) & 0x33333333u) : (x & 0x33333333u) | ((z << 2) & 0xCCCCCCCCu);
    }
    const uint64_t gw = (uint64_t)part * 64u + lane;
    if (gw < a.W) static_cast<uint64_t *>(a.dst)[slot * a.dst_stride + gw] = ((uint64_t)bits[1] << 32) | bits[0];
}

} // namespace fo
