// Selection among the compiled variants of the dither + sign + pack kernel (included by fo_enc.hip, which
// instantiates the variants without the diagnostic counters, and by fo_enc_stats.hip, which instantiates those with).
#pragma once
#include "fo_host.h"
#include "fo_enc_wave.h"

namespace fo_host {

// The packing kernels are compiled per (dither on/off, transform length below 256).
template <int IN, bool STATS>
int launch_pack_s(fo_plan *pl, int kid, dim3 grid, hipStream_t st, const ContigArgs &c, const PtrTab &tab)
{
    const bool dither = c.dither == FO_DITHER_UNIFORM, small = c.S < 8;
    const dim3 block(kThreads);
    if (c.K > 1) { // the K-fold quantiser of the server's message
        if (dither && small) return launch(pl, kid, k_contig<IN, OUT_PACK, true, true, 0, true, STATS>, grid, block, st, c, tab);
        if (dither) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 0, true, STATS>, grid, block, st, c, tab);
        return launch(pl, kid, k_contig<IN, OUT_PACK, false, false, 0, true, STATS>, grid, block, st, c, tab);
    }
    if (dither && c.S == 15) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 15, false, STATS>, grid, block, st, c, tab);
    if constexpr (IN == IN_GRAD && !STATS) {
        // Blocks inside a wave's 4096 coordinates, each length compiled for itself; what lies inside the input whole goes to a
        // variant without the per-chunk end-of-input checks.
        if (dither && c.S <= 12) {
            const uint64_t wgs = (pl->ntot + 4095u) >> 12, full = c.len_in >> 12;
            const uint32_t nfull = (uint32_t)(full < wgs ? full : wgs), rest = (uint32_t)wgs - nfull;
            ContigArgs cc = c;
            auto both = [&](auto sc) -> int {
                constexpr int SC = decltype(sc)::value;
                if (nfull) FO_TRY(launch(pl, KID_ENC_WAVE, k_enc_wave<SC, false>, dim3(nfull, grid.y), dim3(kWvThreads), st, cc, tab));
                cc.tile0 = nfull;
                if (rest) FO_TRY(launch(pl, KID_ENC_WAVE, k_enc_wave<SC, true>, dim3(rest, grid.y), dim3(kWvThreads), st, cc, tab));
                return FO_OK;
            };
            switch (c.S) {
            case 6: return both(std::integral_constant<int, 6>{});
            case 7: return both(std::integral_constant<int, 7>{});
            case 8: return both(std::integral_constant<int, 8>{});
            case 9: return both(std::integral_constant<int, 9>{});
            case 10: return both(std::integral_constant<int, 10>{});
            case 11: return both(std::integral_constant<int, 11>{});
            default: return both(std::integral_constant<int, 12>{});
            }
        }
        // blocks of 2^14, likewise compiled for their stage count and without checks where they can be
        if (dither && c.S == 14) {
            const uint64_t full64 = c.len_in >> kTileLog2;
            const uint32_t nfull = (uint32_t)(full64 < grid.x ? full64 : grid.x);
            ContigArgs cc = c;
            auto go = [&](auto guarded, uint32_t tile0, uint32_t ntile) -> int {
                cc.tile0 = tile0;
                return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 14, false, false, decltype(guarded)::value>, dim3(ntile, grid.y), block,
                              st, cc, tab);
            };
            if (nfull) FO_TRY(go(std::false_type{}, 0u, nfull));
            if (nfull < grid.x) FO_TRY(go(std::true_type{}, nfull, grid.x - nfull));
            return FO_OK;
        }
    }
    if constexpr (STATS) {
        if (dither && small) return launch(pl, kid, k_contig<IN, OUT_PACK, true, true, 0, false, STATS>, grid, block, st, c, tab);
    }
    if (dither) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 0, false, STATS>, grid, block, st, c, tab);
    return launch(pl, kid, k_contig<IN, OUT_PACK, false, false, 0, false, STATS>, grid, block, st, c, tab);
}

} // namespace fo_host
