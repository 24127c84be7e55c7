// Selection among the compiled variants of the dither + sign + pack kernel (included by fo_enc.hip, which
// instantiates the variants without the diagnostic counters, and by fo_enc_stats.hip, which instantiates those with).
#pragma once
#include "fo_host.h"
#include "fo_enc_wave.h"

namespace fo_host {

// The packing kernels are compiled per dither on/off and, for blocks inside a tile, transform length below 256.
template <int IN, bool STATS>
int launch_pack_s(fo_plan *pl, int kid, dim3 grid, hipStream_t st, const ContigArgs &c, const PtrTab &tab)
{
    const bool dither = c.dither == FO_DITHER_UNIFORM, multik = c.K > 1; // the K-fold quantiser of the server's message
    const dim3 block(kThreads);
    if constexpr (IN == IN_F32) { // low passes: all fifteen stages
        if (multik && dither) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 0, true, STATS>, grid, block, st, c, tab);
        if (multik) return launch(pl, kid, k_contig<IN, OUT_PACK, false, false, 0, true, STATS>, grid, block, st, c, tab);
        if (c.partials) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 15, false, STATS, false, true>, grid, block, st, c, tab);
        if (dither) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 15, false, STATS>, grid, block, st, c, tab);
        return launch(pl, kid, k_contig<IN, OUT_PACK, false, false, 0, false, STATS>, grid, block, st, c, tab);
    } else {
        const bool small = c.S < 8;
        if (multik && dither && small) return launch(pl, kid, k_contig<IN, OUT_PACK, true, true, 0, true, STATS>, grid, block, st, c, tab);
        if (multik && dither) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 0, true, STATS>, grid, block, st, c, tab);
        if (multik) return launch(pl, kid, k_contig<IN, OUT_PACK, false, false, 0, true, STATS>, grid, block, st, c, tab);
        if (!dither) return launch(pl, kid, k_contig<IN, OUT_PACK, false, false, 0, false, STATS>, grid, block, st, c, tab);
        if (c.S == 15) return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 15, false, STATS>, grid, block, st, c, tab);
        if constexpr (STATS) {
            if (small) return launch(pl, kid, k_contig<IN, OUT_PACK, true, true, 0, false, STATS>, grid, block, st, c, tab);
        } else {
            // blocks inside a wave's 4096 coordinates, each length compiled for itself
            auto go = [&](auto sc) -> int {
                return launch(pl, KID_ENC_WAVE, k_enc_wave<decltype(sc)::value>, dim3((unsigned)((pl->ntot + 4095u) >> 12), grid.y), dim3(kWvThreads),
                              st, c, tab);
            };
            switch (c.S) {
            case 6: return go(std::integral_constant<int, 6>{});
            case 7: return go(std::integral_constant<int, 7>{});
            case 8: return go(std::integral_constant<int, 8>{});
            case 9: return go(std::integral_constant<int, 9>{});
            case 10: return go(std::integral_constant<int, 10>{});
            case 11: return go(std::integral_constant<int, 11>{});
            case 12: return go(std::integral_constant<int, 12>{});
            case 14: return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 14>, grid, block, st, c, tab);
            }
        }
        return launch(pl, kid, k_contig<IN, OUT_PACK, true, false, 0, false, STATS>, grid, block, st, c, tab);
    }
}

} // namespace fo_host
