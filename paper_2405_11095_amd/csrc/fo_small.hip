// Launch sequences for short vectors (fo_small.h); fo_host.h says which calls come here.
#include "fo_host.h"
#include "fo_small.h"

namespace fo { // next to SmallArgs: launch() finds them there

inline bool args_ok(const SmallArgs &a, int kid)
{
    const uint32_t S = a.logb < (uint32_t)kSmLog2 ? a.logb : (uint32_t)kSmLog2;
    if (a.logb < 6 || a.logb > 20 || a.S != S || a.M < 1 || a.M > FO_MAX_WORKERS) return false;
    if (a.K < 1 || a.planes < 1 || a.planes > kSmPlanes || a.Kin < 1 || a.planes_in < 1 || a.planes_in > kSmPlanes) return false;
    switch (kid) {
    case KID_SM_ENC_GRAD: case KID_SM_ENC_MID: return (a.src || a.use_tab) && a.scales && (a.bits_out || a.scales_only);
    case KID_SM_DEC: return a.bits_in && a.out && a.scales;
    case KID_SM_DEC_LOW: return a.bits_in && a.mid;
    case KID_SM_SERVER: return a.bits_in && a.scales_up && a.scales && a.bits_out;
    }
    return a.logb > (uint32_t)kSmLog2 && (a.src || a.use_tab) && (kid == KID_SM_DEC_HIGH ? a.out && a.scales : a.mid != nullptr);
}
inline bool args_ok(const SmallArgs &a, const PtrTab &tab, int kid) { return args_ok(a, kid) && (!a.use_tab || tab.p[0]); }

} // namespace fo

namespace fo_host {

namespace {

SmallArgs small_base(const fo_plan *pl, const Rng &r)
{
    SmallArgs a;
    std::memset(&a, 0, sizeof(a));
    a.W = pl->W;
    a.nblocks = pl->nblocks;
    a.ntiles = pl->sm_tiles;
    a.S = pl->logb < (uint32_t)kSmLog2 ? pl->logb : (uint32_t)kSmLog2;
    a.logb = pl->logb;
    a.dither = pl->p.dither;
    a.M = pl->p.M;
    a.K = a.planes = a.Kin = a.planes_in = 1;
    a.k0 = r.k0; a.k1 = r.k1; a.round_lo = r.round_lo; a.round_dev = r.round_dev;
    a.sqrtb = pl->sqrtb;
    a.len_in = a.len_out = pl->ntot;
    return a;
}

// Whether four groups of threads share the workers in the server's kernels: from four workers (three in two groups: n = 2^16 24.8
// us a step and 24.8, d = 10^6 in blocks of 2^12 21.0 and 21.4; two: 2^20 35.7 and 35.4, otherwise the same) and a tile for every
// compute unit at most (512 tiles, M = 8, b = 2^16: 79 us a step with one group, 81 with four; blocks of 2^9, d = 2 * 10^6, M = 4
// 34.3 and 41.4).
constexpr int kServerGroups = 4;
bool share_workers(const fo_plan *pl, const SmallArgs &a)
{
    return !a.count && a.M >= (uint32_t)kServerGroups && pl->sm_tiles <= pl->num_cus;
}

// Stages above the contiguous tile, b > 2^12.
template <int MODE, int G = 1>
int launch_high(fo_plan *pl, uint32_t nslots, hipStream_t st, const SmallArgs &a, const PtrTab &tab)
{
    if constexpr (MODE == SMH_SERVER && G == 1) {
        if (share_workers(pl, a)) return launch_high<MODE, kServerGroups>(pl, nslots, st, a, tab);
    }
    const int kid = MODE == SMH_ENC ? KID_SM_ENC_HIGH : MODE == SMH_SERVER ? KID_SM_SERVER_HIGH : KID_SM_DEC_HIGH;
    const dim3 grid((unsigned)pl->sm_tiles, nslots), block(kSmThreads * G);
    switch (pl->logb - kSmLog2) {
    case 1: return launch(pl, kid, k_small_high<MODE, 1, G>, grid, block, st, a, tab);
    case 2: return launch(pl, kid, k_small_high<MODE, 2, G>, grid, block, st, a, tab);
    case 3: return launch(pl, kid, k_small_high<MODE, 3, G>, grid, block, st, a, tab);
    case 4: return launch(pl, kid, k_small_high<MODE, 4, G>, grid, block, st, a, tab);
    case 5: return launch(pl, kid, k_small_high<MODE, 5, G>, grid, block, st, a, tab);
    case 6: return launch(pl, kid, k_small_high<MODE, 6, G>, grid, block, st, a, tab);
    case 7: return launch(pl, kid, k_small_high<MODE, 7, G>, grid, block, st, a, tab);
    case 8: return launch(pl, kid, k_small_high<MODE, 8, G>, grid, block, st, a, tab);
    }
    return FO_EINVAL;
}

template <int IN, bool DEC>
int launch_low(fo_plan *pl, uint32_t nslots, hipStream_t st, const SmallArgs &a, const PtrTab &tab)
{
    const dim3 grid((unsigned)pl->sm_tiles, nslots), block(kSmThreads);
    const bool dither = a.dither == FO_DITHER_UNIFORM;
    const int kid = IN == SMI_GRAD ? KID_SM_ENC_GRAD : KID_SM_ENC_MID;
    if (a.K > 1) {
        if (dither) return launch(pl, kid, k_small_encode<IN, true, true, DEC>, grid, block, st, a, tab);
        return launch(pl, kid, k_small_encode<IN, false, true, DEC>, grid, block, st, a, tab);
    }
    if (dither) return launch(pl, kid, k_small_encode<IN, true, false, DEC>, grid, block, st, a, tab);
    return launch(pl, kid, k_small_encode<IN, false, false, DEC>, grid, block, st, a, tab);
}

template <bool UPDATE, int G = 1>
int launch_mean(fo_plan *pl, hipStream_t st, const SmallArgs &a)
{
    if constexpr (G == 1) {
        if (share_workers(pl, a)) return launch_mean<UPDATE, kServerGroups>(pl, st, a);
    }
    const dim3 grid((unsigned)pl->sm_tiles), block(kSmThreads * G);
    const bool dither = a.dither == FO_DITHER_UNIFORM;
    if (a.K > 1) {
        if (dither) return launch(pl, KID_SM_SERVER, k_small_server<true, true, UPDATE, G>, grid, block, st, a);
        return launch(pl, KID_SM_SERVER, k_small_server<false, true, UPDATE, G>, grid, block, st, a);
    }
    if (dither) return launch(pl, KID_SM_SERVER, k_small_server<true, false, UPDATE, G>, grid, block, st, a);
    return launch(pl, KID_SM_SERVER, k_small_server<false, false, UPDATE, G>, grid, block, st, a);
}

// Both passes of the encoder in one launch, 2^12 < b <= 2^16.
template <int HB>
int launch_block(fo_plan *pl, hipStream_t st, const SmallArgs &a)
{
    const dim3 grid((unsigned)pl->sm_tiles), block(kSmThreads * small_block_groups(HB));
    const bool dither = a.dither == FO_DITHER_UNIFORM;
    if (a.stat_clipped) return FO_EINVAL;
    if (a.K > 1) {
        if (dither) return launch(pl, KID_SM_ENC_GRAD, k_small_block<HB, true, true>, grid, block, st, a);
        return launch(pl, KID_SM_ENC_GRAD, k_small_block<HB, false, true>, grid, block, st, a);
    }
    if (dither) return launch(pl, KID_SM_ENC_GRAD, k_small_block<HB, true, false>, grid, block, st, a);
    return launch(pl, KID_SM_ENC_GRAD, k_small_block<HB, false, false>, grid, block, st, a);
}

// What the decoder of one party's message (`party`) needs besides its input.
void set_decode(SmallArgs &a, const fo_plan *pl, uint32_t party, const float *scales, float *out, uint32_t store_mode, float delta)
{
    a.Kin = party == FO_PARTY_SERVER ? pl->p.K : 1u;
    a.planes_in = party == FO_PARTY_SERVER ? pl->planes : 1u;
    a.scales = const_cast<float *>(scales);
    a.eps_in = eps_party_of(pl, party);
    a.out = out; a.len_out = pl->p.d; a.store_mode = store_mode; a.delta = delta;
    a.out_coef = pl->rsqrtb * 2.f / (float)a.Kin; // half values; D = (lambda / K) D_eps H^T q
}

void set_stats(SmallArgs &a, const fo_plan *pl, uint32_t party)
{
    if (!pl->stats) return;
    const uint32_t at = party == FO_PARTY_SERVER ? FO_MAX_WORKERS : party;
    a.stat_clipped = pl->stats->clipped + at;
    a.stat_near = pl->stats->near_tie + at;
}

// What the server's message needs: amplitude rule, eps, quantiser.
void set_server(SmallArgs &a, const fo_plan *pl, const float *scales_up, uint64_t *bits_down, float *scales_down)
{
    const bool l2s = pl->p.server_scale == FO_SERVER_SCALE_L2;
    a.scale_mode = l2s ? SMS_MEASURED : SMS_SERVER;
    a.coef = l2s ? pl->coef_lambda_s : pl->coef_s;
    a.scales_up = scales_up;
    a.scales = scales_down; a.scales_stride = 0;
    a.bits_out = bits_down; a.bits_out_stride = 0;
    a.party0 = FO_PARTY_SERVER; a.eps_party0 = eps_party_of(pl, FO_PARTY_SERVER);
    a.K = pl->p.K; a.planes = pl->planes;
    set_stats(a, pl, FO_PARTY_SERVER);
}

// `dec`: leave the decoder's low stages of the messages in buf_a, one slot per party (b > 2^12).  tmp == nullptr (no scratch
// to be had, fo_encode_noalloc): one vector of blocks of at most 2^16 coordinates.
int encode(fo_plan *pl, const PtrTab *tab, const float *src, uint64_t src_stride, uint64_t len_in, uint32_t nslots, uint32_t party0,
           uint64_t round, bool scales_given, uint64_t *bits, uint64_t bits_stride, float *scales, uint64_t scales_stride, float *tmp,
           uint64_t tmp_stride, hipStream_t st, bool common, bool dec)
{
    PtrTab none;
    std::memset(&none, 0, sizeof(none));
    SmallArgs a = small_base(pl, rng_of(pl, round));
    a.src = src; a.src_stride = src_stride; a.use_tab = tab ? 1u : 0u; a.len_in = len_in;
    a.bits_out = bits; a.bits_out_stride = bits_stride;
    a.scales = scales; a.scales_stride = scales_stride;
    a.party0 = party0; a.eps_party0 = eps_party_of(pl, party0);
    a.scale_mode = scales_given ? SMS_GIVEN : SMS_MEASURED;
    a.coef = party0 == FO_PARTY_SERVER ? pl->coef_lambda_s : pl->coef_lambda;
    if (party0 == FO_PARTY_SERVER) { a.K = pl->p.K; a.planes = pl->planes; }
    set_stats(a, pl, party0);
    if (pl->logb <= (uint32_t)kSmLog2) {
        if (common && !scales_given) {
            a.scales_only = 1u;
            FO_TRY((launch_low<SMI_GRAD, false>(pl, nslots, st, a, tab ? *tab : none)));
            FO_TRY(launch_common_scales(pl, st, scales, nslots));
            a.scales_only = 0u;
            a.scale_mode = SMS_GIVEN;
        }
        return launch_low<SMI_GRAD, false>(pl, nslots, st, a, tab ? *tab : none);
    }
    if (!tmp) {
        if (tab || nslots != 1 || dec) return FO_EINVAL;
        switch (pl->logb - kSmLog2) {
        case 1: return launch_block<1>(pl, st, a);
        case 2: return launch_block<2>(pl, st, a);
        case 3: return launch_block<3>(pl, st, a);
        case 4: return launch_block<4>(pl, st, a);
        }
        return FO_EINVAL;
    }
    a.mid = tmp; a.mid_stride = tmp_stride;
    a.partials = pl->partials;
    FO_TRY(launch_high<SMH_ENC>(pl, nslots, st, a, tab ? *tab : none));
    a.src = tmp; a.src_stride = tmp_stride; a.use_tab = 0u;
    a.common = common ? nslots : 0u;
    if (dec) return launch_low<SMI_MID, true>(pl, nslots, st, a, none); // in place
    return launch_low<SMI_MID, false>(pl, nslots, st, a, none);
}

// `mid`: the decoder's low stages already done (else from `bits`)
int decode(fo_plan *pl, const uint64_t *bits, const float *mid, const float *scales, uint64_t round, uint32_t party, float *out,
           uint32_t store_mode, float delta, float *tmp, hipStream_t st)
{
    PtrTab none;
    std::memset(&none, 0, sizeof(none));
    SmallArgs a = small_base(pl, rng_of(pl, round));
    set_decode(a, pl, party, scales, out, store_mode, delta);
    const dim3 grid((unsigned)pl->sm_tiles), block(kSmThreads);
    a.bits_in = bits;
    if (pl->logb <= (uint32_t)kSmLog2) return launch(pl, KID_SM_DEC, k_small_decode<true>, grid, block, st, a);
    if (!mid) {
        a.mid = tmp;
        FO_TRY(launch(pl, KID_SM_DEC_LOW, k_small_decode<false>, grid, block, st, a));
        mid = tmp;
    }
    a.src = mid;
    return launch_high<SMH_DEC>(pl, 1, st, a, none);
}

// `mids`: the workers' messages are in buf_a with the decoder's low stages done.  x: also decode the server's message
// and update x.
int server(fo_plan *pl, const uint64_t *bits_up, const float *scales_up, bool mids, uint64_t round, uint64_t *bits_down,
           float *scales_down, float *gbar, float *x, float delta, hipStream_t st)
{
    PtrTab none;
    std::memset(&none, 0, sizeof(none));
    const bool shared = pl->p.eps_mode != FO_EPS_INDEPENDENT;
    SmallArgs a = small_base(pl, rng_of(pl, round));
    if (x) set_decode(a, pl, FO_PARTY_SERVER, scales_down, x, STORE_AXPY, delta);
    set_server(a, pl, scales_up, bits_down, scales_down);
    a.bits_in = bits_up; a.bits_in_stride = pl->W; // messages lie W words apart
    a.count = shared ? 1u : 0u;
    a.eps_in = shared ? kPartyAllWorkers : 0u;
    a.in_coef = 2.f * (pl->rsqrtb / (float)pl->p.M); // half values
    a.gbar = gbar;
    if (pl->logb <= (uint32_t)kSmLog2) return x ? launch_mean<true>(pl, st, a) : launch_mean<false>(pl, st, a);
    const uint32_t nmsg = shared ? 1u : pl->p.M;
    if (!mids) {
        SmallArgs d = a;
        d.mid = pl->buf_a; d.mid_stride = pl->ntot;
        FO_TRY(launch(pl, KID_SM_DEC_LOW, k_small_decode<false>, dim3((unsigned)pl->sm_tiles, nmsg), dim3(kSmThreads), st, d));
    }
    a.src = pl->buf_a; a.src_stride = pl->ntot;
    a.mid = pl->buf_b;
    a.partials = a.scale_mode == SMS_MEASURED ? pl->partials : nullptr;
    FO_TRY(launch_high<SMH_SERVER>(pl, 1, st, a, none));
    a.src = pl->buf_b;
    if (!x) return launch_low<SMI_MID, false>(pl, 1, st, a, none);
    FO_TRY((launch_low<SMI_MID, true>(pl, 1, st, a, none))); // in place
    return decode(pl, nullptr, pl->buf_b, scales_down, round, FO_PARTY_SERVER, x, STORE_AXPY, delta, nullptr, st);
}

} // namespace

int small_encode(fo_plan *pl, const PtrTab *tab, const float *src, uint64_t src_stride, uint64_t len_in, uint32_t nslots,
                 uint32_t party0, uint64_t round, bool scales_given, uint64_t *bits, uint64_t bits_stride, float *scales,
                 uint64_t scales_stride, float *tmp, uint64_t tmp_stride, hipStream_t st, bool common)
{
    return encode(pl, tab, src, src_stride, len_in, nslots, party0, round, scales_given, bits, bits_stride, scales, scales_stride,
                  tmp, tmp_stride, st, common, false);
}

int small_decode(fo_plan *pl, const uint64_t *bits, const float *scales, uint64_t round, uint32_t party, float *out,
                 uint32_t store_mode, float delta, float *tmp, hipStream_t st)
{
    return decode(pl, bits, nullptr, scales, round, party, out, store_mode, delta, tmp, st);
}

int small_server(fo_plan *pl, const uint64_t *bits_up, const float *scales_up, uint64_t round, uint64_t *bits_down,
                 float *scales_down, float *gbar_or_null, hipStream_t st)
{
    return server(pl, bits_up, scales_up, false, round, bits_down, scales_down, gbar_or_null, nullptr, 0.f, st);
}

int small_step(fo_plan *pl, const PtrTab &tab, float *x, float delta, uint64_t round, bool scales_given, hipStream_t st)
{
    const uint32_t M = pl->p.M, mode = pl->p.eps_mode;
    // with independent eps the server decodes every message, so the workers' kernel goes on with the decoder
    const bool mids = mode == FO_EPS_INDEPENDENT && pl->logb > (uint32_t)kSmLog2;
    FO_TRY(encode(pl, &tab, nullptr, 0, pl->p.d, M, 0, round, scales_given, pl->bits_up, pl->W, pl->scales_up, pl->nblocks,
                  pl->buf_a, pl->ntot, st, mode != FO_EPS_INDEPENDENT, mids));
    if (mode == FO_EPS_SHARED_ALL) { // no transform on the server
        FO_TRY(launch_server(pl, pl->bits_up, pl->scales_up, round, pl->bits_down, pl->scales_down, nullptr, st));
        return decode(pl, pl->bits_down, nullptr, pl->scales_down, round, FO_PARTY_SERVER, x, STORE_AXPY, delta, pl->buf_a, st);
    }
    return server(pl, pl->bits_up, pl->scales_up, mids, round, pl->bits_down, pl->scales_down, nullptr, x, delta, st);
}

} // namespace fo_host
