"""Transforms of 2^26 and 2^27 points take two passes (eleven and twelve stages over rows of 16 and 8 columns), longer
ones three.  The first two against the oracle; the three-pass server with several workers against the decoder and
the encoder, which test_gpu_max_size.py checks at that length."""
import numpy as np
import pytest

from tests.parity import check_round_trip, gates

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,M,blk,kw", [
    ((1 << 26) + 5, 2, 0, {}),                                     # twelve stages, most of the second half padding
    ((1 << 27) - 3, 2, 27, {"eps_mode": 1, "server_scale": 1}),    # one summed transform, measured-norm amplitude
    ((1 << 26) + 70_001, 1, 26, {"K": 3}),                         # two blocks of eleven stages, int32 intermediate
    (50_000_001, 2, 0, {}),                                        # eleven stages, independent workers, plain signs
    (1, 1, 26, {}),                                                # one coordinate: every tile but the first reads padding
    ((3 << 15) + 31, 1, 27, {}),                                   # ends inside a register's rows, on an odd coordinate
    ((1 << 26) + 300_001, 2, 26, {}),                              # two blocks, so regions of more than one, plain signs both ways
    ((1 << 25) + 40_003, 1, 25, {"dither": 1}),                    # ten stages in two blocks, quantiser without dither
    ((1 << 25) + 9, 1, 25, {"K": 5}),                              # and the K-fold one
], ids=["2p27", "2p27_shared_l2", "two_blocks_2p26_K3", "2p26", "one", "odd_end", "two_blocks_2p26", "two_blocks_2p25_no_dither",
        "two_blocks_2p25_K5"])
def test_two_pass_transforms_of_narrow_rows(oracle, d, M, blk, kw):
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    gs = [inputs.heavy_tailed(d, m) for m in range(M)]
    print(f"d={d} M={M} block_log2={blk} {kw}", flush=True)
    rep = check_round_trip(oracle, B, gs, d=d, M=M, block_log2=blk, seed=0x5A + M, rnd=3, delta=0.05,
                           device=torch.device("cuda:0"), threads=16, **kw)
    print(rep, flush=True)
    gates(rep)


def test_three_pass_server_with_several_workers():
    """n = 2^28: the mean is the average of the decoded messages (each exact but for one rounding of 2^-24, and M + 1
    roundings of the sum: 1e-6 covers them), and the downlink is the server's own encode of that mean."""
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    d, M, rnd = (1 << 27) + 9, 3, 5
    plan = B.Plan(d=d, M=M, seed=77)
    assert plan.ntot == 1 << 28
    gen = torch.Generator(device=dev)
    gen.manual_seed(4)
    bits_up = torch.randint(-(1 << 63), (1 << 63) - 1, (M, plan.W), generator=gen, device=dev, dtype=torch.int64)
    lam = torch.rand(M, 1, generator=gen, device=dev) + 0.5
    down = torch.zeros(1, plan.W, dtype=torch.int64, device=dev)
    lam_s = torch.zeros(1, device=dev)
    gbar = torch.zeros(plan.ntot, device=dev)
    plan.fo_server_aggregate(bits_up, lam, rnd, down, lam_s, gbar)
    want = torch.zeros(d, device=dev)
    out = torch.zeros(d, device=dev)
    for m in range(M):
        plan.fo_decode(bits_up[m], lam[m], rnd, m, out)
        want += out / M
    assert float((gbar[:d] - want).norm() / want.norm()) < 1e-6
    again = torch.zeros(plan.W, dtype=torch.int64, device=dev)
    plan.fo_encode(gbar, rnd, B.PARTY_SERVER, again, lam_s, flags=B.FORCE_SCALE)
    differ = (again ^ down[0]) != 0
    assert float(differ.float().mean()) < 1e-5   # near ties only: the fused pass adds in another order


@pytest.mark.parametrize("low", [8, 14])
@pytest.mark.parametrize("logb", [22, 25, 26, 27])
def test_top_stages_come_first(logb, low):
    """The encoder's strided pass takes the top index bits: the padding lies there, and a sum with one of its zeros is exact.
    Two entries of 2^26 that the top bit alone tells apart cancel in half of the transform, and what is left is the entry 1,
    whose sum with 2^26 would have been 2^26."""
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    top = 1 << (logb - 1)
    d = top + (1 << 15) + 3
    plan = B.Plan(d=d, M=1, dither=B.DITHER_NONE, seed=41)
    assert plan.b == 1 << logb and plan.nblocks == 1
    lam = torch.ones(1, device=dev)

    def encode(entries):
        g = torch.zeros(d, device=dev)
        for i, x in entries.items():
            g[i] = x
        bits = torch.zeros(plan.W, dtype=torch.int64, device=dev)
        plan.fo_encode(g, 7, 0, bits, lam, flags=B.FORCE_SCALE)
        return bits

    eps = [1 if int(encode({i: 1.0})[0]) & 1 else -1 for i in (0, top, 1 << low)]    # coordinate 0 of the transform of e_i
    got = encode({0: 2.0 ** 26, top: 2.0 ** 26, 1 << low: 1.0}).view(2, -1)
    lower_cancels = eps[0] != eps[1]
    left = got[0 if lower_cancels else 1]
    word = torch.arange(left.numel(), device=dev)
    positive = (((word >> (low - 6)) & 1) == 0) == (eps[2] > 0)
    assert torch.equal(left, -positive.long())
    assert torch.equal(got[1 if lower_cancels else 0], torch.full_like(left, -1 if eps[0] > 0 else 0))
    plan.close()
