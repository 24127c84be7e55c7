"""The kernels for short vectors (tiles of 2^12 coordinates) at the edges of their range: every number of stages above
the tile, blocks from 2^6 up, ragged ends inside a tile, both quantisers, the three eps modes and server amplitudes, the
longest plan that takes them and the first that does not.  Every stage against the oracle."""
import pytest

from tests.parity import check_round_trip, gates

pytestmark = pytest.mark.gpu

CASES = [
    # d, M, block_log2, options
    (4096, 3, 0, {}),                                            # one whole tile
    (4097, 2, 0, {}),                                            # one stage above the tile
    (10_001, 2, 0, {"K": 3}),
    (3 * 8192 + 1, 2, 0, {"server_scale": 1}),                   # three stages, measured-norm amplitude
    (40_000, 33, 0, {}),                                         # four: the last without an exchange
    (70_001, 2, 0, {"eps_mode": 1}),                             # five
    (200_003, 2, 0, {"eps_mode": 2, "server_scale": 2}),         # six
    (300_001, 2, 0, {"K": 15}),                                  # seven
    (1_000_003, 2, 0, {"eps_mode": 1, "server_scale": 1, "K": 4}),  # eight
    (4096 + 63, 2, 6, {"K": 255}),                               # second tile: one block, its last coordinate padding
    (4096 * 3 + 1, 2, 7, {"server_scale": 1}),
    (12_345, 64, 9, {"eps_mode": 1}),
    (9_000, 2, 12, {"eps_mode": 2, "K": 2}),
    (50_000, 2, 11, {"scale_rule": 0, "Bnorm": 60.0}),           # amplitude from the bound
    (60_000, 2, 14, {"scale_rule": 0, "Bnorm": 60.0}),
    (20_000, 2, 0, {"dither": 1}),
    (3_000, 2, 8, {"dither": 1, "K": 3}),
    (1 << 22, 2, 12, {}),                                        # the longest one-pass plan, and one block more
    ((1 << 22) + 1, 2, 12, {}),
    (1 << 20, 2, 20, {}),                                        # the longest transform, and the next
    ((1 << 20) + 1, 2, 0, {}),
    (9_001, 3, 0, {}),                                           # workers one after the other, then dealt to four groups, unevenly
    (20_003, 5, 0, {"server_scale": 1}),
    (150_001, 7, 0, {"K": 3}),
    (1 << 20, 4, 0, {"server_scale": 1}),                        # a tile for every compute unit; one tile more
    ((1 << 20) + 5, 3, 13, {}),
    (20_011, 4, 12, {}),                                         # blocks of a tile and less: workers dealt to four groups
    (30_007, 7, 10, {"K": 3, "server_scale": 1}),
    (9_001, 35, 8, {"dither": 1}),                               # a second draw of eps words, for three workers
    (1 << 20, 5, 12, {}),                                        # a tile for every compute unit; one tile more
    ((1 << 20) + 5, 5, 9, {}),
]


@pytest.mark.parametrize("d,M,blk,kw", CASES, ids=[f"{c[0]}-{c[1]}-{c[2]}" for c in CASES])
def test_short_vectors(oracle, d, M, blk, kw):
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    gs = [inputs.heavy_tailed(d, m) for m in range(M)]
    print(f"d={d} M={M} block_log2={blk} {kw}", flush=True)
    rep = check_round_trip(oracle, B, gs, d=d, M=M, block_log2=blk, seed=0x5E + M, rnd=(1 << 32) + 3, delta=0.05,
                           device=torch.device("cuda:0"), threads=16, **kw)
    print(rep, flush=True)
    gates(rep)


@pytest.mark.parametrize("d,blk", [(5_000, 0), (10_000, 9), (4096 + 63, 6), (70_001, 0), (12_288, 12)])
def test_counters_of_short_vectors(oracle, d, blk):
    """fo_stats with every wave of every workgroup adding to the counters (an amplitude a quarter of the rule's clips a
    known share of the coordinates) and with none adding (the rule's own), against counts from the oracle's vector: equal
    but for coordinates within rounding of a threshold, of which there are fewer than three in a million."""
    import numpy as np
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    dev = torch.device("cuda:0")
    plan = B.Plan(d=d, M=2, block_log2=blk, seed=71)
    p = oracle.params(d=d, M=2, block_log2=blk, seed=71)
    stats = torch.zeros(2 * (B.MAX_WORKERS + 1), dtype=torch.int64, device=dev)
    plan.fo_set_stats(stats)
    g = inputs.gaussian(d, 1)
    gd = torch.from_numpy(g).to(dev)
    bits = torch.zeros(plan.W, dtype=torch.int64, device=dev)
    lam = torch.zeros(plan.nblocks, device=dev)
    plan.fo_encode(gd, 2, 1, bits, lam)
    torch.cuda.synchronize()
    near = B.MAX_WORKERS + 1
    free = stats.cpu().numpy()
    lam *= 0.25
    stats.zero_()
    plan.fo_encode(gd, 2, 1, bits, lam, flags=B.FORCE_SCALE)
    torch.cuda.synchronize()
    forced = stats.cpu().numpy()
    for h, f in ((free, 4.0), (forced, 1.0)):
        lam64 = lam.cpu().numpy().astype(np.float64) * f
        r = oracle.encode(p, g.astype(np.float64), 2, 1, lam=lam64, want_margin=True, want_z=True)
        each = np.repeat(lam64, plan.b)[:plan.ntot]
        assert abs(int(h[1]) - int(np.count_nonzero(np.abs(r["z"]) > each))) <= 2
        assert abs(int(h[near + 1]) - int(np.count_nonzero(np.abs(r["margin"]) < 1e-6 * each))) <= 2
        assert h[0] == 0 and h[near] == 0 and h[B.MAX_WORKERS] == 0
    assert forced[1] > plan.ntot // 100
    plan.close()


# log2 of the block, blocks in a tile for every compute unit at most and in more; 2^16: up to 2^24 coordinates of all workers
@pytest.mark.parametrize("blk,few,many,M", [(blk, few, many, M)
                                            for blk, few, many in ((6, 700, 19_300), (9, 20, 2_400), (12, 250, 300), (16, 8, 32), (17, 1, 16), (20, 1, 2))
                                            for M in (2, 3, 4, 5, 7, 8, 11) if (blk, M) != (16, 11)])
def test_groups_add_in_the_workers_order(blk, few, many, M):
    """Up to a tile for every compute unit, groups of threads share the workers; beyond, one group takes them one after the
    other.  The mean of a block is the same to the bit: the groups hand one another exact values only."""
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    assert (few << blk) / 4096 <= cus < (many << blk) / 4096
    gen = torch.Generator(device=dev)
    gen.manual_seed(M)
    bits = torch.randint(-(1 << 63), (1 << 63) - 1, (M, (many << blk) // 64), generator=gen, device=dev, dtype=torch.int64)
    lam = torch.rand(M, many, generator=gen, device=dev) + 0.5
    means = []
    for nb in (few, many):
        plan = B.Plan(d=nb << blk, M=M, block_log2=blk, seed=17)
        down, lam_s = torch.zeros(1, plan.W, dtype=torch.int64, device=dev), torch.zeros(nb, device=dev)
        gbar = torch.zeros(plan.ntot, device=dev)
        plan.fo_profile_begin()
        plan.fo_server_aggregate(bits[:, :plan.W].contiguous(), lam[:, :nb].contiguous(), 6, down, lam_s, gbar)
        torch.cuda.synchronize()
        assert any(k.startswith("k_small") for k in plan.fo_profile_end())
        means.append(gbar)
        plan.close()
    assert torch.equal(means[0], means[1][:few << blk])
