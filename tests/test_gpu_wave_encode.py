"""The encoder of blocks of 2^6 to 2^12 coordinates in which a wave does everything: blocks that share a wave's 4096
coordinates do not touch one another, whatever one of them holds, and the ends of its range (a part that is partly padding,
amplitudes given instead of measured).  Whole rounds against the oracle at these lengths are in test_gpu_long_plans.py."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("blk", [6, 7, 8, 9, 10, 11, 12])
def test_blocks_of_a_wave_are_independent(blk):
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    d = (1 << 22) + 3 * 4096 + 77                  # past the short vectors; the last part holds 77 coordinates
    gen = torch.Generator(device=dev)
    gen.manual_seed(blk)
    g = torch.randn(d, generator=gen, device=dev)
    plan = B.Plan(d=d, M=1, block_log2=blk, seed=31)

    def encode(v, lam=None):
        bits = torch.zeros(plan.W, dtype=torch.int64, device=dev)
        scales = torch.zeros(plan.nblocks, device=dev) if lam is None else lam.clone()
        plan.fo_encode(v, 9, 0, bits, scales, flags=0 if lam is None else B.FORCE_SCALE)
        return bits.view(plan.nblocks, -1), scales

    plan.fo_profile_begin()
    bits, lam = encode(g)
    torch.cuda.synchronize()
    assert set(plan.fo_profile_end()) == {"k_enc_wave"}
    norms = torch.nn.functional.pad(g.double(), (0, plan.ntot - d)).view(plan.nblocks, -1).norm(dim=1)
    coef = 2.0 * (torch.log(torch.tensor(float(plan.b), dtype=torch.float64)) / plan.b).sqrt().item()
    assert float((lam.double() / (coef * norms) - 1).abs().max()) < 1e-6

    special = {0: float("nan"), 5: 0.0, 6: 1e15, 7: float("inf"), plan.nblocks - 1: float("nan")}   # factor on the whole block
    h = torch.nn.functional.pad(g, (0, plan.ntot - d)).view(plan.nblocks, -1).clone()
    for j, f in special.items():
        h[j] *= f
    bits2, lam2 = encode(h.view(-1)[:d].contiguous())
    rest = torch.ones(plan.nblocks, dtype=torch.bool, device=dev)
    rest[list(special)] = False
    assert torch.equal(bits2[rest], bits[rest]) and torch.equal(lam2[rest], lam[rest])
    assert not bits2[0].any() and not bits2[plan.nblocks - 1].any() and bool(lam2[0].isnan())   # NaN compares false
    assert bool((bits2[5] == -1).all()) and float(lam2[5]) == 0                                 # zeros are +1
    assert float(lam2[7]) == float("inf")
    # amplitudes handed in: the measured ones give the same message
    again, _ = encode(g, lam)
    assert torch.equal(again, bits)
    plan.close()


@pytest.mark.parametrize("blk", [6, 7, 8, 9, 10, 11, 12, 13, 15])
def test_every_kernel_finds_the_same_amplitude(blk):
    """Counters attached, a K-fold quantiser and none of the dither take another kernel than the plain message: the amplitudes
    they measure are the same to the bit."""
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    d = (1 << 22) + 5 * 4096 + 333
    gen = torch.Generator(device=dev)
    gen.manual_seed(100 + blk)
    first = None
    for kw in ({}, {"K": 3}, {"dither": 1}):
        plan = B.Plan(d=d, M=1, block_log2=blk, seed=31, **kw)
        if first is None:
            g = torch.randn(plan.ntot, generator=gen, device=dev)
        bits = torch.zeros(plan.planes, plan.W, dtype=torch.int64, device=dev)
        for stats in (None, torch.zeros(2 * (B.MAX_WORKERS + 1), dtype=torch.int64, device=dev)):
            plan.fo_set_stats(stats)
            lam = torch.zeros(plan.nblocks, device=dev)
            plan.fo_encode(g, 9, B.PARTY_SERVER, bits, lam)
            torch.cuda.synchronize()
            first = lam if first is None else first
            print(f"2^{blk} {kw} counters {stats is not None}: {int((lam != first).sum())} of {plan.nblocks} differ", flush=True)
            assert torch.equal(lam, first)
        plan.fo_set_stats(None)
        plan.close()
