"""Blocks of 2^16: the encode in which a workgroup walks over blocks, with a block for every compute unit at most (no walk), one
block more than that, several rounds whose last is not full, workers whose blocks share a workgroup, and a ragged last block,
which is walked beside only from more than five whole blocks for every compute unit on.  The timing facility says which kernels
ran; the lines follow the device's number of compute units, the comments are for 256."""
import pytest

from tests.parity import check_round_trip, gates

pytestmark = pytest.mark.gpu

CASES = [
    # blocks of 2^16, coordinates past them, M, options
    (40, 0, 1, {}),                                      # a workgroup each
    (257, 0, 1, {}),                                     # one workgroup takes two
    (90, 777, 3, {}),                                    # 270 whole blocks and the ragged ones: a workgroup each
    (61, 1, 9, {"eps_mode": 1, "server_scale": 1}),      # a pass for the norms, then the common amplitude
    (300, 65_535, 2, {"scale_rule": 0, "Bnorm": 60.0}),  # amplitude from the bound; the mean's 301 blocks are walked over
    (90, 0, 3, {}),                                      # 270 blocks of three workers, whose blocks share workgroups
    (430, 777, 3, {}),                                   # 1290 whole blocks walked over, the ragged ones in a launch of their own
    (430, 1, 3, {"eps_mode": 1}),                        # the same with a common amplitude
]


def _expected(cus, blocks, rest, M):
    """{kernel: launches} of one fo_step with independent eps: the workers' encode and the encode of the mean."""
    want = {"k_contig_pair": 0, "k_contig_pair_walk": 0}
    if blocks * M > (5 if rest else 1) * cus:
        want["k_contig_pair_walk"] += 1
        want["k_contig_pair"] += 1 if rest else 0
    else:
        want["k_contig_pair"] += 1
    mean = blocks + (1 if rest else 0)
    want["k_contig_pair_walk" if mean > cus else "k_contig_pair"] += 1
    return {k: n for k, n in want.items() if n}


@pytest.mark.parametrize("blocks,rest,M,kw", CASES, ids=[f"{c[0]}-{c[1]}-{c[2]}" for c in CASES])
def test_walk_over_blocks(oracle, blocks, rest, M, kw):
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    d = (blocks << 16) + rest
    gs = [inputs.heavy_tailed(d, m) for m in range(M)]
    print(f"d={d} M={M} {kw}", flush=True)
    rep = check_round_trip(oracle, B, gs, d=d, M=M, block_log2=16, seed=0x16 + M, rnd=(1 << 32) + 3, delta=0.05,
                           device=torch.device("cuda:0"), threads=16, **kw)
    print(rep, flush=True)
    gates(rep)
    if not kw:
        dev = torch.device("cuda:0")
        plan = B.Plan(d=d, M=M, block_log2=16, seed=1)
        x = torch.zeros(d, device=dev)
        gd = [torch.from_numpy(g).to(dev) for g in gs]
        plan.fo_profile_begin()
        plan.fo_step(gd, x, 0.05, 1)
        torch.cuda.synchronize()
        ran = {k: n for k, (n, _) in plan.fo_profile_end().items() if k.startswith("k_contig_pair")}
        plan.close()
        assert ran == _expected(torch.cuda.get_device_properties(dev).multi_processor_count, blocks, rest, M)
