"""Blocks of 2^16: the encode in which a workgroup walks over blocks, with one block per workgroup, a ragged last block
beside the walk, one block more than there are compute units, several rounds whose last is not full, and workers whose
blocks share a workgroup."""
import pytest

from tests.parity import check_round_trip, gates

pytestmark = pytest.mark.gpu

CASES = [
    # blocks of 2^16, coordinates past them, M, options
    (40, 0, 1, {}),                                      # a workgroup each
    (257, 0, 1, {}),                                     # one workgroup takes two
    (90, 777, 3, {}),                                    # 270 whole blocks, the ragged ones in a launch of their own
    (61, 1, 9, {"eps_mode": 1, "server_scale": 1}),      # a pass for the norms, then the common amplitude
    (300, 65_535, 2, {"scale_rule": 0, "Bnorm": 60.0}),  # amplitude from the bound
]


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
