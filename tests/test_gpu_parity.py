"""GPU parity tests: every call goes through the C ABI (libfo.so) and is compared with the CPU
oracle element by element.  Sizes span several 2^15 tiles, ragged tails, every kernel path
(short vectors, single-pass, two-pass; blocked and full-length; three passes are in
test_gpu_three_pass.py, plans just past the short ones in test_gpu_long_plans.py)."""
import numpy as np
import pytest

from tests.parity import check_round_trip, gates

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(oracle):
    import torch
    from paper_2405_11095_amd import binding, inputs
    assert torch.cuda.is_available()
    binding.load_library()
    return oracle, binding, inputs, torch.device("cuda:0")


CASES = [
    # name, d, M, block_log2, generator
    ("one_coordinate", 1, 2, 0, "gaussian"),
    ("one_word", 64, 3, 0, "gaussian"),
    ("one_word_plus_one", 65, 2, 0, "gaussian"),
    ("tiny_single_tile", 1000, 2, 0, "gaussian"),
    ("max_workers", 4096, 64, 0, "gaussian"),
    ("one_tile_exact", 1 << 15, 3, 0, "gaussian"),
    ("c1_two_pass_hb1", 1 << 16, 4, 0, "gaussian"),
    ("ragged_two_pass", 70_001, 3, 0, "gaussian"),
    ("two_pass_hb5", 1 << 20, 2, 0, "sparse"),
    ("ragged_hb7", (1 << 21) + 12345, 2, 0, "heavy"),
    ("blocked_b64", 5000, 2, 6, "gaussian"),
    ("blocked_b128", 40_000, 2, 7, "gaussian"),
    ("blocked_b256", 3000, 2, 8, "gaussian"),
    ("blocked_b512", 70_000, 2, 9, "gaussian"),
    ("blocked_b1024_ragged", 100_003, 3, 10, "layered"),
    ("blocked_b2048", 50_000, 2, 11, "heavy"),
    ("blocked_b4096", 1 << 18, 2, 12, "layered"),
    ("blocked_b8192", 100_000, 2, 13, "gaussian"),
    ("blocked_b16384", (1 << 18) + 77, 2, 14, "layered"),
    ("blocked_b32768", 100_000, 2, 15, "gaussian"),
    ("blocked_b65536", (1 << 19) + 5, 2, 16, "layered"),
    # blocks of two tiles: the last block's upper tile partly filled, then its lower tile partly filled
    ("blocked_b65536_upper_ragged", (1 << 16) + 40_000, 3, 16, "heavy"),
    ("blocked_b65536_lower_ragged", (1 << 17) + 9_999, 2, 16, "gaussian"),
    # the benchmark's geometry (n = 2^25: ten strided stages, the specialised kernels), fewer workers
    ("c3_geometry_n2p25", 25_557_032, 3, 0, "heavy"),
    # the same geometry with one worker (no prefetch of a next worker in the server pass), and two blocks of 2^25
    # (server tiles of the second block start 2^25 coordinates up), the second partly filled
    ("n2p25_single_worker", (1 << 24) + 1, 1, 0, "gaussian"),
    ("blocked_b2p25_two_blocks", (1 << 25) + 300_001, 2, 25, "gaussian"),
    # eleven strided stages (n = 2^26) with several workers: the fused server over the grouped int16 intermediates
    ("n2p26_with_three_workers", (1 << 25) + 77, 3, 0, "heavy"),
]


def _gen(inputs, kind, d, m):
    return {"gaussian": inputs.gaussian, "sparse": inputs.sparse_gaussian, "heavy": inputs.heavy_tailed,
            "layered": inputs.layered}[kind](d, m)


@pytest.mark.parametrize("name,d,M,blk,kind", CASES, ids=[c[0] for c in CASES])
def test_round_trip_parity(env, name, d, M, blk, kind):
    O, B, inputs, dev = env
    gs = [_gen(inputs, kind, d, m) for m in range(M)]
    print(f"case {name}: d={d} M={M} block_log2={blk}", flush=True)
    rep = check_round_trip(O, B, gs, d=d, M=M, block_log2=blk, seed=0xF05D + len(name), rnd=7, delta=0.05, device=dev)
    print(rep, flush=True)
    gates(rep)


def test_c3_at_full_size_in_the_benchmark_configuration(env):
    """The benchmark's workload as bench.py runs it (d = 25,557,032, n = 2^25, M = 16, batched launches through
    fo_step): every uplink bit of all 16 workers, the mean, every downlink bit, the decoded vector and the updated
    iterate against the oracle; fo_step's messages equal the ones of the calls made by hand."""
    O, B, inputs, dev = env
    wl = inputs.WORKLOADS["c3"]
    gs = inputs.workload("c3")
    rep = check_round_trip(O, B, gs, d=wl["d"], M=wl["M"], block_log2=0, seed=0xF05D + 3, rnd=2, delta=1e-3, device=dev,
                           threads=16)
    print(rep, flush=True)
    gates(rep)
    assert rep["uplink_exempt"] < 5000 and rep["downlink_exempt"] < 500   # near ties: about one coordinate in a million
