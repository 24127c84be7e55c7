"""fo_encode_noalloc (the entry point for callers that cannot allocate: static device scratch, no plan) against
fo_encode on the same inputs: same packed signs and same amplitudes, bit for bit, on calls made one after the
other that share the static array, each smaller than the one before."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SERVER = 0xFFFFFFFF


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2405_11095_amd import binding, inputs
    assert torch.cuda.is_available()
    binding.load_library()
    return binding, inputs, torch.device("cuda:0")


def _encode_both(B, torch, dev, g, d, M, blk, party, rnd, seed, force=None):
    plan = B.Plan(d=d, M=M, block_log2=blk, seed=seed)
    W, nb = plan.W, plan.nblocks
    bits_a = torch.zeros(W, dtype=torch.int64, device=dev)
    bits_b = torch.full((W,), -1, dtype=torch.int64, device=dev)
    lam_a = torch.zeros(nb, dtype=torch.float32, device=dev)
    lam_b = torch.full((nb,), -1.0, dtype=torch.float32, device=dev)
    flags = 0
    if force is not None:
        lam_a[:] = force
        lam_b[:] = force
        flags = B.FORCE_SCALE
    plan.fo_encode(g, rnd, party, bits_a, lam_a, flags=flags)
    B.fo_encode_noalloc(plan.params, g, rnd, party, bits_b, lam_b, flags=flags)
    torch.cuda.synchronize()
    plan.close()
    return bits_a.cpu().numpy(), bits_b.cpu().numpy(), lam_a.cpu().numpy(), lam_b.cpu().numpy()


def test_noalloc_encode_equals_plan_encode_on_consecutive_calls(env):
    import torch
    B, inputs, dev = env
    # (d, block_log2): the largest vector the entry point takes (n = 2^22, seven strided stages), then smaller ones
    # that reuse the same static array: a ragged two-pass one, blocks of 2^16 (one pass), a single tile
    cases = [((1 << 22) - 4321, 0), (70_001, 0), ((1 << 19) + 5, 16), (30_000, 0), (200_003, 12), (1 << 21, 0)]
    for k, (d, blk) in enumerate(cases):
        print(f"noalloc case d={d} block_log2={blk}", flush=True)
        g = torch.from_numpy(inputs.heavy_tailed(d, k)).to(dev)
        a, b, la, lb = _encode_both(B, torch, dev, g, d, 3, blk, party=k % 3, rnd=5 + k, seed=77 + k)
        assert np.array_equal(la, lb) and np.all(la > 0)
        assert np.array_equal(a, b)
        assert 0.3 < np.unpackbits(a.view(np.uint8)).mean() < 0.7     # a real message, not a cleared buffer
    # forced amplitudes and the server's party (input of the padded length)
    d = 150_000
    plan = B.Plan(d=d, M=2, seed=9)
    nt = plan.ntot
    plan.close()
    g = torch.from_numpy(inputs.gaussian(nt, 1)).to(dev)
    a, b, la, lb = _encode_both(B, torch, dev, g[:d].clone(), d, 2, 0, party=1, rnd=3, seed=9, force=0.01)
    assert np.array_equal(a, b) and np.array_equal(la, lb)


def test_noalloc_rejects_what_it_cannot_take(env):
    import torch
    B, inputs, dev = env
    d = B.NOALLOC_MAX_N + 1
    g = torch.zeros(64, dtype=torch.float32, device=dev)
    bits = torch.zeros(64, dtype=torch.int64, device=dev)
    lam = torch.zeros(64, dtype=torch.float32, device=dev)
    p = B.Params(d, 1, 0, 1, 0, 1, 0, 2.0, 2.0, 1.0, 1, 0)
    with pytest.raises(B.FoError) as e:
        B.fo_encode_noalloc(p, g, 0, 0, bits, lam)
    assert e.value.code == B.ESIZE and "FO_NOALLOC_MAX_N" in str(e.value)
    p = B.Params(1000, 1, 0, 1, 0, 1, 0, 1.0, 2.0, 1.0, 1, 0)      # alpha < 2
    with pytest.raises(B.FoError) as e:
        B.fo_encode_noalloc(p, g, 0, 0, bits, lam)
    assert e.value.code == B.EINVAL
    p = B.Params(1000, 2, 0, 1, 0, 1, 0, 2.0, 2.0, 1.0, 1, 0)
    with pytest.raises(B.FoError) as e:
        B.fo_encode_noalloc(p, g, 0, 2, bits, lam)                  # party out of range
    assert e.value.code == B.EINVAL
    with pytest.raises(B.FoError) as e:
        B.fo_encode_noalloc(p, g[1:], 0, 0, bits, lam)              # gradient not 16-byte aligned
    assert e.value.code == B.EALIGN


# every number of stages above a tile of 2^12, whole and ragged, one block and several; both quantisers, both dithers, both
# sources of the amplitude
ONE_LAUNCH = [
    # d, block_log2, party, options
    (8192, 0, 0, {}),
    (4097, 0, 1, {}),                                     # all of the second row but one coordinate is padding
    (10_001, 0, SERVER, {"K": 3}),
    (16_385 + 4096, 0, 0, {"dither": 1}),
    (32_767, 0, 1, {"scale_rule": 0, "B": 60.0}),
    (65_536, 0, 0, {}),
    (40_000, 0, SERVER, {"K": 255}),
    (33_000, 0, SERVER, {"K": 2, "dither": 1}),
    (100_001, 13, 1, {}),
    ((1 << 20) - 1, 14, 0, {"eps_mode": 1}),
    (70_000, 15, SERVER, {}),
    ((1 << 21) - 70_001, 16, 1, {}),
]


@pytest.mark.parametrize("d,blk,party,kw", ONE_LAUNCH, ids=[f"{c[0]}-{c[1]}" for c in ONE_LAUNCH])
def test_noalloc_encode_in_one_launch_equals_plan_encode(env, d, blk, party, kw):
    """Transforms of 2^13 to 2^16 points: the plan's two kernels and the one without scratch, to the bit."""
    import torch
    B, inputs, dev = env
    print(f"d={d} block_log2={blk} party={party:#x} {kw}", flush=True)
    plan = B.Plan(d=d, M=2, block_log2=blk, seed=d, **kw)
    n = plan.ntot if party == SERVER else d
    g = torch.from_numpy(inputs.heavy_tailed(n, 1)).to(dev)
    planes = plan.planes if party == SERVER else 1
    for flags in (0, B.FORCE_SCALE):
        out = []
        for noalloc in (False, True):
            bits = torch.full((planes, plan.W), 0x55 if noalloc else 0xAA, dtype=torch.int64, device=dev)
            lam = torch.full((plan.nblocks,), 0.02 if flags else -1.0, device=dev)
            if noalloc:
                B.fo_encode_noalloc(plan.params, g, 3, party, bits, lam, flags=flags)
            else:
                plan.fo_encode(g, 3, party, bits, lam, flags=flags)
            out.append((bits, lam))
        assert torch.equal(out[0][1], out[1][1]) and bool((out[0][1] > 0).all())
        assert torch.equal(out[0][0], out[1][0])
    plan.close()


def test_noalloc_encodes_of_short_transforms_may_overlap(env):
    """No scratch is shared by transforms of up to 2^16 points: calls in flight on four streams at once give what each
    gives alone."""
    import torch
    B, inputs, dev = env
    streams = [torch.cuda.Stream() for _ in range(4)]
    shapes = [(65_536, 0), (30_000, 0), (150_000, 14), (9_000, 0)]
    work = []
    for k, (d, blk) in enumerate(shapes):
        plan = B.Plan(d=d, M=1, block_log2=blk, seed=k)
        g = torch.from_numpy(inputs.gaussian(d, k)).to(dev)
        rounds = []
        for r in range(12):
            want, lam = torch.zeros(plan.W, dtype=torch.int64, device=dev), torch.zeros(plan.nblocks, device=dev)
            plan.fo_encode(g, r, 0, want, lam)
            rounds.append((want, lam, torch.zeros_like(want), torch.zeros_like(lam)))
        work.append((plan, g, rounds))
    torch.cuda.synchronize()
    for r in range(12):
        for s, (plan, g, rounds) in zip(streams, work):
            B.fo_encode_noalloc(plan.params, g, r, 0, rounds[r][2], rounds[r][3], stream=s.cuda_stream)
    torch.cuda.synchronize()
    for plan, g, rounds in work:
        for want, lam, bits, lam2 in rounds:
            assert torch.equal(bits, want) and torch.equal(lam2, lam)
        plan.close()
