"""Plans just past what the kernels for short vectors take: the kernels that serve every longer plan, at sizes that the oracle
computes in a second or two.  Whole rounds over every block length from 2^6 up with both quantisers, no dither and the three eps
modes; the diagnostic counters; messages that are rows of the Walsh matrix; and a seeded sweep over random configurations.
The timing facility says which kernels ran: none of those for short vectors but the decoder of blocks of at most 2^12, which is
one at every length."""
import numpy as np
import pytest

from tests.parity import SERVER, _peek, check_round_trip, compare_bits, gates

pytestmark = pytest.mark.gpu

# the longest padded length that the kernels for short vectors take, by log2 of the transform length (any number of workers)
LONGEST = {**{k: 1 << 22 for k in range(6, 13)}, 13: 1 << 20, 14: 1 << 20, 15: 1 << 20, **{k: 1 << 21 for k in range(16, 21)}, 21: 0}

CASES = [
    # log2 of the block length, coordinates past the line, M, options
    (6, 101, 1, {}),
    (6, 1, 1, {"K": 3}),
    (6, 77, 2, {"eps_mode": 1, "server_scale": 1}),
    (7, 129, 2, {}),
    (7, 65, 1, {"K": 2, "eps_mode": 1}),
    (7, 5, 1, {"dither": 1}),
    (8, 33, 1, {"K": 5, "dither": 1}),
    (9, 700, 2, {"server_scale": 1}),
    (9, 1, 1, {"eps_mode": 2, "K": 3}),
    (10, 1, 2, {"K": 4}),
    (11, 9_999, 2, {"server_scale": 1}),
    (12, 4097, 1, {"K": 129}),
    (12, 1, 2, {"scale_rule": 0, "Bnorm": 60.0}),
    (13, 1, 2, {}),
    (13, 70_001, 2, {"K": 3}),
    (14, 20_001, 2, {"dither": 1}),
    (14, 1, 3, {"eps_mode": 1, "K": 2}),
    (15, 1, 2, {}),
    (15, 40_000, 2, {"K": 3}),
    (15, 9, 2, {"eps_mode": 1, "server_scale": 1}),
    (15, 3, 1, {"dither": 1}),
    (16, 1, 2, {"K": 3}),
    (16, 40_001, 2, {"dither": 1}),
    (16, 9_999, 1, {"dither": 1, "K": 2}),
    (16, 65_535, 2, {"eps_mode": 2, "server_scale": 2}),
    (17, 1, 2, {}),                                             # two strided stages; then three, four, five, six
    (17, 1, 1, {"eps_mode": 1, "server_scale": 1}),
    (18, 200_001, 2, {}),
    (18, 5, 2, {"K": 3, "server_scale": 1}),
    (19, 7, 2, {}),
    (19, 300_001, 1, {"dither": 1, "eps_mode": 1}),
    (20, 11, 2, {"scale_rule": 0, "Bnorm": 60.0}),
    (20, 1, 1, {"K": 15}),
    (21, 1_300_001, 2, {}),
    (21, 2_000_001, 1, {"eps_mode": 2, "K": 3}),
]


def _kernels(torch, binding, gs, d, M, blk, **kw):
    """Names of the kernels that a step launches."""
    dev = torch.device("cuda:0")
    plan = binding.Plan(d=d, M=M, block_log2=blk, seed=1, **kw)
    x = torch.zeros(d, device=dev)
    gd = [torch.from_numpy(g).to(dev) for g in gs]
    plan.fo_profile_begin()
    plan.fo_step(gd, x, 0.1, 1)
    torch.cuda.synchronize()
    names = set(plan.fo_profile_end())
    plan.close()
    return names


def _assert_long(names, blk):
    assert {k for k in names if k.startswith("k_small")} == ({"k_small_decode<FINAL>"} if blk <= 12 else set()), names


@pytest.mark.parametrize("blk,past,M,kw", CASES, ids=[f"b{c[0]}-{c[1]}" for c in CASES])
def test_rounds_of_long_plans(oracle, blk, past, M, kw):
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    d = LONGEST[blk] + past
    gs = [inputs.heavy_tailed(d, m) for m in range(M)]
    print(f"d={d} M={M} block_log2={blk} {kw}", flush=True)
    plan_kw = {("B" if k == "Bnorm" else k): v for k, v in kw.items()}
    _assert_long(_kernels(torch, B, gs, d, M, blk, **plan_kw), blk)
    rep = check_round_trip(oracle, B, gs, d=d, M=M, block_log2=blk, seed=0x70 + M + blk, rnd=(1 << 32) + 3, delta=0.05,
                           device=torch.device("cuda:0"), threads=16, **kw)
    print(rep, flush=True)
    gates(rep)


def test_workers_alone_can_make_a_plan_long(oracle):
    """The lines are on the length times the number of workers as well."""
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    for d, blk in (((1 << 18) + 1, 9), ((1 << 17) + 1, 14), ((1 << 18) + 1, 16)):
        M = 64
        gs = [inputs.gaussian(d, m) for m in range(M)]
        print(d, blk, flush=True)
        _assert_long(_kernels(torch, B, gs, d, M, blk), blk)
        rep = check_round_trip(oracle, B, gs, d=d, M=M, block_log2=blk, seed=0x64, rnd=3, delta=0.05, device=torch.device("cuda:0"),
                               threads=16)
        gates(rep)


@pytest.mark.parametrize("blk,past,K,party,dither", [
    (6, 77, 1, 0, 0), (7, 5, 3, SERVER, 0), (9, 1, 1, 1, 0), (11, 3, 1, 0, 1), (12, 9, 2, SERVER, 0), (13, 1, 1, 0, 0), (15, 1, 1, 1, 0),
    (15, 7, 3, SERVER, 1), (16, 1, 1, 0, 0), (16, 40_001, 2, SERVER, 0), (16, 1, 1, 1, 1), (18, 1, 1, 1, 0), (18, 5, 4, SERVER, 0),
])
def test_counters_of_long_plans(oracle, blk, past, K, party, dither):
    """fo_stats of one encode with a quarter of the rule's amplitude, against counts from the oracle's vector; and the message,
    which the counting variants form by the definition, against the oracle's."""
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    dev = torch.device("cuda:0")
    d, seed = LONGEST[blk] + past, 21 + blk
    plan = B.Plan(d=d, M=2, block_log2=blk, K=K, dither=dither, seed=seed)
    p = oracle.params(d=d, M=2, block_log2=blk, K=K, dither=dither, seed=seed)
    stats = torch.zeros(2 * (B.MAX_WORKERS + 1), dtype=torch.int64, device=dev)
    plan.fo_set_stats(stats)
    g = np.zeros(plan.ntot if party == SERVER else d, dtype=np.float32)
    g[:d] = inputs.gaussian(d, 1)
    gd = torch.from_numpy(g).to(dev)
    planes = plan.planes if party == SERVER else 1
    bits = torch.zeros(planes, plan.W, dtype=torch.int64, device=dev)
    lam = torch.zeros(plan.nblocks, device=dev)
    plan.fo_encode(gd, 2, party, bits, lam)
    lam *= 0.25
    stats.zero_()
    plan.fo_encode(gd, 2, party, bits, lam, flags=B.FORCE_SCALE)
    torch.cuda.synchronize()
    h = stats.cpu().numpy()
    lam64 = lam.cpu().numpy().astype(np.float64)
    k = K if party == SERVER else 1
    r = oracle.encode(p, g[:d].astype(np.float64), 2, party, K=1, lam=lam64, want_margin=True, want_z=True)  # the first dither
    each = np.repeat(lam64, plan.b)[:plan.ntot]
    at, near = (B.MAX_WORKERS if party == SERVER else party), B.MAX_WORKERS + 1
    # a coordinate within rounding (2e-7 lambda) of a threshold may be counted on either side: one or two in 2^22
    assert abs(int(h[at]) - int(np.count_nonzero(np.abs(r["z"]) > each))) <= 5 and h[at] > plan.ntot // 100
    assert abs(int(h[near + at]) - int(np.count_nonzero(np.abs(r["margin"]) < 1e-6 * each))) <= 5
    assert int(h.sum()) == int(h[at] + h[near + at])
    if k == 1:
        bad, exempt, raw = compare_bits(bits[0].cpu().numpy().view(np.uint64), r["margin"], lam64, plan.b)
        assert bad == 0, (bad, exempt, raw)
    plan.close()


@pytest.mark.parametrize("blk,past", [(12, 1), (13, 1), (14, 1), (15, 1), (16, 1), (17, 1), (20, 1)])
def test_walsh_rows_through_long_plans(oracle, blk, past):
    """Every block of every message is row j of the Walsh matrix: b at coordinate j of the block, the largest integer of the
    decode side, and zeros elsewhere, through the decoder and the server's mean."""
    import torch
    from paper_2405_11095_amd import binding as B
    O, dev, M, seed, rnd = oracle, torch.device("cuda:0"), 2, 23, 6
    plan = B.Plan(d=LONGEST[blk] + past, M=M, block_log2=blk, seed=seed)
    n, b, nb, W = plan.ntot, plan.b, plan.nblocks, plan.W
    lam = torch.stack([torch.linspace(1.0, 2.0, nb, device=dev), torch.linspace(0.25, 0.5, nb, device=dev)])
    down, lam_s = torch.zeros(W, dtype=torch.int64, device=dev), torch.zeros(nb, device=dev)
    gbar, out = torch.zeros(n, device=dev), torch.zeros(plan.d, device=dev)
    for j in (0, b - 1, (b >> 1) | 33):
        i = np.arange(b, dtype=np.uint64) & np.uint64(j)
        for s in (16, 8, 4, 2, 1):
            i ^= i >> np.uint64(s)
        word = O.pack(np.tile(1 - 2 * (i & np.uint64(1)).astype(np.int32), nb))
        bits = torch.from_numpy(word.view(np.int64)).to(dev).repeat(M, 1)
        at = np.arange(nb) * b + j
        eps = [O.eps(seed, rnd, O.eps_party(0, m), at) for m in range(M)]
        plan.fo_decode(bits[1], lam[1], rnd, 1, out)
        plan.fo_server_aggregate(bits, lam, rnd, down, lam_s, gbar)
        torch.cuda.synchronize()
        got, mean, lam64 = out.cpu().numpy(), gbar.cpu().numpy(), lam.cpu().numpy().astype(np.float64)
        inside = at < plan.d
        want = lam64[1] * eps[1] * np.sqrt(b)
        assert np.count_nonzero(got) == np.count_nonzero(inside)
        assert np.allclose(got[at[inside]], want[inside], rtol=1e-6, atol=0)
        want = (lam64[0] * eps[0] + lam64[1] * eps[1]) * np.sqrt(b) / M
        assert np.count_nonzero(mean) == nb and np.allclose(mean[at], want, rtol=1e-6, atol=0)
    plan.close()


def _draw(rng):
    blk = int(rng.choice([6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19, 20, 21]))
    most = {21: 21, 13: 21, 14: 21, 15: 21}.get(blk, 23)
    d = int(rng.integers(max(LONGEST[blk] + 1, 1 << 20), 1 << most))
    return dict(d=d, M=int(rng.choice([1, 1, 2, 3])), blk=blk, K=int(rng.choice([1, 1, 2, 5])), eps_mode=int(rng.choice([0, 0, 1, 2])),
                server_scale=int(rng.choice([0, 1])), dither=int(rng.choice([0, 0, 0, 1])), scale_rule=int(rng.choice([1, 1, 0])),
                kind=str(rng.choice(["gaussian", "heavy", "sparse"])))


CONFIGS = [_draw(np.random.default_rng([2405, 11095, 77, i])) for i in range(24)]


@pytest.mark.parametrize("cfg", CONFIGS, ids=[f"{i:02d}" for i in range(len(CONFIGS))])
def test_random_long_plans(oracle, cfg):
    import torch
    from paper_2405_11095_amd import binding as B, inputs
    gen = {"gaussian": inputs.gaussian, "heavy": inputs.heavy_tailed, "sparse": inputs.sparse_gaussian}[cfg["kind"]]
    gs = [gen(cfg["d"], m) for m in range(cfg["M"])]
    bnorm = 1.5 * max(float(np.linalg.norm(g.astype(np.float64))) for g in gs) + 1e-3
    print(cfg, flush=True)
    rep = check_round_trip(oracle, B, gs, cfg["d"], cfg["M"], cfg["blk"], seed=0xC0FFEE + cfg["d"], rnd=3, delta=1e-2,
                           device=torch.device("cuda:0"), threads=16, K=cfg["K"], eps_mode=cfg["eps_mode"],
                           server_scale=cfg["server_scale"], dither=cfg["dither"], scale_rule=cfg["scale_rule"], Bnorm=bnorm)
    gates(rep)


@pytest.mark.parametrize("M,blk", [(1, 17), (6, 17), (7, 17), (1, 22), (6, 22)])
def test_amplitudes_of_two_pass_plans(M, blk):
    """The low pass adds up the strided pass's partial sums in plans of up to four tiles for every compute unit (1024), a
    kernel of its own beyond; either way every block has its norm's amplitude, a block of NaN its NaN."""
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    d = (160 << 15) - 77                                # 160 tiles of 2^15: six workers are within, seven are not
    gen = torch.Generator(device=dev)
    gen.manual_seed(blk)
    g = torch.randn(d, generator=gen, device=dev)
    g[3] = float("nan")
    plan = B.Plan(d=d, M=M, block_log2=blk, seed=5)
    bits, lam = torch.zeros(plan.W, dtype=torch.int64, device=dev), torch.zeros(plan.nblocks, device=dev)
    plan.fo_profile_begin()
    plan.fo_encode(g, 1, 0, bits, lam)
    torch.cuda.synchronize()
    tiles = plan.ntot >> 15
    assert ("scale kernels" in plan.fo_profile_end()) == (M * tiles > 1024)
    norms = torch.nn.functional.pad(g.double(), (0, plan.ntot - d)).view(plan.nblocks, -1).norm(dim=1)
    coef = 2.0 * (torch.log(torch.tensor(float(plan.b), dtype=torch.float64)) / plan.b).sqrt().item()
    assert bool(lam[0].isnan())
    assert plan.nblocks == 1 or float((lam[1:].double() / (coef * norms[1:]) - 1).abs().max()) < 1e-6
    plan.close()


def test_step_and_call_by_hand_add_partial_sums_alike():
    """fo_encode adds up a block's partial sums in its low pass, fo_step with a shared eps in a kernel of its own.  Squares whose
    sum is m^2 for an odd m of 25 bits, and two more of 0.4 ulp of it, which reach it in one addition or in two: the root rounds
    to m - 1 or m + 1."""
    import torch
    from paper_2405_11095_amd import binding as B
    dev = torch.device("cuda:0")
    d = 1 << 23                                            # 256 tiles of 128 columns; entries lie in the first row
    coef = np.float32(2.0 * np.sqrt(np.log(d) / d))
    m = 3 * (1 << 23) + 1                                  # an ulp of m^2 is an eighth and moves the root by 0.67 ulp
    while (m // 2) % 2 or coef * np.float32(m - 1) == coef * np.float32(m + 1):    # a tie that goes down, and shows
        m += 2
    squares, rest = [], m * m
    while rest:                                            # m^2 as squares of twelve bits
        k = max(0, (rest.bit_length() - 23) // 2)
        x = min(int(np.sqrt(float(rest))) >> k, 4095) << k
        squares.append(x)
        rest -= x * x
    assert len(squares) < 64 and sum(x * x for x in squares) == m * m and squares[0] ** 2 > 1 << 49
    g = torch.zeros(d, device=dev)
    for tile, x in enumerate(squares):
        g[128 * tile] = float(x)
    for tile in (64, 192):
        g[128 * tile] = 0.05 ** 0.5
    plan = B.Plan(d=d, M=1, eps_mode=B.EPS_SHARED_WORKERS, seed=3)
    assert plan.nblocks == 1 and plan.b == d
    bits, lam = torch.zeros(plan.W, dtype=torch.int64, device=dev), torch.zeros(1, device=dev)
    plan.fo_encode(g, 1, 0, bits, lam)
    plan.fo_step([g], torch.zeros(d, device=dev), 0.1, 1)
    torch.cuda.synchronize()
    step = _peek(torch, plan.fo_step_messages()[1], 1, torch.float32, dev)
    assert float(lam[0]) in (float(coef * np.float32(m - 1)), float(coef * np.float32(m + 1)))
    assert float(step[0]) == float(lam[0])
    plan.close()
