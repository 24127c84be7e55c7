"""Transforms of three passes (longer than 2^27 points): whole rounds with several workers at n = 2^28, in every eps mode, with
the K-fold downlink and both measured amplitudes; and messages that are rows of the Walsh matrix, whose inverse transform
is the largest integer there is, at the lengths that keep their stages in int32 (2^26, 2^27 and 2^28).

The reference is the definition in fp64: eps from the oracle, the transform as 28 butterfly stages over torch's fp64 tensors on
the device, the quantiser (Def. 3.2) by the oracle on ranges of the transformed vector.  Stages are fed the library's own
upstream messages and fp32 amplitudes, as in parity.py, with its gates."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from tests.parity import SERVER, TIE, _peek

pytestmark = pytest.mark.gpu

RANGES = 1 << 16   # coordinates in each range on which signs are compared


def _wht(x):
    """Unnormalised transform, in place."""
    h = 1
    while h < x.numel():
        y = x.view(-1, 2, h)
        d = y[:, 0, :] - y[:, 1, :]
        y[:, 0, :] += y[:, 1, :]
        y[:, 1, :] = d
        h *= 2
    return x


def _signs(torch, bits, K=1):
    """Bit planes [P][W] -> the code 2 c - K as fp64, c the count that the planes hold (K = 1: the signs)."""
    shift = torch.arange(64, device=bits.device)
    c = torch.zeros(bits.shape[-1], 64, dtype=torch.float64, device=bits.device)
    for p, plane in enumerate(bits.view(-1, bits.shape[-1])):
        c += ((plane[:, None] >> shift) & 1) * float(1 << p)
    return c.mul_(2.0).sub_(float(K)).view(-1)


def _ranges(n):
    rs = np.random.default_rng(28)
    return [0, n - RANGES] + [int(i) * RANGES for i in rs.integers(1, n // RANGES - 1, size=6)]


def _check_codes(O, torch, q, z, lam, K, seed, rnd, party):
    for i0 in _ranges(z.numel()):
        want, margin = O.quantize(z[i0:i0 + RANGES].cpu().numpy(), lam, K=K, seed=seed, rnd=rnd, party=party, i0=i0, want_margin=True)
        got = q[i0:i0 + RANGES].cpu().numpy()
        assert not np.any((got != want) & (np.abs(margin) >= TIE * lam)), (party, i0)


def _rel(a, b):
    return float((a - b).norm() / b.norm())


@pytest.mark.parametrize("M,K,eps_mode,server_scale", [
    (3, 1, 0, 0),
    (2, 3, 0, 1),
    (3, 1, 1, 0),
    (2, 1, 1, 1),
    (2, 2, 2, 1),
    (3, 1, 2, 2),
], ids=["independent", "independent_K3_l2", "shared", "shared_l2", "all_K2_l2", "all_sup"])
def test_round_of_three_pass_transforms(oracle, M, K, eps_mode, server_scale):
    import torch
    from paper_2405_11095_amd import binding as B
    O, dev = oracle, torch.device("cuda:0")
    d, seed, rnd, delta = (1 << 27) + 9, 0x3A + M, (1 << 32) + 5, 0.25
    plan = B.Plan(d=d, M=M, K=K, eps_mode=eps_mode, server_scale=server_scale, seed=seed)
    n, W, rootn = plan.ntot, plan.W, float(1 << 14)
    assert n == 1 << 28
    print(f"n=2^28 M={M} K={K} eps={eps_mode} server={server_scale}", flush=True)

    with ThreadPoolExecutor(max_workers=4) as ex:
        streams = {O.eps_party(eps_mode, p) for p in [*range(M), SERVER]}
        filled = dict(zip(streams, ex.map(lambda s: O.eps_fill(seed, rnd, s, 0, n), streams)))
    eps_of = lambda party: torch.from_numpy(filled[O.eps_party(eps_mode, party)]).to(dev)

    gen = torch.Generator(device=dev)
    gen.manual_seed(M + 10 * K)
    gs = [torch.randn(d, generator=gen, device=dev) for _ in range(M)]
    bits = torch.zeros(M, W, dtype=torch.int64, device=dev)
    lam = torch.zeros(M, 1, device=dev)
    for m in range(M):
        plan.fo_encode(gs[m], rnd, m, bits[m], lam[m])
    for m in range(M):
        want = O.lam_rule(2.0, float(gs[m].double().norm()), n)
        assert abs(float(lam[m]) - want) <= 1e-6 * want
    if eps_mode:
        lam[:] = lam.max()
        for m in range(M):
            plan.fo_encode(gs[m], rnd, m, bits[m], lam[m], flags=B.FORCE_SCALE)
    down = torch.zeros(plan.planes, W, dtype=torch.int64, device=dev)
    lam_s = torch.zeros(1, device=dev)
    gbar = torch.zeros(n, device=dev)
    out = torch.zeros(d, device=dev)
    plan.fo_server_aggregate(bits, lam, rnd, down, lam_s, gbar)
    plan.fo_decode(down, lam_s, rnd, SERVER, out)

    # uplink and mean
    mean = torch.zeros(n, dtype=torch.float64, device=dev)
    for m in range(M):
        e, q = eps_of(m), _signs(torch, bits[m])
        z = torch.zeros(n, dtype=torch.float64, device=dev)
        z[:d] = gs[m]
        _check_codes(O, torch, q, _wht(z.mul_(e)).div_(rootn), float(lam[m]), 1, seed, rnd, m)
        mean += _wht(q).mul_(e).mul_(float(lam[m]) / (rootn * M))
        del z, q, e
    assert _rel(gbar.double(), mean) <= 1e-6
    # amplitude and downlink
    want = (O.lam_rule(2.0, float(mean.norm()), n) if server_scale == 1 else float(lam.max()) if server_scale == 2 else
            2.0 * float(lam.max()) * np.sqrt(np.log(n)))
    assert abs(float(lam_s) - want) <= 1e-6 * want
    e, q = eps_of(SERVER), _signs(torch, down, K)
    _check_codes(O, torch, q, _wht(mean.mul_(e)).div_(rootn), float(lam_s), K, seed, rnd, SERVER)
    del mean
    # decode
    assert _rel(out.double(), _wht(q).mul_(e).mul_(float(lam_s) / (rootn * K))[:d]) <= 1e-6
    del q, e
    # a step: the same messages, and the update
    x0 = torch.randn(d, generator=gen, device=dev)
    x = x0.clone()
    plan.fo_step(gs, x, delta, rnd)
    torch.cuda.synchronize()
    pb_up, ps_up, pb_dn, ps_dn = plan.fo_step_messages()
    for addr, mine in ((pb_up, bits), (ps_up, lam), (pb_dn, down), (ps_dn, lam_s)):
        assert np.array_equal(_peek(torch, addr, mine.numel(), mine.dtype, dev), mine.cpu().numpy().reshape(-1))
    assert float((x - (x0 - delta * out)).abs().max()) <= 2.0 ** -22 * float(x0.abs().max() + delta * out.abs().max())
    # linear in the amplitude, whatever its sign
    if eps_mode == 0:
        minus, mean2 = torch.zeros(d, device=dev), torch.zeros(n, device=dev)
        plan.fo_decode(bits[1], lam[1], rnd, 1, out)
        plan.fo_decode(bits[1], -lam[1], rnd, 1, minus)
        assert float(out.abs().max()) > 0 and torch.equal(minus, -out)
        lam[1] = -lam[1]
        plan.fo_server_aggregate(bits, lam, rnd, down, lam_s, mean2)
        assert _rel(mean2[:d], gbar[:d] - 2.0 * out / M) <= 1e-6
    plan.close()


@pytest.mark.parametrize("logn,eps_mode", [(26, 0), (27, 0), (28, 0), (26, 1), (27, 1), (28, 1)])
def test_walsh_rows_through_long_transforms(oracle, logn, eps_mode):
    """Every worker sends row j of the Walsh matrix (j = 0: all ones).  H^T of it is n at coordinate j and zero elsewhere, 2^27 in
    half values at n = 2^28: past what fp32 counts in.  Decode, mean and downlink have closed forms."""
    import torch
    from paper_2405_11095_amd import binding as B
    O, dev = oracle, torch.device("cuda:0")
    n, M, seed, rnd = 1 << logn, 3, 51, 2
    plan = B.Plan(d=n, M=M, eps_mode=eps_mode, seed=seed)
    W, rootn = plan.W, float(n) ** 0.5
    lams = [0.75] * M if eps_mode else [1.0, 0.5, 0.8125]
    lam = torch.tensor(lams, device=dev).view(M, 1)
    down = torch.zeros(W, dtype=torch.int64, device=dev)
    lam_s, gbar, out = torch.zeros(1, device=dev), torch.zeros(n, device=dev), torch.zeros(n, device=dev)
    eps_at = lambda party, i: float(O.eps(seed, rnd, O.eps_party(eps_mode, party), [i])[0])
    for j in (0, n - 1, (n >> 1) | (n >> 12) | 33):
        i = torch.arange(n, device=dev) & j
        for s in (16, 8, 4, 2, 1):
            i ^= i >> s
        row = ((i & 1) == 0).view(W, 64)
        weights = torch.ones(64, dtype=torch.int64, device=dev) << torch.arange(64, device=dev)
        word = (row * weights).sum(1)                  # wraps into the sign bit, as the packed words do
        del i, row
        bits = word.repeat(M, 1)
        for party in (1, SERVER):
            plan.fo_decode(bits[1], lam[1], rnd, party, out)
            assert int((out != 0).sum()) == 1
            want = lams[1] * rootn * eps_at(party, j)
            assert abs(float(out[j]) - want) <= 1e-6 * abs(want)
        plan.fo_server_aggregate(bits, lam, rnd, down, lam_s, gbar)
        assert int((gbar != 0).sum()) == 1
        want = sum(l * eps_at(m, j) for m, l in enumerate(lams)) * rootn / M
        assert abs(float(gbar[j]) - want) <= 1e-6 * abs(want)
        # H D_eps of that spike is row j again, times its value
        q = _signs(torch, down)
        z = _signs(torch, word).mul_(want * eps_at(SERVER, j) / rootn)
        _check_codes(O, torch, q, z, float(lam_s), 1, seed, rnd, SERVER)
        del q, z
    plan.close()
