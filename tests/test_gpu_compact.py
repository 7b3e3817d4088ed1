"""K1 with compact suffix states (FP32, serial schedule, long rows) against
the general item body.

Both run the same operations in the same order, so every output must be
equal bit for bit.  Two shots per wavefront run the general body, one runs
the compact one (decode, ragged, no-allocation).  Graphs: columns of up to
6 and up to 8 checks (the two widths of the column sums), chunk counts that
are no multiple of the group, columns and checks without edges, priors above
1/2, equal priors (ties everywhere), and orders in which the messages rise
along the sweep, so that nearly every edge is a record and the chunks fall
back to their states.
"""
import numpy as np
import pytest

from synth.dem import circuit_dem, dem_from_dense, phenomenological_dem
from synth.sample import permutations, sample

from parity_helpers import check_valid

pytestmark = pytest.mark.gpu

DET = [0, 1, 2, 4, 5, 6]  # stats fields that do not depend on timing


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_15743_amd as P

    P.lib()
    return torch


def _random(m, n, deg, seed, equal=False, high=False):
    rng = np.random.default_rng(seed)
    h = np.zeros((m, n), np.uint8)
    for v in range(n):
        if v % 97 == 5:
            continue  # in no check
        h[rng.choice(m - 1, size=min(int(rng.integers(1, deg + 1)), m - 1), replace=False), v] = 1  # the last check stays empty
    if deg > 6:
        h[rng.choice(m - 1, size=deg, replace=False), 0] = 1
    pri = np.full(n, 2e-3) if equal else np.exp(rng.uniform(np.log(1e-4), np.log(2e-2), n))
    if high:
        pri[rng.choice(n, 9, replace=False)] = rng.uniform(0.51, 0.7, 9)
    return dem_from_dense(h, pri, rng.integers(0, 2, (2, n)).astype(np.uint8))


# (graph, L, M, T, order of the sweep)
CASES = {
    "circuit d=3": (lambda: circuit_dem(3, 3, 4e-3), 6, 2, 12, None),
    "circuit d=7": (lambda: circuit_dem(7, 7, 1e-3), 8, 3, 20, None),
    "circuit d=5, rising": (lambda: circuit_dem(5, 5, 2e-3), 4, 4, 10, "rising"),
    "columns of 6": (lambda: _random(33, 1501, 6, 1), 5, 5, 9, None),
    "columns of 8": (lambda: _random(60, 2003, 8, 2), 4, 1, 9, None),
    "columns of 8, rising": (lambda: _random(25, 997, 8, 3), 3, 2, 8, "rising"),
    "equal priors": (lambda: _random(40, 1700, 5, 4, equal=True), 4, 2, 10, None),
    "priors above 1/2": (lambda: _random(30, 900, 6, 5, high=True), 4, 2, 10, None),
}


def _graph(P, key, seed):
    mk, L, M, T, order = CASES[key]
    dem = mk()
    perms = permutations(dem.n, L, seed)
    if order == "rising":  # lambda ascending along the sweep
        perms = np.stack([np.argsort(-dem.priors + 1e-9 * np.random.default_rng(i).random(dem.n)) for i in range(L)])
    G = P.Graph.from_dem(dem, perms.astype(np.uint32), L=L, M=M, T_max=T, lsd_order=2)
    return dem, G


def _same(torch, a, b):
    (c1, o1, s1), (c2, o2, s2) = a, b
    assert torch.equal(c1, c2)
    assert torch.equal(o1, o2)
    assert torch.equal(s1[:, DET], s2[:, DET])


@pytest.mark.parametrize("key", list(CASES))
def test_compact_equals_general(torch_cuda, key):
    import paper_2508_15743_amd as P

    torch = torch_cuda
    print(f"case {key}", flush=True)
    dem, G = _graph(P, key, 11)
    synd = sample(dem, 203, 12).syndromes
    synd[3] = 0
    s = torch.from_numpy(synd).to("cuda:0")
    G.set_launch(slab_in_lds=0, shots_per_wave=2)
    ref = G.decode(s)
    for grid in (0, 5):  # full, and one that makes every block run many items
        G.set_launch(slab_in_lds=0, grid=grid, shots_per_wave=1)
        got = G.decode(s)
        _same(torch, got, ref)
    _same(torch, G.decode(s[:1].contiguous()), tuple(x[:1] for x in ref))
    _same(torch, G.decode(s, noalloc=True), ref)
    G.set_alpha([0.5, 0.7, 0.9])
    a = G.decode(s)
    G.set_launch(slab_in_lds=0, shots_per_wave=2)
    _same(torch, G.decode(s), a)
    torch.cuda.synchronize()
    check_valid(dem, P.unpack_bits(ref[0], dem.n), synd, ref[2].cpu().numpy())
    G.close()


def test_compact_ragged_with_general_segments(torch_cuda):
    """One ragged launch over compact graphs of both widths and a graph
    without compact data (short rows): each request as its own decode."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    pairs = []
    for i, key in enumerate(("circuit d=7", "columns of 8", "priors above 1/2")):
        dem, G = _graph(P, key, 20 + i)
        G.set_launch(slab_in_lds=0, shots_per_wave=1)
        pairs.append((G, torch.from_numpy(sample(dem, (70, 1, 33)[i], 30 + i).syndromes).to("cuda:0")))
    dem = phenomenological_dem(7, 7, 0.01, 0.01)
    G = P.Graph.from_dem(dem, permutations(dem.n, 8, 3), L=8, M=3, T_max=20)
    G.set_launch(slab_in_lds=0, shots_per_wave=1)
    pairs.append((G, torch.from_numpy(sample(dem, 90, 40).syndromes).to("cuda:0")))
    want = [G.decode(s) for G, s in pairs]
    rt = P.Runtime()
    for a, b in zip(rt.decode(pairs), want):
        _same(torch, a, b)
    ex = P.Exec(pairs)
    for _ in range(2):
        ex.launch()
        torch.cuda.synchronize()
        for a, b in zip(ex.outs, want):
            _same(torch, a, b)
    ex.close()
    rt.close()
    for G, _ in pairs:
        G.close()


def test_server_serves_what_only_the_general_body_fits(torch_cuda):
    """A pool that holds a request's general footprint but not its compact
    one: the request is admitted as before and decoded."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    dem, G = _graph(P, "circuit d=7", 50)
    G.set_launch(slab_in_lds=0, shots_per_wave=1)
    s = torch.from_numpy(sample(dem, 16, 51).syndromes).to("cuda:0")
    want = G.decode(s)
    torch.cuda.synchronize()
    # the general footprint: bisect the smallest budget that admits it
    lo, hi = 1 << 16, 1 << 30
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        srv = P.Server([G], slots=1, max_batch_shots=64, hbm_budget=mid)
        try:
            t, _ = srv.submit(0, s)
            srv.wait(t)
            hi = mid
        except P.VibeError:
            lo = mid
        srv.close()
    srv = P.Server([G], slots=1, max_batch_shots=64, hbm_budget=hi)
    t, got = srv.submit(0, s)
    srv.wait(t)
    torch.cuda.synchronize()
    _same(torch, got, want)
    assert srv.info()["peak_bytes"] <= hi
    srv.close()
    G.close()


@pytest.mark.parametrize("key", ["circuit d=7", "columns of 6", "columns of 8", "equal priors", "priors above 1/2"])
def test_compact_parallel_equals_general(torch_cuda, key):
    """The parallel schedule's one-pass body (a row's two least magnitudes)
    against the general one, which ragged launches run; posteriors of every
    iteration's last sweep against the general FP64 body within FP32's
    rounding (1e-4 of max(|L|, 1), where no decision is near a tie)."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    print(f"parallel, case {key}", flush=True)
    mk, L, M, T, _ = CASES[key]
    dem = mk()
    for L in (1, 3):
        perms = permutations(dem.n, L, 60)
        G = P.Graph.from_dem(dem, perms, L=L, M=1, T_max=T, schedule="parallel")
        synd = sample(dem, 203, 61).syndromes
        synd[3] = 0
        s = torch.from_numpy(synd).to("cuda:0")
        rt = P.Runtime()
        want = rt.decode([(G, s)])[0]
        _same(torch, G.decode(s), want)
        G.set_launch(slab_in_lds=0, grid=7)
        _same(torch, G.decode(s), want)
        G.set_launch(slab_in_lds=0)
        _same(torch, G.decode(s, noalloc=True), want)
        rt.close()
        G64 = P.Graph.from_dem(dem, perms, L=L, M=1, T_max=T, schedule="parallel", message_bits=64)
        _, p32, e32 = G.bp_ensemble(s[:40], T_run=3, stop=False)
        _, p64, e64 = G64.bp_ensemble(s[:40], T_run=3, stop=False)
        err = (p32.double() - p64).abs() / p64.abs().clamp(min=1.0)
        assert float(err.max()) <= 1e-4
        if not bool((p64.abs() < 1e-3).any()):
            assert torch.equal(e32, e64)
        torch.cuda.synchronize()
        G.close()
        G64.close()
