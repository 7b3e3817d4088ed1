"""Calls that must not take longer than what they took on the general item
body: each is timed against a call on the same graph that runs that body.
The bounds leave room for what the two bodies differ by where both reside
alike; the faults they guard against were larger."""
import time

import numpy as np
import pytest

from synth.dem import circuit_dem, dem_from_dense
from synth.sample import permutations, sample

pytestmark = pytest.mark.gpu

DET = [0, 1, 2, 4, 5, 6]  # stats fields that do not depend on timing


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _random(m, n, lo, hi, seed):
    rng = np.random.default_rng(seed)
    h = np.zeros((m, n), np.uint8)
    for v in range(n):
        h[rng.choice(m, int(rng.integers(lo, hi + 1)), replace=False), v] = 1
    return dem_from_dense(h, np.exp(rng.uniform(np.log(1e-4), np.log(1e-2), n)), rng.integers(0, 2, (1, n)).astype(np.uint8))


def _ms(torch, call, reps=5):
    out = call()
    torch.cuda.synchronize()
    best = 1e9
    for _ in range(reps):
        t = time.perf_counter()
        out = call()
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
    return best * 1e3, out


def test_ragged_round_of_mostly_general_work(torch_cuda):
    """A few shots of a graph with compact data beside many of one without
    (columns of up to 15 checks): no longer than the two apart."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    pairs = []
    for dem, B in ((_random(200, 4000, 8, 15, 2), 1200), (circuit_dem(3, 3, 1e-3), 10)):
        G = P.Graph.from_dem(dem, permutations(dem.n, 16, 1), L=16, M=5, T_max=12)
        pairs.append((G, torch.from_numpy(sample(dem, B, 3).syndromes).to("cuda:0")))
    rt = P.Runtime()
    apart, want = _ms(torch, lambda: [rt.decode([p])[0] for p in pairs], 3)
    ms, got = _ms(torch, lambda: rt.decode(pairs), 3)
    print(f"one round {ms:.2f} ms, two calls {apart:.2f} ms", flush=True)
    for a, b in zip(got, want):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2][:, DET], b[2][:, DET])
    assert ms <= 1.06 * apart
    # more compact work than that: the compact launch runs the other's items too
    few = [(pairs[0][0], pairs[0][1][:7].contiguous()), (pairs[1][0], pairs[1][1].repeat(300, 1))]
    for a, b in zip(rt.decode(few), [rt.decode([p])[0] for p in few]):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2][:, DET], b[2][:, DET])
    rt.close()
    for G, _ in pairs:
        G.close()


def test_thousands_of_checks_with_short_rows(torch_cuda):
    """The compact bodies' row states let few wavefronts reside on 3000 checks;
    a ragged round on the parallel schedule runs the general body."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    dem = _random(3000, 3000, 2, 3, 4)
    G = P.Graph.from_dem(dem, permutations(dem.n, 8, 1), L=8, M=8, T_max=20, schedule="parallel")
    s = torch.from_numpy(sample(dem, 3000, 2).syndromes).to("cuda:0")
    rt = P.Runtime()
    general, want = _ms(torch, lambda: rt.decode([(G, s)])[0])
    ms, got = _ms(torch, lambda: G.decode(s))
    print(f"decode {ms:.2f} ms, general body {general:.2f} ms", flush=True)
    assert torch.equal(got[0], want[0]) and torch.equal(got[2][:, DET], want[2][:, DET])
    assert ms <= 1.3 * general
    # few items reside in any case
    few = torch.equal(G.decode(s[:40].contiguous())[0], want[0][:40])
    assert few
    rt.close()
    G.close()


def test_members_are_built_side_by_side(torch_cuda):
    """Creating a graph of 32 members takes less than half of 32 graphs of one
    member (one after the other: three quarters)."""
    import paper_2508_15743_amd as P

    dem = circuit_dem(5, 5, 1e-3)

    def create(L):
        perms, best = permutations(dem.n, L, 1), 1e9
        for _ in range(5):
            t = time.perf_counter()
            G = P.Graph.from_dem(dem, perms, L=L, M=1, T_max=20)
            best = min(best, time.perf_counter() - t)
            G.close()
        return best * 1e3

    one, all_ = create(1), create(32)
    print(f"one member {one:.2f} ms, 32 members {all_:.2f} ms", flush=True)
    assert all_ <= 16 * one
