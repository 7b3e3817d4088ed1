"""K1 with one lane per shot: lanes that take new shots, the correction limit,
and the saturation mark.

A wavefront has more shots than lanes here (20000 shots of 16 members on about
2000 wavefronts), so lanes take new ones at any iteration.  The slab in LDS
runs one wavefront per shot and member; every output that does not depend on
timing must be the same.
"""
import numpy as np
import pytest

from synth.dem import code_capacity_dem, dem_from_dense
from synth.sample import permutations, sample

pytestmark = pytest.mark.gpu

DET = [0, 1, 2, 4, 5, 6]  # stats fields that do not depend on timing


@pytest.fixture(scope="module")
def torch_cuda():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _random(m, n, row, col, seed):
    rng = np.random.default_rng(seed)
    h = np.zeros((m, n), np.uint8)
    for v in range(n - 1):  # the last column is in no check
        free = np.flatnonzero(h.sum(1) < row)
        if len(free):
            h[rng.choice(free, size=min(int(rng.integers(1, col + 1)), len(free)), replace=False), v] = 1
    return dem_from_dense(h, np.exp(rng.uniform(np.log(1e-2), np.log(0.2), n)), rng.integers(0, 2, (2, n)).astype(np.uint8))


# graph, L, M, T, shots, clamp
CASES = {
    "d=3, several shots a lane": (lambda: code_capacity_dem(3, 0.05), 16, 5, 32, 20000, 1e6),
    "d=5, one correction of 64": (lambda: code_capacity_dem(5, 0.01), 64, 1, 64, 5003, 1e6),
    "d=5, many at the limit": (lambda: code_capacity_dem(5, 0.12), 16, 16, 11, 20000, 1e6),
    "d=5, messages at the clamp": (lambda: code_capacity_dem(5, 0.08), 16, 5, 20, 9001, 4.0),
    "d=7, few wavefronts": (lambda: code_capacity_dem(7, 0.03), 4, 2, 16, 30001, 1e6),
    "rows of 8, columns of 4, clamp": (lambda: _random(18, 50, 8, 4, 1), 20, 2, 9, 9000, 5.0),
    "two checks": (lambda: _random(2, 6, 3, 2, 2), 3, 2, 5, 70000, 1e6),
}


@pytest.mark.parametrize("key", list(CASES))
def test_lanes_that_take_new_shots(torch_cuda, key):
    import paper_2508_15743_amd as P

    torch = torch_cuda
    print(f"case {key}", flush=True)
    mk, L, M, T, B, clamp = CASES[key]
    dem = mk()
    G = P.Graph.from_dem(dem, permutations(dem.n, L, 5), L=L, M=M, T_max=T, clamp=clamp)
    s = torch.from_numpy(sample(dem, B, 6).syndromes).to("cuda:0")
    G.set_launch(slab_in_lds=1)
    want = G.decode(s)
    G.set_launch(slab_in_lds=0)
    for _ in range(2):
        got = G.decode(s)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert torch.equal(got[2][:, DET], want[2][:, DET])
    if clamp < 100:  # VIBE_FLAG_SATURATED on some shots, not on all
        flags = want[2][:, 0]
        assert 0 < int((flags & P.FLAG_SATURATED != 0).sum()) < B
    torch.cuda.synchronize()
    G.close()


def test_a_set_grid_holds(torch_cuda):
    """Launch settings on the form with one lane per shot: a grid below the
    member count makes wavefronts run several members; a grid of one block
    takes longer than all of them."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    dem = code_capacity_dem(5, 0.05)
    G = P.Graph.from_dem(dem, permutations(dem.n, 16, 5), L=16, M=5, T_max=8)
    s = torch.from_numpy(sample(dem, 20000, 6).syndromes).to("cuda:0")
    want = G.decode(s)
    ms = {}
    for grid in (0, 33, 7, 1):
        G.set_launch(slab_in_lds=0, grid=grid)
        P.vibe_profile_enable(G.handle, True)
        got = G.decode(s)
        torch.cuda.synchronize()
        ms[grid] = P.vibe_profile_read(G.handle)["bp_ensemble"][0]
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
        assert torch.equal(got[2][:, DET], want[2][:, DET])
    print(f"BP ms by grid: {ms}", flush=True)
    assert ms[1] > 5 * ms[0]
    G.close()


def test_autotune_times_no_setting_that_changes_nothing(torch_cuda):
    """Where the batch runs one lane per shot, neither a smaller grid nor the
    decisions' place is a choice, so none is stored."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    dem = code_capacity_dem(5, 0.05)
    s = torch.from_numpy(sample(dem, 4000, 6).syndromes).to("cuda:0")
    for L in (9, 11, 13, 15):
        G = P.Graph.from_dem(dem, permutations(dem.n, L, 5), L=L, M=3, T_max=19)
        ch = G.autotune(s)
        print(f"{L} members: {ch}", flush=True)
        if ch["slab_in_lds"] == 0 and ch["shots_per_wave"] == 1:
            assert ch["grid"] == 0 and ch["decisions_global"] <= 0
        G.close()


def test_members_past_the_correction_limit_stop(torch_cuda):
    """With M = 1, members that do not converge must not run to the iteration
    limit on shots that another member decides early."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    dem = code_capacity_dem(5, 0.12)
    L, T = 64, 64
    G = P.Graph.from_dem(dem, permutations(dem.n, L, 5), L=L, M=1, T_max=T)
    s = torch.from_numpy(sample(dem, 2000, 6).syndromes).to("cuda:0")
    stats = G.decode(s)[2]
    t_conv = G.bp_ensemble(s, T_run=T)[0].view(2000, L)
    alone = torch.where(t_conv > 0, t_conv, torch.full_like(t_conv, T)).sum(1)
    some = (t_conv > 0).any(1)
    ran, free = int(stats[some, 7].sum()), int(alone[some].sum())
    print(f"iterations run {ran}, without the limit {free}", flush=True)
    assert ran <= 0.75 * free
    G.close()
