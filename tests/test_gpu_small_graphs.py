"""K1 with one lane per shot (graphs of at most 64 checks, 64 columns and 160
edges, in batches of at least 6 columns^2 shots x members) against one
wavefront per shot and member.

Both form every message by the same operations in the same order, so all
outputs must be equal.  The batch is decoded whole and in pieces below the
size at which the other form runs.  Batches are no multiple of the wavefront;
graphs reach both cuts of the kernel (rows of up to 6 and 8 checks, columns of
up to 3 and 4), columns without checks and priors above 1/2 included, with
the correction limit at both ends.
"""
import numpy as np
import pytest

from synth.dem import code_capacity_dem, dem_from_dense
from synth.sample import permutations, sample

from parity_helpers import check_valid

pytestmark = pytest.mark.gpu

DET = [0, 1, 2, 4, 5, 6]  # stats fields that do not depend on timing


def _random(m, n, row, col, seed, high=False):
    rng = np.random.default_rng(seed)
    h = np.zeros((m, n), np.uint8)
    for v in range(n - 1):  # the last column is in no check
        free = np.flatnonzero(h.sum(1) < row)
        if len(free):
            h[rng.choice(free, size=min(int(rng.integers(1, col + 1)), len(free)), replace=False), v] = 1
    pri = np.exp(rng.uniform(np.log(1e-2), np.log(0.2), n))
    if high:
        pri[[0, n // 2, n - 1]] = [0.6, 0.7, 0.55]
    return dem_from_dense(h, pri, rng.integers(0, 2, (2, n)).astype(np.uint8))


CASES = {
    "code capacity d=3": (lambda: code_capacity_dem(3, 0.08), 5, 1, 7),
    "code capacity d=5": (lambda: code_capacity_dem(5, 0.05), 16, 5, 32),
    "code capacity d=9": (lambda: code_capacity_dem(9, 0.06), 24, 24, 12),
    "rows of 8, columns of 4": (lambda: _random(19, 57, 8, 4, 1), 20, 2, 12),
    "priors above 1/2": (lambda: _random(20, 64, 6, 3, 2, high=True), 24, 4, 9),
    "one check": (lambda: _random(1, 5, 3, 1, 3), 2, 1, 3),
}


@pytest.mark.parametrize("key", list(CASES))
def test_one_lane_per_shot_equals_one_wavefront(key):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_15743_amd as P

    print(f"case {key}", flush=True)
    mk, L, M, T = CASES[key]
    dem = mk()
    G = P.Graph.from_dem(dem, permutations(dem.n, L, 5), L=L, M=M, T_max=T, lsd_order=1)
    synd = sample(dem, 1000 + 37, 6).syndromes
    synd[70] = 0
    s = torch.from_numpy(np.ascontiguousarray(synd)).to("cuda:0")
    for alpha in (None, [0.5, 0.8, 1.1]):
        G.set_alpha(alpha)
        c, o, st = G.decode(s)
        parts = [G.decode(s[a:a + 13].contiguous()) for a in range(0, len(synd), 13)]
        pc, po, ps = (torch.cat([p[i] for p in parts]) for i in range(3))
        assert torch.equal(c, pc) and torch.equal(o, po) and torch.equal(st[:, DET], ps[:, DET])
        for other in (G.decode(s, noalloc=True), G.decode_packed(_pack(torch, s))):
            assert torch.equal(c, other[0]) and torch.equal(o, other[1]) and torch.equal(st[:, DET], other[2][:, DET])
    torch.cuda.synchronize()
    check_valid(dem, P.unpack_bits(c, dem.n), synd, st.cpu().numpy())
    G.close()


def _pack(torch, s):
    wide = torch.zeros((s.shape[0], 64), dtype=torch.int64, device=s.device)
    wide[:, :s.shape[1]] = s.to(torch.int64)
    return (wide << torch.arange(64, device=s.device)).sum(1, keepdim=True)
