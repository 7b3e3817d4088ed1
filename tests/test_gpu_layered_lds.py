"""The layered sweep with the posteriors in LDS against the one with them in
global memory (which ragged launches run): the same values in every message,
so all outputs are equal bit for bit, in FP32 and FP64.  Rows of one edge,
rows of more than 256 edges (which keep the global form), an empty
check, columns without checks, row counts around a block of 64 checks, ties
(equal priors) and a small clamp, at which messages saturate and row minima
tie.
"""
import numpy as np
import pytest

from synth.dem import circuit_dem, code_capacity_dem, dem_from_dense
from synth.sample import permutations, sample

pytestmark = pytest.mark.gpu

DET = [0, 1, 2, 4, 5, 6]  # stats fields that do not depend on timing


def _rows(m, n, seed, long=0, equal=False):
    rng = np.random.default_rng(seed)
    h = (rng.random((m, n)) < 3.0 / m).astype(np.uint8)
    h[:, 3] = 0  # a column in no check
    if m > 4:
        h[2] = 0  # an empty check
        h[1] = 0
        h[1, 7] = 1  # a row of one edge
    if long:
        h[0, :long] = 1
        h[0, 3] = 0
    for v in np.flatnonzero(h.sum(0) > 15):
        h[rng.permutation(np.flatnonzero(h[:, v]))[15:], v] = 0
    pri = np.full(n, 0.01) if equal else np.exp(rng.uniform(np.log(1e-3), np.log(0.05), n))
    return dem_from_dense(h, pri, rng.integers(0, 2, (1, n)).astype(np.uint8))


CASES = {
    "code capacity": (lambda: code_capacity_dem(5, 0.05), 1e6),
    "circuit d=5": (lambda: circuit_dem(5, 5, 2e-3), 1e6),
    "circuit d=7, a block of wavefronts": (lambda: circuit_dem(7, 7, 2e-3), 1e6),
    "63 checks": (lambda: _rows(63, 400, 1), 1e6),
    "64 checks, equal priors": (lambda: _rows(64, 500, 2, equal=True), 1e6),
    "65 checks, a row of 300": (lambda: _rows(65, 401, 3, long=300), 1e6),
    "65 checks, a row of 250": (lambda: _rows(65, 401, 5, long=250), 1e6),
    "129 checks, a row of 120": (lambda: _rows(129, 300, 6, long=120), 1e6),
    "small clamp": (lambda: _rows(130, 700, 4), 3.0),
}


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("key", list(CASES))
def test_layered_lds_equals_global(key, bits):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_15743_amd as P

    print(f"case {key}, {bits} bits", flush=True)
    mk, clamp = CASES[key]
    dem = mk()
    L, M, T = 5, 2, 9
    G = P.Graph.from_dem(dem, permutations(dem.m, L, 70), L=L, M=M, T_max=T, schedule="layered", clamp=clamp,
                         message_bits=bits)
    synd = sample(dem, 90, 71).syndromes
    synd[1] = 0
    s = torch.from_numpy(np.ascontiguousarray(synd)).to("cuda:0")
    rt = P.Runtime()
    for alpha in (None, [0.4, 0.9]):
        G.set_alpha(alpha)
        want = rt.decode([(G, s)])[0]
        for got in (G.decode(s), G.decode(s, noalloc=True), G.decode(s, plain=True)):
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
            assert torch.equal(got[2][:, DET], want[2][:, DET])
    torch.cuda.synchronize()
    rt.close()
    G.close()
