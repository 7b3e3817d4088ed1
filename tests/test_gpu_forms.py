"""Each form of K1 on inputs the other tests leave out: messages at the clamp
(the saturation mark), graphs that no compact form takes, layered graphs whose
posteriors exceed LDS."""
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
    return torch


def _random(m, n, lo, hi, seed):
    rng = np.random.default_rng(seed)
    h = np.zeros((m, n), np.uint8)
    for v in range(n):
        h[rng.choice(m, int(rng.integers(lo, hi + 1)), replace=False), v] = 1
    return dem_from_dense(h, np.exp(rng.uniform(np.log(1e-4), np.log(1e-2), n)), rng.integers(0, 2, (1, n)).astype(np.uint8))


def _same(torch, a, b):
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert torch.equal(a[2][:, DET], b[2][:, DET])


# graph, clamp: between the channel LLRs and what messages reach
SATURATING = {
    "circuit d=5": (lambda: circuit_dem(5, 5, 2e-3), 11.5),
    "circuit d=5, channel LLRs at the clamp": (lambda: circuit_dem(5, 5, 1e-3), 6.0),
    "phenomenological d=7": (lambda: phenomenological_dem(7, 7, 0.01, 0.01), 6.5),
}


@pytest.mark.parametrize("key", list(SATURATING))
def test_saturation_mark_of_the_compact_bodies(torch_cuda, key):
    """Serial: against several shots per wavefront; parallel: against a ragged
    round.  Both are the general body."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    mk, clamp = SATURATING[key]
    dem = mk()
    s = torch.from_numpy(sample(dem, 300, 6).syndromes).to("cuda:0")
    marks = []
    for schedule in ("serial", "parallel"):
        G = P.Graph.from_dem(dem, permutations(dem.n, 8, 5), L=8, M=3, T_max=20, clamp=clamp, schedule=schedule)
        if schedule == "serial":
            G.set_launch(slab_in_lds=0, shots_per_wave=2)
            want = G.decode(s)
            G.set_launch(slab_in_lds=0, shots_per_wave=1)
        else:
            rt = P.Runtime()
            want = rt.decode([(G, s)])[0]
            rt.close()
            G.set_launch(slab_in_lds=0)
        _same(torch, G.decode(s), want)
        marks.append(int((want[2][:, 0] & P.FLAG_SATURATED != 0).sum()))
        torch.cuda.synchronize()
        G.close()
    print(f"{key}: {marks} of 300 shots marked (serial, parallel)", flush=True)
    assert min(marks) > 0


def test_saturation_mark_of_layered_forms(torch_cuda):
    """A row of one check raises its column to alpha x clamp; columns 0 to 9
    are in no check.  Posteriors in LDS, in global memory (a ragged round) and
    in FP64, against the oracle."""
    import paper_2508_15743_amd as P
    from oracle import oracle as O

    torch = torch_cuda
    h = np.zeros((12, 38), np.uint8)
    for r in range(12):
        h[r, 10 + 2 * r:12 + 2 * r + (r % 3)] = 1
    h[5] = 0
    h[5, 37] = 1
    dem = dem_from_dense(h, np.full(38, 0.01), np.ones((1, 38), np.uint8))
    perms = permutations(12, 4, 5)
    synd = sample(dem, 40, 6).syndromes
    synd[:, 0] = 1
    s = torch.from_numpy(synd).to("cuda:0")
    kw = dict(L=4, M=1, T_max=3, alpha=1.25, schedule="layered")
    G, G64 = P.Graph.from_dem(dem, perms, **kw), P.Graph.from_dem(dem, perms, message_bits=64, **kw)
    rt = P.Runtime()
    forms = {"LDS": G.decode(s), "ragged": rt.decode([(G, s)])[0], "FP64": G64.decode(s), "FP64 ragged": rt.decode([(G64, s)])[0]}
    flags = {k: (o[2][:, 0] & P.FLAG_SATURATED).cpu().numpy() for k, o in forms.items()}
    ref = O.decode(O.OracleGraph(dem), perms, synd, L=4, M=1, T=3, alpha=1.25, schedule="layered")
    want = ref["saturated"] * P.FLAG_SATURATED
    print({k: int((f != 0).sum()) for k, f in flags.items()}, int((want != 0).sum()), flush=True)
    for k, f in flags.items():
        assert np.array_equal(f, want), k
    rt.close()
    G.close()
    G64.close()


def test_forms_of_the_general_body(torch_cuda):
    """Columns of 9 to 15 checks in FP32: every chunk on the general body, in
    its persistent and latency forms, decisions in LDS and in global memory,
    one, two and four shots per wavefront."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    dem = _random(120, 1500, 9, 15, 3)
    G = P.Graph.from_dem(dem, permutations(dem.n, 6, 5), L=6, M=2, T_max=8)
    assert G.info()["chunks_min"] >= 100
    s = torch.from_numpy(sample(dem, 700, 6).syndromes).to("cuda:0")
    G.set_launch(slab_in_lds=0, grid=512)  # fewer blocks than items
    want = G.decode(s)
    for kw in (dict(decisions_global=0), dict(decisions_global=1), dict(decisions_global=1, grid=300),
               dict(shots_per_wave=2), dict(shots_per_wave=4), dict(shots_per_wave=2, decisions_global=1)):
        G.set_launch(slab_in_lds=0, **kw)
        _same(torch, G.decode(s), want)
    G.set_launch(slab_in_lds=0)
    for a in (0, 1, 699):  # every item resides
        _same(torch, G.decode(s[a:a + 1].contiguous()), tuple(x[a:a + 1] for x in want))
    torch.cuda.synchronize()
    check_valid(dem, P.unpack_bits(want[0], dem.n), s.cpu().numpy(), want[2].cpu().numpy())
    G.close()


def test_layered_posteriors_beyond_lds(torch_cuda):
    """45000 columns: the posteriors stay in global memory.  One order and one
    iteration is check by check what the definition says."""
    import paper_2508_15743_amd as P

    torch = torch_cuda
    rng = np.random.default_rng(4)
    m, n = 400, 45000
    rows = [np.sort(rng.choice(n, 60, replace=False)) for _ in range(m)]
    h = np.zeros((m, n), np.uint8)
    for r, c in enumerate(rows):
        h[r, c] = 1
    dem = dem_from_dense(h, np.exp(rng.uniform(np.log(1e-4), np.log(1e-3), n)), rng.integers(0, 2, (1, n)).astype(np.uint8))
    order = permutations(m, 1, 5)
    G = P.Graph.from_dem(dem, order, L=1, M=1, T_max=1, schedule="layered")
    synd = sample(dem, 5, 6).syndromes
    _, post, _ = G.bp_ensemble(torch.from_numpy(synd).to("cuda:0"), T_run=1, stop=False)
    got = post.cpu().numpy().reshape(5, n)
    lam = np.log((1.0 - dem.priors) / dem.priors)
    for b in range(5):
        L = lam.copy()
        for r in order[0]:
            c = rows[r]
            mu = L[c]
            order_ = np.argsort(np.abs(mu))
            least = np.where(np.arange(len(c)) == order_[0], np.abs(mu[order_[1]]), np.abs(mu[order_[0]]))
            sign = np.where(mu < 0, -1.0, 1.0)
            L[c] = mu + 0.625 * least * sign * np.prod(sign) * (-1.0 if synd[b, r] else 1.0)
        # sums of at most a few FP32 terms of size 10
        np.testing.assert_allclose(got[b], L, rtol=0, atol=1e-4)
    G.close()
