"""A server's pool sized for several batches by their smallest footprint holds
that many at once: the faster item body's larger footprint must not keep the
second batch waiting."""
import re

import pytest

from synth.dem import circuit_dem
from synth.sample import permutations, sample

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [2, 3])
def test_pool_of_several_footprints_runs_them_together(slots):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2508_15743_amd as P

    dem = circuit_dem(7, 7, 2e-3)
    G = P.Graph.from_dem(dem, permutations(dem.n, 16, 1), L=16, M=5, T_max=60)
    s = torch.from_numpy(sample(dem, 60, 2).syndromes).to("cuda:0")
    want = G.decode(s)
    torch.cuda.synchronize()
    tiny = P.Server([G], slots=1, max_batch_shots=60, hbm_budget=4096)
    with pytest.raises(P.VibeError) as e:
        tiny.submit(0, s)
    tiny.close()
    one = int(re.search(r"footprint \((\d+) bytes", str(e.value)).group(1))
    # 960 items reside with either body, so the compact one's larger slab makes
    # its footprint the larger.  The decode takes milliseconds, the submissions
    # far less.
    srv = P.Server([G], slots=slots, max_batch_requests=1, max_batch_shots=60, hbm_budget=slots * one)
    sent = [srv.submit(0, s) for _ in range(slots)]
    for t, _ in sent:
        srv.wait(t)
    torch.cuda.synchronize()
    info = srv.info()
    print(f"footprint {one}, {info}", flush=True)
    for _, got in sent:
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert info["batches"] == slots and info["peak_bytes"] >= slots * one
    srv.close()
    G.close()
