"""Reads of K1's compact body past a member's last chunk.

The compact body runs a member's chunks in groups of four, an even number of
groups: up to seven chunks past the last one have no record in the member's
schedule.  The resource of those records (osch) spans exactly the member's
chunks, and the bounds check of a raw buffer access covers the lane offset,
not the scalar one.  So every load from it has to carry the chunk in the lane
offset; the last member's padding would else be read past the allocation.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_15743_amd", "csrc")


def _calls(text, name):
    """Argument lists of the calls of `name`, split at top-level commas."""
    for m in re.finditer(re.escape(name) + r"(?:<[^>]*>)?\(", text):
        depth, args, cur = 1, [], ""
        for ch in text[m.end():]:
            depth += (ch == "(") - (ch == ")")
            if depth == 0:
                break
            if ch == "," and depth == 1:
                args.append(cur.strip())
                cur = ""
            else:
                cur += ch
        yield args + [cur.strip()]


def test_chunk_records_are_addressed_by_lane_offsets():
    text = open(os.path.join(CSRC, "bp_compact.h")).read()
    loads = [a for n in ("bload", "bload4") for a in _calls(text, n) if a[0] == "x.osch"]
    assert len(loads) >= 4
    for a in loads:
        assert a[2] == "0", f"scalar offset {a[2]} is outside the bounds check"


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1025, 1290, 1466])
def test_padding_chunks_of_the_last_member(n):
    """Members whose chunk counts leave one to seven chunks of padding, with
    posteriors (which read the columns' indices in every chunk): decode and
    ensemble against the general body and its FP64 form."""
    import numpy as np
    import torch

    import paper_2508_15743_amd as P
    from synth.dem import dem_from_dense
    from synth.sample import permutations, sample

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(n)
    h = np.zeros((90, n), np.uint8)
    for v in range(n):
        h[rng.choice(90, size=int(rng.integers(1, 5)), replace=False), v] = 1
    dem = dem_from_dense(h, np.exp(rng.uniform(np.log(1e-4), np.log(1e-2), n)), rng.integers(0, 2, (1, n)).astype(np.uint8))
    perms = permutations(n, 3, n)
    G = P.Graph.from_dem(dem, perms, L=3, M=3, T_max=6)
    G64 = P.Graph.from_dem(dem, perms, L=3, M=3, T_max=6, message_bits=64)
    i = G.info()
    print(f"n = {n}: {i['chunks_min']} to {i['chunks_max']} chunks", flush=True)
    assert i["chunks_min"] >= 16 and any(c % 8 for c in range(i["chunks_min"], i["chunks_max"] + 1))
    s = torch.from_numpy(sample(dem, 65, 3).syndromes).to("cuda:0")
    _, p32, _ = G.bp_ensemble(s, T_run=2, stop=False)
    _, p64, _ = G64.bp_ensemble(s, T_run=2, stop=False)
    # two iterations of sums of at most five FP32 terms
    assert float(((p32.double() - p64).abs() / p64.abs().clamp(min=1.0)).max()) <= 1e-4
    got = G.decode(s)
    G.set_launch(slab_in_lds=0, shots_per_wave=2)  # the general body
    want = G.decode(s)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    torch.cuda.synchronize()
    G.close()
    G64.close()
