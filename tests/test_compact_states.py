"""The compact form of the suffix states (csrc/bp_compact.h) against the
states themselves, on the CPU.

The general item body keeps, per edge, the least magnitude and the sign
parity of its row's later messages.  The compact body keeps one state per
row and, per chunk, the messages' signs, a mask of the records (messages
smaller than all later ones of their row) and the least later magnitude of
each record; a chunk with more records than fit keeps its states.  Stepping
the row states over the chunks must give every edge its suffix state, for
any messages: ties, zeros, negative ones, rows that only rise (every edge a
record) or only fall, and empty rows.
"""
import numpy as np
import pytest

FIT = 12  # record values per chunk


def direct(chunks, msgs, m, top):
    low, par = np.full(m, top), np.zeros(m, bool)
    out = [None] * len(chunks)
    for k in range(len(chunks) - 1, -1, -1):
        rows, x = chunks[k], msgs[k]
        out[k] = (low[rows].copy(), par[rows].copy())
        low[rows] = np.minimum(low[rows], np.abs(x))
        par[rows] ^= x < 0
    return out


def compact(chunks, msgs, m, top):
    low, par = np.full(m, top), np.zeros(m, bool)
    recs = [None] * len(chunks)
    for k in range(len(chunks) - 1, -1, -1):
        rows, x = chunks[k], msgs[k]
        rec = np.abs(x) < low[rows]
        kept = (low[rows].copy(), par[rows].copy()) if rec.sum() > FIT else None
        recs[k] = (x < 0, rec, low[rows][rec], kept)
        low[rows] = np.minimum(low[rows], np.abs(x))
        par[rows] ^= x < 0
    out = []
    for rows, (neg, rec, vals, kept) in zip(chunks, recs):
        if kept is None:
            mag, sgn = low[rows].copy(), par[rows] ^ neg
            mag[rec] = vals
        else:
            mag, sgn = kept
        out.append((mag, sgn))
        low[rows], par[rows] = mag, sgn
    return out


@pytest.mark.parametrize("kind", ["random", "ties", "rising", "falling", "zeros"])
@pytest.mark.parametrize("m,width", [(3, 3), (40, 24), (540, 64), (70, 64)])
def test_records_give_every_suffix_state(kind, m, width):
    rng = np.random.default_rng(m * 7 + width)
    n = 60
    chunks = [np.sort(rng.choice(m - 1 if m > 3 else m, size=min(width, m - 1), replace=False)) for _ in range(n)]
    msgs = []
    for k, rows in enumerate(chunks):
        x = rng.normal(size=len(rows))
        if kind == "ties":
            x = rng.choice([-2.0, -1.0, 1.0, 2.0], size=len(rows))
        elif kind == "rising":
            x = np.sign(x) * (k + 1.0)
        elif kind == "falling":
            x = np.sign(x) * (n - k + 0.0)
        elif kind == "zeros":
            x = np.where(rng.random(len(rows)) < 0.3, 0.0, x)
        msgs.append(x)
    for (a, b), (c, d) in zip(direct(chunks, msgs, m, 1e6), compact(chunks, msgs, m, 1e6)):
        assert np.array_equal(a, c) and np.array_equal(b, d)
