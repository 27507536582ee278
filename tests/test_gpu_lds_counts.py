"""GPU: out-degrees counted in LDS while a work-group walks several chunks of
tables, where every wave adds to the same members: each chunk's counters are
complete before they go out (key-sum ordered path, the two 64-member chunks of
M >= 11 and the wide tables below)."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [5, 10, 11, 12, 16])
def test_counts_of_two_runs_of_equal_rows(M, monkeypatch):
    import torch
    monkeypatch.setenv("NSGA3_PAIRS", "0")
    rng = np.random.Generator(np.random.PCG64(M))
    f = np.empty((3000, M), np.float32)
    f[:1500], f[1500:] = rng.random(M), 2.0
    f = f[rng.permutation(3000)]
    din, dout = oracle.dominance(f)[:2]
    ctx = nsga3.Context(0)
    refs = torch.eye(M, device="cuda") + 0.1
    for _ in range(3):
        res = nsga3.select(torch.from_numpy(f).cuda(), refs, 1500, ctx=ctx)
        assert np.array_equal(res.dom_in.cpu().numpy(), din)
        assert np.array_equal(res.dom_out.cpu().numpy(), dout)
