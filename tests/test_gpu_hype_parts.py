"""GPU: HypE selection where its kernels branch (one part of the samples or
several, the last part ragged; few or many members of the last front; equal
estimates across the cut; both dominance paths below it), against the oracle
and, for the choice itself, against the library's own estimates: the last
front's members in descending order, the lower index first."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3
import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,s,n,kind", [
    (1, 2, 1, 1, "sphere"), (300, 3, 511, 150, "sphere"), (300, 3, 513, 299, "front"),
    (1000, 2, 4096, 500, "sphere"), (1000, 5, 4097, 500, "front"), (5000, 3, 9001, 2500, "same"),
    (2000, 4, 1030, 1999, "same"), (33000, 3, 700, 16000, "sphere"),
])
@pytest.mark.parametrize("pairs", ["1", "0"])
def test_hype_branches(N, M, s, n, kind, pairs, monkeypatch):
    import torch
    monkeypatch.setenv("NSGA3_PAIRS", pairs)
    rng = np.random.Generator(np.random.PCG64(N + s))
    f = workloads.sphere_shell(rng, N, M, lambda r, c: r.uniform(0, 0.5, c), 0.2)
    if kind != "sphere":
        f /= np.linalg.norm(f, axis=1, keepdims=True)     # one front
    if kind == "same":
        f = f[rng.integers(0, max(1, N // 50), N)]        # equal estimates by the dozen
    f = f.astype(np.float32)
    vref = (f.max(0) * 1.1 + 0.01).astype(np.float32)
    U = rng.random((s, M)).astype(np.float32)
    r = nsga3.hype_select(torch.from_numpy(f).cuda(), torch.from_numpy(vref).cuda(),
                          torch.from_numpy(U).cuda(), n, ctx=nsga3.Context(0))
    d, rank = r.d.cpu().numpy(), r.rank.cpu().numpy()
    o = oracle.hype_select(f, vref, U, n)
    assert r.info().status == 0 and np.array_equal(rank, o.rank)
    np.testing.assert_allclose(d, o.d, rtol=1e-10, atol=1e-300)
    l = o.last_front
    last = np.nonzero(rank == l)[0]
    take = last[np.argsort(-d[last], kind="stable")][: n - int((rank < l).sum())]
    want = np.sort(np.concatenate([np.nonzero(rank < l)[0], take]))
    assert np.array_equal(r.selected.cpu().numpy(), want)
