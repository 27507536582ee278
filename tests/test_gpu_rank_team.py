"""GPU: the rank launch with fewer work-groups than it wants (others hold the
CUs), more, or a small number wanted (few CUs): the team that forms works
through every 64-point group, against the oracle.  N at one group a wave and
several, in LDS at once or in turns."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3
from tests.test_gpu_pairs import _objs

pytestmark = pytest.mark.gpu

_want = {}


def _oracle(kind, N, M):
    if (kind, N, M) not in _want:
        f = _objs(kind, N, M, N + M)
        _want[kind, N, M] = f, oracle.dominance(f)[:2], oracle.ranks(f)[0]
    return _want[kind, N, M]


@pytest.mark.parametrize("kind,N,M", [("quant", 1100, 2), ("sphere", 20001, 3), ("corr", 9000, 16),
                                      ("sphere", 33000, 5), ("quant", 66000, 3)])
@pytest.mark.parametrize("groups,started", [(0, 1), (0, 2), (0, 13), (0, 80), (1, 0), (3, 0), (5, 2)])
def test_any_team_ranks_every_point(kind, N, M, groups, started, monkeypatch):
    import torch
    monkeypatch.setenv("NSGA3_RANK_GROUPS", str(groups))
    monkeypatch.setenv("NSGA3_RANK_STARTED", str(started))
    f, (din, dout), rank = _oracle(kind, N, M)
    o, r = torch.from_numpy(f).cuda(), torch.eye(M, device="cuda") + 0.1
    ctx = nsga3.Context(0)
    for _ in range(2):
        res = nsga3.select(o, r, N // 2, ctx=ctx)
        assert res.info().status == 0
        assert np.array_equal(res.rank.cpu().numpy(), rank)
        assert np.array_equal(res.dom_in.cpu().numpy(), din)
        assert np.array_equal(res.dom_out.cpu().numpy(), dout)
    ctx.close()


def test_streams_of_both_paths_at_once():
    """Four contexts on four streams: above the spatial path's limit (cooperative
    peel), with fronts taken off first, one rank launch, one work-group."""
    import torch
    probs = [(_objs("sphere", n, m, n), m) for n, m in ((210000, 4), (120000, 5), (20000, 3), (900, 2))]
    refs = [torch.eye(m, device="cuda") + 0.1 for _, m in probs]
    objs = [torch.from_numpy(f).cuda() for f, _ in probs]
    ctx = [nsga3.Context(0) for _ in probs]
    want = [nsga3.select(o, r, len(o) // 2, ctx=c) for o, r, c in zip(objs, refs, ctx)]
    streams = [torch.cuda.Stream() for _ in probs]
    torch.cuda.synchronize()
    got = []
    for _ in range(4):
        for o, r, c, s in zip(objs, refs, ctx, streams):
            with torch.cuda.stream(s):
                got.append(nsga3.select(o, r, len(o) // 2, ctx=c))
    torch.cuda.synchronize()
    for q, g in enumerate(got):
        w = want[q % len(probs)]
        assert g.info().status == 0
        for k in ("rank", "dom_in", "dom_out", "selected"):
            assert torch.equal(getattr(g, k), getattr(w, k)), (q, k)


@pytest.mark.parametrize("kind,N,M", [("sphere", 120000, 5), ("quant", 66000, 3), ("sphere", 210000, 4),
                                      ("corr", 205000, 3)])
def test_counts_not_published_are_made_by_the_block_that_waits(kind, N, M, monkeypatch):
    """No look at an earlier block's count but the first (front copies of the spatial
    path, splits of the key-sum order)."""
    import torch
    o, r = torch.from_numpy(_objs(kind, N, M, N)).cuda(), torch.eye(M, device="cuda") + 0.1
    want = nsga3.select(o, r, N // 2, ctx=nsga3.Context(0))
    monkeypatch.setenv("NSGA3_LOOK_POLLS", "0")
    ctx = nsga3.Context(0)
    for _ in range(3):
        got = nsga3.select(o, r, N // 2, ctx=ctx)
        assert got.info() == want.info() and got.info().status == 0
        for k in ("rank", "dom_in", "dom_out", "selected"):
            assert torch.equal(getattr(got, k), getattr(want, k)), k
