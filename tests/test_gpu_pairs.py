"""GPU: the spatially ordered dominance path at the sizes where it can go wrong
(64-point groups, 128-point blocks, one rank work-group / several, the first
fronts taken off), and the key-sum ordered path that larger problems and capped
workspaces take, both against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3
import workloads

pytestmark = pytest.mark.gpu


def _objs(kind, N, M, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    if kind == "sphere":
        f = workloads.sphere_shell(rng, N, M, lambda r, n: r.exponential(0.25, n), 0.2)
    elif kind == "quant":
        f = np.round(workloads.sphere_shell(rng, N, M, lambda r, n: r.uniform(0, 0.5, n), 0.2) * 64) / 64
    elif kind == "corr":       # near-chains: most pairs of blocks keep masks
        f = rng.random((N, 1)) + 0.02 * rng.random((N, M))
    elif kind == "same":       # runs of identical rows longer than a work-group
        f = rng.random((N, M))
        f[: N // 2] = f[0]
        f[N // 2: N // 2 + 1500] = 2.0
    else:                      # signs and wide ranges
        f = rng.standard_normal((N, M)) * np.exp(rng.uniform(-20, 20, (N, M)))
    return np.ascontiguousarray(f[rng.permutation(N)].astype(np.float32))


def _check(objs, monkeypatch=None, pairs=True):
    import torch
    N, M = objs.shape
    if not pairs:
        monkeypatch.setenv("NSGA3_PAIRS", "0")
    refs = np.eye(M, dtype=np.float32) + 0.1
    ctx = nsga3.Context(0)
    o, r = torch.from_numpy(objs).cuda(), torch.from_numpy(refs.astype(np.float32)).cuda()
    res = nsga3.select(o, r, max(1, N // 2), ctx=ctx)
    only = nsga3.select(o, r, max(1, N // 2), ctx=ctx, want_counts=False)
    info = res.info()
    assert info.status == 0, info
    din, dout = oracle.dominance(objs)[:2]
    rank = oracle.ranks(objs)[0]
    assert np.array_equal(res.dom_in.cpu().numpy(), din)
    assert np.array_equal(res.dom_out.cpu().numpy(), dout)
    assert np.array_equal(res.rank.cpu().numpy(), rank)
    assert np.array_equal(only.rank.cpu().numpy(), rank)
    assert np.array_equal(only.selected.cpu().numpy(), res.selected.cpu().numpy())
    l = int(np.sort(rank)[max(1, N // 2) - 1])
    assert (info.num_fronts, info.last_front) == (int(rank.max()) + 1, l)
    assert info.last_front_size == int((rank == l).sum())


@pytest.mark.parametrize("N,M,kind", [
    (1, 2, "sphere"), (2, 16, "sphere"), (63, 3, "quant"), (65, 4, "wide"), (128, 2, "corr"),
    (129, 7, "sphere"), (511, 5, "quant"), (1024, 3, "sphere"), (1025, 3, "same"),
    (4096, 2, "quant"), (4097, 6, "wide"), (8321, 16, "sphere"), (12000, 12, "quant"),
    (20001, 3, "corr"), (32768, 4, "quant"), (32769, 5, "sphere"), (33000, 3, "corr"),
    (40000, 2, "same"), (65600, 3, "quant"), (70001, 9, "sphere"), (90000, 3, "corr"),
])
def test_ranks_and_degrees_match_oracle(N, M, kind):
    _check(_objs(kind, N, M, 17 * N + M))


@pytest.mark.parametrize("N,M,kind", [(300, 3, "quant"), (5000, 2, "quant"), (9000, 5, "sphere"),
                                      (3000, 12, "same")])
def test_key_sum_order_matches_oracle(N, M, kind, monkeypatch):
    _check(_objs(kind, N, M, 3 * N + M), monkeypatch, pairs=False)


def test_four_streams_at_once():
    """Contexts on four streams, each with rank launches that wait for their own
    work-groups, beside each other."""
    import torch
    probs = [(_objs("sphere", n, m, n), m) for n, m in ((90000, 5), (70000, 4), (30000, 3), (8000, 2))]
    refs = [torch.eye(m, device="cuda") + 0.1 for _, m in probs]
    objs = [torch.from_numpy(f).cuda() for f, _ in probs]
    ctx = [nsga3.Context(0) for _ in probs]
    want = [nsga3.select(o, r, len(o) // 2, ctx=c).rank.clone() for o, r, c in zip(objs, refs, ctx)]
    streams = [torch.cuda.Stream() for _ in probs]
    torch.cuda.synchronize()
    got = []
    for _ in range(5):
        for o, r, c, s in zip(objs, refs, ctx, streams):
            with torch.cuda.stream(s):
                got.append(nsga3.select(o, r, len(o) // 2, ctx=c))
    torch.cuda.synchronize()
    for q, g in enumerate(got):
        assert g.info().status == 0 and torch.equal(g.rank, want[q % len(probs)])
