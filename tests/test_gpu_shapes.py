"""GPU: populations whose first fronts are small (uniform, normal, objectives that
move together in part).  No call slower than in the key-sum order, and the pairs
whose dominator masks are not stored against the oracle."""
from __future__ import annotations

import time

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3

pytestmark = pytest.mark.gpu


def _objs(kind, N, M):
    rng = np.random.Generator(np.random.PCG64(N + M))
    if kind == "normal":
        f = rng.standard_normal((N, M))
    elif kind == "cube":
        f = rng.random((N, M))
    else:      # a common part, and so much of their own
        f = rng.random((N, 1)) + float(kind) * rng.random((N, M))
    return np.ascontiguousarray(f.astype(np.float32))


@pytest.mark.parametrize("N,M,kind", [(200000, 3, "cube"), (200000, 5, "cube"), (50000, 5, "cube"),
                                      (200000, 4, "normal"), (200000, 5, "0.2"), (200000, 5, "1.0"),
                                      (100000, 8, "1.0"), (33000, 4, "0.5"), (60000, 16, "0.3"),
                                      (34000, 16, "0.5"), (1024, 16, "cube"), (765, 13, "normal"),
                                      (1000, 5, "cube"), (600, 8, "normal"), (300, 10, "cube")])
@pytest.mark.parametrize("counts", [True, False])
def test_no_slower_than_the_key_sum_order(N, M, kind, counts, monkeypatch):
    import torch
    o, r = torch.from_numpy(_objs(kind, N, M)).cuda(), torch.eye(M, device="cuda") + 0.1
    best, out = {}, {}
    for pairs in ("1", "0"):
        monkeypatch.setenv("NSGA3_PAIRS", pairs)
        ctx = nsga3.Context(0)
        best[pairs] = 1e9
        for _ in range(4 if N > 5000 else 40):
            torch.cuda.synchronize()
            t = time.perf_counter()
            out[pairs] = nsga3.select(o, r, N // 2, ctx=ctx, want_counts=counts)
            torch.cuda.synchronize()
            best[pairs] = min(best[pairs], time.perf_counter() - t)
        ctx.close()
    for k in ("rank", "selected") + (("dom_in", "dom_out") if counts else ()):
        assert torch.equal(getattr(out["1"], k), getattr(out["0"], k)), k
    assert best["1"] <= 1.05 * best["0"], best


@pytest.mark.parametrize("units", [0, 64, 6400])
@pytest.mark.parametrize("N,M,kind", [(300, 2, "cube"), (5000, 3, "normal"), (9000, 16, "1.0"),
                                      (20001, 5, "cube"), (40000, 4, "0.5"), (70000, 3, "cube")])
def test_pairs_without_stored_masks(N, M, kind, units, monkeypatch):
    """None of the masks stored, one a counter, or a share of them."""
    import torch
    monkeypatch.setenv("NSGA3_MASK_UNITS", str(units))
    f = _objs(kind, N, M)
    f[: N // 8] = f[N // 2: N // 2 + N // 8]     # (identical rows do not dominate each other)
    ctx = nsga3.Context(0)
    res = nsga3.select(torch.from_numpy(f).cuda(), torch.eye(M, device="cuda") + 0.1, N // 2, ctx=ctx)
    assert res.info().status == 0
    assert np.array_equal(res.rank.cpu().numpy(), oracle.ranks(f)[0])
    ctx.close()


@pytest.mark.parametrize("N", [35000, 70000])
@pytest.mark.parametrize("layers", [0, 1, 2, 3, 4, 5, 6])
def test_fronts_taken_off(N, layers):
    """So many large fronts before the small ones of a uniform rest: the fronts
    that are taken off first end after each of them."""
    import torch
    rng = np.random.Generator(np.random.PCG64(N + layers))
    f = 3.0 + rng.random((N, 2))
    n = N // 8
    for j in range(layers):
        x = rng.random(n)
        f[j * n:(j + 1) * n] = np.stack([x, 1.0 + 0.2 * j - x], 1)
    f = np.ascontiguousarray(f[rng.permutation(N)].astype(np.float32))
    res = nsga3.select(torch.from_numpy(f).cuda(), torch.eye(2, device="cuda") + 0.1, N // 2,
                       ctx=nsga3.Context(0))
    rank = oracle.ranks(f)[0]
    l = int(np.sort(rank)[N // 2 - 1])
    i = res.info()
    assert np.array_equal(res.rank.cpu().numpy(), rank)
    assert (i.status, i.num_fronts, i.last_front, i.last_front_size) == (
        0, int(rank.max()) + 1, l, int((rank == l).sum()))


@pytest.mark.parametrize("N,M", [(512, 2), (513, 2), (341, 3), (342, 3), (204, 5), (205, 5), (64, 16),
                                 (65, 16), (1024, 16), (2, 16), (1, 2)])
def test_small_orders(N, M):
    """By one work-group up to N x M = 1024 keys, by cells above."""
    import torch
    f = _objs("normal", N, M)
    f[: N // 3] = f[N // 2: N // 2 + N // 3]
    res = nsga3.select(torch.from_numpy(f).cuda(), torch.eye(M, device="cuda") + 0.1, (N + 1) // 2,
                       ctx=nsga3.Context(0))
    din, dout = oracle.dominance(f)[:2]
    assert res.info().status == 0
    assert np.array_equal(res.rank.cpu().numpy(), oracle.ranks(f)[0])
    assert np.array_equal(res.dom_in.cpu().numpy(), din)
    assert np.array_equal(res.dom_out.cpu().numpy(), dout)


@pytest.mark.parametrize("N,M,H", [(4096, 3, 1), (4097, 2, 511), (16384, 3, 512), (16385, 5, 513),
                                   (32769, 3, 255), (32769, 4, 256), (65536, 2, 700), (65537, 3, 5000),
                                   (40000, 10, 4097), (70000, 16, 300)])
def test_association_lanes(N, M, H):
    """Where another number of lanes shares a point, and references beyond one
    staged chunk: niches and distances against float64 over all references."""
    import torch
    from tests.gpu_helpers import compare_full, gpu_select
    rng = np.random.Generator(np.random.PCG64(N + H))
    u = np.abs(rng.standard_normal((N, M)))
    f = (u / np.linalg.norm(u, axis=1, keepdims=True) * (1 + 0.02 * rng.random((N, 1)))).astype(np.float32)
    refs = (rng.random((H, M)) + 1e-3).astype(np.float32)
    assert torch.cuda.is_available()
    rep = compare_full(f, refs, N // 2, gpu_select(f, refs, N // 2))
    rep.pop("near_ties")
    assert not any(rep.values()), rep
