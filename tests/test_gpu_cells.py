"""GPU: populations that put many points into one cell of the spatial order
(identical rows, objectives that move together): the order inside wide cells
against the oracle, at the sizes where a cell becomes wide and where wide cells
meet inside a work-group, and no call slower than in the key-sum order."""
from __future__ import annotations

import time

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3

pytestmark = pytest.mark.gpu


def _objs(kind, N, M):
    rng = np.random.Generator(np.random.PCG64(N + M))
    f = rng.random((N, M))
    if kind == "same":
        f[:] = f[0]
    elif kind.startswith("run"):       # so many identical rows, the others anywhere
        f[: int(kind[3:])] = 0.5
    elif kind == "two":
        f = f[rng.integers(0, 2, N)]
    elif kind == "few":
        f = np.floor(4 * f)
    elif kind == "line":               # near one line, a quarter of the rows repeated
        f = rng.random((N, 1)) + 0.01 * f
        f[: N // 4] = f[rng.integers(0, N, N // 4)]
    return np.ascontiguousarray(f[rng.permutation(N)].astype(np.float32))


@pytest.mark.parametrize("N,M,kind", [
    (1025, 2, "same"), (3000, 3, "run128"), (3000, 3, "run129"), (3000, 3, "run1025"),
    (5000, 16, "same"), (4096, 3, "line"), (4097, 3, "same"),
    (2600, 2, "two"), (9001, 4, "two"), (20000, 3, "line"), (12000, 2, "few"), (30000, 10, "line"),
    (40000, 5, "run17000"),
])
def test_wide_cells_match_oracle(N, M, kind):
    import torch
    f = _objs(kind, N, M)
    res = nsga3.select(torch.from_numpy(f).cuda(), torch.eye(M, device="cuda") + 0.1, N // 2,
                       ctx=nsga3.Context(0))
    din, dout = oracle.dominance(f)[:2]
    assert res.info().status == 0
    assert np.array_equal(res.rank.cpu().numpy(), oracle.ranks(f)[0])
    assert np.array_equal(res.dom_in.cpu().numpy(), din)
    assert np.array_equal(res.dom_out.cpu().numpy(), dout)


@pytest.mark.parametrize("N,M,kind", [(200000, 5, "same"), (200000, 2, "same"), (200000, 5, "two"),
                                      (200000, 3, "few"), (50000, 3, "run25000"), (20000, 3, "same"),
                                      (200000, 10, "line")])
def test_wide_cells_cost_no_more_than_the_key_sum_order(N, M, kind, monkeypatch):
    import torch
    o, r = torch.from_numpy(_objs(kind, N, M)).cuda(), torch.eye(M, device="cuda") + 0.1
    best, out = {}, {}
    for pairs in ("1", "0"):
        monkeypatch.setenv("NSGA3_PAIRS", pairs)
        ctx = nsga3.Context(0)
        best[pairs] = 1e9
        for _ in range(4):
            torch.cuda.synchronize()
            t = time.perf_counter()
            out[pairs] = nsga3.select(o, r, N // 2, ctx=ctx)
            torch.cuda.synchronize()
            best[pairs] = min(best[pairs], time.perf_counter() - t)
        ctx.close()
    for k in ("rank", "dom_in", "dom_out", "selected"):
        assert torch.equal(getattr(out["1"], k), getattr(out["0"], k)), k
    assert best["1"] <= 1.1 * best["0"], best
