"""GPU: the key-sum ordered path, which problems above 204,800 points and capped
contexts take, at the sizes where it matters: whole selections against the
oracle, calls that size their launches by the previous call's levels, and both
sides of the spatially ordered path's limit."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_2503_20286_amd as nsga3
import workloads
from tests.gpu_helpers import compare_full, gpu_select
from tests.test_gpu_parity import _oracle_full, _zero
from tests.test_gpu_pairs import _objs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    nsga3.load()


@pytest.mark.parametrize("name", ["large", "many"])
def test_full_size(name, monkeypatch):
    monkeypatch.setenv("NSGA3_PAIRS", "0")
    w, s = _oracle_full(name)
    ctx = nsga3.Context(0)
    ctx.reserve(w.N, w.M, w.H)
    for _ in range(3):       # the second and third follow the first one's level sizes
        _zero(compare_full(w.objs, w.refs, w.K, gpu_select(w.objs, w.refs, w.K, ctx=ctx), s=s))
    ctx.close()


def test_calls_follow_the_previous_level_profile(monkeypatch):
    monkeypatch.setenv("NSGA3_PAIRS", "0")
    cases = {"ties": workloads.make("ties", N=8000, seed=41),
             "large": workloads.make("large", N=6000, seed=42),
             "small": workloads.make("small", N=200, seed=43)}
    want = {k: oracle.select(w.objs, w.refs, w.K, with_counts=True) for k, w in cases.items()}
    ctx = nsga3.Context(0)
    for name in ("ties", "ties", "ties", "large", "ties", "large", "large", "small", "ties"):
        w = cases[name]
        _zero(compare_full(w.objs, w.refs, w.K, gpu_select(w.objs, w.refs, w.K, ctx=ctx), s=want[name]))
    ctx.close()


@pytest.mark.parametrize("N", [204800, 204801])
@pytest.mark.parametrize("M,kind", [(3, "quant"), (6, "wide")])
def test_both_sides_of_the_limit(N, M, kind, monkeypatch):
    import torch
    o = torch.from_numpy(_objs(kind, N, M, N + M)).cuda()
    r = torch.eye(M, device="cuda") + 0.1
    got = nsga3.select(o, r, N // 2, ctx=nsga3.Context(0))
    monkeypatch.setenv("NSGA3_PAIRS", "0")
    want = nsga3.select(o, r, N // 2, ctx=nsga3.Context(0))
    for k in ("rank", "dom_in", "dom_out", "niche", "dist", "selected"):
        assert torch.equal(getattr(got, k), getattr(want, k)), k
    assert got.info() == want.info() and got.info().status == 0


def test_hype_of_both_paths_at_size(monkeypatch):
    import torch
    o = torch.from_numpy(_objs("sphere", 100000, 4, 5)).cuda()
    U = torch.rand((2000, 4), device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    v = (o.max(0).values * 1.1).contiguous()
    got = nsga3.hype_select(o, v, U, 50000, ctx=nsga3.Context(0))
    monkeypatch.setenv("NSGA3_PAIRS", "0")
    want = nsga3.hype_select(o, v, U, 50000, ctx=nsga3.Context(0))
    assert got.info().status == 0
    for k in ("rank", "d", "selected"):
        assert torch.equal(getattr(got, k), getattr(want, k)), k


@pytest.mark.parametrize("N,kind", [(8191, "same"), (8192, "same"), (8193, "one"), (65537, "one"),
                                    (204800, "one"), (204801, "one"), (204801, "same")])
def test_hype_cut_of_long_last_fronts(N, kind):
    """The last front's members with the largest estimates, the lower index first,
    by digits and above the limit by a sort."""
    import torch
    rng = np.random.Generator(np.random.PCG64(N))
    f = np.abs(rng.standard_normal((N, 3)))
    f /= np.linalg.norm(f, axis=1, keepdims=True)
    if kind == "same":
        f = f[rng.integers(0, 40, N)]
    o = torch.from_numpy(f.astype(np.float32)).cuda()
    U = torch.rand((600, 3), device="cuda", generator=torch.Generator("cuda").manual_seed(N))
    v = (o.max(0).values * 1.1).contiguous()
    n = N // 3
    r = nsga3.hype_select(o, v, U, n, ctx=nsga3.Context(0))
    d, rank, l = r.d.cpu().numpy(), r.rank.cpu().numpy(), r.info().last_front
    last = np.nonzero(rank == l)[0]
    take = last[np.argsort(-d[last], kind="stable")][: n - int((rank < l).sum())]
    assert r.info().status == 0 and len(take)
    assert np.array_equal(r.selected.cpu().numpy(),
                          np.sort(np.concatenate([np.nonzero(rank < l)[0], take])))
