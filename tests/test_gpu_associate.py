"""GPU: the association's lane splits and its list of survivors (more than four
of a point, references beyond one staged chunk, N at the edges of the splits),
the last work-group's intercepts, and the one-work-group compaction, against
the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import paper_2503_20286_amd as nsga3
import workloads
from tests.gpu_helpers import compare_full, gpu_select

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,H,bf16", [
    (1, 2, 2, False), (17, 3, 5000, False), (4096, 5, 300, False), (4097, 2, 97, False),
    (32768, 3, 1300, False), (32769, 4, 35, False), (65536, 2, 11, False), (65537, 2, 11, False),
    (3000, 10, 700, True), (500, 16, 1000, False),
])
@pytest.mark.parametrize("near", [False, True])
def test_association_splits(N, M, H, bf16, near):
    rng = np.random.Generator(np.random.PCG64(N + H))
    f = workloads.sphere_shell(rng, N, M, lambda r, n: r.uniform(0, 0.5, n), 0.2).astype(np.float32)
    # `near`: references in bunches closer than the screen tells apart, and repeated
    d = rng.random((max(1, H // 8), M)) + 0.05
    refs = (np.repeat(d, 8, 0) * (1 + 1e-8 * rng.random((8 * len(d), 1))) if near
            else rng.random((H, M)) + 1e-3).astype(np.float32)[:H]
    K = max(1, N // 2)
    g = gpu_select(f, refs, K, assoc=nsga3.ASSOC_BF16 if bf16 else nsga3.ASSOC_FP32)
    rep = compare_full(f, refs, K, g)
    rep.pop("near_ties")
    assert not any(rep.values()), rep


@pytest.mark.parametrize("N,M,H,kind", [
    (2, 2, 1, "sphere"), (200, 3, 91, "sphere"), (1023, 5, 1, "front"), (1024, 3, 2048, "same"),
    (1024, 16, 2049, "front"), (1024, 2, 4097, "sphere"), (1025, 3, 91, "same"),
])
def test_small_problems(N, M, H, kind):
    """One work-group's order and niching, and the sizes where they end."""
    rng = np.random.Generator(np.random.PCG64(N * H))
    f = workloads.sphere_shell(rng, N, M, lambda r, n: r.uniform(0, 0.5, n), 0.2)
    if kind == "front":
        f /= np.linalg.norm(f, axis=1, keepdims=True)
    if kind == "same":
        f = f[rng.integers(0, N // 3, N)]
    f, refs = f.astype(np.float32), (rng.random((H, M)) + 1e-3).astype(np.float32)
    for K in sorted({1, N // 2, N}):
        rep = compare_full(f, refs, K, gpu_select(f, refs, K))
        rep.pop("near_ties")
        assert not any(rep.values()), (K, rep)
