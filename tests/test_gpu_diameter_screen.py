"""The diameter's fp16 screening at the edges of its operand layout and scale.

M + 4 operand features (the coordinates, and each norm in two fp16 parts) or,
where those do not fit the padded feature count, M + 2: M = 28 to 31 and 60 to
64 lie on both sides. The operands are scaled by a power of two found from the
data, so data of any magnitude must give the pair and the fp64 value of the
oracle, bit for bit. "antipodal" holds 1,500 pairs within 4e-6 of the largest
distance, inside the band that the screening leaves to the fp64 decision;
"offset" lies far from the origin against its spread."""
import numpy as np
import pytest
import torch

import oracle
import paper_1402_3788_amd as km

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0") if torch.cuda.is_available() else None


def _data(n, M, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "antipodal":
        u = rng.standard_normal((n // 2, M))
        u /= np.linalg.norm(u, axis=1, keepdims=True)
        u *= 1.0 + 1e-6 * rng.random((n // 2, 1))
        X = np.concatenate([u, -u, 0.1 * rng.standard_normal((n - 2 * (n // 2), M))])
        X = X[rng.permutation(n)]
    else:
        X = rng.standard_normal((n, M)) + (300.0 if kind == "offset" else 0.0)
    return X


@pytest.mark.parametrize("kind", ["normal", "antipodal", "offset"])
@pytest.mark.parametrize("scale", [1.0, 1e-13, 7e15, 3e-19])
@pytest.mark.parametrize("M", [1, 5, 28, 29, 30, 31, 60, 61, 62, 63, 64])
def test_screening_keeps_the_farthest_pair(M, scale, kind):
    print(f"[screen] M={M} scale={scale} {kind}", flush=True)
    X = np.ascontiguousarray((_data(3_001, M, kind, M) * scale).astype(np.float32))
    d2, pair, _ = km.kmeans_diameter(torch.from_numpy(X).to(DEV))
    want = oracle.diameter(X)
    assert float(d2.item()) == float(want[0])
    assert tuple(pair.cpu().tolist()) == want[1:]


def _band_pairs(X):
    """Pairs within 0.4 % of the largest centred norm of the longest: in the
    band of the first screening whatever its products round to."""
    x = X.astype(np.float64) - X.astype(np.float64).mean(axis=0)
    nrm = (x * x).sum(axis=1)
    d = nrm[:, None] + nrm[None, :] - 2.0 * (x @ x.T)
    return int((d >= d.max() - 0.004 * nrm.max()).sum()) // 2


def _counted(X):
    """Diameter of X, and the pairs that were taken in fp64: the fifth counter
    at the workspace's start."""
    n, M = X.shape
    ws = torch.empty(km.kmeans_diameter_workspace_bytes(n, M), dtype=torch.uint8, device=DEV)
    d2, pair, _ = km.kmeans_diameter(torch.from_numpy(X).to(DEV), ws=ws)
    return float(d2.item()), tuple(pair.cpu().tolist()), int(ws[16:20].cpu().view(torch.int32).item())


@pytest.mark.parametrize("M,kind", [(2, "sphere"), (3, "sphere")] +
                         [(M, "groups") for M in (2, 3, 25, 29, 32, 62, 64)])
def test_few_of_many_pairs_near_the_longest_are_taken_in_fp64(M, kind):
    """Points on a sphere, and two groups of sigma 3e-5 at distance 1."""
    print(f"[screen] M={M} {kind}", flush=True)
    rng = np.random.default_rng(M)
    X = rng.standard_normal((3_001, M))
    if kind == "sphere":
        X /= np.linalg.norm(X, axis=1, keepdims=True)
    else:
        X *= 3e-5
        X[1_500:, 0] += 1.0
    X = np.ascontiguousarray(X.astype(np.float32))
    d2, pair, taken = _counted(X)
    want = oracle.diameter(X)
    assert (d2, pair) == (float(want[0]), want[1:])
    print(f"[screen] {taken} pairs", flush=True)
    assert 1 <= taken < _band_pairs(X) // 4


@pytest.mark.parametrize("scale", [1e-15, 1e-16, 1e-17, 2e-18])
@pytest.mark.parametrize("M", [5, 25, 64])
def test_small_spreads_are_screened(M, scale):
    """Squared norms down to 1e-35 are screened like any others."""
    print(f"[screen] M={M} scale={scale}", flush=True)
    X = np.ascontiguousarray((_data(3_001, M, "normal", M) * scale).astype(np.float32))
    d2, pair, taken = _counted(X)
    want = oracle.diameter(X)
    assert (d2, pair) == (float(want[0]), want[1:])
    print(f"[screen] {taken} pairs", flush=True)
    assert 1 <= taken < 1_000
