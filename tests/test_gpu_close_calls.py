"""Close calls of the matrix-core kernels and the two-launch form of large K x M.

Objects whose split-precision scores leave the label open are noted during a
launch and decided after its last tile, among the centres within their limit
or, when a wave's list overflowed, over all centres. The data here leave most
objects open (one broad cluster away from the origin, so that the guard band is
wide against the distances between centres), at the feature counts where the
form of the split products changes (a last chunk of at most 8, at most 16, more
features), at ragged n, and at shapes whose sums are formed in a second launch
(K x M too large for one workgroup's LDS). Labels and counts must equal the
oracle's exactly; a centre is an fp64 mean rounded once, so a sum in another
order moves it by at most one unit in the last place (2^-23 relative)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1402_3788_amd as km
import test_plans

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0") if torch.cuda.is_available() else None


def _case(n, M, K, seed, kind):
    rng = np.random.default_rng(seed)
    if kind == "dups":                       # exact ties, also between centres
        vals = rng.integers(-2, 3, (12, M)).astype(np.float32) + 5
        X = vals[rng.integers(0, 12, n)]
        C = vals[rng.integers(0, 12, K)]
    else:
        X = (rng.standard_normal((n, M)) + (20.0 if kind == "offset" else 1.0)).astype(np.float32)
        C = (rng.standard_normal((K, M)) + (20.0 if kind == "offset" else 1.0)).astype(np.float32)
        X[: min(n, K) // 2] = C[: min(n, K) // 2]
    return np.ascontiguousarray(X), np.ascontiguousarray(C)


def _check(X, C, path):
    n, K = X.shape[0], C.shape[0]
    Xg, Cg = torch.from_numpy(X).to(DEV), torch.from_numpy(C).to(DEV)
    want, d1, _ = oracle.assign(X, C, with_dist=True)
    lab, d2 = km.kmeans_assign(Xg, Cg, with_min_d2=True, path=path)
    assert np.array_equal(lab.cpu().numpy(), want)
    np.testing.assert_allclose(d2.cpu().numpy(), d1, rtol=(X.shape[1] + 2) * 2.0**-22, atol=1e-30)
    olab, oC, ocnt, _ = oracle.run(X, K, C, 2, fixed=True)
    glab, gC, gcnt, _ = km.kmeans_run(Xg, K, Cg, 2, fixed_iters=True, path=path)
    assert np.array_equal(glab.cpu().numpy(), olab)
    assert np.array_equal(gcnt.cpu().numpy(), ocnt)
    scale = np.maximum(np.abs(oC).max(axis=1, keepdims=True), 1e-30)
    assert (np.abs(gC.cpu().numpy().astype(np.float64) - oC) <= 2.0**-23 * scale).all()
    again = km.kmeans_run(Xg, K, Cg, 2, fixed_iters=True, path=path)
    assert torch.equal(again[1].view(torch.int32), gC.view(torch.int32))


# K <= 64 with M <= 32: one object per lane, with one, two and four centre
# blocks; otherwise tiles, with M at the edges of the product forms, K = 65 ...
# 256 the fused launch, larger K x M the two-launch form
SHAPES = [(1, 3, 5), (65, 10, 8), (5_001, 25, 16), (4_097, 10, 24), (129, 31, 33), (3_001, 32, 64),
          (1, 8, 65), (63, 9, 100), (64, 16, 129), (4_097, 17, 200), (5_001, 24, 257),
          (4_999, 32, 65), (3_000, 33, 70), (5_003, 40, 20), (2_049, 41, 150), (3_001, 49, 90),
          (2_000, 64, 17), (4_097, 16, 1024), (3_001, 32, 512), (2_003, 64, 256), (4_001, 25, 600),
          (70, 2, 1000)]


@pytest.mark.parametrize("kind", ["near", "offset", "dups"])
@pytest.mark.parametrize("n,M,K", SHAPES)
def test_close_calls_follow_the_oracle(n, M, K, kind):
    print(f"[close] n={n} M={M} K={K} {kind}", flush=True)
    X, C = _case(n, M, K, n + M + K, kind)
    _check(X, C, None)


@pytest.mark.parametrize("n,M,K,path", [(20_003, 64, 186, "tiles"), (20_003, 24, 471, "tiles"),
                                        (20_003, 17, 545, "tiles"),
                                        (20_000, 64, 187, "tiles"), (20_001, 7, 40, "tiles")])
def test_overflowing_lists_follow_the_oracle(n, M, K, path):
    """One-wave workgroups whose list of close calls holds 68, 2, 64 and 2
    objects beside the slab (the first four; up to 128 are open), with nearly
    every object open: the objects are found again by the marks in their
    labels."""
    print(f"[overflow] n={n} M={M} K={K}", flush=True)
    X, C = _case(n, M, K, n + M, "offset")
    _check(X, C, path)


@pytest.mark.parametrize("with_d2", [False, True])
def test_overflowing_lists_of_the_lane_kernel(with_d2):
    """More close calls per wave than the list holds (444 beside the slabs of
    K = 64, M = 32): the labels equal those of the direct form, whose calls do
    not go through a list, and the centres to one unit in the last place.
    (Without distances to overflow, the assignment alone fits its longer lists
    here; test_every_kind_of_list_overflows has the sizes for it.)"""
    n, M, K = 1_200_003, 32, 64
    print(f"[overflow lane] n={n} M={M} K={K}", flush=True)
    X, C = _case(n, M, K, 5, "offset")
    Xg, Cg = torch.from_numpy(X).to(DEV), torch.from_numpy(C).to(DEV)
    if with_d2:
        lab, d2 = km.kmeans_assign(Xg, Cg, with_min_d2=True)
        want, wd2 = km.kmeans_assign(Xg, Cg, with_min_d2=True, path="direct")
        assert torch.equal(lab, want)
        torch.testing.assert_close(d2, wd2, rtol=(M + 2) * 2.0**-22, atol=1e-30)
        return
    lab, cen, cnt, _ = km.kmeans_run(Xg, K, Cg, 1, fixed_iters=True)
    want, wcen, wcnt, _ = km.kmeans_run(Xg, K, Cg, 1, fixed_iters=True, path="direct")
    assert torch.equal(lab, want) and torch.equal(cnt, wcnt)
    scale = wcen.abs().amax(1, keepdim=True)
    assert ((cen - wcen).abs() <= 2.0**-23 * scale).all()


@pytest.mark.parametrize("n,M,K,kernel,mode", [
    (4_300_003, 3, 64, "lane", "assign"), (920_009, 32, 64, "lane", "run"),
    (460_003, 64, 186, "tile", "assign"), (550_003, 40, 20, "tile", "run"),
    (1_010_009, 17, 100, "tile", "run"), (570_011, 25, 300, "tile", "run"),
    (1_860_001, 33, 65, "tile", "run")])
def test_every_kind_of_list_overflows(n, M, K, kernel, mode):
    """Every centre is there twice, so every object is open, and there are more
    objects than all lists hold together: the assignments with and without
    distances, private slabs (two forms) and slabs that six or eight waves
    share in turn."""
    print(f"[overflow] n={n} M={M} K={K} {kernel} {mode}", flush=True)
    plan = test_plans.plan_tile if kernel == "tile" else test_plans.plan_lane_mfma
    p = plan(n, M, K, test_plans.ASSIGN if mode == "assign" else test_plans.ASSIGN_ACCUM)
    assert p.waves >= 6 and n > p.waves * p.groups * p.list_cap
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    X = torch.randn(n, M, device=DEV, generator=g)
    C = torch.randn(K, M, device=DEV, generator=g)
    C[K // 2:K // 2 * 2] = C[:K // 2]
    if K % 2:
        C[K - 1] = 1e6                          # the nearest of no object
    ws = km.workspace(n, M, K, DEV)
    lab, cen, cnt, _ = km.kmeans_run(X, K, C, 1, fixed_iters=True, ws=ws)
    want, wd2 = km.kmeans_assign(X, C, with_min_d2=True, path="direct")
    assert km.ctl_fallbacks(ws) == n            # all open
    assert torch.equal(lab, want)
    wcen, wcnt = km.kmeans_update(X, want, K, C)
    assert torch.equal(cnt, wcnt)
    scale = wcen.abs().amax(1, keepdim=True)
    assert ((cen - wcen).abs() <= 2.0**-23 * scale).all()
    if mode == "assign":
        assert torch.equal(km.kmeans_assign(X, C), want)
        lab, d2 = km.kmeans_assign(X, C, with_min_d2=True)
        assert torch.equal(lab, want)
        torch.testing.assert_close(d2, wd2, rtol=(M + 2) * 2.0**-22, atol=1e-30)


@pytest.mark.parametrize("n,M,K", [(1, 16, 1024), (64, 16, 1024), (65, 63, 260), (40_007, 15, 1000),
                                   (40_007, 64, 256), (9_999, 41, 399)])
def test_sums_from_labels_follow_the_oracle(n, M, K):
    """The sums' own launch, by slices of features (M a multiple of four or
    not, labels out of range ignored)."""
    print(f"[sums] n={n} M={M} K={K}", flush=True)
    rng = np.random.default_rng(n + M)
    X = rng.uniform(-60, 60, (n, M)).astype(np.float32)
    labels = rng.integers(0, K, n).astype(np.int32)
    prev = rng.standard_normal((K, M)).astype(np.float32)
    bad = labels.copy()
    bad[::7] = np.where(np.arange(len(bad[::7])) % 2 == 0, -1, K)
    for lab in (labels, bad):
        C, cnt = km.kmeans_update(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), K,
                                  torch.from_numpy(prev).to(DEV))
        keep = (lab >= 0) & (lab < K)
        if keep.any():
            oC, ocnt = oracle.update(X[keep], lab[keep], K, prev)
        else:
            oC, ocnt = prev, np.zeros(K, np.int32)
        assert np.array_equal(cnt.cpu().numpy(), ocnt)
        scale = np.maximum(np.abs(oC).max(axis=1, keepdims=True), 1e-30)
        assert (np.abs(C.cpu().numpy().astype(np.float64) - oC) <= 2.0**-23 * scale).all()


@pytest.mark.parametrize("n,M,K", [(40_007, 57, 140), (40_007, 50, 200), (65_600, 33, 300),
                                   (20_003, 61, 100), (40_001, 64, 20), (40_000, 48, 100),
                                   (30_011, 25, 512), (65, 64, 17)])
def test_sums_in_slices_of_eight_and_sixteen_features(n, M, K):
    """Whole slices and remainders of every kind (9, 2, 1, 13 features, none)."""
    print(f"[slices] n={n} M={M} K={K}", flush=True)
    rng = np.random.default_rng(n + M)
    X = rng.uniform(-60, 60, (n, M)).astype(np.float32)
    lab = rng.integers(-1, K + 1, n).astype(np.int32)
    prev = rng.standard_normal((K, M)).astype(np.float32)
    C, cnt = km.kmeans_update(torch.from_numpy(X).to(DEV), torch.from_numpy(lab).to(DEV), K,
                              torch.from_numpy(prev).to(DEV))
    keep = (lab >= 0) & (lab < K)
    oC, ocnt = oracle.update(X[keep], lab[keep], K, prev)
    assert np.array_equal(cnt.cpu().numpy(), ocnt)
    scale = np.maximum(np.abs(oC).max(axis=1, keepdims=True), 1e-30)
    assert (np.abs(C.cpu().numpy().astype(np.float64) - oC) <= 2.0**-23 * scale).all()
