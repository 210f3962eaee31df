"""Edges of the landmark update and of online SOM training against the FP64
oracle: slices and ranges of the LDS sums, landmark counts beyond them, budgeted
contexts, strided and invalid nearest lists, and small and large batches."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# FP64 sums on both sides and one rounding to FP32 (2^-24 relative); the sums
# themselves differ by at most n 2^-53 relative to the summed magnitudes
RTOL = 2.0 ** -23


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _reference(X, L, l, near, kind, alpha, sigma):
    g, d = L.shape
    S, c = np.zeros((g, d)), np.zeros(g)
    ok = (near >= 0) & (near < g)
    np.add.at(S, near[ok], X[ok].astype(np.float64))
    np.add.at(c, near[ok], 1.0)
    counts = c.astype(np.int32)
    if kind == "som":
        d2 = ((l[:, None].astype(np.float64) - l[None]) ** 2).sum(2)
        h = np.exp(-d2 / (2.0 * float(np.float32(sigma)) ** 2)) if sigma > 0 else np.eye(g)
        S, c = h @ S, h @ c
    a = float(np.float32(alpha))
    mean = np.where(c[:, None] > 0, S / np.where(c > 0, c, 1.0)[:, None], L)
    return L + a * (mean - L), counts


# n on both sides of a range (1024) and of all ranges; d around the slice widths
# 16, 32 and 64; g with one slice, several, and past the LDS sums (1163)
@pytest.mark.parametrize("n,d,g,kind,sigma,stride,tight", [
    (1, 1, 3, "kmeans", 0.0, 1, False), (1025, 17, 49, "som", 1.5, 3, False),
    (70_001, 33, 700, "kmeans", 0.0, 16, False), (70_001, 33, 700, "kmeans", 0.0, 16, True),
    (30_000, 64, 1024, "som", 0.7, 20, True), (5000, 65, 300, "som", 0.0, 1, False),
    (3000, 130, 100, "kmeans", 0.0, 2, False), (4000, 255, 60, "som", 2.0, 1, False),
    (300_000, 16, 1163, "kmeans", 0.0, 1, False), (20_000, 16, 1300, "som", 1.0, 2, False)])
def test_update_paths(torch_dev, n, d, g, kind, sigma, stride, tight):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(n + d)
    X = rng.normal(0, 2, (n, d)).astype(np.float32)
    L = rng.normal(0, 2, (g, d)).astype(np.float32)
    l = rng.normal(0, 2, (g, 2)).astype(np.float32)
    near = rng.integers(-1, g + 1, n).astype(np.int32)  # -1 and g are ignored
    near[: n // 3] = g // 2                              # one landmark with a long list
    wide = np.full((n, stride), -7, np.int32)
    wide[:, 0] = near
    # the budget: the counters and what the counting sort takes for this shape
    al = lambda b: (b + 255) & ~255
    chunks = n // 4096 + g + 1
    room = 128 + al(8 * g * (d + 1)) + al(4 * g) + 2 * al(8 * (g + 1)) + al(4 * n) + 2 * al(4 * chunks) + 256
    ctx = esom.Context(0, room if tight else 0)
    try:
        print("case update n=%d d=%d g=%d %s stride=%d tight=%s" % (n, d, g, kind, stride, tight), flush=True)
        Ld = _dev(torch_dev, L)
        cnt = ctx.landmark_update(_dev(torch_dev, X), Ld, _dev(torch_dev, l), kind=kind, alpha=0.3, sigma=sigma,
                                  nearest=_dev(torch_dev, wide)[:, 0], counts=True)
        got, cnt = Ld.cpu().numpy(), cnt.cpu().numpy()
    finally:
        ctx.close()
    ref, rc = _reference(X, L, l, near, kind, 0.3, sigma)
    np.testing.assert_array_equal(cnt, rc)
    np.testing.assert_allclose(got, ref, rtol=RTOL, atol=RTOL * np.abs(ref).max())


# batches around the points per wavefront (1, 2, 4) and the direct path's limit
# (4096), d around the lanes per row (16, 32, 64) and the tile sizes
@pytest.mark.parametrize("B,d,g", [(1, 16, 3), (7, 17, 65), (1025, 33, 300), (2049, 64, 257), (300, 65, 129),
                                   (64, 129, 70), (33, 256, 40), (4096, 5, 400), (4097, 5, 400), (3, 2, 4097)])
def test_som_train_paths(torch_dev, oracle_mod, B, d, g):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(B + d)
    n, T = 3000, 3
    X = rng.integers(-3, 4, (n, d)).astype(np.float32)
    L = rng.integers(-3, 4, (g, d)).astype(np.float32)  # exact ties: the lower index wins
    L[g - 1] = L[0]
    l = rng.normal(0, 3, (g, 2)).astype(np.float32)
    rows = rng.integers(-1, n + 1, (T, B)).astype(np.int32)  # -1 and n present no point
    frozen = (rng.random(g) < 0.1).astype(np.uint8)
    sigma, alpha = np.float32([1.5, 0.0, 0.7]), np.float32([0.5, 0.25, 0.1])
    ctx = esom.Context(0)
    try:
        print("case som train B=%d d=%d g=%d" % (B, d, g), flush=True)
        Ld = _dev(torch_dev, L)
        # a strided sample
        wide = np.zeros((n, d + 3), np.float32)
        wide[:, :d] = X
        ctx.som_train(_dev(torch_dev, wide)[:, :d], Ld, _dev(torch_dev, l), _dev(torch_dev, rows), list(sigma),
                      list(alpha), frozen=_dev(torch_dev, frozen))
        got = Ld.cpu().numpy()
    finally:
        ctx.close()
    ref = oracle_mod.som_train(X, L, l, rows, sigma.astype(np.float64), alpha.astype(np.float64), frozen=frozen)
    # one FP32 rounding a step on both sides, from FP64 values
    np.testing.assert_allclose(got, ref, rtol=T * RTOL, atol=T * RTOL * 3)
    np.testing.assert_array_equal(got[frozen == 1], L[frozen == 1])


# an infinite batch point is equally far from all landmarks (the lowest index), a NaN
# point has no nearest; on both sides of the direct path's largest batch
@pytest.mark.parametrize("B", [1, 70, 4096, 4097])
def test_som_train_non_finite_rows(torch_dev, B):
    from paper_2201_00701_amd import esom
    n, d, g = 64, 9, 130
    rng = np.random.default_rng(B)
    X = rng.integers(-3, 4, (n, d)).astype(np.float32)
    L = rng.integers(-3, 4, (g, d)).astype(np.float32)
    l = rng.normal(0, 2, (g, 2)).astype(np.float32)
    X[0, 2], X[9, 2], X[11, 4] = np.inf, -np.inf, np.nan
    rows = np.full((1, B), -1, np.int32)
    m = min(B, n)
    rows[0, :m] = rng.permutation(n)[:m] if B > 1 else 0
    ctx = esom.Context(0)
    try:
        print("case som train non-finite rows B=%d" % B, flush=True)
        Ld = _dev(torch_dev, L)
        ctx.som_train(_dev(torch_dev, X), Ld, _dev(torch_dev, l), _dev(torch_dev, rows), [1.5], [0.5])
        got = Ld.cpu().numpy()
    finally:
        ctx.close()
    x = X[rows[0, :m]].astype(np.float64)
    x = x[~np.isnan(x).any(1)]
    near = ((x[:, None] - L[None].astype(np.float64)) ** 2).sum(2).argmin(1)
    d2 = ((l[:, None].astype(np.float64) - l[None]) ** 2).sum(2)
    h = np.exp(-d2 / (2.0 * 1.5 ** 2))[:, near]
    ok = np.arange(d) != 2  # the infinite dimension spreads to every landmark
    ref = L[:, ok] + 0.5 / B * (h @ x[:, ok] - h.sum(1)[:, None] * L[:, ok])
    np.testing.assert_allclose(got[:, ok], ref, rtol=RTOL, atol=RTOL * 3)
    assert not np.isfinite(got[:, 2]).any()
