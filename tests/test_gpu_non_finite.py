"""Projection calls with non-finite rows: the other rows keep their bits, a NaN row
gives NaN and no list, an infinite one is equally far from all landmarks (the lowest
indices, the centroid of their positions)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


# landmark counts that leave 1 to 63 padded positions; every list size with k equal to
# it and below; landmark rows in LDS (few landmarks), from memory, and points in
# locality order; the wide path
@pytest.mark.parametrize("n,d,g,k,mode", [
    (300, 20, 70, 8, "bf16"), (300, 20, 70, 16, "bf16"), (300, 20, 65, 12, "fp32"), (200, 33, 127, 20, "bf16"),
    (200, 17, 97, 24, "fp32"), (200, 40, 161, 32, "bf16"), (300, 40, 1001, 7, "bf16"), (300, 40, 1001, 16, "fp32"),
    (300, 100, 400, 16, "bf16"), (200, 64, 1087, 20, "fp32"), (200, 48, 1025, 30, "bf16"), (200, 16, 400, 16, "bf16"),
    (66_000, 24, 513, 16, "bf16"), (66_000, 24, 577, 12, "fp32"), (300, 100, 130, 16, "fp32"), (50, 12, 70, 40, "bf16")])
def test_non_finite_rows(torch_dev, n, d, g, k, mode):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(n + d + g + k)
    L = rng.normal(0, 2, (g, d)).astype(np.float32)
    l = rng.normal(0, 3, (g, 2)).astype(np.float32)
    X = rng.normal(0, 2, (n, d)).astype(np.float32)
    Xb = X.copy()
    nans, infs = [1, 6, n // 2], [2, n // 3, n - 1]
    Xb[nans, [0, d - 1, 5]] = np.nan
    Xb[infs, [d - 1, 0, 4]] = [np.inf, -np.inf, np.inf]
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = esom.Context(0)
    try:
        print("case non-finite rows n=%d d=%d g=%d k=%d %s" % (n, d, g, k, mode), flush=True)
        res = [[t.cpu().numpy() for t in ctx.embed(dev(x), dev(L), dev(l), k=k, mode=mode, knn=True)] for x in (X, Xb)]
        alone = ctx.embed(dev(Xb), dev(L), dev(l), k=k, mode=mode).cpu().numpy()
    finally:
        ctx.close()
    (out, idx, d2), (outb, idxb, d2b) = res
    rest = np.setdiff1d(np.arange(n), nans + infs)
    np.testing.assert_array_equal(outb[rest], out[rest])
    np.testing.assert_array_equal(idxb[rest], idx[rest])
    np.testing.assert_array_equal(d2b[rest], d2[rest])
    assert np.isnan(outb[nans]).all() and (idxb[nans] == -1).all() and np.isnan(alone[nans]).all()
    np.testing.assert_array_equal(idxb[infs], np.tile(np.arange(k), (3, 1)))
    assert np.isinf(d2b[infs]).all()
    centre = np.tile(l[:k].astype(np.float64).mean(0), (3, 1))  # FP64 sums, one rounding
    for o in (outb, alone):
        np.testing.assert_allclose(o[infs], centre, rtol=2.0 ** -23, atol=2.0 ** -23)


# finite rows whose norms leave FP32 (above 1.8e19): the squared distances to the
# nearest landmarks still fit, but most landmarks' keys are infinite and only two of the
# key groups hold a finite one, fewer than k
@pytest.mark.parametrize("mode", ["bf16", "fp32"])
def test_norms_beyond_fp32(torch_dev, oracle_mod, mode):
    from paper_2201_00701_amd import esom
    n, d, g, k = 70, 16, 128, 3
    rng = np.random.default_rng(4)
    L, X = rng.normal(0, 1e17, (g, d)), rng.normal(0, 1e17, (n, d))
    L[:, 0] += 1.86e19 * np.where(np.arange(g) % 2, 1, -1)
    L[[0, 1, 64, 65], 0] = -0.3e19
    X[:, 0] += 0.9e19
    X, L = X.astype(np.float32), L.astype(np.float32)
    l = rng.normal(0, 3, (g, 2)).astype(np.float32)
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = esom.Context(0)
    try:
        print("case norms beyond fp32 %s" % mode, flush=True)
        out, idx, d2 = [t.cpu().numpy() for t in ctx.embed(dev(X), dev(L), dev(l), k=k, mode=mode, knn=True)]
    finally:
        ctx.close()
    ref = oracle_mod.embed(X, L, l, k, threads=8)
    np.testing.assert_array_equal(idx, ref["idx"][:, :k])
    np.testing.assert_allclose(d2, ref["d2"][:, :k], rtol=2.0 ** -23)
    assert np.abs(out - ref["out"]).max() <= 1e-4 * max(float(np.ptp(l, axis=0).max()), np.abs(ref["out"]).max())
