"""Edges of the wide-data path (dimensions beyond the fused kernel's) against the
FP64 oracle: key counts around the instantiations, one point and one past a block,
all landmarks as neighbours, and more candidates than a wavefront holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.mark.parametrize("n,d,g,k,mode,copies", [
    (1, 65, 3, 3, "fp32", 1), (65, 129, 256, 32, "bf16", 1), (64, 80, 257, 5, "fp32", 1),
    (300, 67, 2048, 32, "fp32", 1), (130, 256, 2049, 16, "bf16", 1), (500, 70, 32, 32, "fp32", 1),
    (200, 90, 200, 8, "fp32", 100)])
def test_wide_paths(torch_dev, oracle_mod, n, d, g, k, mode, copies):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(n + d + g)
    X = rng.normal(0, 2, (n, d)).astype(np.float32)
    L = rng.normal(0, 2, (g, d)).astype(np.float32)
    L[:copies] = L[0]  # coincident landmarks: ties at tau, decided by the index
    X[: n // 2] = L[rng.integers(0, g, n // 2)] + rng.normal(0, 0.5, (n // 2, d)).astype(np.float32)
    l = rng.normal(0, 3, (g, 2)).astype(np.float32)
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = esom.Context(0)
    try:
        print("case wide n=%d d=%d g=%d k=%d %s copies=%d" % (n, d, g, k, mode, copies), flush=True)
        out, idx, _ = ctx.embed(dev(X), dev(L), dev(l), k=k, mode=mode, knn=True)
        out, idx = out.cpu().numpy().astype(np.float64), idx.cpu().numpy()
    finally:
        ctx.close()
    ref = oracle_mod.embed(X, L, l, k, threads=8)
    np.testing.assert_array_equal(idx, ref["idx"][:, :k])
    # the library's coordinate bar: 1e-4 of the grid span
    span = float(np.ptp(l, axis=0).max())
    scale = np.maximum(span, np.abs(ref["out"]).max(axis=1))
    assert (np.abs(out - ref["out"]).max(axis=1) / scale).max() <= 1e-4
