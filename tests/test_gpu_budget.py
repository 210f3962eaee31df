"""Contexts with a memory budget: what a call takes only to be faster is given back to
a later call that needs the room, and results do not depend on the budget."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

G, D, K = 500, 16, 8


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


@pytest.fixture(scope="module")
def data(torch_dev):
    rng = np.random.default_rng(3)
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()
    X = dev(rng.normal(0, 2, (300_000, D)).astype(np.float32))
    near = dev(rng.integers(0, G, 300_000).astype(np.int32))
    return X, dev(rng.normal(0, 2, (G, D)).astype(np.float32)), dev(rng.normal(0, 3, (G, 3)).astype(np.float32)), near


def _call(ctx, what, data):
    """One call of each kind; its outputs as one array each."""
    from paper_2201_00701_amd import esom
    X, L, l3, near = data
    l = l3[:, :2].contiguous()
    if what == "embed":  # 300k points: the largest scratch
        return [ctx.embed(X, L, l, k=K)]
    if what == "embed3":  # 40k points: a pair table of G x G doubles
        return list(ctx.embed3(X[:40_000], L, l3, k=K, knn=True))
    if what == "layout":  # edge lists of G x 64 entries
        nbr, _ = esom.landmark_graph(L, 6)
        ctx.graph_layout(L, nbr, l, steps=3)
        return [l]
    L1 = L.clone()  # an update: partial sums as room allows
    cnt = ctx.landmark_update(X, L1, l, kind="kmeans", alpha=0.5, nearest=near, counts=True)
    return [L1, cnt]


def _least(todo, data):
    """The least budget (to 4 KB) of a context that does these calls."""
    from paper_2201_00701_amd import esom
    lo, hi = 0, 64 << 20
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        ctx = esom.Context(0, mid)
        try:
            for what in todo:
                _call(ctx, what, data)
            hi = mid
        except esom.EsomError as e:
            assert e.code == esom.ESOM_ENOMEM
            lo = mid
        finally:
            ctx.close()
    return hi


def _given_back(data, first, needs):
    """The optional memory first, then the call that needs its room, then the first
    again, within the embedding's own least budget and `needs` bytes, which the first
    call takes in any case."""
    from paper_2201_00701_amd import esom
    free, ctx = esom.Context(0), esom.Context(0, _least(["embed"], data) + needs + 4096)
    try:
        print("case optional memory %s" % first, flush=True)
        for what in (first, "embed", first, "embed"):
            want = _call(free, what, data)
            for a, b in zip(_call(ctx, what, data), want):
                # FP64 sums in another split, one rounding to FP32; all else is the same
                np.testing.assert_allclose(a.cpu().numpy(), b.cpu().numpy(), rtol=2.0 ** -23, atol=2.0 ** -22)
    finally:
        ctx.close()
        free.close()


# the list of 3-D neighbours beside the table; the layout's second positions beside
# the edge lists
@pytest.mark.parametrize("first,needs", [("embed3", 4 * 40_000 * K), ("layout", 8 * G)])
def test_optional_memory_is_given_back(torch_dev, data, first, needs):
    _given_back(data, first, needs)


# the partial sums take the room there is, and give it back
def test_update_workspace_is_given_back(torch_dev, data):
    _given_back(data, "update", 8 * G * (D + 1))


# the least workspace of an update (the sums alone), room for a few ranges of partial
# sums, for all of them, and for the compact copy of a strided list
@pytest.mark.parametrize("ranges,copy", [(0, 0), (1, 0), (3, 0), (3, 1), (300, 0), (300, 1)])
def test_update_in_the_room_there_is(torch_dev, data, ranges, copy):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(8)
    n, d, g = 40_001, 64, 700
    X = rng.integers(-8, 9, (n, d)).astype(np.float32)
    L = rng.normal(0, 2, (g, d)).astype(np.float32)
    near = rng.integers(-1, g + 1, (n, 3)).astype(np.int32)
    al = lambda b: (b + 255) & ~255
    sums = 8 * g * (d + 1)
    dev = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()
    ctx = esom.Context(0, 128 + al(sums) + al(ranges * sums) + copy * al(4 * n) + 256)
    try:
        print("case update room ranges=%d copy=%d" % (ranges, copy), flush=True)
        Ld = dev(L)
        cnt = ctx.landmark_update(dev(X), Ld, dev(L[:, :2]), kind="kmeans", alpha=1.0, nearest=dev(near)[:, 0],
                                  counts=True)
        got, cnt = Ld.cpu().numpy(), cnt.cpu().numpy()
    finally:
        ctx.close()
    ok = (near[:, 0] >= 0) & (near[:, 0] < g)
    c = np.bincount(near[ok, 0], minlength=g)
    S = np.zeros((g, d))
    np.add.at(S, near[ok, 0], X[ok].astype(np.float64))
    np.testing.assert_array_equal(cnt, c)
    # whole sums are exact; one rounding of the mean, and two FP64 operations on the way
    want = np.where(c[:, None] > 0, S / np.maximum(c, 1)[:, None], L)
    np.testing.assert_allclose(got, want, rtol=2.0 ** -23, atol=2.0 ** -50)
