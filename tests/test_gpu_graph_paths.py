"""Edges of the landmark-graph and layout kernels against the FP64 oracle: tile
and list-capacity boundaries, hub nodes, empty list entries, and the layout
without room for its edge lists."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


# dimensions on both sides of the 4-wavefront limit (128), kg on both sides of
# the list capacities 8 and 16, g one past a tile of 64 or 256 rows
@pytest.mark.parametrize("g,d,kg", [(257, 129, 8), (65, 256, 17), (5, 3, 4), (300, 128, 9), (513, 20, 32),
                                    (256, 1, 16)])
def test_landmark_graph_edges(torch_dev, oracle_mod, g, d, kg):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(g + d)
    # small integers: many exact ties, which the index decides
    L = rng.integers(-2, 3, (g, d)).astype(np.float32)
    print("case graph edges g=%d d=%d kg=%d" % (g, d, kg), flush=True)
    nbr, dist = esom.landmark_graph(torch_dev.from_numpy(L).cuda(), kg)
    rn, rd = oracle_mod.landmark_graph(L, kg)
    np.testing.assert_array_equal(nbr.cpu().numpy(), rn)
    np.testing.assert_array_equal(dist.cpu().numpy(), rd.astype(np.float32))


@pytest.mark.parametrize("g,kg,steps", [(2, 1, 1), (65, 5, 3), (700, 32, 2)])
@pytest.mark.parametrize("room", [True, False])
def test_layout_hub_and_empty_entries(torch_dev, oracle_mod, g, kg, steps, room):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(g)
    L = rng.normal(size=(g, 7)).astype(np.float32)
    l0 = rng.normal(0, 3, (g, 2)).astype(np.float32)
    l0[1] = l0[0]  # coincident positions: no spring force
    nbr = rng.integers(-1, g, (g, kg)).astype(np.int32)  # -1, own and repeated entries among them
    nbr[:, 0] = 0  # every node lists node 0
    # the budget holds the counters and the position buffer, not the edge lists
    ctx = esom.Context(0, 0 if room else 128 + 256 * ((8 * g + 255) // 256))
    try:
        print("case layout g=%d kg=%d steps=%d room=%s" % (g, kg, steps, room), flush=True)
        ld = torch_dev.from_numpy(l0).cuda()
        ctx.graph_layout(torch_dev.from_numpy(L).cuda(), torch_dev.from_numpy(nbr).cuda(), ld, steps=steps,
                         scale=0.3)
        got = ld.cpu().numpy().astype(np.float64)
    finally:
        ctx.close()
    ref = oracle_mod.layout(L, nbr, l0, steps=steps, scale=0.3, repulsion=0.05, soft=0.5, step=0.1, max_move=0.5)
    # FP64 forces on both sides, summed in different orders; a position is
    # rounded to a float after every step (2^-24 of its size each), and a step
    # carries a difference on by at most a factor of the force's gradient
    assert np.abs(got - ref).max() <= steps * 4.0 * 2.0 ** -24 * max(1.0, np.abs(ref).max())


# infinite landmarks: their distances compete by index, as in a plain FP64 evaluation
@pytest.mark.parametrize("g,d,kg", [(5, 3, 4), (70, 17, 32), (300, 48, 10), (40, 130, 30), (33, 5, 8)])
def test_graph_of_infinite_landmarks(torch_dev, g, d, kg):
    from paper_2201_00701_amd import esom
    rng = np.random.default_rng(g + d)
    L = rng.integers(-3, 4, (g, d)).astype(np.float32)
    L[1, 0], L[g - 2, d - 1] = np.inf, -np.inf
    print("case graph of infinite landmarks g=%d d=%d kg=%d" % (g, d, kg), flush=True)
    nbr, d2 = esom.landmark_graph(torch_dev.from_numpy(L).cuda(), kg)
    D = ((L[:, None].astype(np.float64) - L[None]) ** 2).sum(2)  # whole numbers or infinite, NaN on the diagonal
    want = np.stack([np.lexsort((np.arange(g)[np.arange(g) != u], D[u, np.arange(g) != u])) for u in range(g)])[:, :kg]
    want = want + (want >= np.arange(g)[:, None])
    np.testing.assert_array_equal(nbr.cpu().numpy(), want)
    np.testing.assert_array_equal(d2.cpu().numpy(), np.take_along_axis(D, want, 1))
