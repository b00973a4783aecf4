"""Cell lists at the limits of the one-workgroup construction (up to 4 096 atoms and what fits its LDS): the neighbour sets
against the oracle's, on both sides of the line, with segments that share waves, span them, are empty or hold one atom."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _sizes(rng, n, n_seg):
    cuts = np.sort(rng.integers(0, n + 1, size=n_seg - 1))   # (equal cuts: empty segments)
    return np.diff(np.concatenate([[0], cuts, [n]]))


@pytest.mark.parametrize("n,n_seg,periodic", [
    (1, 1, False), (64, 1, False), (65, 3, False), (1023, 40, False), (1025, 2, False), (2240, 64, False), (3000, 3, True),
    (4096, 1, False), (4096, 17, False), (4097, 17, False),          # the limit in atoms
    (1500, 1100, False), (2000, 250, False), (3900, 300, False),     # the limits in segments and in LDS
])
def test_neighbour_sets(n, n_seg, periodic):
    import torch
    import oracle as O
    from paper_2601_16622_amd import binding as B, workloads as W
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(n + n_seg)
    cfg = dict(L=1, C=32, H=2, B=8, lf=1, cutoff=3.0, dtype="f32")
    box = None
    if periodic:
        wl = W.periodic_boxes((1000, 1500, 500), seed=3, L=1, C=32, H=2, B=8, cutoff=3.0, dtype="f32")
        box = wl["box"]
    else:
        parts = [(rng.random((s, 3)) * max(1.0, s / 0.1) ** (1.0 / 3.0) + rng.uniform(-50, 50, 3)).astype(np.float32)
                 for s in _sizes(rng, n, n_seg)]
        wl = W._pack(cfg, parts, rng, elements=False)
    P = B.Problem(wl)
    try:
        P.build_cells()
        _, offs, idx = P.neighbors()
        if box is None:
            ref = O.neighbor_list(wl["pos"], wl["seg"], np.float32(3.0))
        else:
            ref = O.neighbor_list_periodic(wl["pos"], wl["seg"], np.float32(3.0), box)
        assert np.array_equal(offs, ref[0]) and np.array_equal(idx, ref[1])
    finally:
        P.close()


@pytest.mark.parametrize("periodic", [False, True])
def test_nearest_neighbours_on_both_sides_of_every_path(periodic):
    """The K nearest of 64, 65, 256, 257, 512 and 513 neighbours: found by counting up to 256 of them (64 to a register), by
    a radix select over keys in LDS up to 512, by repeated walks beyond.  Clusters on a lattice of 0.25, so that most
    distances are shared by many atoms and exact in binary32 (ties go to the lower index), open and across a box's faces."""
    import torch
    import oracle as O
    from paper_2601_16622_amd import binding as B, workloads as W
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(4)
    sites = np.stack(np.meshgrid(*[np.arange(9)] * 3, indexing="ij"), -1).reshape(-1, 3) * 0.25   # diagonal 3.5
    sizes = (65, 66, 257, 258, 513, 514)
    parts = [(sites[rng.permutation(len(sites))[:s]] - (1.0 if periodic else 20.0)).astype(np.float32) for s in sizes]
    wl = W._pack(dict(L=1, C=32, H=2, B=8, lf=1, cutoff=5.0, dtype="f32"), parts, rng, elements=False)
    if periodic:
        wl["box"] = np.full((len(sizes), 3), 16.0, dtype=np.float32)
        off, idx, shift = O.neighbor_list_periodic(wl["pos"], wl["seg"], np.float32(5.0), wl["box"])
        assert shift.any()
        tr = O.edge_translations(wl["seg"], wl["box"], off, shift)
        pos = O.wrap_positions(wl["pos"], wl["seg"], wl["box"])
    else:
        (off, idx), tr, pos = O.neighbor_list(wl["pos"], wl["seg"], np.float32(5.0)), None, wl["pos"]
    assert sorted(set(np.diff(off))) == [s - 1 for s in sizes]
    P = B.Problem(wl)
    try:
        P.build_cells()
        for K in (1, 20, 63, 64, 65, 200, 255, 256, 257, 400, 511, 512, 513):
            table, count = (x.cpu().numpy() for x in P.neighbor_table(K))
            ref = O.cap_neighbors(pos, off, idx, K, tr)
            assert np.array_equal(count, np.diff(ref[0]))
            for i in range(P.N):
                row = table[i]
                assert (row[count[i]:] == -1).all()
                assert np.array_equal(np.sort(row[:count[i]]), np.sort(ref[1][ref[0][i]:ref[0][i + 1]])), (i, K)
    finally:
        P.close()
