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
