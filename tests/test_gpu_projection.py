"""The two fp32 projections at 64 and 128 channels, weights in registers and per tile, at the edges of their tiles, of the plan
(tiles per workgroup by degree) and of the rule between them: the forward pass, which reads the layouts they write, against the
materialized call, whose projection is another kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CUTOFF = 4.0
LCAP = 240   # slot groups that a tile's candidate list holds


def compare(L, C, H, parts, seed):
    import torch
    from paper_2601_16622_amd import binding as B, workloads as W
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    cfg = dict(L=L, C=C, H=H, B=8, lf=min(1, L), cutoff=CUTOFF, dtype="f32")
    P = B.Problem(W._pack(cfg, [p.astype(np.float32) for p in parts], np.random.default_rng(seed), elements=False))
    try:
        P.build_cells()
        ref = torch.full_like(P.out, float("nan"))
        P.forward_materialized(ref)
        P.attn_ws.fill_(255)   # nothing that the call above left is found again
        P.out.fill_(float("nan"))
        P.forward()
        torch.cuda.synchronize()
        got, want = P.out.double(), ref.double()
        assert torch.isfinite(got).all()
        assert float(want.norm()) > 0.0
        # both are some 8e-7 of the norm from 64 bits
        assert float((got - want).norm()) <= 5e-6 * float(want.norm())
    finally:
        P.close()


def box(rng, N):
    return rng.random((N, 3)) * (N / 0.1) ** (1.0 / 3.0)


@pytest.mark.parametrize("L,C,N,H", [
    (1, 64, 15, 4), (2, 64, 17, 4), (4, 64, 203, 4),         # a lone tile, ragged ends
    (2, 64, 40, 2), (2, 64, 999, 2), (2, 64, 1000, 2),       # heads of 32 channels, plain layouts only: both sides of their rule
    (0, 64, 1105, 4), (0, 128, 2599, 8), (2, 128, 1499, 4), (2, 128, 1500, 4),
    (2, 128, 949, 8), (2, 128, 950, 8), (3, 128, 913, 8), (4, 128, 899, 8), (4, 128, 1027, 8),   # with the tile layouts
    # tiles per workgroup by degree, from L down, the last workgroup of a degree short of them:
    (4, 64, 3010, 4),     # 1, 2, 2, 4, 14; 0, 1, 1, 1, 7 left
    (4, 128, 4000, 8),    # 3, 3, 5, 9, 27; 1, 1, 0, 7, 7 left
    (4, 128, 6000, 8),    # 1, 1, 2, 3, 10 in 1 101 workgroups, four rounds of them; 0, 0, 1, 0, 5 left
])
def test_forward_against_the_materialized_call(L, C, N, H):
    compare(L, C, H, [box(np.random.default_rng(N), N)], N)


@pytest.mark.parametrize("L,C,H", [(1, 64, 4), (2, 128, 8)])
def test_crowded_tiles_read_the_plain_layouts(L, C, H):
    """964 atoms that all see each other, whose tiles are left to the kernel that reads the plain q, k and v, and a second
    system of 100, whose lists fit (at most 26 groups a pass, 9 passes)."""
    rng = np.random.default_rng(C)
    ball = rng.uniform(-1.1, 1.1, size=(964, 3)).astype(np.float32)
    seen = (np.linalg.norm(ball[:, None].astype(np.float64) - ball[None], axis=-1) < CUTOFF).sum(1)
    assert seen.min() > 4 * LCAP   # a list with all of them has more groups of four than fit
    compare(L, C, H, [ball, box(rng, 100)], C)
