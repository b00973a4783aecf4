"""The fp32 projection with the weights in registers (64 and 128 channels) at the edges of its tiles, of its
plan (tiles per workgroup by degree) and of its rule: the forward pass, which reads the layouts it writes, against the
materialized call, whose projection is another kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,C,N,H", [
    (1, 64, 1, 4), (2, 64, 15, 4), (2, 64, 17, 4), (4, 64, 203, 4),      # a lone tile, ragged ends
    (2, 64, 40, 2), (2, 64, 999, 2), (2, 64, 1000, 2),                   # heads of 32 channels, plain layouts only: both sides of their rule
    (0, 64, 1105, 4), (0, 128, 2599, 8), (2, 128, 1499, 4), (2, 128, 1500, 4),
    (2, 128, 949, 8), (2, 128, 950, 8), (3, 128, 913, 8), (4, 128, 899, 8), (4, 128, 1027, 8),   # with the tile layouts
    (1, 128, 2303, 8),                                                   # several tiles per workgroup in every degree
])
def test_forward_against_the_materialized_call(L, C, N, H):
    import torch
    from paper_2601_16622_amd import binding as B, workloads as W
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(N)
    cfg = dict(L=L, C=C, H=H, B=8, lf=min(1, L), cutoff=4.0, dtype="f32")
    box = rng.random((N, 3)) * (N / 0.1) ** (1.0 / 3.0)
    dense = min(N // 2, 60)   # some atoms crowded together: tiles whose list does not fit read the plain layouts
    box[:dense] = box[0] + 0.3 * rng.random((dense, 3))
    P = B.Problem(W._pack(cfg, [box.astype(np.float32)], rng, elements=False))
    try:
        P.build_cells()
        ref = torch.full_like(P.out, float("nan"))
        P.forward_materialized(ref)
        P.out.fill_(float("nan"))
        P.forward()
        torch.cuda.synchronize()
        got, want = P.out.double(), ref.double()
        assert torch.isfinite(got).all()
        # both are some 8e-7 of the norm from 64 bits
        assert float((got - want).norm()) <= 5e-6 * max(float(want.norm()), 1e-30)
    finally:
        P.close()
