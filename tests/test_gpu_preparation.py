"""The preparation in extra workgroups of the per-tile projection's launch (fp32), at every channel count of that kernel: with
more to prepare than there are atoms and the other way round, against the materialized call, which prepares in a launch of
its own and projects in another kernel."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,C,N,H", [
    (0, 16, 3, 1), (1, 16, 33, 2), (1, 32, 2500, 2), (2, 48, 65, 3), (3, 128, 60, 8), (2, 256, 60, 16), (4, 256, 130, 16),
    (0, 256, 2100, 16),
])
def test_forward_against_the_materialized_call(L, C, N, H):
    import torch
    from paper_2601_16622_amd import binding as B, workloads as W
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    rng = np.random.default_rng(N)
    cfg = dict(L=L, C=C, H=H, B=8, lf=min(1, L), cutoff=4.0, dtype="f32")
    pos = (rng.random((N, 3)) * (N / 0.1) ** (1.0 / 3.0)).astype(np.float32)   # (3 atoms: within each other's reach)
    P = B.Problem(W._pack(cfg, [pos], rng, elements=False))
    try:
        P.build_cells()
        ref = torch.full_like(P.out, float("nan"))
        P.forward_materialized(ref)
        P.attn_ws.fill_(255)   # nothing prepared by the call above is found again
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
