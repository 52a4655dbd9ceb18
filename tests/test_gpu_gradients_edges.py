"""Both adjoint gradients at lmax beside the 64 values of l of a beam tile and the eight rows its waves take,
with mbmax 0 to lmax, against the oracle; and the sky gradient of the launch that makes both against the one
made alone, for a beam whose rows are unrelated (both then add the same terms in the same order)."""
import numpy as np
import pytest

from paper_1002_1050_amd import synthetic as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-11   # of the gradient's norm, as for every gradient here


@pytest.mark.parametrize("L, M", [(0, 0), (1, 1), (7, 3), (8, 0), (62, 5), (63, 63), (64, 2), (65, 1), (127, 4),
                                  (128, 3), (161, 2)])
def test_gradients_at_tile_edges(L, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_1002_1050_amd import _binding as B
    nring = 19
    x = S.ring_cosines(nring)
    alm, blm, G = S.sky_alm(L, 5), S.random_beam(L, M, 6), S.random_cbar(L, M, nring, 7)
    print(f"[gpu] gradients at tile edges L={L} M={M}", flush=True)
    dev = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (alm, blm, G)]
    ga, gb = B.totalconv_adj_x(L, M, x, *dev)
    ra, rb = oracle.totalconv_adj(L, M, x, alm, blm, G)
    for got, ref in ((ga, ra), (gb, rb)):
        got = got.cpu().numpy()
        assert np.isfinite(got).all()
        assert np.linalg.norm(got - ref) <= TOL * max(np.linalg.norm(ref), 1e-300)
    alone, _ = B.totalconv_adj_x(L, M, x, *dev, want_blm=False)
    assert torch.linalg.vector_norm(alone - ga) <= TOL * torch.linalg.vector_norm(ga)
