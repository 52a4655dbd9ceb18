"""The sky gradients of the summed polarised adjoint asked for alone: bit for bit those of a scalar adjoint
that forms both gradients; a scalar adjoint of the sky alone may form one sum per column instead of
two, which changes the rounding only (both within a few times 1e-15 of the exact gradient, bound 1e-13)."""
import pytest

from paper_1002_1050_amd import synthetic as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M,nring", [(40, 3, 61), (180, 5, 700)])
def test_summed_sky_gradients_alone(L, M, nring):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1002_1050_amd import _binding as B

    def dev(a):
        return torch.from_numpy(a).to("cuda")

    beta = S.ring_colatitudes(nring)
    alms = [dev(S.sky_alm(L, 1 + p)) for p in range(3)]
    blms = [dev(S.beam_blm(L, M, 300.0, 0.1 * p)) for p in range(2)] + [dev(S.random_beam(L, M, 4))]
    G = dev(S.random_cbar(L, M, nring, 5))
    print(f"[gpu] totalconv_adj_pol, summed, sky alone: L={L} M={M} nring={nring}", flush=True)
    ga, _ = B.totalconv_adj_pol(L, M, beta, alms, blms, [G], B.TC_POL_SUM, True, False)
    for p in range(3):
        both, _ = B.totalconv_adj(L, M, beta, alms[p], blms[p], G)
        alone, _ = B.totalconv_adj(L, M, beta, alms[p], blms[p], G, True, False)
        assert torch.equal(ga[p], both), p
        assert float(torch.linalg.vector_norm(alone - both) / torch.linalg.vector_norm(both)) <= 1e-13, p
