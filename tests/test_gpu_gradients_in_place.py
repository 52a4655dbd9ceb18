"""totalconv_adj through the C ABI with the beam gradient written over the beam it is taken at: both
gradients equal those written beside their inputs, bit for bit (the sky gradient reads the beam
before the beam gradient replaces it)."""
import pytest

from paper_1002_1050_amd import synthetic as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,M,nring", [(5, 2, 4), (64, 4, 130), (300, 9, 601)])
def test_beam_gradient_over_the_beam(L, M, nring):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1002_1050_amd import _binding as B

    def dev(a):
        return torch.from_numpy(a).to("cuda")

    beta = S.ring_colatitudes(nring)
    alm, blm = dev(S.sky_alm(L, 1)), dev(S.random_beam(L, M, 2))
    G = dev(S.random_cbar(L, M, nring, 3))
    print(f"[gpu] totalconv_adj, blm_bar over blm: L={L} M={M} nring={nring}", flush=True)
    want_a, want_b = B.totalconv_adj(L, M, beta, alm, blm, G)
    over, got_a = blm.clone(), torch.empty_like(alm)
    ws = torch.empty(B.workspace_bytes(B.TC_OP_ADJ, L, M, beta), dtype=torch.uint8, device="cuda")
    rc = B.lib().totalconv_adj(L, M, nring, B._hptr(beta), B._dptr(alm), B._dptr(over), B._dptr(G), B._dptr(got_a),
                               B._dptr(over), B._dptr(ws), ws.numel(), B._stream_handle(torch, alm.device))
    assert rc == 0, B.last_error()
    assert torch.equal(got_a, want_a) and torch.equal(over, want_b)
