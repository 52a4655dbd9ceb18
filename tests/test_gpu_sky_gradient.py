"""The sky gradient alone (no beam gradient): columns whose beam rows mb and -mb are equal up to a sign
form one sum instead of two.  Against the oracle, and against the call that returns both gradients.

Tolerance: the two forms add the same terms in another order (d (G + s G') for d G + s d G'), a rounding
apart per term, so both are gated at the repository's 1e-11 of the gradient's norm."""
import numpy as np
import pytest

from paper_1002_1050_amd import synthetic as S

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-11


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1002_1050_amd import _binding
    _binding.lib()
    return _binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def beam(kind, L, M):
    """gauss: real, even rows; signs: odd rows antisymmetric; mixed: some rows unrelated, some zero."""
    if kind == "gauss":
        return S.beam_blm(L, M, 200.0, 0.3)
    b = S.random_beam(L, M, 31)
    if kind == "complex":
        return b
    for m in range(1, M + 1):
        if kind == "signs" or m % 3 == 1:
            b[M - m] = (-1) ** m * b[M + m]
        elif m % 3 == 0:
            b[M - m] = b[M + m] = 0.0
    return b


@pytest.mark.parametrize("kind", ["gauss", "signs", "mixed", "complex"])
@pytest.mark.parametrize("L, M, nring", [(40, 4, 97), (33, 0, 40), (9, 1, 1), (70, 3, 130), (48, 5, 1101),
                                         (24, 3, 2100), (16, 2, 4097), (12, 3, 8192)])
def test_sky_gradient_alone(B, kind, L, M, nring):
    import oracle
    x = S.ring_cosines(nring)
    alm_h, blm_h, G_h = S.sky_alm(L, 41), beam(kind, L, M), S.random_cbar(L, M, nring, 42)
    print(f"[gpu] sky gradient alone L={L} M={M} nring={nring} {kind}", flush=True)
    alm, blm, G = dev(alm_h), dev(blm_h), dev(G_h)
    ga, gb = B.totalconv_adj_x(L, M, x, alm, blm, G, want_blm=False)
    assert gb is None
    both, _ = B.totalconv_adj_x(L, M, x, alm, blm, G)
    ref, _ = oracle.totalconv_adj(L, M, x, alm_h, blm_h, G_h)
    ga = ga.cpu().numpy()
    assert np.linalg.norm(ga - ref) <= TOL * np.linalg.norm(ref)
    assert np.linalg.norm(ga - both.cpu().numpy()) <= TOL * np.linalg.norm(ref)


def test_single_rings_and_polarised_pairs(B):
    """Rings without a mirror partner; three pairs with a cotangent each, sky gradients alone."""
    import oracle
    L, M = 37, 4
    x = np.sort(np.cos(np.linspace(0.1, 1.4, 50)))[::-1].copy()      # one hemisphere: no mirror pairs
    kinds = ["gauss", "mixed", "complex"]
    alm_h = [S.sky_alm(L, 50 + i) for i in range(3)]
    blm_h = [beam(k, L, M) for k in kinds]
    G_h = [S.random_cbar(L, M, x.size, 60 + i) for i in range(3)]
    print("[gpu] sky gradients alone, three pairs", flush=True)
    ga, gb = B.totalconv_adj_pol_x(L, M, x, [dev(a) for a in alm_h], [dev(b) for b in blm_h], [dev(g) for g in G_h],
                                   want_blm=False)
    assert gb == [None] * 3
    for i in range(3):
        ref, _ = oracle.totalconv_adj(L, M, x, alm_h[i], blm_h[i], G_h[i])
        assert np.linalg.norm(ga[i].cpu().numpy() - ref) <= TOL * np.linalg.norm(ref)
