"""Polarised pairs with separate outputs on columns where every pair's beam rows mb and -mb are related by
a sign (the even / odd form), where some are, and where none is: each output against the oracle.

Tolerance: the repository's gate of 1e-11 of a column's largest value, as for the scalar forward, whose
sums these are."""
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


def beam(kind, L, M, seed):
    """even / odd: row -mb = +- row mb; zero: no rows but mb = 0; some: unrelated rows at mb = +-1 only."""
    b = S.random_beam(L, M, seed)
    for m in range(1, M + 1):
        if kind == "even" or (kind == "some" and m > 1):
            b[M - m] = b[M + m]
        elif kind == "odd":
            b[M - m] = -b[M + m]
        elif kind == "zero":
            b[M - m] = b[M + m] = 0.0
    return b


@pytest.mark.parametrize("kinds", [("even", "even", "odd"), ("even", "zero", "odd"), ("some", "even", "odd"),
                                   ("complex", "even", "odd"), ("complex", "complex", "complex"), ("odd", "even"),
                                   ("complex", "odd")])
@pytest.mark.parametrize("L, M, nring", [(40, 3, 61), (21, 0, 30), (70, 2, 1101), (24, 4, 2100), (10, 1, 1)])
def test_separate_outputs(B, kinds, L, M, nring):
    import oracle
    x = S.ring_cosines(nring)
    alm_h = [S.sky_alm(L, 70 + i) for i in range(len(kinds))]
    blm_h = [beam(k, L, M, 80 + i) for i, k in enumerate(kinds)]
    print(f"[gpu] polarised rows L={L} M={M} nring={nring} {kinds}", flush=True)
    outs = B.totalconv_fwd_pol_x(L, M, x, [dev(a) for a in alm_h], [dev(b) for b in blm_h])
    for i in range(len(kinds)):
        got = outs[i].cpu().numpy().reshape(-1, nring)
        ref = oracle.totalconv_fwd(L, M, x, alm_h[i], blm_h[i]).reshape(-1, nring)
        num, den = np.abs(got - ref).max(axis=1), np.abs(ref).max(axis=1)
        assert np.all(num[den == 0] == 0)
        assert np.all(num[den > 0] <= TOL * den[den > 0]), kinds[i]
