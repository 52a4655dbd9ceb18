"""Data cube: the alpha pass over pairs of mb and of alpha, at numbers of alpha around its 4, 8 and 16 slots
(odd and even, with and without alpha = pi), and at mbmax beside the number of values read together."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


@pytest.mark.parametrize("M", [0, 1, 3, 4, 9])
@pytest.mark.parametrize("Na", [1, 2, 7, 8, 9, 16, 17, 31, 32, 33, 64, 65])
def test_cube_alpha_pairs(orc, M, Na):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1002_1050_amd import _binding as B
    print("cube alpha pairs", M, Na, flush=True)
    L, n, Ng = 11, 17, 32
    rng = np.random.Generator(np.random.PCG64(100 * M + Na))
    C = rng.standard_normal((2 * M + 1, L + 1, n)) + 1j * rng.standard_normal((2 * M + 1, L + 1, n))
    got = B.totalconv_datacube(L, M, torch.from_numpy(C).cuda(), Na, Ng).cpu().numpy()
    ref = orc.datacube(L, M, C, Na, Ng)
    # every one of the (2M+1)(2L+1) terms is rounded at most 2M + 1 + 4 log2(ngamma) times on its way
    bound = EPS * (2 * M + 5 + 4 * np.log2(Ng)) * 2 * np.abs(C).sum(axis=(0, 1))
    assert (np.abs(got - ref).reshape(n, -1).max(axis=1) <= bound).all()
