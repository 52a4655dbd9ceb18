"""Data cube: the builds of the gamma pass at and beside their largest row, rows of alpha sums that
are and are not whole lines, and the larger of the two workspaces against the smaller one."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1002_1050_amd import _binding
    _binding.lib()
    return _binding


# (lmax, mbmax, nring, nalpha, ngamma): half lengths 512 to 8192, lmax + 1 = -1, 0, 1 and 4 modulo 8, rings and
# msky beside a multiple of 16, alpha beside the widths 8, 16 and 32 of the alpha pass
CASES = [(510, 1, 17, 8, 1024), (511, 2, 16, 9, 2048), (1024, 1, 15, 16, 2048), (1023, 0, 3, 17, 4096),
         (1500, 1, 3, 32, 4096), (2048, 1, 2, 33, 8192), (3, 3, 40, 66, 8192), (4095, 0, 2, 2, 8192),
         (8192, 0, 1, 1, 16384)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "L%d_M%d_n%d_a%d_g%d" % c)
def test_cube_rows_against_oracle(B, orc, case):
    L, M, n, Na, Ng = case
    print("cube", case, flush=True)
    rng = np.random.Generator(np.random.PCG64(L + Ng))
    C = rng.standard_normal((2 * M + 1, L + 1, n)) + 1j * rng.standard_normal((2 * M + 1, L + 1, n))
    got = B.totalconv_datacube(L, M, torch.from_numpy(C).cuda(), Na, Ng).cpu().numpy()
    pts = 300
    j, a, g = rng.integers(0, n, pts), rng.integers(0, Na, pts), rng.integers(0, Ng, pts)
    j[:2], a[:2], g[:2] = [0, n - 1], [0, Na - 1], [0, Ng - 1]
    ref = orc.datacube(L, M, C, Na, Ng, points=(j, a, g))
    # each term rounded a few times on the way through mb sums and log2(ngamma) stages: the root sum of squares
    # of the row's terms is at most the largest |c| times a small factor
    tol = 16 * EPS * (2 * M + 1 + np.log2(Ng))
    scale = np.abs(got).reshape(n, -1).max(axis=1)[j]
    assert float((np.abs(got[j, a, g] - ref) / scale).max()) <= tol


def test_cube_smaller_workspace_gives_the_same_cube(B):
    """1.7 GB of alpha sums: one chunk in the workspace asked for now, three in 1.5 GB of the size asked for
    by two chunks of 768 MB; one byte less is refused."""
    L, M, n, Na, Ng = 1022, 1, 3600, 29, 2048
    C = torch.randn((2 * M + 1, L + 1, n), dtype=torch.complex128, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(7))
    lib = B.lib()
    whole = B.totalconv_datacube(L, M, C, Na, Ng)
    out = torch.full_like(whole, float("nan"))
    chunk = ((768 << 20) // (16 * Na * (L + 1))) // 16 * 16
    up = lambda b: -(-b // 256) * 256
    old = up(16 * 32 * (2 * M + 1)) + up(16 * Ng) + 2 * up(16 * Na * (L + 1) * chunk)
    assert old < int(lib.totalconv_datacube_workspace_bytes(L, M, n, Na, Ng))
    ws = torch.empty(old, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert lib.totalconv_datacube(L, M, n, C.data_ptr(), Na, Ng, out.data_ptr(), ws.data_ptr(), old - 1, stream) == -3
    assert lib.totalconv_datacube(L, M, n, C.data_ptr(), Na, Ng, out.data_ptr(), ws.data_ptr(), old, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(whole, out)
