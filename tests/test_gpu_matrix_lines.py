"""The full matrix where its store pieces begin and end: l around the rows a workgroup owns (112), walks
(128) and the steps it gathers (128, 144 with those held back), and outputs that start anywhere
within a line.  Every element against the oracle, and nothing outside the output is written.

Gate: 1e-12 absolute up to l = 300, the repository's gate for this size."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

RINGS = np.array([0.37, -0.81, 1.0, 2.0 ** -30])


@pytest.mark.parametrize("l, offset", [(3, 1), (15, 0), (16, 5), (111, 3), (112, 0), (113, 15), (126, 7), (127, 2), (128, 9),
                                       (143, 4), (144, 12), (223, 6), (224, 11), (239, 14), (240, 8), (257, 13)])
def test_every_element_at_any_alignment(l, offset):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    from paper_1002_1050_amd import _binding as B
    n, w = RINGS.size, 2 * l + 1
    print(f"[gpu] matrix lines l={l} offset={offset}", flush=True)
    buf = torch.full((offset + n * w * w + 16,), float("nan"), dtype=torch.float64, device="cuda")
    out = buf[offset:offset + n * w * w].view(n, w, w)
    B.wigner_d_matrix_x(l, RINGS, out=out)
    got = out.cpu().numpy()
    assert torch.isnan(buf[:offset]).all() and torch.isnan(buf[offset + n * w * w:]).all()
    m = np.repeat(np.arange(-l, l + 1), w)
    mp = np.tile(np.arange(-l, l + 1), w)
    ref = oracle.wigner_d(l, m, mp, RINGS)[:, l, :].T.reshape(n, w, w)
    assert np.abs(got - ref).max() <= 1e-12
