"""Calls of more than 2^32 work items: one launch holds fewer, so they take several, and every
element is written.  The matrix at l = 1 on 4194303 + 700 rings (one launch takes 4194303): equal
bit for bit, around the launches' border and at the end, to calls on those rings alone.  wigner_d_rings
at l = 0 of 4200000 pairs on 1000 rings (one launch takes 4194303 pairs): d^0_00 = 1 everywhere."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1002_1050_amd import _binding
    _binding.lib()
    yield _binding
    torch.cuda.empty_cache()


def test_matrix_on_many_rings(B):
    n = 4194303 + 700
    x = np.random.Generator(np.random.PCG64(7)).uniform(-1.0, 1.0, n)
    out = torch.full((n, 3, 3), float("nan"), dtype=torch.float64, device="cuda")
    print(f"[gpu] wigner_d_matrix l=1 nring={n}", flush=True)
    B.wigner_d_matrix_x(1, x, out=out)
    assert bool(torch.isfinite(out).all())
    for j in (0, 4194303 - 100, 4194303, n - 100):
        assert torch.equal(out[j:j + 100], B.wigner_d_matrix_x(1, x[j:j + 100])), j


def test_wigner_rings_of_many_pairs(B):
    npair, n = 4200000, 1000
    x = np.random.Generator(np.random.PCG64(8)).uniform(-1.0, 1.0, n)
    zero = np.zeros(npair, np.int32)
    out = torch.full((npair, n), float("nan"), dtype=torch.float64, device="cuda")
    ws = torch.empty(B.workspace_bytes_x(B.TC_OP_WIGNER, 0, npair, x), dtype=torch.uint8, device="cuda")
    print(f"[gpu] wigner_d_rings lmax=0 npair={npair} nring={n}", flush=True)
    rc = B.lib().wigner_d_rings_x(0, npair, B._hptr(zero), B._hptr(zero), n, B._hptr(x), B._dptr(out), B._dptr(ws),
                                  ctypes.c_size_t(ws.numel()), B._stream_handle(torch, out.device))
    assert rc == 0, B.last_error()
    ones = 0
    for k in range(0, npair, 600000):
        ones += int((out[k:k + 600000] == 1.0).sum())
    assert ones == npair * n
