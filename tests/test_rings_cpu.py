"""Rings from colatitudes (CPU only): the oracle's ring grid pinned to its definition, and the
library's ring prep (tc_rings_from_beta, run on the host) equal to it bit for bit.

Reading of the paper: the problem is stated on colatitudes beta_j (Sec. 4.1); the ring is
x_j = cos(beta_j) rounded once to double (Sec. 4.2.2 precomputes cos(beta) per ring); rings j
and k = nring-1-j whose colatitudes add up to pi to within 2^-48 are an exact mirror pair
(Sec. 4.2.3), the one with the larger colatitude taking exactly -x of the other.
"""
import mpmath as mp
import numpy as np
import pytest

from paper_1002_1050_amd import synthetic as S

TOL = mp.mpf(2) ** -48


def grids():
    rng = np.random.Generator(np.random.PCG64(48))
    pi_l = np.arccos(np.longdouble(-1.0))
    out = {f"equispaced {n}": S.ring_colatitudes(n) for n in (1, 2, 3, 4, 129, 2048, 8192, 16384)}
    for n in (7, 1000):
        j = np.arange(n, dtype=np.longdouble)
        out[f"long-double grid {n}"] = (pi_l * (j + np.longdouble(0.5)) / n).astype(np.float64)
        out[f"with poles {n}"] = (pi_l * j / (n - 1)).astype(np.float64)
    out["descending"] = S.ring_colatitudes(64)[::-1].copy()
    out["shifted (no pairs)"] = S.ring_colatitudes(64) + 1e-9
    out["random"] = np.sort(rng.uniform(0.0, np.pi, 500))
    near = S.ring_colatitudes(40)
    near[3] = np.pi - near[36] + 2.0 ** -47      # gap 2^-47: not a pair
    near[5] = np.pi - near[34] + 2.0 ** -50      # gap about 2^-50: a pair
    out["near the bound"] = near
    return out


def exact_pairs(beta):
    """(j, k) with |beta_j + beta_k - pi| <= 2^-48, in exact arithmetic; checks that no gap
    lies so close to the bound that long double could decide it differently."""
    mp.mp.dps = 60
    n = beta.size
    pairs = []
    for j in range(n // 2):
        k = n - 1 - j
        gap = abs(mp.mpf(float(beta[j])) + mp.mpf(float(beta[k])) - mp.pi)
        assert abs(gap - TOL) > mp.mpf(2) ** -60, "test grid too close to the pairing bound"
        if gap <= TOL:
            pairs.append((j, k))
    return pairs


@pytest.mark.parametrize("name", list(grids()))
def test_oracle_ring_grid_follows_its_definition(orc, name):
    beta = grids()[name]
    x = orc.ring_grid_x(beta)
    plain = orc.ring_x(beta)            # cos rounded once, pinned against mpmath
    paired = set()
    for j, k in exact_pairs(beta):
        lo, hi = (j, k) if beta[k] >= beta[j] else (k, j)
        assert x[lo] == plain[lo] and x[hi] == -plain[lo]
        paired |= {j, k}
    rest = [i for i in range(beta.size) if i not in paired]
    assert np.array_equal(x[rest], plain[rest])


def test_equispaced_grids_pair_every_ring(orc):
    for n in (2048, 8192, 16384):
        assert len(exact_pairs(S.ring_colatitudes(n))) == n // 2
    assert exact_pairs(S.ring_colatitudes(64) + 1e-9) == []


@pytest.mark.parametrize("name", list(grids()))
def test_library_rings_equal_the_oracle(orc, name):
    from paper_1002_1050_amd import _binding as B
    beta = grids()[name]
    got = B.rings_from_beta(beta)
    ref = orc.ring_grid_x(beta)
    assert got.tobytes() == ref.tobytes()


@pytest.mark.parametrize("name", ["random", "equator", "table points", "poles", "midpoints", "descending pairs"])
def test_ring_cosines_equal_long_double_rounded_once(orc, name):
    """The library's own cosine against the oracle's, where its rounding is hardest to be sure of: many
    random colatitudes, the equator (tiny cosines), its table's points k/32 and their midpoints, the poles."""
    from paper_1002_1050_amd import _binding as B
    rng = np.random.Generator(np.random.PCG64(32))
    k = np.arange(101)
    beta = {
        "random": rng.uniform(0.0, np.pi, 200001),
        "equator": np.pi / 2 + np.concatenate([np.linspace(-1e-3, 1e-3, 20001), 2.0 ** -np.arange(1, 60), [0.0]]),
        "table points": np.concatenate([k / 32.0, np.nextafter(k[1:] / 32.0, 0.0), np.nextafter(k[:100] / 32.0, 4.0)]),
        "poles": np.concatenate([np.linspace(0.0, 1e-3, 5001), 2.0 ** -np.arange(1.0, 1070.0, 7.0),
                                 np.pi - np.linspace(0.0, 1e-6, 5001), [np.nextafter(np.pi, 0.0)]]),
        "midpoints": (k[:100] + 0.5) / 32.0,
        "descending pairs": S.ring_colatitudes(3001)[::-1].copy(),
    }[name]
    assert B.rings_from_beta(beta).tobytes() == orc.ring_grid_x(beta).tobytes()
