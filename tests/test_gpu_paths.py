"""Kernel variants at the edges of their tiles and dispatch rules, against the oracle."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import spai_oracle as O
from paper_2511_09753_amd import workloads as W
from tests.helpers import oracle_rule, require_gpu

pytestmark = pytest.mark.gpu


def _spai():
    require_gpu()
    from paper_2511_09753_amd import spai as S
    S.load()
    return S


def _random_symmetric(n, per_row, seed):
    rng = np.random.default_rng(seed)
    m = n * per_row // 2
    r, c, v = rng.integers(0, n, m), rng.integers(0, n, m), rng.standard_normal(m)
    U = sp.triu(sp.coo_matrix((v, (r, c)), shape=(n, n)).tocsr(), 1)
    A = (U + U.T + sp.diags(rng.standard_normal(n))).tocsr()
    A.sort_indices()
    return A


@pytest.mark.parametrize("n,steps,per_row", [
    (1, 1, 0), (2, 2, 2), (255, 63, 6), (256, 64, 6), (257, 65, 40), (300, 130, 6),
    (1025, 68, 9)])
def test_lanczos_passes_at_tile_edges(n, steps, per_row):
    """Rows around a 256-row tile, basis vectors around the 64 a workgroup takes at once,
    rows of up to about 40 entries (four lanes share one).  Both sides run the same
    process in float64 and differ by the order of their sums: 1e-9 of the spectral scale."""
    S = _spai()
    A = _random_symmetric(n, per_row, n)
    v0 = np.random.default_rng(steps).standard_normal(n)
    g = S.spectrum(A, v0, steps=steps)
    o = O.lanczos(A, steps, v0)
    scale = max(abs(o[0]), abs(o[1]))
    assert g[4] == o[4]
    assert abs(g[0] - o[0]) <= 1e-9 * scale and abs(g[1] - o[1]) <= 1e-9 * scale
    assert abs(g[2] - o[2]) <= 1e-7 * scale and abs(g[3] - o[3]) <= 1e-7 * scale


def test_lanczos_stops_in_an_invariant_subspace():
    """Three distinct eigenvalues: the process ends after three steps, although the host
    looks only every 64."""
    S = _spai()
    A = sp.diags(np.repeat([1.0, 2.0, 5.0], 200)).tocsr()
    lo, hi, _, _, k = S.spectrum(A, np.random.default_rng(0).standard_normal(600), steps=200)
    assert k == 3
    assert lo == pytest.approx(1.0, rel=1e-12) and hi == pytest.approx(5.0, rel=1e-12)
