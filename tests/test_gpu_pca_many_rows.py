"""PCA projections of many rows of few pixels, where each wave takes a row tile
of its own: at the edges of its tiles, its steps of 16 pixels and its groups of
four components, against the oracle in 64 bits; and rows without a centre.
"""

import numpy as np
import pytest

from oracle import surrogate as OSG

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


@pytest.mark.parametrize(
    "n,P,k",
    [
        (160, 1, 1),         # one pixel of one component, the last block with two tiles
        (1681, 15, 3),       # no whole step; one row past the tiles
        (1601, 16, 66),      # one whole step, four components that begin before the second tile
        (2047, 17, 4),       # one pixel past it
        (5309, 47, 63),
        (16385, 161, 130),   # ten steps, three component tiles
    ],
)
def test_many_rows_of_few_pixels(n, P, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[pca-rows] n {n} P {P} k {k}", flush=True)
    rng = np.random.default_rng(n + P + k)
    D = rng.normal(1.0, 0.1, (n, P + 3)).astype(np.float32)
    M = rng.normal(1.0, 0.1, (3, P)).astype(np.float32)
    idx = rng.integers(0, 3, n).astype(np.int32)
    V = rng.normal(0.0, 1.0, (P, k)).astype(np.float32)
    coef = torch.full((n + 1, k), 7.0, dtype=torch.float32, device="cuda")
    L.soap_pca_project(_dev(D), _dev(M), _dev(V), coef[:n], mean_index=torch.from_numpy(idx).cuda(), n_pix=P)
    got = coef.cpu().numpy()
    d = D[:, :P].astype(np.float64) - M[idx].astype(np.float64)
    want = OSG.pca_project(d, np.zeros(P), V.astype(np.float64))
    tol = 4.0 * P * 2.0**-24 * np.abs(d).max() * np.abs(V).max()
    assert np.abs(got[:n] - want).max() <= tol
    assert np.all(got[n] == 7.0)  # nothing past the last row
    bad = idx.copy()
    bad[n - 1] = 3
    bad[0] = -1
    L.soap_pca_project(_dev(D), _dev(M), _dev(V), coef[:n], mean_index=torch.from_numpy(bad).cuda(), n_pix=P)
    again = coef.cpu().numpy()
    assert np.all(np.isnan(again[[0, n - 1]]))
    np.testing.assert_array_equal(again[1:n - 1], got[1:n - 1])
