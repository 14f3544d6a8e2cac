"""Surrogate RVs at the edges of the matrix kernels' tiles: sample counts around
16, component counts around one tile, one LDS pass and one block's columns,
velocity grids from less than a group of 16 to several LDS passes, every member
count class.  The mean RV equals the linear fit's bit for bit; the spread is
compared with first-order propagation in numpy at the fitted parameters."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


def _sensitivity(v, y, c0, a, mu, s):
    """dRV/dy of the least-squares fit of c0 - a exp(-(v - mu)^2 / (2 s^2)) to y."""
    q = (v - mu) / s
    e = np.exp(-0.5 * q * q)
    r = c0 - a * e - y
    J = np.stack([np.ones_like(e), -e, -a * e * q / s, -a * e * q * q / s], axis=1)
    H = J.T @ J
    for i, j, d2 in ((1, 2, -e * q / s), (1, 3, -e * q * q / s), (2, 2, -a * e * (q**2 - 1) / s**2),
                     (2, 3, -a * e * (q**3 - 2 * q) / s**2), (3, 3, -a * e * (q**4 - 3 * q**2) / s**2)):
        H[i, j] += r @ d2
        if i != j:
            H[j, i] += r @ d2
    return J @ np.linalg.solve(H, np.array([0.0, 0.0, 1.0, 0.0]))


@pytest.mark.parametrize(
    "n,k,E,n_v",
    [(1, 1, 2, 12), (15, 16, 3, 64), (17, 33, 4, 161), (48, 128, 4, 161), (33, 129, 5, 193), (16, 300, 2, 200),
     (40, 31, 9, 385), (3, 64, 16, 768), (20, 7, 4, 16)],
)
def test_matrix_kernels_at_tile_edges(n, k, E, n_v):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-rv] n {n} k {k} E {E} n_v {n_v}", flush=True)
    rng = np.random.default_rng(1000 * k + n_v)
    star = W.make_tiny(3, n_grid=24, n_pix=900, precision=W.PREC_FP32)
    ctx = L.soap_grid_init(star)
    m = star.mask
    dv = 24.0 / (n_v - 1)
    mask = W.Mask(m.ln_lambda, m.weight, 0.3, -12.0, dv, n_v)
    # the context's velocity grid is the last mask's
    L.soap_ccf_rv(ctx, torch.ones(1, star.n_pix, device="cuda"), mask,
                  ccf_out=torch.empty(1, n_v, dtype=torch.float64, device="cuda"))
    v = W.make_velocity_grid(-12.0, dv, n_v)
    base = np.stack([10.0 - 4.0 * np.exp(-0.5 * ((v - x) / 3.0) ** 2) for x in (0.3, -0.7)])
    basis = 0.02 * np.stack([np.sin(2 * np.pi * (j % 9 + 1) * v / 24.0 + j) for j in range(k)]) / np.sqrt(k)
    coef = rng.normal(size=(n, k)).astype(np.float32)
    mem = (coef[None] + 0.05 * rng.normal(size=(E, n, k))).astype(np.float32)
    rows = rng.integers(0, 2, n).astype(np.int32)
    if n > 1:
        rows[n - 1] = 2  # no such star
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    rv = torch.empty(n, dtype=torch.float64, device="cuda")
    err = torch.empty(n, dtype=torch.float64, device="cuda")
    fb = torch.empty(n, dtype=torch.int32, device="cuda")
    rec = torch.empty(n * L.RV_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
    L.soap_surrogate_rv(ctx, dev(coef), dev(mem), dev(base), dev(basis), 1.5, 1e9, rv, fb, err_kms=err, rv_out=rec,
                        base_index=dev(rows))
    got = np.frombuffer(rec.cpu().numpy().tobytes(), dtype=L.RV_DTYPE)
    for b in (0, 1):
        lin = torch.empty(n * L.RV_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        L.soap_ccf_linear_rv(ctx, dev(coef), dev(base[b]), dev(basis), None, lin)
        ref = np.frombuffer(lin.cpu().numpy().tobytes(), dtype=L.RV_DTYPE)
        np.testing.assert_array_equal(got["rv_kms"][rows == b], ref["rv_kms"][rows == b])
    e_got, f_got = err.cpu().numpy(), fb.cpu().numpy()
    for i in range(n):
        if rows[i] == 2:
            assert np.isinf(e_got[i]) and f_got[i] == 1 and got["status"][i] == 2
            continue
        assert got["status"][i] == 0 and f_got[i] == 0
        y = base[rows[i]] + coef[i].astype(np.float64) @ basis
        g = _sensitivity(v, y, got["c0"][i], got["amp"][i], got["rv_kms"][i], got["sigma_kms"][i])
        d = (mem[:, i].astype(np.float64) - coef[i]) @ (basis @ g)
        # the parameters' distance from the minimum (the fit's stopping rule,
        # about 1e-8) enters the sensitivity to first order
        np.testing.assert_allclose(e_got[i], 1.5 * np.std(d, ddof=1), rtol=1e-5)
    L.soap_destroy(ctx)
