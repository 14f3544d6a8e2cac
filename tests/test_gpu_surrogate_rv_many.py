"""Surrogate RVs of many samples and few components, whose spreads take blocks
of fewer waves: the RVs and records of calls of a few samples bit for bit, and
their spreads to the rounding of the sums, which add in another order."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


@pytest.mark.parametrize(
    "n,k,E,n_v",
    [
        (4097, 64, 3, 161),  # two waves, the fewest samples; the last block has one
        (4110, 17, 16, 31),
        (8193, 32, 9, 201),  # one wave
        (8200, 5, 8, 49),
    ],
)
def test_many_samples_equal_few(n, k, E, n_v):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-rv-many] n {n} k {k} E {E} n_v {n_v}", flush=True)
    rng = np.random.default_rng(n)
    star = W.make_tiny(3, n_grid=24, n_pix=900, precision=W.PREC_FP32)
    ctx = L.soap_grid_init(star)
    dv = 24.0 / (n_v - 1)
    mask = W.Mask(star.mask.ln_lambda, star.mask.weight, 0.3, -12.0, dv, n_v)
    # the context's velocity grid is the last mask's
    L.soap_ccf_rv(ctx, torch.ones(1, star.n_pix, device="cuda"), mask,
                  ccf_out=torch.empty(1, n_v, dtype=torch.float64, device="cuda"))
    v = W.make_velocity_grid(-12.0, dv, n_v)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    base = dev(np.stack([10.0 - 4.0 * np.exp(-0.5 * ((v - x) / 3.0) ** 2) for x in (0.3, -0.7)]))
    basis = dev(0.02 * np.stack([np.sin(2 * np.pi * (j % 9 + 1) * v / 24.0 + j) for j in range(k)]) / np.sqrt(k))
    coef = rng.normal(size=(n, k)).astype(np.float32)
    mem = (coef[None] + 0.05 * rng.normal(size=(E, n, k))).astype(np.float32)
    rows = rng.integers(0, 2, n).astype(np.int32)

    def call(a, b):
        m = b - a
        rv, err = (torch.empty(m, dtype=torch.float64, device="cuda") for _ in range(2))
        fb = torch.empty(m, dtype=torch.int32, device="cuda")
        rec = torch.empty(m * L.RV_DTYPE.itemsize, dtype=torch.uint8, device="cuda")
        L.soap_surrogate_rv(ctx, dev(coef[a:b]), dev(mem[:, a:b]), base, basis, 1.5, 1e9, rv, fb, err_kms=err,
                            rv_out=rec, base_index=dev(rows[a:b]))
        return rv.cpu().numpy(), err.cpu().numpy(), fb.cpu().numpy(), rec.cpu().numpy().reshape(m, -1)

    rv, err, fb, rec = call(0, n)
    assert np.all(np.isfinite(err)) and not fb.any()
    for a, b in ((0, 40), (n // 2 - 3, n // 2 + 30), (n - 17, n)):
        r, e, f, c = call(a, b)
        assert np.array_equal(rv[a:b], r) and np.array_equal(fb[a:b], f) and np.array_equal(rec[a:b], c)
        # 64 x 201 terms in double whose sums cancel by less than 1e3
        np.testing.assert_allclose(err[a:b], e, rtol=1e-10)
    L.soap_destroy(ctx)
