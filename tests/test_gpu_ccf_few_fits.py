"""Calls of few spectra (two spectra a block, more loads in flight) give the CCFs
and the fit records of a large call bit for bit, on both sides of the number of
waves up to which they are taken, for one and seven waves of velocities per
block and two velocities per thread."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")

C_KMS = 299792.458


@pytest.mark.parametrize(
    "prec,n_v,n_few",
    [
        (W.PREC_FP32, 161, (1, 7, 213, 568, 569)),  # three line blocks of three waves: 71 blocks of eight spectra are few
        (W.PREC_FP32, 401, (2, 240, 241)),          # seven waves: 30 blocks of eight are
        (W.PREC_FP64, 161, (3, 568, 569)),
        (W.PREC_FP32, 600, (1, 340)),               # two velocities per thread
    ],
)
def test_ccf_and_fit_of_few_spectra(prec, n_v, n_few):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[ccf-few] prec {prec} n_v {n_v}", flush=True)
    n_pix, n_lines, n_many = 2000, 70, 2400
    star = W.make_tiny(53, n_grid=8, n_pix=n_pix, n_mu=2, precision=prec, n_phases=1)
    ctx = L.soap_grid_init(star)
    rng = np.random.default_rng(n_v)
    dt = torch.float64 if prec == W.PREC_FP64 else torch.float32
    # lines of 4 pixels' width at known places, so that every CCF has a dip and its fit converges
    centre = np.sort(rng.uniform(60.0, n_pix - 60.0, n_lines))
    x = np.arange(n_pix)[:, None] - centre[None, :]
    dip = (0.5 * np.exp(-0.5 * (x / 4.0) ** 2)).sum(axis=1)
    flux = 1.0 - dip[None, :] * rng.uniform(0.5, 1.0, (n_many, 1)) + rng.normal(0.0, 1e-3, (n_many, n_pix))
    flux = torch.from_numpy(flux).to(dt).cuda()
    px_kms = C_KMS * star.dln_lambda
    dv = 46.0 * px_kms / (n_v - 1)
    mask = W.Mask(star.ln_lambda0 + centre * star.dln_lambda, rng.uniform(0.5, 1.5, n_lines), 0.45 * px_kms,
                  -0.5 * dv * (n_v - 1), dv, n_v)

    def run(n):
        ccf = torch.empty(n, n_v, dtype=torch.float64, device="cuda")
        rv = L.rv_records(n)
        L.soap_ccf_rv(ctx, flux[:n], mask, ccf_out=ccf, rv_out=rv)
        torch.cuda.synchronize()
        return ccf, rv

    many, rv_many = run(n_many)
    assert np.all(rv_many["status"] == 0)
    for n in n_few:
        few, rv = run(n)
        assert torch.equal(few, many[:n]), n
        assert rv.tobytes() == rv_many[:n].tobytes(), n
    L.soap_destroy(ctx)
