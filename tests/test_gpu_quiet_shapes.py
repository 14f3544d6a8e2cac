"""Quiet spectrum and padded rows at the edges of their kernels: one and many
bins, disks of more than one LDS pass of columns, no rotation (one offset),
wide rotation (several runs of offsets per bin), pixel counts off every block;
device spectra, copied in one pass, give what host spectra give, and a
non-finite value in any row is found."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle import spectrum as OS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


def _quiet(star, dt):
    ctx = L.soap_grid_init(star)
    q = torch.empty(star.n_pix, dtype=dt, device="cuda")
    L.soap_quiet_spectrum(ctx, q)
    a = torch.empty(len(star.phases), star.n_pix, dtype=dt, device="cuda")
    L.soap_active_spectra(ctx, star.regions, star.phases, W.EFFECT_TOT, a)
    torch.cuda.synchronize()
    L.soap_destroy(ctx)
    return q.cpu().numpy(), a.cpu().numpy()


@pytest.mark.parametrize(
    "precision,n_grid,n_pix,n_mu,vsini",
    [
        (W.PREC_FP32, 2, 257, 1, 0.0),
        (W.PREC_FP32, 65, 1023, 20, 12.0),
        (W.PREC_FP32, 1030, 300, 3, 1.0),   # two passes over the columns
        (W.PREC_FP64, 33, 1025, 7, 15.0),
        (W.PREC_FP64, 1025, 256, 2, 0.3),
    ],
)
def test_quiet_and_rows(precision, n_grid, n_pix, n_mu, vsini):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[quiet] prec {precision} N {n_grid} P {n_pix} B {n_mu} vsini {vsini}", flush=True)
    star = W.make_tiny(61, n_grid=n_grid, n_pix=n_pix, n_mu=n_mu, precision=precision, n_phases=2, vsini_kms=vsini,
                       contrast_mode=W.CONTRAST_PLANCK)
    dt = torch.float32 if precision == W.PREC_FP32 else torch.float64
    host, act = _quiet(star, dt)
    want = OS.quiet(star)
    # FP32: column sums in Kahan FP32 (2^-24 per cell weight), rows and result
    # rounded to FP32; FP64: sums of positive terms
    tol = 1e-6 if precision == W.PREC_FP32 else 1e-9
    assert np.max(np.abs(host - want) / np.maximum(np.abs(want), 1e-3 * np.abs(want).max())) <= tol
    dev = dataclasses.replace(star, spectra=[None if s is None else torch.from_numpy(np.ascontiguousarray(s)).cuda()
                                             for s in star.spectra])
    q, a = _quiet(dev, dt)
    np.testing.assert_array_equal(q, host)
    np.testing.assert_array_equal(a, act)
    for t in range(3):
        if dev.spectra[t] is None:
            continue
        for m in (0, n_pix - 1):
            bad = [None if s is None else s.clone() for s in dev.spectra]
            bad[t][n_mu - 1, m] = float("inf")
            with pytest.raises(L.SoapError):
                L.soap_grid_init(dataclasses.replace(dev, spectra=bad))
