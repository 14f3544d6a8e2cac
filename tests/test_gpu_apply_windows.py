"""Shift-and-sum windows: wide shifts (several windows of eight offsets per
group, list lengths below and above the windows in flight), pixel counts at
the edges of a wave's and a block's tile, every table mode, against the
oracle."""
import numpy as np
import pytest

import workloads as W
from oracle import spectrum as OS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


@pytest.mark.parametrize(
    "precision,contrast,effect,vsini,n_pix,n_regions",
    [
        (W.PREC_FP32, W.CONTRAST_PLANCK, W.EFFECT_TOT, 15.0, 1023, 3),   # paired with contrast
        (W.PREC_FP32, W.CONTRAST_PLANCK, W.EFFECT_FLUX, 0.0, 257, 1),    # one offset pair, few windows
        (W.PREC_FP32, W.CONTRAST_SCALAR, W.EFFECT_TOT, 15.0, 1025, 2),   # split
        (W.PREC_FP32, W.CONTRAST_SCALAR, W.EFFECT_BCONV, 8.0, 255, 2),   # paired without contrast
        (W.PREC_FP32, W.CONTRAST_ARRAY, W.EFFECT_TOT, 4.0, 2049, 4),     # a spot contrast row per bin
        (W.PREC_FP64, W.CONTRAST_ARRAY, W.EFFECT_FLUX, 15.0, 513, 3),
        (W.PREC_FP64, W.CONTRAST_SCALAR, W.EFFECT_TOT, 15.0, 511, 2),
        (W.PREC_FP64, W.CONTRAST_PLANCK, W.EFFECT_BCONV, 8.0, 129, 1),
    ],
)
def test_windows_match_the_oracle_in_every_shape(precision, contrast, effect, vsini, n_pix, n_regions):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[windows] prec {precision} contrast {contrast} effect {effect} vsini {vsini} P {n_pix}", flush=True)
    star = W.make_tiny(41, n_grid=24, n_pix=n_pix, n_mu=3, precision=precision, contrast_mode=contrast, n_phases=19,
                       vsini_kms=vsini, n_regions=n_regions)
    ctx = L.soap_grid_init(star)
    dt = torch.float32 if precision == W.PREC_FP32 else torch.float64
    pcs = (0, 8, 16) if precision == W.PREC_FP32 else (0, 4, 8)
    ref = None
    for pc in pcs:
        for depth in (2, 3):
            L.soap_set_apply_shape(ctx, depth, 0, pc)
            out = torch.full((len(star.phases) + 1, n_pix), 7.0, dtype=dt, device="cuda")
            L.soap_active_spectra(ctx, star.regions, star.phases, effect, out[:-1])
            got = out.cpu().numpy()
            assert np.all(got[-1] == 7.0)  # nothing past the last row
            if ref is None:
                ref = got
                tol = 1e-6 if precision == W.PREC_FP32 else 1e-9
                for p in range(0, len(star.phases), 3):
                    f = OS.integrated(star, star.phases[p], effect)
                    e = np.max(np.abs(got[p] - f) / np.maximum(np.abs(f), 1e-3 * np.abs(f).max()))
                    assert e <= tol, (p, e)
            else:
                np.testing.assert_array_equal(got, ref, err_msg=f"pc {pc}, depth {depth}")
    L.soap_destroy(ctx)
