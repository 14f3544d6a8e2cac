"""The profile's count of issued operations is what the shift-and-sum kernel's
loop issues: FP32 with eight phases per chunk adds both groups of four at every
offset it walks and forms one difference there (9 operations), with sixteen the
pairs of groups that have a tap; FP64 the pairs of phases with a tap."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")

WINDOW = 8  # offsets of a window: at most so many are walked per offset with a tap


@pytest.mark.parametrize("precision,pc,contrast", [(W.PREC_FP32, 8, W.CONTRAST_PLANCK), (W.PREC_FP32, 8, W.CONTRAST_SCALAR),
                                                   (W.PREC_FP32, 16, W.CONTRAST_PLANCK),
                                                   (W.PREC_FP64, 4, W.CONTRAST_PLANCK)])
def test_issued_operations(precision, pc, contrast):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    # one small spot: visible, and at a chunk's offsets, for part of the phases only
    star = W.make_tiny(71, n_grid=40, n_pix=600, n_mu=4, precision=precision, contrast_mode=contrast, n_phases=64,
                       vsini_kms=10.0, n_regions=1)
    star.regions = [W.Region(W.SPOT, 10.0, 0.0, 0.12, 0.6)]
    ctx = L.soap_grid_init(star)
    L.soap_set_apply_shape(ctx, 2, 0, pc)
    dt = torch.float32 if precision == W.PREC_FP32 else torch.float64
    out = torch.empty((64, star.n_pix), dtype=dt, device="cuda")
    L.soap_profile_enable(ctx, True)
    L.soap_active_spectra(ctx, star.regions, star.phases, W.EFFECT_TOT, out)
    p = L.soap_profile_read(ctx)
    print("[issued]", precision, pc, contrast, {k: p[k] for k in ("taps_nonzero", "taps_offsets", "fma_issued")}, flush=True)
    issued, taps, offs = p["fma_issued"], p["taps_nonzero"], p["taps_offsets"]
    diff = 0 if contrast == W.CONTRAST_SCALAR else 1  # split tables form none
    if pc == 8 and precision == W.PREC_FP32:
        assert issued % (8 + diff) == 0
        walked = issued // (8 + diff)
        assert walked >= offs and 8 * walked >= taps
        assert walked > offs or 8 * offs > taps
    elif pc == 16:
        # every walked offset, and 8 operations per pair of groups with a tap
        assert offs + 8 * offs <= issued <= 17 * (offs * WINDOW)
        assert issued - taps >= offs
    else:
        assert issued >= taps + offs and issued <= 2 * taps + offs * WINDOW
    L.soap_destroy(ctx)
