"""Synthesis calls enqueued one after another without a wait (their table
kernels then run beside the pending work, in rotating table sets and
parameter slots) give bit for bit what the same calls give one at a time, for
region counts and phase counts at the edges of the parameter kernel's lanes
and blocks; both agree with the oracle.  A captured stream is refused."""
import numpy as np
import pytest

import workloads as W
from oracle import spectrum as OS

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


@pytest.mark.parametrize(
    "precision,n_regions,n_phases,diff_rot",
    [
        (W.PREC_FP32, 1, 1, 0.0),
        (W.PREC_FP32, 3, 129, 0.0),    # four lanes per phase, last block ragged
        (W.PREC_FP32, 33, 5, 0.0),     # a wave per phase
        (W.PREC_FP64, 64, 3, 0.0),
        (W.PREC_FP64, 5, 17, 0.25),
    ],
)
def test_enqueued_calls_match_single_calls(precision, n_regions, n_phases, diff_rot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[queue] prec {precision} regions {n_regions} phases {n_phases} diff_rot {diff_rot}", flush=True)
    star = W.make_tiny(17, n_grid=24, n_pix=2000, n_mu=3, precision=precision, contrast_mode=W.CONTRAST_PLANCK,
                       n_phases=n_phases, vsini_kms=8.0, n_regions=n_regions)
    star.diff_rot = diff_rot
    ctx = L.soap_grid_init(star)
    dt = torch.float32 if precision == W.PREC_FP32 else torch.float64
    rng = np.random.default_rng(n_phases)
    n_calls = 14  # more than the table sets and the parameter slots
    # another set of phases and another part of the region list in every call
    calls = [(star.regions[: 1 + k % n_regions], np.asarray(rng.uniform(0.0, 1.0, n_phases - k % min(3, n_phases))))
             for k in range(n_calls)]
    single = []
    for regions, phases in calls:
        out = torch.empty(len(phases), star.n_pix, dtype=dt, device="cuda")
        L.soap_active_spectra(ctx, regions, phases, W.EFFECT_TOT, out)
        torch.cuda.synchronize()
        single.append(out.cpu().numpy())
    for _ in range(3):
        outs = [torch.full((len(p), star.n_pix), 7.0, dtype=dt, device="cuda") for _, p in calls]
        torch.cuda.synchronize()
        for (regions, phases), out in zip(calls, outs):
            L.soap_active_spectra(ctx, regions, phases, W.EFFECT_TOT, out)
        torch.cuda.synchronize()
        for k, out in enumerate(outs):
            np.testing.assert_array_equal(out.cpu().numpy(), single[k], err_msg=f"call {k}")
    tol = 1e-6 if precision == W.PREC_FP32 else 1e-9
    k = n_regions - 1 if n_regions <= n_calls else n_calls - 1
    star.regions = calls[k][0]
    f = OS.integrated(star, calls[k][1][0], W.EFFECT_TOT)
    e = np.max(np.abs(single[k][0] - f) / np.maximum(np.abs(f), 1e-3 * np.abs(f).max()))
    assert e <= tol, e
    L.soap_destroy(ctx)


def test_capture_is_refused():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    star = W.make_tiny(18, n_grid=24, n_pix=500, n_mu=3, precision=W.PREC_FP32, n_phases=2)
    s = torch.cuda.Stream()
    x = torch.zeros(8, device="cuda")
    with torch.cuda.stream(s):
        ctx = L.soap_grid_init(star)
        out = torch.empty(2, star.n_pix, dtype=torch.float32, device="cuda")
        L.soap_active_spectra(ctx, star.regions, star.phases, W.EFFECT_TOT, out)
    torch.cuda.synchronize()
    ref = out.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        x.add_(1.0)
        with pytest.raises(L.SoapError):
            L.soap_active_spectra(ctx, star.regions, star.phases, W.EFFECT_TOT, out)
    g.replay()
    torch.cuda.synchronize()
    assert torch.all(x == 1.0)
    out.zero_()
    with torch.cuda.stream(s):
        L.soap_active_spectra(ctx, star.regions, star.phases, W.EFFECT_TOT, out)
    torch.cuda.synchronize()
    assert torch.equal(out, ref)
    L.soap_destroy(ctx)
