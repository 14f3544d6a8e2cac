"""CCFs of more than 512 velocities, several to a thread: large calls (blocks of
eight spectra) and batches against the oracle, in both precisions; batches bit
for bit the single calls."""
import numpy as np
import pytest

import workloads as W
from oracle import ccf as OC

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")

C_KMS = 299792.458


@pytest.mark.parametrize("prec", [W.PREC_FP32, W.PREC_FP64])
@pytest.mark.parametrize("n_v,hole_px,n_spec", [(513, 0.9, 701), (577, 3.0, 704), (768, 1.4, 640)])
def test_large_calls_and_batches_match_oracle(prec, n_v, hole_px, n_spec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[ccf-wide] prec {prec} n_v {n_v} hole {hole_px} px spectra {n_spec}", flush=True)
    n_pix, n_lines = 2000, 70  # three line blocks: at least 240 blocks of three waves or more
    star = W.make_tiny(53, n_grid=8, n_pix=n_pix, n_mu=2, precision=prec, n_phases=1)
    ctx = L.soap_grid_init(star)
    rng = np.random.default_rng(n_v)
    px_kms = C_KMS * star.dln_lambda
    dv = 200.0 * px_kms / (n_v - 1)
    v0 = -0.5 * dv * (n_v - 1)
    q = np.sort(rng.uniform(-20.0, n_pix + 20.0, n_lines))
    mask = W.Mask(star.ln_lambda0 + (q - 0.5) * star.dln_lambda, rng.uniform(0.5, 1.5, n_lines),
                  0.5 * hole_px * px_kms, v0, dv, n_v)
    dt = np.float64 if prec == W.PREC_FP64 else np.float32
    flux = rng.uniform(0.2, 1.0, (n_spec, n_pix)).astype(dt)
    ccf = torch.full((n_spec + 1, n_v), -7.0, dtype=torch.float64, device="cuda")
    L.soap_ccf_rv(ctx, torch.from_numpy(flux).cuda(), mask, ccf_out=ccf[:n_spec])
    got = ccf.cpu().numpy()
    assert np.all(got[-1] == -7.0)
    rows = [0, 7, 8, n_spec // 2, n_spec - 1]

    def off(got, flux):
        ref = OC.ccf(flux.astype(np.float64), star.ln_lambda0, star.dln_lambda, mask.ln_lambda, mask.weight,
                     mask.half_width_kms, W.make_velocity_grid(v0, dv, n_v))
        return np.max(np.abs(got - ref) / np.abs(ref))

    # FP64: hole edges differ by ~1e-10 pixel.  FP32: partials of at most 32
    # lines x 10 pixels, each FMA within 2^-24 of the running positive sum
    tol = 1e-9 if prec == W.PREC_FP64 else 2e-5
    assert off(got[rows], flux[rows]) < tol
    # the work-list form, on spectra that the batch makes itself
    regs = [W.Region(W.SPOT, 20.0, 40.0, 0.2, 0.6)]
    out = torch.empty((17, n_pix), dtype=torch.float64 if prec == W.PREC_FP64 else torch.float32, device="cuda")
    cb = torch.empty((17, n_v), dtype=torch.float64, device="cuda")
    b = L.soap_batch_create([ctx], [regs], [np.linspace(0.0, 0.9, 17)], W.EFFECT_TOT, [out], mask=mask, ccf_outs=[cb])
    L.soap_batch_run(b)
    torch.cuda.synchronize()
    one = torch.empty((17, n_v), dtype=torch.float64, device="cuda")
    L.soap_ccf_rv(ctx, out, mask, ccf_out=one)
    assert torch.equal(cb, one)
    assert off(cb.cpu().numpy()[:3], out.cpu().numpy()[:3]) < tol
    L.soap_batch_destroy(b)
    L.soap_destroy(ctx)
