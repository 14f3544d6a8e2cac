"""CCF against the oracle at velocity counts around the block sizes: whole
waves and one past them, the last grid with one velocity per thread and the
first with two, the widest; narrow and wide stages, one spectrum and a
remainder of the spectra per block."""
import numpy as np
import pytest

import workloads as W
from oracle import ccf as OC

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")

C_KMS = 299792.458


@pytest.mark.parametrize(
    "prec,n_v,hole_px,span_px,n_spec",
    [
        (W.PREC_FP32, 192, 0.9, 60.0, 9),
        (W.PREC_FP32, 193, 0.9, 60.0, 1),
        (W.PREC_FP32, 449, 1.4, 120.0, 8),
        (W.PREC_FP32, 512, 0.9, 300.0, 3),
        (W.PREC_FP32, 513, 0.9, 130.0, 10),
        (W.PREC_FP32, 768, 3.0, 400.0, 2),
        (W.PREC_FP64, 385, 0.9, 100.0, 5),
        (W.PREC_FP64, 768, 0.9, 200.0, 9),
    ],
)
def test_velocity_counts_match_oracle(prec, n_v, hole_px, span_px, n_spec):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n_pix, n_lines = 3000, 70
    star = W.make_tiny(51, n_grid=8, n_pix=n_pix, n_mu=2, precision=prec, n_phases=1)
    print(f"[ccf-lanes] prec {prec} n_v {n_v} hole {hole_px} px span {span_px} px spectra {n_spec}", flush=True)
    ctx = L.soap_grid_init(star)
    rng = np.random.default_rng(n_v)
    px_kms = C_KMS * star.dln_lambda
    dv = span_px * px_kms / (n_v - 1)
    v0 = -0.5 * dv * (n_v - 1)
    q = np.sort(rng.uniform(-0.2 * span_px, n_pix + 0.2 * span_px, n_lines))
    mask = W.Mask(star.ln_lambda0 + (q - 0.5) * star.dln_lambda, rng.uniform(0.5, 1.5, n_lines),
                  0.5 * hole_px * px_kms, v0, dv, n_v)
    dt = np.float64 if prec == W.PREC_FP64 else np.float32
    flux = rng.uniform(0.2, 1.0, (n_spec, n_pix)).astype(dt)
    ccf = torch.full((n_spec + 1, n_v), -7.0, dtype=torch.float64, device="cuda")
    L.soap_ccf_rv(ctx, torch.from_numpy(flux).cuda(), mask, ccf_out=ccf[:n_spec])
    torch.cuda.synchronize()
    got = ccf.cpu().numpy()
    assert np.all(got[-1] == -7.0)
    ref = OC.ccf(flux.astype(np.float64), star.ln_lambda0, star.dln_lambda, mask.ln_lambda, mask.weight,
                 mask.half_width_kms, W.make_velocity_grid(v0, dv, n_v))
    # FP64: hole edges differ by ~1e-10 pixel.  FP32: partials of at most 32
    # lines x 10 pixels, each FMA within 2^-24 of the running positive sum
    rel = np.max(np.abs(got[:-1] - ref) / np.abs(ref))
    assert rel < (1e-9 if prec == W.PREC_FP64 else 2e-5), rel
    L.soap_destroy(ctx)


@pytest.mark.parametrize("prec,hole_px,n_lines", [(W.PREC_FP32, 0.9, 70), (W.PREC_FP32, 3.0, 33),
                                                  (W.PREC_FP64, 0.9, 1), (W.PREC_FP64, 1.4, 64)])
def test_few_spectra_equal_many(prec, hole_px, n_lines):
    """Calls of few blocks take two spectra a block with more loads in flight;
    every spectrum's CCF and fit is bit for bit that of a large call."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[ccf-lanes] few: prec {prec} hole {hole_px} px lines {n_lines}", flush=True)
    n_pix, n_v, n_many = 3000, 161, 1100  # at least 138 blocks of eight spectra
    star = W.make_tiny(52, n_grid=8, n_pix=n_pix, n_mu=2, precision=prec, n_phases=1)
    ctx = L.soap_grid_init(star)
    rng = np.random.default_rng(n_lines)
    px_kms = C_KMS * star.dln_lambda
    dv = 46.0 * px_kms / (n_v - 1)
    q = np.sort(rng.uniform(-5.0, n_pix + 5.0, n_lines))
    mask = W.Mask(star.ln_lambda0 + (q - 0.5) * star.dln_lambda, rng.uniform(0.5, 1.5, n_lines),
                  0.5 * hole_px * px_kms, -0.5 * dv * (n_v - 1), dv, n_v)
    dt = torch.float64 if prec == W.PREC_FP64 else torch.float32
    flux = torch.from_numpy(rng.uniform(0.2, 1.0, (n_many, n_pix))).to(dt).cuda()
    many = torch.empty(n_many, n_v, dtype=torch.float64, device="cuda")
    L.soap_ccf_rv(ctx, flux, mask, ccf_out=many)
    for n in (1, 2, 7):
        few = torch.empty(n, n_v, dtype=torch.float64, device="cuda")
        L.soap_ccf_rv(ctx, flux[:n], mask, ccf_out=few)
        assert torch.equal(few, many[:n]), n
    L.soap_destroy(ctx)
