"""Predictions of many rows, or of very wide networks, take other launch shapes
than those of a few rows of ordinary ones: what a row's prediction is must not
depend on how many rows are with it.  Every output is compared bit for bit with
the same rows' in calls of at most 32 rows; the values themselves are tested
against the oracle in test_gpu_surrogate_rows.py.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


@pytest.mark.parametrize(
    "n_in,H,O,E,B",
    [
        (12, 32, 32, 16, 3072),  # narrow, the fewest rows of the two-wave blocks
        (32, 64, 64, 8, 6160),   # narrow, every column tile used; the last block half full
        (1, 64, 32, 5, 9872),    # a single input
        (12, 1792, 32, 1, 240),  # wide, the fewest rows of the row kernel; of fewer the general kernels
        (12, 2048, 96, 3, 352),  # wider, more columns and members
    ],
)
def test_rows_do_not_depend_on_the_batch(n_in, H, O, E, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-shapes] n_in {n_in} H {H} O {O} E {E} B {B}", flush=True)
    rng = np.random.default_rng(B)
    s = L.soap_surrogate_create(n_in, H, O, E, seed=5)
    x = torch.as_tensor(rng.normal(size=(B, n_in)).astype(np.float32), device="cuda")
    coef = torch.empty((B, O), dtype=torch.float32, device="cuda")
    mem = torch.full((E + 1, B, O), 7.0, dtype=torch.float32, device="cuda")
    L.soap_surrogate_predict(s, x, coef, mem[:E])
    assert torch.all(mem[E] == 7.0)
    for r in sorted({*range(0, B, max(32, B // 5 // 16 * 16)), B - 16}):
        n = min(32, B - r)
        c = torch.empty((n, O), dtype=torch.float32, device="cuda")
        m = torch.empty((E, n, O), dtype=torch.float32, device="cuda")
        L.soap_surrogate_predict(s, x[r:r + n].contiguous(), c, m)
        assert torch.equal(m, mem[:E, r:r + n]) and torch.equal(c, coef[r:r + n]), r


@pytest.mark.parametrize("members", [False, True])
def test_few_rows_of_a_wide_network_without_memory(monkeypatch, members):
    """After a call of many rows, one of few is refused neither under a byte cap
    nor in a captured graph; its outputs are the same."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    H, O, E, B = 1792, 64, 2, 512
    rng = np.random.default_rng(7)
    x = torch.as_tensor(rng.normal(size=(B, 12)).astype(np.float32), device="cuda")
    few = x[:32].contiguous()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = L.soap_surrogate_create(12, H, O, E, seed=5)

        def call(x):
            coef = torch.zeros((len(x), O), dtype=torch.float32, device="cuda")
            mem = torch.zeros((E, len(x), O), dtype=torch.float32, device="cuda") if members else None
            L.soap_surrogate_predict(s, x, coef, mem)
            return coef, mem

        want, mem = call(x)
        monkeypatch.setenv("SOAP_MAX_DEVICE_BYTES", str(L.device_bytes() + 4096))
        held = L.device_bytes()
        got, m = call(few)
        assert torch.equal(got, want[:32]) and (not members or torch.equal(m, mem[:, :32]))
        assert L.device_bytes() == held
        monkeypatch.delenv("SOAP_MAX_DEVICE_BYTES")
        coef = torch.zeros((32, O), dtype=torch.float32, device="cuda")
        m = torch.zeros((E, 32, O), dtype=torch.float32, device="cuda") if members else None
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            L.soap_surrogate_predict(s, few, coef, m)
        for _ in range(3):
            coef.zero_()
            g.replay()
            assert torch.equal(coef, want[:32])
        got, m = call(few)  # (the general kernels)
        assert torch.equal(got, want[:32]) and (not members or torch.equal(m, mem[:, :32]))


@pytest.mark.parametrize("H", [64, 800])  # trained by the row kernels, by the general ones
def test_prediction_captured_after_training(H):
    """A training step leaves the buffers that a prediction of its batch needs:
    one can be captured without an eager call before it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        s = L.soap_surrogate_create(12, H, 32, 2, seed=5)
        x, t = torch.randn(64, 12, device="cuda"), torch.randn(64, 32, device="cuda")
        L.soap_surrogate_train_step(s, x, t, 1e-3)
        coef, want = (torch.zeros((64, 32), dtype=torch.float32, device="cuda") for _ in range(2))
        stream.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            L.soap_surrogate_predict(s, x, coef)
        L.soap_surrogate_predict(s, x, want)
        for _ in range(3):
            coef.zero_()
            g.replay()
            assert torch.equal(coef, want)
