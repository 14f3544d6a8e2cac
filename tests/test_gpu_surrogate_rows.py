"""Surrogate training and inference in the row kernels, at the widths where
their tiles, rounds and k steps end, and past the width that they hold (general
kernels): gradients, the updated parameters' outputs and the second step's
gradients against the oracle with bfloat16 operands; large inference batches
bit for bit the same as small ones."""
import numpy as np
import pytest

from oracle import surrogate as OSG

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _grads(s, e, P, x, t, n_in, H, O):
    """Relative error of every tensor's gradient against the bfloat16 oracle."""
    g = L.soap_surrogate_get_grads(s, e).astype(np.float64)
    _, g_q = OSG.backward(P, x, t, n_in, H, O, bf16=True)
    lay, _ = OSG.layout(n_in, H, O)
    return {k: np.linalg.norm(g[sl] - g_q[sl]) / np.linalg.norm(g_q[sl]) for k, (sl, _) in lay.items()}


@pytest.mark.parametrize(
    "n_in,H,O,E,B",
    [
        (32, 32, 32, 1, 32),     # one tile pair, every input used
        (12, 256, 128, 2, 160),  # one round of the block's waves; the last 128-row chunk is short
        (12, 288, 160, 3, 96),   # a second round and a second set of k steps
        (3, 736, 32, 1, 640),    # nearly all of the LDS; more chunks than waves
        (5, 800, 64, 1, 64),     # trains in the general kernels, predicts in the row kernel
    ],
)
def test_two_steps_match_oracle(n_in, H, O, E, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-rows] n_in {n_in} H {H} O {O} E {E} B {B}", flush=True)
    rng = np.random.default_rng(H + B)
    s = L.soap_surrogate_create(n_in, H, O, E, seed=H)
    x = rng.normal(size=(B, n_in)).astype(np.float32)
    t = rng.normal(size=(B, O)).astype(np.float32)
    for _ in range(2):
        P = [L.soap_surrogate_get_params(s, e) for e in range(E)]
        L.soap_surrogate_train_step(s, _dev(x), _dev(t), lr=1e-3)
        for e in range(E):
            # one-ulp bfloat16 flips of activations and errors: the bound that
            # the gradients of the other widths are held to
            for k, err in _grads(s, e, P[e], x, t, n_in, H, O).items():
                assert err <= 1e-2, (e, k, err)
    mem = torch.empty((E, B, O), dtype=torch.float32, device="cuda")
    coef = torch.empty((B, O), dtype=torch.float32, device="cuda")
    L.soap_surrogate_predict(s, _dev(x), coef, mem)
    for e in range(E):
        P = L.soap_surrogate_get_params(s, e)
        y_q, _ = OSG.forward(P, x, n_in, H, O, bf16=True)
        y_x, _ = OSG.forward(P, x, n_in, H, O, bf16=False)
        assert np.abs(mem[e].cpu().numpy() - y_q).max() <= 2e-3 * np.abs(y_x).max()


@pytest.mark.parametrize("H,O,E,B", [(256, 128, 4, 4112), (96, 32, 2, 16400), (2400, 32, 1, 48)])
def test_large_batches_equal_small_ones(H, O, E, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-rows] predict H {H} O {O} E {E} B {B}", flush=True)
    rng = np.random.default_rng(B)
    s = L.soap_surrogate_create(12, H, O, E, seed=5)
    x = _dev(rng.normal(size=(B, 12)))
    coef = torch.empty((B, O), dtype=torch.float32, device="cuda")
    mem = torch.full((E + 1, B, O), 7.0, dtype=torch.float32, device="cuda")
    L.soap_surrogate_predict(s, x, coef, mem[:E])
    only = torch.empty_like(coef)
    L.soap_surrogate_predict(s, x, only)  # the members in the library's own buffer
    assert torch.equal(only, coef) and torch.all(mem[E] == 7.0)
    for r in range(0, B, max(16, B // 3 // 16 * 16)):
        n = min(32, B - r)
        c = torch.empty((n, O), dtype=torch.float32, device="cuda")
        m = torch.empty((E, n, O), dtype=torch.float32, device="cuda")
        L.soap_surrogate_predict(s, x[r:r + n].contiguous(), c, m)
        assert torch.equal(m, mem[:E, r:r + n]) and torch.equal(c, coef[r:r + n])
