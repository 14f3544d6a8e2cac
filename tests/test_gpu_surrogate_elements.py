"""Every element of two surrogate training steps, in the row kernels and past the
width that they hold: gradients within eight times the error propagated through
the oracle's bfloat16 network (FP32 sums of any order, their errors adding up at
random; a rounded value is off only where the error reaches the next bfloat16),
and the Adam update of the device's own gradients."""
import numpy as np
import pytest

from oracle import surrogate as OSG

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")

U = 2.0**-24  # half a unit in the last place of FP32, relative


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _product(a, ea, b, eb=0.0):
    """a @ b and the size of its error for operands off by ea, eb at random, added in FP32."""
    var = ea**2 @ b**2 if np.ndim(ea) else 0.0
    var = var + (a**2 @ eb**2 if np.ndim(eb) else 0.0)
    return a @ b, np.sqrt(var + (a.shape[1] + 2) * U * U * (a**2 @ b**2))


def _rounded(v, e):
    """bfloat16 of v, and how far another value within 4 e of v can round from it."""
    q = OSG.bf16_round(v)
    return q, np.maximum(np.abs(OSG.bf16_round(v + 4 * e) - q), np.abs(OSG.bf16_round(v - 4 * e) - q))


def _silu(z, ez):
    h = OSG.silu(z)
    return _rounded(h, 1.1 * ez + 2.0**-20 * np.abs(h))  # |silu'| < 1.1; expf and the division: a few ulps


def _back(lin, elin, z, ez):
    """lin silu'(z): |silu''| <= 1/2, silu' from FP32 terms of size up to 1 + |z|."""
    g = OSG.silu_grad(z)
    eg = 0.5 * ez + 2.0**-20 * (1.0 + np.abs(z))
    v = lin * g
    return v, elin * (np.abs(g) + eg) + np.abs(lin) * eg + 4 * U * np.abs(v)


def _bounds(p, x, t, n_in, H, O):
    """Gradient of the oracle (flat) and eight times the error of each element."""
    w = OSG.unpack(p, n_in, H, O)
    W1, W2, W3 = (OSG.bf16_round(w[k]) for k in ("W1", "W2", "W3"))
    B = x.shape[0]
    a0 = OSG.bf16_round(x)

    def bias(v, e, b):
        return v + b, e + U * (np.abs(v) + np.abs(b))

    z1, e1 = bias(*_product(a0, 0.0, W1), w["b1"])
    a1, ea1 = _silu(z1, e1)
    z2, e2 = bias(*_product(a1, ea1, W2), w["b2"])
    a2, ea2 = _silu(z2, e2)
    y, ey = bias(*_product(a2, ea2, W3), w["b3"])
    sc = 2.0 / (B * O)
    dy = sc * (y - t)
    dyq, edy = _rounded(dy, sc * ey + 4 * U * np.abs(dy))
    dz2, ed2 = _back(*_product(dyq, edy, W3.T), z2, e2)
    dz2q, ed2q = _rounded(dz2, ed2)
    dz1, ed1 = _back(*_product(dz2q, ed2q, W2.T), z1, e1)
    dz1q, ed1q = _rounded(dz1, ed1)
    g, e = {}, {}
    g["W3"], e["W3"] = _product(a2.T, ea2.T, dyq, edy)
    g["W2"], e["W2"] = _product(a1.T, ea1.T, dz2q, ed2q)
    g["W1"], e["W1"] = _product(a0.T, 0.0, dz1q, ed1q)
    for k, d, ed in (("b3", dyq, edy), ("b2", dz2, ed2), ("b1", dz1, ed1)):
        g[k], e[k] = d.sum(axis=0), np.sqrt((ed**2).sum(axis=0) + (B + 2) * U * U * (d**2).sum(axis=0))
    return OSG.pack(g, n_in, H, O), 8.0 * OSG.pack(e, n_in, H, O)


@pytest.mark.parametrize(
    "n_in,H,O,E,B",
    [
        (32, 32, 32, 1, 32),     # one tile pair, every input used
        (12, 256, 128, 2, 160),  # one round of the block's waves; the last 128-row chunk is short
        (12, 288, 160, 3, 96),   # a second round and a second set of k steps
        (3, 736, 32, 1, 640),    # nearly all of the LDS; more chunks than waves
        (5, 800, 64, 1, 64),     # the general kernels
    ],
)
def test_elements_of_two_steps(n_in, H, O, E, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-elements] n_in {n_in} H {H} O {O} E {E} B {B}", flush=True)
    rng = np.random.default_rng(H + B)
    s = L.soap_surrogate_create(n_in, H, O, E, seed=H)
    x = rng.normal(size=(B, n_in)).astype(np.float32)
    t = rng.normal(size=(B, O)).astype(np.float32)
    lr, b1, b2, eps = 1e-3, np.float32(0.9), np.float32(0.999), 1e-8
    m, v = np.zeros(E, object), np.zeros(E, object)
    for step in (1, 2):
        before = [L.soap_surrogate_get_params(s, e).astype(np.float64) for e in range(E)]
        L.soap_surrogate_train_step(s, _dev(x), _dev(t), lr=lr)
        for e in range(E):
            got = L.soap_surrogate_get_grads(s, e).astype(np.float64)
            want, off = _bounds(before[e], x.astype(np.float64), t.astype(np.float64), n_in, H, O)
            worst = np.argmax(np.abs(got - want) - off)
            assert np.all(np.abs(got - want) <= off), (step, e, worst, got[worst], want[worst], off[worst])
            # (of the oracle alone: below the first step's gradients, so that misplaced elements cannot pass)
            assert step > 1 or np.median(off) < 0.2 * np.median(np.abs(want))
            # the update from the device's gradients: constants in FP32 as the
            # kernel has them, where 1 - 0.999^k carries 3e-5 of rounding
            m[e] = float(b1) * m[e] + float(np.float32(1) - b1) * got
            v[e] = float(b2) * v[e] + float(np.float32(1) - b2) * got * got
            c1, c2 = float(np.float32(1) - b1**np.float32(step)), float(np.float32(1) - b2**np.float32(step))
            p = before[e] - lr * (m[e] / c1) / (np.sqrt(v[e] / c2) + eps)
            after = L.soap_surrogate_get_params(s, e).astype(np.float64)
            assert np.all(np.abs(after - p) <= 1e-4 * lr + 2 * U * np.abs(p)), (step, e)
