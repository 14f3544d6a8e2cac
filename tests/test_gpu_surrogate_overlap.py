"""Surrogate inference whose member outputs lie over its inputs, or over its
means, gives what separate arrays give (the members win where they overlap the
means), in the row kernel and past the width that it holds."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


@pytest.mark.parametrize("H,O,E,B", [(64, 32, 3, 48), (256, 128, 4, 4112), (2400, 32, 2, 32)])
def test_outputs_over_inputs(H, O, E, B):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[sg-overlap] H {H} O {O} E {E} B {B}", flush=True)
    n_in = 12
    s = L.soap_surrogate_create(n_in, H, O, E, seed=3)
    x = torch.from_numpy(np.random.default_rng(B).normal(size=(B, n_in)).astype(np.float32)).cuda()
    coef = torch.empty((B, O), dtype=torch.float32, device="cuda")
    mem = torch.empty((E, B, O), dtype=torch.float32, device="cuda")
    L.soap_surrogate_predict(s, x, coef, mem)
    # inputs at the end of the members
    buf = torch.zeros(E * B * O, dtype=torch.float32, device="cuda")
    xin = buf[E * B * O - B * n_in:].view(B, n_in)
    xin.copy_(x)
    c2 = torch.empty_like(coef)
    L.soap_surrogate_predict(s, xin, c2, buf.view(E, B, O))
    assert torch.equal(buf.view(E, B, O), mem) and torch.equal(c2, coef)
    # means over the first member, and over the inputs
    m2 = torch.zeros((E, B, O), dtype=torch.float32, device="cuda")
    L.soap_surrogate_predict(s, x, m2[0], m2)
    assert torch.equal(m2, mem)
    buf = torch.zeros(B * O, dtype=torch.float32, device="cuda")
    buf[:B * n_in].view(B, n_in).copy_(x)
    m3 = torch.empty_like(mem)
    L.soap_surrogate_predict(s, buf[:B * n_in].view(B, n_in), buf.view(B, O), m3)
    assert torch.equal(m3, mem) and torch.equal(buf.view(B, O), coef)
