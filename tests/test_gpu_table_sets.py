"""Synthesis calls made while the stream is certainly busy (matrix products are
enqueued first, and still run when the calls return): the table kernels run on
the side stream through all of their table sets.  One context and several in
turn, fresh ones among them, give bit for bit what the calls give one at a
time; a byte cap that holds one or two table sets refuses none of them."""
import gc

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
L = pytest.importorskip("paper_2301_04259_amd", reason="libsoap.so not built")


@pytest.fixture(scope="module", autouse=True)
def _device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    # a context that the garbage collector destroys waits for its stream: none in the middle of a burst
    gc.collect()
    gc.disable()
    yield
    gc.enable()


@pytest.fixture(scope="module")
def busy():
    """Enqueues some 60 ms of work on the current stream and returns the event after it."""
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    c = torch.empty_like(a)
    b = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)

    def go():
        for _ in range(80):
            torch.mm(a, b, out=c)
        ev = torch.cuda.Event()
        ev.record()
        return ev

    go().synchronize()
    return go


def _star(seed, precision, n_pix, n_phases, n_regions, diff_rot=0.0, n_grid=24):
    star = W.make_tiny(seed, n_grid=n_grid, n_pix=n_pix, n_mu=3, precision=precision, contrast_mode=W.CONTRAST_PLANCK,
                       n_phases=n_phases, vsini_kms=8.0, n_regions=n_regions)
    star.diff_rot = diff_rot
    return star


def _out(star, n, fill=7.0):
    dt = torch.float32 if star.precision == W.PREC_FP32 else torch.float64
    return torch.full((n, star.n_pix), fill, dtype=dt, device="cuda")


def _calls(star, n_calls, seed):
    """Another part of the region list and other phases in every call."""
    rng = np.random.default_rng(seed)
    n = len(star.phases)
    return [(star.regions[: 1 + k % len(star.regions)], rng.uniform(0.0, 1.0, max(1, n - k % 3)))
            for k in range(n_calls)]


def _single(ctx, star, calls):
    want = []
    for regions, phases in calls:
        out = _out(star, len(phases))
        L.soap_active_spectra(ctx, regions, phases, W.EFFECT_TOT, out)
        torch.cuda.synchronize()
        want.append(out)
    return want


@pytest.mark.parametrize(
    "precision,n_regions,n_phases,diff_rot",
    [(W.PREC_FP32, 3, 100, 0.0), (W.PREC_FP32, 64, 7, 0.0), (W.PREC_FP64, 2, 33, 0.25)],
)
@pytest.mark.parametrize("fresh", [False, True])
def test_calls_behind_pending_work(busy, precision, n_regions, n_phases, diff_rot, fresh):
    print(f"[sets] prec {precision} regions {n_regions} phases {n_phases} diff_rot {diff_rot} fresh {fresh}", flush=True)
    star = _star(17, precision, 2000, n_phases, n_regions, diff_rot)
    calls = _calls(star, 12, n_phases)
    ref = L.soap_grid_init(star)
    want = _single(ref, star, calls)
    ctx = L.soap_grid_init(star) if fresh else ref
    outs = [_out(star, len(p)) for _, p in calls]
    torch.cuda.synchronize()
    ev = busy()
    for k, (regions, phases) in enumerate(calls):
        L.soap_active_spectra(ctx, regions, phases, W.EFFECT_TOT, outs[k])
        if k == 1:
            assert not ev.query()  # no call can have begun: the second one's tables have the side stream
    torch.cuda.synchronize()
    for k, out in enumerate(outs):
        assert torch.equal(out, want[k]), k


def test_contexts_in_turn_on_one_stream(busy):
    stars = [_star(30 + i, W.PREC_FP64 if i == 2 else W.PREC_FP32, 1500 + 300 * i, 9 + 20 * i, 1 + i, 0.2 * (i == 3))
             for i in range(4)]
    calls = [_calls(s, 9, 5 + i) for i, s in enumerate(stars)]
    want = []
    for s, c in zip(stars, calls):
        ctx = L.soap_grid_init(s)
        want.append(_single(ctx, s, c))
        L.soap_destroy(ctx)
    ctxs = [L.soap_grid_init(s) for s in stars]
    for again in range(2):  # first with fresh contexts
        outs = [[_out(s, len(p)) for _, p in c] for s, c in zip(stars, calls)]
        torch.cuda.synchronize()
        ev = busy()
        for k in range(len(calls[0])):
            for i, s in enumerate(stars):
                regions, phases = calls[i][k]
                L.soap_active_spectra(ctxs[i], regions, phases, W.EFFECT_TOT, outs[i][k])
            if k == 0 and not again:  # (a set that grows is freed first, which may wait)
                assert not ev.query()
        # one context of the stream goes while the others still have work pending
        if again:
            L.soap_destroy(ctxs.pop(0))
        torch.cuda.synchronize()
        for i in range(len(stars)):
            for k in range(len(calls[0])):
                assert torch.equal(outs[i][k], want[i][k]), (again, i, k)


@pytest.mark.parametrize("n_phases,sets", [(600, 1), (600, 2), (9000, 1), (9000, 2), (60000, 1), (60000, 2)])
def test_byte_cap_that_holds_the_sets(busy, monkeypatch, n_phases, sets):
    star = _star(51, W.PREC_FP32, 400, n_phases, 2)
    ctx = L.soap_grid_init(star)
    base = L.device_bytes()
    calls = [(star.regions, np.random.default_rng(k).uniform(0.0, 1.0, n_phases)) for k in range(6)]
    want = _single(ctx, star, calls)
    one = L.device_bytes() - base  # the tables of calls that are waited for
    print(f"[sets] cap: {n_phases} phases, tables of {one} bytes, {sets} allowed", flush=True)
    outs = [_out(star, n_phases) for _ in calls]
    torch.cuda.synchronize()
    monkeypatch.setenv("SOAP_MAX_DEVICE_BYTES", str(base + sets * one + 4096))
    ev = busy()
    for k, (regions, phases) in enumerate(calls):
        L.soap_active_spectra(ctx, regions, phases, W.EFFECT_TOT, outs[k])
        if k == 0:
            assert not ev.query()
    torch.cuda.synchronize()
    for k, out in enumerate(outs):
        assert torch.equal(out, want[k]), k
    monkeypatch.delenv("SOAP_MAX_DEVICE_BYTES")
    for k, (regions, phases) in enumerate(calls):
        L.soap_active_spectra(ctx, regions, phases, W.EFFECT_TOT, outs[k])
    torch.cuda.synchronize()
    assert L.device_bytes() - base <= (3 if one <= 64 << 20 else 2) * one + 4096
    # other workspaces take the memory of sets that are not needed
    monkeypatch.setenv("SOAP_MAX_DEVICE_BYTES", str(base + one + one // 2))
    q = np.empty(star.n_pix, dtype=np.float32)
    L.soap_quiet_spectrum(ctx, q)
    L.soap_destroy(ctx)


def test_threads_with_contexts_on_one_stream():
    import threading

    stars = [_star(61 + i, W.PREC_FP32, 1200 + 500 * i, 11 + 40 * i, 2 + i) for i in range(2)]
    calls = [_calls(s, 40, 9 + i) for i, s in enumerate(stars)]
    want, outs, ctxs = [], [], []
    for s, c in zip(stars, calls):
        ref = L.soap_grid_init(s)
        want.append(_single(ref, s, c))
        L.soap_destroy(ref)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for s, c in zip(stars, calls):
            ctxs.append(L.soap_grid_init(s))
            outs.append([_out(s, len(p)) for _, p in c])
    torch.cuda.synchronize()
    print("[sets] two threads, one stream", flush=True)
    errors = []

    def work(i):
        try:
            for k, (regions, phases) in enumerate(calls[i]):
                L.soap_active_spectra(ctxs[i], regions, phases, W.EFFECT_TOT, outs[i][k])
            if i == 0:  # this context goes while the other one's calls are pending
                L.soap_destroy(ctxs[0])
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for i in range(2):
        for k in range(len(calls[i])):
            assert torch.equal(outs[i][k], want[i][k]), (i, k)
