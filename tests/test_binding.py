"""The native binding refuses what the entry points do not take, with the exception types and
messages of the Python layer, before anything is launched."""
import pytest

torch = pytest.importorskip("torch")


def _inputs(dev, B=1, T=8, H=2, dk=32, dv=16, dtype=torch.float32):
    z = lambda *s: torch.full(s, 0.5, device=dev, dtype=dtype)
    return [z(B, T, H, dk), z(B, T, H, dk), z(B, T, H, dv), z(B, T, H, dk), z(B, T, H, dk), z(B, T, H)]


def test_cpu_tensors_are_refused():
    import paper_2602_10743_amd as K
    x = _inputs("cpu")
    with pytest.raises(ValueError, match="must live on a GPU"):
        K.kla_forward(*x)
    with pytest.raises(ValueError, match="must live on a GPU"):
        K.kla_backward(*x, None, None, x[2])
    with pytest.raises(ValueError, match="GPU tensors"):
        K.kla_decode_step(*[t[:, 0] for t in x], torch.ones(1, 2, 32), torch.zeros(1, 2, 32, 16))


@pytest.mark.gpu
def test_bad_tensors_are_refused():
    import paper_2602_10743_amd as K
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = "cuda:0"
    x = _inputs(dev)

    def bad(i, t, exc, match):
        y = list(x)
        y[i] = t
        with pytest.raises(exc, match=match):
            K.kla_forward(*y)

    bad(0, x[0].double(), TypeError, "unsupported dtype torch.float64; use float32 or bfloat16")
    bad(0, x[0][0], ValueError, r"q must be \[B, T, H, dk\]")
    bad(1, x[1][:, :4].contiguous(), ValueError, r"k has shape \(1, 4, 2, 32\), expected \(1, 8, 2, 32\)")
    bad(3, x[3].bfloat16(), ValueError, "a must share q's dtype and device")
    bad(2, x[2].transpose(1, 2).contiguous().transpose(1, 2), ValueError, "v must be contiguous")
    bad(5, x[5].cpu(), ValueError, "r must share q's dtype and device")
    with pytest.raises(ValueError, match=r"lam0 must be a contiguous float32 tensor of shape \(1, 2, 32\) on cuda:0"):
        K.kla_forward(*x, torch.ones(2, 32, device=dev))
    with pytest.raises(ValueError, match="dy must be a contiguous"):
        K.kla_backward(*x, None, None, x[0])
    wide = [t.repeat_interleave(2, -1)[..., :24].contiguous() if t.dim() == 4 else t for t in x]   # widths of 24
    with pytest.raises(K.KLAError) as e:
        K.kla_forward(*wide)
    assert e.value.status == 2   # KLA_ERR_SHAPE
    with pytest.raises(ValueError, match="k must be a contiguous"):
        K.kla_decode_step(x[0][:, 0], x[1][:, 0, :1], x[2][:, 0], x[3][:, 0], x[4][:, 0], x[5][:, 0],
                          torch.ones(1, 2, 32, device=dev), torch.zeros(1, 2, 32, 16, device=dev))


@pytest.mark.gpu
def test_absent_ou_parameters_are_refused():
    """An OU entry point without one of a, p, delta is refused, and per-token gates are not taken
    in their place."""
    import paper_2602_10743_amd as K
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    q, k, v, a, p, r = _inputs("cuda:0")
    par = [torch.ones(2, 32, device="cuda:0") for _ in range(3)]
    lam, eta = torch.ones(1, 2, 32, device="cuda:0"), torch.zeros(1, 2, 32, 16, device="cuda:0")
    one = [t[:, 0].contiguous() for t in (q, k, v, r)]
    for i in range(3):
        some = [None if j == i else t for j, t in enumerate(par)]
        for call in (lambda: K.kla_forward_ou(q, k, v, *some, r),
                     lambda: K.kla_backward_ou(q, k, v, *some, r, None, None, v),
                     lambda: K.kla_decode_step_ou(*one[:3], *some, one[3], lam, eta)):
            with pytest.raises(K.KLAError) as e:
                call()
            assert e.value.status == 1   # KLA_ERR_NULL
    with pytest.raises(ValueError, match="a must be a contiguous float32"):
        K.kla_forward_ou(q, k, v, a, p, None, r)
    with pytest.raises(K.KLAError):
        K.kla_decode_step_ou(*one[:3], *par, one[3], None, eta)


@pytest.mark.gpu
def test_unused_outputs_have_no_gradient():
    """Gradients through y alone, through lamT alone and through both agree with their sum."""
    import paper_2602_10743_amd as K
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = [t.clone().requires_grad_(True) for t in _inputs("cuda:0", T=70)]
    y, lamT, etaT = K.kla_filter(*x)
    gy = torch.autograd.grad(y.sum(), x, retain_graph=True)
    gl = torch.autograd.grad(lamT.sum(), x, retain_graph=True)
    both = torch.autograd.grad(y.sum() + lamT.sum(), x)
    for a, b, c in zip(gy, gl, both):
        assert torch.allclose(a + b, c, rtol=1e-5, atol=1e-5 * float(c.abs().max() + 1))


@pytest.mark.gpu
def test_other_threads_run_during_a_call(monkeypatch):
    """The interpreter lock is given up in a call: under KLA_CHECK=1 it waits for the stream,
    here behind some 0.3 s of other work, and another thread goes on meanwhile."""
    import threading
    import time

    import paper_2602_10743_amd as K
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = _inputs("cuda:0")
    monkeypatch.setenv("KLA_CHECK", "1")
    K.kla_forward(*x)
    start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    start.record()
    torch.cuda._sleep(10_000_000)
    end.record()
    torch.cuda.synchronize()
    cycles = int(10_000_000 * 300.0 / start.elapsed_time(end))
    calls = [lambda: K.kla_forward(*x), lambda: K.kla_backward(*x, None, None, x[2])]
    for call in calls:
        torch.cuda._sleep(cycles)
        took = []

        def work():
            t0 = time.perf_counter()
            call()
            took.append(time.perf_counter() - t0)

        t = threading.Thread(target=work)
        last, gap = time.perf_counter(), 0.0
        t.start()
        while t.is_alive():
            time.sleep(0.001)
            now = time.perf_counter()
            last, gap = now, max(gap, now - last)
        t.join()
        torch.cuda.synchronize()
        assert took[0] > 0.1, "the call did not wait for the stream"
        assert gap < 0.5 * took[0], f"held the interpreter lock for {gap:.2f} of {took[0]:.2f} s"
