"""The segment-parallel bf16 forward and backward (few sequences, csrc/chunk_seg.hip) against
the fp64 oracle: ragged lengths, segments of one chunk, the last segment of one token, wide
and 64-channel value tiles, per-token and OU gates, with and without a saved context.

Tolerances as in test_parity_gpu.py: bf16 outputs 2e-2, fp32 beliefs and variances 1e-4
(etaT, whose products are split-bf16: 2e-2)."""
import numpy as np
import pytest

import kla_inputs as K
import oracle
from kla_testutil import TOL, log, rel_err, rel_err_sum, to_np, to_torch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOKEN = ("q", "k", "v", "a", "p", "r")


@pytest.fixture(scope="module")
def kla():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_10743_amd as lib
    lib._load()
    return lib


def _f32(x):
    return torch.tensor(np.asarray(x, dtype=np.float32), device=DEV)


def _check(got, ref, names, tol):
    for n in names:
        x = to_np(got[n])
        assert np.all(np.isfinite(x)), f"{n} not finite"
        r = K.quantise(ref[n], "bf16") if n == "y" else ref[n]
        e = rel_err(x, r)
        assert e <= tol, f"{n}: {e:.2e}"


@pytest.mark.parametrize("B,T,H,dk,dv", [
    (1, 705, 2, 128, 128),   # wide tiles; a last segment of one token
    (1, 1000, 1, 64, 128),   # wide tiles, segments of one chunk
    (2, 513, 3, 64, 64), (1, 640, 2, 32, 32), (1, 799, 1, 32, 128), (3, 900, 20, 64, 32), (1, 600, 2, 128, 16)])
@pytest.mark.parametrize("ou", [False, True])
def test_against_oracle(kla, B, T, H, dk, dv, ou):
    log(f"segments B{B} T{T} H{H} dk{dk} dv{dv} ou={ou}")
    case = K.random_case(B, T, H, dk, dv, "bf16", seed=T + dk, dist="lm")
    g = np.random.default_rng(T)
    q32 = lambda x: x.astype(np.float32).astype(np.float64)
    lam0, eta0 = q32(0.5 + g.random((B, H, dk))), q32(g.standard_normal((B, H, dk, dv)))
    dlamT, detaT = q32(g.standard_normal((B, H, dk))), q32(g.standard_normal((B, H, dk, dv)))
    dyvar = q32(g.standard_normal((B, T, H)))
    x = {n: to_torch(case[n], "bf16", DEV) for n in TOKEN + ("dy",)}
    if ou:
        P = K.ou_params(H, dk, seed=T)
        Pd = [P[n].astype(np.float64) for n in ("a", "p", "delta")]
        pt = [_f32(P[n]) for n in ("a", "p", "delta")]
        fa = (x["q"], x["k"], x["v"], *pt, x["r"], _f32(lam0), _f32(eta0))
        oa = (case["q"], case["k"], case["v"], *Pd, case["r"], lam0, eta0)
        fwd, bwd, ofwd = kla.kla_forward_ou, kla.kla_backward_ou, oracle.forward_ou
        rg = oracle.backward_ou(*oa, case["dy"], dlamT, detaT, dyvar=dyvar, with_mass=True)
        tok = ("dq", "dk", "dv", "dr")
    else:
        fa = tuple(x[n] for n in TOKEN) + (_f32(lam0), _f32(eta0))
        oa = tuple(case[n] for n in TOKEN) + (lam0, eta0)
        fwd, bwd, ofwd = kla.kla_forward, kla.kla_backward, oracle.forward
        rg = oracle.backward(*oa, case["dy"], dlamT, detaT, dyvar=dyvar)
        tok = ("dq", "dk", "dv", "da", "dp", "dr")
    ref = ofwd(*oa)
    for save in (False, True):
        out = fwd(*fa, want_var=True, save=save)
        _check(out, ref, ("y", "etaT"), TOL["bf16"])
        _check(out, ref, ("yvar", "lamT"), TOL["f32"])
    if dv == 16:
        return   # its saved context and backward are the token-recurrent ones
    for saved in (out["saved"], None):
        got = bwd(*fa, x["dy"], _f32(dlamT), _f32(detaT), saved=saved, dyvar=_f32(dyvar))
        _check(got, rg, tok + ("dlam0", "deta0"), TOL["bf16"])
        if ou:
            for n in ("da", "dp", "ddelta"):
                e = rel_err_sum(to_np(got[n]), rg[n], rg["mass_" + n])
                assert e <= TOL["bf16"], f"{n}: {e:.2e}"


def _lm(B, T, H, dk, dv, seed):
    g = torch.Generator(device=DEV).manual_seed(seed)
    z = lambda *s: torch.randn(*s, generator=g, device=DEV)
    x = dict(q=z(B, T, H, dk), k=torch.nn.functional.normalize(z(B, T, H, dk), dim=-1), v=z(B, T, H, dv),
             r=0.1 + z(B, T, H).abs(), a=torch.sigmoid(z(B, T, H, dk) + 3), p=0.05 * z(B, T, H, dk).abs(),
             dy=z(B, T, H, dv))
    x = {n: t.bfloat16() for n, t in x.items()}
    x.update(lam0=0.5 + torch.rand(B, H, dk, generator=g, device=DEV), eta0=z(B, H, dk, dv), dlamT=z(B, H, dk),
             detaT=z(B, H, dk, dv), dyvar=z(B, T, H))
    return x, z


def _gates(z, H, dk):
    """OU parameters: a in 1 .. 3, p above 1, delta about 0.001 .. 0.1."""
    return [1 + torch.sigmoid(z(H, dk)) * 2, z(H, dk).abs() + 1, 0.001 + 0.03 * z(H, dk).abs()]


# the allocation-free backward works in 64 MiB: the same segments in windows, bit for bit
@pytest.mark.parametrize("B,T,H,dk,dv", [(2, 2048, 16, 128, 128), (1, 30011, 8, 32, 64), (1, 20000, 5, 64, 128)])
def test_windows_agree(kla, B, T, H, dk, dv):
    log(f"segment windows B{B} T{T} H{H} {dk} x {dv}")
    x, _ = _lm(B, T, H, dk, dv, T)
    fa = [x[n] for n in TOKEN] + [x["lam0"], x["eta0"]]
    saved = kla.kla_forward(*fa, save=True)["saved"]
    args = fa + [x["dy"], x["dlamT"], x["detaT"]]
    ref = kla.kla_backward(*args, saved=saved, dyvar=x["dyvar"])
    got = kla.kla_backward_noalloc(*args, saved=saved, dyvar=x["dyvar"])
    torch.cuda.synchronize()
    for n in ("dq", "dk", "dv", "da", "dp", "dr", "dlam0", "deta0"):
        assert torch.equal(got[n], ref[n]), n


def test_ou_windows_agree_with_halves(kla):
    """A sequence whose segments need two windows against its halves (one window each), joined
    through the belief and its gradient.  Each side is within the bf16 tolerance of the exact
    gradients, so the two are within twice it; the parameter gradients sum 384000 tokens' fp32 terms
    in another order, 1e-3 in the 2-norm."""
    T, H, d, m = 24000, 16, 128, 12000
    log(f"OU segment windows T{T} H{H} {d} x {d}")
    x, z = _lm(1, T, H, d, d, 7)
    gates = _gates(z, H, d)

    def run(s, lam0, eta0):
        return [x[n][:, s].contiguous() for n in ("q", "k", "v")] + gates + [x["r"][:, s].contiguous(), lam0, eta0]

    def grads(fa, s, dlamT, detaT, saved):
        return kla.kla_backward_ou(*fa, x["dy"][:, s].contiguous(), dlamT, detaT, saved=saved,
                                   dyvar=x["dyvar"][:, s].contiguous())

    every, one, two = slice(0, T), slice(0, m), slice(m, T)
    fa = run(every, x["lam0"], x["eta0"])
    ref = grads(fa, every, x["dlamT"], x["detaT"], kla.kla_forward_ou(*fa, save=True)["saved"])
    f1 = run(one, x["lam0"], x["eta0"])
    o1 = kla.kla_forward_ou(*f1, save=True)
    f2 = run(two, o1["lamT"], o1["etaT"])
    g2 = grads(f2, two, x["dlamT"], x["detaT"], kla.kla_forward_ou(*f2, save=True)["saved"])
    g1 = grads(f1, one, g2["dlam0"], g2["deta0"], o1["saved"])
    for n in ("dq", "dk", "dv", "dr"):
        e = rel_err(to_np(torch.cat([g1[n], g2[n]], 1)), to_np(ref[n]))
        assert e <= 2 * TOL["bf16"], f"{n}: {e:.2e}"
    for n in ("dlam0", "deta0"):
        e = rel_err(to_np(g1[n]), to_np(ref[n]))
        assert e <= 2 * TOL["bf16"], f"{n}: {e:.2e}"
    for n in ("da", "dp", "ddelta"):
        a, b = (g1[n] + g2[n]).double(), ref[n].double()
        e = float((a - b).norm() / b.norm())
        assert e <= 1e-3, f"{n}: {e:.2e}"


@pytest.mark.parametrize("B,T,H,dk,dv", [(1, 2011, 4, 128, 128), (1, 1500, 3, 64, 32)])
@pytest.mark.parametrize("ou", [False, True])
def test_recomputed_context_agrees(kla, B, T, H, dk, dv, ou):
    """Without a saved context the backward forms it by the forward's own (segmented) kernels:
    the same gradients bit for bit."""
    log(f"recomputed context B{B} T{T} H{H} {dk} x {dv} ou={ou}")
    x, z = _lm(B, T, H, dk, dv, T)
    if ou:
        gates = _gates(z, H, dk)
        fa = [x["q"], x["k"], x["v"], *gates, x["r"], x["lam0"], x["eta0"]]
        fwd, bwd = kla.kla_forward_ou, kla.kla_backward_ou
    else:
        fa = [x[n] for n in TOKEN] + [x["lam0"], x["eta0"]]
        fwd, bwd = kla.kla_forward, kla.kla_backward
    args = fa + [x["dy"], x["dlamT"], x["detaT"]]
    ref = bwd(*args, saved=fwd(*fa, save=True)["saved"], dyvar=x["dyvar"])
    got = bwd(*args, dyvar=x["dyvar"])
    for n in ref:
        assert torch.equal(got[n], ref[n]), n
