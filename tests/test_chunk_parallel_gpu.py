"""The chunk-parallel fp64 path (fp32 inputs, csrc/chunk64_par.hip) against the fp64 oracle:
the lengths around its threshold and its chunks, every width and gate form, the windows it
cuts long problems into, and the token-by-token fallback when a chunk leaves fp64's range.

Tolerance 1e-5: outputs are fp64 results rounded once to fp32 (6e-8); what is left is the
fp64 recursions' own rounding, below that."""
import numpy as np
import pytest

import kla_inputs as K
import oracle
from kla_testutil import log, rel_err, rel_err_sum, to_np, to_torch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 1e-5
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


def _extras(B, T, H, dk, dv, seed):
    g = np.random.default_rng(seed)
    r = lambda x: x.astype(np.float32).astype(np.float64)
    return dict(lam0=r(0.5 + g.random((B, H, dk))), eta0=r(g.standard_normal((B, H, dk, dv))),
                dlamT=r(g.standard_normal((B, H, dk))), detaT=r(g.standard_normal((B, H, dk, dv))),
                dyvar=r(g.standard_normal((B, T, H))))


def _all(got, ref, names, tol=TOL):
    for n in names:
        x = to_np(got[n])
        assert np.all(np.isfinite(x)), f"{n} not finite"
        e = rel_err(x, ref[n])
        assert e <= tol, f"{n}: {e:.2e}"


# one token past two chunks, a whole number of chunks, a ragged end; at widths up to 32 few
# sequences and enough chunks to take this path (65 tokens there: the sequential one)
@pytest.mark.parametrize("B,T,H,dk,dv", [(1, 65, 3, 64, 64), (2, 96, 1, 64, 16), (1, 97, 2, 16, 64), (1, 161, 1, 128, 128),
                                         (2, 129, 1, 32, 128), (1, 320, 2, 32, 32), (1, 289, 3, 16, 32),
                                         (1, 65, 2, 32, 16)])
@pytest.mark.parametrize("ou", [False, True])
def test_against_oracle(kla, B, T, H, dk, dv, ou):
    log(f"chunk-parallel fp64 B{B} T{T} H{H} dk{dk} dv{dv} ou={ou}")
    case = K.random_case(B, T, H, dk, dv, "f32", seed=T + dk, dist="lm")
    e = _extras(B, T, H, dk, dv, T)
    x = {n: to_torch(case[n], "f32", DEV) for n in TOKEN + ("dy",)}
    d = {n: _f32(v) for n, v in e.items()}
    if ou:
        P = K.ou_params(H, dk, seed=T)
        Pd = {n: v.astype(np.float64) for n, v in P.items()}
        pt = [_f32(P[n]) for n in ("a", "p", "delta")]
        out = kla.kla_forward_ou(x["q"], x["k"], x["v"], *pt, x["r"], d["lam0"], d["eta0"], want_var=True, save=True)
        free = kla.kla_forward_ou(x["q"], x["k"], x["v"], *pt, x["r"], d["lam0"], d["eta0"], want_var=True)
        args = (x["q"], x["k"], x["v"], *pt, x["r"], d["lam0"], d["eta0"], x["dy"], d["dlamT"], d["detaT"])
        got = kla.kla_backward_ou(*args, saved=out["saved"], dyvar=d["dyvar"])
        again = kla.kla_backward_ou(*args, dyvar=d["dyvar"])
        oa = (case["q"], case["k"], case["v"], Pd["a"], Pd["p"], Pd["delta"], case["r"], e["lam0"], e["eta0"])
        ref = oracle.forward_ou(*oa)
        rg = oracle.backward_ou(*oa, case["dy"], e["dlamT"], e["detaT"], dyvar=e["dyvar"], with_mass=True)
        names = ("dq", "dk", "dv", "dr", "dlam0", "deta0")
        for n in ("da", "dp", "ddelta"):
            err = rel_err_sum(to_np(got[n]), rg[n], rg["mass_" + n])
            assert err <= TOL, f"{n}: {err:.2e}"
    else:
        args = tuple(x[n] for n in TOKEN) + (d["lam0"], d["eta0"])
        out = kla.kla_forward(*args, want_var=True, save=True)
        free = kla.kla_forward(*args, want_var=True)
        got = kla.kla_backward(*args, x["dy"], d["dlamT"], d["detaT"], saved=out["saved"], dyvar=d["dyvar"])
        again = kla.kla_backward(*args, x["dy"], d["dlamT"], d["detaT"], dyvar=d["dyvar"])
        oa = tuple(case[n] for n in TOKEN) + (e["lam0"], e["eta0"])
        ref = oracle.forward(*oa)
        rg = oracle.backward(*oa, case["dy"], e["dlamT"], e["detaT"], dyvar=e["dyvar"])
        names = ("dq", "dk", "dv", "da", "dp", "dr", "dlam0", "deta0")
    _all(out, ref, ("y", "yvar", "lamT", "etaT"))
    _all(got, rg, names)
    for n in ("y", "yvar", "lamT", "etaT"):
        assert torch.equal(out[n], free[n]), f"{n} differs without a saved context"
    for n in names:
        assert torch.equal(got[n], again[n]), f"{n} differs with a recomputed context"


def test_out_of_range_chunk_falls_back(kla):
    """abar = 1e-12 over two chunks of one head: P underflows fp64 inside a chunk, which the
    token-recurrent kernels take; without and with a saved context, and then a call in range
    on the same workspace sizes (the flag is cleared).  The token-recurrent kernels round
    q / lam and the partial sums of the readout to fp32: 64 terms of 6e-8 of their size, judged
    against 1% of the rms, where they cancel: 64 x 6e-8 / 0.01 = 4e-4 at worst, the fp32 gate of
    1e-4 in practice."""
    B, T, H, dk, dv = 2, 150, 2, 64, 32
    case = K.random_case(B, T, H, dk, dv, "f32", seed=3, dist="lm")
    low = dict(case, a=case["a"].copy())
    low["a"][1, 40:110, 1] = np.float32(1e-12)
    e = _extras(B, T, H, dk, dv, 4)
    for name, c, tol in (("low", low, 1e-4), ("in range", case, TOL)):
        log(f"range fallback: {name}")
        x = {n: to_torch(c[n], "f32", DEV) for n in TOKEN + ("dy",)}
        d = {n: _f32(v) for n, v in e.items()}
        args = tuple(x[n] for n in TOKEN) + (d["lam0"], d["eta0"])
        out = kla.kla_forward(*args, want_var=True, save=True)
        free = kla.kla_forward(*args, want_var=True)
        got = kla.kla_backward(*args, x["dy"], d["dlamT"], d["detaT"], saved=out["saved"], dyvar=d["dyvar"])
        oa = tuple(c[n] for n in TOKEN) + (e["lam0"], e["eta0"])
        ref = oracle.forward(*oa)
        rg = oracle.backward(*oa, c["dy"], e["dlamT"], e["detaT"], dyvar=e["dyvar"])
        _all(out, ref, ("y", "yvar", "lamT", "etaT"), tol)
        _all(free, ref, ("y", "yvar", "lamT", "etaT"), tol)
        _all(got, rg, ("dq", "dk", "dv", "dp", "dr", "dlam0", "deta0"), tol)
        da, rda = to_np(got["da"]), rg["da"]
        keep = c["a"] > 1e-6   # at abar = 1e-12 the gradient is 1 / abar times a cancelling sum
        assert rel_err(da[keep], rda[keep]) <= tol


# windows: batches of sequences and windows of one sequence's chunks (the allocation-free
# backward works in 56 MiB, the others in 192), with a carry from window to window, are the
# same kernels on the same chunks: bit for bit the same results
@pytest.mark.parametrize("B,T,H", [(1, 9600, 1), (3, 3000, 2)])
def test_windows_agree(kla, B, T, H):
    log(f"windows B{B} T{T} H{H} 128 x 128")
    g = torch.Generator(device=DEV).manual_seed(5)
    z = lambda *s: torch.randn(*s, generator=g, device=DEV)
    dk = dv = 128
    q, v, dy = z(B, T, H, dk), z(B, T, H, dv), z(B, T, H, dv)
    k = torch.nn.functional.normalize(z(B, T, H, dk), dim=-1)
    a, p, r = torch.sigmoid(z(B, T, H, dk) + 3), 0.05 * z(B, T, H, dk).abs(), 0.1 + z(B, T, H).abs()
    dlamT, detaT = z(B, H, dk), z(B, H, dk, dv)
    saved = kla.kla_forward(q, k, v, a, p, r, save=True)["saved"]
    ref = kla.kla_backward(q, k, v, a, p, r, None, None, dy, dlamT, detaT, saved=saved)
    got = kla.kla_backward_noalloc(q, k, v, a, p, r, None, None, dy, dlamT, detaT, saved=saved)
    torch.cuda.synchronize()
    for n in ("dq", "dk", "dv", "da", "dp", "dr", "dlam0", "deta0"):
        assert torch.equal(got[n], ref[n]), n


def test_forward_windows_agree(kla):
    T, d = 48000, 128   # 1500 chunks without a saved context: two windows; with one: one
    log(f"forward windows T{T} {d} x {d}")
    g = torch.Generator(device=DEV).manual_seed(6)
    z = lambda *s: torch.randn(*s, generator=g, device=DEV)
    q, v = z(1, T, 1, d), z(1, T, 1, d)
    k = torch.nn.functional.normalize(z(1, T, 1, d), dim=-1)
    a, p, r = torch.sigmoid(z(1, T, 1, d) + 3), 0.05 * z(1, T, 1, d).abs(), 0.1 + z(1, T, 1).abs()
    one = kla.kla_forward(q, k, v, a, p, r, want_var=True, save=True)
    two = kla.kla_forward(q, k, v, a, p, r, want_var=True)
    torch.cuda.synchronize()
    for n in ("y", "yvar", "lamT", "etaT"):
        assert torch.equal(one[n], two[n]), n


# OU gates, whose sums are carried over windows and placed by batches, with a belief, its gradient
# and dyvar: a sequence of two windows against its halves (joined through fp32 values, so to TOL),
# and two batches of sequences against each sequence alone (the same kernels on the same chunks,
# bit for bit; the parameters' sums over the sequences to TOL).
@pytest.mark.parametrize("B,T,halves", [(1, 48000, True), (6, 9600, False)])
def test_ou_windows_and_batches_agree(kla, B, T, halves):
    log(f"OU windows B{B} T{T} 128 x 128")
    d = 128
    g = torch.Generator(device=DEV).manual_seed(8)
    z = lambda *s: torch.randn(*s, generator=g, device=DEV)
    x = dict(q=z(B, T, 1, d), k=torch.nn.functional.normalize(z(B, T, 1, d), dim=-1), v=z(B, T, 1, d),
             r=0.1 + z(B, T, 1).abs(), dy=z(B, T, 1, d), dyvar=z(B, T, 1))
    par = [1 + 2 * torch.sigmoid(z(1, d)), z(1, d).abs() + 1, 0.001 + 0.03 * z(1, d).abs()]
    lam0, eta0, dlamT, detaT = z(B, 1, d).abs() + 0.5, z(B, 1, d, d), z(B, 1, d), z(B, 1, d, d)

    def fwd(b, t, l0, e0):
        ins = [x[n][b, t].contiguous() for n in ("q", "k", "v")] + par + [x["r"][b, t].contiguous(), l0, e0]
        return ins, kla.kla_forward_ou(*ins, save=True)

    def bwd(ins, out, b, t, dl, de):
        return kla.kla_backward_ou(*ins, x["dy"][b, t].contiguous(), dl, de, saved=out["saved"],
                                   dyvar=x["dyvar"][b, t].contiguous())

    every, m = slice(0, T), T // 2 // 32 * 32
    ref = bwd(*fwd(slice(0, B), every, lam0, eta0), slice(0, B), every, dlamT, detaT)
    params = ("da", "dp", "ddelta")
    if halves:
        one, two, b = slice(0, m), slice(m, T), slice(0, B)
        i1, o1 = fwd(b, one, lam0, eta0)
        g2 = bwd(*fwd(b, two, o1["lamT"], o1["etaT"]), b, two, dlamT, detaT)
        g1 = bwd(i1, o1, b, one, g2["dlam0"], g2["deta0"])
        got = {n: torch.cat([g1[n], g2[n]], 1) for n in ("dq", "dk", "dv", "dr")}
        got.update(dlam0=g1["dlam0"], deta0=g1["deta0"], **{n: g1[n] + g2[n] for n in params})
        for n in got:
            a, w = got[n].double(), ref[n].double()
            assert float((a - w).norm() / w.norm()) <= TOL, n
    else:
        parts = []
        for i in range(B):
            b = slice(i, i + 1)
            parts.append(bwd(*fwd(b, every, lam0[b], eta0[b]), b, every, dlamT[b], detaT[b]))
        for n in ("dq", "dk", "dv", "dr", "dlam0", "deta0"):
            assert torch.equal(torch.cat([p[n] for p in parts]), ref[n]), n
        for n in params:
            a, w = sum(p[n].double() for p in parts), ref[n].double()
            assert float((a - w).norm() / w.norm()) <= TOL, n


# A value that is not finite reaches the tokens that the recursion carries it to and no other: y
# and yvar of its own and later tokens, gradients of its own and earlier ones (dv and dr after it,
# and everything else there, stay those of the oracle).  Token 53 of 150: in the second of its
# chunk's two tiles of 16, with tokens of the tile and whole chunks on both sides.
@pytest.mark.parametrize("name", ["v", "q", "dy", "dyvar"])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("dk,dv", [(64, 64), (128, 16)])
def test_non_finite_values_stay_causal(kla, name, bad, dk, dv):
    log(f"non-finite {name} {bad} {dk} x {dv}")
    B, T, H, t = 2, 150, 2, 53
    case = K.random_case(B, T, H, dk, dv, "f32", seed=9, dist="lm")
    e = _extras(B, T, H, dk, dv, 9)
    c = {n: case[n].copy() for n in TOKEN + ("dy",)}
    c["dyvar"] = e["dyvar"].copy()
    c[name][(1, t, 1) if name == "dyvar" else (1, t, 1, 3)] = bad
    x = {n: to_torch(c[n], "f32", DEV) for n in TOKEN + ("dy",)}
    d = {n: _f32(v) for n, v in dict(e, dyvar=c["dyvar"]).items()}
    args = tuple(x[n] for n in TOKEN) + (d["lam0"], d["eta0"])
    out = kla.kla_forward(*args, want_var=True, save=True)
    free = kla.kla_forward(*args, want_var=True)
    got = kla.kla_backward(*args, x["dy"], d["dlamT"], d["detaT"], saved=out["saved"], dyvar=d["dyvar"])
    again = kla.kla_backward(*args, x["dy"], d["dlamT"], d["detaT"], dyvar=d["dyvar"])
    oa = tuple(c[n] for n in TOKEN) + (e["lam0"], e["eta0"])
    with np.errstate(all="ignore"):
        ref = oracle.forward(*oa)
        rg = oracle.backward(*oa, c["dy"], e["dlamT"], e["detaT"], dyvar=c["dyvar"])
    outs, grads = ("y", "yvar", "lamT", "etaT"), ("dq", "dk", "dv", "da", "dp", "dr")
    for res, want, names in ((out, ref, outs), (free, ref, outs), (got, rg, grads), (again, rg, grads)):
        for n in names:
            o, w = to_np(res[n]), np.asarray(want[n])
            keep = np.isfinite(w)
            assert keep.mean() > 0.5, n
            wrong = np.argwhere(keep & ~np.isfinite(o))[:4].tolist()
            assert not wrong, f"{n}: not finite at {wrong}"
            err = rel_err(o[keep], w[keep])
            assert err <= 1e-4, f"{n}: {err:.2e}"   # as the token-recurrent kernels' (see above)
