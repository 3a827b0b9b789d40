"""The per-channel kernels pick their lanes per channel and channels per workgroup by how far
the channels of all heads fill the chip: one sequence alone (few channels) against the same
sequence in a batch that fills it.  The two differ in the order of sums over n <= 128 channels
whose terms are rounded to fp32 (fp32 inputs: the key-side gradients): n 6e-8 of a term, judged
against 1% of the sums' rms of about sqrt(n) terms, 6e-8 sqrt(n) / 0.01 = 7e-5 at n = 128; and
by one bf16 rounding."""
import pytest

from kla_testutil import log, rel_err, to_np

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,dk,dv,dtype", [(19, 16, 128, "bf16"), (8, 128, 128, "bf16"), (33, 64, 64, "f32"),
                                           (17, 32, 32, "bf16"), (9, 128, 16, "f32"),
                                           (11, 128, 128, "f32"), (10, 64, 128, "f32")])
@pytest.mark.parametrize("ou", [False, True])
def test_few_and_many_channels_agree(T, dk, dv, dtype, ou):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_10743_amd as K
    log(f"per-channel lanes T{T} {dk} x {dv} {dtype} ou={ou}")
    B, H = 8192 // dv // 2 + 1, 2          # at least 8192 channels in the batch
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(T + dk)
    z = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, k, v, r = z(B, T, H, dk), z(B, T, H, dk) / dk ** 0.5, z(B, T, H, dv), 0.1 + z(B, T, H, dv).abs()
    dy, dyvar = z(B, T, H, dv).to(t), z(B, T, H, dv)
    q, k, v, r = (x.to(t) for x in (q, k, v, r))
    if ou:
        gates = [1 + 15 * torch.rand(H, dk, dv, generator=g, device="cuda"), z(H, dk, dv).abs() + 1,
                 0.001 + 0.1 * torch.rand(H, dk, dv, generator=g, device="cuda")]
        fwd = lambda s: K.kla_forward_pc_ou(q[s], k[s], v[s], *gates, r[s], want_var=True, save=True)
        bwd = lambda s, o: K.kla_backward_pc_ou(q[s], k[s], v[s], *gates, r[s], None, None, dy[s], saved=o["saved"],
                                                dyvar=dyvar[s])
        names = ("dq", "dk", "dv", "dr", "dlam0", "deta0")
    else:
        a, p = torch.sigmoid(z(B, T, H, dk) + 3).to(t), (0.05 * z(B, T, H, dk).abs()).to(t)
        fwd = lambda s: K.kla_forward_pc(q[s], k[s], v[s], a[s], p[s], r[s], want_var=True, save=True)
        bwd = lambda s, o: K.kla_backward_pc(q[s], k[s], v[s], a[s], p[s], r[s], None, None, dy[s], saved=o["saved"],
                                             dyvar=dyvar[s])
        names = ("dq", "dk", "dv", "da", "dp", "dr", "dlam0", "deta0")
    whole, one = slice(0, B), slice(B - 1, B)
    om, of = fwd(whole), fwd(one)
    gm, gf = bwd(whole, om), bwd(one, of)
    tol = 1.2e-2 if dtype == "bf16" else 1e-4   # bf16: one rounding apart is 2^-7 of the value
    for n in ("y", "yvar", "lamT", "etaT"):
        e = rel_err(to_np(of[n]), to_np(om[n][one]))
        assert e <= (tol if n == "y" else 1e-4), f"{n}: {e:.2e}"
    for n in names:
        e = rel_err(to_np(gf[n]), to_np(gm[n][one]))
        assert e <= (tol if gf[n].dtype == t else 1e-4), f"{n}: {e:.2e}"


# the fp64 forward at 128 key slots by its waves per SIMD: one, two and three (two with OU gates)
@pytest.mark.parametrize("heads,dv", [(512, 16), (520, 16), (1040, 16), (256, 32), (258, 32), (514, 32), (172, 128)])
@pytest.mark.parametrize("ou", [False, True])
def test_waves_per_simd_agree(heads, dv, ou):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_10743_amd as K
    log(f"per-channel forward, {heads} heads of 128 x {dv} ou={ou}")
    B, T, H, dk = heads // 2, 19, 2, 128
    g = torch.Generator(device="cuda").manual_seed(heads + dv)
    z = lambda *s: torch.randn(*s, generator=g, device="cuda")
    q, k, v, r = z(B, T, H, dk), z(B, T, H, dk) / dk ** 0.5, z(B, T, H, dv), 0.1 + z(B, T, H, dv).abs()
    if ou:
        gates = [1 + 15 * torch.rand(H, dk, dv, generator=g, device="cuda"), z(H, dk, dv).abs() + 1,
                 0.001 + 0.1 * torch.rand(H, dk, dv, generator=g, device="cuda")]
        fwd = lambda s, **kw: K.kla_forward_pc_ou(q[s], k[s], v[s], *gates, r[s], save=True, **kw)
    else:
        a, p = torch.sigmoid(z(B, T, H, dk) + 3), 0.05 * z(B, T, H, dk).abs()
        fwd = lambda s, **kw: K.kla_forward_pc(q[s], k[s], v[s], a[s], p[s], r[s], save=True, **kw)
    for one in (slice(0, 1), slice(B - 1, B)):
        om, on, of = fwd(slice(0, B), want_var=True), fwd(slice(0, B)), fwd(one, want_var=True)
        for n in ("y", "yvar", "lamT", "etaT"):   # fp64 sums of 128 terms in another order, stored in fp32
            e = rel_err(to_np(of[n]), to_np(om[n][one]))
            assert e <= 1e-4, f"{n}: {e:.2e}"
        assert torch.equal(on["y"], om["y"]) and torch.equal(on["etaT"], om["etaT"])
