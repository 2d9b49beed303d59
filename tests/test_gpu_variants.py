"""Feature-map variants and attention from given features (HIP path through the C
ABI) against the float64 oracle of the variants (oracle/luna_variants.py).

Inputs are rounded to the call's dtype before the oracle sees them (X and W), so
that the comparison measures the kernels' arithmetic.  Tolerances as everywhere:
normwise per (b, h) slice (per row for causal outputs), 1e-4 for fp32, 2e-2 for bf16.
"""
import math
import zlib

import numpy as np
import pytest

from gpu_util import assert_close, assert_close_rows, say, to_np, torch_dtype
from oracle import luna_variants as VAR
from paper_2512_08061_amd import luna

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _device():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    luna.load_library()
    yield
    torch.cuda.synchronize()


def _variant_params(rng, kind, M, d, L=4, hidden=16, act="relu", shared=False, nonneg=True, env=False, bank=False,
                    ch_rms=False, per_head=0):
    lead = (per_head,) if per_head else ()
    s = 1.0 / math.sqrt(d)
    p = {"kind": kind, "act": act, "M": M, "per_head": bool(per_head)}
    if kind == "performer":  # omega / d^(1/4), omega ~ N(0, I): unbiased for exp(x . y / sqrt(d))
        p["W"] = rng.standard_normal(lead + (M, d)) / d ** 0.25
        p["b"] = np.zeros(lead + (M,))
    elif kind in ("rff_cos", "rff_sincos"):
        p["W"] = rng.standard_normal(lead + (M, d)) * s
        p["b"] = rng.uniform(0, 2 * math.pi, lead + (M,))
    else:
        C1 = 1 if shared else L
        p.update(W=rng.standard_normal(lead + (M, d)) * s, b=rng.standard_normal(lead + (M,)) * s,
                 fc1_w=rng.standard_normal(lead + (C1, hidden)), fc1_b=rng.standard_normal(lead + (C1, hidden)),
                 fc2_w=rng.standard_normal(lead + (L, hidden)) * 0.3, fc2_b=rng.standard_normal(lead + (L,)) * 0.3 + 0.2,
                 L=L, hidden=hidden, nonneg=nonneg, shared_channels=shared)
        if env:
            p["env_w"] = rng.standard_normal(lead + (L, d)) * s
            p["env_b"] = rng.standard_normal(lead + (L,))
        if bank:
            p["bank"] = rng.standard_normal(lead + (L,))
        if ch_rms:
            p["ch_rms"], p["ch_rms_target"] = True, 0.05
    return p


def _upload_rounded(x, dtype):
    """x on the device in dtype, and the same values (rounded) for the oracle."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(x)).to("cuda").to(torch_dtype(dtype)).contiguous()
    return t, to_np(t)


def _run_variant(p, X, dtype, out_dtype=None):
    import torch
    Xt, Xr = _upload_rounded(X, dtype)
    v = luna.PhiVariant.from_arrays(p, torch.device("cuda:0"), torch_dtype(dtype))
    q = dict(p, W=to_np(v.base.W))  # the oracle takes W as the device holds it
    got = to_np(luna.featuremap_variant(Xt, v, out_dtype))
    return got, VAR.featuremap_variant(Xr, q)


MAP_CASES = [  # (kind, act, dtype, d, M, options)
    ("rff_cos", "relu", "f32", 64, 40, {}), ("rff_cos", "relu", "bf16", 128, 128, {}),
    ("rff_sincos", "relu", "f32", 32, 24, {}), ("rff_sincos", "relu", "bf16", 64, 64, {}),
    ("performer", "relu", "f32", 64, 48, {}), ("performer", "relu", "bf16", 128, 256, {}),
    ("mlp", "relu", "f32", 64, 16, {}), ("mlp", "gelu", "f32", 64, 16, {}), ("mlp", "silu", "bf16", 64, 20, {}),
    ("mlp", "tanh", "f32", 128, 9, dict(shared=True, nonneg=False)),
    ("mlp", "gelu", "f32", 32, 16, dict(env=True)), ("mlp", "relu", "bf16", 64, 16, dict(env=True, shared=True)),
    ("mlp", "silu", "f32", 64, 33, dict(bank=True)), ("mlp", "relu", "f32", 64, 16, dict(env=True, bank=True)),
    ("mlp", "tanh", "f32", 64, 12, dict(per_head=3, env=True)),
    ("rff_sincos", "relu", "f32", 64, 16, dict(per_head=3)),
]


@pytest.mark.parametrize("kind,act,dtype,d,M,opts", MAP_CASES)
def test_featuremap_variant(kind, act, dtype, d, M, opts):
    say(f"variant map {kind} act={act} {dtype} d={d} M={M} {opts}")
    rng = np.random.default_rng(zlib.crc32(f"{kind}/{act}/{d}/{M}/{sorted(opts)}".encode()))
    p = _variant_params(rng, kind, M, d, act=act, **opts)
    X = rng.standard_normal((2, 3, 77, d))
    got, ref = _run_variant(p, X, dtype)
    assert_close(got, ref, dtype, "phi")
    if dtype == "bf16":  # fp32 output from bf16 input at the fp32 bar
        import torch
        got32, _ = _run_variant(p, X, dtype, torch.float32)
        assert_close(got32, ref, "f32", "phi, fp32 out")


@pytest.mark.parametrize("dtype,bank", [("f32", False), ("bf16", False), ("f32", True)])
def test_featuremap_variant_channel_rms(dtype, bank):
    """Listing 1's channel RMS over the whole call (two passes), with channels both
    above the target (scaled down) and below it (unchanged)."""
    say(f"variant channel RMS {dtype} bank={bank}")
    rng = np.random.default_rng(41)
    p = _variant_params(rng, "mlp", 16, 64, L=4, act="gelu", ch_rms=True, bank=bank)
    p["fc2_b"] = np.array([2.0, 0.01, 0.5, 0.0])  # channel 0 large, channel 1 tiny
    p["ch_rms_target"] = 0.3
    X = rng.standard_normal((2, 3, 200, 64))
    got, ref = _run_variant(p, X, dtype)
    assert_close(got, ref, dtype, "phi with channel RMS")


ATTN_CASES = [  # (feature dtype, value dtype, d, D, n, causal)
    ("f32", "f32", 64, 64, 97, False), ("f32", "f32", 64, 100, 333, True), ("bf16", "bf16", 128, 256, 700, False),
    ("bf16", "bf16", 128, 256, 1000, True), ("bf16", "bf16", 64, 128, 333, True), ("bf16", "f32", 32, 48, 129, True),
    ("f32", "bf16", 128, 256, 65, True),
    # widths that only the fp32 GEMM path takes, over several chunks and 512-token pieces
    ("f32", "f32", 48, 100, 130, True), ("bf16", "f32", 48, 100, 1100, False), ("bf16", "bf16", 64, 300, 700, True),
    ("f32", "bf16", 64, 300, 1025, False), ("f32", "f32", 256, 512, 200, True), ("bf16", "bf16", 256, 512, 600, False),
    ("f32", "f32", 9, 1, 65, True), ("f32", "f32", 33, 512, 513, False), ("bf16", "bf16", 48, 257, 64, True),
]


@pytest.mark.parametrize("fdt,vdt,d,D,n,causal", ATTN_CASES)
def test_attn_from_features(fdt, vdt, d, D, n, causal):
    """Positive random features (exp of a Gaussian projection), so that denominators
    stay away from 0.  The bf16 causal cases with (d, D) = (128, 256) and (64, 128) run on
    the causal scan kernel; d in {32, 64, 128} with D <= 256 otherwise on the kernels that
    read the features as they are (non-causal) or the fp32 chunk kernels (causal); all other
    widths on fp32 GEMMs."""
    say(f"attention from features {fdt}/{vdt} d={d} D={D} n={n} causal={causal}")
    rng = np.random.default_rng(42 + n)
    B, H = 2, 3
    fq = np.exp(rng.standard_normal((B, H, n, D)) * 0.5) / math.sqrt(D)
    fk = np.exp(rng.standard_normal((B, H, n, D)) * 0.5) / math.sqrt(D)
    V = rng.standard_normal((B, H, n, d))
    (tq, rq), (tk, rk), (tv, rv) = (_upload_rounded(a, dt) for a, dt in ((fq, fdt), (fk, fdt), (V, vdt)))
    got = to_np(luna.attn_fwd_features(tq, tk, tv, causal=causal))
    ref = VAR.attn_from_features(rq, rk, rv, causal=causal)
    tol_dt = "f32" if (fdt == "f32" and vdt == "f32") else "bf16"
    (assert_close_rows if causal else assert_close)(got, ref, tol_dt, "out")


@pytest.mark.parametrize("kind,causal", [("performer", False), ("performer", True), ("rff_sincos", True),
                                         ("mlp", False)])
def test_variant_attention_end_to_end(kind, causal):
    """A variant map of Q and K, then attention from the features, against the oracle's
    composition.  The sin/cos features are taken at small inputs, where the kernel
    cos(u_x - u_y) stays near 1 (positive denominators)."""
    import torch
    say(f"variant attention {kind} causal={causal}")
    rng = np.random.default_rng(43)
    B, H, n, d = 2, 2, 150, 64
    p = _variant_params(rng, kind, 32, d, L=4, act="silu", env=(kind == "mlp"))
    scale = 0.2 if kind == "rff_sincos" else 0.7
    Q, K = rng.standard_normal((B, H, n, d)) * scale, rng.standard_normal((B, H, n, d)) * scale
    V = rng.standard_normal((B, H, n, d))
    v = luna.PhiVariant.from_arrays(p, torch.device("cuda:0"), torch.float32)
    tq, tk, tv = (torch.from_numpy(a).float().cuda().contiguous() for a in (Q, K, V))
    out = to_np(luna.attn_fwd_features(luna.featuremap_variant(tq, v), luna.featuremap_variant(tk, v), tv,
                                       causal=causal))
    ref = VAR.attn_from_features(VAR.featuremap_variant(Q, p), VAR.featuremap_variant(K, p), V, causal=causal)
    (assert_close_rows if causal else assert_close)(out, ref, "f32", "out")


def test_features_of_the_base_map():
    """luna_featuremap's own output through attention from features equals luna_attn_fwd
    (the same eq. (9) on the same features, to the bf16 bar)."""
    import torch
    from gpu_util import inputs, small_workload, upload
    w = small_workload("bf16", B=2, H=3, n=300, d=64, M=16, L=8)
    Q, K, V, p = inputs(w, seed=44)
    (Qt, Kt, Vt), pt = upload(w, [Q, K, V], p)
    f32 = torch.float32
    out = to_np(luna.attn_fwd_features(luna.featuremap(Qt, pt, f32), luna.featuremap(Kt, pt, f32), Vt))
    assert_close(out, to_np(luna.attn_fwd(Qt, Kt, Vt, pt)), "bf16", "features vs fused")


@pytest.mark.parametrize("pdt,dt,d,D,n", [
    ("bf16", "bf16", 32, 5, 31), ("bf16", "bf16", 64, 64, 512), ("bf16", "bf16", 64, 72, 513), ("bf16", "f32", 64, 128, 33),
    ("bf16", "bf16", 128, 256, 1100), ("f32", "bf16", 32, 130, 97), ("f32", "f32", 128, 250, 600), ("f32", "f32", 64, 16, 1),
    ("f32", "bf16", 128, 129, 257), ("bf16", "f32", 128, 200, 40)])
def test_attn_features_noncausal_edges(pdt, dt, d, D, n):
    """Non-causal attention from features of either type beside values of either type, at
    the edges of the 32-token tiles, 512-token pieces and 16- and 64-feature blocks, with
    feature rows that are not whole 16-byte pieces."""
    say(f"features non-causal phi={pdt} {dt} d={d} D={D} n={n}")
    rng = np.random.default_rng(1000 * D + n)
    fq, fqr = _upload_rounded(np.abs(rng.standard_normal((2, 3, n, D))), pdt)
    fk, fkr = _upload_rounded(np.abs(rng.standard_normal((2, 3, n, D))), pdt)
    V, Vr = _upload_rounded(rng.standard_normal((2, 3, n, d)), dt)
    out = to_np(luna.attn_fwd_features(fq, fk, V))
    assert_close(out, VAR.attn_from_features(fqr, fkr, Vr), dt, "out")


@pytest.mark.parametrize("kind,dtype,d,M,n", [
    ("performer", "bf16", 64, 128, 200), ("performer", "f32", 128, 64, 63), ("rff_cos", "bf16", 32, 8, 65),
    ("rff_cos", "f32", 64, 36, 64), ("rff_cos", "bf16", 128, 72, 1), ("rff_sincos", "bf16", 64, 12, 129),
    ("rff_sincos", "f32", 32, 32, 130), ("rff_sincos", "bf16", 128, 64, 77), ("performer", "bf16", 64, 96, 128)])
def test_featuremap_variant_rows(kind, dtype, d, M, n):
    """One-feature kinds with rows of whole 16-byte pieces up to 256 bytes: one, two and four
    projection blocks across the waves, piece counts that are and are not powers of two,
    feature counts off the 8- and 32-projection steps, rows off the 64-row items."""
    say(f"variant rows {kind} {dtype} d={d} M={M} n={n}")
    rng = np.random.default_rng(zlib.crc32(f"rows/{kind}/{d}/{M}/{n}".encode()))
    p = _variant_params(rng, kind, M, d)
    X = rng.standard_normal((2, 3, n, d))
    got, ref = _run_variant(p, X, dtype)
    assert_close(got, ref, dtype, "phi")


def _positive_features(rng, shape):
    return np.exp(rng.standard_normal(shape) * 0.5) / math.sqrt(shape[-1])


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,D,n", [(32, 48, 200), (64, 128, 700), (128, 256, 200)])
def test_attn_features_infinite_values(d, D, n, causal):
    """A bf16 infinity in V beside fp32 features: its column is infinite (not NaN) for every
    row that sees it, the other columns are as without it."""
    say(f"features beside infinite values d={d} D={D} n={n} causal={causal}")
    rng = np.random.default_rng(45 + D)
    fq, rq = _upload_rounded(_positive_features(rng, (1, 2, n, D)), "f32")
    fk, rk = _upload_rounded(_positive_features(rng, (1, 2, n, D)), "f32")
    V, rv = _upload_rounded(rng.standard_normal((1, 2, n, d)), "bf16")
    t, c = 70, 3
    for h, x in enumerate((math.inf, -math.inf)):
        V[0, h, t, c] = x
        rv[0, h, t, c] = 0.0
    got = to_np(luna.attn_fwd_features(fq, fk, V, causal=causal))
    ref = VAR.attn_from_features(rq, rk, rv, causal=causal)
    first = t if causal else 0
    assert (got[0, 0, first:, c] == math.inf).all() and (got[0, 1, first:, c] == -math.inf).all()
    cols = [i for i in range(d) if i != c]
    assert_close_rows(got[..., cols], ref[..., cols], "bf16", "other columns")
    if causal:  # (rows before t in its own 64-token tile meet it as 0 times infinity)
        assert_close_rows(got[:, :, :64], ref[:, :, :64], "bf16", "rows before its tile")


@pytest.mark.parametrize("d,M", [(128, 256), (128, 200), (64, 100)])
def test_attn_state_infinite_value(d, M):
    """The same in the state of shapes whose features are held in fp32."""
    from gpu_util import inputs, small_workload, upload
    import torch
    n, t, c = 600, 70, 3
    w = small_workload("bf16", B=1, H=2, n=n, d=d, M=M, L=1)
    say(f"state beside an infinite value {w.name}")
    _, K, V, p = inputs(w, seed=46)
    p = dict(p, fc2_b=np.abs(p["fc2_b"]) + 1.0)
    (Kt, Vt), pt = upload(w, [K, V], p)
    Vt[:, :, t, c] = 0.0
    S0, z0 = luna.attn_state(Kt, Vt, pt)
    Vt[0, :, t, c] = torch.tensor([math.inf, -math.inf])
    S, z = luna.attn_state(Kt, Vt, pt)
    phi = luna.featuremap(Kt, pt, torch.float32)[0, :, t]  # [H][M]
    assert (phi > 0).float().mean() > 0.5
    for h, x in enumerate((math.inf, -math.inf)):
        assert (S[0, h, phi[h] > 0, c] == x).all()
    cols = [i for i in range(d) if i != c]
    # (the columns beside it may be summed in another order: twice n roundings of the terms)
    phi_all = luna.featuremap(Kt, pt, torch.float32)
    Vt[:, :, t, c] = 0.0
    terms = torch.matmul(phi_all.transpose(-1, -2).contiguous(), Vt.float().abs())
    assert ((S - S0)[..., cols].abs() <= 2 * n * 2.0 ** -24 * terms[..., cols]).all()
    assert torch.equal(z, z0)


@pytest.mark.parametrize("pdt,dt,D,n,causal", [("bf16", "f32", 64, 40, False), ("f32", "bf16", 1, 1, True),
                                               ("bf16", "f32", 48, 1, False)])
def test_attn_features_largest_values(pdt, dt, D, n, causal):
    """fp32 operands above the largest bf16 value: sums that fp32 holds stay finite."""
    import torch
    say(f"largest fp32 values phi={pdt} {dt} D={D} n={n} causal={causal}")
    big = 3.4e38
    V = torch.full((1, 1, n, 32), 0.5, dtype=torch_dtype(dt), device="cuda")
    if dt == "f32":  # (statistics of up to 3.4e38 from features of 1, read out by features of 2^-8)
        fq = torch.full((1, 1, n, D), 2.0 ** -8, dtype=torch_dtype(pdt), device="cuda")
        fk = torch.ones((1, 1, n, D), dtype=torch_dtype(pdt), device="cuda")
        V[0, 0, 0, ::2], V[0, 0, 0, 1::2] = big, -big
        ref = V.double().sum(2, keepdim=True) / n
    else:  # one token whose kernel value is 3.4e38
        fq = torch.full((1, 1, n, D), 1.8e19, dtype=torch.float32, device="cuda")
        fk = torch.full((1, 1, n, D), 1.8888e19, dtype=torch.float32, device="cuda")
        ref = V.double()
    got = luna.attn_fwd_features(fq, fk, V, causal=causal, eps=0.0)
    assert_close(to_np(got), ref.expand(got.shape).cpu().numpy(), dt, "out")


def test_attn_features_without_workspace():
    """A short causal call on the scan kernel, for which no workspace is asked: one part a head."""
    import torch
    rng = np.random.default_rng(48)
    n, d, D = 255, 64, 128
    say(f"features without workspace n={n}")
    (fq, rq), (fk, rk) = (_upload_rounded(_positive_features(rng, (2, 3, n, D)), "bf16") for _ in range(2))
    V, rv = _upload_rounded(rng.standard_normal((2, 3, n, d)), "bf16")
    out = torch.empty_like(V)
    st = luna.load_library().luna_attn_fwd_features(fq.data_ptr(), fk.data_ptr(), luna.LUNA_BF16, V.data_ptr(),
                                                    luna.LUNA_BF16, 2, 3, n, d, D, 1, 64, 1e-6, out.data_ptr(), None, 0,
                                                    torch.cuda.current_stream().cuda_stream)
    assert st == luna.LUNA_OK
    assert_close_rows(to_np(out), VAR.attn_from_features(rq, rk, rv, causal=True), "bf16", "out")


@pytest.mark.parametrize("causal", [False, True])
def test_attn_features_more_heads_than_one_launch(causal):
    """8.4 million heads and more, of one or two tokens: the launches of every kernel are cut
    at 2^31 threads."""
    import torch
    heads, n, d, eps = (1 << 23) + 1001, 2 if causal else 1, 32, 1e-3
    say(f"features, {heads} heads causal={causal}")
    g = torch.Generator(device="cuda").manual_seed(47)
    fq, fk = (torch.rand((1, heads, n, 1), generator=g, device="cuda") + 0.5 for _ in range(2))
    V = torch.randn((1, heads, n, d), generator=g, device="cuda").to(torch.bfloat16)
    out = luna.attn_fwd_features(fq, fk, V, causal=causal, eps=eps)
    num = (torch.cumsum(fk * V.float(), 2) if causal else fk * V.float()) * fq
    den = (torch.cumsum(fk, 2) if causal else fk) * fq + eps
    # (the only rounding beyond fp32 sums of at most two terms is the output's own to bf16)
    assert ((out.float() - num / den).abs() <= 2.0 ** -8 * (num / den).abs() + 1e-6).all()


@pytest.mark.parametrize("pdt,dt,d,D,B,H,n", [
    ("f32", "f32", 128, 256, 1, 150, 70), ("f32", "bf16", 128, 200, 2, 65, 33), ("bf16", "bf16", 64, 256, 1, 129, 64),
    ("f32", "f32", 64, 128, 1, 257, 45), ("bf16", "f32", 32, 256, 1, 100, 40), ("bf16", "bf16", 128, 72, 1, 140, 97)])
def test_attn_features_many_heads(pdt, dt, d, D, B, H, n):
    """Non-causal attention from features with as many pieces as the state kernel gives all, or
    half, of their features to one workgroup (few pieces give a quarter)."""
    say(f"features many heads phi={pdt} {dt} d={d} D={D} B={B} H={H} n={n}")
    rng = np.random.default_rng(2000 * D + n)
    fq, fqr = _upload_rounded(np.abs(rng.standard_normal((B, H, n, D))), pdt)
    fk, fkr = _upload_rounded(np.abs(rng.standard_normal((B, H, n, D))), pdt)
    V, Vr = _upload_rounded(rng.standard_normal((B, H, n, d)), dt)
    assert_close(to_np(luna.attn_fwd_features(fq, fk, V)), VAR.attn_from_features(fqr, fkr, Vr), dt, "out")
