"""The C ABI without a GPU: the library loads, exports what include/luna.h declares,
and rejects bad arguments on the host with the documented status codes."""
import ctypes

import pytest

from paper_2512_08061_amd import luna

FAKE = 0x10000  # non-null pointer value; validation never dereferences it


def _params(M=16, L=8, hidden=64, shared=0, nonneg=1, per_head=0, nullW=False):
    return luna.PhiParamsC(M, L, hidden, shared, nonneg, per_head, 0 if nullW else FAKE, FAKE, FAKE, FAKE, FAKE,
                           FAKE)


@pytest.fixture(scope="module")
def lib():
    return luna.load_library()


def test_exports_every_declared_symbol(lib):
    names = luna.header_functions()
    assert set(names) == {"luna_workspace_bytes", "luna_featuremap", "luna_attn_fwd", "luna_attn_fwd_causal",
                          "luna_attn_state", "luna_attn_causal_step", "luna_status_string", "luna_last_error",
                          "luna_attn_fwd_causal_noalloc", "luna_noalloc_scratch_bytes", "luna_attn_bwd",
                          "luna_phi_variant_features", "luna_featuremap_variant_workspace_bytes",
                          "luna_featuremap_variant", "luna_attn_features_workspace_bytes", "luna_attn_fwd_features",
                          "luna_distill_workspace_bytes", "luna_distill"}
    for name in names:
        assert hasattr(lib, name), name


def test_status_strings(lib):
    for s in range(5):
        assert lib.luna_status_string(s)
    assert lib.luna_status_string(99) == b"unknown status"


def _attn(lib, B=2, H=3, n=100, d=64, p=None, eps=1e-6, ws=FAKE, ws_bytes=1 << 40, q=FAKE, dt=luna.LUNA_BF16):
    p = p or _params()
    return lib.luna_attn_fwd(q, FAKE, FAKE, dt, B, H, n, d, ctypes.byref(p), eps, FAKE, ws, ws_bytes, None)


def _causal(lib, chunk=64, d=128, M=32, dt=luna.LUNA_BF16, **kw):
    p = _params(M=M)
    return lib.luna_attn_fwd_causal(FAKE, FAKE, FAKE, dt, 1, 1, 100, d, ctypes.byref(p), chunk, 1e-6, FAKE,
                                    FAKE, 1 << 40, None)


@pytest.mark.parametrize("kw,status", [
    (dict(n=0), luna.LUNA_ERR_INVALID_ARG),
    (dict(B=0), luna.LUNA_ERR_INVALID_ARG),
    (dict(d=48), luna.LUNA_ERR_UNSUPPORTED),
    (dict(q=0), luna.LUNA_ERR_INVALID_ARG),
    (dict(eps=-1.0), luna.LUNA_ERR_INVALID_ARG),
    (dict(eps=float("nan")), luna.LUNA_ERR_INVALID_ARG),
    (dict(ws_bytes=1024), luna.LUNA_ERR_WORKSPACE),
    (dict(ws=FAKE + 8), luna.LUNA_ERR_INVALID_ARG),
    (dict(p=_params(M=0)), luna.LUNA_ERR_INVALID_ARG),
    (dict(p=_params(M=32, L=16)), luna.LUNA_ERR_INVALID_ARG),
    (dict(p=_params(hidden=65)), luna.LUNA_ERR_INVALID_ARG),
    (dict(p=_params(nonneg=2)), luna.LUNA_ERR_INVALID_ARG),
    (dict(p=_params(nullW=True)), luna.LUNA_ERR_INVALID_ARG),
    (dict(p=_params(L=16, hidden=64)), luna.LUNA_ERR_UNSUPPORTED),
    (dict(dt=7), luna.LUNA_ERR_INVALID_ARG),
])
def test_noncausal_rejects(lib, kw, status):
    assert _attn(lib, **kw) == status
    assert lib.luna_last_error()  # a reason is recorded


def test_causal_rejects_chunk(lib):
    assert _causal(lib, chunk=32) == luna.LUNA_ERR_UNSUPPORTED
    assert b"chunk" in lib.luna_last_error()


def test_featuremap_rejects(lib):
    p = _params()
    assert lib.luna_featuremap(FAKE, luna.LUNA_BF16, 1, 1, 10, 64, ctypes.byref(p), FAKE, 5, FAKE, 1 << 40,
                               None) == luna.LUNA_ERR_INVALID_ARG
    assert lib.luna_featuremap(0, luna.LUNA_BF16, 1, 1, 10, 64, ctypes.byref(p), FAKE, luna.LUNA_BF16, FAKE,
                               1 << 40, None) == luna.LUNA_ERR_INVALID_ARG
    p3 = _params(L=3)
    assert lib.luna_featuremap(FAKE, luna.LUNA_BF16, 1, 1, 10, 64, ctypes.byref(p3), FAKE, luna.LUNA_BF16, FAKE,
                               1 << 40, None) == luna.LUNA_ERR_UNSUPPORTED


def test_state_and_step_reject(lib):
    p = _params()
    st = lambda **kw: lib.luna_attn_state(kw.get("k", FAKE), FAKE, luna.LUNA_BF16, 2, 3, kw.get("n", 100), 64,
                                          ctypes.byref(kw.get("p", p)), kw.get("acc", 0), kw.get("S", FAKE), FAKE,
                                          FAKE, kw.get("ws_bytes", 1 << 40), None)
    assert st(k=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(S=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(acc=2) == luna.LUNA_ERR_INVALID_ARG
    assert st(n=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(ws_bytes=256) == luna.LUNA_ERR_WORKSPACE
    assert st(p=_params(L=3)) == luna.LUNA_ERR_UNSUPPORTED
    stp = lambda **kw: lib.luna_attn_causal_step(FAKE, FAKE, FAKE, luna.LUNA_BF16, 2, 3, kw.get("m", 4), 64,
                                                 ctypes.byref(kw.get("p", p)), kw.get("eps", 1e-6),
                                                 kw.get("ready", 0), kw.get("S", FAKE), FAKE, kw.get("out", FAKE),
                                                 FAKE, kw.get("ws_bytes", 1 << 40), None)
    assert stp(S=0) == luna.LUNA_ERR_INVALID_ARG
    assert stp(out=0) == luna.LUNA_ERR_INVALID_ARG
    assert stp(eps=-1.0) == luna.LUNA_ERR_INVALID_ARG
    assert stp(m=0) == luna.LUNA_ERR_INVALID_ARG
    assert stp(ready=2) == luna.LUNA_ERR_INVALID_ARG
    assert stp(ws_bytes=256) == luna.LUNA_ERR_WORKSPACE
    assert stp(p=_params(L=3)) == luna.LUNA_ERR_UNSUPPORTED
    assert lib.luna_last_error()
    # workspace: tables plus the new tokens' features (fp32) for a step; tables plus
    # partial statistics for the state
    nb1 = lib.luna_workspace_bytes(luna.OP_CAUSAL_STEP, luna.LUNA_BF16, 2, 3, 1, 64, ctypes.byref(p), 64)
    nb9 = lib.luna_workspace_bytes(luna.OP_CAUSAL_STEP, luna.LUNA_BF16, 2, 3, 9, 64, ctypes.byref(p), 64)
    assert 0 < nb1 < nb9 and nb9 % 256 == 0
    assert lib.luna_workspace_bytes(luna.OP_STATE, luna.LUNA_BF16, 8, 16, 16384, 128, ctypes.byref(_params(M=32)),
                                    64) > 0


def test_workspace_sizes(lib):
    # the five measured problems all have kernels and finite workspaces
    for (dt, B, H, n, d, M, op) in [(luna.LUNA_F32, 1, 1, 256, 32, 8, luna.OP_ATTN),
                                    (luna.LUNA_BF16, 32, 12, 512, 64, 8, luna.OP_ATTN),
                                    (luna.LUNA_BF16, 64, 12, 197, 64, 16, luna.OP_ATTN),
                                    (luna.LUNA_BF16, 32, 8, 4096, 64, 16, luna.OP_ATTN),
                                    (luna.LUNA_BF16, 8, 16, 16384, 128, 32, luna.OP_ATTN_CAUSAL)]:
        p = _params(M=M)
        nb = lib.luna_workspace_bytes(op, dt, B, H, n, d, ctypes.byref(p), 64)
        assert 0 < nb < 1 << 30, (n, nb)
        assert nb % 256 == 0
        nbf = lib.luna_workspace_bytes(luna.OP_FEATUREMAP, dt, B, H, n, d, ctypes.byref(p), 64)
        assert nbf > 0
    p = _params()
    assert lib.luna_workspace_bytes(9, luna.LUNA_BF16, 1, 1, 1, 64, ctypes.byref(p), 64) == 0
    # per-head parameters need one table per head
    ph = _params(per_head=1)
    one = lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 2, 4, 64, 64, ctypes.byref(p), 64)
    four = lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 2, 4, 64, 64, ctypes.byref(ph), 64)
    assert four > one


def test_generic_path_planning(lib):
    """Shapes without a fused kernel run in fp32: their workspace holds the features of the
    queries and keys and the statistics of pieces of 128 tokens (causal) or 512 tokens, and
    the piece count is capped; M above 256 is invalid."""
    d, n, B, H = 128, 16384, 8, 16
    rows = B * H * n
    p200 = _params(M=200, L=1)
    for op, piece in [(luna.OP_ATTN_CAUSAL, 128), (luna.OP_ATTN, 512)]:
        nb = lib.luna_workspace_bytes(op, luna.LUNA_BF16, B, H, n, d, ctypes.byref(p200), 64)
        floor = rows * 2 * 200 * 4 + B * H * (n // piece) * 200 * 129 * 4
        assert floor <= nb <= floor + (1 << 20), (op, nb, floor)
    # one channel per projection with 256 features at d = 128, causal: the features of
    # Q and K in bf16, then the scan kernel (its state pieces are a few MB)
    p1 = _params(M=256, L=1)
    nb = lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, B, H, n, d, ctypes.byref(p1), 64)
    assert rows * 256 * 2 * 2 <= nb <= rows * 256 * 2 * 2 + (64 << 20), nb
    # fused shapes keep their small workspaces
    assert lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, B, H, n, d, ctypes.byref(_params(M=32)),
                                    64) < 1 << 30
    # the fused one-channel non-causal kernel (M = 128, d = 64) needs only the tables
    assert lib.luna_workspace_bytes(luna.OP_ATTN, luna.LUNA_BF16, 32, 8, 4096, 64, ctypes.byref(_params(M=128, L=1)),
                                    64) < 1 << 20
    assert lib.luna_workspace_bytes(luna.OP_STATE, luna.LUNA_BF16, 2, 3, 1000, 128, ctypes.byref(p1), 64) > 0
    # chunk counts above 65535 are refused before anything runs
    big = lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 1, 1, 65535 * 64 + 1, d, ctypes.byref(p200),
                                   64)
    assert big == 0
    assert lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 1, 1, 65535 * 64, d, ctypes.byref(p200),
                                    64) > 0
    assert lib.luna_workspace_bytes(luna.OP_ATTN, luna.LUNA_BF16, 1, 1, 65535 * 512 + 1, d, ctypes.byref(p200),
                                    64) == 0
    p257 = _params(M=257, L=1)
    assert lib.luna_workspace_bytes(luna.OP_ATTN, luna.LUNA_BF16, 1, 1, 64, d, ctypes.byref(p257), 64) == 0
    assert _attn(lib, p=p257) == luna.LUNA_ERR_INVALID_ARG
    # an L the feature-map kernel is not built for stays unsupported
    assert _attn(lib, p=_params(M=16, L=3)) == luna.LUNA_ERR_UNSUPPORTED


def test_noalloc_refuses_beyond_scratch_on_host(lib):
    """A causal problem whose workspace exceeds the static scratch is refused before
    any HIP call (per-head parameters: one table per head, 1024 heads)."""
    p = _params(M=32, per_head=1)
    need = lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 1, 1024, 64, 128, ctypes.byref(p), 64)
    assert need > lib.luna_noalloc_scratch_bytes() == 64 << 20
    st = lib.luna_attn_fwd_causal_noalloc(FAKE, FAKE, FAKE, luna.LUNA_BF16, 1, 1024, 64, 128, ctypes.byref(p), 64,
                                          1e-6, FAKE, None)
    assert st == luna.LUNA_ERR_WORKSPACE
    assert b"static scratch" in lib.luna_last_error()


def _variant(lib, kind=0, act=0, M=16, L=8, hidden=64, env=False, bank=False, ch_rms=0, target=0.1, base=None):
    base = base or _params(M=M, L=L, hidden=hidden)
    v = luna.PhiVariantC(kind, act, ctypes.pointer(base), FAKE if env else None, FAKE if env else None,
                         FAKE if bank else None, ch_rms, target)
    v._base = base  # keep the parameters alive
    return v


def test_variant_features_and_rejects(lib):
    """Feature counts of the variants and their argument checks, on the host."""
    feats = lambda v: lib.luna_phi_variant_features(ctypes.byref(v))  # noqa: E731
    assert feats(_variant(lib)) == 128                      # M L
    assert feats(_variant(lib, bank=True)) == 16            # Bank+Coef: M
    assert feats(_variant(lib, kind=1)) == 16               # RFF cos: M
    assert feats(_variant(lib, kind=2)) == 32               # sin/cos: 2 M
    assert feats(_variant(lib, kind=3)) == 16               # Performer: M
    assert feats(_variant(lib, kind=4)) == -1               # unknown kind
    assert feats(_variant(lib, act=7)) == -1                # unknown activation
    assert feats(_variant(lib, kind=1, env=True)) == -1     # envelope only with the MLP kind
    assert feats(_variant(lib, kind=3, ch_rms=1)) == -1
    assert feats(_variant(lib, ch_rms=1, target=0.0)) == -1
    assert feats(_variant(lib, ch_rms=1, target=float("nan"))) == -1
    assert feats(_variant(lib, M=64, L=16)) == -1           # more than 512 features
    assert feats(_variant(lib, M=300, L=1)) == -1
    # workspace: the channel RMS partials, else none
    ws = lambda v: lib.luna_featuremap_variant_workspace_bytes(luna.LUNA_BF16, 2, 3, 100, 64, ctypes.byref(v))  # noqa: E731
    assert ws(_variant(lib)) == 0 and ws(_variant(lib, ch_rms=1)) > 0
    v = _variant(lib)
    st = lambda **kw: lib.luna_featuremap_variant(kw.get("x", FAKE), luna.LUNA_BF16, 2, 3, kw.get("n", 100),  # noqa: E731
                                                   kw.get("d", 64), ctypes.byref(kw.get("v", v)), FAKE,
                                                   kw.get("odt", luna.LUNA_BF16), FAKE, 1 << 40, None)
    assert st(x=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(n=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(d=48) == luna.LUNA_ERR_UNSUPPORTED
    assert st(odt=5) == luna.LUNA_ERR_INVALID_ARG
    assert st(v=_variant(lib, kind=9)) == luna.LUNA_ERR_INVALID_ARG
    rms = _variant(lib, ch_rms=1)
    assert lib.luna_featuremap_variant(FAKE, luna.LUNA_BF16, 2, 3, 100, 64, ctypes.byref(rms), FAKE, luna.LUNA_BF16,
                                       FAKE, 256, None) == luna.LUNA_ERR_WORKSPACE


def test_attn_features_planning(lib):
    """Attention from given features: the causal scan kernel for bf16 features with
    (d, D) = (128, 256) (state pieces only), otherwise fp32 (copies of bf16 features, states
    of 128-token pieces); argument checks on the host."""
    B, H, n = 8, 16, 16384
    wsb = lambda pdt, dt, d, D, causal, chunk=64: lib.luna_attn_features_workspace_bytes(  # noqa: E731
        pdt, dt, B, H, n, d, D, causal, chunk)
    given = wsb(luna.LUNA_BF16, luna.LUNA_BF16, 128, 256, 1)
    assert 0 < given < 64 << 20
    rows = B * H * n
    states = B * H * (n // 128) * 256 * 129 * 4
    fp32 = wsb(luna.LUNA_F32, luna.LUNA_BF16, 128, 256, 1)
    assert states <= fp32 < states + (1 << 20)
    widened = wsb(luna.LUNA_BF16, luna.LUNA_F32, 128, 256, 1)
    assert 0 <= widened - fp32 - rows * 256 * 8 < 1 << 20  # plus the fp32 copies
    assert wsb(luna.LUNA_BF16, luna.LUNA_BF16, 128, 256, 1, chunk=32) == 0
    assert wsb(luna.LUNA_BF16, luna.LUNA_BF16, 128, 600, 0) == 0
    assert wsb(luna.LUNA_BF16, luna.LUNA_BF16, 300, 64, 0) == 0
    assert wsb(luna.LUNA_BF16, 7, 64, 64, 0) == 0
    call = lambda **kw: lib.luna_attn_fwd_features(FAKE, FAKE, luna.LUNA_BF16, kw.get("v", FAKE), luna.LUNA_BF16, 2,  # noqa: E731
                                                   3, 100, 64, 64, kw.get("causal", 0), 64, kw.get("eps", 1e-6),
                                                   FAKE, FAKE, kw.get("ws", 1 << 40), None)
    assert call(v=0) == luna.LUNA_ERR_INVALID_ARG
    assert call(causal=2) == luna.LUNA_ERR_INVALID_ARG
    assert call(eps=-1.0) == luna.LUNA_ERR_INVALID_ARG
    assert call(ws=16) == luna.LUNA_ERR_WORKSPACE


def test_distill_planning_and_rejects(lib):
    """The distillation loss: supported feature counts per dtype, a workspace that grows
    with the gradients (feature gradients and the feature-map backward's buffers), and
    argument checks on the host."""
    wsb = lambda M, L, dt=luna.LUNA_BF16, d=64, grads=0, n=300: lib.luna_distill_workspace_bytes(  # noqa: E731
        dt, 2, 3, n, d, ctypes.byref(_params(M=M, L=L)), grads)
    assert wsb(16, 8) > 0 and wsb(8, 8) > 0 and wsb(32, 8) > 0 and wsb(256, 1) > 0   # D = 128, 64, 256, 256
    assert wsb(16, 8, luna.LUNA_F32) > 0 and wsb(32, 8, luna.LUNA_F32) == 0          # fp32: D <= 128
    assert wsb(12, 8) == 0 and wsb(3, 5) == 0 and wsb(16, 4) > 0                     # D = 96, 15, 64
    rows, D = 2 * 3 * 300, 128
    with_grads = wsb(16, 8, grads=1)
    assert with_grads - wsb(16, 8) >= 2 * rows * D * 4  # fp32 feature gradients of Q and K
    assert wsb(16, 8, d=48) == 0
    p = _params()
    st = lambda **kw: lib.luna_distill(kw.get("q", FAKE), FAKE, kw.get("dt", luna.LUNA_BF16), 2, 3,  # noqa: E731
                                       kw.get("n", 300), 64, ctypes.byref(kw.get("p", p)), kw.get("causal", 0),
                                       kw.get("eps", 1e-6), kw.get("loss", FAKE), None, FAKE, kw.get("ws", 1 << 40),
                                       None)
    assert st(q=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(loss=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(causal=2) == luna.LUNA_ERR_INVALID_ARG
    assert st(eps=-1.0) == luna.LUNA_ERR_INVALID_ARG
    assert st(n=0) == luna.LUNA_ERR_INVALID_ARG
    assert st(p=_params(M=12, L=8)) == luna.LUNA_ERR_UNSUPPORTED
    assert st(ws=256) == luna.LUNA_ERR_WORKSPACE


# (op, dtype, heads, n, d, M, L): bytes that the call has to do with, fewer than it asks for
SMALL_WORKSPACES = [
    (luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 16, 1024, 128, 32, 8, 17013248),
    (luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 8, 1999, 128, 256, 1, 32332288),
    (luna.OP_ATTN_CAUSAL, luna.LUNA_F32, 3, 321, 64, 16, 8, 304640),
    (luna.OP_ATTN, luna.LUNA_F32, 1, 256, 32, 8, 8, 146432),
    (luna.OP_ATTN, luna.LUNA_F32, 1, 1999, 128, 32, 8, 6790656),
    (luna.OP_ATTN, luna.LUNA_BF16, 1, 600, 128, 256, 1, 2217472),
    (luna.OP_STATE, luna.LUNA_BF16, 4, 1000, 64, 16, 8, 637440),
    (luna.OP_STATE, luna.LUNA_F32, 1, 2000, 128, 32, 8, 3713536),
    (luna.OP_ATTN_BWD, luna.LUNA_F32, 1, 1999, 128, 32, 8, 10601984),
]


@pytest.mark.parametrize("op,dt,heads,n,d,M,L,few", SMALL_WORKSPACES)
def test_small_workspaces(lib, op, dt, heads, n, d, M, L, few):
    """A workspace that holds the statistics in few pieces (the cut of a causal head in two,
    512 tokens, token ranges of 256) is accepted although the call asks for more; one that
    holds no table is refused.  (The size is checked before the pointer, which is
    misaligned, so that nothing is enqueued.)"""
    p = _params(M=M, L=L)
    assert lib.luna_workspace_bytes(op, dt, 1, heads, n, d, ctypes.byref(p), 64) > few
    g = luna.PhiGradsC(*[FAKE] * 6)

    def call(nb):
        head = (FAKE, FAKE, FAKE)
        shape = (dt, 1, heads, n, d, ctypes.byref(p))
        tail = (FAKE + 8, nb, None)
        if op == luna.OP_ATTN:
            return lib.luna_attn_fwd(*head, *shape, 1e-6, FAKE, *tail)
        if op == luna.OP_ATTN_CAUSAL:
            return lib.luna_attn_fwd_causal(*head, *shape, 64, 1e-6, FAKE, *tail)
        if op == luna.OP_STATE:
            return lib.luna_attn_state(*head[:2], *shape, 0, FAKE, FAKE, *tail)
        return lib.luna_attn_bwd(*head, FAKE, *shape, 0, 1e-6, FAKE, FAKE, FAKE, ctypes.byref(g), *tail)

    assert call(few) == luna.LUNA_ERR_INVALID_ARG and b"aligned" in lib.luna_last_error()
    assert call(1 << 16) == luna.LUNA_ERR_WORKSPACE


@pytest.mark.parametrize("heads,n", [(8, 4992), (3, 13376), (17, 2432), (42, 1024)])
def test_noalloc_scratch_holds_fewer_pieces(lib, heads, n):
    """One channel per projection with 256 features at d = 128 holds its features in the
    workspace too; the static scratch is enough for these shapes with the states of a cut in
    two, though not for those of equal parts."""
    p = _params(M=256, L=1)
    cap = lib.luna_noalloc_scratch_bytes()
    assert lib.luna_workspace_bytes(luna.OP_ATTN_CAUSAL, luna.LUNA_BF16, 1, heads, n, 128, ctypes.byref(p), 64) > cap
    assert lib.luna_attn_fwd_causal(FAKE, FAKE, FAKE, luna.LUNA_BF16, 1, heads, n, 128, ctypes.byref(p), 64, 1e-6, FAKE,
                                    FAKE + 8, cap, None) == luna.LUNA_ERR_INVALID_ARG
    assert b"aligned" in lib.luna_last_error()


def test_features_without_workspace(lib):
    """Short causal calls on the scan kernel do without any workspace (it is asked for from
    the length on where states come in)."""
    assert lib.luna_attn_features_workspace_bytes(luna.LUNA_BF16, luna.LUNA_BF16, 1, 1, 255, 64, 128, 1, 64) == 0
    st = lib.luna_attn_fwd_features(FAKE, FAKE, luna.LUNA_BF16, FAKE, luna.LUNA_BF16, 1, 1, 255, 64, 128, 1, 64, -1.0,
                                    FAKE, None, 0, None)
    assert st == luna.LUNA_ERR_INVALID_ARG and b"eps" in lib.luna_last_error()
    assert lib.luna_attn_fwd_features(FAKE, FAKE, luna.LUNA_BF16, FAKE, luna.LUNA_BF16, 1, 1, 400, 64, 128, 1, 64, 1e-6,
                                      FAKE, None, 0, None) == luna.LUNA_ERR_WORKSPACE


@pytest.mark.parametrize("dt,heads,n,pieces", [
    (luna.LUNA_F32, 1, 100, 1), (luna.LUNA_F32, 1, 512, 8), (luna.LUNA_F32, 128, 100, 1), (luna.LUNA_F32, 300, 1024, 2),
    (luna.LUNA_BF16, 1, 100, 1), (luna.LUNA_BF16, 64, 512, 1), (luna.LUNA_BF16, 1, 512, 8)])
def test_state_pieces(lib, dt, heads, n, pieces):
    """Non-causal calls on 256 given features cut their tokens only where the pieces pay."""
    nb = lib.luna_attn_features_workspace_bytes(dt, dt, 1, heads, n, 128, 256, 0, 64)
    assert nb == heads * pieces * 256 * 129 * 4
