"""The extension module's way from a call to its launch against the binding's own checks and marshalling: the same
bits for every entry point that takes it, and the same answer for tensors that it leaves to them."""
import pytest
import torch

from paper_2503_13565_amd import binding as B, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _inputs(m, n, k):
    w = synth.weights_student_t(n, k, seed=3, device=DEV)
    x = synth.activations_outlier_channels(m, k, seed=4, device=DEV)
    q, s = B.mxfp4_direct_cast(w)
    return x, w, q, s


def _calls(m, n, k):
    """name -> call without an output buffer."""
    x, w, q, s = _inputs(m, n, k)
    bias = torch.linspace(-1, 1, n, device=DEV, dtype=torch.bfloat16)
    res = torch.ones((m, n + 8), device=DEV, dtype=torch.bfloat16)[:, :n]       # rows further apart than they are long
    half = torch.ones((m, n // 2), device=DEV, dtype=torch.bfloat16)
    ws = torch.empty((max(B.mxfp4_woq_gemm_workspace_bytes(m, n, k), 256),), dtype=torch.uint8, device=DEV)
    pick = torch.empty((B.mxfp4_woq_gemm_argmax_workspace_bytes(m, n, k),), dtype=torch.uint8, device=DEV)
    pick16 = torch.empty((B.mxfp4_bf16_gemm_argmax_workspace_bytes(m, n, k),), dtype=torch.uint8, device=DEV)
    draft = torch.zeros((m - 1,), dtype=torch.int32, device=DEV)
    tiles = B.mxfp4_tile_repack(q, s)
    e4, e2 = B.mxfp4_e4m3_direct_cast(w), B.mxfp4_e2m3_direct_cast(w)
    calls = {
        "plain": lambda: B.mxfp4_woq_gemm(x, q, s),
        "wide": lambda: B.mxfp4_woq_gemm(torch.cat([x, x], 1)[:, :k], q, s),    # (rows 2 K apart)
        "workspace": lambda: B.mxfp4_woq_gemm(x, q, s, workspace=ws),
        "path": lambda: B.mxfp4_woq_gemm(x, q, s, path=B.PATH_VALU_CVT),
        "grad": lambda: B.mxfp4_woq_gemm(x.clone().requires_grad_(), torch.nn.Parameter(q, requires_grad=False), s),
        "fused": lambda: B.mxfp4_woq_gemm_fused(x, q, s, bias=bias, residual=res, workspace=ws),
        "gate": lambda: B.mxfp4_woq_gemm_fused(x, q, s, act=B.ACT_SWIGLU, residual=half),
        "tiled": lambda: B.mxfp4_woq_gemm_tiled(x, tiles),
        "tiled_ws": lambda: B.mxfp4_woq_gemm_tiled(x, tiles, workspace=ws),
        "tiled_fused": lambda: B.mxfp4_woq_gemm_tiled_fused(x, tiles, bias=bias, act=B.ACT_SWIGLU, residual=half),
        "bf16": lambda: B.mxfp4_bf16_gemm(x, w),
        "bf16_wide": lambda: B.mxfp4_bf16_gemm(x, torch.cat([w, w], 1)[:, :k]),
        "e4m3": lambda: B.mxfp4_e4m3_woq_gemm(x, *e4),
        "e2m3": lambda: B.mxfp4_e2m3_woq_gemm(x, *e2),
        "verify": lambda: B.mxfp4_woq_gemm_verify(x, q, s, draft, workspace=pick),
        "verify_tiled": lambda: B.mxfp4_woq_gemm_tiled_verify(x, tiles, draft, workspace=pick),
        "verify_bf16": lambda: B.mxfp4_bf16_gemm_verify(x, w, draft, workspace=pick16),
    }
    if m == 1:
        calls["verify_none"] = lambda: B.mxfp4_woq_gemm_verify(x, q, s, None, workspace=pick)
    for fmt in (B.FMT_E5M2, B.FMT_E3M2, B.FMT_T2):
        pair = B.mxfp4_fmt_direct_cast(fmt, w)
        calls["fmt%d" % fmt] = lambda fmt=fmt, pair=pair: B.mxfp4_fmt_woq_gemm(fmt, x, *pair)
    return calls


@pytest.mark.parametrize("m", [1, 3, 17])
def test_same_bits_as_the_binding_itself(m, monkeypatch):
    calls = _calls(m, 2056, 512)
    taken = []
    product, verify = B._product, B._verify
    with monkeypatch.context() as patch:
        patch.setattr(B, "_product", lambda *a: taken.append(product(*a)) or taken[-1])
        patch.setattr(B, "_verify", lambda *a: taken.append(verify(*a)) or taken[-1])
        native = {name: call() for name, call in calls.items()}
    assert len(taken) == len(calls) and all(t is not None for t in taken)
    monkeypatch.setattr(B, "_product", lambda *a: None)
    monkeypatch.setattr(B, "_verify", lambda *a: None)
    for name, call in calls.items():
        got, want = native[name], call()
        for a, b in zip(got if isinstance(got, tuple) else [got], want if isinstance(want, tuple) else [want], strict=True):
            assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and not a.requires_grad, name
            assert torch.equal(a, b), name


def test_the_current_stream_and_the_device_of_a_mode():
    x, _, q, s = _inputs(4, 2048, 512)
    want = B.mxfp4_woq_gemm(x, q, s)
    side, busy = torch.cuda.Stream(), torch.ones((8192, 8192), device=DEV)
    late = torch.zeros_like(x)                      # what a product on another stream would read
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(8):
            busy = busy @ busy                      # (some tens of ms: the call returns long before its input is there)
        late.copy_(x)
        got = B.mxfp4_woq_gemm(late, q, s)
    side.synchronize()
    assert torch.equal(got, want)
    with torch.device("cpu"):                       # an active mode: the binding's own way
        assert torch.equal(B.mxfp4_woq_gemm(x, q, s), want)


@pytest.mark.parametrize("what", ["dtype", "stride", "dims", "host", "q_stride", "s_shape", "bias", "residual", "workspace", "subclass"])
def test_what_does_not_fit_is_answered_as_before(what, monkeypatch):
    x, _, q, s = _inputs(4, 2048, 512)
    kw = {}
    if what == "dtype":
        x = x.float()
    elif what == "stride":
        x = x.t().contiguous().t()
    elif what == "dims":
        x = x[None]
    elif what == "host":
        x = x.cpu()
    elif what == "q_stride":
        q = torch.cat([q, q], 1)[:, :256]
    elif what == "s_shape":
        s = s[:, :8].contiguous()
    elif what == "bias":
        kw = {"bias": torch.zeros(7, dtype=torch.bfloat16, device=DEV)}
    elif what == "residual":
        kw = {"residual": torch.zeros((4, 7), dtype=torch.bfloat16, device=DEV)}
    elif what == "workspace":
        kw = {"workspace": torch.zeros(1024, dtype=torch.float32, device=DEV)}
    elif what == "subclass":
        x = x.as_subclass(type("Named", (torch.Tensor,), {}))

    def answer():
        try:
            return B.mxfp4_woq_gemm_fused(x, q, s, **kw)
        except (ValueError, B.Mxfp4Error) as e:
            return type(e), str(e)

    B.load()
    assert B._product(0, x, q, s, 0, 0, True, kw.get("bias"), 0, kw.get("residual"), 0, kw.get("workspace")) is None
    got = answer()
    monkeypatch.setattr(B, "_product", lambda *a: None)
    want = answer()
    assert torch.equal(got, want) if isinstance(want, torch.Tensor) else got == want


def test_numbers_that_do_not_fit_are_answered_as_before():
    x, _, q, s = _inputs(4, 2048, 512)
    tiles = B.mxfp4_tile_repack(q, s)
    with pytest.raises(ValueError, match="BF16 tensor"):
        B.mxfp4_woq_gemm_tiled(x, B.TiledWeights(tiles.q, tiles.s, 2048, 2 ** 70))
    for act in (2 ** 70, 2 ** 32 + 1):              # (marshalled to what an int of the C interface keeps of it)
        assert B._product(0, x, q, s, 0, 0, True, None, act, None, 0, None) is None


@pytest.mark.parametrize("what", ["whole", "one", "wide", "grad", "inference", "dtype", "stride", "dims", "host", "subclass", "block"])
def test_casts(what, monkeypatch):
    w = synth.weights_student_t(1 if what == "one" else 37, 96, seed=3, device=DEV)
    if what == "wide":                              # rows further apart than they are long
        w = torch.cat([w, w], 1)[:, :96]
    elif what == "grad":
        w = torch.nn.Parameter(w)
    elif what == "dtype":
        w = w.float()
    elif what == "stride":
        w = w.t().contiguous().t()
    elif what == "dims":
        w = w[None]
    elif what == "host":
        w = w.cpu()
    elif what == "subclass":
        w = w.as_subclass(type("Named", (torch.Tensor,), {}))
    elif what == "block":
        w = w[:, :80].contiguous()

    def answer():
        try:
            with torch.inference_mode(what == "inference"):
                return B.mxfp4_direct_cast(w)
        except (ValueError, B.Mxfp4Error) as e:
            return type(e), str(e)

    B.load()
    assert (B._cast(w) is not None) == (what in ("whole", "one", "wide", "grad", "inference"))
    got = answer()
    with torch.device("cpu"):                       # an active mode: the binding's own way
        assert B._cast(w) is None
    monkeypatch.setattr(B, "_cast", lambda w: None)
    for a, b in zip(got, answer(), strict=True):
        if isinstance(a, torch.Tensor):
            assert a.dtype == b.dtype and a.shape == b.shape and a.stride() == b.stride() and not a.requires_grad
            assert a.is_inference() == b.is_inference() and torch.equal(a, b)
        else:
            assert a == b


def test_a_status_raises_the_error_of_the_library():
    x, _, q, s = _inputs(4, 2048, 512)
    with pytest.raises(B.Mxfp4Error) as e:
        B.mxfp4_woq_gemm(x, q, s, path=99)
    assert e.value.code != 0 and "path" in str(e.value)
