"""The native marshalling of the tensor helpers (csrc/jet_host.cpp) against the Python path it stands in for: what it
does not take it declines (None), what it takes has the same results, types and errors."""
import warnings

import pytest
import torch

from paper_2601_14243_amd import binding as b

u8, f32, bf = torch.uint8, torch.float32, torch.bfloat16


class _OnGpu(torch.Tensor):
    """A CPU tensor that passes for a GPU one, for checks that come before any launch."""
    is_cuda = property(lambda self: True)


def test_declines_everything_but_the_plain_form():
    h = b._native()
    x, s = torch.zeros((4, 256), dtype=bf), torch.ones((4, 2))
    q, w = torch.zeros((4, 256), dtype=u8), torch.zeros((128, 256), dtype=u8)
    assert h.quant_act(x, None, True, False, None) is None                      # CPU tensors
    assert h.quant_act("x", None, True, False, None) is None                    # no tensor at all
    assert h.rmsnorm_quant(x, x[0], 1e-6, None) is None
    assert h.silu_mul_quant(x, x, None) is None
    assert h.silu_mul_bwd(x, x, x, None) is None
    assert h.quant_weight(x, True, None) is None
    for kind in (0, 1, 2):
        assert h.gemm(kind, q, s, w, s, None) is None
    with pytest.raises(TypeError):
        h.gemm(0, q, s)
    with pytest.raises(TypeError):
        b.quant_act(x)                                                          # the Python path words the error
    with pytest.raises(TypeError):
        b.quant_weight(x)


@pytest.mark.parametrize("broken", ["missing", "of another Python or torch"])
def test_the_helpers_work_without_the_extension(monkeypatch, broken):
    """libjet.so alone is enough: the Python path takes every call, after one warning."""
    monkeypatch.setattr(b, "_host", None)
    if broken == "missing":
        monkeypatch.setattr(b, "_HOST_PATH", b._HOST_PATH + ".none")
    else:
        def undefined(*a):
            raise ImportError("undefined symbol: THPVariableClass")
        monkeypatch.setattr(b.importlib, "import_module", undefined)
    calls = []
    monkeypatch.setattr(b, "_stream", lambda: None)
    monkeypatch.setattr(b, "jet_quant_act", lambda *a: calls.append(a) or 0)
    x = torch.zeros((4, 256), dtype=bf).as_subclass(_OnGpu)
    out = {"q_row": torch.zeros((4, 256), dtype=u8).as_subclass(_OnGpu), "s_row": torch.ones((4, 2)).as_subclass(_OnGpu)}
    with pytest.warns(RuntimeWarning, match="native marshalling"):
        assert b.quant_act(x, out=out) is out
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        b.quant_act(x, out=out)
    assert len(calls) == 2
    h = b._native()
    assert all(getattr(h, name)() is None for name in ("quant_act", "rmsnorm_quant", "silu_mul_quant", "silu_mul_bwd", "quant_weight", "gemm"))


def test_a_failed_build_of_the_extension_leaves_the_library(monkeypatch, tmp_path):
    from paper_2601_14243_amd import build as jb

    def no_compiler(force):
        raise FileNotFoundError("g++")
    stale = tmp_path / "_jet_host.so"
    stale.write_bytes(b"")
    monkeypatch.setattr(jb, "HOST_LIB", str(stale))
    monkeypatch.setattr(jb, "_compile", lambda *a: None)
    monkeypatch.setattr(jb, "_compile_host", no_compiler)
    with pytest.warns(RuntimeWarning, match="not built"):
        assert jb.build() == jb.LIB
    assert not stale.exists()


class _Declines:
    def __getattr__(self, name):
        return lambda *a: None


def _flat(r):
    if isinstance(r, dict):
        return [r[k] for k in sorted(r)]
    return list(r) if isinstance(r, tuple) else [r]


@pytest.mark.gpu
def test_same_results_as_the_python_path(monkeypatch):
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(bf)
    M, N, K = 128, 256, 384
    x, dy, w, gamma, both, dh = rnd(M, K), rnd(M, N), torch.nn.Parameter(rnd(N, K)), rnd(K), rnd(M, 2 * K), rnd(M, K)
    wq = b.quant_weight(w, transposed=True)
    qx, qd = b.quant_act(x, row=True, col=True), b.quant_act(dy, row=True, col=True)

    def calls():
        e = lambda t: torch.empty_like(t)
        o = {k: e(v) for k, v in qx.items()}
        yield lambda: b.quant_act(x)
        yield lambda: b.quant_act(x, row=False, col=True)
        yield lambda: b.quant_act(x, row=True, col=True, out=o)
        yield lambda: b.quant_act(qx["q_row"], qx["s_row"], row=False, col=True)
        yield lambda: b.quant_act(x, col=True, out={"q_row": e(qx["q_row"]), "s_row": e(qx["s_row"])})   # half given: the rest is added
        yield lambda: b.rmsnorm_quant(x, gamma, 1e-6)
        yield lambda: b.rmsnorm_quant(x, gamma, 1, out={"q_row": e(qx["q_row"]), "s_row": e(qx["s_row"])})  # an int eps
        yield lambda: b.silu_mul_quant(both[:, :K], both[:, K:])
        yield lambda: b.silu_mul_bwd(both[:, :K], both[:, K:], dh)
        yield lambda: b.silu_mul_bwd(both[:, :K], both[:, K:], dh, out=torch.empty((M, 2 * K), dtype=bf, device="cuda"))
        yield lambda: b.quant_weight(w)
        yield lambda: b.quant_weight(w, transposed=True)
        yield lambda: b.quant_weight(w, transposed=True, out=tuple(e(t) for t in wq))
        yield lambda: b.quant_weight(w, out=[e(t) for t in wq])
        yield lambda: b.fp8_linear_fwd(qx["q_row"], qx["s_row"], wq[0], wq[1])
        yield lambda: b.fp8_linear_fwd(qx["q_row"], qx["s_row"], wq[0], wq[1], out=torch.empty((M, N), dtype=bf, device="cuda"))
        yield lambda: b.fp8_linear_dgrad(qd["q_row"], qd["s_row"], wq[2], wq[3])
        yield lambda: b.fp8_linear_wgrad(qd["q_colT"], qd["s_colT"], qx["q_colT"], qx["s_colT"])

    for i, call in enumerate(calls()):
        monkeypatch.undo()
        r1 = [t.clone() for t in _flat(call())]
        monkeypatch.setattr(b, "_host", _Declines())
        r2 = _flat(call())
        assert len(r1) == len(r2), i
        for p, q in zip(r1, r2):
            assert p.dtype == q.dtype and p.shape == q.shape and p.stride() == q.stride() and p.device == q.device, i
            assert torch.equal(p.view(u8), q.view(u8)), i
            assert not p.requires_grad and not q.requires_grad
    monkeypatch.undo()


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_same_errors_as_the_python_path(monkeypatch, native):
    if not native:
        monkeypatch.setattr(b, "_host", _Declines())
    z = lambda *s, dt=bf: torch.zeros(s, dtype=dt, device="cuda")
    with pytest.raises(b.JetError) as e:
        b.quant_act(z(4, 200))                              # K % 128: the C ABI's status
    assert e.value.status == 2 and "jet_quant_act" in str(e.value)
    with pytest.raises(b.JetError) as e:
        b.rmsnorm_quant(z(4, 128), z(128), -1.0)
    assert e.value.status == 4
    with pytest.raises(b.JetError):
        b.quant_act(z(100, 128), row=False, col=True)       # M % 128 in column mode
    with pytest.raises(TypeError):
        b.quant_act(z(4, 128, dt=f32))
    with pytest.raises(TypeError):
        b.rmsnorm_quant(z(4, 128), z(256)[::2], 1e-6)
    with pytest.raises(TypeError):
        b.silu_mul_quant(z(4, 128), z(4, 256))
    with pytest.raises(ValueError):
        b.silu_mul_bwd(z(4, 128), z(4, 128), z(8, 128))
    q, s, w, ws = z(4, 256, dt=u8), z(4, 2, dt=f32), z(128, 256, dt=u8), z(1, 2, dt=f32)
    with pytest.raises(ValueError):
        b.fp8_linear_fwd(q, s, w, z(1, 3, dt=f32))
    with pytest.raises(ValueError):
        b.fp8_linear_fwd(q, s, z(128, 128, dt=u8), z(1, 1, dt=f32))
    with pytest.raises(ValueError):
        b.fp8_linear_fwd(q, s, w, ws, out=z(4, 256))
    with pytest.raises(TypeError):
        b.fp8_linear_fwd(q[:, ::2], s, w, ws)


def _bad_buffers(make, other):
    """(name of the call, call) pairs whose output or scales the kernels would run out of or misread.  make(*shape,
    dtype=) makes a tensor on the operand's device, other(*shape, dtype=) one somewhere else."""
    M, K = 128, 384
    x, gamma, both = make(M, K, dtype=bf), make(K, dtype=bf), make(M, 2 * K, dtype=bf)
    q, s = make(M, K, dtype=u8), make(M, K // 128, dtype=f32)
    qT, sT = make(K, M, dtype=u8), make(K, 1, dtype=f32)
    wq = [make(M, K, dtype=u8), make(1, 3, dtype=f32), make(K, M, dtype=u8), make(3, 1, dtype=f32)]
    pairs = [(q, make(M, 2, dtype=f32)), (make(M - 1, K, dtype=u8), s), (make(K, M, dtype=u8), s), (other(M, K, dtype=u8), s),
             (q, other(M, 3, dtype=f32)), (make(M, K, dtype=bf), s), (q, make(M, 3, dtype=torch.float64)), (q, make(M, 3, dtype=bf)),
             (make(M, 2 * K, dtype=u8)[:, :K], s), (make(M, 2 * K, dtype=u8)[:, ::2], s), (q, make(M, 6, dtype=f32)[:, ::2]),
             (q, make(M * 3 - 1, dtype=f32))]
    for i, (a, b_) in enumerate(pairs):
        o = {"q_row": a, "s_row": b_}
        yield f"quant_act {i}", lambda o=o: b.quant_act(x, out=o)
        yield f"quant_act both {i}", lambda o=o: b.quant_act(x, col=True, out={**o, "q_colT": qT, "s_colT": sT})
        yield f"rmsnorm_quant {i}", lambda o=o: b.rmsnorm_quant(x, gamma, 1e-6, out=o)
        yield f"silu_mul_quant {i}", lambda o=o: b.silu_mul_quant(both[:, :K], both[:, K:], out=o)
    for i, (a, b_) in enumerate([(make(M, K, dtype=u8), sT), (qT, make(K - 1, 1, dtype=f32)), (other(K, M, dtype=u8), sT),
                                 (make(K, 2 * M, dtype=u8), sT), (qT, make(K, 1, dtype=torch.float16))]):
        yield f"quant_act col {i}", lambda o={"q_colT": a, "s_colT": b_}: b.quant_act(x, row=False, col=True, out=o)
    for i, xs in enumerate([other(M, 3, dtype=f32), make(M, 2, dtype=f32), make(M - 1, 3, dtype=f32), make(M, 3, dtype=torch.float64),
                            make(M, 3, dtype=torch.float16), make(M, 6, dtype=f32)[:, ::2], make(M, 6, dtype=f32)]):
        yield f"x_scales {i}", lambda xs=xs: b.quant_act(q, xs)
        yield f"x_scales col {i}", lambda xs=xs: b.quant_act(q, xs, row=False, col=True, out={"q_colT": qT, "s_colT": sT})
    for i, bad in enumerate([make(M - 1, K, dtype=u8), make(1, 2, dtype=f32), make(M, K, dtype=u8), make(2, 1, dtype=f32)]):
        o = list(wq)
        o[i] = bad
        yield f"quant_weight {i}", lambda o=o: b.quant_weight(x, transposed=True, out=tuple(o))
        yield f"quant_weight list {i}", lambda o=o: b.quant_weight(x, transposed=True, out=o)
        o = list(wq)
        o[i] = other(*wq[i].shape, dtype=wq[i].dtype)
        yield f"quant_weight elsewhere {i}", lambda o=o: b.quant_weight(x, transposed=True, out=tuple(o))
    yield "quant_weight without copy", lambda: b.quant_weight(x, out=(wq[0], make(1, 2, dtype=f32)))


def _no_call(name):
    def f(*a):
        raise AssertionError(f"{name} was called with pointers that do not hold the result")
    return f


RAW = ("jet_quant_act", "jet_quant_weight", "jet_rmsnorm_quant", "jet_silu_mul_quant", "jet_silu_mul_bwd")


def test_buffers_that_do_not_hold_the_result_are_refused_before_the_call(monkeypatch):
    """Outputs and scales reach the kernels as raw pointers: too small, of another type, strided, of another row length
    or not on the GPU, they raise in the Python path and the C call is not made."""
    monkeypatch.setattr(b, "_stream", lambda: None)
    for name in RAW:
        monkeypatch.setattr(b, name, _no_call(name))
    make = lambda *sh, dtype: torch.zeros(sh, dtype=dtype).as_subclass(_OnGpu)
    other = lambda *sh, dtype: torch.zeros(sh, dtype=dtype)
    for name, call in _bad_buffers(make, other):
        with pytest.raises((TypeError, ValueError)):
            call()
            pytest.fail(name)


def test_buffers_with_room_are_taken(monkeypatch):
    """Flat workspaces, buffers of a larger batch and one-byte types other than uint8 hold the result as well."""
    seen = []
    monkeypatch.setattr(b, "_stream", lambda: None)
    for name in RAW:
        monkeypatch.setattr(b, name, lambda *a, name=name: seen.append(name) or 0)
    make = lambda *sh, dtype: torch.zeros(sh, dtype=dtype).as_subclass(_OnGpu)
    _good_buffers(make)
    assert seen == ["jet_quant_act"] * 5 + ["jet_rmsnorm_quant", "jet_quant_weight"]


def _good_buffers(make):
    M, K = 128, 384
    x, gamma, q, s = make(M, K, dtype=bf), make(K, dtype=bf), make(M, K, dtype=u8), make(M, 3, dtype=f32)
    b.quant_act(x, out={"q_row": make(M * K, dtype=u8), "s_row": make(M * 3 + 5, dtype=f32)})
    b.quant_act(x, out={"q_row": make(2 * M, K, dtype=u8), "s_row": make(2 * M, 3, dtype=f32)})
    b.quant_act(x, out={"q_row": make(2, M // 2, K, dtype=torch.int8), "s_row": s})
    b.quant_act(x, row=False, col=True, out={"q_colT": make(K, M, dtype=u8), "s_colT": make(K, 1, dtype=f32)})
    b.quant_act(q, make(M + 1, 3, dtype=f32), row=True, out={"q_row": make(M, K, dtype=u8), "s_row": make(M, 3, dtype=f32)})
    b.rmsnorm_quant(x, gamma, 1e-6, out={"q_row": q, "s_row": s})
    b.quant_weight(x, out=(q, make(3, dtype=f32)))


@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_buffers_on_the_gpu(monkeypatch, native):
    """The same calls on GPU tensors: the native path declines them and the Python path raises, both on the host before
    any launch; what has room runs."""
    if not native:
        monkeypatch.setattr(b, "_host", _Declines())
    make = lambda *sh, dtype: torch.zeros(sh, dtype=dtype, device="cuda")
    other = lambda *sh, dtype: torch.zeros(sh, dtype=dtype)
    _good_buffers(make)
    for name in RAW:
        monkeypatch.setattr(b, name, _no_call(name))
    for name, call in _bad_buffers(make, other):
        with pytest.raises((TypeError, ValueError)):
            call()
            pytest.fail(name)
