"""The native argument marshalling of the per-layer calls (csrc/qoq_py.cpp): what it refuses, and on which stream it launches."""
import numpy as np
import pytest
import torch

from paper_2405_04532_amd import api
from paper_2405_04532_amd import workloads as wl

gpu = pytest.mark.gpu
DEV = "cuda:0"
M, K, N = 16, 256, 256
B, T, HKV, H, S, D = 2, 3, 2, 4, 64, 128


@pytest.fixture(scope="module", autouse=True)
def built():
    import os
    if not (os.path.exists(api.LIB_PATH) and os.path.exists(api.NATIVE_PATH)):
        from paper_2405_04532_amd import build
        build.build()


class NoTruth:
    """A flag without a truth value, as an array of several elements has none."""
    def __bool__(self):
        raise ValueError("no truth value")


def test_a_binding_of_another_torch_is_refused(monkeypatch):
    assert api._load_native().torch_version == torch.__version__
    monkeypatch.setattr(api, "_native", None)
    monkeypatch.setattr(torch, "__version__", "0.0")
    with pytest.raises(RuntimeError, match="built for torch"):
        api._load_native()


def test_the_c_library_is_built_without_torch(monkeypatch, tmp_path, capsys):
    import sys

    from paper_2405_04532_amd import build
    ran = []
    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "_compile", lambda source, extra: source)
    monkeypatch.setattr(build.subprocess, "check_call", lambda command, **kw: ran.append(command))
    monkeypatch.setitem(sys.modules, "torch", None)
    assert build.build() == build.LIB
    assert [c for c in ran if build.LIB in c] and not [c for c in ran if build.PY_LIB in c]
    assert "not built" in capsys.readouterr().out


@gpu
def test_a_flag_without_a_truth_value_raises_its_own_error():
    x, gamma = torch.ones((M, K), dtype=torch.float16, device=DEV), torch.ones(K, dtype=torch.float16, device=DEV)
    perm = torch.arange(K, dtype=torch.int32, device=DEV)
    for call in (lambda f: api.quant_act_per_token(x, f), lambda f: api.quant_act_per_token(x, True, f),
                 lambda f: api.quant_act_per_token_reordered(x, perm, f), lambda f: api.quant_act_per_token_reordered(x, perm, True, f),
                 lambda f: api.rmsnorm_quant(x, gamma, 1e-5, f), lambda f: api.rmsnorm_quant(x, gamma, 1e-5, True, f),
                 lambda f: api.rmsnorm_quant(x, gamma, 1e-5, True, True, f),
                 lambda f: api.silu_mul_quant(x, f), lambda f: api.silu_mul_quant(x, True, f), lambda f: api.silu_mul_quant(x, True, True, f)):
        with pytest.raises(ValueError, match="no truth value"):
            call(NoTruth())
        assert len(call(np.bool_(True))) in (4, 5)
    with pytest.raises(ValueError):
        api.rmsnorm_quant(x, gamma, "small")
    for eps in ("1e-5", np.float32(1e-5), torch.tensor(1e-5)):                   # whatever float() takes
        assert len(api.rmsnorm_quant(x, gamma, eps)) == 5


def _inputs(dev):
    """One valid argument list per entry point, as keyword arguments of the public functions."""
    g = torch.Generator().manual_seed(11)
    half = lambda *s: torch.randn(s, generator=g).to(torch.float16).to(dev)
    ints = lambda hi, *s: torch.randint(0, hi, s, generator=g, dtype=torch.int32).to(dev)
    x, qx = half(M, K), torch.randint(-127, 128, (M, K), generator=g, dtype=torch.int8).to(dev)
    sx, rowsum = half(M).abs() + 0.01, qx.sum(1, dtype=torch.int32)
    packed = torch.zeros(max(1, api.packed_bytes(N, K)), dtype=torch.uint8, device=dev)
    cache = api.kv4_new_cache(B, HKV, S, dev)
    return {
        "quant_act_per_token": dict(x=x),
        "quant_act_per_token_reordered": dict(x=x, perm=torch.randperm(K, generator=g).to(torch.int32).to(dev)),
        "rmsnorm_quant": dict(x=x, gamma=half(K), eps=1e-5),
        "silu_mul_quant": dict(gate_up=x),
        "w4a8_gemm": dict(qx=qx, sx=sx, packed=packed, N=N),
        "w4a8_gemm_noalloc": dict(qx=qx, sx=sx, packed=packed, N=N, out=half(M, N)),
        "w4a8_gemm_token_sum": dict(qx=qx, sx=sx, tx=half(M).float(), packed=packed, N=N),
        "w4a8_linear": dict(x=x, packed=packed, N=N),
        "kv4_append": dict(cache=cache, k=half(B, T, HKV, D), v=half(B, T, HKV, D), positions=ints(S - T, B), S_max=S),
        "kv4_attention_decode": dict(q=half(B, H, D), cache=cache, seq_lens=ints(S, B) + 1, Hkv=HKV, S_max=S),
    }


# the tensors whose type, layout and place are checked
CHECKED = {"quant_act_per_token": ["x"], "quant_act_per_token_reordered": ["x", "perm"], "rmsnorm_quant": ["x", "gamma"],
           "silu_mul_quant": ["gate_up"], "w4a8_gemm": ["qx"], "w4a8_gemm_noalloc": ["qx", "out"], "w4a8_gemm_token_sum": ["qx", "tx"],
           "w4a8_linear": ["x"], "kv4_append": ["k", "v", "positions"], "kv4_attention_decode": ["q", "seq_lens"]}
NATIVE = {"quant_act_per_token": ("quant_act", 3), "quant_act_per_token_reordered": ("quant_act_reordered", 4), "rmsnorm_quant": ("rmsnorm_quant", 6),
          "silu_mul_quant": ("silu_mul_quant", 4), "w4a8_gemm": ("w4a8_gemm", 8), "w4a8_gemm_noalloc": ("w4a8_gemm_noalloc", 7),
          "w4a8_gemm_token_sum": ("w4a8_gemm_token_sum", 7), "w4a8_linear": ("w4a8_linear", 9), "kv4_append": ("kv4_append", 5),
          "kv4_attention_decode": ("kv4_attention_decode", 7)}


@pytest.mark.parametrize("name", sorted(CHECKED))
def test_a_tensor_on_the_host_and_a_wrong_argument_count_are_refused(name):
    with pytest.raises(TypeError, match="on the GPU"):
        getattr(api, name)(**_inputs("cpu")[name])
    first = next(iter(k for k in _inputs("cpu")[name] if k in CHECKED[name]))
    with pytest.raises(TypeError, match="tensor"):
        getattr(api, name)(**{**_inputs("cpu")[name], first: [1.0, 2.0]})
    entry, count = NATIVE[name]
    for n in (count - 1, count + 1):
        with pytest.raises(TypeError, match=f"expected {count} arguments, got {n}"):
            getattr(api._load_native(), entry)(*[None] * n)


@gpu
@pytest.mark.parametrize("name", sorted(CHECKED))
def test_wrong_types_layouts_and_shapes_are_refused(name):
    good = _inputs(DEV)[name]
    call = getattr(api, name)
    for arg in CHECKED[name]:
        t = good[arg]
        with pytest.raises(TypeError, match=arg):
            call(**{**good, arg: t.cpu()})
        with pytest.raises(TypeError, match=arg):
            call(**{**good, arg: t.double()})
        if t.dim() >= 2:
            wide = torch.empty((*t.shape[:-1], 2 * t.shape[-1]), dtype=t.dtype, device=DEV)[..., ::2]
            with pytest.raises(TypeError, match=arg):
                call(**{**good, arg: wide})
    first = CHECKED[name][0]
    for shape in ((-1,), (1, 1, 1, 1, -1)):
        with pytest.raises(ValueError, match="dimensions"):
            call(**{**good, first: good[first].reshape(shape)})
    if "N" in good:
        with pytest.raises(TypeError):
            call(**{**good, "N": 1.5})
        with pytest.raises(api.QoqError):                                        # a status of the library, as its exception
            call(**{**good, "N": 100, **({"out": torch.empty((M, 100), dtype=torch.float16, device=DEV)} if name == "w4a8_gemm_noalloc" else {})})


@gpu
@pytest.mark.parametrize("name", sorted(CHECKED))
def test_calls_run_on_the_current_stream(name):
    """The input of a call is finished late on a side stream: a launch anywhere else would read what was there before.  Only
    that stream is waited for."""
    good = _inputs(DEV)[name]
    if "packed" in good:
        mode = api.QOQ_PER_CHANNEL if name == "w4a8_gemm_token_sum" else api.QOQ_GROUP128
        good["packed"] = api.pack_weights(wl.make_weights(N, K, 3, DEV), mode)
    if name == "kv4_attention_decode":
        src = _inputs(DEV)["kv4_append"]
        long = {a: torch.randn(B, S, HKV, D, generator=torch.Generator().manual_seed(i)).to(torch.float16).to(DEV) for i, a in enumerate("kv")}
        api.kv4_append(good["cache"], long["k"], long["v"], torch.zeros_like(src["positions"]), S)
    call = getattr(api, name)

    def outputs():
        r = call(**good)
        r = good["cache"] if r is None else r
        return [t for t in (r if isinstance(r, tuple) else (r,)) if t is not None]

    first = CHECKED[name][0]
    real = good[first].clone()
    want = [t.clone() for t in outputs()]
    if name == "kv4_append":
        good["cache"].zero_()
    late = torch.zeros_like(real)
    good[first] = late
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)
        late.copy_(real)
        got = outputs()
    side.synchronize()
    assert len(got) == len(want) and all(torch.equal(a, b) for a, b in zip(got, want))
    assert any(bool(t.view(torch.uint8).any()) for t in want)


def _calls_without_a_workspace(m, n, k, mode):
    """The GEMM entry points on zeros with every result given: whatever else is allocated is their own workspace."""
    new = lambda dtype, *s: torch.zeros(s, dtype=dtype, device=DEV)
    packed = new(torch.uint8, api.packed_bytes(n, k, mode))
    x, qx, sx, rowsum, out = new(torch.float16, m, k), new(torch.int8, m, k), new(torch.float16, m), new(torch.int32, m), new(torch.float16, m, n)
    calls = [lambda: api.w4a8_gemm(qx, sx, packed, n, mode, rowsum=rowsum, out=out),
             lambda: api.w4a8_linear(x, packed, n, mode, out=out, qx=qx, sx=sx, rowsum=rowsum)]
    return calls + ([lambda: api.w4a8_gemm_token_sum(qx, sx, new(torch.float32, m), packed, n, out=out)] if mode else [])


@gpu
@pytest.mark.parametrize("mode", [0, 1])
def test_a_call_without_a_workspace_zeroes_the_counters_only(mode):
    """Half of the places for partial tiles of this plan are not used: in a block that the allocator has had before they keep what they
    held, while the counters are zeroed."""
    m, n, k = 64, 4096, 11008
    need = api.gemm_workspace_bytes(m, n, k, mode)
    assert need > api.GEMM_COUNTER_BYTES == 256 << 10
    for call in _calls_without_a_workspace(m, n, k, mode):
        block = torch.full((need,), 0x5A, dtype=torch.uint8, device=DEV)
        where = block.data_ptr()
        del block
        call()
        block = torch.empty(need, dtype=torch.uint8, device=DEV)
        assert block.data_ptr() == where
        kept = (block[api.GEMM_COUNTER_BYTES:] == 0x5A).float().mean().item()
        assert not block[:api.GEMM_COUNTER_BYTES].any() and 0.4 < kept < 0.6
        del block


@gpu
@pytest.mark.parametrize("m,n,k,made", [(1024, 4096, 11008, False),       # uncut: nothing is exchanged, whatever a kept workspace is sized for
                                        (65, 15616, 3840, False),         # cut it gains less than zeroing counters takes
                                        (138, 15808, 8192, True), (389, 4096, 11008, True), (64, 4096, 4096, False)])
def test_a_call_without_a_workspace_makes_one_where_that_pays(m, n, k, made):
    for call in _calls_without_a_workspace(m, n, k, 0):
        torch.cuda.reset_peak_memory_stats()
        before = torch.cuda.memory_allocated()
        call()
        assert (torch.cuda.max_memory_allocated() > before) == made
