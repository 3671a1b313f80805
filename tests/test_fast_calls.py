"""The binding's short way (native checks and call in one step) against its long way: the same results, the same
refusals, and nothing taken that is not plainly right."""
import ctypes
import importlib.machinery
import importlib.util
import subprocess

import numpy as np
import pytest
import torch

from paper_2602_09578_amd import binding as B
from paper_2602_09578_amd import inputs as I
from paper_2602_09578_amd.build import FAST_PATH, fast_calls_sources

ENTRIES = ("decode_attn", "token_logprobs", "sample_tokens", "kv_append", "prefill_attn")


def test_what_is_not_a_device_tensor_goes_the_long_way():
    B.load_library()
    if B._fast is None:
        pytest.skip("torch does not tell the current stream")
    shape = B.make_shape(2, 1, 4, 2, 3, 1, 1)
    x = torch.zeros(2, 4, 128, dtype=torch.bfloat16)
    for name in ENTRIES:
        f = getattr(B._fast, name)
        for n in range(14):
            for filler in (None, 3, "no", x, shape):
                assert f(*([shape] + [filler] * (n - 1) if n else [])) is None
    with pytest.raises(ValueError, match="device tensors required"):
        B.marl_token_logprobs(torch.zeros(1, 8, dtype=torch.bfloat16), torch.zeros(1, dtype=torch.int32), 1.0, torch.zeros(1))


def _reloaded(monkeypatch, fast_path, build):
    """The module as a fresh process loads it, with another file and builder of the short way."""
    monkeypatch.setattr(B, "_lib", None)
    monkeypatch.setattr(B, "_fast", None)
    monkeypatch.setattr(B, "FAST_PATH", str(fast_path))
    monkeypatch.setattr(B, "build_fast_calls", build)
    return B.load_library()


def test_a_short_way_that_cannot_be_loaded_or_built_leaves_the_long_way(tmp_path, monkeypatch):
    B.load_library()
    if B._raw_stream is None:
        pytest.skip("torch does not tell the current stream")
    def no_compiler():
        raise FileNotFoundError("g++")
    def fails():
        raise RuntimeError("g++ failed for fast_calls.cpp")
    (tmp_path / "cut.so").write_bytes(b"\x7fELF cut short")
    for path, build in ((tmp_path / "cut.so", fails), (B.LIB_PATH, fails), (tmp_path / "missing.so", no_compiler), (tmp_path / "missing.so", fails)):
        with pytest.warns(RuntimeWarning, match="fast_calls"):
            lib = _reloaded(monkeypatch, path, build)
        assert lib.marl_version() == 1 and B._fast is None
        assert B.marl_workspace_bytes(B.make_shape(2, 1, 4, 2, 3, 1, 1)) > 0
    # another torch's: loads, but is not taken
    with monkeypatch.context() as m, pytest.warns(RuntimeWarning, match="built for torch"):
        m.setattr(torch, "__version__", "0.0.1")
        _reloaded(m, FAST_PATH, fails)
        assert B._fast is None


@pytest.mark.parametrize("sources", [None, "other", "these"])
def test_a_short_way_of_other_sources_leaves_the_long_way(sources, monkeypatch):
    """A module built before its functions changed: it says nothing of its sources, or names others, or cannot be bound."""
    B.load_library()
    if B._raw_stream is None:
        pytest.skip("torch does not tell the current stream")

    class Old:
        torch_version = torch.__version__.split("+")[0]
        def bind(self, *args):
            raise TypeError("bind: a function, two types, six addresses")
    if sources is not None:
        Old.sources = fast_calls_sources() if sources == "these" else sources
    with monkeypatch.context() as m, pytest.warns(RuntimeWarning, match="six addresses" if sources == "these" else "other sources"):
        m.setattr(importlib.util, "module_from_spec", lambda spec: Old())
        m.setattr(importlib.machinery.ExtensionFileLoader, "exec_module", lambda self, module: None)
        lib = _reloaded(m, FAST_PATH, lambda: pytest.fail("built"))
        assert lib.marl_version() == 1 and B._fast is None


def test_a_short_way_without_its_sources_is_taken(tmp_path, monkeypatch):
    """The built package alone: there is nothing to compare."""
    B.load_library()
    if B._raw_stream is None:
        pytest.skip("torch does not tell the current stream")
    with monkeypatch.context() as m:
        m.setattr("paper_2602_09578_amd.build.CSRC", str(tmp_path))
        _reloaded(m, FAST_PATH, lambda: pytest.fail("built"))
        assert B._fast is not None


def test_a_missing_short_way_is_built(tmp_path, monkeypatch):
    B.load_library()
    if B._raw_stream is None:
        pytest.skip("torch does not tell the current stream")
    built = tmp_path / "fast_calls.so"
    _reloaded(monkeypatch, built, lambda: built.write_bytes(open(FAST_PATH, "rb").read()))
    assert B._fast is not None


def _calls():
    """(name, function, arguments, outputs among them) of one right call of each entry."""
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(1)
    attn = I.build_attn_inputs(I.WORKLOADS["tiny"], device=dev)
    call = B.prepare_attn(attn, B.MARL_OUT_F32)
    a = [call.shape, call.workspace, attn.q, attn.k_pages, attn.v_pages, attn.prefix_block_table, attn.suffix_block_table,
         attn.prefix_lens, attn.suffix_lens, attn.group_of_seq, attn.scale, call.out]
    x = I.randn_bf16((5, 1000), 3.0, gen, dev)
    u = torch.rand(5, generator=gen, device=dev)
    i32, f32 = (lambda: torch.zeros(5, dtype=torch.int32, device=dev)), (lambda: torch.zeros(5, device=dev))
    ws = B.alloc_workspace(B.marl_sample_workspace_bytes(5, 1000), dev)
    NS, Hkv = attn.num_seqs, attn.Hkv
    new = [I.randn_bf16((NS, Hkv, 128), 1.0, gen, dev) for _ in range(2)]
    lens = torch.full((NS,), 2, dtype=torch.int32, device=dev)
    pre = I.build_prefill_inputs(8, 2, np.array([20, 33]), np.array([0, 16]), device=dev, seed=1, poison=False)
    pshape, pws, pout = B.prepare_prefill(pre, B.MARL_OUT_BF16)
    return [("decode_attn", B.marl_decode_attn, a, [11]),
            ("token_logprobs", B.marl_token_logprobs, [x, i32(), 0.9, f32(), None], [3]),
            ("sample_tokens", B.marl_sample_tokens, [x, u, 0.9, i32(), f32(), ws], [3, 4]),
            ("sample_tokens_top_p", B.marl_sample_tokens_top_p, [x, u, 0.9, 0.8, i32(), f32()], [4, 5]),
            ("kv_append", B.marl_kv_append, [call.shape, *new, attn.k_pages, attn.v_pages, attn.suffix_block_table, lens], [3, 4]),
            ("prefill_attn", B.marl_prefill_attn, [pshape, pws, pre.q, pre.k_pages, pre.v_pages, pre.prefix_block_table, pre.q_start,
                                                   pre.q_pos0, pre.scale, pout], [9])]


def _native(name, args):
    """What the native function itself says to the binding's arguments: a status, or None for the long way."""
    f = getattr(B._fast, "sample_tokens" if name.startswith("sample") else name)
    if name == "sample_tokens":
        args = [*args[:3], None, *args[3:]]
    elif name == "sample_tokens_top_p":
        args = [*args, None]
    elif name == "kv_append":
        args = [*args, None]
    return f(*args)


def _spoil(args, outs):
    """Outputs that hold what no call writes (a cache page: only the appended token's part is written)."""
    for k in outs:
        if args[k] is not None and torch.is_tensor(args[k]):
            args[k].fill_(-77)


def _outcome(f, args, outs):
    _spoil(args, outs)
    try:
        f(*args)
    except Exception as e:      # noqa: BLE001 (what is compared is which)
        return type(e).__name__ + ": " + str(e)
    torch.cuda.synchronize()
    return [args[k].clone() for k in outs]


@pytest.mark.gpu
@pytest.mark.parametrize("which", range(6))
def test_right_calls_are_taken_by_the_short_way(which):
    """The native function makes the call (status 0 and outputs written), and not for another structure of as many bytes."""
    name, f, right, outs = _calls()[which]
    print("case: fast calls, taken", name, flush=True)
    _spoil(right, outs)
    assert _native(name, right) == 0
    torch.cuda.synchronize()
    for k in outs:
        assert (right[k] != -77).any(), k
        if name != "kv_append":
            assert (right[k] != -77).all(), k
    if isinstance(right[0], ctypes.Structure):
        other = (ctypes.c_byte * ctypes.sizeof(right[0])).from_buffer_copy(right[0])
        assert _native(name, [other, *right[1:]]) is None
        with pytest.raises(AttributeError):
            f(other, *right[1:])


@pytest.mark.gpu
@pytest.mark.parametrize("which", range(6))
def test_both_ways_give_the_same(which, monkeypatch):
    name, f, right, outs = _calls()[which]
    print("case: fast calls", name, flush=True)
    fast = B._fast
    assert fast is not None

    def state():   # (appending changes the lengths: each way gets them as they were)
        return [a.clone() if torch.is_tensor(a) and k == 6 and name == "kv_append" else a for k, a in enumerate(right)]

    def both(changed=None, value=None):
        results = []
        for way in (fast, None):
            monkeypatch.setattr(B, "_fast", way)
            args = state()
            if changed is not None:
                args[changed] = value
            results.append(_outcome(f, args, [k for k in outs if k != changed]))
        monkeypatch.setattr(B, "_fast", fast)
        return results
    short, long = both()
    assert isinstance(short, list) and all(torch.equal(s.view(torch.uint8), g.view(torch.uint8)) for s, g in zip(short, long))
    # one argument wrong at a time: another type, another extent, a stride, host memory, nothing, a number that is none
    for k, a in enumerate(right):
        if torch.is_tensor(a):
            wrong = [a.to(torch.float64), a[:-1], a.cpu(), None, 5]
            if a.dim() > 1:
                wrong.append(a.transpose(0, 1).contiguous().transpose(0, 1))
            if a.dtype == torch.uint8:
                wrong = [a[:100], a.cpu(), a[::2]]   # (a workspace: any number of bytes is looked at by the library)
        elif isinstance(a, float):
            wrong = ["x", float("nan")]
        else:
            continue
        for w in wrong:
            short, long = both(k, w)
            if isinstance(short, str) or isinstance(long, str):
                assert short == long, (k, short, long)


@pytest.mark.gpu
def test_an_exception_in_the_library_is_raised_and_the_call_is_not_repeated(tmp_path):
    """Functions that count their calls and throw, in the place of the library's."""
    print("case: fast calls, exception", flush=True)
    (tmp_path / "boom.cpp").write_text("#include <stdexcept>\n"
                                       'extern "C" int calls = 0;\n'
                                       'extern "C" int boom() { ++calls; throw std::runtime_error("out of paper"); }\n'
                                       'extern "C" int number() { ++calls; throw 7; }\n')
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(tmp_path / "boom.so"), str(tmp_path / "boom.cpp")], check=True)
    boom = ctypes.CDLL(str(tmp_path / "boom.so"))
    calls = ctypes.c_int.in_dll(boom, "calls")
    lib = B.load_library()
    assert B._fast is not None
    try:
        for f, message in ((boom.boom, "out of paper"), (boom.number, "exception in the library")):
            B._bind_fast_calls(B._fast, *[f] * 6)
            for name, call, right, _ in _calls():
                calls.value = 0
                with pytest.raises(RuntimeError, match=message):
                    call(*right)
                assert calls.value == 1, name
    finally:
        B._bind_fast_calls(B._fast, lib.marl_decode_attn, lib.marl_token_logprobs, lib.marl_kv_append, lib.marl_sample_tokens,
                           lib.marl_sample_tokens_top_p, lib.marl_prefill_attn)
    name, call, right, outs = _calls()[1]
    call(*right)
    torch.cuda.synchronize()
    assert torch.isfinite(right[outs[0]]).all()


@pytest.mark.gpu
def test_the_scatter_stays_bound_where_the_other_functions_are_bound_anew():
    print("case: fast calls, six functions bound", flush=True)
    lib = B.load_library()
    B._bind_fast_calls(B._fast, lib.marl_decode_attn, lib.marl_token_logprobs, lib.marl_kv_append, lib.marl_sample_tokens,
                       lib.marl_sample_tokens_top_p, lib.marl_prefill_attn)
    pre = I.build_prefill_inputs(8, 2, np.array([20]), np.array([5]), device="cuda", seed=1, poison=False)
    shape, _, _ = B.prepare_prefill(pre, B.MARL_OUT_BF16)
    assert B._fast.kv_write_prompt(shape, pre.k_new, pre.v_new, pre.k_pages, pre.v_pages, pre.prefix_block_table, pre.q_start,
                                   pre.q_pos0, None) == 0
    torch.cuda.synchronize()


@pytest.mark.gpu
def test_prompt_scatter_by_the_short_way(monkeypatch):
    """The native function makes the plain call, leaves everything else to the long way, and both write the same bytes."""
    print("case: fast calls, prompt scatter", flush=True)
    lib = B.load_library()
    B._bind_fast_calls(B._fast, lib.marl_decode_attn, lib.marl_token_logprobs, lib.marl_kv_append, lib.marl_sample_tokens,
                       lib.marl_sample_tokens_top_p, lib.marl_prefill_attn, lib.marl_kv_write_prompt)
    pre = I.build_prefill_inputs(8, 2, np.array([20, 33]), np.array([0, 16]), device="cuda", seed=1, poison=False)
    shape, _, _ = B.prepare_prefill(pre, B.MARL_OUT_BF16)
    args = lambda: [shape, pre.k_new, pre.v_new, pre.k_pages.clone(), pre.v_pages.clone(), pre.prefix_block_table, pre.q_start, pre.q_pos0]
    short, long = args(), args()
    assert B._fast.kv_write_prompt(*short, None) == 0
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert B._fast.kv_write_prompt(*long, flags) is None            # (with flags: the long way)
    B.marl_kv_write_prompt(*long, flags)
    torch.cuda.synchronize()
    assert int(flags) == 0 and not torch.equal(short[3], pre.k_pages)
    assert torch.equal(short[3], long[3]) and torch.equal(short[4], long[4])
    for k, a in enumerate(args()):
        if not torch.is_tensor(a):
            continue
        for wrong in (a.to(torch.float64), a[:-1], a.cpu(), a.unsqueeze(0), None, 5):
            bad = args()
            bad[k] = wrong
            if wrong is None and k > 1:                             # (no address: what the library itself refuses)
                assert B._fast.kv_write_prompt(*bad, None) == -1    # MARL_INVALID_ARG
            else:
                assert B._fast.kv_write_prompt(*bad, None) is None, k
            said = []
            for way in (B._fast, None):
                with monkeypatch.context() as m, pytest.raises(Exception) as e:
                    m.setattr(B, "_fast", way)
                    B.marl_kv_write_prompt(*bad)
                said.append((e.type, str(e.value)))
            assert said[0] == said[1]
    other = (ctypes.c_byte * ctypes.sizeof(shape)).from_buffer_copy(shape)
    assert B._fast.kv_write_prompt(other, *args()[1:], None) is None
