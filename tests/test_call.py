"""The binding's calls in C++ (csrc/apmm_call.cpp) against the Python functions that they stand for: the same results and the same errors
for every way to give the arguments, plain or not."""
import inspect
import os

import pytest
import torch

from paper_2409_17870_amd import binding

NAMES = ["apmm_pack_weights", "apmm_pack_activations", "apmm_quantize_pack_activations", "apmm_gemm", "apmm_gemm_from_codes"]


def general(name):
    """The Python function behind a call: binding.py once more, without the C++ module."""
    spec = inspect.getsource(binding).replace("from . import _apmm_call as _call", "raise ImportError")
    space = {"__name__": "binding_general", "__file__": binding.__file__}
    with pytest.warns(RuntimeWarning, match="C\\+\\+ marshalling is not used"):  # a program without it is told
        exec(compile(spec, binding.__file__, "exec"), space)
    return space[name]


@pytest.mark.parametrize("name", NAMES)
def test_signatures(name):
    assert binding._call is not None
    assert inspect.signature(getattr(binding, name)) == inspect.signature(general(name))


def outcome(fn, *args, **kw):
    try:
        return fn(*args, **kw)
    except Exception as e:
        return type(e).__name__, str(e)


@pytest.mark.parametrize("name, args, kw", [
    ("apmm_pack_weights", (), {}),
    ("apmm_pack_weights", (torch.zeros(2, 3, dtype=torch.uint8), 2), {}),
    ("apmm_pack_activations", (torch.zeros(6, dtype=torch.uint8), 2), dict(out=torch.zeros(4, dtype=torch.uint8))),
    ("apmm_pack_activations", (1, 2, 3, 4), {}),
    ("apmm_quantize_pack_activations", (torch.zeros(2, 3), 4), {}),
    ("apmm_gemm", (1, 2, 3), dict(p=1, nothing=2)),
    ("apmm_gemm", (1, 2, 3, 4, 5, 6, 7), dict(M=1)),
    ("apmm_gemm_from_codes", (None, 2, 3, 4, None), {}),
])
def test_refused_alike(name, args, kw):
    binding.load()
    got, want = outcome(getattr(binding, name), *args, **kw), outcome(general(name), *args, **kw)
    assert isinstance(got, tuple) and got == want


PLAIN, GENERAL = 0, 1  # marshalled in C++, or handed to the Python function once


@pytest.mark.gpu
def test_results_and_errors_alike():
    dev = torch.device("cuda:0")
    M, N, K, p, q = 5, 70, 300, 3, 2
    g = torch.Generator(device=dev).manual_seed(3)
    a = torch.randint(0, 1 << p, (M, K), generator=g, device=dev, dtype=torch.uint8)
    w = torch.randint(0, 1 << q, (N, K), generator=g, device=dev, dtype=torch.uint8)
    x = torch.randn((M, K), generator=g, device=dev).half()
    sa, sw = torch.rand(M, generator=g, device=dev).half(), torch.rand(N, generator=g, device=dev).half()
    general_of = {name: general(name) for name in NAMES}

    def empty(n):
        return torch.zeros(n, dtype=torch.uint8, device=dev)

    na, nw = binding.apmm_packed_activation_bytes(M, K, p), binding.apmm_packed_bytes(N, K, q)
    ap, wp = binding.apmm_pack_activations(a, p), binding.apmm_pack_weights(w, q)
    c32, c16 = (lambda: torch.zeros((M, N), dtype=torch.int32, device=dev)), (lambda: torch.zeros((M, N), dtype=torch.float16, device=dev))

    class Sub(torch.Tensor):
        pass

    calls = [
        ("apmm_pack_weights", PLAIN, lambda: ((w, q), dict(out=empty(nw)))),
        ("apmm_pack_weights", PLAIN, lambda: ((w, q, empty(nw)), {})),
        ("apmm_pack_weights", PLAIN, lambda: ((w,), dict(q=q))),
        ("apmm_pack_weights", GENERAL, lambda: ((w, q), dict(out=empty(nw - 1)))),
        ("apmm_pack_weights", GENERAL, lambda: ((w, 9), dict(out=empty(nw)))),
        ("apmm_pack_weights", GENERAL, lambda: ((w.t(), q), dict(out=empty(nw)))),
        ("apmm_pack_weights", GENERAL, lambda: ((w.int(), q), dict(out=empty(nw)))),
        ("apmm_pack_activations", PLAIN, lambda: ((a, p), dict(out=empty(na + 64)[16:]))),
        ("apmm_pack_activations", PLAIN, lambda: ((a, p), dict(out=empty(na + 64)[8:]))),
        ("apmm_pack_activations", GENERAL, lambda: ((a.as_subclass(Sub), p), dict(out=empty(na)))),
        ("apmm_quantize_pack_activations", PLAIN, lambda: ((x, p), dict(out=empty(na), scale_out=torch.zeros(M, dtype=torch.float16, device=dev)))),
        ("apmm_quantize_pack_activations", GENERAL, lambda: ((x, p, empty(na), torch.zeros(M - 1, dtype=torch.float16, device=dev)), {})),
        ("apmm_quantize_pack_activations", PLAIN, lambda: ((x, p), {})),
        ("apmm_quantize_pack_activations", PLAIN, lambda: ((x, p), dict(out=empty(na), scale_out=None))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32()))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), dict(want_i32=False, want_f16=True, w_scale=sw, a_scale=sa, c_f16=c16()))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp, True, True, sw, sa, c32(), c16()), {})),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), {})),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), dict(want_f16=True, w_scale=sw, a_scale=None, c_i32=c32()))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, 9, q, ap, wp), {})),
        ("apmm_gemm", GENERAL, lambda: ((1 << 62, N, K, p, q, ap, wp), {})),  # no such tensor
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32(), workspace=empty(64)))),
        ("apmm_gemm", GENERAL, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32(), workspace=torch.zeros(64, dtype=torch.uint8)))),
        ("apmm_gemm", GENERAL, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32(), algo=None))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), dict(want_i32=False))),
        ("apmm_gemm", GENERAL, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32(), w_scale=sw[:-1]))),
        ("apmm_gemm", GENERAL, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32(), a_scale=sa.float()))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap[1:], wp), dict(c_i32=c32()))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, 1 << 40, p, q, ap, wp), dict(c_i32=c32()))),
        ("apmm_gemm", PLAIN, lambda: ((0, N, K, p, q, ap, wp), dict(c_i32=c32()))),
        ("apmm_gemm", PLAIN, lambda: ((M, N, K, p, q, ap, wp), dict(c_i32=c32(), algo=binding.ALGO_DECODE))),
        ("apmm_gemm_from_codes", PLAIN, lambda: ((a, N, p, q, wp), dict(c_i32=c32(), workspace=empty(na)))),
        ("apmm_gemm_from_codes", PLAIN, lambda: ((a, N, p, q, wp), dict(want_i32=False, want_f16=True, c_f16=c16(), w_scale=sw, a_scale=sa))),
        ("apmm_gemm_from_codes", PLAIN, lambda: ((a, N, p, q, wp), {})),
        ("apmm_gemm_from_codes", PLAIN, lambda: ((a, N, p, q, wp), dict(want_f16=True, a_scale=sa))),
        ("apmm_gemm_from_codes", PLAIN, lambda: ((a, N, p, 9, wp), dict(c_i32=c32()))),
    ]
    stream = torch.cuda.Stream()
    for name, route, make in calls:
        results = []
        asked = []  # times that the C++ call handed over to the Python function

        def handed_over(*args, **kw):
            asked.append(name)
            return general_of[name](*args, **kw)

        binding._call.set_general(name, handed_over)
        try:
            for fn in (getattr(binding, name), general_of[name]):
                args, kw = make()
                stream.wait_stream(torch.cuda.current_stream())
                with torch.cuda.stream(stream):
                    r = outcome(fn, *args, **kw)
                stream.synchronize()
                results.append(r if isinstance(r, tuple) else (r,))
        finally:
            binding._call.set_general(name, binding._general[name])
        assert len(asked) == route, (name, asked)
        got, want = results
        assert len(got) == len(want), (name, got, want)
        for s, t in zip(got, want):
            if isinstance(t, torch.Tensor):
                assert type(s) is type(t) and s.dtype == t.dtype and torch.equal(s, t), name
            else:
                assert s == t, (name, s, t)


@pytest.mark.gpu
def test_forked_process_refused_alike():
    """A process forked from one that uses the GPU must not use it: torch's own refusal comes before anything is launched there."""
    dev = torch.device("cuda:0")
    a, w = (torch.ones((n, 64), dtype=torch.uint8, device=dev) for n in (3, 40))
    x, sa = torch.ones((3, 64), dtype=torch.float16, device=dev), torch.ones(3, dtype=torch.float16, device=dev)
    ap, wp = binding.apmm_pack_activations(a, 2), binding.apmm_pack_weights(w, 2)
    c = torch.zeros((3, 40), dtype=torch.int32, device=dev)
    calls = [("apmm_pack_weights", (w, 2, wp), {}), ("apmm_pack_activations", (a, 2, ap), {}), ("apmm_quantize_pack_activations", (x, 2, ap, sa), {}),
             ("apmm_gemm", (3, 40, 64, 2, 2, ap, wp), dict(c_i32=c)), ("apmm_gemm_from_codes", (a, 40, 2, 2, wp), dict(c_i32=c))]
    torch.cuda.synchronize()
    end, begin = os.pipe()
    child = os.fork()
    if child == 0:  # nothing here touches the GPU
        try:
            outcomes = [outcome(getattr(binding, name), *args, **kw) for name, args, kw in calls]
            os.write(begin, "\n".join("%s %s" % (o[0], str(o[1])[:30]) if isinstance(o[0], str) else "launched" for o in outcomes).encode())
        finally:
            os._exit(0)
    os.close(begin)
    with os.fdopen(end) as f:
        lines = f.read().split("\n")
    os.waitpid(child, 0)
    assert lines == ["RuntimeError Cannot re-initialize CUDA in f"] * len(calls)
