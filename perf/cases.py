"""What this library's users have it do, as cases whose time can be taken.

Every case is one pass through the public entry points of ``paper_2409_17870_amd.binding``, the way a user's program
calls them.  Three kinds:

  "linear"   one linear, C = A W^T, as separate calls from Python.  The weights were packed when the model was loaded;
             the activations arrive with the call, as codes (``source`` "codes": ``apmm_gemm_from_codes``; "pack":
             ``apmm_pack_activations`` + ``apmm_gemm``) or as binary16 features ("f16":
             ``apmm_quantize_pack_activations`` + ``apmm_gemm``).  ``out`` names the results asked for.
  "fresh"    a product of two matrices that both arrive with the call: ``apmm_pack_weights`` is inside as well.
  "layers"   the seven linears of each of ``layers`` decoder layers (q, k, v, o, gate, up, down), in the order of their
             dependencies: the projections that share an input are one ``apmm_gemm_grouped`` call where ``graph`` is
             set (a serving loop that captured its decode step once and replays it), else one ``apmm_gemm`` each.

Inputs are drawn on the GPU from the seed: Bernoulli(1/2) bits for weights and for activations of one or two bits, a
discretised, clipped normal for wider activation codes, N(0,1) with some heavy channels for features, U(0.01, 0.1) for
scales.
"""
import math

import torch

from paper_2409_17870_amd import binding


def listed():
    return [
        # The tiny W1A2 configuration: what any single small product costs a caller, launches and host work included.
        dict(name="tiny_w1a2", kind="linear", M=16, N=256, K=512, p=2, q=1, source="pack", out="i32", scaled=False),
        # One token through one Llama-2-7B linear, called from Python: the latency of a decode step without a graph.
        dict(name="decode_call_w2a2", kind="linear", M=1, N=11008, K=4096, p=2, q=2, source="codes", out="f16",
             scaled=True),
        # Token generation for one sequence: four 7B decoder layers inside a captured step, weights from memory.
        dict(name="decode_layers_w2a2_m1", kind="layers", graph=True, layers=4, M=1, hidden=4096, ffn=11008, p=2, q=2,
             source="codes"),
        # Token generation for a batch of 16 sequences, features quantised on the way: two 13B layers, W4A4.
        dict(name="decode_layers_w4a4_m16", kind="layers", graph=True, layers=2, M=16, hidden=5120, ffn=13824, p=4, q=4,
             source="f16"),
        # A short prompt of an odd number of tokens.
        dict(name="short_prompt_w2a2", kind="linear", M=203, N=4096, K=4096, p=2, q=2, source="codes", out="f16",
             scaled=True),
        # The 13B decoder-layer sweep: a 512-token prefill through all linears of a layer, packing included.
        dict(name="layer13b_w2a4_m512", kind="layers", graph=False, layers=1, M=512, hidden=5120, ffn=13824, p=4, q=2,
             source="codes"),
        # A long prefill through the widest 7B linear, both outputs.
        dict(name="prefill_w2a4_m2048", kind="linear", M=2048, N=11008, K=4096, p=4, q=2, source="pack", out="both",
             scaled=True),
        # The square W1A2 product of the paper's first table: the library's headline figure.
        dict(name="square_w1a2_4096", kind="linear", M=4096, N=4096, K=4096, p=2, q=1, source="pack", out="i32",
             scaled=False),
        # Two matrices that both arrive with the call, no size a multiple of anything.
        dict(name="fresh_w3a3_ragged", kind="fresh", M=1000, N=5003, K=3001, p=3, q=3, source="pack", out="both",
             scaled=True),
        # A prefill at the widest codes of the paper's evaluation, features quantised on the way.
        dict(name="prefill_w4a4_f16", kind="linear", M=1024, N=4096, K=11008, p=4, q=4, source="f16", out="f16",
             scaled=True),
        # Eight-bit weights and activations, the usual fallback for layers that low widths hurt.
        dict(name="prefill_w8a8", kind="linear", M=512, N=4096, K=4096, p=8, q=8, source="pack", out="f16", scaled=True),
        # Low-bit weights under eight-bit activations at a few tokens.
        dict(name="decode_w4a8", kind="linear", M=8, N=11008, K=4096, p=8, q=4, source="codes", out="f16", scaled=True),
    ]


# The most that a drawn case may cost: operations, for wide codes weighted with the number of plane pairs (the general
# kernel's work), and packed plus unpacked bytes of the operands.
_MOST_OPS = 2.0 * 2048 * 11008 * 4096
_MOST_PAIR_OPS = 64 * 2.0 * 512 * 4096 * 4096


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi):
    """A size between lo and hi: often a round one, as model widths are, sometimes any number."""
    x = _log_int(rng, lo, hi)
    how = rng.random()
    step = 256 if how < 0.5 else 16 if how < 0.75 else 1
    return min(hi, max(lo, (x + step - 1) // step * step))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "wide", "layers", "fresh"])
    if kind == "layers":
        graph = rng.random() < 0.7
        hidden = 512 * rng.randint(4, 10)
        return dict(kind="layers", graph=graph, layers=rng.randint(1, 3) if graph else 1,
                    M=_log_int(rng, 1, 64) if graph else _log_int(rng, 65, 512), hidden=hidden,
                    ffn=min(13824, 128 * int(round(hidden * rng.uniform(2.5, 4.0) / 128))), p=rng.randint(1, 4),
                    q=rng.randint(1, 4), source=rng.choice(["codes", "f16"]))
    p, q = rng.randint(1, 4), rng.randint(1, 4)
    if kind == "wide":
        p, q = rng.choice([(8, rng.randint(1, 8)), (rng.randint(5, 8), rng.randint(1, 8)), (rng.randint(1, 8), 8)])
    while True:
        M = _log_int(rng, 1, 4096)
        N, K = _size(rng, 256, 11008), _size(rng, 256, 11008)
        ops = 2.0 * M * N * K
        if kind == "wide":
            rows = (M + 63) // 64 * 64  # the general kernel's row tile
            if 2.0 * rows * N * K * p * q <= _MOST_PAIR_OPS:
                break
        elif ops <= _MOST_OPS:
            break
    return dict(kind="fresh" if kind == "fresh" else "linear", M=M, N=N, K=K, p=p, q=q,
                source="pack" if kind == "fresh" else rng.choice(["codes", "pack", "f16"]),
                out=rng.choice(["i32", "f16", "both"]), scaled=rng.random() < 0.8)


# ---------------------------------------------------------------- inputs ----
def _rng(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _bits(g, rows, K, bits):
    return torch.randint(0, 1 << bits, (rows, K), generator=g, device="cuda", dtype=torch.uint8)


def _activation_codes(g, M, K, p):
    if p <= 2:
        return _bits(g, M, K, p)
    half = 1 << (p - 1)
    z = torch.randn((M, K), generator=g, device="cuda")
    # three sigma on the outermost code
    return (torch.floor(z * (half / 3.0)) + half).clamp_(0, 2 * half - 1).to(torch.uint8)


def _features(g, M, K):
    x = torch.randn((M, K), generator=g, device="cuda")
    x[:, ::97] *= 8.0
    return x.to(torch.float16)


def _scales(g, n, bits):
    """U(0.01, 0.1) at up to four bits; a wider grid has finer steps over the same range."""
    s = 0.01 + 0.09 * torch.rand(n, generator=g, device="cuda")
    return (s * min(1.0, 15.0 / ((1 << bits) - 1))).to(torch.float16)


class _Linear:
    """What a program holds for one linear: packed weights, scales, outputs."""

    def __init__(self, g, M, N, K, q, out, scaled):
        self.N, self.K = N, K
        self.w = binding.apmm_pack_weights(_bits(g, N, K, q), q)
        self.w_scale = _scales(g, N, q) if scaled else None
        self.c_i32 = torch.empty((M, N), dtype=torch.int32, device="cuda") if out in ("i32", "both") else None
        self.c_f16 = torch.empty((M, N), dtype=torch.float16, device="cuda") if out in ("f16", "both") else None


class _Activations:
    """One activation matrix as it arrives, and room for its packed form."""

    def __init__(self, g, M, K, p, source, scaled):
        self.x = _features(g, M, K) if source == "f16" else _activation_codes(g, M, K, p)
        self.packed = torch.empty(binding.apmm_packed_activation_bytes(M, K, p), dtype=torch.uint8, device="cuda")
        self.scale = None
        if source == "f16":
            self.scale = torch.empty(M, dtype=torch.float16, device="cuda")
        elif scaled:
            self.scale = _scales(g, M, p)


def prepare(case, seed):
    g = _rng(seed)
    s = dict(case=case)
    M, p, q = case["M"], case["p"], case["q"]
    if case["kind"] == "layers":
        h, f = case["hidden"], case["ffn"]
        s["layers"] = []
        for _ in range(case["layers"]):
            layer = []
            for names_k, widths in ((h, (h, h, h)), (h, (h,)), (h, (f, f)), (f, (h,))):
                acts = _Activations(g, M, names_k, p, case["source"], True)
                layer.append((acts, [_Linear(g, M, n, names_k, q, "f16", True) for n in widths]))
            s["layers"].append(layer)
        if case["graph"]:
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                _layers_step(s)
            torch.cuda.current_stream().wait_stream(stream)
            s["step"] = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s["step"], stream=stream):
                _layers_step(s)
        return s
    s["a"] = _Activations(g, M, case["K"], p, case["source"], case["scaled"])
    s["linear"] = _Linear(g, M, case["N"], case["K"], q, case["out"], case["scaled"])
    if case["kind"] == "fresh":
        s["w_codes"] = _bits(g, case["N"], case["K"], q)
    return s


# ------------------------------------------------------------------- run ----
def _pack(acts, p, source):
    if source == "f16":
        binding.apmm_quantize_pack_activations(acts.x, p, out=acts.packed, scale_out=acts.scale)
    else:
        binding.apmm_pack_activations(acts.x, p, out=acts.packed)


def _layers_step(s):
    case = s["case"]
    M, p, q, source, grouped = case["M"], case["p"], case["q"], case["source"], case["graph"]
    outs = []
    for layer in s["layers"]:
        for acts, linears in layer:
            if grouped and source == "codes" and len(linears) == 1:
                lin = linears[0]
                binding.apmm_gemm_from_codes(acts.x, lin.N, p, q, lin.w, want_i32=False, want_f16=True,
                                             w_scale=lin.w_scale, a_scale=acts.scale, c_f16=lin.c_f16,
                                             workspace=acts.packed)
            else:
                _pack(acts, p, source)
                if grouped and len(linears) > 1:
                    binding.apmm_gemm_grouped([dict(M=M, N=lin.N, K=lin.K, a_packed=acts.packed, w_packed=lin.w,
                                                    c_f16=lin.c_f16, w_scale=lin.w_scale, a_scale=acts.scale)
                                               for lin in linears], p, q)
                else:
                    for lin in linears:
                        binding.apmm_gemm(M, lin.N, lin.K, p, q, acts.packed, lin.w, want_i32=False, want_f16=True,
                                          w_scale=lin.w_scale, a_scale=acts.scale, c_f16=lin.c_f16)
            outs += [lin.c_f16 for lin in linears]
    return outs


def run(state):
    case = state["case"]
    if case["kind"] == "layers":
        if case["graph"]:
            state["step"].replay()
            return [lin.c_f16 for layer in state["layers"] for _, linears in layer for lin in linears]
        return _layers_step(state)
    M, N, K, p, q = case["M"], case["N"], case["K"], case["p"], case["q"]
    a, lin = state["a"], state["linear"]
    want = dict(want_i32=lin.c_i32 is not None, want_f16=lin.c_f16 is not None, w_scale=lin.w_scale, a_scale=a.scale,
                c_i32=lin.c_i32, c_f16=lin.c_f16)
    if case["source"] == "codes":
        out = binding.apmm_gemm_from_codes(a.x, N, p, q, lin.w, workspace=a.packed, **want)
        return [c for c in out if c is not None]
    if case["kind"] == "fresh":
        binding.apmm_pack_weights(state["w_codes"], q, out=lin.w)
    _pack(a, p, case["source"])
    out = [c for c in binding.apmm_gemm(M, N, K, p, q, a.packed, lin.w, **want) if c is not None]
    return out + [a.scale] if case["source"] == "f16" else out


# ------------------------------------------------------------------ work ----
def _linear_work(M, N, K, p, q, out, fresh=False):
    weights = N * K if fresh else N * K * q / 8.0
    results = M * N * ((4 if out in ("i32", "both") else 0) + (2 if out in ("f16", "both") else 0))
    return weights + results + 2 * N + 2 * M, 2.0 * M * N * K


def work(case):
    """Activations read once as they arrive (one byte a code, two a feature), packed weights once, outputs once."""
    M, p, q = case["M"], case["p"], case["q"]
    unit = 2 if case["source"] == "f16" else 1
    if case["kind"] == "layers":
        h, f = case["hidden"], case["ffn"]
        nbytes = unit * M * (3 * h + f)
        ops = 0.0
        for n, k in [(h, h)] * 4 + [(f, h)] * 2 + [(h, f)]:
            b, o = _linear_work(M, n, k, p, q, "f16")
            nbytes, ops = nbytes + b, ops + o
        return {"bytes": case["layers"] * nbytes, "flops": case["layers"] * ops}
    nbytes, ops = _linear_work(M, case["N"], case["K"], p, q, case["out"], case["kind"] == "fresh")
    return {"bytes": nbytes + unit * M * case["K"], "flops": ops}


def tolerance(case):
    """int32 results are exact.  A binary16 result is C a_scale w_scale, two single-precision products and one rounding:
    against the same in double precision one result in 17000 lands on the neighbouring binary16 number (a part in 1024
    at most), 6e-6 in the 2-norm."""
    if case["kind"] != "layers" and case["out"] == "i32" and case["source"] != "f16":
        return "exact"
    return {"rel": 2.5e-5, "max": 1e-3}
