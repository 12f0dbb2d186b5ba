"""The work that programs on this library have it do, as cases that can be timed and checked.

Three kinds of pass:

* ``layers``: the four projections of `layers` decoder layers (QKV, O, gate+up with the gated epilogue, down) on `m`
  rows, captured once into a HIP graph and replayed: how a serving loop runs the decode of a batch.  Each projection
  has input rows of its own (attention, norms and residuals between them belong to the caller); the weights of the
  layers are distinct, so that a replay streams them from memory.
* ``single``: one projection launched eagerly, from unquantised rows (`path` "fused"), int8 rows ("a8") or bf16 rows
  that stay unquantised ("a16"): one-off calls, chunks of a prompt, whole prompts.
* ``quantize`` and ``prepack``: the activation quantiser on its own (rows that feed several projections are quantised
  once) and the conversion of a checkpoint's codes and scales to the device layout.

Values follow the benchmark's recipe: codes uniform over the codec's alphabet, group scales uniform in
[0.005, 0.05] rounded to bf16, activations N(0, 1).
"""
import math

import torch

from paper_2508_06753_amd import binding as w2

ACTS = {"none": w2.ACT_NONE, "silu": w2.ACT_SILU, "silu_mul": w2.ACT_SILU_MUL}
CODECS = {"int2": w2.CODEC_INT2, "ternary": w2.CODEC_TERNARY}

# the largest pass: 2048 rows through an 8192 x 57344 projection
MOST_MACS = 2048 * 8192 * 57344


def listed():
    return [
        # one token of one user: the weight stream of an 8B-class model, one launch per projection
        dict(name="decode_8b_m1_a8", kind="layers", hidden=4096, qkv=6144, ff=14336, layers=5, m=1, path="fused", x="f32",
             group=128, codec="int2"),
        # a few users (or one user with drafted tokens) whose activations are not to be quantised
        dict(name="decode_8b_m4_a16", kind="layers", hidden=4096, qkv=6144, ff=14336, layers=5, m=4, path="a16", x="bf16",
             group=128, codec="int2"),
        # a small batch on a 27B-class ternary model
        dict(name="decode_27b_m8_a8_ternary", kind="layers", hidden=5120, qkv=7168, ff=17408, layers=3, m=8, path="fused",
             x="bf16", group=128, codec="ternary"),
        # continuous batching: dozens of users, each with one token per pass
        dict(name="batch_8b_m48_a8", kind="layers", hidden=4096, qkv=6144, ff=14336, layers=5, m=48, path="fused", x="bf16",
             group=128, codec="int2"),
        dict(name="batch_8b_m64_a16", kind="layers", hidden=4096, qkv=6144, ff=14336, layers=5, m=64, path="a16", x="bf16",
             group=128, codec="int2"),
        # the smallest call: one row through one small projection, launched from Python; latency
        dict(name="single_2048_m1", kind="single", k=2048, n=2048, m=1, path="fused", x="f32", group=128, codec="int2",
             bias=False, act="none"),
        # the tail chunk of a prompt through a deep 70B-class projection, on rows that are quantised already
        dict(name="chunk_70b_down_m100_a8", kind="single", k=28672, n=8192, m=100, path="a8", x="bf16", group=128,
             codec="int2", bias=True, act="none"),
        # a prompt of odd length, finer groups, gated epilogue
        dict(name="prefill_8b_m1000_g64", kind="single", k=4096, n=28672, m=1000, path="fused", x="bf16", group=64,
             codec="ternary", bias=False, act="silu_mul"),
        # prompts through a 70B-class model: without and with quantised activations
        dict(name="prefill_70b_down_m512_a16", kind="single", k=28672, n=8192, m=512, path="a16", x="bf16", group=128,
             codec="int2", bias=False, act="none"),
        dict(name="prefill_70b_m2048_a8", kind="single", k=8192, n=57344, m=2048, path="fused", x="bf16", group=128,
             codec="int2", bias=False, act="silu_mul"),
        # rows of a prompt, quantised once for the projections that share them
        dict(name="quantize_m2048_k8192", kind="quantize", m=2048, k=8192, x="bf16", group=128, gsum=False),
        # a checkpoint's projection on its way to the device layout
        dict(name="prepack_4096x28672", kind="prepack", k=4096, n=28672, group=128, codec="int2"),
    ]


def _log(rng, lo, hi, step=1):
    """A multiple of `step` between lo and hi, spread over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def draw(rng):
    group = rng.choice([128, 128, 64])
    codec = rng.choice(["int2", "ternary"])
    kind = rng.choice(["decode", "batch", "decode", "batch", "single", "single", "single", "prompt", "prompt",
                       "quantize", "prepack"])
    if kind in ("decode", "batch"):
        hidden = _log(rng, 1024, 8192, 256)
        qkv = hidden + 256 * rng.randint(2, hidden // 512)
        ff = min(28672, 256 * int(hidden * rng.uniform(2.5, 3.6) / 256))
        macs = hidden * (hidden + qkv + 3 * ff)
        path = rng.choice(["fused", "fused", "a16"])
        return dict(kind="layers", hidden=hidden, qkv=qkv, ff=ff, layers=max(1, min(8, int(1.1e9 / macs))),
                    m=_log(rng, 1, 16) if kind == "decode" else _log(rng, 17, 256), path=path,
                    x="bf16" if path == "a16" else rng.choice(["f32", "bf16"]), group=group, codec=codec)
    if kind in ("single", "prompt"):
        path = rng.choice(["fused", "a8", "a16"])
        act = rng.choice(["none", "none", "silu", "silu_mul"])
        m = _log(rng, 1, 512) if kind == "single" else _log(rng, 129, 4096)
        k = _log(rng, 1024, 28672, 256)
        n = _log(rng, 1024, 57344, 32 if act == "silu_mul" else 8)
        if m * k * n > MOST_MACS:
            m = MOST_MACS // (k * n)
        return dict(kind="single", k=k, n=n, m=m, path=path, x="bf16" if path == "a16" else rng.choice(["f32", "bf16"]),
                    group=group, codec=codec, bias=rng.random() < 0.3, act=act)
    if kind == "quantize":
        return dict(kind="quantize", m=_log(rng, 1, 4096), k=_log(rng, 1024, 28672, 256), x=rng.choice(["f32", "bf16"]),
                    group=group, gsum=rng.random() < 0.3)
    # (K in steps of 1024: the blob then ends with its last scale, without alignment bytes of undefined content)
    return dict(kind="prepack", k=_log(rng, 1024, 28672, 1024), n=_log(rng, 1024, 16384, 8), group=group, codec=codec)


def _projections(case):
    """(K, N, activation) of each projection of one layer; one entry for a single call."""
    if case["kind"] == "layers":
        h, q, f = case["hidden"], case["qkv"], case["ff"]
        return [(h, q, "none"), (h, h, "none"), (h, 2 * f, "silu_mul"), (f, h, "none")]
    return [(case["k"], case["n"], case["act"])]


def _weights(case, K, N, gen):
    codes = torch.randint(0, 4 if case["codec"] == "int2" else 3, (K, N), dtype=torch.uint8, device="cuda", generator=gen)
    scales = torch.empty((K // case["group"], N), dtype=torch.float32, device="cuda")
    return codes, scales.uniform_(0.005, 0.05, generator=gen).to(torch.bfloat16)


def _rows(case, M, K, gen):
    return torch.randn((M, K), dtype=torch.float32, device="cuda", generator=gen).to(
        torch.float32 if case["x"] == "f32" else torch.bfloat16)


def _calls(case, seed):
    """The inputs of each call of a pass: (K, N, activation, codes, scales, rows, bias)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    for _ in range(case.get("layers", 1)):
        for K, N, act in _projections(case):
            codes, scales = _weights(case, K, N, gen)
            rows = _rows(case, case["m"], K, gen)
            bias = (torch.randn(N, dtype=torch.float32, device="cuda", generator=gen).to(torch.bfloat16)
                    if case.get("bias") else None)
            yield K, N, act, codes, scales, rows, bias


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "quantize":
        return {"case": case, "x": _rows(case, case["m"], case["k"], gen)}
    if case["kind"] == "prepack":
        codes, scales = _weights(case, case["k"], case["n"], gen)
        return {"case": case, "codes": codes, "scales": scales}
    G, M, path = case["group"], case["m"], case["path"]
    room = max(w2.workspace_size(M, K, N, G, a16=path == "a16") for K, N, _ in _projections(case))
    ws = torch.empty(max(16, room), dtype=torch.uint8, device="cuda")
    calls = []
    for K, N, act, codes, scales, rows, bias in _calls(case, seed):
        packed = w2.prepack(codes, scales, G, CODECS[case["codec"]])
        if path == "a8":
            xq, sx, _ = w2.quantize_rows(rows, G)
            rows = (xq, sx)
        calls.append({"packed": packed, "K": K, "N": N, "rows": rows, "bias": bias, "act": act, "out": None})
    state = {"case": case, "calls": calls, "ws": ws, "graph": None}
    if case["kind"] == "layers":
        for c in calls:
            c["out"] = torch.empty((M, c["N"] // 2 if c["act"] == "silu_mul" else c["N"]), dtype=torch.bfloat16,
                                   device="cuda")
        _pass(state)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _pass(state)
        state["graph"] = graph
    return state


def _pass(state):
    """Every projection of the pass through its public call."""
    G, path, ws, outs = state["case"]["group"], state["case"]["path"], state["ws"], []
    for c in state["calls"]:
        args = (c["packed"], c["K"], c["N"], G)
        plain = c["bias"] is None and c["act"] == "none"
        more = {"out": c["out"], "workspace": ws}
        if not plain:
            more.update(bias=c["bias"], act=ACTS[c["act"]])
        if path == "a8":
            outs.append((w2.matmul_a8 if plain else w2.matmul_a8_epi)(*args, *c["rows"], **more))
        elif path == "a16":
            outs.append((w2.matmul_a16 if plain else w2.matmul_a16_epi)(*args, c["rows"], **more))
        else:
            outs.append((w2.matmul_a8_fused if plain else w2.matmul_a8_fused_epi)(*args, c["rows"], **more))
    return outs


def run(state):
    case = state["case"]
    if case["kind"] == "quantize":
        xq, sx, gsum = w2.quantize_rows(state["x"], case["group"], want_gsum=case["gsum"])
        return [xq, sx, gsum] if case["gsum"] else [xq, sx]
    if case["kind"] == "prepack":
        return w2.prepack(state["codes"], state["scales"], case["group"], CODECS[case["codec"]])
    if state["graph"] is not None:
        state["graph"].replay()
        return [c["out"] for c in state["calls"]]
    return _pass(state)


def work(case):
    if case["kind"] == "quantize":
        M, K = case["m"], case["k"]
        size = 4 if case["x"] == "f32" else 2
        return {"bytes": M * K * (size + 1) + 4 * M + (4 * M * (K // case["group"]) if case["gsum"] else 0),
                "flops": 2 * M * K}
    if case["kind"] == "prepack":
        K, N, G = case["k"], case["n"], case["group"]
        return {"bytes": K * N + 2 * (K // G) * N + w2.packed_size(K, N, G), "flops": 0}
    M, G = case["m"], case["group"]
    row_bytes = {"a8": lambda K: K + 4, "a16": lambda K: 2 * K,
                 "fused": lambda K: (4 if case["x"] == "f32" else 2) * K}[case["path"]]
    total = flops = 0
    for K, N, act in _projections(case):
        n_out = N // 2 if act == "silu_mul" else N
        total += K * N // 4 + 2 * (K // G) * N + M * row_bytes(K) + 2 * M * n_out + (2 * N if case.get("bias") else 0)
        flops += 2 * M * K * N
    layers = case.get("layers", 1)
    return {"bytes": layers * total, "flops": layers * flops}


def tolerance(case):
    """Codes, row scales and the packed layout are defined bit for bit.  Outputs are bf16: one rounding apart, over
    fp32 sums in any order (a rounding to bf16 moves a value by 1.7e-3 in the root mean square, by 2^-8 at most; a
    gated output multiplies two sums)."""
    if case["kind"] in ("quantize", "prepack"):
        return "exact"
    return {"rel": 2e-3, "max": 2e-2}


def _quantized(rows):
    """int8 codes and row scales by the quantiser's definition: every operation in binary32, one rounding each (the
    64-bit quotient or product of two 32-bit numbers, rounded to 32 bits, is that)."""
    x = rows.to(torch.float32).to(torch.float64)
    amax = x.abs().amax(dim=1, keepdim=True)
    inv = torch.where(amax > 0, 127.0 / amax, torch.zeros_like(amax)).to(torch.float32).to(torch.float64)
    codes = (x * inv).to(torch.float32).round().clamp_(-127, 127)
    return codes.to(torch.float64), (amax / 127.0).to(torch.float32).to(torch.float64)


def exact(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "prepack":
        return None
    if case["kind"] == "quantize":
        _, sx = _quantized(_rows(case, case["m"], case["k"], gen))
        return [None, sx.reshape(-1)] + ([None] if case["gsum"] else [])
    outs = []
    for K, N, act, codes, scales, rows, bias in _calls(case, seed):
        if case["path"] == "a16":
            x, sx = rows.to(torch.float64), None
        else:
            x, sx = _quantized(rows)
        z = torch.empty((case["m"], N), dtype=torch.float64, device="cuda")
        for n in range(0, N, 8192):                       # in slices of columns: the weights in 64 bits are large
            q = codes[:, n:n + 8192].to(torch.float64) - (2 if case["codec"] == "int2" else 1)
            q *= scales[:, n:n + 8192].to(torch.float64).repeat_interleave(case["group"], dim=0)
            z[:, n:n + 8192] = x @ q
        if sx is not None:
            z *= sx
        if bias is not None:
            z += bias.to(torch.float64)
        if act == "silu":
            z = z * torch.sigmoid(z)
        elif act == "silu_mul":                           # blocks of 16 columns: gate, up, gate, up, ...
            z = z.reshape(case["m"], N // 32, 2, 16)
            z = (z[:, :, 0] * torch.sigmoid(z[:, :, 0]) * z[:, :, 1]).reshape(case["m"], N // 2)
        outs.append(z)
    return outs
