"""What a program that serves XFP-compressed layers asks of this library, as cases that can be timed.

A pass is what such a program does between two points of its own: one token (or one batch of tokens) through the
compressed matrices of a few layers, with the weights on the GPU and the calls written as in the README.  Several
layers are several matrices of one shape, because a decoder reads every matrix once per token: a pass over a single
small matrix, repeated, would find it in the last-level cache, which no decoder does.

The fields of a case:
  call     "gemv" (xfp_gemv), "noalloc" (xfp_gemv_noalloc) or "experts" (a routed-expert layer: gate/up with SiLU, then
           down with the router's weighted sum; N, K are those of the gate/up matrix, the down matrix is K x N / 2)
  format   "v2" (a codebook per row), "v2a" (a library of L codebooks, an id per group of 128 weights) or "record" (v2a
           with the scale and the mid-point per group of the paper's 40-bit group record)
  tokens   M of the call; for "experts" the tokens that are decoded one after the other, each with a routing of its own
  density  share of the weights that are outliers in CSR form
"""
import math

import torch

import paper_2605_14844_amd as xfp

GROUP = 128
DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16, "fp32": torch.float32}
#: A decoder's weights exceed the 256 MB last-level cache; the states that are walked in turn do so together.
COLD_BYTES = 140e6
#: The largest call: the benchmark's largest matrix (28672 x 8192) with a prompt of 2048 tokens.
MOST_WEIGHTS = 28672 * 8192
MOST_MACS = MOST_WEIGHTS * 2048


def _case(name, call="gemv", format="v2", bits=4, N=0, K=0, L=0, tokens=1, layers=1, density=0.003, x="fp16", y="fp16",
          experts=1, active=1):
    case = {"call": call, "format": format, "bits": bits, "N": N, "K": K, "L": L, "tokens": tokens, "layers": layers,
            "density": density, "x": x, "y": y, "experts": experts, "active": active}
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest matrix of the benchmark, a single token: what a call costs whatever it computes
        _case("small_matrix", call="noalloc", N=512, K=1024),
        # the headline shape: a token through the 4-bit projections of several layers
        _case("decode_4bit", N=8192, K=4096, layers=8),
        # the same with library tensors at 3 bits, which are small: launches count as much as bytes
        _case("decode_library_3bit", format="v2a", bits=3, N=4096, K=4096, L=32, layers=24, density=0.001),
        # the full group record of the paper in a model that keeps bf16 activations; rows that fill no power of two
        _case("decode_record_bf16", format="record", bits=4, N=6144, K=5120, L=32, layers=10, density=0.001, x="bf16", y="bf16"),
        # the widest index widths, which the sensitive layers of a model fall back to
        _case("decode_5bit", bits=5, N=8192, K=4096, layers=6, x="bf16", y="bf16"),
        # a down projection of a large model: rows longer than a wave holds
        _case("decode_long_rows", N=8192, K=28672, layers=2),
        # a routed-expert layer, 8 of 256 experts, for the tokens of four requests
        _case("experts_3bit", call="experts", bits=3, N=2048, K=4096, experts=256, active=8, tokens=4, density=0.0005),
        # a few requests at once (or a handful of drafted tokens) on 2-bit matrices of ragged size
        _case("few_tokens_2bit", bits=2, N=7001, K=5504, tokens=5, layers=6, x="bf16", y="bf16"),
        # a batch of 16 requests on the benchmark's largest matrix
        _case("batch_16", N=28672, K=8192, tokens=16),
        # a batch of 64 requests, library tensors
        _case("batch_64_library", format="v2a", bits=3, N=28672, K=8192, L=32, tokens=64),
        # a short prompt of odd length
        _case("prompt_333_library", format="v2a", bits=2, N=4096, K=4096, L=32, tokens=333, layers=4, density=0.001),
        # a long prompt on the largest matrix
        _case("prompt_2048", N=28672, K=8192, tokens=2048, x="bf16", y="bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    x = rng.choice(["fp16", "fp16", "bf16"])
    y = x if rng.random() < 0.8 else "fp32"
    density = rng.choice([0.0005, 0.001, 0.003, 0.003, 0.01])
    if rng.random() < 0.2:
        bits, I, H = rng.choice([2, 3, 3, 4]), GROUP * _log_int(rng, 2, 16), GROUP * _log_int(rng, 8, 48)
        E = _log_int(rng, 8, 256)
        E = max(8, min(E, int(1.3e9 / (3 * I * H * bits / 8))))
        return _case(None, call="experts", format=rng.choice(["v2", "v2", "v2", "v2a"]), bits=bits, N=2 * I, K=H, L=32,
                     experts=E, active=rng.randint(2, 8), tokens=rng.randint(1, 4), density=min(density, 0.001), x=x, y=y)
    format = rng.choice(["v2", "v2", "v2", "v2a", "v2a", "record"])
    bits = rng.choice([4, 4, 3, 3, 2, 2, 5, 6] if format == "v2" else [4, 3, 3, 2, 2])
    size = rng.choice([1, 1, 1, 16, 64, 2048])                  # a token, a few, a batch, a prompt
    tokens = 1 if size == 1 else _log_int(rng, {16: 2, 64: 17, 2048: 65}[size], size)
    # what runs token by token today is asked for a few tokens only, as its users do
    tokens = min(tokens, 4 if bits > 4 else 64 if format == "record" else 2048)
    K = GROUP * _log_int(rng, 4, 224)
    most = min(32768, MOST_WEIGHTS // K, (MOST_MACS // 4 if tokens > 64 else MOST_MACS) // (K * tokens))
    N = _log_int(rng, 256, max(257, most))
    layers = max(1, min(32, int(COLD_BYTES / 2 / (N * K * bits / 8)))) if tokens <= 64 else 1
    return _case(None, format=format, bits=bits, N=N, K=K, L=rng.choice([16, 32, 32, 48]) if format != "v2" else 0, tokens=tokens,
                 layers=layers, density=density, x=x, y=y)


# ---------------------------------------------------------------- inputs

def _nnz(case, N, K):
    return int(round(case["density"] * N * K))


def _index_words(gen, words, bits):
    """Packed indices whose levels occur as often as a codebook fitted to bell-shaped weights uses them: the inner
    ones more often than the outer ones.  16 random bits pick 4 indices (2 at 4 bits, 1 at 5 and 6) from a table."""
    n = {2: 4, 3: 4, 4: 2}.get(bits)
    if n is None:                                               # 5 and 6 bits: uniform words, as the tests have them
        return torch.randint(-2**31, 2**31, (words,), generator=gen, device="cuda", dtype=torch.int32)
    z = torch.linspace(-2.0, 2.0, 1 << bits, dtype=torch.float64)
    edges = torch.cumsum(torch.softmax(-z * z / 3.0, 0), 0)
    per = int(round(65536 ** (1.0 / n)))                        # random digits per index: 16 or 256
    level = torch.searchsorted(edges, (torch.arange(per, dtype=torch.float64) + 0.5) / per).clamp_(max=(1 << bits) - 1)
    r = torch.arange(per**n)
    table = sum(level[(r // per**i) % per] << (bits * i) for i in range(n)).to(torch.int32).cuda()
    if bits == 3:                                               # 12 bits each: two of them are 3 bytes
        pick = table[torch.randint(0, 65536, (words * 8 // 3 + 2,), generator=gen, device="cuda", dtype=torch.int32)[: words * 8 // 3 // 2 * 2]]
        v = pick[0::2] | (pick[1::2] << 12)
        out = torch.stack([v & 255, (v >> 8) & 255, v >> 16], 1).to(torch.uint8).reshape(-1)
        return out.view(torch.int32)[:words]
    pick = torch.randint(0, 65536, (words * 4,), generator=gen, device="cuda", dtype=torch.int32)
    return table.to(torch.uint8)[pick].view(torch.int32)


def _weights(case, N, K, E, gen):
    """One bank of E matrices [N, K] on the GPU, in the layout of include/xfp.h."""
    bits, lib = case["bits"], case["format"] != "v2"
    words = N * K * bits // 32
    indices = torch.empty((E, words), dtype=torch.int32, device="cuda")
    step = max(1, (1 << 25) // words)
    for e in range(0, E, step):
        n = min(step, E - e)
        indices[e:e + n] = _index_words(gen, n * words, bits).reshape(n, words)
    rows = case["L"] if lib else N
    if case["format"] == "record":                              # library shapes are normalised to [-1, 1]
        books = torch.rand((E, rows, 1 << bits), generator=gen, device="cuda") * 2 - 1
    else:
        books = torch.randn((E, rows, 1 << bits), generator=gen, device="cuda") * 0.02
    books = books.sort(-1).values.half()
    ids = scale = mid = None
    if lib:
        ids = torch.randint(0, rows, (E, N, K // GROUP), generator=gen, device="cuda", dtype=torch.uint8)
    if case["format"] == "record":
        scale = (torch.rand((E, N, K // GROUP), generator=gen, device="cuda") * 0.04 + 0.02).half()
        mid = (torch.randn((E, N, K // GROUP), generator=gen, device="cuda") * 0.002).half()
    nnz = E * _nnz(case, N, K)
    pos = torch.unique(torch.randint(0, E * N * K, (int(nnz * 1.03) + 64,), generator=gen, device="cuda", dtype=torch.int64))
    pos = pos[torch.randperm(pos.numel(), generator=gen, device="cuda")[:nnz]].sort().values
    row_ptr = torch.zeros(E * N + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.searchsorted(pos, torch.arange(1, E * N + 1, device="cuda") * K).to(torch.int32)
    val = (torch.randn(nnz, generator=gen, device="cuda") * 0.5).half()
    return xfp.binding.make_descriptor(xfp.XFP_MODE_V2A if lib else xfp.XFP_MODE_V2, bits, N, K, rows if lib else 0, E,
                                       indices, books.view(torch.int16), ids, row_ptr, (pos % K).to(torch.int32),
                                       val.view(torch.int16), group_scale=scale if scale is None else scale.view(torch.int16),
                                       group_mid=mid if mid is None else mid.view(torch.int16))


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    N, K, M = case["N"], case["K"], case["tokens"]
    state = {"call": case["call"], "y": DTYPES[case["y"]],
             "x": torch.randn((M, K), generator=gen, device="cuda").to(DTYPES[case["x"]])}
    if case["call"] == "experts":
        E, T = case["experts"], case["active"]
        state["gate_up"], state["down"] = _weights(case, N, K, E, gen), _weights(case, K, N // 2, E, gen)
        routing = torch.rand((M, E), generator=gen, device="cuda").topk(T, 1)
        state["ids"] = list(routing.indices.to(torch.int32))
        state["router"] = list((routing.values / routing.values.sum(1, keepdim=True)).contiguous())
    else:
        state["layers"] = [_weights(case, N, K, 1, gen) for _ in range(case["layers"])]
    if case["call"] == "noalloc":
        state["out"] = torch.empty((M, N), dtype=state["y"], device="cuda")
    return state


def run(state):
    x, y = state["x"], state["y"]
    if state["call"] == "noalloc":
        return [xfp.xfp_gemv_noalloc(W, x, state["out"]) for W in state["layers"]]
    if state["call"] == "gemv":
        return [xfp.xfp_gemv(W, x, y_dtype=y) for W in state["layers"]]
    out = []
    for t, ids in enumerate(state["ids"]):
        h = xfp.xfp_gemv_moe_silu_mul(state["gate_up"], ids, x[t], h_dtype=x.dtype)
        out += [h, xfp.xfp_gemv_moe_combine(state["down"], ids, h, state["router"][t], y_dtype=y)]
    return out


def _matrix_bytes(case, N, K):
    b = N * K * case["bits"] / 8 + 6 * _nnz(case, N, K) + 4 * (N + 1)
    if case["format"] == "v2":
        return b + N * 2 * 2 ** case["bits"]
    return b + case["L"] * 2 * 2 ** case["bits"] + N * K // GROUP * (5 if case["format"] == "record" else 1)


def work(case):
    N, K, M, T = case["N"], case["K"], case["tokens"], case["active"]
    xs, ys = DTYPES[case["x"]].itemsize, DTYPES[case["y"]].itemsize
    if case["call"] == "experts":
        I = N // 2
        per = T * (_matrix_bytes(case, N, K) + _matrix_bytes(case, K, I)) + K * xs + 2 * T * I * xs + K * ys
        return {"bytes": M * per, "flops": M * T * 2 * (N * K + _nnz(case, N, K) + K * I + _nnz(case, K, I))}
    return {"bytes": case["layers"] * (_matrix_bytes(case, N, K) + M * N * ys) + M * K * xs,
            "flops": case["layers"] * 2 * M * (N * K + _nnz(case, N, K))}


def tolerance(case):
    # sums are fp32 whatever the order; what is left is the one rounding of the output type (of h too, for experts)
    if case["call"] == "experts":
        return {"rel": 4e-3 if "bf16" in (case["x"], case["y"]) else 1e-3}
    return {"rel": {"fp32": 1e-5, "fp16": 5e-4, "bf16": 4e-3}[case["y"]]}
