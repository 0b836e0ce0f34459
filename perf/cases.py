"""The calls that a program built on this library makes, as cases that can be timed: the linear
layers of Llama-shaped decoder blocks in the draft mode (quantiser or fused producer, then the
W4A4 product), in the verify mode (the W4A16 product) and over a prompt, and the acceptance and
KV overwrite that end a cycle.  Shapes and value distributions are those of
`paper_2410_11305_amd.synth`: codes uniform in [-8, 7], scales uniform in [0.002, 0.01),
activations N(0, 1) with one channel in a hundred twenty times larger.

A decoding server runs its draft and verify passes with fixed shapes and buffers and replays them
as HIP graphs (as bench.py does), so those cases hold a captured graph over their own buffers;
the single layer and the prompt, whose length changes from request to request, are called eagerly.
Every linear layer of a pass has its own input, so that one layer's last-bit differences do not
turn into other codes in the next.
"""
from __future__ import annotations

import math

import torch

from paper_2410_11305_amd import binding as B

GROUP = 128
EPS = 1e-5

# (hidden size, qkv outputs, MLP intermediate size) of the benchmark configurations
SHAPES = {"7b": (4096, 12288, 11008), "13b": (5120, 15360, 13824), "70b": (8192, 10240, 28672)}


def _block(name, kind, shape, M, blocks, producer="fused"):
    H, Q, I = SHAPES[shape]
    return dict(name=name, kind=kind, H=H, Q=Q, I=I, M=M, blocks=blocks, producer=producer)


def listed():
    return [
        # one small layer, called eagerly in both modes on the same weights (4 sequences, one
        # draft token each, then 3 drafts + 1): latency, launches and the host's share
        dict(name="linear_1024", kind="linear", K=1024, N=1024, M=4, Mv=16),
        # a single user's draft token: everything is weight streaming and launch gaps
        _block("draft_7b_m1", "draft", "7b", 1, 2),
        # small batches, both modes (8 sequences, 3 drafts + 1)
        _block("draft_7b_m8", "draft", "7b", 8, 2),
        _block("verify_7b_m32", "verify", "7b", 32, 2),
        # medium batches, the draft with the per-group rotation against outlier channels
        _block("draft_7b_m32_rotate", "draft", "7b", 32, 2, "rotate"),
        _block("verify_7b_m128", "verify", "7b", 128, 2),
        # 64 sequences, 5 drafts + 1, the plain quantiser in front of every layer
        _block("draft_13b_m64_plain", "draft", "13b", 64, 1, "plain"),
        _block("verify_13b_m384", "verify", "13b", 384, 1),
        # 128 sequences, 3 drafts + 1: the largest decoding configuration
        _block("draft_70b_m128", "draft", "70b", 128, 1),
        _block("verify_70b_m512", "verify", "70b", 512, 1),
        # a prompt of odd length through one block in the high-precision mode
        _block("prompt_7b_m2050", "prompt", "7b", 2050, 1),
        # the end of a cycle: greedy acceptance over the verify logits, then the K and V rows of
        # the accepted tokens of two layers
        dict(name="accept_b128", kind="accept", batch=128, gamma=3, V=32000, D=4096, S=128, layers=2),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("linear", "draft", "draft", "draft", "verify", "verify", "verify", "prompt", "accept"))
    if kind == "linear":
        return dict(kind=kind, K=GROUP * rng.randint(4, 32), N=16 * rng.randint(32, 256),
                    M=_log_int(rng, 1, 32), Mv=_log_int(rng, 4, 128))
    if kind == "accept":
        return dict(kind=kind, batch=_log_int(rng, 1, 128), gamma=rng.randint(2, 6), V=rng.randint(16000, 64000),
                    D=8 * rng.randint(64, 512), S=rng.randint(64, 256), layers=rng.randint(1, 4))
    H = GROUP * rng.randint(16, 64)
    Q = H + 16 * (rng.randint(H // 4, 2 * H) // 16)           # grouped to full key / value heads
    I = GROUP * int(H * rng.uniform(2.5, 3.5) / GROUP)
    weights = _weights(H, Q, I)
    if kind == "draft":
        M = _log_int(rng, 1, 256)
    elif kind == "verify":
        M = _log_int(rng, 4, 512)
    else:
        M = _log_int(rng, 200, 2050)
    # no dearer than a pass of 512 tokens through the largest listed block
    H0, Q0, I0 = SHAPES["70b"]
    M = max(1, min(M, 512 * _weights(H0, Q0, I0) // weights))
    blocks = 1 if kind == "prompt" else max(1, min(4, round(2e8 / weights), 512 * _weights(H0, Q0, I0) // (weights * M)))
    producer = rng.choice(("fused", "fused", "plain", "rotate", "reorder")) if kind == "draft" else "fused"
    return dict(kind=kind, H=H, Q=Q, I=I, M=M, blocks=blocks, producer=producer)


def _weights(H, Q, I):
    return Q * H + H * H + 2 * I * H + H * I


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _pack(gen, N, K):
    codes = torch.randint(-8, 8, (N, K), dtype=torch.int8, device="cuda", generator=gen)
    scales = (torch.rand((N, K // GROUP), device="cuda", generator=gen) * 0.008 + 0.002).half()
    return B.pack_weights(codes, scales)


def _activations(gen, M, K):
    x = torch.randn((M, K), device="cuda", generator=gen)
    channels = torch.randperm(K, device="cuda", generator=gen)[:max(1, round(0.01 * K))]
    x[:, channels] *= 20.0
    return x.half()


def _captured(fn):
    """fn's launches as a HIP graph; fn runs once eagerly first, as torch asks of a capture."""
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        fn()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        fn()
    return graph


def _layers(case):
    """(outputs, inputs) of the four linear layers of a block."""
    H, Q, I = case["H"], case["Q"], case["I"]
    return ((Q, H), (H, H), (2 * I, H), (H, I))


def _prepare_linear(case, gen):
    K, N, M, Mv = case["K"], case["N"], case["M"], case["Mv"]
    packed = _pack(gen, N, K)
    x, xv = _activations(gen, M, K), _activations(gen, Mv, K)
    wide = B.w4a4_takes_wide(M, N, K)
    qa = torch.empty((M, K) if wide else (M, K // 2), dtype=torch.int8 if wide else torch.uint8, device="cuda")
    sa = torch.empty((M, K // GROUP), dtype=torch.float32, device="cuda")
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    yv = torch.empty((Mv, N), dtype=torch.float16, device="cuda")
    ws = B.alloc_workspace(max(B.workspace_bytes(M, N, K), B.workspace_bytes(Mv, N, K)))
    quantise, product = (B.quant_act_wide, B.gemm_w4a4_wide) if wide else (B.quant_act, B.gemm_w4a4)

    def call():
        quantise(x, qa, sa)
        product(packed, qa, sa, N, y=y, workspace=ws)
        B.gemm_w4a16(packed, xv, N, y=yv, workspace=ws)
        return y, yv
    return dict(call=call)


def _prepare_verify(case, gen):
    M, blocks = case["M"], case["blocks"]
    layers = _layers(case)
    packed = [[_pack(gen, N, K) for N, K in layers] for _ in range(blocks)]
    x = [_activations(gen, M, K) for _, K in layers]
    y = [[torch.empty((M, N), dtype=torch.float16, device="cuda") for N, _ in layers] for _ in range(blocks)]
    ws = B.alloc_workspace(max(B.workspace_bytes(M, N, K) for N, K in layers))

    def call():
        for b in range(blocks):
            for i, (N, _) in enumerate(layers):
                B.gemm_w4a16(packed[b][i], x[i], N, y=y[b][i], workspace=ws)
        return y
    return dict(call=call) if case["kind"] == "prompt" else dict(call=call, graph=_captured(call), y=y)


def _prepare_draft(case, gen):
    M, I, blocks, producer = case["M"], case["I"], case["blocks"], case["producer"]
    # the reordering quantiser carries its outlier group as two groups
    layers = [(N, K + (GROUP if producer == "reorder" else 0)) for N, K in _layers(case)]
    packed = [[_pack(gen, N, K) for N, K in layers] for _ in range(blocks)]
    y = [[torch.empty((M, N), dtype=torch.float16, device="cuda") for N, _ in layers] for _ in range(blocks)]
    ws = B.alloc_workspace(max(B.workspace_bytes(M, N, K) for N, K in layers))
    makers, products = [], []
    for i, (N, K) in enumerate(layers):
        kind = producer
        if producer in ("fused", "rotate"):                   # norm, attention, norm, SiLU * up
            kind = ("norm", "plain", "norm", "silu")[i]
            if kind == "plain" and producer == "rotate":
                kind = "hadamard"
        # only the quantisers of the packed format exist for the last two
        wide = B.w4a4_takes_wide(M, N, K) and kind not in ("hadamard", "reorder")
        qa = torch.empty((M, K) if wide else (M, K // 2), dtype=torch.int8 if wide else torch.uint8, device="cuda")
        sa = torch.empty((M, K // GROUP), dtype=torch.float32, device="cuda")
        makers.append(_maker(kind, gen, M, K, I, qa, sa, wide, producer == "rotate"))
        products.append((B.gemm_w4a4_wide if wide else B.gemm_w4a4, qa, sa, N))

    def call():
        for b in range(blocks):
            for i, (product, qa, sa, N) in enumerate(products):
                makers[i]()
                product(packed[b][i], qa, sa, N, y=y[b][i], workspace=ws)
        return y
    return dict(call=call, graph=_captured(call), y=y)


def _maker(kind, gen, M, K, I, qa, sa, wide, rotate):
    """The call that writes a draft-mode layer's activation codes and scales."""
    if kind == "norm":
        x = _activations(gen, M, K)
        w = (1.0 + 0.1 * torch.randn(K, device="cuda", generator=gen)).half()
        return lambda: B.rmsnorm_quant(x, w, EPS, qa, sa, rotate=rotate, wide=wide)
    if kind == "silu":
        gate_up = (torch.randn((M, 2 * I), device="cuda", generator=gen) * 1.5).half()
        return lambda: B.silu_mul_quant(gate_up, qa, sa, rotate=rotate, wide=wide)
    if kind == "reorder":
        x = _activations(gen, M, K - GROUP)
        perm = torch.argsort(x.float().abs().amax(dim=0)).int()          # the largest channels last
        return lambda: B.reorder_quant(x, perm, 1, qa, sa)
    x = _activations(gen, M, K)
    if kind == "hadamard":
        return lambda: B.hadamard_quant(x, qa, sa)
    return (lambda: B.quant_act_wide(x, qa, sa)) if wide else (lambda: B.quant_act(x, qa, sa))


def _prepare_accept(case, gen):
    n, gamma, V, D, S, layers = (case[k] for k in ("batch", "gamma", "V", "D", "S", "layers"))
    logits = (torch.randn((n, gamma + 1, V), device="cuda", generator=gen) * 2.0).half()
    top = logits.argmax(dim=2).int()
    miss = torch.rand((n, gamma), device="cuda", generator=gen) >= 0.8
    draft = torch.where(miss, (top[:, :gamma] + 1) % V, top[:, :gamma]).int().contiguous()
    pos = torch.randint(0, S - gamma - 1, (n,), device="cuda", generator=gen).int()
    caches = [torch.randn((n, S, D), device="cuda", generator=gen).half() for _ in range(2 * layers)]
    rows = [torch.randn((n, gamma + 1, D), device="cuda", generator=gen).half() for _ in range(2 * layers)]
    n_accept = torch.empty((n,), dtype=torch.int32, device="cuda")
    tokens = torch.zeros((n, gamma + 1), dtype=torch.int32, device="cuda")
    ws = torch.empty(max(B.accept_workspace_bytes(n, gamma, V), 16), dtype=torch.uint8, device="cuda")

    def call():
        B.greedy_accept(logits, draft, n_accept, tokens, ws)
        for cache, kv in zip(caches, rows):
            B.kv_overwrite(cache, kv, n_accept, pos)
        return n_accept, tokens, caches
    return dict(call=call, graph=_captured(call), y=(n_accept, tokens, caches))


def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    if kind == "linear":
        return _prepare_linear(case, gen)
    if kind == "accept":
        return _prepare_accept(case, gen)
    return _prepare_draft(case, gen) if kind == "draft" else _prepare_verify(case, gen)


def run(state):
    if "graph" in state:
        state["graph"].replay()
        return state["y"]
    return state["call"]()


# ------------------------------------------------------------------ what a pass cannot do without
def _packed_bytes(N, K):
    return N * K // 2 + 2 * N * (K // GROUP)


def work(case):
    kind = case["kind"]
    if kind == "linear":
        K, N, M, Mv = case["K"], case["N"], case["M"], case["Mv"]
        return dict(bytes=2 * _packed_bytes(N, K) + 2 * (M + Mv) * (K + N), flops=2 * (M + Mv) * N * K)
    if kind == "accept":
        n, gamma, V, D, layers = (case[k] for k in ("batch", "gamma", "V", "D", "layers"))
        rows = n * min(gamma, 2.4) + n                        # rows copied at four accepted drafts in five
        return dict(bytes=2 * n * (gamma + 1) * V + 2 * layers * rows * D * 2 * 2, flops=n * (gamma + 1) * V)
    M, I = case["M"], case["I"]
    n_bytes = flops = 0
    for i, (N, K) in enumerate(_layers(case)):
        inputs = 2 * I if kind == "draft" and i == 3 and case["producer"] in ("fused", "rotate") else K
        n_bytes += _packed_bytes(N, K) + 2 * M * (inputs + N)
        flops += 2 * M * N * K
    return dict(bytes=case["blocks"] * n_bytes, flops=case["blocks"] * flops)


def tolerance(case):
    if case["kind"] == "accept":
        return "exact"
    # Against float64 on the same codes and scales the fp16 rounding of a result measures 2.1e-4
    # (largest 5e-4 of a value); where a dequantised weight is rounded to fp16 as well, 2.8e-4
    # (largest 1.2e-3).  Four times that.
    if case["kind"] == "draft":
        return {"rel": 8e-4, "max": 5e-3}
    return {"rel": 1.1e-3, "max": 5e-3}
