"""The work that a user of this framework gives it, as cases that can be timed and compared.

A drafter serves one speculative-decoding request at a time: a few in-flight tokens, the decoder linears pruned and
packed once at load time, everything resident on the GPU.  The cases go through the package's public entry points as
such a program calls them: single linears, the gated MLP block, the decoder stack without and with a key/value cache,
whole drafting rounds with the LM head and the verification, and the masked gradient of sparse fine-tuning.

Shapes are those of ``sd2_workload.CONFIGS`` (a 3B-, a 1.5B- and a 1B-shape drafter) or generic ones.  Weights are
0.02 z pruned by magnitude per row (or 2:4), activations z, z ~ N(0, 1), bf16.  A stack has at most four different
layers' weights (packing is host work); every layer has its own copy in memory, so nothing is read twice from a cache.
"""

import math
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import torch

import paper_2504_08838_amd as sd2

FORMATS = {"bitmask": 1, "2:4": 3}  # blob formats; "dense" is stored as it is
DISTINCT_LAYERS = 4
ROPE_THETA = 500000.0
HEAD_DIM = 128

LLAMA_3B = {"layers": 28, "hidden": 3072, "n_heads": 24, "n_kv": 8, "inter": 8192}
QWEN_1_5B = {"layers": 28, "hidden": 1536, "n_heads": 12, "n_kv": 2, "inter": 8960}


def listed():
    return [
        # one small linear on one token: the smallest call, launch latency and little else
        {"name": "linear-512", "kind": "linear", "n_out": 512, "k_in": 512, "sparsity": 50, "k_tok": 1, "format": "bitmask"},
        # a linear whose rows and columns fit no tile, on an odd number of tokens, at the sparsest setting of the one-shot grid
        {"name": "linear-ragged", "kind": "linear", "n_out": 5003, "k_in": 4160, "sparsity": 75, "k_tok": 13, "format": "bitmask"},
        # the gated MLP block of the 1B shape at a usual draft length
        {"name": "mlp-1b", "kind": "mlp", "hidden": 2048, "inter": 8192, "sparsity": 50, "k_tok": 5, "format": "bitmask"},
        # the benchmark's headline: the 3B-shape stack on five draft tokens, then the verification of a batch of drafts
        {"name": "forward-3b", "kind": "forward", **LLAMA_3B, "sparsity": 50, "k_tok": 5, "format": "bitmask", "verify": 64},
        # the smaller drafter, sparser, on fewer tokens: short phases, where synchronisation counts
        {"name": "forward-1.5b", "kind": "forward", **QWEN_1_5B, "sparsity": 60, "k_tok": 3, "format": "bitmask", "verify": 0},
        # the 2:4 drafter that the paper evaluates next to the unstructured one
        {"name": "forward-3b-2of4", "kind": "forward", **LLAMA_3B, "sparsity": 50, "k_tok": 5, "format": "2:4", "verify": 0},
        # the wide regime (token trees, several requests in one call): the most tokens that a call takes
        {"name": "forward-3b-wide", "kind": "forward", **LLAMA_3B, "sparsity": 50, "k_tok": 64, "format": "bitmask", "verify": 0},
        # the unpruned drafter that the pruned one is compared with
        {"name": "forward-1.5b-dense", "kind": "forward", **QWEN_1_5B, "sparsity": 0, "k_tok": 5, "format": "dense", "verify": 0},
        # prefill: a chunk of the prompt enters the cache behind what is there already
        {"name": "prefill-1.5b", "kind": "decode", **QWEN_1_5B, "sparsity": 50, "k_tok": 64, "format": "bitmask", "pos0": 448, "max_pos": 1024},
        # decode: one token against a cache (a 300-token prompt and half of 256 generated tokens)
        {"name": "decode-3b", "kind": "decode", **LLAMA_3B, "sparsity": 50, "k_tok": 1, "format": "bitmask", "pos0": 428, "max_pos": 1024},
        # a whole speculative round: five sequential draft tokens against the cache, each through the LM head, then verified
        {"name": "round-3b", "kind": "round", **LLAMA_3B, "sparsity": 50, "k_tok": 5, "format": "bitmask", "pos0": 428, "max_pos": 1024,
         "vocab": 128256},
        # the masked-gradient step of sparse fine-tuning on the largest matrix of the 3B shape
        {"name": "gradient-3b", "kind": "gradient", "n_out": 16384, "k_in": 3072, "sparsity": 50, "dtype": "float32"},
    ]


# ------------------------------------------------------------------ drawn cases


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _draw_stack(rng):
    """A decoder between a quarter of the 1.5B shape's width and the 3B shape's, grouped heads, ragged widths among them."""
    heads = rng.randint(4, 24)
    n_kv = rng.choice([g for g in range(1, heads + 1) if heads % g == 0 and 2 <= heads // g <= 6] or [heads])
    hidden = HEAD_DIM * heads
    inter = min(8192, 64 * rng.randint(2 * hidden // 64, 5 * hidden // 64))
    return {"layers": _log_int(rng, 4, 28), "hidden": hidden, "n_heads": heads, "n_kv": n_kv, "inter": inter}


def _draw_format(rng):
    fmt = rng.choice(["bitmask", "bitmask", "bitmask", "2:4", "dense"])
    return {"format": fmt, "sparsity": {"bitmask": rng.choice([50, 60, 66, 70, 75]), "2:4": 50, "dense": 0}[fmt]}


def draw(rng):
    kind = rng.choice(["linear", "linear", "mlp", "forward", "forward", "forward", "wide", "prefill", "decode", "round", "gradient"])
    if kind == "linear":
        return {"kind": "linear", "n_out": _log_int(rng, 48, 16384), "k_in": 64 * _log_int(rng, 1, 144), "k_tok": _log_int(rng, 1, 64),
                **_draw_format(rng)}
    if kind == "mlp":
        return {"kind": "mlp", "hidden": 64 * rng.randint(8, 64), "inter": 64 * _log_int(rng, 16, 160), "k_tok": _log_int(rng, 1, 64),
                **_draw_format(rng)}
    if kind in ("forward", "wide"):
        k_tok = rng.randint(1, 8) if kind == "forward" else _log_int(rng, 9, 64)
        return {"kind": "forward", **_draw_stack(rng), **_draw_format(rng), "k_tok": k_tok, "verify": rng.choice([0, 64])}
    if kind in ("prefill", "decode"):
        k_tok = _log_int(rng, 1, 8) if kind == "decode" else _log_int(rng, 16, 64)
        pos0 = _log_int(rng, 16, 3000)
        return {"kind": "decode", **_draw_stack(rng), **_draw_format(rng), "k_tok": k_tok, "pos0": pos0,
                "max_pos": pos0 + k_tok + rng.randint(0, 500)}
    if kind == "round":
        pos0, k_tok = _log_int(rng, 16, 3000), rng.randint(2, 6)
        return {"kind": "round", **_draw_stack(rng), "format": "bitmask", "sparsity": rng.choice([50, 60, 66, 70, 75]), "k_tok": k_tok,
                "pos0": pos0, "max_pos": pos0 + k_tok + rng.randint(0, 500), "vocab": _log_int(rng, 32000, 128256)}
    return {"kind": "gradient", "n_out": _log_int(rng, 256, 16384), "k_in": 64 * _log_int(rng, 4, 128), "sparsity": rng.choice([50, 60, 70]),
            "dtype": rng.choice(["float32", "bfloat16"])}


# ------------------------------------------------------------------ what a program has in hand before the call


def _keep(k_in, sparsity):
    return k_in - (sparsity * k_in) // 100


def _weight(gen, n_out, k_in, sparsity, fmt):
    """bf16 weights on the GPU, pruned entries zero."""
    w = torch.empty((n_out, k_in), dtype=torch.float32, device="cuda").normal_(0.0, 0.02, generator=gen)
    if fmt == "2:4":
        groups = w.abs().view(n_out, k_in // 4, 4)
        mask = torch.zeros_like(groups, dtype=torch.bool).scatter_(2, groups.topk(2, dim=2, sorted=False).indices, True).view(n_out, k_in)
        w = torch.where(mask, w, torch.zeros_like(w))
    elif sparsity:
        # the smallest magnitude that a row keeps
        threshold = w.abs().topk(_keep(k_in, sparsity), dim=1, sorted=False).values.amin(dim=1, keepdim=True)
        w = torch.where(w.abs() >= threshold, w, torch.zeros_like(w))
    return w.to(torch.bfloat16)


class _Packed:
    """A matrix as the library takes it: the packed blob (or the dense matrix) on the GPU and its descriptor."""

    def __init__(self, w, fmt):
        self.n_out, self.k_in = w.shape
        if fmt == "dense":
            self.host, self.dev = None, w
            self.m = sd2.matrix_init_dense(w.data_ptr(), self.n_out, self.k_in)
        else:
            self.host = sd2.pack_sparse(w.view(torch.int16).cpu().numpy().view(np.uint16), FORMATS[fmt])
            self.dev = torch.from_numpy(self.host).cuda()
            self.m = sd2.matrix_init_sparse(self.host, self.dev.data_ptr())

    def copy(self):
        """The same weights at an address of their own."""
        other = object.__new__(_Packed)
        other.n_out, other.k_in, other.host, other.dev = self.n_out, self.k_in, self.host, self.dev.clone()
        other.m = (sd2.matrix_init_dense(other.dev.data_ptr(), self.n_out, self.k_in) if self.host is None
                   else sd2.matrix_init_sparse(self.host, other.dev.data_ptr()))
        return other


def _layer_shapes(case):
    hidden, inter, kv = case["hidden"], case["inter"], case["n_kv"] * HEAD_DIM
    q_out = case["n_heads"] * HEAD_DIM
    return [(q_out + 2 * kv, hidden), (hidden, q_out), (2 * inter, hidden), (hidden, inter)]  # q|k|v, o, gate|up, down


def _pack_all(weights, fmt):
    with ThreadPoolExecutor(max_workers=16) as pool:
        return list(pool.map(lambda w: _Packed(w, fmt), weights))


def _model(case, gen):
    distinct = min(case["layers"], DISTINCT_LAYERS)
    weights = [_weight(gen, n, k, case["sparsity"], case["format"]) for _ in range(distinct) for n, k in _layer_shapes(case)]
    packed = _pack_all(weights, case["format"])
    mats = [packed[i] if i < len(packed) else packed[i % len(packed)].copy() for i in range(4 * case["layers"])]
    shape = sd2.ModelShape(case["layers"], case["hidden"], case["n_heads"] * HEAD_DIM, case["n_kv"] * HEAD_DIM, case["inter"],
                           case["n_heads"], case["n_kv"], HEAD_DIM)
    return sd2.model_create(shape, [m.m for m in mats], keep=mats)


def _bf16(gen, *shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda").normal_(generator=gen).to(torch.bfloat16)


def _buffer(n_bytes):
    return torch.empty(max(n_bytes, 16), dtype=torch.uint8, device="cuda")


def _cache(gen, case):
    c = torch.zeros((case["layers"], case["n_kv"], case["max_pos"], HEAD_DIM), dtype=torch.bfloat16, device="cuda")
    c[:, :, : case["pos0"]] = _bf16(gen, case["layers"], case["n_kv"], case["pos0"], HEAD_DIM)
    return c


def _targets(gen, batch, k, vocab, likely):
    """The target model's greedy tokens: equal to `likely` with probability 0.85 at each position."""
    other = torch.randint(0, vocab, (batch, k + 1), generator=gen, device="cuda")
    hit = torch.rand((batch, k + 1), generator=gen, device="cuda") < 0.85
    return torch.where(hit, likely, other).to(torch.int32).contiguous()


class _State:
    pass


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    s = _State()
    s.case = case
    s.stream = torch.cuda.current_stream().cuda_stream
    kind = case["kind"]
    k = case.get("k_tok", 0)
    if kind == "linear":
        s.mat = _Packed(_weight(gen, case["n_out"], case["k_in"], case["sparsity"], case["format"]), case["format"])
        s.x = _bf16(gen, k, case["k_in"])
        s.y = torch.empty((k, case["n_out"]), dtype=torch.float32, device="cuda")
        s.ws_bytes = sd2.linear_workspace_size(s.mat.m, k)
    elif kind == "mlp":
        hidden, inter = case["hidden"], case["inter"]
        s.gate_up, s.down = _pack_all([_weight(gen, 2 * inter, hidden, case["sparsity"], case["format"]),
                                       _weight(gen, hidden, inter, case["sparsity"], case["format"])], case["format"])
        s.x = _bf16(gen, k, hidden)
        s.y = torch.empty((k, hidden), dtype=torch.float32, device="cuda")
        s.ws_bytes = sd2.mlp_workspace_size(s.gate_up.m, s.down.m, k)
    elif kind == "gradient":
        s.mat = _Packed(_weight(gen, case["n_out"], case["k_in"], case["sparsity"], "bitmask"), "bitmask")
        s.grad = torch.empty((case["n_out"], case["k_in"]), dtype=torch.float32, device="cuda").normal_(generator=gen)
        s.grad = s.grad.to(getattr(torch, case["dtype"]))
        s.ws_bytes = 0
    else:
        s.model = _model(case, gen)
        s.h_out = torch.empty((k, case["hidden"]), dtype=torch.float32, device="cuda")
        if kind == "forward":
            s.h_in = _bf16(gen, k, case["hidden"])
            s.ws_bytes = sd2.drafter_workspace_size(s.model, k)
            if case["verify"]:
                vocab, batch = 128256, case["verify"]
                s.draft = torch.randint(0, vocab, (batch, k), generator=gen, device="cuda").to(torch.int32)
                s.target = _targets(gen, batch, k, vocab, torch.cat([s.draft, s.draft[:, :1]], dim=1))
                s.accepted = torch.empty(batch, dtype=torch.int32, device="cuda")
                s.tokens = torch.empty((batch, k + 1), dtype=torch.int32, device="cuda")
        else:
            s.k_cache, s.v_cache = _cache(gen, case), _cache(gen, case)
            if kind == "decode":
                s.h_in = _bf16(gen, k, case["hidden"])
                s.ws_bytes = sd2.drafter_decode_workspace_size(s.model, k)
            else:
                # embedding tied to the head, 3 z: the choice then has a clear margin, as a confident drafter's has (with
                # random rows of any size the largest of 100 000 logits would be a near-tie every few steps)
                s.emb = _bf16(gen, case["vocab"], case["hidden"]).mul_(3.0)
                s.start = torch.randint(0, case["vocab"], (1,), generator=gen, device="cuda").to(torch.int32)
                s.ids = torch.empty((1, k), dtype=torch.int32, device="cuda")
                s.target = _targets(gen, 1, k, case["vocab"], s.start)
                s.accepted = torch.empty(1, dtype=torch.int32, device="cuda")
                s.tokens = torch.empty((1, k + 1), dtype=torch.int32, device="cuda")
                s.ws_bytes = sd2.draft_round_cached_workspace_size(s.model, case["vocab"], k)
    s.ws = _buffer(s.ws_bytes)
    return s


# ------------------------------------------------------------------ one pass


def run(s):
    case, k, stream = s.case, s.case.get("k_tok", 0), s.stream
    kind = case["kind"]
    if kind == "linear":
        call = sd2.dense_linear if case["format"] == "dense" else sd2.sparse_linear
        call(s.mat.m, s.x.data_ptr(), k, s.y.data_ptr(), s.ws.data_ptr(), s.ws_bytes, stream)
        return s.y
    if kind == "mlp":
        sd2.sparse_mlp_forward(s.gate_up.m, s.down.m, s.x.data_ptr(), k, s.y.data_ptr(), s.ws.data_ptr(), s.ws_bytes, stream)
        return s.y
    if kind == "gradient":
        sd2.mask_gradient(s.mat.m, s.grad.data_ptr(), case["dtype"] == "bfloat16", stream)
        return s.grad
    if kind == "forward":
        sd2.sparse_drafter_forward(s.model, s.h_in.data_ptr(), k, s.h_out.data_ptr(), s.ws.data_ptr(), s.ws_bytes, stream)
        if not case["verify"]:
            return s.h_out
        sd2.greedy_verify(s.draft.data_ptr(), s.target.data_ptr(), case["verify"], k, 128256, s.accepted.data_ptr(), s.tokens.data_ptr(), stream)
        return {"h": s.h_out, "accepted": s.accepted, "tokens": s.tokens}
    if kind == "decode":
        sd2.sparse_drafter_decode(s.model, s.h_in.data_ptr(), k, case["pos0"], s.k_cache.data_ptr(), s.v_cache.data_ptr(), case["max_pos"],
                                  ROPE_THETA, s.h_out.data_ptr(), s.ws.data_ptr(), s.ws_bytes, stream)
        return {"h": s.h_out, "k_cache": s.k_cache, "v_cache": s.v_cache}
    sd2.draft_round_cached(s.model, s.emb.data_ptr(), case["vocab"], s.start.data_ptr(), k, case["pos0"], s.k_cache.data_ptr(),
                           s.v_cache.data_ptr(), case["max_pos"], ROPE_THETA, s.ids.data_ptr(), s.ws.data_ptr(), s.ws_bytes, stream)
    sd2.greedy_verify(s.ids.data_ptr(), s.target.data_ptr(), 1, k, case["vocab"], s.accepted.data_ptr(), s.tokens.data_ptr(), stream)
    return {"ids": s.ids, "accepted": s.accepted, "tokens": s.tokens, "k_cache": s.k_cache, "v_cache": s.v_cache}


# ------------------------------------------------------------------ what a pass cannot do without


def _matrix_work(n_out, k_in, case):
    """(bytes of the stored matrix, multiply-adds per token)"""
    if case["format"] == "dense":
        return 2 * n_out * k_in, n_out * k_in
    if case["format"] == "2:4":
        return 9 * n_out * k_in // 8, n_out * k_in // 2
    nnz = n_out * _keep(k_in, case["sparsity"])
    return 2 * nnz + n_out * k_in // 8, nnz


def work(case):
    kind, k = case["kind"], case.get("k_tok", 0)
    if kind == "linear":
        b, macs = _matrix_work(case["n_out"], case["k_in"], case)
        return {"bytes": b + 2 * k * case["k_in"] + 4 * k * case["n_out"], "flops": 2 * macs * k}
    if kind == "mlp":
        (b0, m0), (b1, m1) = _matrix_work(2 * case["inter"], case["hidden"], case), _matrix_work(case["hidden"], case["inter"], case)
        return {"bytes": b0 + b1 + 6 * k * case["hidden"], "flops": 2 * (m0 + m1) * k}
    if kind == "gradient":
        size = 4 if case["dtype"] == "float32" else 2
        n = case["n_out"] * case["k_in"]
        return {"bytes": 2 * size * n + n // 8, "flops": 0}
    per_layer = [_matrix_work(n, kk, case) for n, kk in _layer_shapes(case)]
    weights = case["layers"] * sum(b for b, _ in per_layer)
    macs = case["layers"] * sum(m for _, m in per_layer)
    if kind == "forward":
        verify = 4 * case["verify"] * (3 * k + 3)
        return {"bytes": weights + 6 * k * case["hidden"] + verify, "flops": 2 * macs * k}
    row = 4 * case["layers"] * case["n_kv"] * HEAD_DIM  # bytes of one position's keys and values in all layers
    scores = case["layers"] * case["n_heads"] * HEAD_DIM * 2  # multiply-adds per query token and position
    if kind == "decode":
        return {"bytes": weights + 6 * k * case["hidden"] + row * (case["pos0"] + k),
                "flops": 2 * (macs * k + scores * sum(case["pos0"] + t + 1 for t in range(k)))}
    head = 2 * case["vocab"] * case["hidden"]  # every step needs the step before it: each streams the weights and the head
    positions = sum(case["pos0"] + t + 1 for t in range(k))
    return {"bytes": k * (weights + head) + row * positions, "flops": 2 * (k * (macs + head // 2) + scores * positions)}


def tolerance(case):
    kind = case["kind"]
    if kind == "gradient":
        return "exact"
    if kind == "linear":
        return {"rel": 1e-5}  # exact products, sums in 32 bits
    if kind == "mlp":
        return {"rel": 2e-3}  # one rounding of the activations to bf16 between the two linears
    # A stack rounds its activations to bf16 at four points of every layer: values next to a rounding boundary go either way,
    # and that accumulates over the layers.  The tests hold 28 layers to the same bound.  The chosen ids are whole numbers.
    return {"rel": 2e-2, "differ": 0.0}
