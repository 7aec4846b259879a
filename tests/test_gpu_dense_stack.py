"""Dense stacks up to 16 tokens: the norm, the gated product and the residual inside the linears, where each can go wrong -- one to four
column chunks a wavefront and wavefronts without one, longer rows than the norm takes, ragged strips, the last token of a pass,
and layers that mix dense and packed matrices, so that some of the glue stays a launch of its own."""
from types import SimpleNamespace

import numpy as np
import pytest

import sd2_workload as wl
from oracle import decode as od
from oracle import linear as ol
from oracle import stack as os_

pytestmark = pytest.mark.gpu
# Whole-stack bar of tests/test_gpu_stack.py.  Two layers round their activations to bf16 eight times; a value next to a boundary moves by
# one spacing, 2^-8 at most: with one in twenty of them 2^-8 sqrt(8 / 20) = 2.5e-3, and the next linear may amplify that.
TOL = 5e-3


def _shape(hidden, heads, kv, inter, layers=2):
    return SimpleNamespace(layers=layers, hidden=hidden, q_out=128 * heads, kv_out=128 * kv, inter=inter, n_heads=heads, n_kv=kv, head_dim=128)


def _model(shape, seed, dense=(True, True, True, True), make=None):
    import gpu_util as gu
    import paper_2504_08838_amd as sd2
    table = {p: (n, k) for p, n, k in wl.layer_matrix_shapes(shape)}
    cache = {}

    def get(layer, proj):
        if (layer, proj) not in cache:
            cache[(layer, proj)] = make(proj, *table[proj]) if make else wl.gen_weight(seed, layer, proj, *table[proj], 50)
        return cache[(layer, proj)]

    mats = []
    for l in range(shape.layers):
        for parts, is_dense in zip(("qkv", ("o",), ("gate", "up"), ("down",)), dense):
            w = np.concatenate([get(l, p) for p in parts], axis=0)
            mats.append(gu.DenseMat(w) if is_dense else gu.SparseMat(w, 1))
    ms = sd2.ModelShape(shape.layers, shape.hidden, shape.q_out, shape.kv_out, shape.inter, shape.n_heads, shape.n_kv, shape.head_dim)
    return get, sd2.model_create(ms, [m.m for m in mats], keep=mats)


@pytest.mark.parametrize("shape", [
    _shape(128, 2, 1, 128),     # one chunk: seven wavefronts have none
    _shape(1536, 3, 1, 1088),   # two chunks, half of the wavefronts one; down has 64 columns too many for the stream
    _shape(2304, 2, 2, 8960),   # three chunks, a ragged third; nine in down
    _shape(4096, 2, 1, 640),    # four chunks; 256 strips
    _shape(4224, 2, 1, 4224),   # longer than the norm takes; 33 chunks
], ids=lambda s: str(s.hidden))
@pytest.mark.parametrize("k_tok", [1, 5, 16, 17])
def test_dense_forward(shape, k_tok):
    import gpu_util as gu
    get, model = _model(shape, 71)
    h = wl.gen_x(71, 0, "q", k_tok, shape.hidden)
    out = gu.run_forward(model, h, shape.hidden)
    assert ol.rel_l2(out, os_.drafter_forward(shape, get, h)) <= TOL
    assert np.array_equal(gu.run_forward(model, h, shape.hidden), out)


@pytest.mark.parametrize("shape", [
    _shape(128, 2, 1, 128),
    _shape(1536, 3, 1, 1088),
    _shape(2304, 2, 2, 1152),   # an odd number of column chunks in the norm
    _shape(3072, 2, 1, 640),
    _shape(4096, 2, 1, 640),
    _shape(4224, 2, 1, 1280),
], ids=lambda s: str(s.hidden))
@pytest.mark.parametrize("k_tok", [1, 5, 16])
def test_glue_inside_the_linears_changes_no_bit(shape, k_tok):
    """A traced forward keeps every step a launch of its own: the norm, the gated product and the residual inside the linears add the
    same numbers in the same order."""
    import gpu_util as gu
    get, model = _model(shape, 77)
    for i in range(6):  # a sum of squares that is off by its last bit changes few activations
        h = wl.gen_x(77 + i, 0, "q", k_tok, shape.hidden)
        apart, _, _ = gu.run_forward_trace(model, h, shape)
        assert np.array_equal(gu.run_forward(model, h, shape.hidden), apart)


@pytest.mark.parametrize("shape", [_shape(h, 3, 1, i, layers=1) for h, i in ((128, 128), (1536, 1280), (2304, 640), (4096, 8960), (4224, 384))],
                         ids=lambda s: str(s.hidden))
@pytest.mark.parametrize("k_tok", [1, 5, 16])
@pytest.mark.parametrize("half", ["attention", "mlp"])
def test_one_layer_exact_integers(shape, k_tok, half):
    """Every value between the launches is a whole number that its type holds: the norm's result (the residual's mean square is a power of
    four), the values of the heads (the same for every token, so their average too), silu(32 m) = 32 m for m >= 0 (no gate is negative)."""
    import gpu_util as gu
    rng = np.random.default_rng([89, shape.hidden, k_tok])
    hidden, shared = shape.hidden, shape.hidden // 2  # columns that all tokens share, up to their scale
    few = min(1.0, 48 / hidden)

    a = np.repeat([2, 1, 0], [hidden // 8, hidden // 2, hidden - hidden // 8 - hidden // 2])  # mean square 1
    common = rng.permutation(a)
    a = np.concatenate([np.broadcast_to(common[:shared], (k_tok, shared)), rng.permuted(np.broadcast_to(common[shared:], (k_tok, hidden - shared)), axis=1)],
                       axis=1)
    a = a * np.where(np.arange(hidden) < shared, rng.integers(0, 2, hidden) * 2 - 1, rng.integers(0, 2, (k_tok, hidden)) * 2 - 1)

    def make(proj, n, k):
        w = rng.integers(-2, 3, size=(n, k)) * (rng.random((n, k)) < few)
        if proj in ("v", "gate"):
            w[:, shared:] = 0
        if proj == "gate":
            w = 32 * abs(w) * np.sign(a[0])
        if proj in (("down", "q") if half == "attention" else ("v", "q")):
            w[:] = 0
        weights[proj] = w
        return _bits(w.astype(np.float32))

    weights = {}
    _, model = _model(shape, 0, make=make)
    h = a * (4.0 * 2.0 ** (np.arange(k_tok) % 3))[:, None]
    if half == "attention":
        ctx = a @ weights["v"].T
        assert abs(ctx).max() <= 256
        ref = h + np.tile(ctx.reshape(k_tok, 1, 128), (1, 3, 1)).reshape(k_tok, -1) @ weights["o"].T
    else:
        gated = ((a @ weights["gate"].T) * (a @ weights["up"].T)).astype(np.float32)
        gated = (wl.f32_to_bf16_bits(gated).astype(np.uint32) << 16).view(np.float32).astype(np.float64)
        ref = h + gated @ weights["down"].T
    assert abs(ref).max() < 2 ** 24
    assert np.array_equal(gu.run_forward(model, _bits(h.astype(np.float32)), hidden), ref)


@pytest.mark.parametrize("dense", [(True, False, False, False), (False, True, False, False), (False, False, True, False),
                                   (False, False, False, True), (True, False, True, True)])
@pytest.mark.parametrize("k_tok", [5, 17])
def test_mixed_layers(dense, k_tok):
    import gpu_util as gu
    shape = _shape(768, 2, 1, 640)
    get, model = _model(shape, 73, dense)
    h = wl.gen_x(73, 0, "q", k_tok, shape.hidden)
    assert ol.rel_l2(gu.run_forward(model, h, shape.hidden), os_.drafter_forward(shape, get, h)) <= TOL


@pytest.mark.parametrize("k_tok", [1, 13])
def test_dense_decode(k_tok):
    import gpu_util as gu
    from test_gpu_decode import _decode, THETA
    shape, pos0 = _shape(1152, 4, 2, 1216), 37
    get, model = _model(shape, 79)
    rng = np.random.default_rng([79, k_tok])
    kc, vc = (wl.f32_to_bf16_bits(rng.standard_normal((2, 2, 64, 128)).astype(np.float32)) for _ in range(2))
    h = wl.gen_x(79, 0, "q", k_tok, shape.hidden)
    out = _decode(model, shape, h, gu.dev(kc), gu.dev(vc), 64, pos0)
    assert ol.rel_l2(out, od.drafter_decode(shape, get, h, kc.copy(), vc.copy(), pos0, THETA)) <= TOL


@pytest.mark.parametrize("hidden,inter", [(128, 64), (1536, 8960), (4224, 1088)])
@pytest.mark.parametrize("k_tok", [1, 7, 16])
def test_dense_mlp(hidden, inter, k_tok):
    import torch
    import gpu_util as gu
    import paper_2504_08838_amd as sd2
    wg, wu, wd = (wl.gen_weight(2, 1, p, n, k, 50) for p, n, k in (("gate", inter, hidden), ("up", inter, hidden), ("down", hidden, inter)))
    x_bits = wl.gen_x(2, 1, "gate", k_tok, hidden)
    ref, _ = os_.mlp_block(wg, wu, wd, x_bits)
    g_u, dn, x = gu.DenseMat(np.concatenate([wg, wu], axis=0)), gu.DenseMat(wd), gu.dev(x_bits)
    y = torch.full((k_tok, hidden), float("nan"), dtype=torch.float32, device="cuda")
    nb = sd2.mlp_workspace_size(g_u.m, dn.m, k_tok)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    sd2.sparse_mlp_forward(g_u.m, dn.m, x.data_ptr(), k_tok, y.data_ptr(), ws.data_ptr(), nb, gu.stream_ptr())
    torch.cuda.synchronize()
    assert ol.rel_l2(y.cpu().numpy(), ref) <= 2e-3  # as the bitmask blocks: one rounding to bf16 between the linears


@pytest.mark.parametrize("k", [4224, 5248, 6272])
def test_infinite_weight_with_five_and_seven_chunks(k):
    """33, 41 and 49 column chunks on eight wavefronts: some have one or two chunks fewer than the kernel is built for."""
    import gpu_util as gu
    w = np.random.default_rng([83, k]).integers(1, 9, size=(40, k)).astype(np.float32)
    w[7, k - 128] = np.inf
    x = np.random.default_rng([84, k]).integers(1, 5, size=(5, k)).astype(np.float32)
    assert np.array_equal(gu.run_linear(gu.DenseMat(_bits(w)), _bits(x), sparse=False), x @ w.T)


@pytest.mark.parametrize("n_out", [7, 1000, 2041, 2048, 2049])
@pytest.mark.parametrize("k", [2048, 2176, 9216])
@pytest.mark.parametrize("k_tok", [1, 16, 17])
def test_strips_of_eight_rows(n_out, k, k_tok):
    """Whole numbers on either side of where strips have eight rows: rows, columns and tokens, and last strips that are not whole."""
    import gpu_util as gu
    rng = np.random.default_rng([101, n_out, k, k_tok])
    w, x = (rng.integers(-4, 5, size=(n, k)).astype(np.float32) for n in (n_out, k_tok))
    assert np.array_equal(gu.run_linear(gu.DenseMat(_bits(w)), _bits(x), sparse=False), x @ w.T)


def _bits(a):
    return wl.f32_to_bf16_bits(a)


def _attends_as_apart(hidden, heads, kv, k_tok):
    import gpu_util as gu
    shape = _shape(hidden, heads, kv, 128, layers=1)
    get, model = _model(shape, 97)
    h = wl.gen_x(97, 0, "q", k_tok, shape.hidden)
    out = gu.run_forward(model, h, shape.hidden)
    assert ol.rel_l2(out, os_.drafter_forward(shape, get, h)) <= TOL
    apart, _, _ = gu.run_forward_trace(model, h, shape)
    assert np.array_equal(out, apart)


@pytest.mark.parametrize("heads,kv", [(1, 1), (8, 2), (9, 3), (16, 4), (17, 17), (25, 5), (32, 4), (33, 11)])
@pytest.mark.parametrize("k_tok", [1, 2, 3, 5, 6, 8, 9])
def test_attention_inside_the_output_projection(heads, kv, k_tok):
    """One to four heads a wavefront and wavefronts without one, every count of token slots, heads and tokens on either side of where the
    linear attends by itself: the traced forward's attention is a launch of its own and gives the same bits."""
    _attends_as_apart(256, heads, kv, k_tok)


@pytest.mark.parametrize("hidden,heads,kv", [(2112, 8, 8), (2112, 9, 3), (3072, 16, 4), (3072, 24, 8), (4096, 32, 8)])
@pytest.mark.parametrize("k_tok", [1, 2, 3, 5])
def test_attention_inside_strips_of_sixteen_rows(hidden, heads, kv, k_tok):
    """The same on more than 2048 rows, whose strips have sixteen rows: one to four heads a wavefront on two slots, one and two on five."""
    _attends_as_apart(hidden, heads, kv, k_tok)


@pytest.mark.parametrize("heads,kv,hidden", [(2, 1, 256), (9, 3, 1152), (24, 8, 3072), (33, 11, 4224)])
@pytest.mark.parametrize("k_tok", [1, 2, 3, 5, 8])
def test_attention_over_the_whole_range_of_values(heads, kv, hidden, k_tok):
    """Values of 2^127 at every token average to 2^127, and token 0's weight of exp(-89.8), which has no normal fp32 number, still brings
    its 2^127 in front of the other tokens' zeros: in the linear that attends and in a launch of its own.  Every entry of h is 1 but
    column 0, which is -1 at token 0, and the norm's result is h."""
    import gpu_util as gu
    shape = _shape(hidden, heads, kv, 128, layers=1)
    w = {p: np.zeros((n, k), dtype=np.float32) for p, n, k in wl.layer_matrix_shapes(shape)}
    w["q"][::128, 1] = 1.0
    w["k"][::128, 0] = 508.0                                             # scores +-508 / sqrt(128): 89.8 apart
    w["v"][1::128, 2] = 2.0 ** 127                                       # dimension 1: the same at every token
    w["v"][2::128, 1], w["v"][2::128, 0] = 2.0 ** 126, -(2.0 ** 126)     # dimension 2: 2^127 at token 0, else 0
    w["o"][3, 1], w["o"][4, 128 * heads - 126] = 2.0 ** -120, 1.0        # the first head's dimension 1, the last one's dimension 2
    w["o"][5, 2] = 2.0 ** -120
    _, model = _model(shape, 0, make=lambda proj, n, k: _bits(w[proj]))
    h = np.ones((k_tok, hidden))
    h[0, 0] = -1.0
    ref = h.copy()
    far = np.array([2.0 ** 127] + [np.exp(-2 * 508 / np.sqrt(128.0)) * 2.0 ** 127 / t for t in range(1, k_tok)])  # 0.17 / t
    ref[:, 3] += 128.0
    ref[:, 4] += far
    ref[:, 5] += far * 2.0 ** -120
    out = gu.run_forward(model, _bits(h.astype(np.float32)), hidden)
    assert (abs(out - ref) <= 2.0 ** -8 * abs(ref - h) + 2.0 ** -22 * abs(ref)).all()  # the context's rounding to bf16
