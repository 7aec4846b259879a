"""The kernel for 17 to 64 tokens at the edges of its tiling -- ragged rows and columns, one strip, odd unit counts, halves of
tiles denser than its staging, every token group -- on all three formats, and the attention kernels behind it."""
from types import SimpleNamespace

import numpy as np
import pytest

import sd2_workload as wl
from oracle import decode as od
from oracle import linear as ol
from oracle import stack as os_

pytestmark = pytest.mark.gpu


def _ints(a):
    return wl.f32_to_bf16_bits(np.asarray(a, dtype=np.float32))


def _matrix(rng, n, k, fmt):
    w = rng.integers(-8, 9, size=(n, k))
    if fmt == "2:4":
        drop = rng.permuted(np.broadcast_to(np.array([True, True, False, False]), (n, k // 4, 4)), axis=2)
        w[drop.reshape(n, k)] = 0
    elif fmt == "bitmask":
        w[rng.random((n, k)) < 0.5] = 0
    elif fmt == "crowded":  # every tile's values in one half of it, far more than the staged part holds
        w[:, (np.arange(k) // 128) % 2 == (1 if n % 2 else 0)] = 0
    return w


@pytest.mark.parametrize("fmt", ["bitmask", "crowded", "2:4", "dense"])
@pytest.mark.parametrize("n,k,k_tok", [
    (16, 64, 17),       # one strip, half a unit
    (33, 192, 64),      # ragged rows, one unit and a half
    (333, 320, 33),     # n_out not a multiple of 4: scalar stores
    (4112, 1536, 32),   # more strips than one group per workgroup, ragged last block
    (96, 8960, 49),     # a long contraction: split over workgroups or passes
    (5003, 832, 49),    # ragged rows, six units and a half, too many strips for passes of 16 or 32 tokens
    (5008, 768, 33),    # bitmask: 2817 tiles in passes of 16 tokens
    (2048, 512, 33),    # passes of 16 tokens, the last of one
    (2041, 1600, 64),   # two passes of 32 tokens, one slab per wavefront (bitmask), ragged rows
    (2500, 3392, 17),   # one pass of 32 tokens, two slabs per wavefront (bitmask)
    (2500, 2048, 49),   # bitmask: all 64 and all 48 tokens in one pass
    (4096, 1024, 64),
    (2500, 3008, 40),
    (3300, 960, 48),
    (8192, 64, 31),     # one short tile per strip; a dense matrix of one slab
    (8000, 192, 24),
    (1536, 512, 49),    # dense: passes of 32 tokens, one to four column chunks per wavefront
    (2040, 2048, 64),
    (1600, 3072, 40),
    (2560, 4096, 17),
    (600, 10240, 33),   # dense: more columns than the streaming kernel takes
])
def test_wide_linear_exact_integers(n, k, k_tok, fmt):
    import gpu_util as gu
    rng = np.random.default_rng([5, n, k, k_tok])
    w = _matrix(rng, n, k, fmt)
    x = rng.integers(-4, 5, size=(k_tok, k))
    if fmt == "2:4" and k > 9216:
        pytest.skip("more columns than a 2:4 matrix may have")
    mat = gu.DenseMat(_ints(w)) if fmt == "dense" else gu.SparseMat(_ints(w), 3 if fmt == "2:4" else 1)
    y = gu.run_linear(mat, _ints(x), sparse=fmt != "dense")
    assert np.array_equal(y, x.astype(np.float64) @ w.T.astype(np.float64))  # sums below 2^24: exact in fp32 in any order


@pytest.mark.parametrize("fmt", ["bitmask", "2:4", "dense"])
@pytest.mark.parametrize("n,k,k_tok", [
    (16640, 64, 64),    # four groups of two wavefronts over the strips
    (32960, 320, 50),   # the same, three units: two passes
    (8208, 576, 17),    # twelve wavefronts in two groups
    (24800, 576, 33),   # the same with two strip groups per workgroup, one after the other
    (32960, 832, 64),   # eight wavefronts along the contraction, three strip groups
])
def test_wide_linear_many_strips_exact_integers(n, k, k_tok, fmt):
    """Short contractions of many strips: wavefronts share out the strips, and a workgroup takes several groups of them."""
    import gpu_util as gu
    rng = np.random.default_rng([7, n, k, k_tok])
    w = _matrix(rng, n, k, fmt)
    x = rng.integers(-4, 5, size=(k_tok, k))
    mat = gu.DenseMat(_ints(w)) if fmt == "dense" else gu.SparseMat(_ints(w), 3 if fmt == "2:4" else 1)
    y = gu.run_linear(mat, _ints(x), sparse=fmt != "dense")
    assert np.array_equal(y, x.astype(np.float32) @ w.T.astype(np.float32))  # sums below 2^24: exact in any order


@pytest.mark.parametrize("fmt", ["bitmask", "2:4", "dense"])
@pytest.mark.parametrize("hidden,inter,k_tok", [(192, 48, 17), (512, 1200, 64),
                                                (512, 2048, 33),   # bitmask gate|up in passes of 16 tokens, 256 workgroups and
                                                (1216, 2048, 64),  # in passes of 32, one slab per wavefront
                                                (448, 4096, 40),   # the same, short tiles
                                                (1344, 4160, 20),  # one pass of 32, six slabs
                                                (576, 12416, 40),  # gate|up: two groups of six wavefronts, two strip groups
                                                (320, 16512, 64)])  # gate|up: four groups of two wavefronts, two passes
def test_wide_mlp_gated(hidden, inter, k_tok, fmt):
    import torch
    import paper_2504_08838_amd as sd2
    import gpu_util as gu
    if fmt == "2:4" and inter > 9216:
        pytest.skip("the down matrix has more columns than a 2:4 matrix may have")
    pattern = dict(pattern="2:4") if fmt == "2:4" else {}
    inter = (inter + 63) // 64 * 64
    wg, wu, wd = (wl.gen_weight(2, 1, p, n, k, 50, **pattern) for p, n, k in (("gate", inter, hidden), ("up", inter, hidden), ("down", hidden, inter)))
    x_bits = wl.gen_x(2, 1, "gate", k_tok, hidden)
    ref, _ = os_.mlp_block(wg, wu, wd, x_bits)
    mk = gu.DenseMat if fmt == "dense" else (lambda w: gu.SparseMat(w, 3 if fmt == "2:4" else 1))
    g_u, dn = mk(np.concatenate([wg, wu], axis=0)), mk(wd)
    x = gu.dev(x_bits)
    y = torch.full((k_tok, hidden), float("nan"), dtype=torch.float32, device="cuda")
    nb = sd2.mlp_workspace_size(g_u.m, dn.m, k_tok)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    sd2.sparse_mlp_forward(g_u.m, dn.m, x.data_ptr(), k_tok, y.data_ptr(), ws.data_ptr(), nb, gu.stream_ptr())
    torch.cuda.synchronize()
    assert ol.rel_l2(y.cpu().numpy(), ref) <= 2e-3


SHAPE = SimpleNamespace(layers=2, hidden=768, q_out=768, kv_out=128, inter=640, n_heads=6, n_kv=1, head_dim=128)


@pytest.mark.parametrize("k_tok", [9, 16, 17, 33, 64])
def test_wide_inflight_attention(k_tok):
    import gpu_util as gu
    from test_gpu_decode import _model
    get, model = _model(SHAPE, 41)
    h = wl.gen_x(41, 0, "q", k_tok, SHAPE.hidden)
    assert ol.rel_l2(gu.run_forward(model, h, SHAPE.hidden), os_.drafter_forward(SHAPE, get, h)) <= 1e-3


@pytest.mark.parametrize("hidden", [64, 1088, 4096, 4160, 8256])
@pytest.mark.parametrize("k_tok", [5, 20])
def test_residual_norm_widths(hidden, k_tok, sd2_options):
    """Less than a wavefront's columns, a ragged last wavefront, one to four pieces per thread; one and several partial results."""
    import gpu_util as gu
    from test_gpu_decode import _model
    sd2_options.set("forward_multi", 1)
    shape = SimpleNamespace(layers=1, hidden=hidden, q_out=256, kv_out=128, inter=1024, n_heads=2, n_kv=1, head_dim=128)
    get, model = _model(shape, 47)
    h = wl.gen_x(47, 0, "q", k_tok, hidden)
    assert ol.rel_l2(gu.run_forward(model, h, hidden), os_.drafter_forward(shape, get, h)) <= 1e-3


@pytest.mark.parametrize("k_tok,pos0", [(1, 0), (3, 31), (17, 255), (33, 256), (64, 1000)])
def test_wide_cached_attention(k_tok, pos0, sd2_options):
    """Histories around the tiles of 32 positions and the 256 of a workgroup's pass, six query heads per key/value head."""
    import gpu_util as gu
    from test_gpu_decode import _cache_close, _decode, _model, THETA
    sd2_options.set("forward_multi", 1)
    get, model = _model(SHAPE, 43)
    max_pos = pos0 + k_tok + 5
    rng = np.random.default_rng([43, k_tok, pos0])
    kc, vc = (wl.f32_to_bf16_bits(rng.standard_normal((SHAPE.layers, SHAPE.n_kv, max_pos, 128)).astype(np.float32)) for _ in range(2))
    h = wl.gen_x(43, 0, "q", k_tok, SHAPE.hidden)
    kd, vd = gu.dev(kc), gu.dev(vc)
    out = _decode(model, SHAPE, h, kd, vd, max_pos, pos0)
    ref_k, ref_v = kc.copy(), vc.copy()
    ref = od.drafter_decode(SHAPE, get, h, ref_k, ref_v, pos0, THETA)
    assert ol.rel_l2(out, ref) <= 1e-3
    # the first layer's rows: the second's inputs already differ by bf16 roundings that went the other way
    _cache_close(kd.cpu().numpy().view(np.uint16)[:1], ref_k[:1])
    _cache_close(vd.cpu().numpy().view(np.uint16)[:1], ref_v[:1])


@pytest.mark.parametrize("k_tok,bad", [(12, 10), (40, 37), (64, 0)])
@pytest.mark.parametrize("pos0", [None, 0, 40])
def test_a_token_that_is_not_finite_leaves_the_earlier_ones_alone(k_tok, bad, pos0, sd2_options):
    """Causal attention: tokens before the bad one come out as without it, the bad one and those after it are not finite."""
    import gpu_util as gu
    from test_gpu_decode import _decode, _model
    sd2_options.set("forward_multi", 1)
    get, model = _model(SHAPE, 53)
    h = wl.gen_x(53, 0, "q", k_tok, SHAPE.hidden)
    h_bad = h.copy()
    h_bad[bad] = 0x7FC0  # NaN
    max_pos = (pos0 or 0) + k_tok

    def forward(x):
        if pos0 is None:
            return gu.run_forward(model, x, SHAPE.hidden)
        rng = np.random.default_rng([53, pos0])
        cache = [gu.dev(wl.f32_to_bf16_bits(rng.standard_normal((SHAPE.layers, SHAPE.n_kv, max_pos, 128)).astype(np.float32))) for _ in range(2)]
        return _decode(model, SHAPE, x, *cache, max_pos, pos0)

    got, clean = forward(h_bad), forward(h)
    assert not np.isfinite(got[bad:]).any()
    if bad:
        assert ol.rel_l2(got[:bad], clean[:bad]) <= 1e-3


@pytest.mark.parametrize("k_tok,pos0", [(5, 40), (33, 300)])
def test_infinite_key_follows_the_sign_of_its_score(k_tok, pos0, sd2_options):
    """Minus infinity times a positive query component is a weight of zero: that head's row stays finite.  Plus infinity is NaN.
    The first head meets the infinite key.  The oracle takes the largest number in its place, and a token is finite where the
    value at that position does not count."""
    import gpu_util as gu
    from test_gpu_decode import _decode, _model, THETA
    sd2_options.set("forward_multi", 1)
    shape = SimpleNamespace(layers=1, hidden=512, q_out=512, kv_out=512, inter=1024, n_heads=4, n_kv=4, head_dim=128)
    get, model = _model(shape, 61)
    max_pos = pos0 + k_tok
    rng = np.random.default_rng([61, k_tok])
    kc, vc = (wl.f32_to_bf16_bits(rng.standard_normal((1, 4, max_pos, 128)).astype(np.float32)) for _ in range(2))
    h = wl.gen_x(61, 0, "q", k_tok, shape.hidden)
    kc[0, 0, 7, 70] = 0xFF7F
    ref = od.drafter_decode(shape, get, h, kc.copy(), vc.copy(), pos0, THETA)
    other = vc.copy()
    other[0, 0, 7] = 0x4480  # 1024
    finite = (od.drafter_decode(shape, get, h, kc.copy(), other, pos0, THETA) == ref).all(axis=1)
    assert finite.any() and not finite.all()
    kc[0, 0, 7, 70] = 0xFF80  # -inf
    got = _decode(model, shape, h, gu.dev(kc), gu.dev(vc), max_pos, pos0)
    assert np.array_equal(np.isfinite(got).all(axis=1), finite)
    assert ol.rel_l2(got[finite], ref[finite]) <= 1e-3


@pytest.mark.parametrize("fmt", ["bitmask", "dense"])
@pytest.mark.parametrize("k", [320, 384, 1152])
@pytest.mark.parametrize("k_tok", [5, 17, 64])
def test_infinite_weight_stays_in_its_row(k_tok, k, fmt):
    """The infinity sits in the first column of the last 64 or 128, where a kernel that reads absent columns as existing ones
    would multiply it with zero: a half unit, wavefronts without a column chunk, a second chunk that one wavefront has."""
    import gpu_util as gu
    rng = np.random.default_rng([59, k_tok])
    w = rng.integers(1, 9, size=(40, k)).astype(np.float32)
    w[7, k - (64 if k == 320 else 128)] = np.inf
    x = rng.integers(1, 5, size=(k_tok, k)).astype(np.float32)
    mat = gu.DenseMat(_ints(w)) if fmt == "dense" else gu.SparseMat(_ints(w), 1)
    assert np.array_equal(gu.run_linear(mat, _ints(x), sparse=fmt != "dense"), x @ w.T)
