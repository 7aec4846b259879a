"""The C-ABI library loads, exports every symbol the header declares, and rejects bad
arguments on the host before any launch (so these run without a GPU)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import paper_2504_08838_amd as sd2
import sd2_workload as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "sd2.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(sd2_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported():
    names = _declared()
    for must in ("sd2_pack_sparse", "sd2_sparse_linear", "sd2_sparse_drafter_forward", "sd2_greedy_verify",
                 "sd2_dense_linear", "sd2_sparse_mlp_forward"):
        assert must in names
    raw = C.CDLL(sd2.lib_path())
    for n in names:
        assert hasattr(raw, n), n
    assert sd2.version() >= 100


def test_binding_has_the_same_names():
    for n in _declared():
        assert hasattr(sd2, n[len("sd2_"):]), n


def _host_matrix():
    w = wl.gen_weight(12, 5, "q", 64, 512, 50)
    blob = sd2.pack_sparse(w, 1)
    return blob, sd2.matrix_init_sparse(blob, 0x1000)   # fake, aligned device address: never dereferenced here


def test_linear_argument_checks():
    blob, m = _host_matrix()
    assert m.info.n_slabs == 2
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    assert sd2.linear_workspace_size(m, 5) == 2 * 5 * 64 * 4
    assert L.sd2_sparse_linear(None, fake, 1, fake, fake, 1 << 20, None) == -1
    assert L.sd2_sparse_linear(C.byref(m), None, 1, fake, fake, 1 << 20, None) == -1
    assert L.sd2_sparse_linear(C.byref(m), fake, 0, fake, fake, 1 << 20, None) == -6
    assert L.sd2_sparse_linear(C.byref(m), fake, 65, fake, fake, 1 << 20, None) == -6
    assert L.sd2_sparse_linear(C.byref(m), C.c_void_p(0x2002), 1, fake, fake, 1 << 20, None) == -4
    assert L.sd2_sparse_linear(C.byref(m), fake, 5, fake, fake, 100, None) == -4      # workspace too small
    assert L.sd2_sparse_linear(C.byref(m), fake, 5, fake, None, 0, None) == -1        # split matrix needs one
    assert L.sd2_dense_linear(C.byref(m), fake, 1, fake, fake, 1 << 20, None) == -3   # wrong kind
    with pytest.raises(sd2.SD2Error) as e:
        sd2.matrix_init_sparse(blob, 0x1001)
    assert e.value.status == -4
    bad = blob.copy(); bad[0] = 0
    with pytest.raises(sd2.SD2Error) as e:
        sd2.matrix_init_sparse(bad, 0x1000)
    assert e.value.status == -5
    with pytest.raises(sd2.SD2Error) as e:
        sd2.matrix_init_dense(0x1000, 64, 100)
    assert e.value.status == -2


def test_model_argument_checks():
    shape = sd2.ModelShape(1, 256, 256, 128, 512, 2, 1, 128)
    dims = [(512, 256), (256, 256), (1024, 256), (256, 512)]
    mats = [sd2.matrix_init_dense(0x1000, n, k) for n, k in dims]
    model = sd2.model_create(shape, mats)
    assert sd2.drafter_workspace_size(model, 5) > 0
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    assert L.sd2_sparse_drafter_forward(model.handle, fake, 5, fake, fake, 16, None) == -4
    assert L.sd2_sparse_drafter_forward(model.handle, fake, 99, fake, fake, 1 << 30, None) == -6
    assert L.sd2_sparse_drafter_forward(None, fake, 5, fake, fake, 1 << 30, None) == -1
    model.close()
    with pytest.raises(sd2.SD2Error) as e:
        sd2.model_create(shape, mats[:3])
    assert e.value.status == -2
    with pytest.raises(sd2.SD2Error) as e:
        sd2.model_create(shape, [mats[1], mats[0], mats[2], mats[3]])
    assert e.value.status == -2
    with pytest.raises(sd2.SD2Error):
        sd2.model_create(sd2.ModelShape(1, 256, 256, 128, 512, 3, 1, 128), mats)


def test_verify_argument_checks():
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    assert L.sd2_greedy_verify(fake, fake, -1, 5, 100, fake, fake, None) == -2
    assert L.sd2_greedy_verify(fake, fake, 4, 5, 0, fake, fake, None) == -6
    assert L.sd2_greedy_verify(None, fake, 4, 5, 100, fake, fake, None) == -1
    assert L.sd2_greedy_verify(fake, fake, 0, 5, 100, fake, fake, None) == 0          # empty batch: nothing to do
    sd2.check_token_ids_host(np.array([0, 5, 99], dtype=np.int32), 100)
    with pytest.raises(sd2.SD2Error) as e:
        sd2.check_token_ids_host(np.array([0, 100], dtype=np.int32), 100)
    assert e.value.status == -6
    with pytest.raises(sd2.SD2Error):
        sd2.check_token_ids_host(np.array([-1], dtype=np.int32), 100)


def test_lm_head_argument_checks():
    """Every rejection happens on the host, before any launch."""
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    n = sd2.lm_head_workspace_size(128256, 3072, 5)
    assert n > 0 and n % 16 == 0
    args = lambda **kw: [kw.get("w", fake), kw.get("vocab", 1000), kw.get("hidden", 1024), kw.get("h", fake),
                         kw.get("k", 5), kw.get("ids", fake), None, None, kw.get("ws", fake), kw.get("wsb", n), None]
    assert L.sd2_lm_head_argmax(*args(w=None)) == -1
    assert L.sd2_lm_head_argmax(*args(h=None)) == -1
    assert L.sd2_lm_head_argmax(*args(ids=None)) == -1
    assert L.sd2_lm_head_argmax(*args(ws=None)) == -1
    assert L.sd2_lm_head_argmax(*args(vocab=0)) == -2
    assert L.sd2_lm_head_argmax(*args(hidden=1000)) == -2      # not a multiple of 128
    assert L.sd2_lm_head_argmax(*args(hidden=9216 + 128)) == -2
    assert L.sd2_lm_head_argmax(*args(k=0)) == -6
    assert L.sd2_lm_head_argmax(*args(k=65)) == -6
    assert L.sd2_lm_head_argmax(*args(wsb=n - 1)) == -4
    assert L.sd2_lm_head_argmax(*args(w=C.c_void_p(0x2008))) == -4  # misaligned
    with pytest.raises(sd2.SD2Error):
        sd2.lm_head_workspace_size(1000, 100, 5)


def test_format_3_descriptors():
    """A 2:4 blob gives a sparse descriptor; a width the 2:4 kernel cannot split over its wavefronts is refused."""
    import sd2_workload as wl
    w = wl.gen_weight(71, 0, "q", 32, 512, 50, pattern="2:4")
    blob = sd2.pack_sparse(w, 3)
    m = sd2.matrix_init_sparse(blob, 0x10000)
    assert m.info.format == 3 and m.info.n_slabs == 2 and m.info.total_bytes == 128 + 4608 * m.info.n_tiles
    assert sd2.linear_workspace_size(m, 5) == 0  # the 2:4 kernel writes final values: no split-K partials
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    wide = wl.gen_weight(71, 0, "q", 16, 9216 + 256, 50, pattern="2:4")  # 37 slabs
    mw = sd2.matrix_init_sparse(sd2.pack_sparse(wide, 3), 0x10000)
    assert L.sd2_sparse_linear(C.byref(mw), fake, 5, fake, None, 0, None) == -8


def test_mask_gradient_argument_checks():
    import sd2_workload as wl
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    m = sd2.matrix_init_sparse(sd2.pack_sparse(wl.gen_weight(72, 0, "q", 32, 256, 50), 1), 0x10000)
    assert L.sd2_mask_gradient(C.byref(m), None, 0, None) == -1
    assert L.sd2_mask_gradient(C.byref(m), C.c_void_p(0x2004), 0, None) == -4
    assert L.sd2_mask_gradient(C.byref(m), fake, 2, None) == -6
    assert L.sd2_mask_gradient(None, fake, 0, None) == -1
    m24 = sd2.matrix_init_sparse(sd2.pack_sparse(wl.gen_weight(72, 0, "q", 32, 256, 50, pattern="2:4"), 3), 0x10000)
    assert L.sd2_mask_gradient(C.byref(m24), fake, 0, None) == -8
    d = sd2.matrix_init_dense(0x10000, 32, 256)
    assert L.sd2_mask_gradient(C.byref(d), fake, 0, None) == -3


def test_prune_argument_checks():
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    assert L.sd2_prune_magnitude(None, 16, 256, 50, 0, None) == -1
    assert L.sd2_prune_magnitude(C.c_void_p(0x2002), 16, 256, 50, 0, None) == -4
    assert L.sd2_prune_magnitude(fake, 0, 256, 50, 0, None) == -2
    assert L.sd2_prune_magnitude(fake, 16, 100, 50, 0, None) == -2
    assert L.sd2_prune_magnitude(fake, 16, 256, 100, 0, None) == -6
    assert L.sd2_prune_magnitude(fake, 16, 256, 60, 1, None) == -6      # 2:4 is 50 %
    assert L.sd2_prune_magnitude(fake, 16, 320, 50, 0, None) == -8      # rows need k_in % 256 == 0
    assert L.sd2_prune_magnitude(fake, 16, 9216 + 256, 50, 0, None) == -8
    assert L.sd2_prune_magnitude(fake, 16, 256, 50, 7, None) == -3


def test_draft_round_argument_checks():
    import sd2_workload as wl
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    shape = sd2.ModelShape(1, 256, 256, 128, 512, 2, 1, 128)
    ws = {"qkv": (512, 256), "o": (256, 256), "gu": (1024, 256), "dn": (256, 512)}
    mats = [sd2.matrix_init_sparse(sd2.pack_sparse(wl.gen_weight(73, 0, "q", n, k, 50), 1), 0x10000) for n, k in ws.values()]
    model = sd2.model_create(shape, mats)
    n = sd2.draft_round_workspace_size(model, 1000, 5)
    assert n > 0 and n % 256 == 0
    args = lambda **kw: [kw.get("model", model.handle), kw.get("emb", fake), kw.get("vocab", 1000), kw.get("start", fake),
                         kw.get("k", 5), kw.get("ids", fake), kw.get("ws", fake), kw.get("wsb", n), None]
    assert L.sd2_draft_round(*args(emb=None)) == -1
    assert L.sd2_draft_round(*args(start=None)) == -1
    assert L.sd2_draft_round(*args(ids=None)) == -1
    assert L.sd2_draft_round(*args(ws=None)) == -1
    assert L.sd2_draft_round(*args(k=0)) == -6
    assert L.sd2_draft_round(*args(k=65)) == -6
    assert L.sd2_draft_round(*args(vocab=0)) == -2
    assert L.sd2_draft_round(*args(wsb=n - 1)) == -4
    assert L.sd2_draft_round(*args(model=None)) == -1
    sd2.model_destroy(model)


def test_decode_argument_checks():
    import sd2_workload as wl
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    shape = sd2.ModelShape(1, 256, 256, 128, 512, 2, 1, 128)
    ws = {"qkv": (512, 256), "o": (256, 256), "gu": (1024, 256), "dn": (256, 512)}
    mats = [sd2.matrix_init_sparse(sd2.pack_sparse(wl.gen_weight(73, 0, "q", n, k, 50), 1), 0x10000) for n, k in ws.values()]
    model = sd2.model_create(shape, mats)
    n = sd2.drafter_decode_workspace_size(model, 5)
    assert n > sd2.drafter_workspace_size(model, 5) * 0 and n % 256 == 0
    args = lambda **kw: [kw.get("model", model.handle), kw.get("h_in", fake), kw.get("k", 5), kw.get("pos0", 10),
                         kw.get("kc", fake), kw.get("vc", fake), kw.get("max_pos", 64), kw.get("theta", 5.0e5),
                         kw.get("h_out", fake), kw.get("ws", fake), kw.get("wsb", n), None]
    for name in ("model", "h_in", "kc", "vc", "h_out", "ws"):
        assert L.sd2_sparse_drafter_decode(*args(**{name: None})) == -1, name
    assert L.sd2_sparse_drafter_decode(*args(k=0)) == -6
    assert L.sd2_sparse_drafter_decode(*args(k=65)) == -6
    assert L.sd2_sparse_drafter_decode(*args(pos0=-1)) == -6
    assert L.sd2_sparse_drafter_decode(*args(pos0=60)) == -6        # 60 + 5 > 64
    assert L.sd2_sparse_drafter_decode(*args(max_pos=0)) == -6
    assert L.sd2_sparse_drafter_decode(*args(theta=1.0)) == -6
    assert L.sd2_sparse_drafter_decode(*args(theta=float("nan"))) == -6
    assert L.sd2_sparse_drafter_decode(*args(max_pos=1 << 20)) == -8  # scores of a head no longer fit in LDS
    assert L.sd2_sparse_drafter_decode(*args(wsb=n - 1)) == -4
    assert L.sd2_sparse_drafter_decode(*args(kc=C.c_void_p(0x2004))) == -4
    sd2.model_destroy(model)


def test_cached_round_argument_checks():
    import sd2_workload as wl
    L = sd2.lib()
    fake = C.c_void_p(0x2000)
    shape = sd2.ModelShape(1, 256, 256, 128, 512, 2, 1, 128)
    ws = {"qkv": (512, 256), "o": (256, 256), "gu": (1024, 256), "dn": (256, 512)}
    mats = [sd2.matrix_init_sparse(sd2.pack_sparse(wl.gen_weight(73, 0, "q", n, k, 50), 1), 0x10000) for n, k in ws.values()]
    model = sd2.model_create(shape, mats)
    n = sd2.draft_round_cached_workspace_size(model, 1000, 5)
    assert n > 0 and n % 256 == 0
    args = lambda **kw: [kw.get("model", model.handle), kw.get("emb", fake), kw.get("vocab", 1000), kw.get("start", fake),
                         kw.get("k", 5), kw.get("pos0", 10), kw.get("kc", fake), kw.get("vc", fake), kw.get("max_pos", 64),
                         kw.get("theta", 5.0e5), kw.get("ids", fake), kw.get("ws", fake), kw.get("wsb", n), None]
    for name in ("model", "emb", "start", "kc", "vc", "ids", "ws"):
        assert L.sd2_draft_round_cached(*args(**{name: None})) == -1, name
    assert L.sd2_draft_round_cached(*args(k=0)) == -6
    assert L.sd2_draft_round_cached(*args(k=65)) == -6
    assert L.sd2_draft_round_cached(*args(pos0=-1)) == -6
    assert L.sd2_draft_round_cached(*args(pos0=60)) == -6
    assert L.sd2_draft_round_cached(*args(theta=0.5)) == -6
    assert L.sd2_draft_round_cached(*args(vocab=0)) == -2
    assert L.sd2_draft_round_cached(*args(wsb=n - 1)) == -4
    sd2.model_destroy(model)


def test_improvement_factor_matches_eq3_and_the_oracle():
    from oracle import macs
    # Eq. 3 by hand: 4.16 tokens per round, 5 drafts, drafter step 5 % of a target step -> 4.16 / 1.25
    assert sd2.improvement_factor(4.16, 5, 0.05) == pytest.approx(3.328, rel=1e-12)
    assert sd2.improvement_factor(4.0, 5, 0.0) == 4.0
    for mal, k, c in [(1.0, 0, 0.3), (3.61, 5, 0.11), (6.0, 8, 1.0), (2.5, 3, 2.0)]:
        assert sd2.improvement_factor(mal, k, c) == pytest.approx(macs.improvement_factor(mal, k, c), rel=1e-15)
    L = sd2.lib()
    out = C.c_double(0.0)
    assert L.sd2_improvement_factor(4.0, 5, 0.1, None) == -1
    assert L.sd2_improvement_factor(-1.0, 5, 0.1, C.byref(out)) == -6
    assert L.sd2_improvement_factor(4.0, -1, 0.1, C.byref(out)) == -6
    assert L.sd2_improvement_factor(4.0, 5, float("nan"), C.byref(out)) == -6
    assert L.sd2_improvement_factor(float("inf"), 5, 0.1, C.byref(out)) == -6


def test_options_round_trip_and_ranges():
    L = sd2.lib()
    for which, good, bad in ((sd2.OPT_FORWARD_MULTI, 1, 2), (sd2.OPT_LINEAR_PARTIALS, 1, -1), (sd2.OPT_SPIN_LIMIT, 7, -2),
                             (sd2.OPT_MEGA_TIMING, 2, 3), (sd2.OPT_FIXED_BITS, 15, 30)):
        before = sd2.get_option(which)
        sd2.set_option(which, good)
        assert sd2.get_option(which) == good
        assert L.sd2_set_option(which, bad) == -6
        assert sd2.get_option(which) == good
        sd2.set_option(which, before)
    assert L.sd2_set_option(99, 0) == -6 and L.sd2_set_option(-1, 0) == -6
    assert L.sd2_get_option(0, None) == -1


def test_validate_rejects_mask_bits_outside_a_ragged_matrix():
    # 40 rows: the last strip has 8 rows outside the matrix; set a mask bit there and repair directory and checksum
    # by hand, so that only the out-of-range position is wrong
    t = 2                                             # strip 2, slab 0
    w = wl.gen_weight(12, 6, "q", 40, 256, 50).copy()
    w[39, np.flatnonzero(w[39])[0]] = 0               # one value fewer: the last tile's padding has room for one more
    blob = sd2.pack_sparse(w, 1).copy()
    info = sd2.blob_info(blob)
    assert info.n_strips == 3
    masks = blob[info.mask_off:info.mask_off + 512 * info.n_tiles].view(np.uint16).reshape(info.n_tiles, 64, 4)
    lane = 15                                         # row 47 of the matrix: outside
    assert masks[t, lane].sum() == 0
    sd2.blob_validate(blob)
    # the last run (q = 3, nibble 3) of the tile takes one more value: no run base changes, only the tile's count
    masks[t, lane, 3] |= 0x8000
    d = blob[128 + 48 * t:128 + 48 * (t + 1)].view(np.uint32)
    old_nnz = int(d[1])
    assert (old_nnz + 1 + 7) // 8 == (old_nnz + 7) // 8   # the extra value fits the tile's padding: offsets stay
    d[1] = old_nnz + 1
    hdr64 = blob[40:48].view(np.uint64)
    hdr64[0] += 1
    if old_nnz + 1 > info.max_tile_nnz:
        blob[32:36].view(np.uint32)[0] = old_nnz + 1
    words = blob[128:].view(np.uint32).astype(np.uint64)
    s1 = int(words.sum() & 0xFFFFFFFF)
    s2 = int((words * np.arange(1, words.size + 1, dtype=np.uint64)).sum() & 0xFFFFFFFF)
    blob[88:92].view(np.uint32)[0] = s1 ^ (((s2 << 16) | (s2 >> 16)) & 0xFFFFFFFF)
    with pytest.raises(sd2.SD2Error) as e:
        sd2.blob_validate(blob)
    assert e.value.status == -5


def test_model_create_rejects_head_sizes_the_attention_kernels_cannot_split():
    L = sd2.lib()
    _, m = _host_matrix()
    handle = C.c_void_p()
    bad = sd2.ModelShape(0, 1600, 1600, 400, 64, 16, 4, 100)   # head_dim 100: not a multiple of 8
    assert L.sd2_model_create(C.byref(bad), None, 0, C.byref(handle)) == -2
    ok = sd2.ModelShape(0, 1664, 1664, 416, 64, 16, 4, 104)
    assert L.sd2_model_create(C.byref(ok), None, 0, C.byref(handle)) == 0
    L.sd2_model_destroy(handle)


def _fake_stack(shape, fmt):
    """A one-layer model of blobs at fake addresses: sizes only, nothing is launched."""
    mats, keep = [], []
    for n, k in ((shape.q_out + 2 * shape.kv_out, shape.hidden), (shape.hidden, shape.q_out), (2 * shape.inter, shape.hidden), (shape.hidden, shape.inter)):
        if fmt == "dense":
            mats.append(sd2.matrix_init_dense(0x1000, n, k))
            continue
        w = np.full((n, k), 0x3F80, dtype=np.uint16)
        w[:, 1::2] = 0
        keep.append(sd2.pack_sparse(w, 3 if fmt == "2:4" else 1))
        mats.append(sd2.matrix_init_sparse(keep[-1], 0x1000))
    return sd2.model_create(sd2.ModelShape(shape.layers, shape.hidden, shape.q_out, shape.kv_out, shape.inter, shape.n_heads, shape.n_kv, 128),
                            mats, keep=keep)


@pytest.mark.parametrize("heads,n_kv,inter,fmt", [(20, 4, 6912, "dense"), (13, 13, 4800, "dense"), (13, 13, 4800, "2:4"), (13, 13, 4800, "bitmask"),
                                                  (4, 1, 2048, "dense"), (4, 1, 2048, "2:4"), (4, 1, 2048, "bitmask")])
def test_a_workspace_serves_every_smaller_call(heads, n_kv, inter, fmt, sd2_options):
    """More than 8 tokens are always one launch per step; how a linear is cut there depends on the token count, the room for
    its partial results must not.  Neither may the switches change what a workspace holds."""
    from types import SimpleNamespace
    shape = SimpleNamespace(layers=1, hidden=128 * heads, q_out=128 * heads, kv_out=128 * n_kv, inter=inter, n_heads=heads, n_kv=n_kv)
    model = _fake_stack(shape, fmt)
    for size in (sd2.drafter_workspace_size, sd2.drafter_decode_workspace_size):
        sizes = [size(model, t) for t in range(9, 65)]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), sizes
        for value in (1, 2):
            sd2_options.set("linear_partials", value)
            assert [size(model, t) for t in range(9, 65)] == sizes
            sd2_options.reset()


def test_greedy_verify_host_against_the_hand_cases_and_the_range_rule(golden_dir):
    path = os.path.join(golden_dir, "verify_hand_cases.txt")
    for line in open(path):
        if line.startswith("#") or not line.strip():
            continue
        d, t, n, out = [np.array(f.split(), dtype=np.int32) for f in line.split("|")]
        acc, toks = sd2.greedy_verify_host(d.reshape(1, -1), t.reshape(1, -1), vocab=100)
        assert acc.tolist() == n.tolist() and toks[0].tolist() == out.tolist()
    draft, target = wl.gen_verify(5, 64, 5, 128256, 0.85)
    acc, toks = sd2.greedy_verify_host(draft, target, 128256)
    from oracle import verify as ov
    ref_acc, ref_toks = ov.greedy_verify(draft, target, vocab=128256)
    assert np.array_equal(acc, ref_acc) and np.array_equal(toks, ref_toks)
    bad = target.copy()
    bad[3, 2] = 128256
    with pytest.raises(sd2.SD2Error) as e:
        sd2.greedy_verify_host(draft, bad, 128256)
    assert e.value.status == -6
