"""Masked-gradient step of sparse fine-tuning (Sec. 2.4) on the GPU against the oracle: bit-exact."""
import numpy as np
import pytest

import sd2_workload as wl
from oracle import finetune as oft
from oracle import linear as ol

pytestmark = pytest.mark.gpu


def _run(w, grad, is_bf16):
    import torch
    import paper_2504_08838_amd as sd2
    import gpu_util as gu
    mat = gu.SparseMat(w, 1)
    g = gu.dev(grad)
    sd2.mask_gradient(mat.m, g.data_ptr(), is_bf16, gu.stream_ptr())
    torch.cuda.synchronize()
    out = g.cpu().numpy()
    return out.view(np.uint16) if is_bf16 else out


@pytest.mark.parametrize("n,k,pct,pattern", [(48, 320, 50, "row"), (100, 768, 70, "global"), (16, 64, 60, "row"),
                                             (1000, 3072, 50, "row"), (4096, 8192, 50, "row")])
def test_fp32_gradient_bit_exact(n, k, pct, pattern):
    w = wl.gen_weight(91, 0, "q", n, k, pct, pattern=pattern)
    g = np.random.default_rng(91).standard_normal((n, k)).astype(np.float32)
    out = _run(w, g, False)
    ref = oft.mask_gradient(w, g)
    assert np.array_equal(out.view(np.uint32), ref.view(np.uint32))


@pytest.mark.parametrize("n,k", [(48, 320), (1000, 3072)])
def test_bf16_gradient_bit_exact(n, k):
    w = wl.gen_weight(92, 0, "q", n, k, 50)
    g = wl.f32_to_bf16_bits(np.random.default_rng(92).standard_normal((n, k)).astype(np.float32))
    out = _run(w, g, True)
    ref = np.where(ol.nonzero_mask(w), g, np.uint16(0))
    assert np.array_equal(out, ref)


def test_non_finite_values_at_pruned_positions_vanish_and_kept_ones_survive():
    w = wl.gen_weight(93, 0, "q", 64, 512, 50)
    g = np.random.default_rng(93).standard_normal((64, 512)).astype(np.float32)
    kept = ol.nonzero_mask(w)
    g[~kept] = np.nan
    pos = tuple(np.argwhere(kept)[5])
    g[pos] = np.inf
    out = _run(w, g, False)
    assert not out[~kept].any() and not np.signbit(out[~kept]).any()
    assert np.isinf(out[pos]) and np.array_equal(out[kept], g[kept])


def test_zero_sparsity_changes_nothing_and_full_sparsity_clears_everything():
    g = np.random.default_rng(94).standard_normal((32, 256)).astype(np.float32)
    dense = wl.gen_weight_dense(94, 0, "q", 32, 256)
    assert np.array_equal(_run(dense, g, False), np.where(ol.nonzero_mask(dense), g, 0))
    assert not _run(np.zeros((32, 256), dtype=np.uint16), g, False).any()


@pytest.mark.parametrize("is_bf16", [False, True])
@pytest.mark.parametrize("n,k", [(1, 64), (8, 256), (9, 192), (17, 448), (31, 1088), (40, 2304)])
def test_edges_of_tiles_and_workgroups_bit_exact(n, k, is_bf16):
    """Rows around half strips and strips, columns around slabs, one to nine slabs; neighbours of the buffer stay as they are."""
    import torch
    import paper_2504_08838_amd as sd2
    import gpu_util as gu
    w = wl.gen_weight(95, 0, "q", n, k, 50)
    g = np.random.default_rng(95).standard_normal((n + 2, k)).astype(np.float32)
    g = wl.f32_to_bf16_bits(g) if is_bf16 else g
    mat, d = gu.SparseMat(w, 1), gu.dev(g)
    sd2.mask_gradient(mat.m, d[1:].data_ptr(), is_bf16, gu.stream_ptr())
    torch.cuda.synchronize()
    out, ref = d.cpu().numpy().view(g.dtype), g.copy()
    ref[1:-1] = np.where(ol.nonzero_mask(w), ref[1:-1], ref.dtype.type(0))
    assert np.array_equal(out.view(np.uint8), ref.view(np.uint8))
