"""The single-launch forward where its pieces end: blocks of one to sixteen strips leaving a compute unit (items of four strips and
a token, up to three per wavefront), last blocks that are not whole, and tile streams from empty to the longest that fits."""
from types import SimpleNamespace

import numpy as np
import pytest

import sd2_workload as wl
from oracle import linear as ol
from oracle import stack as os_

pytestmark = pytest.mark.gpu
E2E_TOL = 5e-3  # whole-stack bar of tests/test_gpu_stack.py: activations near a bf16 boundary round either way


def _shape(hidden, heads, kv, inter, layers=1):
    return SimpleNamespace(layers=layers, hidden=hidden, q_out=128 * heads, kv_out=128 * kv, inter=inter, n_heads=heads, n_kv=kv, head_dim=128)


@pytest.mark.parametrize("shape,k_tok,pct", [
    (_shape(256, 2, 1, 30080), 8, 50),       # gate|up: sixteen strips a workgroup, 32 items
    (_shape(256, 2, 1, 30080), 3, 50),       # ... 12 items
    (_shape(320, 3, 3, 704, layers=2), 7, 40),   # few strips, 64-column remainder, streams of nearly 5 KiB
    (_shape(1088, 4, 2, 4160, layers=2), 5, 95),  # short streams
])
def test_forward_blocks_and_streams(shape, k_tok, pct):
    import gpu_util as gu
    table = {p: (n, k) for p, n, k in wl.layer_matrix_shapes(shape)}
    cache = {}

    def get(layer, proj):
        if (layer, proj) not in cache:
            w = wl.gen_weight(21, layer, proj, *table[proj], pct)
            if pct == 95:
                w = w.copy()
                w[16:48, :256] = 0  # tiles without a value
            cache[(layer, proj)] = w
        return cache[(layer, proj)]

    h_in = wl.gen_x(21, 0, "q", k_tok, shape.hidden)
    ref = os_.drafter_forward(shape, get, h_in)
    model = gu.build_model(shape, get)
    out = gu.run_forward(model, h_in, shape.hidden)
    assert ol.rel_l2(out, ref) <= E2E_TOL
    assert np.array_equal(gu.run_forward(model, h_in, shape.hidden), out)  # integer sums: bit-identical


@pytest.mark.parametrize("k_tok", range(1, 9))
@pytest.mark.parametrize("fmt", [1, 3])
def test_every_count_of_tokens(k_tok, fmt):
    """Prologues run on 1, 2, 3, 4, 5 or 8 token slots, the smallest count that holds the tokens: slots beyond them read nothing and
    add nothing, and attention's rows end unevenly on the wavefronts of a head."""
    import gpu_util as gu
    shape = _shape(384, 3, 1, 1088, layers=2)
    table = {p: (n, k) for p, n, k in wl.layer_matrix_shapes(shape)}
    cache = {}

    def get(layer, proj):
        if (layer, proj) not in cache:
            cache[(layer, proj)] = wl.gen_weight(22, layer, proj, *table[proj], 50, **({"pattern": "2:4"} if fmt == 3 else {}))
        return cache[(layer, proj)]

    h_in = wl.gen_x(22, 0, "q", k_tok, shape.hidden)
    ref = os_.drafter_forward(shape, get, h_in)
    model = gu.build_model(shape, get, fmt=fmt)
    out = gu.run_forward(model, h_in, shape.hidden)
    assert out.shape[0] == k_tok and ol.rel_l2(out, ref) <= E2E_TOL
    assert np.array_equal(gu.run_forward(model, h_in, shape.hidden), out)
