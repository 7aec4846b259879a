"""Wide linears whose workgroups take several passes over several groups of strips, and bitmask halves around the size of their stage.
Small integers: every sum is exact in fp32, results equal to the last bit."""
import numpy as np
import pytest

from test_gpu_wide_formats import _ints, _matrix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["bitmask", "crowded", "2:4", "dense"])
@pytest.mark.parametrize("n,k,k_tok", [
    (33000, 1088, 64),  # nine strips a workgroup, eight units and a half
    (33000, 1088, 17),  # tokens in the second group: one
    (17000, 2112, 49),  # five strips a workgroup, 16.5 units, tokens in the last group: one
])
def test_wide_linear_passes_and_groups(n, k, k_tok, fmt):
    import gpu_util as gu
    rng = np.random.default_rng([6, n, k, k_tok])
    w = _matrix(rng, n, k, fmt)
    x = rng.integers(-4, 5, size=(k_tok, k))
    mat = gu.DenseMat(_ints(w)) if fmt == "dense" else gu.SparseMat(_ints(w), 3 if fmt == "2:4" else 1)
    y = gu.run_linear(mat, _ints(x), sparse=fmt != "dense")
    assert np.array_equal(y, x.astype(np.float64) @ w.T.astype(np.float64))


# values of a half tile's two 64-column steps of sixteen rows: the stage holds 1276 with their slack, a step has at most 1024
STEPS = [(1024, 252), (1024, 253), (252, 1024), (253, 1024), (1024, 1024), (1023, 254), (639, 638), (300, 300), (1024, 0), (0, 1024)]


@pytest.mark.parametrize("n,k,k_tok", [(1600, 1280, 17), (33000, 640, 40), (8200, 1344, 64)])
def test_halves_around_the_stage(n, k, k_tok):
    """Bitmask halves that just fit the staged part of their stream and halves that just do not, next to each other in a round."""
    import gpu_util as gu
    rng = np.random.default_rng([8, n, k, k_tok])
    w = rng.integers(1, 9, size=(n, k))
    kept = np.zeros((-(-n // 16), k // 64, 1024), dtype=bool)
    for strip in range(kept.shape[0]):
        for half in range(-(-k // 128)):
            for q, count in enumerate(STEPS[(strip + 3 * half) % len(STEPS)][:k // 64 - 2 * half]):
                kept[strip, 2 * half + q, rng.permutation(1024)[:count]] = True
    mask = kept.reshape(-1, k // 64, 16, 64).transpose(0, 2, 1, 3).reshape(-1, k)[:n]
    w[~mask] = 0
    x = rng.integers(-4, 5, size=(k_tok, k))
    y = gu.run_linear(gu.SparseMat(_ints(w), 1), _ints(x))
    assert np.array_equal(y, x.astype(np.float64) @ w.T.astype(np.float64))
