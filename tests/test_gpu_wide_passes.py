"""Wide linears whose workgroups take several passes over several groups of strips: the next pass's activations travel while this
one's are used, and not across the end of a group.  Small integers: every sum is exact in fp32, results equal to the last bit."""
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
