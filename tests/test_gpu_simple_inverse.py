"""GPU parity: the symmetric elimination of the simple method at the edges of its blocks, against the float64 oracle.

G^{-1} is formed in 64 bits and rounded to 32: relative to the exact one an error of 2^-24 in each element, and the last
product adds about as much times sqrt(n).  Against the result (whose norm the large eigenvalues of G make smaller than
|G^{-1}| |X|, here by 10 at most) that stays under 2^-24 * (1 + sqrt(257)) * 10 = 1.0e-5.
"""
import numpy as np
import pytest

from oracle.simple_ng import simple_ng
from test_gpu_simple_ng import data, gpu_call, rel

pytestmark = pytest.mark.gpu


# pivot blocks of 32: one (a single pivot, nearly full, full), two to nine: odd and even counts of blocks and of 64 x 64 tiles,
# the last ones full, nearly empty and ragged; column space and row space
@pytest.mark.parametrize("n", [1, 2, 3, 5, 31, 32, 33, 63, 64, 65, 95, 97, 128, 129, 160, 161, 193, 224, 225, 257])
@pytest.mark.parametrize("rows", [False, True], ids=["columns", "rows"])
def test_edges_of_pivot_blocks(ngsgd, n, rows):
    import torch
    if rows and n < 2:
        pytest.skip("the method needs two rows")
    rng = np.random.default_rng(4000 + n)
    N, D = (n, n + 45) if rows else (n + 45, n)
    M = data(rng, N, D)
    got, g_g, _ = gpu_call(torch, ngsgd.SimplePreconditioner(N, D), M)
    want, g_o, _ = simple_ng(M.astype(np.float64))
    assert rel(got, want) < 1.0e-5
    assert g_g == pytest.approx(g_o, rel=1.0e-5)
