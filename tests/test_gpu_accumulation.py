"""Accumulation of the row kernels from 5 rows on where it shows: outputs that the zero-offset cancels almost entirely, with activations of which a few are
far larger than the others, so that what an instruction loses of the small products is not hidden by the rounding of y."""
import numpy as np
import pytest

import oracle
import tolerance
from gpu_util import C, WIDTHS, run_linear, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", WIDTHS)
@pytest.mark.parametrize("M", (5, 8, 9, 16, 20))
@pytest.mark.parametrize("groups,large", [(1, (5, 77)), (1, (0,)), (7, (5, 131, 400, 770))])
def test_small_products_beside_large_ones(M, r, groups, large):
    # Per element: rounding to fp16 and 8 fp32 unit round-offs of the magnitudes added up (tests/tolerance.py, (ii)).  The matrix instruction aligns a product
    # as if its weight were 2^-14 at least; codes of 2, 6 and 8 bits reach up to there, those of 3 and 4 bits to a half and a quarter of it, so
    # the largest activation counts with a code of 256 (512, 1024) whatever it has.  (With 6-bit codes at bit 0 of an operand the error is 1.2 of this bound, 19 round-offs of the magnitudes.)
    N, K = 512, 128 * groups
    rng = np.random.default_rng([1001, r, groups, len(large)])
    x1 = rng.standard_normal(K) + 1.0
    x1[list(large)] *= 100
    x1 = x1.astype(np.float16)
    parent = rng.integers(0, 256, (N, K), dtype=np.uint8)
    S = oracle.slice_codes(parent, C, r).astype(np.float64).reshape(N, groups, 128)
    xg = x1.astype(np.float64).reshape(groups, 128)
    zeros = (np.einsum("ngk,gk->ng", S, xg) / xg.sum(1)).astype(np.float16)
    L = {"parent": parent, "scales": np.ones((N, groups), np.float16), "zeros": zeros, "x": np.repeat(x1[None], M, axis=0)}
    ref = oracle.linear(L["x"], parent, L["scales"], zeros, C, r, 128)
    _, B = tolerance.term_scales(L["x"], parent, L["scales"], zeros, C, r, 128)
    err = np.abs(run_linear(L, r).cpu().numpy().astype(np.float64) - ref)
    over = err / (2.0 ** -10 * np.abs(ref) + 2.0 ** -24 + 8 * tolerance.U32 * (B + {3: 512, 4: 1024}.get(r, 256) * np.abs(x1.astype(np.float64)).max()))
    assert over.max() <= 1, (over.max(), (err / B).max() * 2 ** 24)
