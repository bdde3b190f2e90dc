"""mq_linear_bf16 on single packed layers, M = 1 .. 4, bit for bit: the low-latency launch converts the bf16 activations itself.
Inputs whose fp32 sums are exact in any order (activations that are small multiples of 1/4, scales that are powers of two),
so the result has to be the bf16 rounding of the exact value; and activations at the ends of what fp16 holds."""
import numpy as np
import pytest

import oracle
import paper_2602_03537_amd as mq
from paper_2602_03537_amd import synth
from gpu_util import C, DEV, WIDTHS, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# one workgroup; ragged, one K slice's rows of waves; ragged, eight K slices; several row blocks and slices; four slices
SHAPES = [(13, 128), (200, 768), (1000, 4096), (4100, 1280), (333, 11008)]
# of one activation in an otherwise empty row: fp16 subnormals, halfway cases and what lies below them; the largest bf16 inside
# fp16's range
EDGES = [2.0 ** -14, 1.5 * 2.0 ** -15, 1.9921875 * 2.0 ** -15, 2.0 ** -24, 1.5 * 2.0 ** -24, 1.5 * 2.0 ** -25, 2.0 ** -25, 2.0 ** -26,
         1e-30, 65280.0, -65280.0, -1.25 * 2.0 ** -20]
BEYOND = [65536.0, -65536.0, 1e38, float("inf"), float("-inf"), float("nan")]   # infinities in fp16


def _layer(N, K, seed):
    rng = np.random.default_rng(seed)
    G = K // 128
    return {"parent": rng.integers(0, 256, (N, K), dtype=np.uint8),
            "scales": np.exp2(-rng.integers(7, 9, (N, G)).astype(np.float64)).astype(np.float16),
            "zeros": rng.integers(0, 256, (N, G)).astype(np.float16)}


def _bf16_bits(a):
    """exact values (float64, all of them fp32 numbers) -> bits of the nearest bf16, ties to even"""
    assert np.array_equal(a.astype(np.float32).astype(np.float64), a)
    b = a.astype(np.float32).view(np.uint32).astype(np.uint64)
    return ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).astype(np.uint16)


def _calls(L, r, x):
    """mq_linear_bf16 on x (bf16, CPU) and mq_linear on the same values as fp16"""
    N, K = L["parent"].shape
    M = x.shape[0]
    lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), r)
    args = (lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, mq.new_workspace(M, N, K, r))
    yb = mq.mq_linear_bf16(x.to(DEV), *args)
    yh = mq.mq_linear(x.to(torch.float16).to(DEV), *args)
    torch.cuda.synchronize()
    assert yb.dtype == torch.bfloat16 and yh.dtype == torch.float16
    return yb.cpu(), yh.cpu()


@pytest.mark.parametrize("M", [1, 2, 3, 4])
@pytest.mark.parametrize("N,K", SHAPES)
@pytest.mark.parametrize("r", WIDTHS)
def test_result_is_the_rounding_of_the_exact_sum(N, K, M, r):
    L = _layer(N, K, [401, N, K, r])
    rng = np.random.default_rng([402, N, K, M])
    x = torch.from_numpy(rng.integers(-8, 9, (M, K)) / 4.0).to(torch.bfloat16)
    yb, yh = _calls(L, r, x)
    ref = oracle.linear(x.to(torch.float16).numpy(), L["parent"], L["scales"], L["zeros"], C, r, 128)
    assert np.array_equal(yb.view(torch.int16).numpy().view(np.uint16), _bf16_bits(ref))
    assert np.array_equal(yh.numpy(), ref.astype(np.float16))   # the same sums from the same values given as fp16


@pytest.mark.parametrize("M", [1, 2, 3, 4])
@pytest.mark.parametrize("r", WIDTHS)
def test_activations_at_the_ends_of_the_fp16_range(M, r):
    N, K = 200, 768
    L = _layer(N, K, [403, r])
    rng = np.random.default_rng([404, M, r])
    for first in range(0, len(EDGES), M):
        x = np.zeros((M, K), np.float64)
        for m in range(M):
            x[m, rng.integers(K)] = EDGES[(first + m) % len(EDGES)]
        x = torch.from_numpy(x).to(torch.bfloat16)
        yb, _ = _calls(L, r, x)
        ref = oracle.linear(x.to(torch.float16).numpy(), L["parent"], L["scales"], L["zeros"], C, r, 128)
        ref = np.where(ref == 0, 0.0, ref)
        got = yb.view(torch.int16).numpy().view(np.uint16)
        assert np.array_equal(np.where(got == 0x8000, 0, got), _bf16_bits(ref)), (x[x != 0], first)


@pytest.mark.parametrize("M", [1, 3, 4])
def test_activations_beyond_the_fp16_range_are_infinities(M):
    # such a row is infinite or no number, as it is for the infinity given as fp16; the other rows do not see it
    N, K = 200, 768
    for r in WIDTHS:
        L = _layer(N, K, [405, r])
        rng = np.random.default_rng([406, M, r])
        for i, v in enumerate(BEYOND):
            x = rng.integers(-8, 9, (M, K)) / 4.0
            x[i % M, rng.integers(K)] = v
            x = torch.from_numpy(x).to(torch.bfloat16)
            yb, yh = _calls(L, r, x)
            assert torch.equal(yb.isnan(), yh.isnan()) and torch.equal(yb.isinf(), yh.isinf()), (r, v)
            assert not yb[i % M].isfinite().any() and yb[[m for m in range(M) if m != i % M]].isfinite().all()
