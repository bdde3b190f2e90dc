"""Inputs that leave the common path of the candidate search may not hold up a whole launch: times against the same call on
ordinary inputs.  A search that sweeps the codes there takes 10 to 30 times as long; the bounds leave room for noise."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import paper_2602_03537_amd as mq  # noqa: E402
from paper_2602_03537_amd import synth  # noqa: E402

pytestmark = pytest.mark.gpu


def _inputs(N, K, seed):
    W = synth.make_weights(N, K, seed)
    _, s, z = synth.quantize_parent(W)
    return [torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0") for a in (W, s, z)]


def _fastest(prepare, call, reps=7):
    times = []
    for i in range(reps):
        prepare()
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    return min(times[1:])


def _quant_time(W, s, z, widths, lam):
    Q = torch.empty(W.shape, dtype=torch.uint8, device=W.device)
    return _fastest(lambda: None, lambda: mq.mq_quant_matgptq(W, s, z, widths, lam, out=Q))


def _loop_time(W, s, z, widths, lam):
    work, Q = torch.empty_like(W), torch.empty(W.shape, dtype=torch.uint8, device=W.device)
    U = torch.eye(W.shape[1], device=W.device) + torch.triu(torch.full((W.shape[1],) * 2, 0.003, device=W.device), 1)
    return _fastest(lambda: work.copy_(W), lambda: mq.mq_matgptq_quantize(work, U, s, z, widths, lam, out=Q))


def _odd_scales(kind, W, s, z):
    W, s = W.clone(), s.clone()
    rows = slice(7, 8) if kind.endswith("one row") else slice(None)
    if kind.startswith("zero"):
        W[rows], s[rows] = 0, 0
    else:
        s[rows] = -s[rows]
    return W, s, z


@pytest.mark.parametrize("widths", [(3, 4, 8), (1, 2, 3, 4, 5, 6, 7, 8)])
@pytest.mark.parametrize("kind", ["zero, one row", "zero", "negative, one row", "negative"])
def test_odd_scales_do_not_hold_up_a_launch(kind, widths):
    lam = [1.0] * len(widths)
    plain = _inputs(2048, 1024, 311)
    odd = _odd_scales(kind, *plain)
    assert _quant_time(*odd, widths, lam) < 3 * _quant_time(*plain, widths, lam)
    plain = [t[:, :256 // (1 if t.shape[1] > 8 else 128)].contiguous() for t in plain]
    odd = _odd_scales(kind, *plain)
    assert _loop_time(*odd, widths, lam) < 3 * _loop_time(*plain, widths, lam)


@pytest.mark.parametrize("lam", [(1.0, 1.0, 1e-7), (1.0, 1e-3, 1e-9), (1e-30, 1e-20, 1e-38)])
def test_uneven_lambdas_do_not_hold_up_a_launch(lam):
    # the sums absorb the finer terms: long runs of codes have the same error
    W, s, z = _inputs(2048, 1024, 312)
    assert _quant_time(W, s, z, (3, 4, 8), lam) < 6 * _quant_time(W, s, z, (3, 4, 8), (1.0, 1.0, 1.0))
    W, s, z = W[:, :256].contiguous(), s[:, :2].contiguous(), z[:, :2].contiguous()
    assert _loop_time(W, s, z, (3, 4, 8), lam) < 6 * _loop_time(W, s, z, (3, 4, 8), (1.0, 1.0, 1.0))


def test_far_outliers_do_not_hold_up_a_launch():
    # so far out that no step shows: every code has the same error
    W, s, z = _inputs(2048, 256, 313)
    far = W.clone()
    far[7, ::5] = 1e16
    assert _loop_time(far, s, z, (3, 4, 8), (1.0, 1.0, 1.0)) < 6 * _loop_time(W, s, z, (3, 4, 8), (1.0, 1.0, 1.0))
