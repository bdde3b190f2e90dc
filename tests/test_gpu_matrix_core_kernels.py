"""Matrix-core kernels in the calls that the low-latency launch does not take: the persistent launch of the row kernels at 9 .. 16 rows, the wide
kernel above.  The shapes are chosen by the rules of csrc/mq_routes.h: a single layer of 233 groups (eight K slices leave a wave eight tiles; under
the wide kernel its row blocks are finished by a launch of their own), a stack of 17 layers up to 16 rows (more than a low-latency launch takes) and
any stack above (row blocks finished by their last contributor).  tests/test_routes.py holds that they take these ways."""
import numpy as np
import pytest

import oracle
import paper_2602_03537_amd as mq
from paper_2602_03537_amd import synth
from gpu_util import C, DEV, WIDTHS, check_layer, dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LONG = 233 * 128
# 16 columns; one to four chunks of 32
BATCHES = (9, 16, 17, 64, 65, 128)
ROUTES = ("single", "stack")


def _shape(route):
    return (200, LONG) if route == "single" else (321, 1280)


def _y(M, N, dtype):
    buf = torch.full((M * N + 128,), float("nan"), dtype=dtype, device=DEV)
    return buf, buf[64:64 + M * N].view(M, N)


def _run(route, lay, x, dtype=torch.float16):
    """y of `lay` from the persistent launch of the row kernels (up to 16 rows) or the wide kernel: three times, the same bits, nothing written around it."""
    M, N, K, r = x.shape[0], lay["N"], lay["K"], lay["r"]
    buf, y = _y(M, N, dtype)
    if route == "single":
        call, ws = mq.mq_linear if dtype == torch.float16 else mq.mq_linear_bf16, mq.new_workspace(M, N, K, r)
        def run():
            call(x, lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, ws, y=y)
    else:
        flags = (mq.MQ_X_BF16 | mq.MQ_Y_BF16) if dtype == torch.bfloat16 else 0
        layers = [dict(lay, x=x, y=y, flags=flags)]
        if M <= 16:
            fill = [mq.prepare_layer(*(dev(a) for a in _filler(i)), WIDTHS[i % 5]) for i in range(16)]
            fx = torch.ones((M, 256), dtype=torch.float16, device=DEV)
            layers = [dict(f, x=fx, y=torch.empty((M, f["N"]), dtype=torch.float16, device=DEV)) for f in fill]
            layers.insert(8, dict(lay, x=x, y=y, flags=flags))
        plan = mq.mq_stack_plan(layers, M, device=DEV)
        def run():
            mq.mq_linear_stack(plan)
    outs = []
    for _ in range(3):
        y.fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        outs.append(y.clone())
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert torch.isnan(buf[:64]).all() and torch.isnan(buf[64 + M * N:]).all()
    return outs[0]


_FILLERS = {}


def _filler(i):
    if i not in _FILLERS:
        L = synth.make_layer(70 + 64 * (i % 3), 256, seed=[601, i])
        _FILLERS[i] = (L["parent"], L["scales"], L["zeros"])
    return _FILLERS[i]


def _layer(kind, route, M):
    N, K = _shape(route)
    if kind != "random":
        return synth.make_layer(N, K, M=M, seed=[602, M, K])
    L = synth.make_random_codes_layer(N, K, M=M, seed=[603, M, K])
    # (sums of 29 824 terms within the absolute bar's range of fp16)
    return dict(L, scales=(L["scales"].astype(np.float32) * (1 / 8 if K == LONG else 1)).astype(np.float16))


@pytest.mark.parametrize("M", BATCHES)
@pytest.mark.parametrize("route", ROUTES)
@pytest.mark.parametrize("kind", ["quantised", "random"])   # integer zeros; every code value, zeros with fraction bits
def test_against_the_oracle(kind, route, M):
    L = _layer(kind, route, M)
    p, s, z, x = dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), dev(L["x"])
    for r in WIDTHS:
        check_layer(_run(route, mq.prepare_layer(p, s, z, r), x), L, r, f"{kind} {route} M={M} r={r}")


@pytest.mark.parametrize("M", BATCHES)
@pytest.mark.parametrize("route", ROUTES)
def test_symmetric_layers(route, M):
    L = _layer("quantised", route, M)
    L["zeros"] = np.full_like(L["zeros"], 128.0)
    p, s, z, x = dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), dev(L["x"])
    for r in (2, 3, 8):
        y = _run(route, mq.prepare_layer(p, s, None, r), x)
        check_layer(y, L, r, f"symmetric {route} M={M} r={r}")
        assert torch.equal(y, _run(route, mq.prepare_layer(p, s, z, r), x))


@pytest.mark.parametrize("M", BATCHES)
@pytest.mark.parametrize("route", ROUTES)
def test_bf16_activations_and_outputs(route, M):
    L = _layer("quantised", route, M)
    xb = torch.from_numpy(L["x"].astype(np.float32)).to(torch.bfloat16)
    p, s, z = dev(L["parent"]), dev(L["scales"]), dev(L["zeros"])
    for r in (2, 4, 6):
        lay = mq.prepare_layer(p, s, z, r)
        got = _run(route, lay, xb.to(DEV), torch.bfloat16).float().cpu().numpy().astype(np.float64)
        ref = oracle.linear(xb.to(torch.float16).numpy(), L["parent"], L["scales"], L["zeros"], C, r, 128)
        # half a bf16 spacing from the rounding, the rest from the fp32 sums
        assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 3e-3), f"bf16 {route} M={M} r={r}"
        assert np.linalg.norm(got - ref) <= 2.5e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("M", (9, 16))
def test_noalloc_9_to_16_rows(M):
    # few schedule shares (the array's room): row blocks of two and three contributors and of one
    N, K, r = 321, LONG, 3
    L = synth.make_layer(N, K, M=M, seed=[604, M])
    lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), r)
    buf, y = _y(M, N, torch.float16)
    for _ in range(2):
        y.fill_(float("nan"))
        mq.mq_linear_noalloc(dev(L["x"]), lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, y)
        torch.cuda.synchronize()
        check_layer(y, L, r, f"noalloc M={M}")
    assert torch.isnan(buf[:64]).all() and torch.isnan(buf[64 + M * N:]).all()
