"""The persistent launch of the row kernels, whose shares belong to workgroups: row blocks cut into many shares, whole ones, shares shorter than a
workgroup has waves, few groups a row block; from 5 rows on with activations at any address of a pair."""
import functools

import pytest

import paper_2602_03537_amd as mq
from gpu_util import DEV, WIDTHS, check_layer, dev, torch
from paper_2602_03537_amd import synth

pytestmark = pytest.mark.gpu

# 17 layers are more than a low-latency launch takes: (rows, columns) of one, 15 small ones, and one of 8 bits and 20 groups that has most row blocks and
# most of the work, so that shares belong to workgroups (tests/test_persistent_shares.py)
LONG, MANY, SMALL, WHOLE = (130, 28672), (1100, 640), (65, 128), (64 * 40, 3200)


def stack_of(shape, M):
    shapes = [shape] + [(64, 128 * (1 + i % 2)) for i in range(15)] + [(12200, 2560)]
    return shapes, [WIDTHS[(i + M) % 5] for i in range(16)] + [8]


@functools.lru_cache(maxsize=1)
def _big():
    return synth.make_layer(12200, 2560, M=16, seed=[603])


@pytest.mark.parametrize("shape", [LONG, MANY, SMALL, WHOLE], ids=["cut", "few_groups", "short", "about_whole"])
@pytest.mark.parametrize("M", (1, 2, 4, 5, 8, 9, 16))
def test_shares(M, shape):
    shapes, widths = stack_of(shape, M)
    host = [synth.make_layer(N, K, M=M, seed=[601, M, N, i]) for i, (N, K) in enumerate(shapes[:-1])] + [dict(_big(), x=_big()["x"][:M])]
    layers = []
    for i, L in enumerate(host):
        lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), widths[i])
        x = torch.empty(M * lay["K"] + 2, dtype=torch.float16, device=DEV)[2:].view(M, lay["K"])  # 4 bytes past an aligned address
        x.copy_(dev(L["x"]))
        layers.append(dict(lay, x=x, y=torch.full((M, lay["N"]), float("nan"), dtype=torch.float16, device=DEV)))
    plan = mq.mq_stack_plan(layers, M, device=DEV)
    outs = []
    for _ in range(3):                                   # the counters are left as they were found
        mq.mq_linear_stack(plan)
        torch.cuda.synchronize()
        outs.append([lay["y"].clone() for lay in layers])
    for i, (lay, L) in enumerate(zip(layers, host)):
        check_layer(outs[0][i], L, lay["r"], f"layer {i} {lay['N']}x{lay['K']} M={M} r={lay['r']}")
        assert torch.equal(outs[0][i], outs[1][i]) and torch.equal(outs[0][i], outs[2][i])   # fixed summation order


# 238 and 240 tiles, a share each: grids that are not and that are a multiple of the eight dies
def few_shares(tiles):
    return [(64, 1792)] * 17 if tiles == 238 else [(64, 1792)] * 16 + [(60, 2048)]


@pytest.mark.parametrize("tiles", (238, 240))
@pytest.mark.parametrize("M", (1, 3, 8, 16))
def test_fewer_shares_than_compute_units(M, tiles):
    host = [synth.make_layer(N, K, M=M, seed=[604, i, M]) for i, (N, K) in enumerate(few_shares(tiles))]
    layers = [dict(mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), 8), x=dev(L["x"]),
                   y=torch.full((M, L["parent"].shape[0]), float("nan"), dtype=torch.float16, device=DEV)) for L in host]
    plan = mq.mq_stack_plan(layers, M, device=DEV)
    for _ in range(2):
        mq.mq_linear_stack(plan)
    torch.cuda.synchronize()
    for i, (lay, L) in enumerate(zip(layers, host)):
        check_layer(lay["y"], L, 8, f"layer {i} M={M}")


# single layers whose 256 shares are whole row blocks, halves and eighths of one
@pytest.mark.parametrize("N,K", [(16384, 1024), (16384, 4096), (4096, 4096), (2048, 8192)])
@pytest.mark.parametrize("M", (9, 16))
def test_even_shares(M, N, K):
    L = synth.make_layer(N, K, M=M, seed=[602, N, K])
    lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), 3)
    ws = mq.new_workspace(M, N, K, 3)
    outs = [mq.mq_linear(dev(L["x"]), lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, 3, 128, ws).clone() for _ in range(2)]
    torch.cuda.synchronize()
    check_layer(outs[0], L, 3, f"{N}x{K} M={M}")
    assert torch.equal(outs[0], outs[1])
