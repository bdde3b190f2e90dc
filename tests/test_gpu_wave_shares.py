"""The persistent launch whose shares belong to waves: row blocks cut into many shares, whole ones, one group a row block, shares of one tile, layers computed from
their parent, single layers, and a small workspace.  tests/test_persistent_shares.py holds that these calls take it."""
import numpy as np
import pytest

import oracle
import paper_2602_03537_amd as mq
from paper_2602_03537_amd import synth
from gpu_util import C, DEV, WIDTHS, check_layer, check_y, dev, torch

pytestmark = pytest.mark.gpu

# the first of 17 layers (more than a low-latency launch takes), and the widths of all
STACKS = {"cut": ((130, 28672), (2,)), "few_groups": ((4100, 640), WIDTHS), "one_group": ((64 * 300 - 7, 128), WIDTHS), "short": ((65, 128), WIDTHS),
          "three_bits": ((64 * 40, 3200), (3, 2)), "eight_groups": ((64 * 90, 1024), (8, 6, 4))}
SINGLES = ((64 * 300 - 9, 16000), (64 * 2100, 2432))


def _shapes(name):
    return [STACKS[name][0]] + [(64 * (1 + i % 3), 128 * (1 + i % 2)) for i in range(16)]


# (from the parent all tiles are of 8 bits: the stacks of few groups a row block)
@pytest.mark.parametrize("M,parent,name", [(M, 0, name) for M in (1, 2, 3, 4, 5, 8, 9, 16) for name in STACKS] +
                         [(M, 1, name) for M in (1, 2, 3, 4) for name in ("few_groups", "one_group", "short", "eight_groups")])
def test_shares_of_waves(M, parent, name):
    widths = STACKS[name][1]
    host = [synth.make_layer(N, K, M=M, seed=[611, M, N, i]) for i, (N, K) in enumerate(_shapes(name))]
    layers = []
    for i, L in enumerate(host):
        lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), 8 if parent else widths[i % len(widths)])
        x = torch.empty(M * lay["K"] + 2, dtype=torch.float16, device=DEV)[2:].view(M, lay["K"])  # 4 bytes past an aligned address
        x.copy_(dev(L["x"]))
        layers.append(dict(lay, r=widths[i % len(widths)], from_parent=parent, x=x, y=torch.full((M, lay["N"]), float("nan"), dtype=torch.float16, device=DEV)))
    plan = mq.mq_stack_plan(layers, M, device=DEV)
    outs = []
    for _ in range(3):                                   # the counters are left as they were found
        mq.mq_linear_stack(plan)
        torch.cuda.synchronize()
        outs.append([lay["y"].clone() for lay in layers])
    for i, (lay, L) in enumerate(zip(layers, host)):
        check_layer(outs[0][i], L, lay["r"], f"{name} layer {i} {lay['N']}x{lay['K']} M={M} r={lay['r']}")
        assert torch.equal(outs[0][i], outs[1][i]) and torch.equal(outs[0][i], outs[2][i])   # fixed summation order


@pytest.mark.parametrize("N,K", SINGLES)
def test_single_layers_sampled_rows(N, K):
    L = synth.make_random_codes_layer(N, K, M=4, seed=[612, N])
    rows = np.unique(np.concatenate([[0, 63, 64, N - 2, N - 1], np.random.default_rng(613).integers(0, N, 100)]))
    rt = torch.from_numpy(rows).to(DEV)
    lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), 2)
    for M in (2, 3, 4):
        ref = oracle.linear_rows(L["x"][:M], L["parent"], L["scales"], L["zeros"], C, 2, 128, rows)
        x, outs = dev(L["x"][:M]), []
        ws = mq.new_workspace(M, N, K, 2)
        for _ in range(2):
            outs.append(mq.mq_linear(x, lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, 2, 128, ws).clone())
        y = torch.empty_like(outs[0])
        mq.mq_linear_noalloc(x, lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, 2, 128, y)
        torch.cuda.synchronize()
        assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
        for out in (outs[0], y):
            check_y(out[:, rt], ref, f"{N}x{K} M={M}")
