"""Small stacks and single layers whose layers are not cut along K, or in fewer slices than alone, on either side of each line of those rules, and the one-row
stacks of up to four bits, which have a kernel of their own: one tile a wave, several, none for some waves, row blocks with rows that do not exist."""
import pytest

import paper_2602_03537_amd as mq
from gpu_util import DEV, check_layer, dev, torch
from paper_2602_03537_amd import synth

pytestmark = pytest.mark.gpu

# (rows, groups) of the layers
STACKS = {
    "8_groups": [(65, 8), (130, 3), (64, 1)],
    "9_groups": [(64 * 63, 9), (60, 2)],
    "16_groups_63": [(64 * 40, 16), (64 * 23 - 1, 16)],
    "16_groups_64": [(64 * 40, 16), (64 * 24 - 1, 17 - 1)],
    "17_groups_96": [(64 * 95, 17), (1, 17)],
    "33_groups_160": [(64 * 100, 33), (64 * 60 - 3, 33)],
    "49_groups_192": [(64 * 190, 49), (100, 49)],
    "256_blocks": [(64 * 200, 5), (64 * 56, 16)],
    "40_groups_208": [(64 * 150, 40), (64 * 58, 7)],
    "cut_in_4_of_64": [(64 * 32, 31), (64 * 32 - 5, 24)],
    "cut_in_4": [(64 * 20, 32), (64 * 28, 48)],
    "cut_in_2_of_128": [(64 * 100, 33), (64 * 28, 64)],
    "257_blocks": [(64 * 200, 5), (64 * 57, 16)],
}


@pytest.mark.parametrize("name", STACKS)
@pytest.mark.parametrize("M,widths", [(1, (2, 3)), (1, (4, 3)), (1, (4, 6)), (1, (8, 2)), (2, (3, 6)), (3, (8, 4)), (4, (2, 4)), (6, (3, 4)), (8, (8, 2)), (13, (4, 6))])
def test_small_stacks(name, M, widths):
    host = [synth.make_layer(N, 128 * G, M=M, seed=[901, M, N, G]) for N, G in STACKS[name]]
    layers = []
    for i, L in enumerate(host):
        lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), widths[i % 2])
        layers.append(dict(lay, x=dev(L["x"]), y=torch.full((M, lay["N"]), float("nan"), dtype=torch.float16, device=DEV)))
    plan = mq.mq_stack_plan(layers, M, device=DEV)
    outs = []
    for _ in range(2):
        mq.mq_linear_stack(plan)
        torch.cuda.synchronize()
        outs.append([lay["y"].clone() for lay in layers])
    for i, (lay, L) in enumerate(zip(layers, host)):
        check_layer(outs[0][i], L, lay["r"], f"{name} layer {i} M={M} r={lay['r']}")
        assert torch.equal(outs[0][i], outs[1][i])
        ws = mq.new_workspace(M, lay["N"], lay["K"], lay["r"])
        y = mq.mq_linear(lay["x"], lay["packed_W"], lay["scales_t"], lay["zeros_t"], lay["N"], lay["K"], lay["r"], 128, ws)
        torch.cuda.synchronize()
        check_layer(y, L, lay["r"], f"{name} layer {i} alone M={M} r={lay['r']}")
