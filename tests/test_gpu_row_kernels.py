"""Batches where one kernel takes over from another, 2 .. 256 rows: the row kernels (built for 2, 3, 4, 8 and 16 rows; by 4x4x4 and from 5 rows on
16x16x32 matrix instructions), single layers, small stacks, stacks of more layers than travel with a launch, and bf16."""
import numpy as np
import pytest

import oracle
import paper_2602_03537_amd as mq
from paper_2602_03537_amd import synth
from gpu_util import C, DEV, WIDTHS, check_layer, check_y, dev, run_linear

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BATCHES = (2, 3, 4, 5, 7, 8, 9, 12, 13, 16)


@pytest.mark.parametrize("r", WIDTHS)
@pytest.mark.parametrize("M", BATCHES)
@pytest.mark.parametrize("shape", [(65, 128), (200, 1152), (1000, 2176)])   # one group; fewer and more groups than waves; K slices
def test_single_layers(r, M, shape):
    L = synth.make_random_codes_layer(*shape, M=M, seed=[501, M, *shape])
    check_layer(run_linear(L, r), L, r, f"{shape} M={M} r={r}")


@pytest.mark.parametrize("r", WIDTHS)
@pytest.mark.parametrize("M", (17, 33, 100, 128))
@pytest.mark.parametrize("shape", [(1, 128), (65, 128), (200, 1152), (1000, 2176), (4100, 640)])
def test_single_layers_in_chunks_of_16_rows(r, M, shape):
    # (row blocks with a last chunk of 1 and 4 rows; not, one, and several times cut along K; one counter for all chunks of a row block; exact
    # products, which the bar for short outputs asks for)
    N, K = shape
    L = synth.make_random_codes_layer(N, K, M=M, seed=[507, M, N, K])
    lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), r)
    ws, x = mq.new_workspace(M, N, K, r), dev(L["x"])
    buf = torch.full((M * N + 128,), float("nan"), dtype=torch.float16, device=DEV)
    outs = []
    for _ in range(2):
        y = buf[64:64 + M * N].view(M, N).fill_(float("nan"))
        mq.mq_linear(x, lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, ws, y)
        torch.cuda.synchronize()
        outs.append(y.clone())
    check_layer(outs[0], L, r, f"{shape} M={M} r={r}", fp16_weights=False)
    assert torch.equal(outs[0], outs[1])                # counters left at zero, fixed summation order
    assert torch.isnan(buf[:64]).all() and torch.isnan(buf[64 + M * N:]).all()


@pytest.mark.parametrize("M", (20, 64, 65, 128))        # one to four chunks of the wide kernel, where it still serves single layers
def test_many_rows_keep_the_wide_kernel_sampled_rows(M):
    N, K = 33000 if M <= 32 else 16500, 1152
    L = synth.make_layer(N, K, M=M, seed=[508, M])
    rows = np.unique(np.concatenate([[0, 63, 64, 255, 256, N - 2, N - 1], np.random.default_rng(509).integers(0, N, 60)]))
    for r in WIDTHS:
        y = run_linear(L, r)
        assert torch.isfinite(y).all()
        check_y(y[:, torch.from_numpy(rows).to(DEV)], oracle.linear_rows(L["x"], L["parent"], L["scales"], L["zeros"], C, r, 128, rows),
                f"M={M} r={r}")


@pytest.mark.parametrize("M", (129, 200, 256))          # three and four chunks, two passes
@pytest.mark.parametrize("shape", [(65, 2176), (300, 4096), (1000, 640)])
def test_wide_row_blocks_finished_by_a_launch_of_their_own(M, shape):
    N, K = shape
    L = synth.make_layer(N, K, M=M, seed=[510, M, N, K])
    for r in WIDTHS:
        y = run_linear(L, r)
        check_layer(y, L, r, f"{shape} M={M} r={r}")
        assert torch.equal(y, run_linear(L, r))


@pytest.mark.parametrize("M", (20, 64))                 # one and two chunks, long sums: many shares in a row block
def test_wide_many_shares_in_a_row_block_sampled_rows(M):
    N, K = 4200, 12672
    L = synth.make_layer(N, K, M=M, seed=[511, M])
    rows = np.unique(np.concatenate([[0, 63, 64, 4159, 4160, N - 1], np.random.default_rng(512).integers(0, N, 60)]))
    for r in (3, 6):
        y = run_linear(L, r)
        assert torch.isfinite(y).all()
        check_y(y[:, torch.from_numpy(rows).to(DEV)], oracle.linear_rows(L["x"], L["parent"], L["scales"], L["zeros"], C, r, 128, rows),
                f"M={M} r={r}")


@pytest.mark.parametrize("M", (68, 128, 130))           # three and four chunks, two passes of three
def test_wide_shares_of_half_a_row_block_sampled_rows(M):
    # two shares meet in every row block, and the second adds the first one's sums up itself
    N, K = 8500 if M > 128 else 17000, 2048
    L = synth.make_layer(N, K, M=M, seed=[513, M])
    rows = np.unique(np.concatenate([[0, 63, 64, 255, 256, N - 2, N - 1], np.random.default_rng(514).integers(0, N, 60)]))
    for r in (2, 8):
        y = run_linear(L, r)
        assert torch.isfinite(y).all() and torch.equal(y, run_linear(L, r))
        check_y(y[:, torch.from_numpy(rows).to(DEV)], oracle.linear_rows(L["x"], L["parent"], L["scales"], L["zeros"], C, r, 128, rows),
                f"M={M} r={r}")


def _put(L, r, M):
    lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), None if L["zeros"] is None else dev(L["zeros"]), r)
    N = L["parent"].shape[0]
    return dict(lay, x=dev(L["x"]), y=torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV))


# 3 layers: one launch in the low-latency shape; 17: the persistent launch (of waves' shares up to 8 rows, workgroups' above)
@pytest.mark.parametrize("M", BATCHES)
@pytest.mark.parametrize("n", [3, 17])
def test_stacks(M, n):
    shapes = [(65 + 61 * (i % 5), 128 * (1 + i % 4)) for i in range(n)]
    widths = [WIDTHS[(i + M) % 5] for i in range(n)]
    host = [synth.make_layer(N, K, M=M, seed=[502, M, i]) for i, (N, K) in enumerate(shapes)]
    layers = [_put(L, r, M) for L, r in zip(host, widths)]
    plan = mq.mq_stack_plan(layers, M, device=DEV)
    outs = []
    for _ in range(2):
        mq.mq_linear_stack(plan)
        torch.cuda.synchronize()
        outs.append([lay["y"].clone() for lay in layers])
    for i, (L, r) in enumerate(zip(host, widths)):
        check_layer(outs[0][i], L, r, f"layer {i} of {n} M={M} r={r}")
        assert torch.equal(outs[0][i], outs[1][i])          # fixed summation order


@pytest.mark.parametrize("M", (2, 4, 5, 8, 11, 16, 40))
def test_bf16_is_the_same_arithmetic(M):
    # sums that are exact in any order: the bf16 result is the rounding of the exact value
    N, K = 300, 1280
    rng = np.random.default_rng([503, M])
    parent = rng.integers(0, 256, (N, K), dtype=np.uint8)
    s = np.exp2(-rng.integers(7, 9, (N, K // 128)).astype(np.float64)).astype(np.float16)
    z = rng.integers(0, 256, (N, K // 128)).astype(np.float16)
    x = torch.from_numpy(rng.integers(-8, 9, (M, K)) / 4.0).to(torch.bfloat16)
    for r in WIDTHS:
        lay = mq.prepare_layer(dev(parent), dev(s), dev(z), r)
        y = mq.mq_linear_bf16(x.to(DEV), lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, mq.new_workspace(M, N, K, r))
        ref = oracle.linear(x.to(torch.float16).numpy(), parent, s, z, C, r, 128)
        assert torch.equal(y.cpu(), torch.from_numpy(ref).to(torch.float32).to(torch.bfloat16)), r


@pytest.mark.parametrize("M", (2, 3, 5, 8, 9, 16))
def test_infinities_stay_in_their_batch_row(M):
    N, K = 200, 768
    L = synth.make_layer(N, K, M=M, seed=[504, M])
    for m in (0, M - 1):
        for v in (np.inf, -np.inf, np.nan):
            x = L["x"].copy()
            x[m, 5 + m] = v
            for r in WIDTHS:
                y = run_linear(dict(L, x=x), r).cpu()
                assert not y[m].isfinite().any() and y[[i for i in range(M) if i != m]].isfinite().all(), (m, v, r)


def test_layers_beyond_the_low_latency_shape_sampled_rows():
    # 12 416 tiles: the low-latency launch up to 8 rows, the persistent one above
    N, K = 12401, 8192
    L = synth.make_layer(N, K, M=16, seed=[505])
    rows = np.unique(np.concatenate([[0, 63, 64, N - 2, N - 1], np.random.default_rng(506).integers(0, N, 90)]))
    rt = torch.from_numpy(rows).to(DEV)
    p, s, z = dev(L["parent"]), dev(L["scales"]), dev(L["zeros"])
    for r in WIDTHS:
        lay = mq.prepare_layer(p, s, z, r)
        for M in (2, 3, 4, 5, 8, 9, 16):
            y = mq.mq_linear(dev(L["x"][:M]), lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, mq.new_workspace(M, N, K, r))
            torch.cuda.synchronize()
            assert torch.isfinite(y).all()
            check_y(y[:, rt], oracle.linear_rows(L["x"][:M], L["parent"], L["scales"], L["zeros"], C, r, 128, rows), f"M={M} r={r}")


def test_two_bits_of_many_tiles_single_and_as_a_stack():
    # 5 rows, 62 720 tiles: as a single layer shares of workgroups, as a stack shares of waves.  Products are exact in both; fp32 sums in another
    # order change the fp16 rounding of few values, each by one spacing (2^-10), where all of them would be 4.9e-4 in the 2-norm
    N, K, r, M = 28672, 17920, 2, 5
    L = synth.make_layer_device(N, K, seed=515, device=DEV, want_x=False)
    lay = mq.prepare_layer(L["parent"], L["scales"], L["zeros"], r)
    x = torch.randn((M, K), generator=torch.Generator(device=DEV).manual_seed(516), device=DEV).half()
    y = mq.mq_linear(x, lay["packed_W"], lay["scales_t"], lay["zeros_t"], N, K, r, 128, mq.new_workspace(M, N, K, r))
    ys = torch.full((M, N), float("nan"), dtype=torch.float16, device=DEV)
    mq.mq_linear_stack(mq.mq_stack_plan([dict(lay, x=x, y=ys)], M, device=DEV))
    torch.cuda.synchronize()
    assert torch.isfinite(y).all() and torch.linalg.vector_norm((y - ys).double()) <= 4.9e-4 * torch.linalg.vector_norm(y.double())


@pytest.mark.parametrize("M", (5, 8))
def test_small_stack_with_one_long_layer(M):
    # few enough tiles for the low-latency launch, which would leave a wave of the long layer seven of them: the persistent launch
    host = [synth.make_layer(N, K, M=M, seed=[517, N, M]) for N, K in ((49600, 128), (100, 3200))]
    layers = []
    for L, r in zip(host, (3, 2)):
        lay = mq.prepare_layer(dev(L["parent"]), dev(L["scales"]), dev(L["zeros"]), r)
        layers.append(dict(lay, x=dev(L["x"]), y=torch.full((M, lay["N"]), float("nan"), dtype=torch.float16, device=DEV)))
    plan = mq.mq_stack_plan(layers, M, device=DEV)
    for rep in range(2):
        mq.mq_linear_stack(plan)
        torch.cuda.synchronize()
        for lay, L in zip(layers, host):
            check_layer(lay["y"], L, lay["r"], f"M={M} r={lay['r']} rep {rep}")
            lay["y"].fill_(float("nan"))
