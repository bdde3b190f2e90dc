"""What bench.py counts as work: only operations that the definition asks for and the kernels do."""
import bench


def _column_loop_by_hand(N, K, widths):
    """Algorithm 2 walked through, one count for every rounded operation; Algorithm 1 on |R| + 1 candidates"""
    ops = 0
    for _ in range(N):
        for j in range(K):
            for _ in range(len(widths) + 1):
                terms = 0
                for _ in widths:
                    ops += 3        # S - zero, * scale, w - D
                    ops += 2        # square, * lambda
                    ops += terms > 0
                    terms += 1
                ops += 1            # compare
            for i in range(len(widths)):
                ops += 3 + (i > 0)
            ops += 2                # / |R|, / U[j, j]
            for _ in range(j + 1, K):
                ops += 2            # E * U[j, k], w - that
    return ops


def test_column_loop_operations():
    for N, K, widths in ((1, 1, (8,)), (2, 5, (3, 4, 8)), (3, 16, (2, 3, 4, 6, 8))):
        assert bench.gptq_ops(N, K, len(widths)) == _column_loop_by_hand(N, K, widths)


def test_counted_rate_is_below_the_peak():
    # 4096 x 4096 in 2.5 ms, faster than the loop runs: a count that no hardware rate explains would show here
    assert bench.gptq_ops(4096, 4096, 3) / 2.5e-3 / 1e12 < bench.VECTOR_LANE_OPS_PEAK_T

