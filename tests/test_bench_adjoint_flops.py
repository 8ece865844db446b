"""The adjoint flop counts of bench.py against the operations of the sweeps, walked one by
one: a forward pass once, reverse steps on the kept states, no recomputed step."""
import bench
import workloads


def reverse_step(n, q):
    """FP32 operations of one reverse step (adjoint_kernel.hpp), FMA = 2."""
    ops = 0
    for _ in range(n):
        ops += 2 + 1 + 1               # ell: the FMA, the exponential, the reciprocal
    for _ in range(q):
        for _ in range(n - 1):
            ops += 2 + 2               # R + ell (E R + E)
        for _ in range(n):
            ops += 1                   # W Xbar
            ops += 2                   # P F = R F + F
            ops += 2                   # ellbar += E P F
            ops += 1 + 2 + 1           # x (W Xbar R + ell P F)
            ops += 1 + 2               # lambdabar += (1 + E) of it
            ops += 2 + 2               # F + E (ell F + W Xbar)
    for _ in range(n):
        ops += 1 + 2 + 1               # vol sum += Xbar (dH - kappa' dt) + lambdabar
        ops += 1 + 3                   # 1 - ell, the product of the move's four factors
        ops += 1 + 1                   # its sum, the state adjoint
    return ops


def test_adjoint_flops_are_those_executed():
    ts = workloads.adjoint_greeks()
    N, s = ts.n_rates, ts.steps_per_period
    nodes = [7 - m // 10 for m in range(N)]
    forward = bench.flops_per_path(ts, "full", nodes)
    jacobian = vjp = forward
    for c in range(N):
        for m in range(c + 1):
            jacobian += s * reverse_step(N - c, nodes[m])
        vjp += s * reverse_step(N - c, nodes[c])
    assert bench.adjoint_flops_per_path(ts, nodes) == jacobian
    assert bench.vjp_flops_per_path(ts, nodes) == vjp
