"""Greeks passes in a captured graph: the Jacobian's sweeps fork to side streams, made on the
first Jacobian of a plan, and join the captured stream.  Every replay, with eager passes of the
same plan between them, equals the eager results bit for bit.  The plan's buffers exist before
the capture (a vector-Jacobian product has run); `warm` runs a Jacobian before it too."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("warm", [False, True])
def test_replays_equal_eager_passes(gpu_lib, warm):
    import torch
    N, P = 12, 5000
    ts = workloads.make_structure(N, 0.25, 0.03 + 0.001 * np.arange(N), 3,
                                  workloads.exp_decay_vol(), [1.0])

    def empty(*size):
        return torch.empty(*size, dtype=torch.float64, device="cuda")

    with gpu_lib.Plan(ts, max_paths=P) as plan:
        w = torch.linspace(-1.0, 2.0, N, dtype=torch.float64, device="cuda")
        plan.greeks_vjp_dev(P, w, seed=1)
        if warm:
            plan.greeks(P, seed=1)
        torch.cuda.synchronize()
        out = [empty(N), empty(N, N), empty(N, N), empty(N), empty(N), empty(N), empty(N, 1)]

        def work():
            stream = torch.cuda.current_stream()
            plan.greeks(P, seed=2, stream=stream)
            plan.greeks_results_dev(*out[:3], stream=stream)
            plan.greeks_vjp_dev(P, w, seed=2, stream=stream)
            plan.greeks_vjp_results_dev(*out[3:6], stream=stream)
            plan.execute(gpu_lib.FULL, P, seed=2, stream=stream)
            plan.results_dev(price=out[6], stream=stream)

        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            work()
        work()
        torch.cuda.synchronize()
        ref = [o.clone() for o in out]
        for _ in range(4):
            for o in out:
                o.fill_(float("nan"))
            plan.execute(gpu_lib.FULL, 1000, seed=9)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(out, ref))
