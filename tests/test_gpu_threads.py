"""Calls on one plan from two threads, each on a stream of its own: the inspection calls and the
training data make their 64-node table in buffers of their own, so pricing passes beside
them neither see nor touch it.  (Every pass writes the same set-up tables; the pricing results
belong to one thread.)"""
import threading

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("which", ["tables", "generate"])
def test_passes_beside_calls_that_hold_the_64_node_table(gpu_lib, which):
    import torch
    ts = workloads.learned_drift()
    n, errors = 1000, []
    with gpu_lib.Plan(ts, max_paths=n) as plan, gpu_lib.Mlp(seed=1) as net:
        plan.execute(gpu_lib.FULL, n, seed=3)
        price = plan.results()["price"]
        tables = plan.tables()

        def passes(stream):
            for _ in range(60):
                plan.execute(gpu_lib.FULL, n, seed=3, stream=stream)
                if not np.array_equal(plan.results(stream=stream)["price"], price):
                    errors.append("price")

        def inspections(stream):
            for _ in range(20):
                if which == "tables":
                    got = plan.tables(stream=stream)
                    errors.extend(k for k in tables if not np.array_equal(got[k], tables[k]))
                else:
                    net.generate(plan, 64, 4, seed=5, stream=stream)

        def run(f, stream):
            try:
                f(stream)
            except Exception as e:  # noqa: BLE001 (a thread's exception ends only the thread)
                errors.append(repr(e))

        threads = [threading.Thread(target=run, args=(f, torch.cuda.Stream()))
                   for f in (passes, inspections)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    assert not errors, errors
