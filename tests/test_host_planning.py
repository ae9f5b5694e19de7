"""Host cost of planning.  Times are the least of several runs, compared between
plans made in the same process, so that the machine's speed does not enter."""
import time

import numpy as np
import pytest

import workloads
from paper_2108_06831_amd import Network


def least_seconds(fn, runs=9):
    best = float("inf")
    for _ in range(runs):
        t = time.perf_counter()
        fn()
        best = min(best, time.perf_counter() - t)
    return best


def qaoa_network(n):
    rng = np.random.default_rng(n)
    return Network.from_circuit(workloads.qaoa_circuit(n, workloads.random_regular_graph(n, 3, rng), 3))


@pytest.mark.parametrize("n", [8, 10, 12])
def test_ordered_passes_plan_no_interpreter_tables(n):
    """A sequential circuit of at most 12 qubits is all interpreter steps by size, but runs as one
    ordered pass.  At 14 qubits most steps are too large for the interpreter, so that plan never had
    its tables: the smaller circuits, with fewer gates, must take less time to plan (0.25 to 0.5 of it, and 0.8 to 3.4 with the tables)."""
    small, large = qaoa_network(n), qaoa_network(14)
    assert least_seconds(lambda: small.plan("sequential")) <= 0.75 * least_seconds(lambda: large.plan("sequential"))
