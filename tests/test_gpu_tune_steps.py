"""The autotuner times the products that a call launches and no others."""
import numpy as np
import pytest

import oracle
import workloads
from paper_2108_06831_amd import Network, autotune, contract_path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
@pytest.mark.parametrize("n", [14, 15, 17])
def test_products_of_other_passes_are_left_alone(n, prec):
    """Ordered passes take the steps of a sequential circuit of 14 qubits, and all but the last one of
    15; a chain from |0...0> those of 17 qubits.  Their steps keep the launch shapes of products,
    which nothing runs."""
    circ = workloads.brickwork(n, 3, np.random.default_rng(n))
    net = Network.from_circuit(circ)
    path = net.plan("sequential")
    before = path.gemm_configs(prec)
    assert len(before) > 2 and path.stats["n_product_launches"] == (n == 15)
    rep = autotune(net, path, precision=prec, reps=2)
    assert rep["n_products"] == (n == 15)
    changed = [s for s, shape in path.gemm_configs(prec).items() if shape != before[s]]
    assert len(changed) == rep["n_changed"] and all(s == max(before) for s in changed)
    assert (rep["seconds_before"] > 0) == (n == 15)
    want = oracle.statevector(circ)
    got = contract_path(net, path, precision=prec)[0].cpu().numpy()
    assert np.linalg.norm(got - want) / np.linalg.norm(want) < (1e-5 if prec == "c64" else 1e-3)
