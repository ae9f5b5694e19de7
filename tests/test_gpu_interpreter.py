"""The interpreter of small contractions, lists in LDS and lists that do not fit there: whole circuits whose result it
writes in the caller's order, and lists whose results other products take up, over parameter batches.  Tolerances 1e-5
(complex64) and 1e-3 (BF16x3), normwise, as everywhere."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
TOL = {"c64": 1e-5, "bf16x3": 1e-3}


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
@pytest.mark.parametrize("kind", ["greedy", "search", "sequential"])
@pytest.mark.parametrize("n,layers", [(1, 3), (2, 9), (4, 1), (5, 7), (11, 5), (12, 9), (13, 4), (12, 30)])
def test_small_circuits(n, layers, kind, prec):
    from paper_2108_06831_amd import Network, contract_path
    rng = np.random.default_rng(10 * n + layers)
    if n == 1:
        circ = workloads.Circuit(1, [workloads.Gate("U3", (0,), (0.3 + i, 0.7, 0.2 * i)) for i in range(layers)])
    else:
        circ = workloads.brickwork(n, layers, rng)
    net = Network.from_circuit(circ, fuse=False)
    path = net.plan(kind)
    want = oracle.statevector(circ)
    for _ in range(2):  # the second on a workspace that holds the first's results
        got = contract_path(net, path, precision=prec)[0].cpu().numpy()
        e = float(np.linalg.norm(got - want) / np.linalg.norm(want))
        print(f"n={n} layers={layers} {kind} {prec}: {path.stats['n_small_steps']} of {path.stats['n_steps']} {e:.2e}", flush=True)
        assert e < TOL[prec]


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
def test_parameter_batches(prec):
    from paper_2108_06831_amd import Network, contract_path
    circ = workloads.hea_circuit(7, 3)
    net = Network.from_circuit(circ)
    path = net.plan("greedy")
    params = np.random.default_rng(3).uniform(0, 2 * np.pi, size=(5, circ.n_params))
    got = contract_path(net, path, params, batch=5, precision=prec).cpu().numpy()
    for b in range(5):
        want = oracle.statevector(circ, params[b])
        assert np.linalg.norm(got[b] - want) / np.linalg.norm(want) < TOL[prec]
