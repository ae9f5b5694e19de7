"""Gate passes in register form (states of 2^16 or more elements, complex64):
statevectors, expectations and adjoint gradients against the FP64 oracle, on
circuits whose segments hold every operation of that form (dense one-qubit
gates of each shape, sign and unit diagonals with none, one or two bits in the
registers, count groups), at the smallest states that take it, over parameter
batches.  Tolerance: 1e-5 normwise, the library's bound for complex64 (about
80 roundings of 2^-24 along the deepest wire leave 5e-6)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-5

DIAGONAL = ["RZ", "S", "T", "Z", "CZ", "CPHASE", "ZZPHASE"]
REAL = ["H", "RY", "X"]
RXLIKE = ["RX", "MIXER", "Y"]
GENERIC = ["U3", "SX", "SW"]


def relerr(got, want):
    return float(np.linalg.norm(np.asarray(got) - np.asarray(want)) / np.linalg.norm(np.asarray(want)))


@pytest.mark.parametrize("n", [16, 17, 19])
@pytest.mark.parametrize("kinds", [REAL + DIAGONAL, RXLIKE + DIAGONAL, GENERIC + DIAGONAL, REAL + RXLIKE + GENERIC])
def test_statevector(n, kinds):
    from paper_2108_06831_amd import Network, contract_path
    circ = workloads.random_circuit(n, 150, np.random.default_rng(100 * n + len(kinds)), kinds=kinds)
    # every qubit off the axes first, so that no amplitude stays zero
    circ.gates = [workloads.Gate("H", (q,)) for q in range(n)] + circ.gates
    net = Network.from_circuit(circ)
    path = net.plan("sequential")
    assert path.stats["n_sweep_steps"] > 100
    got = contract_path(net, path)[0].cpu().numpy()
    e = relerr(got, oracle.statevector(circ))
    print(f"n={n} {kinds[0]}: {e:.2e}", flush=True)
    assert e < TOL


@pytest.mark.parametrize("n", [16, 18])
def test_qaoa_expectation_batch(n):
    """Count groups, and edges left alone in their segment, for three parameter vectors."""
    from paper_2108_06831_amd import Network, Observable, expectation
    rng = np.random.default_rng(n)
    edges = workloads.random_regular_graph(n, 3, rng)
    circ = workloads.qaoa_circuit(n, edges, 3)
    m, c = workloads.maxcut_observable(n, edges)
    params = rng.uniform(0, np.pi, size=(3, circ.n_params))
    net = Network.from_circuit(circ)
    got = expectation([net], [net.plan("sequential")], [params], [Observable(m, c)], batch=3).cpu().numpy()[0]
    want = [oracle.circuit_expectation(circ, p, m, c) for p in params]
    assert np.max(np.abs(got - want) / np.maximum(np.abs(want), 1.0)) < TOL


@pytest.mark.parametrize("n,layers", [(18, 3), (19, 2)])
@pytest.mark.parametrize("dense", ["RY", "RX", "MIXER"])
def test_gradients(n, layers, dense):
    """Ansatz layers of one dense and two diagonal gates per qubit and a CZ ring, a
    Z on some wires, two parameter vectors: the gradient of sampled angles by
    the exact parameter shift."""
    from paper_2108_06831_amd import Network, Observable, backward
    rng = np.random.default_rng(7 * n + layers)
    gates, k = [], 0
    for _ in range(layers):
        for q in range(n):
            gates += [workloads.Gate("H", (q,)), workloads.Gate(dense, (q,), (0.0,), (k,)),
                      workloads.Gate("RZ", (q,), (0.0,), (k + 1,)), workloads.Gate("S", (q,))]
            k += 2
        gates += [workloads.Gate("CZ", (q, (q + 1) % n)) for q in range(n)]
        gates += [workloads.Gate("Z", (q,)) for q in range(0, n, 3)]
    circ = workloads.Circuit(n, gates, k)
    m, c = workloads.zz_ring_observable(n)
    params = rng.uniform(0, 2 * np.pi, size=(2, k))
    net = Network.from_circuit(circ)
    value, grad = backward(net, net.plan("sequential"), params, Observable(m, c), batch=2)
    value, grad = value.cpu().numpy(), grad.cpu().numpy()
    which = [int(x) for x in rng.choice(k, size=6, replace=False)]
    for b in range(2):
        assert abs(value[b] - oracle.circuit_expectation(circ, params[b], m, c)) < TOL * n
        g = oracle.param_shift_gradient(circ, params[b], m, c, which=which)
        got = np.array([grad[b][i] for i in which])
        want = np.array([g[i] for i in which])
        # normwise over the whole gradient, of which the sample is a part; RX and MIXER layers
        # after H leave every derivative zero, where the error counts against 1 as a scalar's does
        e = np.linalg.norm(got - want) / max(np.linalg.norm(grad[b]) * np.sqrt(len(which) / k), 1.0)
        print(f"n={n} {dense} vector {b}: {e:.2e}", flush=True)
        assert e < TOL


@pytest.mark.parametrize("n,layers", [(18, 3), (19, 2)])
@pytest.mark.parametrize("dense", ["RX", "MIXER"])
def test_gradients_of_x_generators(n, layers, dense):
    """RY layers between those of X generators, so that every derivative differs from zero: gradients of
    angles of each kind by the exact parameter shift, each kind's normwise, two parameter vectors."""
    from paper_2108_06831_amd import Network, Observable, backward
    rng = np.random.default_rng(11 * n + layers)
    gates, kinds = [], []
    for layer in range(layers):
        for kind in ("RY", dense, "RZ"):
            for q in range(n):
                gates.append(workloads.Gate(kind, (q,), (0.0,), (len(kinds),)))
                kinds.append(kind)
        gates += [workloads.Gate("CZ", (q, (q + 1) % n)) for q in range(n)]
    gates += [workloads.Gate("RY", (q,), (0.3 + 0.1 * q,)) for q in range(n)]
    circ = workloads.Circuit(n, gates, len(kinds))
    m, c = workloads.zz_ring_observable(n)
    params = rng.uniform(0.2, np.pi - 0.2, size=(2, circ.n_params))
    net = Network.from_circuit(circ)
    path = net.plan("sequential")
    value, grad = backward(net, path, params, Observable(m, c), batch=2)
    value, grad = value.cpu().numpy(), grad.cpu().numpy()
    for b in range(2):
        assert abs(value[b] - oracle.circuit_expectation(circ, params[b], m, c)) < TOL * n
        for kind in ("RY", dense, "RZ"):
            mine = [i for i, x in enumerate(kinds) if x == kind]
            which = [int(x) for x in rng.choice(mine, size=4, replace=False)]
            g = oracle.param_shift_gradient(circ, params[b], m, c, which=which)
            want = np.array([g[i] for i in which])
            got = np.array([grad[b][i] for i in which])
            size = np.linalg.norm(grad[b][mine]) * np.sqrt(len(which) / len(mine))
            print(f"n={n} {dense} {kind} vector {b}: oracle norm {np.linalg.norm(want):.2f}, "
                  f"error {np.linalg.norm(got - want):.2e}", flush=True)
            assert np.linalg.norm(want) > 0.05  # (a term left out, or its factor wrong, would show)
            assert np.linalg.norm(got - want) < TOL * max(size, 1.0)
