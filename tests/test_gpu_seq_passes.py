"""Ordered gate passes over small states (sequential orders of 5 to 15 qubits,
reverse sweeps of 5 to 17): statevectors, expectations and gradients against
the FP64 oracle in both precisions, over every gate kind, at the edges of the
chunk sizes (chunks of fewer than 64 threads, one chunk, several chunks and
passes) and over parameter batches.  Tolerances: 1e-5 (complex64) and 1e-3
(BF16x3), normwise, as everywhere; gradients relative to max(norm, 1)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
TOL = {"c64": 1e-5, "bf16x3": 1e-3}
SIZES = [5, 6, 9, 10, 11, 12, 13, 14, 15]


def relerr(got, want):
    return float(np.linalg.norm(np.asarray(got) - np.asarray(want)) / np.linalg.norm(np.asarray(want)))


def start(n):
    """A first layer that leaves no amplitude zero and no symmetry."""
    return [workloads.Gate("U3", (q,), (0.3 + 0.2 * q, 0.7 - 0.1 * q, 0.4 * q)) for q in range(n)]


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("fuse", [False, "dense"])
def test_statevector_every_kind(n, prec, fuse):
    from paper_2108_06831_amd import Network, contract_path
    circ = workloads.random_circuit(n, 120, np.random.default_rng(n))
    circ.gates = start(n) + circ.gates
    net = Network.from_circuit(circ, fuse=fuse)
    got = contract_path(net, net.plan("sequential"), precision=prec)[0].cpu().numpy()
    e = relerr(got, oracle.statevector(circ))
    print(f"n={n} {prec} fuse={fuse}: {e:.2e}", flush=True)
    assert e < TOL[prec]


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
def test_expectations_of_mixed_sizes(prec):
    """Circuits of every size in one call, two parameter vectors each, called twice (the
    second call on the same workspace), some with more gates than one window of LDS holds."""
    from paper_2108_06831_amd import Network, Observable, expectation
    nets, paths, params, obs, want = [], [], [], [], []
    for i, n in enumerate([6, 8, 10, 12, 14, 16, 8, 13, 15]):
        rng = np.random.default_rng(50 + i)
        if n % 2 == 0:
            circ = workloads.qaoa_circuit(n, workloads.random_regular_graph(n, 3, rng), 3 if i != 2 else 24)
        else:
            circ = workloads.hea_circuit(n, 3)
        m, c = workloads.zz_ring_observable(n)
        m, c = np.concatenate([m, np.array([1, 0], dtype=np.uint64)]), np.concatenate([c, [0.7, 0.25]])
        p = rng.uniform(0, 2 * np.pi, size=(2, circ.n_params))
        nets.append(Network.from_circuit(circ))
        paths.append(nets[-1].plan("sequential"))
        params.append(p)
        obs.append(Observable(m, c))
        want.append([oracle.circuit_expectation(circ, p[b], m, c) for b in range(2)])
    for _ in range(2):
        got = expectation(nets, paths, params, obs, batch=2, precision=prec).cpu().numpy()
        e = np.max(np.abs(got - np.array(want)) / np.maximum(np.abs(np.array(want)), 1.0))
        print(f"{prec}: {e:.2e}", flush=True)
        assert e < TOL[prec]


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
@pytest.mark.parametrize("n", SIZES + [16, 17])
def test_gradients_every_kind(n, prec):
    from paper_2108_06831_amd import Network, Observable, backward
    rng = np.random.default_rng(900 + n)
    circ = workloads.random_circuit(n, 90, rng, n_params=7)
    circ.gates = start(n) + circ.gates
    m, c = workloads.zz_ring_observable(n)
    m, c = np.concatenate([m, np.array([1 << (n - 1), 1], dtype=np.uint64)]), np.concatenate([c, [0.7, -1.3]])
    params = rng.uniform(0, 2 * np.pi, size=(3, circ.n_params))
    w = rng.uniform(0.5, 1.5, size=3)
    net = Network.from_circuit(circ)
    value, grad = backward(net, net.plan("sequential"), params, Observable(m, c), batch=3, grad_out=w, precision=prec)
    value, grad = value.cpu().numpy(), grad.cpu().numpy()
    for b in (0, 2):
        want = oracle.circuit_expectation(circ, params[b], m, c)
        assert abs(value[b] - want) / max(abs(want), 1.0) < TOL[prec]
        g = w[b] * oracle.param_shift_gradient(circ, params[b], m, c)
        e = np.linalg.norm(grad[b] - g) / max(np.linalg.norm(g), 1.0)
        print(f"n={n} {prec} vector {b}: {e:.2e}", flush=True)
        assert e < TOL[prec]


def test_long_ansatz_takes_several_windows():
    """More gates than one window of LDS holds, forward and back."""
    from paper_2108_06831_amd import Network, Observable, backward
    n = 9
    circ = workloads.hea_circuit(n, 40)
    circ.gates = start(n) + circ.gates
    rng = np.random.default_rng(3)
    params = rng.uniform(0, 2 * np.pi, size=(1, circ.n_params))
    m, c = workloads.zz_ring_observable(n)
    net = Network.from_circuit(circ)
    value, grad = backward(net, net.plan("sequential"), params, Observable(m, c), batch=1)
    which = [0, 1, 17, circ.n_params // 2, circ.n_params - 2, circ.n_params - 1]
    g = oracle.param_shift_gradient(circ, params[0], m, c, which=which)
    got = grad.cpu().numpy()[0]
    assert np.max(np.abs(got[which] - g[which])) < 1e-5 * max(np.linalg.norm(got), 1.0)
    assert abs(float(value[0]) - oracle.circuit_expectation(circ, params[0], m, c)) < 1e-5 * n


@pytest.mark.parametrize("batch", [1, 3])
def test_captured_expectations_of_many_sizes(batch):
    """Circuits of one chunk and larger ones in one captured call, so that both have stream lanes of their own, and
    more of one chunk than one launch fills: replays, with new parameters between them, against the eager call."""
    import torch
    from paper_2108_06831_amd import Graph, Network, Observable, expectation
    nets, paths, params, obs = [], [], [], []
    for i in range(26):
        n = [10, 12, 14, 16, 8, 10][i % 6]
        rng = np.random.default_rng(i)
        edges = workloads.random_regular_graph(n, 3, rng)
        circ = workloads.qaoa_circuit(n, edges, 2)
        nets.append(Network.from_circuit(circ))
        paths.append(nets[-1].plan("sequential"))
        params.append(torch.as_tensor(rng.uniform(0, 2, size=(batch, circ.n_params)), device="cuda"))
        obs.append(Observable(*workloads.maxcut_observable(n, edges)))
    want = expectation(nets, paths, params, obs, batch=batch).clone()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    ws = torch.empty(1 << 28, dtype=torch.uint8, device="cuda")
    out = torch.empty_like(want)
    expectation(nets, paths, params, obs, batch=batch, workspace=ws, out=out, stream=stream)
    torch.cuda.synchronize()
    graph = Graph(stream)
    with graph.capture():
        expectation(nets, paths, params, obs, batch=batch, workspace=ws, out=out, stream=stream)
    for k in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.launch()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        for p in params:
            p.add_(0.1)
        want = expectation(nets, paths, params, obs, batch=batch).clone()
