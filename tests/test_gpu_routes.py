"""Calls whose leading steps run as an ordered pass or as a chain from |0...0> and whose other steps
do not: amplitudes along the sequential order (projectors follow the gates), and states and
expectations in a graph replayed with other work between."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2108_06831_amd import Graph, Network, Observable, amplitudes, contract_path, expectation

pytestmark = pytest.mark.gpu
TOL = {"c64": 1e-5, "bf16x3": 1e-3}


def relerr(got, want):
    return float(np.linalg.norm(got - want) / np.linalg.norm(want))


@pytest.mark.parametrize("prec", ["c64", "bf16x3"])
@pytest.mark.parametrize("n,depth", [(6, 12), (13, 4), (14, 4), (15, 3), (17, 3)])
@pytest.mark.parametrize("fuse", [False, "dense"])
def test_sequential_amplitudes(n, depth, fuse, prec):
    rng = np.random.default_rng(n + depth)
    circ = workloads.brickwork(n, depth, rng)
    bits = workloads.random_bitstrings(n, 5, rng)
    net = Network.from_circuit(circ, output="amplitudes", n_bitstrings=len(bits), fuse=fuse)
    path = net.plan("sequential")
    want = oracle.amplitudes(oracle.statevector(circ), n, bits)
    for _ in range(2):
        got = amplitudes(net, path, bits, precision=prec).cpu().numpy()
        # a few amplitudes of 2^(-n/2): as a share of the state's norm per amplitude
        assert np.linalg.norm(got - want) < 4 * TOL[prec] * np.sqrt(len(bits)) * 2.0 ** (-n / 2)


@pytest.mark.parametrize("n", [9, 14, 15, 17])
def test_replays_after_other_work(n):
    """A captured contraction and expectation, replayed after eager calls on the same handles and
    workspace with other parameters in place."""
    edges = workloads.random_regular_graph(n if n % 2 == 0 else n + 1, 3, np.random.default_rng(n))
    edges = [e for e in edges if max(e) < n]
    circ = workloads.qaoa_circuit(n, edges, 2)
    mask, coeff = workloads.maxcut_observable(n, edges)
    net = Network.from_circuit(circ)
    path, obs = net.plan("sequential"), Observable(mask, coeff)
    rng = np.random.default_rng(n)
    p = torch.as_tensor(rng.uniform(0, np.pi, size=(1, circ.n_params)), device="cuda")
    state = torch.zeros(1, 1 << n, dtype=torch.complex64, device="cuda")
    out = torch.zeros(1, 1, dtype=torch.float64, device="cuda")
    ws = torch.zeros(1 << 26, dtype=torch.uint8, device="cuda")
    stream = torch.cuda.Stream()

    def calls():
        contract_path(net, path, p, out=state, workspace=ws, stream=stream)
        expectation([net], [path], [p], [obs], workspace=ws, out=out, stream=stream)
    stream.wait_stream(torch.cuda.current_stream())
    calls()
    stream.synchronize()
    graph = Graph(stream)
    with graph.capture():
        calls()
    for _ in range(3):
        host = rng.uniform(0, np.pi, size=(1, circ.n_params))
        p.copy_(torch.as_tensor(host))
        ws.fill_(255)
        state.zero_()
        out.zero_()
        torch.cuda.synchronize()
        graph.launch()
        stream.synchronize()
        want = oracle.statevector(circ, host[0])
        assert relerr(state[0].cpu().numpy(), want) < 1e-5
        e = oracle.circuit_expectation(circ, host[0], mask, coeff)
        assert abs(float(out) - e) < 1e-5 * max(abs(e), 1.0)
        calls()
        stream.synchronize()
