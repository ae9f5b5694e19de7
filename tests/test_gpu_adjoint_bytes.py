"""Bytes that kernel timing counts for a gradient's reverse sweep, per element and parameter vector."""
import numpy as np
import pytest

import workloads
from paper_2108_06831_amd import (Network, Observable, backward, profile_enable, profile_read, profile_reset,
                                  profile_select)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kind,per", [
    (10, "sequential", 16),  # forward and reverse in one launch: psi written and read
    (13, "sequential", 16),
    (10, "greedy", 8),       # psi from other launches: read
    (15, "sequential", None),  # several chunks: psi and lambda read and written by every pass
])
def test_bytes_of_the_reverse_sweep(n, kind, per):
    circ = workloads.hea_circuit(n, 2, True)
    net = Network.from_circuit(circ)
    path, obs = net.plan(kind), Observable(*workloads.zz_ring_observable(n, True))
    params = np.random.default_rng(n).uniform(0, 2 * np.pi, size=(3, circ.n_params))
    backward(net, path, params, obs, batch=3)
    profile_reset()
    profile_select(["adjoint"])
    profile_enable(True)
    backward(net, path, params, obs, batch=3)
    got = profile_read()["adjoint"]
    profile_enable(False)
    profile_select(None)
    if per is None:
        passes = got["bytes"] / (32.0 * 3 * 2 ** n)
        assert passes == int(passes) and passes >= 2
    else:
        assert got["launches"] == 1 and got["bytes"] == per * 3 * 2 ** n
