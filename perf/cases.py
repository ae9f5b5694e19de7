"""Performance cases: what users of this library have it do, through its public entry points.

A case is a dict of plain values.  ``listed()`` are the cases that are followed, ``draw(rng)`` gives more of the
same ranges, ``prepare(case, seed)`` makes what a program has in hand before the call (network, planned path,
device inputs, workspace), ``run(state)`` is one pass, ``work(case)`` the operations and bytes the path cannot do
without, and ``exact(case, seed)`` the same results in 64 bits from plain torch.

Kinds of cases:

  statevector   contract a circuit's network to its 2^n amplitudes (random brickwork circuits and the test circuit
                of Fig. 3.1), from a 4-qubit circuit to a 28-qubit state of 2 GiB;
  amplitudes    amplitudes of a list of bitstrings of a grid circuit (sampling and verification of random circuits);
  expectation   <C> of a batch of QAOA MaxCut circuits of mixed sizes, eager or replayed as one HIP graph;
  gradient      value and adjoint gradient of a hardware-efficient ansatz for a batch of parameter vectors
                (``backward``), or one training step through the autograd function;
  pair          one pairwise contraction of two tensors (``contract_pair``).
"""
import ctypes
import math

import numpy as np
import torch

import paper_2108_06831_amd as tnq
import workloads

DEVICE = "cuda"


def listed():
    return [
        # The smallest call: one small circuit's state, where launches and host time are everything.
        {"name": "state_10q_brickwork", "kind": "statevector", "circuit": "brickwork", "n": 10, "depth": 8,
         "fuse": "none", "plan": "greedy", "precision": "c64"},
        # An ordinary simulation of a mid-sized circuit of an odd qubit count, gate by gate in circuit order.
        {"name": "state_15q_sequential", "kind": "statevector", "circuit": "brickwork", "n": 15, "depth": 10,
         "fuse": "dense", "plan": "sequential", "precision": "c64"},
        # The benchmark's statevector: 24 qubits, depth 16, searched order, large matrix products.
        {"name": "state_24q_brickwork", "kind": "statevector", "circuit": "brickwork", "n": 24, "depth": 16,
         "fuse": "split", "plan": "search", "precision": "c64"},
        # The same in the split-precision mode.
        {"name": "state_24q_bf16x3", "kind": "statevector", "circuit": "brickwork", "n": 24, "depth": 16,
         "fuse": "split", "plan": "search", "precision": "bf16x3"},
        # The largest state: the Fig. 3.1 circuit at the largest size of its sweep, a 2 GiB result.
        {"name": "state_28q_fig31", "kind": "statevector", "circuit": "fig31", "n": 28, "depth": 4,
         "fuse": "split", "plan": "search", "precision": "c64"},
        # Verification of a random grid circuit: 4096 amplitudes of 32 qubits.
        {"name": "amps_4x8_4096", "kind": "amplitudes", "rows": 4, "cols": 8, "depth": 12, "count": 4096,
         "circuit_seed": 2108068312, "plan": "search", "precision": "c64"},
        # A smaller grid and a ragged number of bitstrings.
        {"name": "amps_4x6_1000", "kind": "amplitudes", "rows": 4, "cols": 6, "depth": 12, "count": 1000,
         "circuit_seed": 2108068312, "plan": "greedy", "precision": "c64"},
        # A share of the benchmark's QAOA batch (16 to 26 qubits), replayed as one HIP graph as its loop does.
        {"name": "qaoa_32_16to26", "kind": "expectation", "circuits": 32, "lo": 16, "hi": 26, "step": 2, "p": 4,
         "batch": 1, "graph": True, "precision": "c64"},
        # Small QAOA instances for several parameter vectors each, called eagerly by an optimiser.
        {"name": "qaoa_16_8to14", "kind": "expectation", "circuits": 16, "lo": 8, "hi": 14, "step": 2, "p": 3,
         "batch": 4, "graph": False, "precision": "c64"},
        # The benchmark's gradients: 20 qubits, 10 layers, 64 parameter vectors.
        {"name": "grad_20q_64", "kind": "gradient", "n": 20, "layers": 10, "batch": 64, "autograd": False,
         "precision": "c64"},
        # A mid-sized ansatz of an odd qubit count with an odd batch.
        {"name": "grad_13q_9", "kind": "gradient", "n": 13, "layers": 6, "batch": 9, "autograd": False,
         "precision": "c64"},
        # One pairwise contraction of permuted tensors with a batch mode, as a program with its own order calls it.
        {"name": "pair_4x1024x512x256", "kind": "pair", "b": 2, "m": 10, "n": 9, "k": 8, "order": 3,
         "precision": "c64"},
    ]


def draw(rng):
    def log2(lo, hi):
        return int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))

    prec = rng.choice(["c64", "c64", "c64", "bf16x3"])
    kind = rng.choice(["statevector", "statevector", "amplitudes", "expectation", "gradient", "gradient", "pair"])
    if kind == "statevector":
        if rng.random() < 0.5:
            n, depth, circuit = rng.randint(4, 25), rng.randint(2, 16), "brickwork"
        else:
            n, circuit = 2 * rng.randint(2, 13), "fig31"
            depth = rng.randint(2, 8 if n <= 24 else 5)
        fuse, plan = rng.choice([("split", "search"), ("split", "greedy"), ("none", "sequential"),
                                 ("dense", "sequential")])
        if n <= 10 and rng.random() < 0.5:
            fuse, plan = "none", "greedy"
        return {"kind": kind, "circuit": circuit, "n": n, "depth": depth, "fuse": fuse, "plan": plan,
                "precision": prec}
    if kind == "amplitudes":
        rows, cols = rng.choice([(2, 5), (3, 3), (3, 5), (3, 6), (4, 4), (4, 5), (3, 7), (4, 6)])
        return {"kind": kind, "rows": rows, "cols": cols, "depth": rng.randint(4, 12), "count": log2(1, 4096),
                "circuit_seed": rng.randint(1, 10 ** 6), "plan": rng.choice(["search", "greedy"]),
                "precision": prec}
    if kind == "expectation":
        lo = rng.choice([6, 8, 10, 12, 14, 16, 18])
        hi = min(24, lo + 2 * rng.randint(1, 4))
        return {"kind": kind, "circuits": log2(1, 32 if hi > 18 else 64), "lo": lo, "hi": hi, "step": 2,
                "p": rng.randint(1, 4), "batch": rng.choice([1, 1, 2, 5]) if hi <= 20 else 1,
                "graph": rng.random() < 0.5, "precision": prec}
    if kind == "gradient":
        n = rng.randint(4, 20)
        return {"kind": kind, "n": n, "layers": rng.randint(1, 8), "batch": log2(1, 64 if n <= 17 else 24),
                "autograd": rng.random() < 0.4, "precision": prec}
    m, n, k = rng.randint(3, 12), rng.randint(3, 12), rng.randint(1, 9)
    return {"kind": "pair", "b": rng.randint(0, 4), "m": m, "n": n, "k": k, "order": rng.randint(0, 999),
            "precision": prec}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _state_circuit(case, seed):
    rng = np.random.default_rng(seed)
    make = workloads.brickwork if case["circuit"] == "brickwork" else workloads.paper_test_circuit
    return make(case["n"], case["depth"], rng)


def _grid(case, seed):
    circ = workloads.grid_circuit(case["rows"], case["cols"], case["depth"],
                                  np.random.default_rng(case["circuit_seed"]))
    return circ, workloads.random_bitstrings(circ.n_qubits, case["count"], np.random.default_rng(seed))


def _sizes(case):
    """Qubit counts of a batch of circuits: all sizes of the range in turn, the same for every seed."""
    sizes = list(range(case["lo"], case["hi"] + 1, case["step"]))
    return [sizes[(i * 5 + i // len(sizes)) % len(sizes)] for i in range(case["circuits"])]


def _qaoa(case, seed):
    rng = np.random.default_rng(seed)
    out = []
    for n in _sizes(case):
        edges = workloads.random_regular_graph(n, 3, rng)
        p = case["p"]
        params = np.concatenate([rng.uniform(0.0, np.pi, size=(case["batch"], p)),
                                 rng.uniform(0.0, np.pi / 2, size=(case["batch"], p))], axis=1)
        out.append((workloads.qaoa_circuit(n, edges, p), workloads.maxcut_observable(n, edges), params))
    return out


def _ansatz(case, seed):
    rng = np.random.default_rng(seed)
    circ = workloads.hea_circuit(case["n"], case["layers"], case["n"] > 2)
    params = rng.uniform(0.0, 2.0 * np.pi, size=(case["batch"], circ.n_params))
    weights = rng.uniform(0.5, 1.5, size=case["batch"])
    return circ, workloads.zz_ring_observable(case["n"], case["n"] > 2), params, weights


def _pair(case, seed):
    """Modes of extent 2, 4 or 8 that make up the batch, m, n and k indices, in a shuffled order in each tensor."""
    rng = np.random.default_rng(case["order"])
    modes, ext = {"b": [], "m": [], "n": [], "k": []}, {}
    for what in "bmnk":
        left = case[what]
        while left:
            t = min(left, int(rng.integers(1, 4)))
            ext[len(ext)] = 1 << t
            modes[what].append(len(ext) - 1)
            left -= t
    a, b, c = (list(rng.permutation(np.array(modes["b"] + modes[x] + modes[y], dtype=int)))
               for x, y in (("m", "k"), ("k", "n"), ("m", "n")))
    a, b, c = ([int(v) for v in x] for x in (a, b, c))
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    ta, tb = (torch.randn([ext[v] for v in x], dtype=torch.complex64, device=DEVICE, generator=gen) for x in (a, b))
    return ta, a, tb, b, c


def prepare(case, seed):
    s = {"case": case}
    kind = case["kind"]
    if kind == "statevector":
        circ = _state_circuit(case, seed)
        s["net"] = tnq.Network.from_circuit(circ, fuse=False if case["fuse"] == "none" else case["fuse"])
        s["path"] = s["net"].plan(case["plan"])
        s["out"] = torch.empty(1, 1 << case["n"], dtype=torch.complex64, device=DEVICE)
        s["ws"] = torch.empty(s["path"].workspace_bytes(1), dtype=torch.uint8, device=DEVICE)
    elif kind == "amplitudes":
        circ, bits = _grid(case, seed)
        s["net"] = tnq.Network.from_circuit(circ, output="amplitudes", n_bitstrings=case["count"])
        s["path"] = s["net"].plan(case["plan"], max_log2_intermediate=28)
        s["bits"] = torch.as_tensor(bits.view(np.int64), device=DEVICE)
        s["out"] = torch.empty(case["count"], dtype=torch.complex64, device=DEVICE)
        s["ws"] = torch.empty(s["path"].workspace_bytes(1), dtype=torch.uint8, device=DEVICE)
    elif kind == "expectation":
        items = _qaoa(case, seed)
        s["nets"] = [tnq.Network.from_circuit(c) for c, _, _ in items]
        s["paths"] = [nt.plan("sequential") for nt in s["nets"]]
        s["obs"] = [tnq.Observable(*o) for _, o, _ in items]
        s["params"] = [torch.as_tensor(p, device=DEVICE) for _, _, p in items]
        s["out"] = torch.empty(len(items), case["batch"], dtype=torch.float64, device=DEVICE)
        n = len(items)
        handles = [(ctypes.c_void_p * n)(*[x.handle.value for x in s[k]]) for k in ("nets", "paths")]
        nbytes = tnq.lib().tn_expectation_workspace_bytes(*handles, n, case["batch"])
        s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)
        s["stream"] = None
        if case["graph"]:
            s["stream"] = torch.cuda.Stream()
            s["stream"].wait_stream(torch.cuda.current_stream())
            _expectation(s)  # creates the device-side tables before the capture
            s["stream"].synchronize()
            s["graph"] = tnq.Graph(s["stream"])
            with s["graph"].capture():
                _expectation(s)
    elif kind == "gradient":
        circ, obs, params, weights = _ansatz(case, seed)
        s["net"] = tnq.Network.from_circuit(circ)
        s["path"] = s["net"].plan("sequential")
        s["obs"] = tnq.Observable(*obs)
        s["params"] = torch.as_tensor(params, device=DEVICE)
        s["weights"] = torch.as_tensor(weights, device=DEVICE)
        nbytes = int(tnq.lib().tn_backward_workspace_bytes(s["net"].handle, s["path"].handle, case["batch"]))
        s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEVICE)
    else:
        s["a"], s["modes_a"], s["b"], s["modes_b"], s["modes_c"] = _pair(case, seed)
    return s


def _expectation(s):
    return tnq.expectation(s["nets"], s["paths"], s["params"], s["obs"], batch=s["case"]["batch"],
                           precision=s["case"]["precision"], workspace=s["ws"], out=s["out"], stream=s["stream"])


def run(s):
    case = s["case"]
    kind, prec = case["kind"], case["precision"]
    if kind == "statevector":
        return tnq.contract_path(s["net"], s["path"], precision=prec, out=s["out"], workspace=s["ws"])
    if kind == "amplitudes":
        return tnq.amplitudes(s["net"], s["path"], s["bits"], precision=prec, out=s["out"], workspace=s["ws"])
    if kind == "expectation":
        if not case["graph"]:
            return _expectation(s)
        # the parameters of the next pass are written on the current stream, and the results read there
        cur = torch.cuda.current_stream()
        s["stream"].wait_stream(cur)
        s["graph"].launch()
        cur.wait_stream(s["stream"])
        return s["out"]
    if kind == "gradient":
        if case["autograd"]:
            theta = s["params"].clone().requires_grad_(True)
            value = tnq.Expectation.apply(theta, s["net"], s["path"], s["obs"], prec)
            (value * s["weights"]).sum().backward()
            return value.detach(), theta.grad
        return tnq.backward(s["net"], s["path"], s["params"], s["obs"], batch=case["batch"], grad_out=s["weights"],
                            precision=prec, workspace=s["ws"])
    return tnq.contract_pair(s["a"], s["modes_a"], s["b"], s["modes_b"], s["modes_c"], precision=prec)


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
def work(case):
    """Inputs read once, outputs written once, and the arithmetic of the best known way to the result: a state is
    one product over its middle cut, with the bond its crossing gates make; a gate that is applied to a state of 2^n
    takes 8 2^n operations (a real or RX-like one-qubit gate), a layer of diagonal gates 6 2^n."""
    kind = case["kind"]
    if kind == "statevector":
        n, d = case["n"], case["depth"]
        per_cut = d // 2 if case["circuit"] == "brickwork" else d  # gates across the middle
        bond = min(max(per_cut, 1), n // 2)
        gates = n * d * (3 if case["circuit"] == "brickwork" else 2)
        return {"bytes": 8.0 * 2 ** n + 8.0 * gates, "flops": 8.0 * 2.0 ** (n + bond)}
    if kind == "amplitudes":
        n, d, c = case["rows"] * case["cols"], case["depth"], case["count"]
        bond = min(d * case["rows"] // 8, n // 2)  # one layer in four crosses the middle, on half of the rows' edges
        return {"bytes": 16.0 * c + 8.0 * n * d, "flops": 8.0 * c * 2.0 ** bond}
    if kind == "expectation":
        p, b = case["p"], case["batch"]
        flops = sum(b * 2.0 ** n * (p * (8.0 * n + 6.0) + 4.0) for n in _sizes(case))
        return {"bytes": float(case["circuits"] * b * 8 * (2 * p + 1) + sum(12 * n for n in _sizes(case))),
                "flops": flops}
    if kind == "gradient":
        n, la, b = case["n"], case["layers"], case["batch"]
        # forward: RY and one diagonal a layer; back: the same on two states, and a term for each RY (4) and RZ (1)
        flops = b * 2.0 ** n * la * ((8.0 * n + 6.0) * (4 if case["autograd"] else 3) + 5.0 * n)
        return {"bytes": 8.0 * b * (2 * 2 * n * la + 2), "flops": flops}
    m, n, k, b = (2.0 ** case[x] for x in "mnkb")
    return {"bytes": 8.0 * b * (m * k + k * n + m * n), "flops": 8.0 * b * m * n * k}


# ---------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------
_P = {"X": [[0, 1], [1, 0]], "Y": [[0, -1j], [1j, 0]], "Z": [[1, 0], [0, -1]]}


def _matrix(kind, t):
    """Gate matrix in complex128; angles t are tensors of one value per batch item (leading axis)."""
    c = torch.complex128
    if kind == "H":
        return torch.tensor([[1, 1], [1, -1]], dtype=c) / math.sqrt(2.0)
    if kind in ("SX", "SY", "SW"):
        px, py = (torch.tensor(_P[k], dtype=c) for k in "XY")
        p = {"SX": px, "SY": py, "SW": (px + py) / math.sqrt(2.0)}[kind]
        return ((1 + 1j) * torch.eye(2, dtype=c) + (1 - 1j) * p) / 2
    if kind == "CZ":
        return torch.diag(torch.tensor([1, 1, 1, -1], dtype=c))
    if kind == "CNOT":
        return torch.tensor([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0]], dtype=c)
    if kind in ("RX", "RY", "RZ", "MIXER"):
        p = torch.tensor(_P["X" if kind == "MIXER" else kind[1]], dtype=c)
        h = (t[0] if kind == "MIXER" else t[0] / 2).to(c).reshape(-1, 1, 1)
        return torch.cos(h) * torch.eye(2, dtype=c) - 1j * torch.sin(h) * p
    if kind == "U3":
        th, f, la = (x.to(c).reshape(-1) for x in t)
        co, si = torch.cos(th / 2), torch.sin(th / 2)
        return torch.stack([co, -torch.exp(1j * la) * si, torch.exp(1j * f) * si,
                            torch.exp(1j * (f + la)) * co], dim=1).reshape(-1, 2, 2)
    if kind == "ZZPHASE":
        e = torch.exp(-1j * t[0].to(c).reshape(-1))
        one = torch.ones_like(e)
        return torch.diag_embed(torch.stack([one, e, e, one], dim=1))
    raise ValueError(kind)


def _angles(g, params):
    """Angles of a gate as float64 tensors [batch] (params: [batch, n_params] on the host, or None)."""
    return [params[:, p] if p >= 0 else torch.tensor([a], dtype=torch.float64) for a, p in zip(g.angles, g.params)]


def _apply(psi, n, u, qubits):
    """psi [batch, 2^n] complex128 after the gate u ([., d, d], d = 2 or 4) on the qubits, in place."""
    u = u.to(psi.device)
    u = u.reshape(-1, u.shape[-2], u.shape[-1])
    v = psi.view([psi.shape[0]] + [2] * n)
    parts = []
    for i in range(u.shape[-1]):
        bits = [i] if len(qubits) == 1 else [i >> 1, i & 1]
        w = v
        for q, x in sorted(zip(qubits, bits), reverse=True):
            w = w.select(q + 1, x)
        parts.append(w)
    shape = [-1] + [1] * (parts[0].dim() - 1)
    nz = (u != 0).any(dim=0)
    if not bool((nz & ~torch.eye(u.shape[-1], dtype=torch.bool, device=u.device)).any()):  # diagonal
        one = (u == 1).all(dim=0)
        for i, w in enumerate(parts):
            if not bool(one[i, i]):
                w.mul_(u[:, i, i].reshape(shape))
        return psi
    old = [w.clone() for w in parts]
    for i, w in enumerate(parts):
        cols = [j for j in range(len(parts)) if bool(nz[i, j])]
        torch.mul(old[cols[0]], u[:, i, cols[0]].reshape(shape), out=w)
        for j in cols[1:]:
            w.addcmul_(old[j], u[:, i, j].reshape(shape).expand_as(w))
    return psi


def _simulate(circ, params=None, batch=1):
    psi = torch.zeros(batch, 1 << circ.n_qubits, dtype=torch.complex128, device=DEVICE)
    psi[:, 0] = 1
    for g in circ.gates:
        _apply(psi, circ.n_qubits, _matrix(g.kind, _angles(g, params)), g.qubits)
    return psi


def _diagonal(n, obs):
    x = torch.arange(1 << n, device=DEVICE)
    d = torch.zeros(1 << n, dtype=torch.float64, device=DEVICE)
    for m, c in zip(*obs):
        y = x & int(m)
        for s in (16, 8, 4, 2, 1):
            y = y ^ (y >> s)
        d += float(c) * (1.0 - 2.0 * (y & 1).double())
    return d


_GENERATOR = {"RY": ("Y", 0.5), "RZ": ("Z", 0.5)}


def _adjoint(circ, params, obs):
    """Values and gradients of <psi|D|psi> for a batch of parameter vectors."""
    n, batch = circ.n_qubits, params.shape[0]
    psi = _simulate(circ, params, batch)
    d = _diagonal(n, obs)
    value = (psi.abs().square() * d).sum(dim=1)
    lam = psi * d
    grad = torch.zeros(batch, circ.n_params, dtype=torch.float64, device=DEVICE)
    for g in reversed(circ.gates):
        if g.params and g.params[0] >= 0:
            name, scale = _GENERATOR[g.kind]
            q = g.qubits[0]
            p, la = (x.view(batch, 1 << q, 2, -1) for x in (psi, lam))
            p0, p1, l0, l1 = p[:, :, 0], p[:, :, 1], la[:, :, 0], la[:, :, 1]
            if name == "Z":
                t = ((l0.conj() * p0).imag - (l1.conj() * p1).imag).sum(dim=(1, 2))
            else:
                t = ((l0.conj() * (-1j * p1)).imag + (l1.conj() * (1j * p0)).imag).sum(dim=(1, 2))
            grad[:, g.params[0]] += 2.0 * scale * t
        u = _matrix(g.kind, _angles(g, params))
        u = u.reshape(-1, u.shape[-2], u.shape[-1]).transpose(1, 2).conj()
        _apply(psi, n, u, g.qubits)
        _apply(lam, n, u, g.qubits)
    return value, grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "statevector":
        return _simulate(_state_circuit(case, seed))
    if kind == "amplitudes":
        circ, bits = _grid(case, seed)
        if circ.n_qubits > 28:
            return None
        return _simulate(circ)[0][torch.as_tensor(bits.view(np.int64), device=DEVICE)]
    if kind == "expectation":
        rows = []
        for circ, obs, params in _qaoa(case, seed):
            psi = _simulate(circ, torch.as_tensor(params), case["batch"])
            rows.append((psi.abs().square() * _diagonal(circ.n_qubits, obs)).sum(dim=1))
        return torch.stack(rows)
    if kind == "gradient":
        circ, obs, params, weights = _ansatz(case, seed)
        step = max(1, (1 << 24) >> case["n"])
        p = torch.as_tensor(params)
        parts = [_adjoint(circ, p[i:i + step], obs) for i in range(0, case["batch"], step)]
        value, grad = (torch.cat(x) for x in zip(*parts))
        return value, grad * torch.as_tensor(weights, device=DEVICE)[:, None]
    a, modes_a, b, modes_b, modes_c = _pair(case, seed)
    ext = dict(zip(modes_a, a.shape)) | dict(zip(modes_b, b.shape))
    both = [m for m in modes_a if m in modes_b]
    batch, summed = [m for m in both if m in modes_c], [m for m in both if m not in modes_c]
    am, bn = [m for m in modes_a if m not in both], [m for m in modes_b if m not in both]

    def size(ms):
        return math.prod(ext[m] for m in ms)

    x = a.to(torch.complex128).permute([modes_a.index(m) for m in batch + am + summed])
    y = b.to(torch.complex128).permute([modes_b.index(m) for m in batch + summed + bn])
    x = x.reshape(size(batch), size(am), size(summed)).contiguous()
    y = y.reshape(size(batch), size(summed), size(bn)).contiguous()
    got = batch + am + bn
    z = torch.stack([torch.mm(u, v) for u, v in zip(x, y)]).reshape([ext[m] for m in got])
    return z.permute([got.index(m) for m in modes_c]).contiguous()
