"""The run kernel (small states) and the tile kernel's rotation runs against
the CPU oracle, at the sizes where they can go wrong (needs an MI355X).

Tolerances as in test_gpu_parity: 1e-5 (complex64) and 1e-12 (complex128)
absolute, the bounds every comparison with the oracle holds.
"""

from __future__ import annotations

import numpy as np
import pytest

import oracle
import workloads as W
from parity import check, close

torch = pytest.importorskip("torch")
import paper_2301_03251_amd as Q  # noqa: E402

pytestmark = pytest.mark.gpu

TOL = {"c64": 1e-5, "c128": 1e-12}
ALL = (W.H, W.RX, W.RY, W.RZ, W.CNOT, W.CZ, W.CRX, W.CRY, W.CRZ)


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    Q.load()


def _dev(a, dtype):
    real = torch.float32 if dtype == "c64" else torch.float64
    return torch.from_numpy(np.ascontiguousarray(a)).to(device="cuda", dtype=real)


def _fb(runner, dtype, x, w, g):
    e, gx, gw = runner.forward_backward(_dev(x, dtype), _dev(w, dtype), _dev(g, dtype))
    torch.cuda.synchronize()
    return {"expz": e.cpu().double().numpy(), "grad_inputs": gx.cpu().double().numpy(),
            "grad_weights": gw.cpu().double().numpy()}


def _all_paths(n, gates, F, P, B, dtype, seed, embed=None, pauli_p=None, amplitude=False):
    """Forward + adjoint and forward alone, in the run kernel, and final states,
    each against the oracle."""
    x, w, g = W.random_inputs(B, F, P, n, seed=seed, dtype=dtype)
    if pauli_p is not None:
        x[:, F - len(pauli_p):] = np.random.default_rng(seed).random((B, len(pauli_p))).astype(x.dtype)
    x[0, 0] = 9.0  # well outside [-pi, pi]
    r = Q.Runner(Q.Circuit(n, gates, F, P, embed=embed, pauli_p=pauli_p), dtype)
    what = f"n={n} {dtype} B={B} G={len(gates)}"
    assert [r.c.call_kernel(dtype, B, m) for m in (Q.MODE_FWD, Q.MODE_FWD_BWD)] == ["runs", "runs"], what
    want = oracle.run(n, gates, x, w, grad_out=g, embed=embed, pauli_p=pauli_p, want_state=True)
    check(_fb(r, dtype, x, w, g), want, TOL[dtype], what)
    e = r.forward(_dev(x, dtype), _dev(w, dtype))
    psi = r.state(_dev(x, dtype), _dev(w, dtype))
    torch.cuda.synchronize()
    close(e.cpu().double().numpy(), want["expz"], TOL[dtype], what, "forward")
    close(psi.cpu().numpy(), want["state"], TOL[dtype], what, "state")


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", list(range(1, 13)))
def test_every_gate_kind(n, dtype):
    """Every size of the kernel's layouts (registers, lanes, wavefronts): runs,
    controlled runs, exchanges, signs and Pauli channels."""
    F, P = 4, 6
    # 4096 complex128 amplitudes of psi and lambda leave LDS for a short circuit only
    G = 30 if (n, dtype) == (12, "c128") else 30 + 8 * n
    gates = W.random_circuit(n, G, F, P, seed=900 + n, kinds=ALL)
    channels = np.array([[W.PAULI, q % n, -1, W.SRC_INPUT, F + q] for q in range(3)], np.int32)
    half = len(gates) // 2
    gates = np.concatenate([gates[:half], channels, gates[half:]])
    _all_paths(n, gates, F + 3, P, 3, dtype, seed=n, pauli_p=[[0.3, 0.3, 0.3], [0.2, 0.5, 0.1], [0.1, 0.1, 0.6]])


@pytest.mark.parametrize("n,G,B,dtype", [(5, 700, 2, "c128"), (10, 500, 1, "c64"), (3, 0, 2, "c128"), (9, 0, 1, "c128"),
                                         (6, 80, 1, "c128"), (7, 60, 1, "c64"), (11, 50, 1, "c128")])
def test_long_and_empty(n, G, B, dtype):
    """More steps than one chunk of 64 records, no gates at all, and a single
    sample of one or several wavefronts (whose weight gradients the kernel
    writes itself)."""
    _all_paths(n, W.random_circuit(n, G, 3, 4, seed=G + n, kinds=ALL), 3, 4, B, dtype, seed=n)


@pytest.mark.parametrize("n,dtype", [(2, "c64"), (6, "c128"), (9, "c64"), (12, "c128")])
def test_real_layers(n, dtype):
    """Layers of RY and H only, and one that a later RZ makes complex."""
    gates = np.concatenate([W.random_circuit(n, 60, 3, 5, seed=n, kinds=(W.RY, W.H, W.CZ, W.CNOT)),
                            W.random_circuit(n, 40, 3, 5, seed=n + 1, kinds=(W.RY, W.H, W.RZ, W.CZ))])
    _all_paths(n, gates, 3, 5, 4, dtype, seed=40 + n)


@pytest.mark.parametrize("kind", ["basis", "amplitude"])
@pytest.mark.parametrize("n,dtype", [(1, "c128"), (7, "c64"), (9, "c128"), (12, "c64")])
def test_embeddings(n, dtype, kind):
    F = n if kind == "basis" else 1 << n
    gates = W.random_circuit(n, 50, F, 4, seed=60 + n, kinds=ALL)
    _all_paths(n, gates, F, 4, 3, dtype, seed=61 + n,
               embed=(W.EMBED_BASIS if kind == "basis" else W.EMBED_AMPLITUDE, 0))


@pytest.mark.parametrize("n,dtype", [(4, "c64"), (7, "c128"), (10, "c128")])
def test_param_shift(n, dtype):
    """Shifted circuits, controlled rotations (each half shifted on its own)
    and chunks that cut a sample's circuits apart."""
    F, P, B = 3, 4, 3
    gates = W.random_circuit(n, 30, F, P, seed=80 + n, kinds=ALL)
    x, w, g = W.random_inputs(B, F, P, n, seed=81 + n, dtype=dtype)
    r = Q.Runner(Q.Circuit(n, gates, F, P), dtype)
    e, gx, gw = r.param_shift(_dev(x, dtype), _dev(w, dtype), _dev(g, dtype), max_chunk=29)
    torch.cuda.synchronize()
    got = {"expz": e.cpu().double().numpy(), "grad_inputs": gx.cpu().double().numpy(),
           "grad_weights": gw.cpu().double().numpy()}
    check(got, oracle.run(n, gates, x, w, grad_out=g), TOL[dtype], f"shift n={n} {dtype}")


@pytest.mark.parametrize("n,dtype,limit,circuit", [(11, "c128", 256, "random"), (12, "c64", 256, "random"),
                                                   (11, "c128", 512, "layers"), (12, "c64", 512, "layers")])
def test_batch_rule(n, dtype, limit, circuit):
    """On both sides of the batch from which the tile kernel takes the step: the
    rows of the smaller batch agree, the last row with the oracle, and the weight
    gradients of the larger batch are those of the smaller plus the last row's."""
    F, P = 3, 4
    gates = W.random_circuit(n, 40, F, P, seed=n, kinds=ALL) if circuit == "random" else run_layers(n, 2, F, P, seed=n)
    x, w, g = W.random_inputs(limit + 1, F, P, n, seed=n, dtype=dtype)
    r = Q.Runner(Q.Circuit(n, gates, F, P), dtype)
    assert (r.c.call_kernel(dtype, limit), r.c.call_kernel(dtype, limit + 1)) == ("runs", "tile")
    big, small = _fb(r, dtype, x, w, g), _fb(r, dtype, x[:limit], w, g[:limit])
    last = oracle.run(n, gates, x[-1:], w, grad_out=g[-1:])
    for k in ("expz", "grad_inputs"):
        close(big[k][:limit], small[k], 2 * TOL[dtype], f"n={n} {dtype}", k)  # each within TOL of the truth
        close(big[k][-1:], last[k], TOL[dtype], f"n={n} {dtype}", k)
    close(big["grad_weights"], small["grad_weights"] + last["grad_weights"], 2 * TOL[dtype], f"n={n} {dtype}", "grad_weights")


@pytest.mark.parametrize("n,dtype,limit,circuit", [(12, "c64", 512, "random"), (11, "c128", 512, "random"), (12, "c64", 1536, "layers"),
                                                   (11, "c128", 768, "layers"), (12, "c128", 256, "random"),
                                                   (12, "c128", 768, "layers")])
def test_batch_rule_forward(n, dtype, limit, circuit):
    """The same of the forward: <Z> of both kernels agrees, and the last rows
    with the oracle."""
    F, P = 3, 4
    gates = W.random_circuit(n, 40, F, P, seed=n, kinds=ALL) if circuit == "random" else run_layers(n, 2, F, P, seed=n)
    x, w, _ = W.random_inputs(limit + 1, F, P, n, seed=n, dtype=dtype)
    r = Q.Runner(Q.Circuit(n, gates, F, P), dtype)
    assert [r.c.call_kernel(dtype, limit + i, Q.MODE_FWD) for i in (0, 1)] == ["runs", "tile"]
    big, small = (r.forward(_dev(x[:rows], dtype), _dev(w, dtype)).cpu().double().numpy() for rows in (limit + 1, limit))
    close(big[:limit], small, 2 * TOL[dtype], f"n={n} {dtype}", "expz")
    close(big[-2:], oracle.run(n, gates, x[-2:], w)["expz"], TOL[dtype], f"n={n} {dtype}", "expz")


def run_layers(n, layers, F, P, seed):
    """Layers of two to four rotations per qubit (all orders, so some qubits
    have runs and others do not) and CNOTs, CZs over a brick."""
    rng = np.random.default_rng(seed)
    gates = []
    for _ in range(layers):
        for q in range(n):
            for kind in rng.choice([W.RX, W.RY, W.RZ], size=int(rng.integers(2, 5))):
                src = (W.SRC_INPUT, int(rng.integers(F))) if rng.random() < 0.3 else (W.SRC_WEIGHT, int(rng.integers(P)))
                gates.append((int(kind), q, -1) + src)
        gates += [(W.CNOT if rng.random() < 0.7 else W.CZ, a, b, 0, 0) for a, b in W.entangler_pairs(n, "brick")]
    return np.array(gates, np.int32)


@pytest.mark.parametrize("n,dtype,opts", [(13, "c64", {}), (14, "c128", {}), (15, "c64", dict(log_regs=5, log_threads=7)),
                                          (12, "c64", dict(log_regs=2, log_threads=8)),
                                          (12, "c128", dict(log_regs=3, log_threads=6, max_gates_per_pass=30))])
def test_tile_rotation_runs(n, dtype, opts):
    """Rotation runs of the tile plans, with and without the product prefix:
    forward + adjoint, exact states, and the plan without runs."""
    F, P, B = 4, 6, 2
    gates = run_layers(n, 3, F, P, seed=100 + n)
    x, w, g = W.random_inputs(B, F, P, n, seed=101 + n, dtype=dtype)
    x[0, 0], w[1] = 9.0, -7.5
    want = oracle.run(n, gates, x, w, grad_out=g, want_state=True)
    for extra in (dict(), dict(product_prefix=-1), dict(rz_groups=-1)):
        r = Q.Runner(Q.Circuit(n, gates, F, P, **opts, **extra), dtype)
        check(_fb(r, dtype, x, w, g), want, TOL[dtype], f"runs n={n} {dtype} {extra}")
        psi = r.state(_dev(x, dtype), _dev(w, dtype))
        torch.cuda.synchronize()
        close(psi.cpu().numpy(), want["state"], TOL[dtype], f"runs n={n} {dtype} {extra}", "state")


def test_tile_rotation_runs_param_shift():
    n, F, P, B = 13, 3, 5, 2
    gates = run_layers(n, 1, F, P, seed=7)
    x, w, g = W.random_inputs(B, F, P, n, seed=8, dtype="c128")
    r = Q.Runner(Q.Circuit(n, gates, F, P, product_prefix=-1), "c128")
    e, gx, gw = r.param_shift(_dev(x, "c128"), _dev(w, "c128"), _dev(g, "c128"), max_chunk=37)
    torch.cuda.synchronize()
    got = {"expz": e.cpu().numpy(), "grad_inputs": gx.cpu().numpy(), "grad_weights": gw.cpu().numpy()}
    check(got, oracle.run(n, gates, x, w, grad_out=g), 1e-12, "runs shift")


def test_captured_calls():
    """A captured forward + adjoint call (tables already on the device) replays
    to the eager results, for a run-kernel and a tile circuit."""
    for n in (9, 13):
        gates = W.random_circuit(n, 60, 3, 4, seed=n)
        x, w, g = (_dev(a, "c64") for a in W.random_inputs(4, 3, 4, n, seed=n, dtype="c64"))
        r = Q.Runner(Q.Circuit(n, gates, 3, 4), "c64")
        want = [t.clone() for t in r.forward_backward(x, w, g)]
        outs = tuple(torch.empty_like(t) for t in want)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            r.forward_backward(x, w, g, outs=outs)
        for _ in range(3):
            for t in outs:
                t.zero_()
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(outs, want):
                assert torch.equal(a, b)
            r.forward_backward(x, w, g)


@pytest.mark.parametrize("n", [10, 12])
def test_rounding(n):
    """Relative errors of complex64 in the 2-norm, over six sets of weights of
    eight layers of RY. An amplitude takes two roundings per run, 2^-24 / sqrt(6)
    of it in the root mean square, so <Z> is off by sqrt(2 N) of that after N
    independent ones, and the gradients, whose psi and lambda also come back, by
    sqrt(3) more. Errors common to all amplitudes (matrices that are not quite
    rotations) add up past it."""
    B, layers = 8, 8
    gates = W.layered_circuit(n, "ry", layers, (W.RY,), W.CZ, "ring")
    P = layers * n
    r = Q.Runner(Q.Circuit(n, gates, n, P), "c64")
    err = {"expz": [], "grad_inputs": [], "grad_weights": []}
    for seed in range(6):
        x, w, g = W.random_inputs(B, n, P, n, seed=seed, dtype="c64")
        want = oracle.run(n, gates, x, w, grad_out=g)
        got = _fb(r, "c64", x, w, g)
        for k in err:
            err[k].append(np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k]))
    once = 2.0 ** -24 / np.sqrt(6.0) * np.sqrt(2 * len(gates[gates[:, 0] == W.RY]))
    for k, bound in (("expz", once), ("grad_inputs", np.sqrt(3) * once), ("grad_weights", np.sqrt(3) * once)):
        rms = float(np.sqrt(np.mean(np.square(err[k]))))
        assert rms <= bound, f"{k}: {rms:.2e} > {bound:.2e}"


def test_tile_coefficients_complex128():
    """A tile rotation's coefficients are within a unit in the last place: an RY
    on |0> by shears leaves sin(theta / 2), as bound, on |1>."""
    n, B = 8, 4096
    r = Q.Runner(Q.Circuit(n, np.array([[W.RY, 0, -1, W.SRC_INPUT, 0]], np.int32), 1, 0, force_tiled=1,
                           product_prefix=-1), "c128")
    x = np.random.default_rng(3).uniform(-np.pi, np.pi, (B, 1))
    psi = r.state(_dev(x, "c128"), None)
    torch.cuda.synchronize()
    want = np.sin(x[:, 0].astype(np.longdouble) / 2)
    ulps = np.abs(psi.real[:, 1].cpu().numpy().astype(np.longdouble) - want) / np.spacing(np.abs(want).astype(np.float64))
    assert float(ulps.max()) <= 1.0


# complex64, 2000 gates: an amplitude takes up to 4000 roundings of 2^-24 / sqrt(6)
# in the root mean square, 1.5e-6 of it together, psi and lambda each; ten times
# both at one value. complex128 keeps its bound.
LONG = {"c64": 3e-5, "c128": 1e-12}


@pytest.mark.parametrize("n,G,B,dtype,kernels", [
    (7, 2000, 3, "c128", ("whole", "whole")), (6, 2000, 3, "c64", ("whole", "whole")),
    (7, 1200, 2, "c64", ("runs", "whole")), (4, 1000, 2, "c128", ("runs", "whole")),
    (6, 400, 2100, "c64", ("whole", "whole"))])
def test_long_small_circuits(n, G, B, dtype, kernels):
    """Below 8 qubits: circuits too long for the run kernel's tables, some only
    with a backward (the one-wavefront kernel takes the rest), and many forward
    circuits on request (the LDS kernel)."""
    F, P = 100, 400
    gates = W.random_circuit(n, G, F, P, seed=G + n, kinds=ALL)
    circ = Q.Circuit(n, gates, F, P, **({"force_tiled": -1} if B > 2000 else {}))
    assert tuple(circ.call_kernel(dtype, B, m) for m in (Q.MODE_FWD, Q.MODE_FWD_BWD)) == kernels
    x, w, g = W.random_inputs(B, F, P, n, seed=G, dtype=dtype)
    r = Q.Runner(circ, dtype)
    want = oracle.run(n, gates, x, w, grad_out=g)
    check(_fb(r, dtype, x, w, g), want, LONG[dtype], f"n={n} {dtype} G={G}")
    e = r.forward(_dev(x, dtype), _dev(w, dtype))
    torch.cuda.synchronize()
    close(e.cpu().double().numpy(), want["expz"], LONG[dtype], f"n={n} {dtype} G={G}", "forward")


@pytest.mark.parametrize("n,dtype,limit", [(9, "c64", 512), (9, "c128", 512), (6, "c64", 1024)])
def test_lds_rule(n, dtype, limit):
    """On both sides of the batch up to which a long circuit keeps the run
    kernel: rows agree, and the weight gradients of the larger batch are those of
    the smaller plus the last row's (from the oracle)."""
    F, P = 100, 300
    gates = W.random_circuit(n, 400, F, P, seed=n, kinds=ALL)
    circ = Q.Circuit(n, gates, F, P)
    other = "tile" if n >= 8 else "whole"
    assert (circ.call_kernel(dtype, limit), circ.call_kernel(dtype, limit + 1)) == ("runs", other)
    x, w, g = W.random_inputs(limit + 1, F, P, n, seed=n, dtype=dtype)
    r = Q.Runner(circ, dtype)
    big, small = _fb(r, dtype, x, w, g), _fb(r, dtype, x[:limit], w, g[:limit])
    last = oracle.run(n, gates, x[-1:], w, grad_out=g[-1:])
    for k in ("expz", "grad_inputs"):
        close(big[k][:limit], small[k], 2 * TOL[dtype], f"n={n} {dtype}", k)
        close(big[k][-1:], last[k], TOL[dtype], f"n={n} {dtype}", k)
    close(big["grad_weights"], small["grad_weights"] + last["grad_weights"], 2 * TOL[dtype], f"n={n} {dtype}", "grad_weights")


@pytest.mark.parametrize("n", [9, 13])
def test_first_call_does_not_wait(n):
    """The first call of a handle returns while the stream is busy, calls on
    other streams do not wait for its tables, and all results agree with those
    of later calls."""
    gates = W.random_circuit(n, 60, 3, 4, seed=n)
    x, w, g = (_dev(a, "c64") for a in W.random_inputs(4, 3, 4, n, seed=n, dtype="c64"))
    r, other = (Q.Runner(Q.Circuit(n, gates, 3, 4), "c64") for _ in range(2))
    want = [t.clone() for t in other.forward_backward(x, w, g)]
    side_r = Q.Runner(r.c, "c64")  # the same handle, a workspace of its own
    for q in (r, side_r):
        q.workspace(4, Q.MODE_FWD_BWD)
    side, busy, done = torch.cuda.Stream(), torch.cuda.Event(), torch.cuda.Event()
    torch.cuda.synchronize()
    torch.cuda._sleep(1 << 28)  # about 0.1 s
    busy.record()
    got = r.forward_backward(x, w, g)
    assert not busy.query()
    with torch.cuda.stream(side):
        got_side = side_r.forward_backward(x, w, g)
        done.record()
    done.synchronize()
    assert not busy.query()
    torch.cuda.synchronize()
    again = r.forward_backward(x, w, g)
    torch.cuda.synchronize()
    for a, b, c, d in zip(want, got, got_side, again):
        assert torch.equal(a, b) and torch.equal(a, c) and torch.equal(a, d)


@pytest.mark.parametrize("n,dtype", [(6, "c64"), (9, "c128"), (13, "c64")])
def test_first_call_captured(n, dtype):
    """A handle whose first call is captured (its tables go to the workspace in
    the graph): every replay gives the eager results, with eager calls between."""
    gates = W.random_circuit(n, 60, 3, 4, seed=n)
    x, w, g = (_dev(a, dtype) for a in W.random_inputs(4, 3, 4, n, seed=n, dtype=dtype))
    eager = Q.Runner(Q.Circuit(n, gates, 3, 4), dtype)
    want = [t.clone() for t in eager.forward_backward(x, w, g)]
    r = Q.Runner(Q.Circuit(n, gates, 3, 4), dtype)
    r.workspace(4, Q.MODE_FWD_BWD_KEEP)
    outs = tuple(torch.empty_like(t) for t in want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        r.forward_backward(x, w, g, outs=outs)
    for _ in range(4):
        for t in outs:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs, want))
        mine = Q.Runner(r.c, dtype).forward_backward(x, w, g)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(mine, want))
