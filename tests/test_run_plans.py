"""The run kernel's plans, on the CPU: every step list carried out on the host
(forward and back) equals the circuit's gates applied one by one. Covers every
gate kind, controlled rotations, Pauli channels, embeddings and every qubit
count the kernel takes, and reads no table outside its bounds (g++ sanitizers)."""

from __future__ import annotations

import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2301_03251_amd", "csrc")
ALL = (W.H, W.RX, W.RY, W.RZ, W.CNOT, W.CZ, W.CRX, W.CRY, W.CRZ)


def _record(f, n, gates, F, P, embed=(0, 0), pauli_p=None):
    gates = np.ascontiguousarray(gates, np.int32).reshape(-1, 5)
    pp = np.zeros((0, 3)) if pauli_p is None else np.asarray(pauli_p, np.float64).reshape(-1, 3)
    np.array([n, gates.shape[0], F, P, embed[0], embed[1], pp.shape[0], 1], np.int32).tofile(f)
    gates.tofile(f)
    np.ascontiguousarray(pp, np.float64).tofile(f)


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_run_plans_on_the_host(tmp_path):
    path = str(tmp_path / "circuits.bin")
    with open(path, "wb") as f:
        for name in ("4q", "10q", "qae"):
            wl = W.get(name)
            _record(f, wl.n, wl.gates(), wl.n_inputs, wl.n_weights, embed=getattr(wl, "embed", None) or (0, 0))
        for n in range(1, 13):
            for seed in range(6):
                kinds = [ALL, (W.RX, W.RY, W.RZ, W.CNOT), (W.H, W.RZ, W.CZ, W.RY), (W.CRX, W.CRY, W.CRZ, W.RZ, W.RX),
                         (W.CNOT, W.CZ, W.RZ, W.RX), (W.CNOT, W.CRY, W.H, W.RY)][seed]
                _record(f, n, W.random_circuit(n, 12 * n + 10, 4, 6, seed=100 * n + seed, kinds=kinds), 4, 6,
                        embed=(0, 0))
            layered = W.layered_circuit(n, "h_rz" if n % 2 else "ry", 3, (W.RY, W.RZ), W.CZ if n % 2 else W.CNOT,
                                        ("ring", "linear", "brick")[n % 3])
            noisy, pp, k = W.with_depolarizing(layered, n, n, 0.3, every=max(len(layered) // 4, 1))
            _record(f, n, noisy, n + k, 6 * n, pauli_p=pp)
            _record(f, n, layered, max(n, 1), 6 * n, embed=(W.EMBED_BASIS, 0))
            _record(f, n, W.random_circuit(n, 60, 1 << n, 6, seed=n, kinds=ALL), 1 << n, 6,
                    embed=(W.EMBED_AMPLITUDE, 0))
            _record(f, n, np.zeros((0, 5), np.int32), 1, 1)
    exe = str(tmp_path / "runs_driver")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-Wall", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    f"-I{CSRC}", os.path.join(HERE, "runs_driver.cpp"), os.path.join(CSRC, "runs.cpp"),
                    os.path.join(CSRC, "plan.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe, path, "v"], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "cases 123 " in r.stdout


@pytest.mark.parametrize("n,options,dtype,mode,want", [
    (4, {}, "c64", 1, "runs"), (7, {"force_tiled": 1}, "c128", 0, "runs"), (10, {}, "c64", 2, "runs"),
    (12, {}, "c128", 0, "runs"), (10, {"rz_groups": -1}, "c64", 1, "tile"), (9, {"force_tiled": 1}, "c64", 0, "tile"),
    (11, {"force_tiled": -1}, "c128", 1, "whole"), (5, {"force_tiled": -1}, "c64", 1, "whole"),
    (8, {"force_tiled": -1}, "c128", 0, "whole"), (13, {}, "c64", 1, "tile"),
    (5, {}, "c64", 3, "whole"), (9, {}, "c64", 3, "tile"), (9, {}, "c128", 3, "runs")])
def test_call_kernel(n, options, dtype, mode, want):
    """Which kernel takes a call, and the errors of asking."""
    Q = pytest.importorskip("paper_2301_03251_amd")
    c = Q.Circuit(n, W.random_circuit(n, 30, 3, 4, seed=n), 3, 4, **options)
    assert c.call_kernel(dtype, 8, mode) == want
    for batch, bad in ((0, mode), (8, 4), (8, -1)):
        with pytest.raises(Q.QLError) as e:
            c.call_kernel(dtype, batch, bad)
        assert e.value.code == -1


@pytest.mark.parametrize("n,circuit,dtype,mode,runs,other", [
    (9, "random 400", "c64", 1, 512, 513), (10, "random 400", "c64", 1, 512, 1024), (9, "random 400", "c128", 1, 512, 513),
    (10, "random 400", "c64", 0, 3000, None), (6, "random 700", "c64", 0, 256, 4000), (6, "random 300", "c64", 1, 1024, 4000),
    (10, "layers 20", "c64", 1, 3000, None), (4, "layers 2", "c128", 1, 20000, None), (7, "layers 4", "c64", 0, 40000, None)])
def test_long_circuits_turn_earlier(n, circuit, dtype, mode, runs, other):
    """The LDS of long irregular circuits limits the batch that the run kernel
    takes; layered ones keep it at every batch below 32 KiB of state."""
    Q = pytest.importorskip("paper_2301_03251_amd")
    kind, size = circuit.split()
    if kind == "random":
        gates, F, P = W.random_circuit(n, int(size), 5, 9, seed=n, kinds=ALL), 5, 9
    else:
        gates, F, P = W.layered_circuit(n, "ry", int(size), (W.RX, W.RY, W.RZ), W.CNOT, "linear"), n, 3 * n * int(size)
    c = Q.Circuit(n, gates, F, P)
    assert c.call_kernel(dtype, runs, mode) == "runs"
    if other:
        assert c.call_kernel(dtype, other, mode) == ("tile" if n >= 8 else "whole")
