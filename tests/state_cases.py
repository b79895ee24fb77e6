"""complex64 final states and shots whose bits are fixed: shots are whole
numbers drawn by a state's bits, so how a state rounds stays what it is when
kernels or plans change. ``golden/state_bits.json`` holds a digest per case;
``python tests/state_cases.py`` prints the digests of the package as it is (on
an MI355X).
"""

from __future__ import annotations

import hashlib
import json
import os
import sys

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
GOLDEN = os.path.join(HERE, "golden", "state_bits.json")

# name: (qubits, batch, circuit, extras)
CASES = {
    "2q": (2, 3, "random", {}),
    "5q": (5, 3, "random", {}),
    "6q amplitude": (6, 3, "random", {"embed": "amplitude"}),
    "7q": (7, 3, "random", {}),
    "7q 2100 circuits": (7, 2100, "random", {}),
    "7q layers": (7, 5, "layers", {}),
    "8q": (8, 3, "random", {}),
    "8q layers": (8, 5, "layers", {}),
    "9q amplitude": (9, 3, "random", {"embed": "amplitude"}),
    "10q layers": (10, 5, "layers", {}),
    "11q basis": (11, 3, "random", {"embed": "basis"}),
    "12q": (12, 3, "random", {}),
    "12q 600 circuits": (12, 600, "layers", {}),
    "13q layers": (13, 3, "layers", {}),
    "13q channels": (13, 3, "random", {"channels": True}),
    "14q layers": (14, 2, "layers", {}),
    "14q layers no prefix": (14, 2, "layers", {"product_prefix": -1}),
    "15q": (15, 2, "random", {}),
    "15q single ops": (15, 2, "layers", {"rz_groups": -1}),
    "16q angles": (16, 2, "angles", {}),
}


def digests(name, Q, W, torch):
    """sha256 of a case's states and of 500 shots of each."""
    n, B, kind, extras = CASES[name]
    extras = dict(extras)
    rng = np.random.default_rng(n)
    embed, p = extras.pop("embed", None), None
    F = {None: n, "basis": n, "amplitude": 1 << n}[embed]
    if kind == "layers":  # RX RY RZ on every qubit: the longest products of one-qubit gates
        layers, rotations = 3, (W.RX, W.RY, W.RZ)
        gates, P = W.layered_circuit(n, "ry", layers, rotations, W.CNOT, "brick"), 3 * layers * n
    elif kind == "angles":
        gates, P = W.layered_circuit(n, "h_rz", 4, (W.RY, W.RZ), W.CZ, "ring"), 2 * 4 * n
    else:
        P = 7
        gates = W.random_circuit(n, 120, F, P, seed=3000 + n,
                                 kinds=(W.H, W.RX, W.RY, W.RZ, W.CNOT, W.CZ, W.CRX, W.CRY, W.CRZ))
    if extras.pop("channels", False):
        half = len(gates) // 2
        ch = np.array([[W.PAULI, q, -1, W.SRC_INPUT, F + q] for q in range(n)], np.int32)
        gates, p, F = np.concatenate([gates[:half], ch, gates[half:]]), [[0.2, 0.2, 0.2]] * n, F + n
    x = rng.uniform(-3.5, 3.5, (B, F)).astype(np.float32)
    if p is not None:
        x[:, F - n:] = rng.random((B, n)).astype(np.float32)
    w = rng.uniform(-7, 7, P).astype(np.float32)
    u = rng.random((B, 500))
    kinds = {None: None, "basis": (W.EMBED_BASIS, 0), "amplitude": (W.EMBED_AMPLITUDE, 0)}
    r = Q.Runner(Q.Circuit(n, gates, F, P, embed=kinds[embed], pauli_p=p, **extras), "c64")
    psi = r.state(torch.from_numpy(x).cuda(), torch.from_numpy(w).cuda())
    shots, _ = Q.sample(psi, torch.from_numpy(u).cuda())
    return {"state": hashlib.sha256(psi.cpu().numpy().tobytes()).hexdigest(),
            "shots": hashlib.sha256(shots.cpu().numpy().tobytes()).hexdigest()}


if __name__ == "__main__":
    sys.path.insert(0, os.getcwd())
    import torch
    import paper_2301_03251_amd as Q
    import workloads as W
    print(json.dumps({name: digests(name, Q, W, torch) for name in CASES}, indent=1))
