"""Tile addressing and two-qubit diagonals of the tiled and fused passes,
against the CPU oracle.

Gates on every other qubit leave a tile's outside qubits in more runs than the
kernels unroll (four), in the circuit passes (13- and 12-bit tiles), the fused
passes and the Pauli passes; CZ and RZZ on random pairs meet both operands in
registers, one, or none.  Bars as in test_gpu_parity: |dE| <= 1e-5 S,
|d grad| <= 1e-4 S (complex64), 1e-12 S (complex128), S = sum |c_k|.
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"c64": (1e-5, 1e-4), "c128": (1e-12, 1e-12)}
TDT = {"c64": torch.complex64, "c128": torch.complex128}
RDT = {"c64": torch.float32, "c128": torch.float64}


def comb_circuit(n, n_gates, kinds, r):
    """Random gates of `kinds` on the even qubits."""
    g, p, m = W.random_circuit(n // 2, n_gates, r, kinds=kinds)
    g = g.copy()
    g[:, 1:3] = np.where(g[:, 1:3] >= 0, 2 * g[:, 1:3], -1)
    return g, p, m


@pytest.mark.parametrize("n,dt,mode,kinds,comb", [
    (20, "c64", "tiled", [W.RX, W.RZZ, W.CZ, W.H], True), (20, "c128", "tiled", [W.RX, W.RZZ, W.CZ, W.U1], True),
    (20, "c64", "fused", [W.U2, W.RX, W.RZZ], True), (20, "c64", "tiled", [W.RY, W.RZ, W.CNOT], True),
    (14, "c64", "tiled", [W.RX, W.RZZ, W.CZ, W.Z, W.S], False), (13, "c128", "tiled", [W.RX, W.RZZ, W.CZ, W.Z, W.S], False),
    (11, "c64", "tiled", [W.RX, W.RZZ, W.CZ], False), (10, "c128", "tiled", [W.RX, W.RZZ, W.CZ], False),
    (9, "c64", "fused", [W.U2, W.RZZ], False), (11, "c64", "fused", [W.U2, W.RZZ], False)])
def test_tiles(oracle_mod, n, dt, mode, kinds, comb):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(n)
    gates, params, mats = comb_circuit(n, 60, kinds, r) if comb else W.random_circuit(n, 80, r, kinds=kinds)
    codes, coeffs = W.random_pauli_sum(n, 10, r, max_weight=4)
    if comb:
        codes[:, 1::2] = 0   # X-masks on the even qubits too
    circ, H = P.Circuit(n, gates, len(params), mats), P.PauliSum(n, codes, coeffs)
    init = W.random_state(n, r).astype(np.complex64).astype(np.complex128)
    psi = torch.as_tensor(np.tile(init, (1, 1))).to(device="cuda", dtype=TDT[dt])
    p = torch.as_tensor(params[None, :]).to(device="cuda", dtype=RDT[dt])
    E, g = P.expect_grad(circ, p, H, psi=psi, mode=mode)
    ref = oracle_mod.expect_grad(n, gates, W.round_params(params, dt), codes, coeffs, W.round_mats(mats, dt), init=init)
    S = float(np.abs(coeffs).sum())
    te, tg = TOL[dt]
    assert abs(E.item() - ref["E"]) <= te * S
    assert len(params) == 0 or np.max(np.abs(g.cpu().numpy()[0] - ref["grad"])) <= tg * S


# every gate kind's reverse step, at 256 and 258 workgroups (one a compute unit, and more)
@pytest.mark.parametrize("n,dt", [(14, "c64"), (13, "c128")])
@pytest.mark.parametrize("batch", [128, 129])
def test_reverse_occupancy(oracle_mod, n, dt, batch):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(n)
    gates, params, mats = W.random_circuit(n, 80, r, kinds=[W.RX, W.RY, W.RZ, W.RZZ, W.CZ, W.CNOT, W.FSIM, W.U1, W.U2])
    codes, coeffs = W.random_pauli_sum(n, 10, r, max_weight=4)
    circ, H = P.Circuit(n, gates, len(params), mats), P.PauliSum(n, codes, coeffs)
    many = r.uniform(-np.pi, np.pi, (batch, len(params)))
    E, g = P.expect_grad(circ, torch.as_tensor(many).to(device="cuda", dtype=RDT[dt]), H, dtype=TDT[dt],
                         mode="tiled")
    S = float(np.abs(coeffs).sum())
    te, tg = TOL[dt]
    for b in (0, batch // 2, batch - 1):
        ref = oracle_mod.expect_grad(n, gates, W.round_params(many[b], dt), codes, coeffs, W.round_mats(mats, dt))
        assert abs(E[b].item() - ref["E"]) <= te * S
        assert np.max(np.abs(g.cpu().numpy()[b] - ref["grad"])) <= tg * S
