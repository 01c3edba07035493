"""Small states (2..10 qubits in complex64, 2..9 in complex128): the one-launch
evaluation, against the CPU oracle and against the per-gate kernels.

Sizes: a single quad (2 qubits) up to four waves with two pairs a thread (10);
circuits of every gate kind, more gates and matrix entries than one chunk of the
LDS tables, qubits without a gate, no gates at all, more Pauli terms than
are kept in LDS, large batches.  Bars as in test_gpu_parity: |dE| <= 1e-5 S,
|d grad| <= 1e-4 S (complex64), 1e-12 S (complex128), S = sum |c_k|.  The
complex64 amplitudes equal the per-gate kernels' exactly (the same roundings in
the same order); the float64 sums are taken in another order, so energies and gradients
agree with theirs to 2^-40 S.
"""
import numpy as np
import pytest
import torch

import workloads as W
from tests.bars import assert_amps

pytestmark = pytest.mark.gpu

TOL = {"c64": (1e-5, 1e-4), "c128": (1e-12, 1e-12)}
TDT = {"c64": torch.complex64, "c128": torch.complex128}
RDT = {"c64": torch.float32, "c128": torch.float64}


@pytest.fixture(scope="module")
def P():
    import paper_2602_14167_amd as pkg
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    pkg.lib()
    return pkg


def circuit(shape, n, r):
    if shape == "empty":
        return W.as_gate_array([]), np.zeros(0), np.zeros((0, 4, 4), complex)
    if shape == "singles":   # no two-qubit gate
        return W.random_circuit(n, 4 * n, r, kinds=[k for k in range(14) if k not in W.TWO_QUBIT])
    if shape == "pair":      # 100 gates on one pair of qubits, the others idle
        g, p, m = W.random_circuit(2, 100, r)
        g = g.copy()
        a, b = n - 1, n // 2 if n > 2 else 0
        g[:, 1:3] = np.where(g[:, 1:3] == 0, a, np.where(g[:, 1:3] == 1, b, -1))
        return g, p, m
    return W.random_circuit(n, 400 if shape == "deep" else 40, r)


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,shape,batch,terms", [
    (2, "mixed", 1, 3), (3, "mixed", 3, 8), (4, "singles", 2, 9), (5, "pair", 2, 20), (6, "deep", 2, 300),
    (7, "mixed", 513, 12), (8, "empty", 2, 5), (8, "deep", 3, 24), (9, "mixed", 5, 27), (9, "deep", 1, 40),
    (10, "deep", 2, 30), (10, "singles", 1100, 4)])
def test_small_states(P, oracle_mod, n, shape, batch, terms, dt):
    r = np.random.default_rng(1000 * n + batch)
    gates, params, mats = circuit(shape, n, r)
    npar = len(params)
    codes, coeffs = W.random_pauli_sum(n, terms, r)
    circ, H = P.Circuit(n, gates, npar, mats), P.PauliSum(n, codes, coeffs)
    pb = r.uniform(0, 2 * np.pi, (batch, npar))
    init = W.random_state(n, r).astype(np.complex64).astype(np.complex128)
    psi = torch.as_tensor(np.tile(init, (batch, 1))).to(device="cuda", dtype=TDT[dt])
    p = torch.as_tensor(pb).to(device="cuda", dtype=RDT[dt])
    fwd = psi.clone()
    P.run_circuit(circ, p, fwd)
    E_only = P.expect_pauli(fwd, H).cpu().numpy()
    hpsi, E_h = P.apply_pauli(fwd, H, want_energy=True)
    E, g, gg = P.expect_grad(circ, p, H, psi=psi, want_gate_grad=True)
    E, g, gg = E.cpu().numpy(), g.cpu().numpy(), gg.cpu().numpy()
    S = float(np.abs(coeffs).sum())
    te, tg = TOL[dt]
    for b in {0, batch // 2, batch - 1}:
        ref = oracle_mod.expect_grad(n, gates, W.round_params(pb[b], dt), codes, coeffs, W.round_mats(mats, dt),
                                     init=init, want_state=True, want_lie=True)
        assert abs(E[b] - ref["E"]) <= te * S and abs(E_only[b] - ref["E"]) <= te * S
        assert abs(E_h[b].item() - ref["E"]) <= te * S
        assert npar == 0 or np.max(np.abs(g[b] - ref["grad"])) <= tg * S
        u2 = gates[:, 0] == W.U2   # (the oracle gives every two-qubit gate's; the library the constant ones')
        assert not u2.any() or np.max(np.abs(gg[b][u2] - ref["lie"][u2])) <= tg * S
        assert not np.any(gg[b][~u2])
        assert_amps(fwd.cpu().numpy()[b], ref["state"], dt, max(len(gates), 1), f"n={n} {shape} state")
        e_h = np.vdot(fwd[b].cpu().numpy().astype(complex), hpsi[b].cpu().numpy().astype(complex)).real
        assert abs(e_h - ref["E"]) <= te * S
    # the per-gate kernels
    psi_p = torch.as_tensor(np.tile(init, (batch, 1))).to(device="cuda", dtype=TDT[dt])
    fwd_p = psi_p.clone()
    P.run_circuit(circ, p, fwd_p, mode="plain")
    assert dt == "c128" or torch.equal(fwd, fwd_p)
    E_p, g_p, gg_p = P.expect_grad(circ, p, H, psi=psi_p, want_gate_grad=True, mode="plain")
    assert dt == "c128" or torch.equal(psi, psi_p)
    assert np.max(np.abs(E - E_p.cpu().numpy())) <= 2.0 ** -40 * S
    assert npar == 0 or np.max(np.abs(g - g_p.cpu().numpy())) <= 2.0 ** -40 * S
    assert len(gates) == 0 or np.max(np.abs(gg - gg_p.cpu().numpy())) <= 2.0 ** -40 * S
    assert_amps(psi.cpu().numpy()[0], init, dt, 8 * max(len(gates), 1), f"n={n} {shape} recomputed state")
