"""Pauli sums of many terms on small states (2..10 qubits in complex64, 2..9 in
complex128): H psi and <H> of the small-state kernel against the CPU oracle and
the per-group kernels, and their time against the per-group kernels'.

Sums: one X-mask with one term a class and with classes of several terms (equal
coefficients), some X-masks, random ones; term counts around the four that a wave
loads at once and beyond a thousand.  Bars: H psi as in tests/bars.py, |dE| <= 1e-5
S (complex64), 1e-12 S (complex128) against the oracle, 2^-40 S against the
per-group kernels (float64 sums in another order).
"""
import time

import numpy as np
import pytest
import torch

import workloads as W
from tests.bars import assert_hpsi

pytestmark = pytest.mark.gpu

TOL = {"c64": 1e-5, "c128": 1e-12}
TDT = {"c64": torch.complex64, "c128": torch.complex128}


def pauli_sum(n, terms, kind, r):
    """kind: diag (Z strings), equal (Z strings, coefficients from three values), few (8 X-masks), rand."""
    if kind == "rand":
        return r.integers(0, 4, (terms, n)).astype(np.uint8), r.uniform(-1, 1, terms)
    z = r.integers(0, 2, (terms, n))
    x = r.integers(0, 2, (8, n))[np.arange(terms) % 8] if kind == "few" else np.zeros((terms, n), int)
    codes = np.where(x & z, 2, np.where(x, 1, np.where(z, 3, 0))).astype(np.uint8)
    return codes, r.choice([0.5, -1.0, 0.25], terms) if kind == "equal" else r.uniform(-1, 1, terms)


def states(n, batch, dt, r):
    s = r.standard_normal((batch, 2 ** n)) + 1j * r.standard_normal((batch, 2 ** n))
    s /= np.linalg.norm(s, axis=1, keepdims=True)
    return torch.as_tensor(s).to(device="cuda", dtype=TDT[dt])


@pytest.mark.parametrize("dt", ["c64", "c128"])
@pytest.mark.parametrize("n,terms,kind", [
    (2, 3, "diag"), (3, 64, "rand"), (5, 5, "equal"), (6, 300, "few"), (7, 4, "diag"), (7, 9, "diag"), (8, 255, "equal"),
    (8, 1000, "few"), (9, 7, "rand"), (9, 257, "diag"), (10, 300, "equal"), (10, 1021, "rand"), (10, 0, "diag")])
def test_many_terms(oracle_mod, n, terms, kind, dt):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(100 * n + terms)
    codes, coeffs = pauli_sum(n, terms, kind, r)
    H = P.PauliSum(n, codes, coeffs)
    psi = states(n, 3, dt, r)
    E = P.expect_pauli(psi, H).cpu().numpy()
    hpsi, E2 = P.apply_pauli(psi, H, want_energy=True)
    hp, Ep = P.apply_pauli(psi, H, want_energy=True, mode="plain")
    S = max(float(np.abs(coeffs).sum()), 1e-300)
    assert np.max(np.abs(E - E2.cpu().numpy())) <= 2.0 ** -40 * S
    assert np.max(np.abs(E - Ep.cpu().numpy())) <= 2.0 ** -40 * S
    if not terms:
        assert not torch.any(hpsi) and not np.any(E)
        return
    v = psi.cpu().numpy()
    assert_hpsi(hpsi.cpu().numpy(), hp.cpu().numpy(), v, coeffs, dt, f"n={n} {terms} {kind}, per-group")
    for b in range(3):
        w = v[b].astype(np.complex128)
        ref = oracle_mod.apply_hamiltonian(n, w, codes, coeffs)
        assert_hpsi(hpsi.cpu().numpy()[b], ref, w, coeffs, dt, f"n={n} {terms} {kind}")
        assert abs(E[b] - np.vdot(w, ref).real) <= TOL[dt] * S


# the largest workgroup: full tables of gates (192 one-qubit gates in one chunk) and of
# matrices (64 two-qubit gates in the next), gate gradients, more than 256 X-masks
@pytest.mark.parametrize("n,dt", [(10, "c64"), (9, "c128")])
def test_full_tables(oracle_mod, n, dt):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(n)
    one, params, _ = W.random_circuit(n, 192, r, kinds=[W.RX, W.RY, W.RZ])
    two, _, mats = W.random_circuit(n, 64, r, kinds=[W.U2])
    gates = np.concatenate([one, two])
    codes, coeffs = pauli_sum(n, 300, "rand", r)
    H = P.PauliSum(n, codes, coeffs)
    real = torch.float32 if dt == "c64" else torch.float64
    E, g, gg = P.expect_grad(P.Circuit(n, gates, len(params), mats), torch.as_tensor(params).to("cuda", real), H,
                             dtype=TDT[dt], want_gate_grad=True)
    ref = oracle_mod.expect_grad(n, gates, W.round_params(params, dt), codes, coeffs, W.round_mats(mats, dt), want_lie=True)
    S = float(np.abs(coeffs).sum())
    tg = 1e-4 if dt == "c64" else 1e-12
    assert abs(E.item() - ref["E"]) <= TOL[dt] * S
    assert np.max(np.abs(g.cpu().numpy()[0] - ref["grad"])) <= tg * S
    assert np.max(np.abs(gg.cpu().numpy()[0][192:] - ref["lie"][192:])) <= tg * S


# the small-state kernel serves every sum at these sizes, so it may not be slower than the
# per-group kernels it replaces; a quarter for timing noise.  (One flat load and wait
# per term made single states 2.4 to 4.7 times slower here, and one kernel for all
# uses, with one wave a SIMD, the large batch 7.6 times.)
@pytest.mark.parametrize("n,dt,terms,kind,batch", [
    (10, "c64", 300, "diag", 1), (10, "c64", 1000, "few", 1), (8, "c64", 1000, "diag", 1), (9, "c128", 1000, "diag", 1),
    (9, "c128", 4, "diag", 32768), (9, "c128", 20, "few", 32768), (10, "c64", 4, "diag", 32768)])
def test_not_slower_than_per_group(n, dt, terms, kind, batch):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(terms)
    H = P.PauliSum(n, *pauli_sum(n, terms, kind, r))
    psi = states(n, 1, dt, r).repeat(batch, 1)
    assert best(lambda: P.expect_pauli(psi, H)) <= 1.25 * best(lambda: P.expect_pauli(psi, H, mode="plain"))


def best(f, reps=20, rounds=5):
    f()
    torch.cuda.synchronize()
    out = []
    for _ in range(rounds):
        t0 = time.perf_counter()
        for _ in range(reps):
            f()
        torch.cuda.synchronize()
        out.append((time.perf_counter() - t0) / reps)
    return min(out)
