"""Launches of more work than one grid holds (2^32 threads): the largest batch
(65535) of deep circuits, whose step coefficients, row sums and final sums each
take a thread or wave per entry.  The circuits rotate one qubit, so the results are
known in closed form: RY(t_1) .. RY(t_k) on |0> is a rotation by the sum of the
angles, <Z> = cos, each derivative -sin.  Bars: a = 8 roundoffs per gate on the
amplitudes (tests/bars.py), so 4 a on <Z> (|d|x|^2| <= 2 |dx| twice) and 8 a on a
derivative (two states, swept forward and back).  All members have the same
angles, so all have the same results, to the last bit."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

BATCH = 65535


@pytest.fixture(autouse=True)
def room():
    torch.cuda.empty_cache()   # (up to 150 GB at a time)
    yield
    torch.cuda.empty_cache()


def rotations(count):
    import paper_2602_14167_amd as P
    g = W.as_gate_array([W.gate(W.RY, 0, p0=k) for k in range(count)])
    r = np.random.default_rng(count)
    t = r.uniform(-np.pi, np.pi, count)
    return P, P.Circuit(11, g, count), torch.as_tensor(t, dtype=torch.float32, device="cuda").repeat(BATCH, 1)


def test_coefficients_beyond_a_grid():
    # 1100 steps forward and 1100 in reverse: 65535 x 2200 x 32 threads
    P, circ, params = rotations(1100)
    psi = P.new_state(11, BATCH)
    P.state_init(psi)
    P.run_circuit(circ, params, psi)
    half = 0.5 * float(params[0].double().sum())
    bar = 8 * 1100 * 2.0 ** -24
    for b in (0, 1, BATCH // 2, BATCH - 1):
        a = psi[b].cpu().numpy()
        assert abs(a[0] - np.cos(half)) <= bar and abs(a[1] - np.sin(half)) <= bar and not np.any(a[2:])
    assert torch.equal(psi[0].expand(BATCH, -1), psi)


def test_row_sums_beyond_a_grid():
    # 65535 x (1024 gradient slots + 1 energy row) waves
    P, circ, params = rotations(1024)
    codes = np.zeros((1, 11), np.uint8)
    codes[0, 0] = 3
    E, g = P.expect_grad(circ, params, P.PauliSum(11, codes, np.ones(1)))
    total, bar = float(params[0].double().sum()), 8 * 1024 * 2.0 ** -24
    for b in (0, BATCH // 2, BATCH - 1):
        assert abs(E[b].item() - np.cos(total)) <= 4 * bar
        assert np.max(np.abs(g[b].cpu().numpy() + np.sin(total))) <= 8 * bar
    assert torch.equal(E[:1].expand(BATCH), E) and torch.equal(g[:1].expand(BATCH, -1), g)


def test_final_sums_beyond_a_grid():
    # 65535 x 4100 gates x 16 outputs; gates without angles: every derivative is 0
    import paper_2602_14167_amd as P
    n_gates = 4100
    circ = P.Circuit(1, W.as_gate_array([W.gate(W.X, 0)] * n_gates), 0)
    H = P.PauliSum(1, np.array([[3]], np.uint8), np.ones(1))
    junk = torch.ones(BATCH * n_gates * 15, dtype=torch.float64, device="cuda")   # (the outputs' memory)
    del junk
    E, _, gg = P.expect_grad(circ, None, H, batch=BATCH, mode="plain", want_gate_grad=True)
    assert torch.equal(E, torch.ones_like(E))
    assert gg.abs().amax().item() == 0.0


def test_block_sums_beyond_a_grid():
    # 65535 x 129 or more matrix-core blocks x 512 sums
    import paper_2602_14167_amd as P
    r = np.random.default_rng(9)
    rows = []
    while len(rows) < 2000:
        a, b = r.permutation(9)[:2]
        rows += [W.gate(W.RY, a, p0=int(r.integers(4))), W.gate(W.CNOT, a, b)]
        if len(rows) % 40 == 0 and P.fused_plan_inspect(9, W.as_gate_array(rows), 4)[4] >= 130:
            break
    gates = W.as_gate_array(rows)
    blocks = P.fused_plan_inspect(9, gates, 4)[4]
    assert 130 <= blocks <= 140
    circ = P.Circuit(9, gates, 4)
    codes, coeffs = W.random_pauli_sum(9, 6, r)
    H = P.PauliSum(9, codes, coeffs)
    t = torch.as_tensor(r.uniform(-np.pi, np.pi, 4), dtype=torch.float32, device="cuda")
    E1, g1 = P.expect_grad(circ, t, H, mode="fused")
    E, g = P.expect_grad(circ, t.repeat(BATCH, 1), H, mode="fused")
    assert torch.equal(E[:1].expand(BATCH), E) and torch.equal(g1.expand(BATCH, -1), g)
    # (one member's energy is summed by two workgroups, a member's of the batch by one)
    assert abs(E[0].item() - E1.item()) <= 2.0 ** -40 * np.abs(coeffs).sum()
