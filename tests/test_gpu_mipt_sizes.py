"""Monitored trajectories from the smallest to the largest state (9 to 32 qubits),
against closed forms.

The first step's gates rotate six qubits (or four) of |0...0> by Hadamards, the second's
are identities.  A measured qubit that was not rotated is 0; a rotated one that is measured for
the first time is 0 where its uniform lies in the lower half of the measured range,
with probability 1/2, and keeps its outcome when measured again.  What is left is an
equal superposition over the rotated qubits that were never measured.  Bars: 1e-5 on
amplitudes and log-probabilities (a dozen gate and rescaling steps in float32).
"""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

PROB = 0.5


@pytest.mark.parametrize("n,pairs", [(9, [(0, 8), (4, 2)]), (13, [(0, 12), (5, 9), (2, 7)]), (14, [(13, 0), (5, 9), (12, 6)]),
                                     (20, [(0, 19), (13, 12), (5, 16)]), (31, [(30, 0), (13, 12), (5, 20)]),
                                     (32, [(0, 31), (13, 12), (5, 20)])])
def test_sizes(n, pairs):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(n)
    gates = W.as_gate_array([W.gate(W.U2, a, b, mat=k) for k, (a, b) in enumerate(pairs)])
    H = np.array([[1, 1], [1, -1]]) / np.sqrt(2)
    step = P.Circuit(n, gates, 0, np.stack([np.eye(4)] * len(pairs)))
    mats = np.stack([np.stack([np.kron(H, H)] * len(pairs)), np.stack([np.eye(4)] * len(pairs))])[None]
    u = r.random((1, 2, n))
    rotated = {q for pr in pairs for q in pr}
    u[0, 0, pairs[0][0]], u[0, 0, pairs[0][1]] = 0.9, 0.6      # outcomes 1 and 0
    u[0, 1, pairs[1][0]] = 0.95
    psi = P.new_state(n, 1)
    P.state_init(psi)
    rec, logp, _ = P.mipt_run(step, torch.as_tensor(mats).to("cuda", torch.complex64), psi,
                              torch.as_tensor(u).cuda(), PROB)
    value, lp = {}, 0.0
    for s in range(2):
        mask = bits = 0
        for q in range(n):
            if u[0, s, q] < 1 - PROB:
                continue
            mask |= 1 << q
            if q in rotated and q not in value:
                value[q] = int(u[0, s, q] - (1 - PROB) >= 0.5 * PROB)
                lp += np.log(0.5)
            bits |= value.get(q, 0) << q
        got = [int(v) & 0xFFFFFFFF for v in rec[0, s].cpu()]
        assert got == [mask, bits], (s, [hex(v) for v in got], hex(mask), hex(bits))
    assert abs(logp.item() - lp) <= 1e-5
    free = sorted(rotated - set(value))
    index = [sum(v << q for q, v in value.items()) | sum(((k >> i) & 1) << q for i, q in enumerate(free))
             for k in range(1 << len(free))]
    amps = psi[0, torch.as_tensor(index, device="cuda")].cpu().numpy()
    assert np.max(np.abs(amps - 2.0 ** (-0.5 * len(free)))) <= 1e-5
    assert torch.count_nonzero(torch.view_as_real(psi[0])).item() <= 2 * len(index)
    del psi
    torch.cuda.empty_cache()
