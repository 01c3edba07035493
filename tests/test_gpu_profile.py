"""Launches are booked under the family of the kernel that runs: on small states
the one-launch kernel's own, elsewhere those of the passes."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

SMALL, FAMILIES = 21, 22


def counts(P, f):
    P.check(P.lib().tcng_profile_begin(4096))
    f()
    torch.cuda.synchronize()
    out = {}
    for k in range(FAMILIES):
        n, ms = ctypes.c_int32(), ctypes.c_double()
        P.check(P.lib().tcng_profile_query(k, ctypes.byref(n), ctypes.byref(ms)))
        if n.value:
            out[k] = n.value
    P.check(P.lib().tcng_profile_end())
    return out


@pytest.mark.parametrize("n,small", [(8, True), (10, True), (12, False)])
def test_small_states_have_their_own_family(n, small):
    import paper_2602_14167_amd as P
    w = W.hea_workload(n, 2, -1.0, -0.5, seed=n, batch=2)
    circ, H = P.Circuit(n, w["gates"], w["n_params"]), P.PauliSum(n, w["codes"], w["coeffs"])
    p = torch.as_tensor(np.asarray(w["params"])).to("cuda", torch.float32)
    psi = P.new_state(n, 2)
    P.state_init(psi)
    for f in (lambda: P.run_circuit(circ, p, psi), lambda: P.expect_pauli(psi, H), lambda: P.apply_pauli(psi, H),
              lambda: P.expect_grad(circ, p, H, psi=psi)):
        c = counts(P, f)
        assert (c == {SMALL: 1}) if small else (SMALL not in c and c)
