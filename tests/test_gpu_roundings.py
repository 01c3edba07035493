"""One gate on a state, to the last bit: the per-gate kernels (and on small states
the one-launch kernel) against a CPU model with every rounding written out, from the
C library's fused multiply-add.

u x0 + v x1 + ...: the first product's real part is fma(u.re, x.re, -(u.im x.im)),
its imaginary part fma(u.re, x.im, u.im x.re), or with `swap` fma(u.im, x.re, u.re x.im);
each further product is two fused multiply-adds a part.  `swap` holds for two-qubit
gates on single quads (qubit 0, two qubits, complex128) and for the chunked
kernels (complex64 from 12 qubits, complex128 from 11).
"""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

LIBM = ctypes.CDLL("libm.so.6")
LIBM.fmaf.argtypes, LIBM.fmaf.restype = [ctypes.c_float] * 3, ctypes.c_float
LIBM.fma.argtypes, LIBM.fma.restype = [ctypes.c_double] * 3, ctypes.c_double


def row(u, x, swap, dt):
    """(re, im) of sum_k u[k] x[k]; u, x: pairs (re, im) in the run's real type."""
    fma, real = (LIBM.fmaf, np.float32) if dt == "c64" else (LIBM.fma, np.float64)
    (ur, ui), (xr, xi) = u[0], x[0]
    re = fma(ur, xr, -real(ui * xi))
    im = fma(ui, xr, real(ur * xi)) if swap else fma(ur, xi, real(ui * xr))
    for (ur, ui), (xr, xi) in zip(u[1:], x[1:]):
        re, im = fma(ur, xr, fma(-ui, xi, re)), fma(ur, xi, fma(ui, xr, im))
    return re, im


def model(psi, qubits, U, swap, dt):
    real = np.float32 if dt == "c64" else np.float64
    out = psi.copy()
    pair = lambda z: (real(z.real), real(z.imag))
    k = len(qubits)
    rest = [i for i in range(len(psi)) if not any((i >> q) & 1 for q in qubits)]
    for i in rest:
        idx = [i | sum(((a >> (k - 1 - t)) & 1) << q for t, q in enumerate(qubits)) for a in range(1 << k)]
        x = [pair(psi[j]) for j in idx]
        for a, j in enumerate(idx):
            out[j] = complex(*row([pair(v) for v in U[a]], x, swap, dt))
    return out


@pytest.mark.parametrize("n,qubits,dt", [
    (2, (0, 1), "c64"), (2, (1, 0), "c64"), (2, (1,), "c64"), (3, (0, 2), "c64"), (3, (2, 1), "c64"), (5, (4, 2), "c64"),
    (5, (3, 0), "c64"), (5, (0,), "c64"), (10, (9, 1), "c64"), (10, (6,), "c64"), (11, (10, 3), "c64"), (12, (11, 2), "c64"),
    (12, (0, 5), "c64"), (12, (4,), "c64"), (12, (11,), "c64"), (4, (3, 1), "c128"), (4, (2,), "c128"), (11, (10, 2), "c128"),
    (11, (1,), "c128")])
def test_roundings(n, qubits, dt):
    import paper_2602_14167_amd as P
    r = np.random.default_rng(n)
    cdt, tdt = (np.complex64, torch.complex64) if dt == "c64" else (np.complex128, torch.complex128)
    k = len(qubits)
    U = np.linalg.qr(r.standard_normal((2 ** k, 2 ** k)) + 1j * r.standard_normal((2 ** k, 2 ** k)))[0].astype(cdt)
    mats = np.zeros((1, 4, 4), complex)
    mats[0, :2 ** k, :2 ** k] = U
    circ = P.Circuit(n, W.as_gate_array([W.gate(W.U1 if k == 1 else W.U2, *qubits, mat=0)]), 0, mats)
    psi = W.random_state(n, r).astype(cdt)
    chunked = n >= (12 if dt == "c64" else 11)
    swap = chunked or (k == 2 and (dt == "c128" or n == 2 or 0 in qubits))
    ref = model(psi, qubits, U, swap, dt)
    for mode in ("plain", "tiled") if dt == "c64" and n <= 10 else ("plain",):
        s = torch.as_tensor(psi).to("cuda", tdt).reshape(1, -1)
        P.run_circuit(circ, None, s, mode=mode)
        assert np.array_equal(s.cpu().numpy()[0], ref), (mode, np.max(np.abs(s.cpu().numpy()[0] - ref)))
