// Gate matrices and their products with amplitudes, gate by gate (the per-gate
// kernels and the small-state kernel: the same arithmetic in both).
#pragma once

#include "gates.h"

namespace tcng {

// build the (possibly inverted) 2x2 / 4x4 matrix of a gate for batch member b
template <typename R>
__device__ __forceinline__ void gate_mat1(int kind, const R* prm, int p0, const cx<R>* cm, int mat,
                                          const cx<R>* umat, bool inv, cx<R> u[4]) {
    if (umat) {
        u[0] = umat[0]; u[1] = umat[1]; u[2] = umat[2]; u[3] = umat[3];
    } else if (kind_diagonal(kind)) {
        cx<R> d[2];
        diag1<R>(kind, prm, p0, d);
        u[0] = d[0]; u[1] = {R(0), R(0)}; u[2] = {R(0), R(0)}; u[3] = d[1];
    } else {
        mat1<R>(kind, prm, p0, cm, mat, u);
    }
    if (inv) dagger_inplace<R, 2>(u);
}

template <typename R>
__device__ __forceinline__ void gate_mat2(int kind, const R* prm, int p0, int p1, const cx<R>* cm, int mat,
                                          const cx<R>* umat, bool inv, cx<R> u[16]) {
    if (umat) {
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i] = umat[i];
    } else if (kind == K_FSIM || kind == K_U2) {
        mat2<R>(kind, prm, p0, p1, cm, mat, u);
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) u[i] = {R(0), R(0)};
        if (kind == K_CNOT) {
            u[0] = {R(1), R(0)}; u[5] = {R(1), R(0)}; u[11] = {R(1), R(0)}; u[14] = {R(1), R(0)};
        } else {
            cx<R> d[4];
            diag2<R>(kind, prm, p0, d);
            u[0] = d[0]; u[5] = d[1]; u[10] = d[2]; u[15] = d[3];
        }
    }
    if (inv) dagger_inplace<R, 4>(u);
}

// Products with the roundings written out.  Left to the compiler, which of the two
// products of a sum is rounded first varies between copies of u x, so that two kernels
// that apply the same gate could differ, or change with the compiler.  u x: the real
// part rounds u.im x.im first; the imaginary part u.im x.re, or with SWAP u.re x.im.
// The chunked kernels take SWAP, and two-qubit gates on single quads (qubit 0, two
// qubits in all, complex128) do; everything else takes the other.
template <bool SWAP, typename R>
__device__ __forceinline__ cx<R> rmul(cx<R> u, cx<R> x) {
    return {fmaR(u.re, x.re, -(u.im * x.im)),
            SWAP ? fmaR(u.im, x.re, u.re * x.im) : fmaR(u.re, x.im, u.im * x.re)};
}

template <bool SWAP, typename R>
__device__ __forceinline__ void mv2(const cx<R>* u, cx<R>& a0, cx<R>& a1) {
    const cx<R> x0 = a0, x1 = a1;
    a0 = cfma(u[1], x1, rmul<SWAP>(u[0], x0));
    a1 = cfma(u[3], x1, rmul<SWAP>(u[2], x0));
}

template <bool SWAP, typename R>
__device__ __forceinline__ void mv4(const cx<R>* u, cx<R>* x) {
    const cx<R> x0 = x[0], x1 = x[1], x2 = x[2], x3 = x[3];
#pragma unroll
    for (int a = 0; a < 4; ++a)
        x[a] = cfma(u[4 * a + 3], x3, cfma(u[4 * a + 2], x2, cfma(u[4 * a + 1], x1, rmul<SWAP>(u[4 * a], x0))));
}

}  // namespace tcng
