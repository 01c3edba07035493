// Final sums of one circuit: its energy, angle gradients and per-gate
// Lie-algebra derivatives from the slot and energy row sums (shared by the
// final-sum kernels and the small-state kernel).
#pragma once

#include "kernels.h"

namespace tcng {

// final sums: one thread per (member, output), fixed order everywhere
// output k of one circuit: k = 0 energy, 1..n_params gradient, then 16 per gate
// (when gate_grad is wanted): its 15 Lie-algebra derivatives and one idle
// (one thread per gate left most of a wave's work to 15 serial traces: 171 us
// for 60 circuits of 12 to 20 qubits)
__device__ inline void finish_one(const FinishJob& F, int64_t k) {
    const double* sl = F.slots;
    if (k == 0) {
        double e = 0.0;
        for (int i = 0; i < F.erows; ++i) e += F.erow[i];
        F.energy[0] = e;
    } else if (k <= F.n_params) {
        const int p = int(k - 1);
        double g = 0.0;
        for (int i = F.slot_ptr[p]; i < F.slot_ptr[p + 1]; ++i) g += sl[F.slot_idx[i]];
        F.grad[p] = g;
    } else {
        // per U2 gate: dE/dalpha_k = Im tr(G^dag P_k U), P_k = sigma_a (x) sigma_b, k = 4a + b - 1
        const int64_t r = k - 1 - F.n_params;
        const int gi = int(r / GATE_OUTS), kk = int(r % GATE_OUTS);
        if (kk == 15) return;
        double* out = F.gate_grad + size_t(gi) * 15;
        const int s0 = F.gate_slot[gi];
        if (s0 < 0) {
            out[kk] = 0.0;
            return;
        }
        const double* U = F.u2m + size_t(F.gate_mat[gi]) * 32;
        // single-qubit Paulis: entry (r, c) of sigma_a as (re, im)
        auto sig = [](int a, int r, int c, double& re, double& im) {
            re = 0.0; im = 0.0;
            if (a == 0) re = (r == c) ? 1.0 : 0.0;
            else if (a == 1) re = (r != c) ? 1.0 : 0.0;
            else if (a == 2) im = (r == c) ? 0.0 : (r == 0 ? -1.0 : 1.0);
            else re = (r == c) ? (r == 0 ? 1.0 : -1.0) : 0.0;
        };
        const int a = (kk + 1) >> 2, c = (kk + 1) & 3;
        double tr_im = 0.0;
        for (int x = 0; x < 4; ++x)
            for (int y = 0; y < 4; ++y) {
                // (P U)[y][x] = sum_z P[y][z] U[z][x]
                double pur = 0.0, pui = 0.0;
                for (int z = 0; z < 4; ++z) {
                    double s1r, s1i, s2r, s2i;
                    sig(a, y >> 1, z >> 1, s1r, s1i);
                    sig(c, y & 1, z & 1, s2r, s2i);
                    const double pr = s1r * s2r - s1i * s2i, pi = s1r * s2i + s1i * s2r;
                    const double ur = U[2 * (4 * z + x)], ui = U[2 * (4 * z + x) + 1];
                    pur += pr * ur - pi * ui;
                    pui += pr * ui + pi * ur;
                }
                // conj(G[y][x]) * (PU)[y][x]
                const double gr = sl[s0 + 2 * (4 * y + x)], gim = sl[s0 + 2 * (4 * y + x) + 1];
                tr_im += gr * pui - gim * pur;
            }
        out[kk] = tr_im;
    }
}

}  // namespace tcng
