// Whole evaluations of small states, one workgroup per batch member: forward
// sweep, H psi and <H>, adjoint sweep, gate derivatives and final sums in one
// launch, with the state and the costate in LDS.
//
// What bounds a call on so small a state is latency.  On the per-gate kernels
// it is one launch per gate and sweep: 140 launches and 0.6 ms for 69 gates on
// 8 qubits and 32 parameter sets.  Here a gate costs one LDS round trip and one
// barrier (none while one wave holds all pairs), its matrix comes from an LDS
// table that the workgroup forms at the start, one thread per gate, and a
// derivative is one sum over the wave, added over the waves at the end.  The
// gates are applied one by one in circuit order with the per-gate kernels'
// matrices (plaingate.h), products and roundings, so complex64 amplitudes agree
// with theirs to the last bit; only the float64 sums are taken in another order.
// Measured, 8 qubits, 69 gates, 32 parameter sets, complex64, value and gradient
// through autograd: 0.64 ms a call with the per-gate kernels, 0.12 ms now, of which
// the kernel is 62 us.  (Runs of gates multiplied into 4 x 4 matrices first took 50 us,
// but round differently: energies and gradients moved by 1e-6.)
#include "devutil.h"
#include "finish.h"
#include "plaingate.h"

namespace tcng {

namespace {

constexpr int SM_THREADS = 256;

// LDS layout of a workgroup (bytes): the host sizes the launch with it, by the
// circuit's own tables, so small circuits share a compute unit.  The largest launch
// (every table full) has to stay within the 64 KiB that a launch may ask for without
// a function attribute.
template <typename R>
struct SmallLds {
    size_t psi, lam, mat, ops, red, cot, esum, total;
    __host__ __device__ constexpr SmallLds(int n, int tab_mat, int tab_ops, bool rev, bool cotangents, int nwaves)
        : psi(0),
          lam((size_t(1) << n) * sizeof(cx<R>)),
          mat(lam + (rev ? lam : 0)),
          ops(mat + size_t(tab_mat) * sizeof(cx<R>)),
          red(ops + size_t(tab_ops) * sizeof(SOp)),
          cot(red + size_t(tab_ops) * 2 * nwaves * sizeof(double)),
          esum(cot + (cotangents ? size_t(2) * 32 * nwaves * sizeof(double) : 0)),
          total(esum + SM_THREADS / 64 * sizeof(double)) {}
    __host__ __device__ SmallLds(const SmallJob& J, int nwaves)
        : SmallLds(J.n, J.tab_mat, J.tab_ops, J.do_rev != 0, J.gate_grad != nullptr, nwaves) {}
};
// qubits of the largest state
template <typename R>
constexpr int small_qubits() { return sizeof(R) == 4 ? SM_QUBITS : SM_QUBITS - 1; }
static_assert(SmallLds<float>(small_qubits<float>(), SM_MAT, SM_OPS, true, true, SM_THREADS / 64).total <= 65536 &&
                  SmallLds<double>(small_qubits<double>(), SM_MAT, SM_OPS, true, true, SM_THREADS / 64).total <= 65536,
              "LDS of the largest launch");

__device__ __forceinline__ uint32_t insert_zero(uint32_t v, int q) { return ((v >> q) << (q + 1)) | (v & ((1u << q) - 1u)); }

// a state between global memory and LDS, 16 bytes an access (the state descriptor's
// alignment; four amplitudes or more), two in flight
template <typename R>
__device__ __forceinline__ void copy_state(cx<R>* dst, const cx<R>* src, uint32_t dim, uint32_t t, uint32_t T) {
    typedef float vec16 __attribute__((vector_size(16), may_alias));
    vec16* d = reinterpret_cast<vec16*>(dst);
    const vec16* s = reinterpret_cast<const vec16*>(src);
    const uint32_t chunks = dim * uint32_t(sizeof(cx<R>)) / 16;
    for (uint32_t c = t; c < chunks; c += 2 * T) {
        const bool more = c + T < chunks;
        const vec16 a = s[c], b = s[more ? c + T : c];
        d[c] = a;
        if (more) d[c + T] = b;
    }
}

// order of the LDS operations between gates: a barrier, or nothing but program
// order while one wave does all of them
__device__ __forceinline__ void gate_sync(bool many) {
    if (many) __syncthreads();
    else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

template <typename R>
__device__ __forceinline__ cx<R> dag(const cx<R>* u, int dim, int a, int b, bool inv) {
    return inv ? conj(u[b * dim + a]) : u[a * dim + b];
}

// a two-qubit gate (or its inverse) on one quad; x: local index, q0 = most
// significant; swap: the per-gate forward kernel's rounding of single quads (plaingate.h)
template <typename R>
__device__ __forceinline__ void quad_apply(int kind, const cx<R>* u, bool inv, bool swap, cx<R>* x) {
    if (kind == K_CNOT) {   // (exact either way: the dense product adds zeros)
        const cx<R> s = x[2];
        x[2] = x[3];
        x[3] = s;
    } else {
        cx<R> m[16];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) m[4 * a + b] = dag(u, 4, a, b, inv);
        if (swap) mv4<true>(m, x);
        else mv4<false>(m, x);
    }
}

// H psi and this thread's part of <H>, for its A amplitudes t, t + T, ... (A = 1:
// threads beyond a state smaller than a wave repeat others' work and drop it).
// What bounds it is the latency of the tables' loads: they are the same for every
// lane, so they are scalar loads, one serves A amplitudes, four one-term classes are
// in flight at once, and the next group is loaded ahead.  (The classes and their
// terms stand in group order, so the first term of a class is known before the
// class is loaded.)  <H> of 300 / 1000 Z strings on 10 qubits, complex64: 39 / 124 us;
// one flat load and wait a term for each amplitude took 235 / 801, the per-group
// kernels' four workgroups 50 / 153.
template <bool REV, int A, typename R>
__device__ __forceinline__ double pauli_part(const SmallJob& J, const cx<R>* psi, cx<R>* lam, cx<R>* glam, uint32_t t,
                                             uint32_t T) {
    cptr<PGroupFull> groups = as_const(J.groups);
    cptr<PClassFull> classes = as_const(J.classes);
    cptr<PTermFull> terms = as_const(J.terms);
    const uint32_t dim = 1u << J.n;
    uint32_t i[A];
    cx<R> pj[A], acc[A];
    double e[A];
#pragma unroll
    for (int a = 0; a < A; ++a) {
        i[a] = (t + uint32_t(a) * T) & (dim - 1u);
        pj[a] = psi[i[a]];
        acc[a] = {R(0), R(0)};
        e[a] = 0.0;
    }
    int m = 0;   // first term of class c
    PGroupFull next{};
    if (J.n_groups) next = groups[0];
    for (int g = 0; g < J.n_groups; ++g) {
        const PGroupFull G = next;
        next = groups[g + 1 < J.n_groups ? g + 1 : g];
        uint32_t j[A];
        cx<R> pp[A];
        double cre[A], cim[A];
#pragma unroll
        for (int a = 0; a < A; ++a) {
            j[a] = i[a] ^ uint32_t(G.x);
            pp[a] = psi[j[a]];
            cre[a] = cim[a] = 0.0;
        }
        for (int c = G.class_begin; c < G.class_end;) {
            if (c + 4 <= G.class_end) {   // (at least four terms from m on, then)
                PClassFull K[4];
                uint32_t z[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    K[k] = classes[c + k];
                    z[k] = uint32_t(terms[m + k].z);
                }
                if (K[3].term_end == m + 4) {   // one term each: its sign is the class's factor
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int a = 0; a < A; ++a) {
                            const double s = (__popc(j[a] & z[k]) & 1) ? -1.0 : 1.0;
                            cre[a] = fma(K[k].cre, s, cre[a]);
                            cim[a] = fma(K[k].cim, s, cim[a]);
                        }
                    c += 4;
                    m += 4;
                    continue;
                }
            }
            const PClassFull K = classes[c];
            const int n_terms = K.term_end - m;
            int odd[A];
#pragma unroll
            for (int a = 0; a < A; ++a) odd[a] = 0;
            for (; m + 4 <= K.term_end; m += 4) {
                uint32_t z[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) z[k] = uint32_t(terms[m + k].z);
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int a = 0; a < A; ++a) odd[a] += __popc(j[a] & z[k]) & 1;
            }
            for (; m < K.term_end; ++m) {
                const uint32_t z = uint32_t(terms[m].z);
#pragma unroll
                for (int a = 0; a < A; ++a) odd[a] += __popc(j[a] & z) & 1;
            }
#pragma unroll
            for (int a = 0; a < A; ++a) {
                const double s = double(n_terms - 2 * odd[a]);
                cre[a] = fma(K.cre, s, cre[a]);
                cim[a] = fma(K.cim, s, cim[a]);
            }
            ++c;
        }
#pragma unroll
        for (int a = 0; a < A; ++a) {
            acc[a] = cfma(cx<R>{R(cre[a]), R(cim[a])}, pp[a], acc[a]);
            const double rr = fma(double(pj[a].re), double(pp[a].re), double(pj[a].im) * double(pp[a].im));
            const double ri = fma(double(pj[a].re), double(pp[a].im), -double(pj[a].im) * double(pp[a].re));
            e[a] += cre[a] * rr - cim[a] * ri;
        }
    }
    double sum = 0.0;
    if (A == 1 && t >= dim) return sum;
#pragma unroll
    for (int a = 0; a < A; ++a) {
        if (REV && J.do_rev) lam[i[a]] = acc[a];
        else if (glam) glam[i[a]] = acc[a];
        sum += e[a];
    }
    return sum;
}

// PARTS: what a launch may have to do: Pauli sums only, gates too, or also the
// derivatives of constant two-qubit matrices.  The 32 float64 sums of those take 213
// registers in complex64 and 290 in complex128; without them gates take 106 and 165, and
// Pauli sums alone 93 and 62.  Large batches need the waves that this leaves room for:
// <H> of 4 Z strings on 32768 states of 9 qubits in complex128 took 489 us in one
// kernel for all, where the per-group kernels take 64; now 45.
enum SmallParts { SM_PAULI, SM_GATES, SM_COTANGENTS };

template <typename R, int PARTS>
__global__ void __launch_bounds__(SM_THREADS, PARTS == SM_PAULI ? 5 : 1) k_small(const SmallJob J) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int n = J.n, T = blockDim.x, t = threadIdx.x;
    const int nwaves = T >> 6;
    const int wave = uniform(t >> 6), lane = t & 63;
    const uint32_t dim = 1u << n, pairs = dim >> 1, quads = dim >> 2;
    const bool many = T > 64;
    const SmallLds<R> L(J, nwaves);
    cx<R>* psi = reinterpret_cast<cx<R>*>(smem + L.psi);
    cx<R>* lam = reinterpret_cast<cx<R>*>(smem + L.lam);
    cx<R>* mat = reinterpret_cast<cx<R>*>(smem + L.mat);
    SOp* ops = reinterpret_cast<SOp*>(smem + L.ops);
    double* red = reinterpret_cast<double*>(smem + L.red);
    double* cot = reinterpret_cast<double*>(smem + L.cot);
    double* esum = reinterpret_cast<double*>(smem + L.esum);
    const int64_t b = blockIdx.x;
    cx<R>* gpsi = static_cast<cx<R>*>(J.psi) + b * J.stride;
    cx<R>* glam = J.lam ? static_cast<cx<R>*>(J.lam) + b * J.stride : nullptr;
    const R* prm = J.params ? static_cast<const R*>(J.params) + b * J.n_params : nullptr;
    const cx<R>* cm = static_cast<const cx<R>*>(J.cm);
    double* slots = J.slots ? J.slots + b * J.total_slots : nullptr;

    copy_state(psi, gpsi, dim, t, T);
    // gates [begin, end) of chunk k and their matrices
    auto chunk = [&](int k) { return k ? J.chunks[k] : J.chunk0; };
    auto build = [&](const SChunk& C) {
        for (int i = t; i < C.op_end - C.op_begin; i += T) {
            const SOp o = J.ops[C.op_begin + i];
            ops[i] = o;
            if (o.q1 >= 0) gate_mat2<R>(o.kind, prm, o.p0, o.p1, cm, o.mat, nullptr, false, mat + o.mpos);
            else gate_mat1<R>(o.kind, prm, o.p0, cm, o.mat, nullptr, false, mat + o.mpos);
        }
        __syncthreads();
    };

    if (PARTS >= SM_GATES && J.do_fwd)
        for (int k = 0; k < J.n_chunks; ++k) {
            const SChunk C = chunk(k);
            if (k) __syncthreads();   // the previous chunk's tables
            build(C);
            const int nops = C.op_end - C.op_begin;
            SOp next = ops[0];
            for (int i = 0; i < nops; ++i) {
                const int kind = uniform(next.kind), q0 = uniform(next.q0), q1 = uniform(next.q1);
                const cx<R>* u = mat + uniform(next.mpos);
                next = ops[i + 1 < nops ? i + 1 : i];
                if (q1 < 0) {
                    const cx<R> m[4] = {u[0], u[1], u[2], u[3]};
                    const uint32_t b0 = 1u << q0;
                    for (uint32_t w = t; w < pairs; w += T) {
                        const uint32_t i0 = insert_zero(w, q0);
                        cx<R> x0 = psi[i0], x1 = psi[i0 | b0];
                        mv2<false>(m, x0, x1);
                        psi[i0] = x0;
                        psi[i0 | b0] = x1;
                    }
                } else {
                    const uint32_t b0 = 1u << q0, b1 = 1u << q1;
                    const int lo = q0 < q1 ? q0 : q1, hi = q0 < q1 ? q1 : q0;
                    for (uint32_t w = t; w < quads; w += T) {
                        const uint32_t i0 = insert_zero(insert_zero(w, lo), hi);
                        cx<R> x[4] = {psi[i0], psi[i0 | b1], psi[i0 | b0], psi[i0 | b0 | b1]};
                        quad_apply<R>(kind, u, false, lo == 0 || n == 2, x);
                        psi[i0] = x[0];
                        psi[i0 | b1] = x[1];
                        psi[i0 | b0] = x[2];
                        psi[i0 | b0 | b1] = x[3];
                    }
                }
                gate_sync(many);
            }
        }
    __syncthreads();

    if (J.do_pauli) {
        constexpr bool REV = PARTS >= SM_GATES;
        double e;
        if (sizeof(R) == 4 && dim == 4u * T) e = pauli_part<REV, sizeof(R) == 4 ? 4 : 1>(J, psi, lam, glam, t, T);
        else if (dim == 2u * T) e = pauli_part<REV, 2>(J, psi, lam, glam, t, T);
        else e = pauli_part<REV, 1>(J, psi, lam, glam, t, T);
        e = wave_sum(e);
        if (lane == 0) esum[wave] = e;
        __syncthreads();
        if (t == 0 && J.energy) {
            double s = 0.0;
            for (int w = 0; w < nwaves; ++w) s += esum[w];
            J.energy[b] = s;
        }
    }

    if (PARTS >= SM_GATES && J.do_rev) {
        for (int k = J.n_chunks - 1; k >= 0; --k) {
            const SChunk C = chunk(k);
            if (J.n_chunks > 1) build(C);   // (one chunk: the forward sweep's tables stand)
            const int nops = C.op_end - C.op_begin;
            int buf = 0;
            SOp next = ops[nops - 1];
            for (int i = nops - 1; i >= 0; --i) {
                const int kind = uniform(next.kind), q0 = uniform(next.q0), q1 = uniform(next.q1);
                const int slot = uniform(next.slot);
                const cx<R>* u = mat + uniform(next.mpos);
                next = ops[i > 0 ? i - 1 : 0];
                double g0 = 0.0, g1 = 0.0;
                if (q1 < 0) {
                    const cx<R> m[4] = {conj(u[0]), conj(u[2]), conj(u[1]), conj(u[3])};
                    const uint32_t b0 = 1u << q0;
                    for (uint32_t w = t; w < pairs; w += T) {
                        const uint32_t i0 = insert_zero(w, q0);
                        cx<R> x0 = psi[i0], x1 = psi[i0 | b0], l0 = lam[i0], l1 = lam[i0 | b0];
                        if (slot >= 0) {
                            if (kind == K_RX) g0 += im_conj_mul(l0, x1) + im_conj_mul(l1, x0);
                            else if (kind == K_RY) g0 += re_conj_mul(l1, x0) - re_conj_mul(l0, x1);
                            else g0 += im_conj_mul(l0, x0) - im_conj_mul(l1, x1);   // RZ
                        }
                        mv2<false>(m, x0, x1);
                        mv2<false>(m, l0, l1);
                        psi[i0] = x0;
                        psi[i0 | b0] = x1;
                        lam[i0] = l0;
                        lam[i0 | b0] = l1;
                    }
                } else {
                    const uint32_t b0 = 1u << q0, b1 = 1u << q1;
                    const int lo = q0 < q1 ? q0 : q1, hi = q0 < q1 ? q1 : q0;
                    const bool want_cot = PARTS == SM_COTANGENTS && kind == K_U2 && slot >= 0;
                    double G[32];
                    if (want_cot)
#pragma unroll
                        for (int e = 0; e < 32; ++e) G[e] = 0.0;
                    for (uint32_t w = t; w < quads; w += T) {
                        const uint32_t i0 = insert_zero(insert_zero(w, lo), hi);
                        const uint32_t ix[4] = {i0, i0 | b1, i0 | b0, i0 | b0 | b1};
                        cx<R> x[4], l[4];
#pragma unroll
                        for (int a = 0; a < 4; ++a) {
                            x[a] = psi[ix[a]];
                            l[a] = lam[ix[a]];
                        }
                        if (kind == K_RZZ) {
                            g0 += im_conj_mul(l[0], x[0]) - im_conj_mul(l[1], x[1]) - im_conj_mul(l[2], x[2]) +
                                  im_conj_mul(l[3], x[3]);
                        } else if (kind == K_FSIM) {
                            g0 += 2.0 * (im_conj_mul(l[1], x[2]) + im_conj_mul(l[2], x[1]));
                            g1 += 2.0 * im_conj_mul(l[3], x[3]);
                        }
                        quad_apply<R>(kind, u, true, false, x);
                        if (want_cot)
#pragma unroll
                            for (int a = 0; a < 4; ++a)
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    G[2 * (4 * a + c)] += fma(double(l[a].re), double(x[c].re), double(l[a].im) * double(x[c].im));
                                    G[2 * (4 * a + c) + 1] += fma(double(l[a].im), double(x[c].re), -double(l[a].re) * double(x[c].im));
                                }
                        quad_apply<R>(kind, u, true, false, l);
#pragma unroll
                        for (int a = 0; a < 4; ++a) {
                            psi[ix[a]] = x[a];
                            lam[ix[a]] = l[a];
                        }
                    }
                    if (want_cot) {   // (two buffers: the last barrier orders the one before last)
                        double* dst = cot + buf * 32 * nwaves;
#pragma unroll
                        for (int e = 0; e < 32; ++e) {
                            const double s = wave_sum(G[e]);
                            if (lane == 0) dst[e * nwaves + wave] = s;
                        }
                        gate_sync(many);
                        if (t < 32) {
                            double s = 0.0;
                            for (int w = 0; w < nwaves; ++w) s += dst[t * nwaves + w];
                            slots[slot + t] = s;
                        }
                        buf ^= 1;
                        continue;
                    }
                }
                if (slot >= 0 && kind != K_U2) {
                    g0 = wave_sum(g0);
                    if (kind == K_FSIM) g1 = wave_sum(g1);
                    if (lane == 0) {
                        red[(2 * i) * nwaves + wave] = g0;
                        red[(2 * i + 1) * nwaves + wave] = g1;
                    }
                }
                gate_sync(many);
            }
            __syncthreads();
            for (int i = t; i < nops; i += T) {
                const SOp o = ops[i];
                if (o.slot < 0 || o.kind == K_U2) continue;
                for (int p = 0; p < (o.kind == K_FSIM ? 2 : 1); ++p) {
                    double s = 0.0;
                    for (int w = 0; w < nwaves; ++w) s += red[(2 * i + p) * nwaves + w];
                    slots[o.slot + p] = s;
                }
            }
            __syncthreads();
        }
    }

    if (PARTS >= SM_GATES && J.do_fwd) copy_state(gpsi, psi, dim, t, T);
    if (PARTS >= SM_GATES && J.do_rev) {
        copy_state(glam, lam, dim, t, T);
        FinishJob F{};
        F.slots = slots;
        F.slot_ptr = J.slot_ptr;
        F.slot_idx = J.slot_idx;
        F.gate_slot = J.gate_slot;
        F.u2m = J.u2m;
        F.gate_mat = J.gate_mat;
        F.grad = J.grad ? J.grad + b * J.n_params : nullptr;
        F.gate_grad = J.gate_grad ? J.gate_grad + b * J.n_gates * 15 : nullptr;
        F.n_params = J.n_params;
        F.n_gates = J.n_gates;
        const int64_t per = 1 + int64_t(J.n_params) + (J.gate_grad ? GATE_OUTS * int64_t(J.n_gates) : 0);
        for (int64_t k = 1 + t; k < per; k += T) finish_one(F, k);   // (output 0, the energy, is written)
    }
}

}  // namespace

// a thread per pair of amplitudes, up to 256
template <typename R>
hipError_t launch_small(const SmallJob& job, int64_t batch, hipStream_t st) {
    if (batch <= 0) return hipSuccess;
    if (job.n < 2 || job.n > small_qubits<R>() || job.tab_ops > SM_OPS || job.tab_mat > SM_MAT) return hipErrorInvalidValue;
    const int nt = std::max(64, std::min(SM_THREADS, 1 << (job.n - 1)));
    auto kernel = job.gate_grad ? k_small<R, SM_COTANGENTS> : job.do_fwd ? k_small<R, SM_GATES> : k_small<R, SM_PAULI>;
    hipLaunchKernelGGL(kernel, dim3(unsigned(batch)), dim3(unsigned(nt)), SmallLds<R>(job, nt / 64).total, st, job);
    return hipGetLastError();
}
template hipError_t launch_small<float>(const SmallJob&, int64_t, hipStream_t);
template hipError_t launch_small<double>(const SmallJob&, int64_t, hipStream_t);

}  // namespace tcng
