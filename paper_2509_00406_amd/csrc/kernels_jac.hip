// Residual terms: the global residual vector and the sparse Jacobian (Sec. 4.1 Eq. 3, Sec. 6.1).
// Each element owns NRES consecutive rows of J (element e of a term: rows row_off + e NRES ...), and
// each row holds the element's stencil DOFs v * D + c in ascending order, so the pattern is fixed by
// the stencils and every value is written once by its owner: no atomics, no assembly pass. The local
// Jacobian comes from first-order duals over the element's (translation-reduced) coordinates, mapped
// back to the stencil DOFs exactly as the gradient is.
#include "kernels_common.hpp"

namespace mad {

namespace {

constexpr int kJacBlock = 256;

// One element per lane, in element order: a wave's rows are one contiguous range, written through LDS (per wave
// sv, sr) in the order of memory. Bound by memory: 1000^2 grid, 2,996,001 edges and 1,000,000 vertices
// (260 MB): 72 us on inputs that no cache holds, 131 us with a launch per term and each lane storing its own rows.
template <class Term, typename T>
__device__ __forceinline__ void jacobian_wave(const JacLaunch& L, const JacTerm& A, int64_t e0, T* sv, double* sr) {
    constexpr int NS = Term::NS, D = Term::D, KR = Term::KR, NF = NS * D, M = Term::NRES, NV = M * NF;
    const int lane = threadIdx.x & 63;
    const int64_t e = e0 + lane;
    const int n = (int)(A.n - e0 < 64 ? A.n - e0 : 64);
    bool bad = false;
    if (lane < n) {
        int vs[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) vs[s] = A.stencil[e * NS + s];
        double rest[n_inputs<Term>()];
        gather_inputs<Term>(rest, A.rest, A.n, e, nullptr, vs, nullptr, A.vdata);
        // stencil vertices in ascending order: the row's column order
        int ord[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) ord[s] = s;
#pragma unroll
        for (int a = 1; a < NS; ++a)
#pragma unroll
            for (int b = a; b > 0; --b)
                if (vs[ord[b - 1]] > vs[ord[b]]) {
                    const int tmp = ord[b];
                    ord[b] = ord[b - 1];
                    ord[b - 1] = tmp;
                }
        if (L.pattern) {
            const int64_t row0 = A.row_off + e * M, nz0 = A.nz_off + e * NV;
#pragma unroll
            for (int m = 0; m < M; ++m) {
                L.rowptr[row0 + m] = (int32_t)(nz0 + (int64_t)m * NF);
#pragma unroll
                for (int j = 0; j < NF; ++j) L.colidx[nz0 + (int64_t)m * NF + j] = vs[ord[j / D]] * D + j % D;
            }
            return;
        }
        double xs[NF];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int c = 0; c < D; ++c) {
                xs[s * D + c] = L.x[(int64_t)vs[s] * D + c];
                bad = bad || !finite(xs[s * D + c]);
            }
        double r[KR];
        if constexpr (Term::TI) {
#pragma unroll
            for (int s = 1; s < NS; ++s)
#pragma unroll
                for (int c = 0; c < D; ++c) r[(s - 1) * D + c] = xs[s * D + c] - xs[c];
        } else {
#pragma unroll
            for (int k = 0; k < KR; ++k) r[k] = xs[k];
        }
        using S1 = D1<KR, T>;
        S1 q[KR], res[M];
#pragma unroll
        for (int k = 0; k < KR; ++k) q[k] = var<S1>(k, r[k]);
        Term::template residual<S1>(q, rest, A.prm, res);
#pragma unroll
        for (int m = 0; m < M; ++m) {
            // the row over the stencil DOFs: (D_NS (x) I)^T applied to the reduced row
            T jx[NF];
            if constexpr (Term::TI) {
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    T j0 = T(0);
#pragma unroll
                    for (int s = 1; s < NS; ++s) {
                        jx[s * D + c] = res[m].g[(s - 1) * D + c];
                        j0 -= res[m].g[(s - 1) * D + c];
                    }
                    jx[c] = j0;
                }
            } else {
#pragma unroll
                for (int k = 0; k < NF; ++k) jx[k] = res[m].g[k];
            }
            sr[lane * M + m] = res[m].v;
            bad = bad || !finite(res[m].v);
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                T v = jx[j];
#pragma unroll
                for (int s = 0; s < NS; ++s)
                    if (ord[j / D] == s) v = jx[s * D + j % D];
                sv[lane * NV + m * NF + j] = v;
                bad = bad || !finite(v);
            }
        }
    }
    if (L.pattern) return;
    wave_sync();
    store_run(L.r + A.row_off + e0 * M, sr, n * M, lane);
    store_run(static_cast<T*>(L.vals) + A.nz_off + e0 * NV, sv, n * NV, lane);
    if (bad) atomicOr(L.flags, 1);
}

// all residual terms in one launch: the terms' blocks one after another, neighbouring blocks on one XCD (its L2
// then serves the vertices that they share)
template <typename T>
__global__ __launch_bounds__(kJacBlock) void k_jacobian(JacLaunch L) {
    __shared__ __align__(16) T sv[kJacBlock / 64][64 * 9];
    __shared__ __align__(16) double sr[kJacBlock / 64][64 * 3];
    const int per = (int)(gridDim.x >> 3), rest8 = (int)(gridDim.x & 7), xcd = (int)(blockIdx.x & 7);
    int64_t b = (int64_t)xcd * per + min(xcd, rest8) + (int)(blockIdx.x >> 3);
    const int w = threadIdx.x >> 6;
    for (int t = 0; t < L.n_terms; ++t) {
        const JacTerm& A = L.terms[t];
        const int64_t nb = (A.n + kJacBlock - 1) / kJacBlock;
        if (b < nb) {
            const int64_t e0 = b * kJacBlock + w * 64;
            if (e0 < A.n) {
                if (A.kind == K_RES_EDGE) jacobian_wave<TermResEdge, T>(L, A, e0, sv[w], sr[w]);
                else if (A.kind == K_RES_POSITION) jacobian_wave<TermResPosition, T>(L, A, e0, sv[w], sr[w]);
            }
            return;
        }
        b -= nb;
    }
}

}  // namespace

hipError_t launch_jacobian(const JacLaunch& L, hipStream_t s) {
    int64_t blocks = 0;
    for (int t = 0; t < L.n_terms; ++t) {
        if (L.terms[t].kind != K_RES_EDGE && L.terms[t].kind != K_RES_POSITION) return hipErrorInvalidValue;
        blocks += (L.terms[t].n + kJacBlock - 1) / kJacBlock;
    }
    if (blocks == 0) return hipSuccess;
    if (L.prec == MAD_F32) hipLaunchKernelGGL(k_jacobian<float>, dim3((unsigned)blocks), dim3(kJacBlock), 0, s, L);
    else hipLaunchKernelGGL(k_jacobian<double>, dim3((unsigned)blocks), dim3(kJacBlock), 0, s, L);
    return hipGetLastError();
}

}  // namespace mad
