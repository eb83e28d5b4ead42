// Helpers shared by the assembly kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "element.hpp"
#include "mad_internal.hpp"
#include "terms.hpp"

namespace mad {

constexpr int kBlock = 256;

__device__ __forceinline__ void atomic_add(float* p, float v) { unsafeAtomicAdd(p, v); }
__device__ __forceinline__ void atomic_add(double* p, double v) { unsafeAtomicAdd(p, v); }

// Finiteness by an integer test of the exponent bits, after an empty asm has hidden the value's
// origin: the element kernels are compiled with -ffinite-math-only (so that arithmetic on the
// structurally zero channels of the duals folds away), under which a floating-point test could be
// folded to "finite". The hardware still computes IEEE results; this reads them.
__device__ __forceinline__ bool finite(float v) {
    uint32_t u = __float_as_uint(v);
    asm volatile("" : "+v"(u));
    return (u & 0x7f800000u) != 0x7f800000u;
}
__device__ __forceinline__ bool finite(double v) {
    uint64_t u = (uint64_t)__double_as_longlong(v);
    asm volatile("" : "+v"(u));
    return (u & 0x7ff0000000000000ull) != 0x7ff0000000000000ull;
}

// wave-scope ordering of LDS accesses between the lanes of one wave
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// n values from LDS (16-byte aligned) to memory, a wave together, 16 bytes a lane where memory need only be
// aligned to the value. For results that are written once, in whole lines, and not read
// again: the stores pass by the L2, which keeps x and the element data (rows of a 1000^2 cloth: 187 -> 146 us).
template <typename T>
__device__ __forceinline__ void store_run(T* to, const T* from, int n, int lane) {
    constexpr int N = 16 / sizeof(T);
    typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
    typedef vec vec_any __attribute__((aligned(sizeof(T))));
    const int nv = n / N;
    for (int k = lane; k < nv; k += 64)
        __builtin_nontemporal_store(reinterpret_cast<const vec*>(from)[k], reinterpret_cast<vec_any*>(to + k * N));
    const int k = nv * N + lane;
    if (k < n) __builtin_nontemporal_store(from[k], to + k);
}

// triangle quality 4 sqrt(3) A / (l0^2 + l1^2 + l2^2): 1 for equilateral, 0 for degenerate
__device__ __forceinline__ double tri_quality3(const double* a, const double* b, const double* c) {
    const double e1[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
    const double e2[3] = {c[0] - a[0], c[1] - a[1], c[2] - a[2]};
    const double e3[3] = {c[0] - b[0], c[1] - b[1], c[2] - b[2]};
    const double n[3] = {e1[1] * e2[2] - e1[2] * e2[1], e1[2] * e2[0] - e1[0] * e2[2], e1[0] * e2[1] - e1[1] * e2[0]};
    const double l2 = e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2] + e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2] +
                      e3[0] * e3[0] + e3[1] * e3[1] + e3[2] * e3[2];
    const double area2 = sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    return l2 > 0.0 ? 2.0 * 1.7320508075688772 * area2 / l2 : 0.0;
}
__device__ __forceinline__ double tri_quality2(const double* a, const double* b, const double* c) {
    const double e1[2] = {b[0] - a[0], b[1] - a[1]}, e2[2] = {c[0] - a[0], c[1] - a[1]};
    const double e3[2] = {c[0] - b[0], c[1] - b[1]};
    const double l2 = e1[0] * e1[0] + e1[1] * e1[1] + e2[0] * e2[0] + e2[1] * e2[1] + e3[0] * e3[0] + e3[1] * e3[1];
    const double area2 = fabs(e1[0] * e2[1] - e1[1] * e2[0]);
    return l2 > 0.0 ? 2.0 * 1.7320508075688772 * area2 / l2 : 0.0;
}

// worst current-triangle quality of an element (diamonds: the worse of its two faces)
template <class Term> __device__ __forceinline__ double quality(const double* xs) {
    if constexpr (Term::NS == 3 && Term::D == 3) {
        return tri_quality3(xs, xs + 3, xs + 6);
    } else if constexpr (Term::NS == 3 && Term::D == 2) {
        return tri_quality2(xs, xs + 2, xs + 4);
    } else if constexpr (Term::NS == 4) {
        const double q1 = tri_quality3(xs, xs + 3, xs + 6);   // (x0, x1, x2)
        const double q2 = tri_quality3(xs, xs + 9, xs + 3);   // (x0, x3, x1)
        return q1 < q2 ? q1 : q2;
    } else {
        return 1.0;
    }
}

// Number of per-element inputs a term's energy reads: rest data, then (shell-feature terms) the
// three unit vertex normals, then (learned density) the 28 network outputs.
template <class Term> constexpr int n_inputs() {
    return (Term::NREST + Term::NAUX + Term::NPSI + Term::NVD) > 0 ? Term::NREST + Term::NAUX + Term::NPSI + Term::NVD
                                                                    : 1;
}

// Gather one element's inputs: rest SoA [NREST][n], normals [nv][3] at the element's global
// vertices gv[], network outputs SoA [28][n] (FP32), the caller's per-vertex data [nv][NVD] at gv[].
template <class Term>
__device__ __forceinline__ void gather_inputs(double (&in)[n_inputs<Term>()], const double* rest, int64_t n, int64_t e,
                                              const double* normals, const int* gv, const float* psi,
                                              const double* vdata) {
#pragma unroll
    for (int k = 0; k < Term::NREST; ++k) in[k] = rest[(int64_t)k * n + e];
    if constexpr (Term::NAUX > 0) {
#pragma unroll
        for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int c = 0; c < 3; ++c) in[Term::NREST + 3 * s + c] = normals[(int64_t)gv[s] * 3 + c];
    }
    if constexpr (Term::NPSI > 0) {
#pragma unroll
        for (int k = 0; k < Term::NPSI; ++k) in[Term::NREST + Term::NAUX + k] = double(psi[(int64_t)k * n + e]);
    }
    if constexpr (Term::NVD > 0) {
        constexpr int B = Term::NREST + Term::NAUX + Term::NPSI;
#pragma unroll
        for (int s = 0; s < Term::NS; ++s)
#pragma unroll
            for (int k = 0; k < Term::NVD; ++k) in[B + s * Term::NVD + k] = vdata[(int64_t)gv[s] * Term::NVD + k];
    }
}

// An element's outputs are all finite iff the sum of their magnitudes is (a NaN or an infinity
// anywhere reaches the sum; finite outputs cannot overflow it at the magnitudes that occur here).
template <class Term, typename T>
__device__ __forceinline__ bool out_finite(const ElemOut<Term, T>& o, int mode) {
    constexpr int NF = Term::NS * Term::D;
    T acc = T(0);
    if (mode >= 1) {
#pragma unroll
        for (int i = 0; i < NF; ++i) acc += fabs(o.g[i]);
    }
    if (mode >= 2) {
#pragma unroll
        for (int i = 0; i < Packed<Term::KR>::N; ++i) acc += fabs(o.hr[i]);
    }
    return finite(o.f) && finite(acc);
}

template <class Term, typename T, typename U>
__device__ __forceinline__ void convert_out(const ElemOut<Term, U>& in, ElemOut<Term, T>& out) {
    constexpr int NF = Term::NS * Term::D;
    out.f = in.f;
#pragma unroll
    for (int i = 0; i < NF; ++i) out.g[i] = T(in.g[i]);
#pragma unroll
    for (int i = 0; i < Packed<Term::KR>::N; ++i) out.hr[i] = T(in.hr[i]);
}

__device__ __forceinline__ void block_reduce_store(double v, double* red, double* out) {
    red[threadIdx.x] = v;
    __syncthreads();
#pragma unroll
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// Energy of component c by one workgroup: partial[t * n_patch + p], patches of component c are
// [comp_patch_ptr[c], comp_patch_ptr[c + 1]). Each lane sums a fixed strided subset in a fixed order, then a fixed tree.
__device__ __forceinline__ void energy_component(const EnergyArgs& E, int c, double* red) {
    const int pb = E.comp_patch_ptr[c], pe = E.comp_patch_ptr[c + 1];
    double acc = 0.0;
    for (int t = 0; t < E.n_terms; ++t) {
        const double* pt = E.partial + (int64_t)t * E.n_patch;
        int i = pb + (int)threadIdx.x;
        // eight loads in flight, then the additions in the same order as one at a time
        for (; i + 7 * kBlock < pe; i += 8 * kBlock) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = pt[i + k * kBlock];
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += v[k];
        }
        for (; i < pe; i += kBlock) acc += pt[i];
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (E.batched) E.energy[1 + c] = red[0];
        if (E.n_comp == 1) E.energy[0] = red[0];
        else E.comp_out[c] = red[0];
    }
}

// sum of red[0, kBlock) in a fixed tree order, by the workgroup's first wave (no barrier: the tree's upper two
// levels are each lane's own four values, the others shuffles); red is already filled and visible
__device__ __forceinline__ void block_sum_store(const double* red, double* out) {
    static_assert(kBlock == 256, "four values per lane");
    if (threadIdx.x >= 64) return;
    const int l = threadIdx.x;
    double v = (red[l] + red[l + 128]) + (red[l + 64] + red[l + 192]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
    if (l == 0) *out = v;
}

}  // namespace mad
