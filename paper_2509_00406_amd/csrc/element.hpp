// One element: forward-mode derivatives over the stencil (Sec. 6.2), the
// optional eigenvalue clamp of the local Hessian (Sec. 7.1 Hessian
// filtering), and the map back to the stencil DOFs.
//
// Active variables are the KR = (NS-1)*D relative coordinates
// r = (D_NS (x) I_D) x with D_NS = [-1 | I] (see terms.hpp). Then
//   g_x = (D_NS (x) I)^T g_r,   H_x = (D_NS (x) I)^T H_r (D_NS (x) I),
// and H_x annihilates the D translation directions exactly.
//
// Clamp in the reduced space: let Q (NS x NS-1) be the orthonormal Helmert
// basis of the complement of the constant vector. Because H_x maps
// translations to zero, H_x = (Q (x) I) Hq (Q (x) I)^T with
// Hq = (W (x) I)^T H_r (W (x) I), W = D_NS Q, and the eigenpairs of H_x are
// those of Hq lifted by (Q (x) I) plus the D translations with eigenvalue 0.
// So clamp(H_x) = (Q (x) I) clamp(Hq) (Q (x) I)^T + max(0, eps) T, with T
// the translation projector. The eigen-decomposition runs on a KR x KR matrix
// instead of an NS*D x NS*D one (6 instead of 9 for a triangle in 3D, 9
// instead of 12 for a diamond).
#pragma once
#include <type_traits>

#include "dual.hpp"

namespace mad {

// Helmert basis: column i (0..NS-2) is (-1, ..., -1, i+1, 0, ...) / sqrt((i+1)(i+2)).
__device__ __forceinline__ constexpr double helmert(int s, int i) {
    return s <= i ? -1.0 / (i == 0 ? 1.4142135623730951 : (i == 1 ? 2.449489742783178 : 3.4641016151377544))
                  : (s == i + 1 ? double(i + 1) / (i == 0 ? 1.4142135623730951
                                                          : (i == 1 ? 2.449489742783178 : 3.4641016151377544))
                                : 0.0);
}
// W = D_NS Q: W[s][i] = Q[s+1][i] - Q[0][i]
__device__ __forceinline__ constexpr double wmat(int s, int i) { return helmert(s + 1, i) - helmert(0, i); }

// Result of one element: energy, the stencil gradient, and the Hessian kept in reduced form
// (KR x KR packed): for MODE 2 the raw Hessian in relative coordinates, for MODE 3 the clamped
// Hessian in Helmert coordinates. hfull() expands any stencil entry on demand.
template <class Term, typename T>
struct ElemOut {
    static constexpr int NF = Term::NS * Term::D;
    double f;
    T g[NF];
    T hr[Packed<Term::KR>::N];
};

// entry (i, j) of the stencil Hessian (i, j in 0..NS*D-1) from the reduced form; te = clamp floor
template <class Term, int MODE, typename T>
__device__ __forceinline__ T hfull(const ElemOut<Term, T>& o, int i, int j, T te) {
    constexpr int NS = Term::NS, D = Term::D, KR = Term::KR;
    if constexpr (!Term::TI) return o.hr[Packed<KR>::at(i, j)];   // seeded on the stencil DOFs
    const int si = i / D, ci = i % D, sj = j / D, cj = j % D;
    T acc = T(0);
    if constexpr (MODE == 2) {
        // H_x = (D_NS (x) I)^T H_r (D_NS (x) I)
#pragma unroll
        for (int a = 1; a < NS; ++a) {
            if (si != 0 && a != si) continue;
#pragma unroll
            for (int b = 1; b < NS; ++b) {
                if (sj != 0 && b != sj) continue;
                const T hv = o.hr[Packed<KR>::at((a - 1) * D + ci, (b - 1) * D + cj)];
                acc += ((si == 0) != (sj == 0)) ? -hv : hv;
            }
        }
    } else {
        // clamp(H_x) = (Q (x) I) clamp(Hq) (Q (x) I)^T + max(0, eps) T
#pragma unroll
        for (int a = 0; a < NS - 1; ++a) {
            const double qa = helmert(si, a);
            if (qa == 0.0) continue;
#pragma unroll
            for (int b = 0; b < NS - 1; ++b) {
                const double qb = helmert(sj, b);
                if (qb == 0.0) continue;
                acc += T(qa * qb) * o.hr[Packed<KR>::at(a * D + ci, b * D + cj)];
            }
        }
        if (ci == cj) acc += te * T(1.0 / NS);
    }
    return acc;
}

// Matrix-free product of one element's Hessian with the stencil vector v (Sec. 6.2, matrix-free
// mode): y = H_x v from the reduced form, without expanding H_x. MODE 2: H_x = (D (x) I)^T H_r (D (x) I),
// so u = (D (x) I) v (relative coordinates), w = H_r u, y = (D (x) I)^T w. MODE 3: H_x = (Q (x) I) Hc
// (Q (x) I)^T + te T, so u = (Q (x) I)^T v, w = Hc u, y = (Q (x) I) w + te T v (T the translation projector).
template <class Term, int MODE, typename T>
__device__ __forceinline__ void hvp_apply(const ElemOut<Term, T>& o, T te, const T (&v)[Term::NS * Term::D],
                                          T (&y)[Term::NS * Term::D]) {
    constexpr int NS = Term::NS, D = Term::D, KR = Term::KR;
    if constexpr (!Term::TI) {
        // seeded on the stencil DOFs: y = H v (the clamp, if any, is already in hr)
#pragma unroll
        for (int i = 0; i < KR; ++i) {
            T acc = T(0);
#pragma unroll
            for (int j = 0; j < KR; ++j) acc += o.hr[Packed<KR>::at(i, j)] * v[j];
            y[i] = acc;
        }
        return;
    }
    T u[KR], w[KR];
    if constexpr (MODE == 2) {
#pragma unroll
        for (int s = 1; s < NS; ++s)
#pragma unroll
            for (int c = 0; c < D; ++c) u[(s - 1) * D + c] = v[s * D + c] - v[c];
    } else {
#pragma unroll
        for (int a = 0; a < NS - 1; ++a)
#pragma unroll
            for (int c = 0; c < D; ++c) {
                T acc = T(0);
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const double q = helmert(s, a);
                    if (q != 0.0) acc += T(q) * v[s * D + c];
                }
                u[a * D + c] = acc;
            }
    }
#pragma unroll
    for (int i = 0; i < KR; ++i) {
        T acc = T(0);
#pragma unroll
        for (int j = 0; j < KR; ++j) acc += o.hr[Packed<KR>::at(i, j)] * u[j];
        w[i] = acc;
    }
    if constexpr (MODE == 2) {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            T y0 = T(0);
#pragma unroll
            for (int s = 1; s < NS; ++s) {
                y[s * D + c] = w[(s - 1) * D + c];
                y0 -= w[(s - 1) * D + c];
            }
            y[c] = y0;
        }
    } else {
#pragma unroll
        for (int c = 0; c < D; ++c) {
            T vs = T(0);
#pragma unroll
            for (int s = 0; s < NS; ++s) vs += v[s * D + c];
            const T tv = te * vs * T(1.0 / NS);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                T acc = tv;
#pragma unroll
                for (int a = 0; a < NS - 1; ++a) {
                    const double q = helmert(s, a);
                    if (q != 0.0) acc += T(q) * w[a * D + c];
                }
                y[s * D + c] = acc;
            }
        }
    }
}

// Reciprocal and reciprocal square root: the hardware's in FP32 (about 1 ulp); in FP64 the hardware's
// estimate and Newton steps, at a quarter of the instructions of the IEEE division and square root. Largest error over
// 4 million values: frcp 0.50 ulp (IEEE 1 / x 0.50), frsq 1.0 (1 / sqrt(x) 1.5), fsqrt 1.7 (sqrt(x) 0.50). fsqrt
// only sets a rotation's angle; a step that rounds it to 0.5 ulp left the clamped Hessians as they are (1.9e-15 against 64 bits,
// 101^2 shell) and took 2% more time (708^2 shell 1790 -> 1825 us).
__device__ __forceinline__ float frcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double frcp(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(fma(-x, y, 1.0), y, y);
    return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ float frsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double frsq(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    const double e = fma(-x * y, y, 1.0);   // one Newton step more, to third order
    return fma(y * e, fma(0.375, e, 0.5), y);
}
// sqrt(x) for x no smaller than the least normal number
__device__ __forceinline__ float fsqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fsqrt(double x) { return x * frsq(x); }
__device__ __forceinline__ float least_normal(float) { return 1.17549435e-38f; }
__device__ __forceinline__ double least_normal(double) { return 2.2250738585072014e-308; }

// ---- symmetric eigen-decomposition: Jacobi rotations in round-robin order --------------------
// A sweep visits every pair (p, q) once, grouped into rounds of disjoint pairs (circle method
// over M = N rounded up to even players; pairs with the padding player are skipped): the parallel
// ordering of R. P. Brent and F. T. Luk, "The solution of singular-value and symmetric eigenvalue
// problems on multiprocessor arrays" (SIAM J. Sci. Stat. Comput., 1985). Rotations
// in one round touch disjoint (p, q) planes, so their parameters depend only on entries no other
// rotation of the round changes: they are computed together, giving independent instruction
// streams. The rotation zeroing a_pq uses t = tan(phi) = 2 a_pq / (h + sgn(h) sqrt(h^2 + 4 a_pq^2)),
// h = a_qq - a_pp (the smaller root of t^2 + t h / a_pq - 1 = 0), c = 1/sqrt(1 + t^2),
// s = t c, and A <- J^T A J, V <- V J with J_pp = J_qq = c, J_pq = s, J_qp = -s.
//
// Scaled rotations (the idea of the fast Givens transformation of W. M. Gentleman, 1973, and
// S. Hammarling, 1974, applied to Jacobi rotations): the off-diagonal entries and the eigenvector
// columns are kept with a diagonal scale, 2 a_ij = d_i d_j b_ij (i != j) and V = W diag(d), while the
// diagonal of A is kept as is. A rotation in the (p, q) plane multiplies d_p and d_q by c; the stored entries then
// change by one fused multiply-add each, b_ip -= t (d_q / d_p) b_iq and b_iq += t (d_p / d_q) b_ip (the same for
// W's columns), where the plain rotation needs two products and a multiply-add. With e = 1/d^2 carried along
// (e <- e (1 + t^2)) the two factors are t d_p d_q times e_p and e_q, so no division is needed; the off-diagonal
// entries are doubled once, exactly, since 2 a_pq is what t and the diagonal take (scales that start at sqrt(2)
// instead, which FP32 rounds, made a diagonal matrix come out 6e-8 too small). c >= 1/sqrt(2), so
// after s sweeps d >= 2^(-s (N - 1) / 2): no underflow in FP32 within the sweep limit, and the
// stored entries grow by at most the inverse.
// On return A's diagonal holds the eigenvalues and W diag(d) the eigenvectors. The matrix is
// scaled to max |a_ij| = 1 first (and the eigenvalues scaled back) so squares cannot overflow.
// Returns whether the off-diagonal mass fell below tol of the Frobenius norm within max_sweeps.
__host__ __device__ constexpr int rr_players(int n) { return n + (n & 1); }
// pair k of round r of the circle method over M players: one of the two members
__host__ __device__ constexpr int rr_a(int M, int r, int k) { return k == 0 ? M - 1 : (r + k) % (M - 1); }
__host__ __device__ constexpr int rr_b(int M, int r, int k) { return k == 0 ? r : (r - k + (M - 1)) % (M - 1); }

// off-diagonal mass (of the unscaled entries) below tol of the Frobenius norm
template <int N, typename T>
__device__ __forceinline__ bool jacobi_converged(const T (&A)[Packed<N>::N], const T (&dsc)[N], T tol) {
    T off = T(0), dg = T(0);
#pragma unroll
    for (int p = 0; p < N; ++p) {
        dg += A[Packed<N>::at(p, p)] * A[Packed<N>::at(p, p)];
#pragma unroll
        for (int q = p + 1; q < N; ++q) {
            const T a = dsc[p] * dsc[q] * A[Packed<N>::at(p, q)];   // twice the entry
            off += a * a;
        }
    }
    return off <= tol * tol * (T(4) * dg + T(2) * off);
}

// one sweep: every pair once, round by round
template <int N, typename T>
__device__ __forceinline__ void jacobi_sweep(T (&A)[Packed<N>::N], T (&W)[N][N], T (&dsc)[N], T (&inv)[N]) {
    constexpr int M = rr_players(N), H = M / 2;
#pragma unroll
    for (int r = 0; r < M - 1; ++r) {
        T tn[H], ta[H], ts[H];
        // parameters of the round's rotations (independent of each other)
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const int a = rr_a(M, r, k), b = rr_b(M, r, k);
            if (a >= N || b >= N) continue;
            const int p = a < b ? a : b, q = a < b ? b : a;
            const T dd = dsc[p] * dsc[q];
            const T a2 = dd * A[Packed<N>::at(p, q)];   // 2 a_pq
            const T h2 = A[Packed<N>::at(q, q)] - A[Packed<N>::at(p, p)];
            // the least normal number keeps t finite (and 0 for a_pq = 0) where the squares underflow
            const T root = fsqrt(h2 * h2 + (a2 * a2 + least_normal(a2)));
            const T t = a2 * frcp(h2 + copysign(root, h2));
            tn[k] = t;
            ta[k] = t * a2;
            ts[k] = t * dd;
        }
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const int a = rr_a(M, r, k), b = rr_b(M, r, k);
            if (a >= N || b >= N) continue;
            const int p = a < b ? a : b, q = a < b ? b : a;
            const T w = tn[k] * tn[k] + T(1);
            const T c = frsq(w);
            const T u = ts[k] * inv[p], v = ts[k] * inv[q];
            A[Packed<N>::at(p, p)] -= T(0.5) * ta[k];
            A[Packed<N>::at(q, q)] += T(0.5) * ta[k];
            A[Packed<N>::at(p, q)] = T(0);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                if (i == p || i == q) continue;
                const T g = A[Packed<N>::at(i, p)], h = A[Packed<N>::at(i, q)];
                A[Packed<N>::at(i, p)] = g - u * h;
                A[Packed<N>::at(i, q)] = h + v * g;
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const T g = W[i][p], h = W[i][q];
                W[i][p] = g - u * h;
                W[i][q] = h + v * g;
            }
            dsc[p] *= c;
            dsc[q] *= c;
            inv[p] *= w;
            inv[q] *= w;
        }
    }
}

template <int N, typename T>
__device__ __forceinline__ bool jacobi_eig(T (&A)[Packed<N>::N], T (&W)[N][N], T (&dsc)[N], int max_sweeps, T tol) {
    T inv[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        dsc[i] = T(1);
        inv[i] = T(1);
#pragma unroll
        for (int j = 0; j < N; ++j) W[i][j] = (i == j) ? T(1) : T(0);
    }
    T amax = T(0);
#pragma unroll
    for (int i = 0; i < Packed<N>::N; ++i) amax = fmax(amax, fabs(A[i]));
    const T scale = amax > T(0) ? frcp(amax) : T(1);
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = i; j < N; ++j) A[Packed<N>::at(i, j)] *= i == j ? scale : T(2) * scale;
    bool conv = jacobi_converged<N, T>(A, dsc, tol);
    if (!conv && max_sweeps > 0) {
        // the first sweep on its own: W is still the identity and the scales one there, so the
        // products with their structural zeros and ones fold away at compile time (the element
        // kernels are built without signed zeros and non-finite values)
        jacobi_sweep<N, T>(A, W, dsc, inv);
        // The test costs about a twentieth of a sweep, and the 8x8 of a hinge and the 6x6 of a shell density rarely
        // meet the tolerance within two sweeps, so for those sizes it starts after the third (FP32, tested from the
        // first -> from the third: 1024^2 shell 1222 -> 1210 us, 700 spheres 2395 -> 2381, learned density 671 both;
        // FP64 708^2 shell 1767 -> 1789); a matrix that would have stopped sooner gets one or two more sweeps, which only
        // reduce its off-diagonal mass further. Small matrices are tested after every sweep.
        constexpr int min_sweeps = N >= 6 ? 3 : 1;
        for (int sweep = 1;; ++sweep) {
            if (sweep >= min_sweeps && jacobi_converged<N, T>(A, dsc, tol)) {
                conv = true;
                break;
            }
            if (sweep == max_sweeps) break;
            jacobi_sweep<N, T>(A, W, dsc, inv);
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) A[Packed<N>::at(i, i)] *= amax > T(0) ? amax : T(1);
    return conv;
}

template <typename T> struct JacobiTol;
template <> struct JacobiTol<float> {
    static constexpr float tol = 1.0e-6f;
    static constexpr int sweeps = 15;
};
template <> struct JacobiTol<double> {
    static constexpr double tol = 1.0e-14;
    static constexpr int sweeps = 25;
};

// What element_derivs leaves for element_clamp: the Hessian to clamp, in Helmert coordinates, Hq = (W (x) I)^T
// H_r (W (x) I); for the terms with a frame (below) the part of it that the frame leaves, the frame's axes (the
// columns of R) and, for a hinge, the unit vector of its null direction.
template <class Term, typename T, int FRAME = Term::FRAME>
struct ClampIn {
    T A[Packed<Term::KR>::N];
};
template <class Term, typename T>
struct ClampIn<Term, T, 1> {
    T A[Packed<8>::N], R[3][3], v[3];
};
template <class Term, typename T>
struct ClampIn<Term, T, 2> {
    T A[Packed<4>::N], B[3], R[3][3];
};
template <class Term, typename T>
struct ClampIn<Term, T, 3> {
    T along, across, u[3];
};

// ---- clamp in a frame of the element ----------------------------------------------------------
// Turning the element turns its Hessian, so the derivatives can be taken in orthonormal axes (u, m, n) of the
// current element, where most coordinates vanish (the compiler folds the products with them) and part of the
// Hessian is known to be zero. The eigen-decomposition of the remaining part gives the same clamped matrix.
//
// Edge (FRAME 3: a function of the length of r_1): with u along r_1 the 3 x 3 Hessian is diagonal, one value
// along u and one across it: no rotations at all.
//
// Membrane (FRAME 2: an energy of the triangle's metric r_i . r_j): u along r_1, m in its plane, n its normal.
// The second derivative of r_i . r_j couples equal axes only and its first derivative has no n part, so the
// 6 x 6 Hessian falls into a 4 x 4 in-plane matrix and a 2 x 2 matrix along n: 6 + 1 rotations of 12 and 4
// multiply-adds a sweep instead of 15 of 20, and three sweeps instead of five.
//
// Hinge (FRAME 1: a function of the dihedral angle theta): u along the hinge e, (u, m) the first face. theta
// does not change when any of e, a, b moves along u, which makes the u-u part of the Hessian zero; and the
// stretch along u of the whole element also leaves the gradient as it is, so the Hessian annihilates that
// direction v (x) u, v the unit vector of the Helmert u-coordinates. With the other two u directions in a
// basis orthogonal to v an 8 x 8 matrix remains: 28 rotations of 28 multiply-adds a sweep instead of 36 of 32,
// and four sweeps instead of five (over a wave of 64 elements of the benchmark shell, FP32 emulation).
__device__ __forceinline__ double dot3(const double (&a)[3], const double (&b)[3]) {
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}
__device__ __forceinline__ void cross3(const double (&a)[3], const double (&b)[3], double (&c)[3]) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}
// |e| to within a rounding from e.e and its reciprocal root
__device__ __forceinline__ double length_of(double ee, double il) {
    const double l = ee * il;
    return fma(0.5 * il, fma(-l, l, ee), l);
}
// The unit normal n loses its orthogonality to u as the triangle degenerates: that part is taken out again.
// m = n x u.
template <typename T>
__device__ __forceinline__ void finish_frame(const double (&u)[3], double (&m)[3], double (&n)[3]) {
    const double nu = dot3(n, u);
#pragma unroll
    for (int c = 0; c < 3; ++c) n[c] -= nu * u[c];
    if constexpr (sizeof(T) == 8) {
        const double in2 = frsq(dot3(n, n));
#pragma unroll
        for (int c = 0; c < 3; ++c) n[c] *= in2;
    }
    cross3(n, u, m);
}

// entry (i, ax; j, bx) of the Helmert-coordinate Hessian from the packed one over the relative coordinates
template <class Term, typename T>
__device__ __forceinline__ T helmert_entry(const T (&h)[Packed<Term::KR>::N], int bi, int ci, int bj, int cj) {
    constexpr int NS = Term::NS, D = Term::D, KR = Term::KR;
    T acc = T(0);
#pragma unroll
    for (int a = 0; a < NS - 1; ++a) {
        const double wa = wmat(a, bi);
        if (wa == 0.0) continue;
#pragma unroll
        for (int b = 0; b < NS - 1; ++b) {
            const double wb = wmat(b, bj);
            if (wb == 0.0) continue;
            acc += T(wa * wb) * h[Packed<KR>::at(a * D + ci, b * D + cj)];
        }
    }
    return acc;
}

// Energy and stencil gradient from first-order duals in the caller's axes, as without the clamp: the gradients of
// neighbouring elements cancel and the rounding of the element's own axes would show. (FP64 shell gradients 5e-14 instead of
// 1.3e-14; in FP32 the clamped gradient was 5 to 12% further from 64 bits than the unclamped one, and its FP64 energy 5e-16
// instead of 5e-17; the duals take 1% of a 1024^2 shell, 1200 -> 1211 us.)
template <class Term, typename T>
__device__ __forceinline__ void frame_gradient(const double (&r)[Term::KR], const double* rest, const double* prm,
                                               ElemOut<Term, T>& out) {
    using S = D1<Term::KR, T>;
    S rs[Term::KR];
#pragma unroll
    for (int i = 0; i < Term::KR; ++i) rs[i] = var<S>(i, r[i]);
    const S q = Term::template energy<S>(rs, rest, prm);
    out.f = q.v;
    const T (&gx)[Term::KR] = q.g;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T g0 = T(0);
#pragma unroll
        for (int s = 1; s < Term::NS; ++s) {
            out.g[s * 3 + c] = gx[(s - 1) * 3 + c];
            g0 -= gx[(s - 1) * 3 + c];
        }
        out.g[c] = g0;
    }
}

// hinge: position of (axis, Helmert index) in the 8 x 8 matrix: n 0-2, m 3-5, then the two u directions
__host__ __device__ constexpr int hinge_n(int i) { return i; }
__host__ __device__ constexpr int hinge_m(int i) { return 3 + i; }
__host__ __device__ constexpr int hinge_u(int k) { return 6 + k; }

// rows 1 and 2 of the reflection that takes the first unit vector to -sgn(v_0) v: an orthonormal basis of
// the complement of v
template <typename T>
__device__ __forceinline__ void complement_rows(const T (&v)[3], T (&P)[2][3]) {
    const T w0 = v[0] + copysign(T(1), v[0]), beta = frcp(T(1) + fabs(v[0]));
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const T b = beta * v[1 + k];
        P[k][0] = -b * w0;
        P[k][1] = (k == 0 ? T(1) : T(0)) - b * v[1];
        P[k][2] = (k == 1 ? T(1) : T(0)) - b * v[2];
    }
}

template <class Term, typename T>
__device__ __forceinline__ void hinge_derivs(const double (&r)[9], const double* rest, const double* prm,
                                             ElemOut<Term, T>& out, ClampIn<Term, T, 1>& in) {
    const double e[3] = {r[0], r[1], r[2]}, a[3] = {r[3], r[4], r[5]}, b[3] = {r[6], r[7], r[8]};
    double u[3], m[3], n[3];
    const double ee = dot3(e, e), il = frsq(ee), l = length_of(ee, il);
#pragma unroll
    for (int c = 0; c < 3; ++c) u[c] = e[c] * il;
    cross3(e, a, n);
    const double inn = frsq(dot3(n, n));
    // from the unrounded product: near a flat hinge theta is this small height over the first face's plane
    const double bn = dot3(n, b) * inn;
#pragma unroll
    for (int c = 0; c < 3; ++c) n[c] *= inn;
    finish_frame<T>(u, m, n);
    const double au = dot3(a, u), am = dot3(a, m), bu = dot3(b, u), bm = dot3(b, m);
    using S = HD<9, T>;
    const S rs[9] = {var<S>(0, l),  var<S>(1, 0.0), var<S>(2, 0.0), var<S>(3, au), var<S>(4, am),
                     var<S>(5, 0.0), var<S>(6, bu),  var<S>(7, bm),  var<S>(8, bn)};
    const S f = Term::template energy<S>(rs, rest, prm);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        in.R[c][0] = T(u[c]);
        in.R[c][1] = T(m[c]);
        in.R[c][2] = T(n[c]);
    }
    frame_gradient<Term, T>(r, rest, prm, out);
    const double ru[3] = {l, au, bu};
    T z[3], zz = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double q = 0.0;
#pragma unroll
        for (int s = 0; s < 3; ++s) q += helmert(s + 1, i) * ru[s];
        z[i] = T(q * frsq(l * l + au * au + bu * bu));   // any scale: keeps the squares in range
        zz += z[i] * z[i];
    }
    const T iz = frsq(zz);
#pragma unroll
    for (int i = 0; i < 3; ++i) in.v[i] = z[i] * iz;
    T P[2][3];
    complement_rows<T>(in.v, P);
    auto hq = [&](int i, int ci, int j, int cj) { return helmert_entry<Term, T>(f.h, i, ci, j, cj); };
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            if (j >= i) {
                in.A[Packed<8>::at(hinge_n(i), hinge_n(j))] = hq(i, 2, j, 2);
                in.A[Packed<8>::at(hinge_m(i), hinge_m(j))] = hq(i, 1, j, 1);
            }
            in.A[Packed<8>::at(hinge_n(i), hinge_m(j))] = hq(i, 2, j, 1);
        }
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int ax = 1; ax < 3; ++ax) {
            const T c0 = hq(0, 0, j, ax), c1 = hq(1, 0, j, ax), c2 = hq(2, 0, j, ax);
#pragma unroll
            for (int k = 0; k < 2; ++k)
                in.A[Packed<8>::at(ax == 2 ? hinge_n(j) : hinge_m(j), hinge_u(k))] =
                    P[k][0] * c0 + P[k][1] * c1 + P[k][2] * c2;
        }
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int k2 = k; k2 < 2; ++k2) in.A[Packed<8>::at(hinge_u(k), hinge_u(k2))] = T(0);
}

template <class Term, typename T>
__device__ __forceinline__ void membrane_derivs(const double (&r)[6], const double* rest, const double* prm,
                                                ElemOut<Term, T>& out, ClampIn<Term, T, 2>& in) {
    const double e[3] = {r[0], r[1], r[2]}, a[3] = {r[3], r[4], r[5]};
    double u[3], m[3], n[3];
    const double ee = dot3(e, e), aa = dot3(a, a), il = frsq(ee);
    double l = length_of(ee, il);
#pragma unroll
    for (int c = 0; c < 3; ++c) u[c] = e[c] * il;
    cross3(u, a, n);
    double nn = dot3(n, n);
    if (ee <= 0.0 || nn <= 1e-28 * aa) {
        // The energy is smooth at triangles without a plane, where any axes with u along their line serve: the
        // longer of e and a and the coordinate axis furthest from it take the places of e and a.
        double d[3], axis[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) d[c] = ee < aa ? a[c] : e[c];
        const double x = fabs(d[0]), y = fabs(d[1]), z = fabs(d[2]), top = fmax(x, fmax(y, z));
        const bool ax = x <= y && x <= z, ay = !ax && y <= z;
        axis[0] = ax ? 1.0 : 0.0;
        axis[1] = ay ? 1.0 : 0.0;
        axis[2] = ax || ay ? 0.0 : 1.0;
        if (top <= 0.0) d[1] = 1.0;   // all vertices in one point (the axis is then the first)
        const double it = top > 0.0 ? 1.0 / top : 1.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) d[c] *= it;
        const double id = frsq(dot3(d, d));
#pragma unroll
        for (int c = 0; c < 3; ++c) u[c] = d[c] * id;
        cross3(u, axis, n);
        nn = dot3(n, n);
        l = dot3(e, u);
    }
    const double inn = frsq(nn);
#pragma unroll
    for (int c = 0; c < 3; ++c) n[c] *= inn;
    finish_frame<T>(u, m, n);
    using S = HD<6, T>;
    const S rs[6] = {var<S>(0, l),          var<S>(1, 0.0),        var<S>(2, 0.0),
                     var<S>(3, dot3(a, u)), var<S>(4, dot3(a, m)), var<S>(5, 0.0)};
    const S f = Term::template energy<S>(rs, rest, prm);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        in.R[c][0] = T(u[c]);
        in.R[c][1] = T(m[c]);
        in.R[c][2] = T(n[c]);
    }
    frame_gradient<Term, T>(r, rest, prm, out);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = i; j < 4; ++j)
            in.A[Packed<4>::at(i, j)] = helmert_entry<Term, T>(f.h, i >> 1, i & 1, j >> 1, j & 1);
    in.B[0] = helmert_entry<Term, T>(f.h, 0, 2, 0, 2);
    in.B[1] = helmert_entry<Term, T>(f.h, 0, 2, 1, 2);
    in.B[2] = helmert_entry<Term, T>(f.h, 1, 2, 1, 2);
}

template <class Term, typename T>
__device__ __forceinline__ void edge_derivs(const double (&r)[3], const double* rest, const double* prm,
                                            ElemOut<Term, T>& out, ClampIn<Term, T, 3>& in) {
    const double rr = dot3(r, r), il = rr > 0.0 ? frsq(rr) : 0.0, l = length_of(rr, il);
#pragma unroll
    for (int c = 0; c < 3; ++c) in.u[c] = rr > 0.0 ? T(r[c] * il) : T(c == 0 ? 1 : 0);
    frame_gradient<Term, T>(r, rest, prm, out);
    T h0, h1;
    if constexpr (Term::NRES > 0) {
        static_assert(Term::NRES == 1, "one residual per edge");
        using S1 = D1<3, T>;
        const S1 q[3] = {var<S1>(0, l), var<S1>(1, 0.0), var<S1>(2, 0.0)};
        S1 res[1];
        Term::template residual<S1>(q, rest, prm, res);
        h0 = res[0].g[0] * res[0].g[0];
        h1 = res[0].g[1] * res[0].g[1];
    } else {
        using S = HD<3, T>;
        const S q[3] = {var<S>(0, l), var<S>(1, 0.0), var<S>(2, 0.0)};
        const S f = Term::template energy<S>(q, rest, prm);
        h0 = f.h[Packed<3>::at(0, 0)];
        h1 = f.h[Packed<3>::at(1, 1)];
    }
    constexpr double w = wmat(0, 0);
    in.along = T(w * w) * h0;
    in.across = T(w * w) * h1;
}

// blk (3 x 3 over the axes, the (i, j) block of a clamped matrix) turned back into the caller's axes
template <class Term, typename T>
__device__ __forceinline__ void rotate_block(const T (&B)[3][3], const T (&R)[3][3], int i, int j,
                                             ElemOut<Term, T>& out) {
    T t[3][3];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int b = 0; b < 3; ++b) t[c][b] = R[c][0] * B[0][b] + R[c][1] * B[1][b] + R[c][2] * B[2][b];
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (i == j && d < c) continue;
            out.hr[Packed<Term::KR>::at(3 * i + c, 3 * j + d)] = t[c][0] * R[d][0] + t[c][1] * R[d][1] + t[c][2] * R[d][2];
        }
}

// Derivatives of one element (modes 1-3): energy, stencil gradient, and the reduced Hessian --
// for MODE 2 the raw Hessian in relative coordinates (into out.hr), for MODE 3 the matrix that
// element_clamp takes (into in).
template <class Term, typename T, int MODE>
__device__ __forceinline__ void element_derivs(const double* xs, const double* rest, const double* prm,
                                               ElemOut<Term, T>& out, ClampIn<Term, T>& in) {
    constexpr int NS = Term::NS, D = Term::D, KR = Term::KR;
    double r[KR];
    if constexpr (Term::TI) {
#pragma unroll
        for (int s = 1; s < NS; ++s)
#pragma unroll
            for (int c = 0; c < D; ++c) r[(s - 1) * D + c] = xs[s * D + c] - xs[c];
    } else {
#pragma unroll
        for (int i = 0; i < KR; ++i) r[i] = xs[i];
    }
    if constexpr (MODE == 3 && Term::FRAME == 1) {
        hinge_derivs<Term, T>(r, rest, prm, out, in);
        return;
    } else if constexpr (MODE == 3 && Term::FRAME == 2) {
        membrane_derivs<Term, T>(r, rest, prm, out, in);
        return;
    } else if constexpr (MODE == 3 && Term::FRAME == 3) {
        edge_derivs<Term, T>(r, rest, prm, out, in);
        return;
    } else {
    using S = typename std::conditional<MODE == 1, D1<KR, T>, HD<KR, T>>::type;
    S f;
    if constexpr (Term::NRES > 0) {
        // residual term (Eq. 3): first-order duals give r and J; the scalar form is 1/2 |r|^2 with
        // gradient J^T r and the Gauss-Newton matrix J^T J in place of the Hessian
        using S1 = D1<KR, T>;
        S1 q[KR], res[Term::NRES];
#pragma unroll
        for (int i = 0; i < KR; ++i) q[i] = var<S1>(i, r[i]);
        Term::template residual<S1>(q, rest, prm, res);
        f = cst<S>(0.0);
#pragma unroll
        for (int m = 0; m < Term::NRES; ++m) {
            f.v += 0.5 * res[m].v * res[m].v;
            const T rv = T(res[m].v);
#pragma unroll
            for (int i = 0; i < KR; ++i) f.g[i] += rv * res[m].g[i];
            if constexpr (MODE >= 2) {
#pragma unroll
                for (int i = 0; i < KR; ++i)
#pragma unroll
                    for (int j = i; j < KR; ++j) f.h[Packed<KR>::at(i, j)] += res[m].g[i] * res[m].g[j];
            }
        }
    } else {
        S rs[KR];
#pragma unroll
        for (int i = 0; i < KR; ++i) rs[i] = var<S>(i, r[i]);
        f = Term::template energy<S>(rs, rest, prm);
    }
    out.f = f.v;
    if constexpr (!Term::TI) {
        // active variables are the stencil DOFs: no map back, no Helmert reduction
#pragma unroll
        for (int i = 0; i < KR; ++i) out.g[i] = f.g[i];
        if constexpr (MODE == 2) {
#pragma unroll
            for (int i = 0; i < Packed<KR>::N; ++i) out.hr[i] = f.h[i];
        } else if constexpr (MODE == 3) {
#pragma unroll
            for (int i = 0; i < Packed<KR>::N; ++i) in.A[i] = f.h[i];
        }
        return;
    }
#pragma unroll
    for (int c = 0; c < D; ++c) {
        T g0 = T(0);
#pragma unroll
        for (int s = 1; s < NS; ++s) {
            out.g[s * D + c] = f.g[(s - 1) * D + c];
            g0 -= f.g[(s - 1) * D + c];
        }
        out.g[c] = g0;
    }
    if constexpr (MODE == 2) {
#pragma unroll
        for (int i = 0; i < Packed<KR>::N; ++i) out.hr[i] = f.h[i];
    } else if constexpr (MODE == 3) {
#pragma unroll
        for (int i = 0; i < KR; ++i)
#pragma unroll
            for (int j = i; j < KR; ++j)
                in.A[Packed<KR>::at(i, j)] = helmert_entry<Term, T>(f.h, i / D, i % D, j / D, j % D);
    }
    }
}

// C = U diag(max(lambda, floor)) U^T (U = V diag(dsc)) of the symmetric N x N matrix A; returns whether the
// eigen-decomposition converged
template <int N, typename T>
__device__ __forceinline__ bool clamp_matrix(T (&A)[Packed<N>::N], T te, T (&C)[Packed<N>::N]) {
    T V[N][N], dsc[N];
    const bool conv = jacobi_eig<N, T>(A, V, dsc, JacobiTol<T>::sweeps, JacobiTol<T>::tol);
#pragma unroll
    for (int i = 0; i < Packed<N>::N; ++i) C[i] = T(0);
#pragma unroll
    for (int m = 0; m < N; ++m) {
        // eigenvector m is column m of V times dsc[m]: its scale squared goes with the eigenvalue
        const T lam = A[Packed<N>::at(m, m)];
        const T lp = (lam > te ? lam : te) * (dsc[m] * dsc[m]);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const T li = lp * V[i][m];
#pragma unroll
            for (int j = i; j < N; ++j) C[Packed<N>::at(i, j)] += li * V[j][m];
        }
    }
    return conv;
}

// the clamped Hessian in Helmert coordinates into out.hr; returns whether the eigen-decomposition converged
template <class Term, typename T>
__device__ __forceinline__ bool element_clamp(ClampIn<Term, T>& in, double eps, ElemOut<Term, T>& out) {
    const T te = T(eps > 0.0 ? eps : 0.0);
    if constexpr (Term::FRAME == 1) {
        T C[Packed<8>::N];
        const bool conv = clamp_matrix<8, T>(in.A, te, C);
        T P[2][3];
        complement_rows<T>(in.v, P);
        auto at = [&](int i, int j) { return C[Packed<8>::at(i, j)]; };
        T X[3][6];   // u rows against the m (0-2) and n (3-5) columns
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                X[i][j] = P[0][i] * at(hinge_m(j), hinge_u(0)) + P[1][i] * at(hinge_m(j), hinge_u(1));
                X[i][3 + j] = P[0][i] * at(hinge_n(j), hinge_u(0)) + P[1][i] * at(hinge_n(j), hinge_u(1));
            }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i; j < 3; ++j) {
                T B[3][3];
                const T p0 = P[0][i] * at(hinge_u(0), hinge_u(0)) + P[1][i] * at(hinge_u(0), hinge_u(1));
                const T p1 = P[0][i] * at(hinge_u(0), hinge_u(1)) + P[1][i] * at(hinge_u(1), hinge_u(1));
                B[0][0] = p0 * P[0][j] + p1 * P[1][j] + te * in.v[i] * in.v[j];
                B[0][1] = X[i][j];
                B[1][0] = X[j][i];
                B[0][2] = X[i][3 + j];
                B[2][0] = X[j][3 + i];
                B[1][1] = at(hinge_m(i), hinge_m(j));
                B[1][2] = at(hinge_n(j), hinge_m(i));
                B[2][1] = at(hinge_n(i), hinge_m(j));
                B[2][2] = at(hinge_n(i), hinge_n(j));
                rotate_block<Term, T>(B, in.R, i, j, out);
            }
        return conv;
    } else if constexpr (Term::FRAME == 2) {
        T C[Packed<4>::N], N2[3];
        const bool c4 = clamp_matrix<4, T>(in.A, te, C), c2 = clamp_matrix<2, T>(in.B, te, N2);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = i; j < 2; ++j) {
                T B[3][3];
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int b = 0; b < 2; ++b) B[a][b] = C[Packed<4>::at(2 * i + a, 2 * j + b)];
#pragma unroll
                for (int a = 0; a < 2; ++a) B[a][2] = B[2][a] = T(0);
                B[2][2] = N2[Packed<2>::at(i, j)];
                rotate_block<Term, T>(B, in.R, i, j, out);
            }
        return c4 && c2;
    } else if constexpr (Term::FRAME == 3) {
        const T a = in.along > te ? in.along : te, b = in.across > te ? in.across : te;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = i; j < 3; ++j)
                out.hr[Packed<3>::at(i, j)] = (a - b) * in.u[i] * in.u[j] + (i == j ? b : T(0));
        return true;
    } else {
        return clamp_matrix<Term::KR, T>(in.A, te, out.hr);
    }
}

// Evaluate one element. MODE: 0 passive, 1 gradient, 2 Hessian, 3 clamped Hessian.
// xs: stencil DOFs (NS*D, FP64). Returns false if the eigen-decomposition did not converge.
template <class Term, typename T, int MODE>
__device__ __forceinline__ bool element_eval(const double* xs, const double* rest, const double* prm, double eps,
                                             ElemOut<Term, T>& out) {
    constexpr int NS = Term::NS, D = Term::D, KR = Term::KR;
    if constexpr (MODE == 0) {
        double r[KR];
        if constexpr (Term::TI) {
#pragma unroll
            for (int s = 1; s < NS; ++s)
#pragma unroll
                for (int c = 0; c < D; ++c) r[(s - 1) * D + c] = xs[s * D + c] - xs[c];
        } else {
#pragma unroll
            for (int i = 0; i < KR; ++i) r[i] = xs[i];
        }
        out.f = Term::template energy<double>(r, rest, prm);
        return true;
    } else {
        ClampIn<Term, T> in;
        element_derivs<Term, T, MODE>(xs, rest, prm, out, in);
        if constexpr (MODE == 3) return element_clamp<Term, T>(in, eps, out);
        return true;
    }
}

}  // namespace mad
