// Row-owned assembly of light problems (every term an edge or a vertex term: springs, inertia, edge-length and
// positional residuals). An edge's Hessian touches two rows, so a row computes the elements around its vertex
// itself: every edge twice instead of once (some 80 instructions each), and in exchange nothing is
// accumulated across lanes of different rows: no LDS atomics, no lock, no halo partials and no gather, each
// block and gradient entry written once, in the order of memory, and summed in a fixed order.
//
// One lane per block of the Hessian: a lane with an off-diagonal block (r, c) evaluates the edge (r, c), the lane
// with the diagonal one the vertex terms. A wave takes a unit of consecutive rows with at most 64 blocks
// (nine rows of a triangle grid), so the lanes are full whatever the valences; a longer row is a unit
// of its own and goes through the wave in passes. Each lane leaves its contribution to its row's diagonal block and
// gradient in LDS, the lanes then share out the (row, component) sums over the row's lanes, and the blocks leave
// through LDS in the order of memory (a unit's blocks are one contiguous range).
//
// 1000^2 cloth (2,996,001 springs, 1,000,000 vertex terms, FP32, clamped): 175 us on inputs that no cache holds
// (130 us on warm ones) where the patch kernel took 344 and its gather 26; it moves 162 MB in and 280 MB out of
// the 392 MB that it cannot do without, 2.5 TB/s. Each unit's columns are loaded while the unit before it is worked
// on, and the row sums keep eight LDS reads in flight (189 -> 179 us); five waves per SIMD (96 registers) against
// four 200 -> 179 us, six spill. Two spilled registers cost 8% (190 us), so a unit's table entry, which all lanes
// hold alike, moves to scalar registers as soon as it has arrived.
#include "kernels_common.hpp"

namespace mad {

namespace {

constexpr int kRowWaves = kBlock / 64;
// What a lane leaves in LDS for its row: the diagonal block (upper half: 6 in 3D) or the product (3), then the gradient
// (3); an odd stride. Gradients alone take a third of a Hessian's LDS, so that it does not limit the waves (FP64
// gradient of a 1000^2 cloth 95 -> 87 us; through patches 89).
constexpr int row_comps(int mode, bool hvp) { return mode >= 2 ? (hvp ? 7 : 9) : mode == 1 ? 3 : 1; }
constexpr int row_grad(int mode, bool hvp) { return mode >= 2 ? (hvp ? 3 : 6) : 0; }

// The contributions of a lane's terms, which add up. Energy, gradient and the unclamped Hessian are the caller's
// axes' own derivatives. (Through the edge's axes, below, the unclamped Hessian of a 200^2 cloth was 1.2 times as far from
// 64 bits in FP32 and 1.8 times in FP64.)
// Clamped: an edge term is a function of the edge's length l, so its Hessian is along u u^T + across (I - u u^T)
// with the edge's unit vector u, from forward mode over the edge's own axes, where the two coordinates across it
// vanish (element.hpp). A vertex term is a quadratic with an isotropic Hessian (along = across).
template <typename T, int MODE>
struct RowPart {
    double f;
    T g[3];              // gradient at the column's vertex
    T along, across;     // clamped
};
template <typename T>
struct RowPart<T, 2> {
    double f;
    T g[3], h[6];
};
template <typename T, int MODE>
__device__ __forceinline__ T hess_size(const RowPart<T, MODE>& P) {
    if constexpr (MODE == 2) return fabs(P.h[0]) + fabs(P.h[1]) + fabs(P.h[2]) + fabs(P.h[3]) + fabs(P.h[4]) + fabs(P.h[5]);
    else return fabs(P.along) + fabs(P.across);
}

template <class Term, typename T, int MODE>
__device__ __forceinline__ void add_edge(const RowTerm& A, const double (&in)[4], const double (&r)[3], double l,
                                         double il, T te, RowPart<T, MODE>& P) {
    static_assert(Term::NREST <= 2 && Term::NS == 2 && Term::FRAME == 3 && Term::NRES <= 1, "an edge term");
    const double rest[2] = {in[0], in[1]};
    if constexpr (MODE == 0) {
        P.f += Term::template energy<double>(r, rest, A.prm);
        return;
    } else if constexpr (MODE == 3 && sizeof(T) == 4) {
        // along the edge in FP64, rounded once: no less exact, and in fewer registers than FP32 duals of three
        P.f += Term::template energy<double>(r, rest, A.prm);
        using S = D1<3, double>;
        const S q[3] = {var<S>(0, l), var<S>(1, 0.0), var<S>(2, 0.0)};
        const double gl = Term::template energy<S>(q, rest, A.prm).g[0] * il;
#pragma unroll
        for (int c = 0; c < 3; ++c) P.g[c] += T(gl * r[c]);
    } else if constexpr (Term::NRES > 0) {
        using S = D1<3, T>;
        const S q[3] = {var<S>(0, r[0]), var<S>(1, r[1]), var<S>(2, r[2])};
        S res[1];
        Term::template residual<S>(q, rest, A.prm, res);
        P.f += 0.5 * res[0].v * res[0].v;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            P.g[a] += T(res[0].v) * res[0].g[a];
            if constexpr (MODE == 2)
#pragma unroll
                for (int b = a; b < 3; ++b) P.h[Packed<3>::at(a, b)] += res[0].g[a] * res[0].g[b];
        }
    } else {
        using S = typename std::conditional<MODE == 2, HD<3, T>, D1<3, T>>::type;
        const S q[3] = {var<S>(0, r[0]), var<S>(1, r[1]), var<S>(2, r[2])};
        const S f = Term::template energy<S>(q, rest, A.prm);
        P.f += f.v;
#pragma unroll
        for (int c = 0; c < 3; ++c) P.g[c] += f.g[c];
        if constexpr (MODE == 2)
#pragma unroll
            for (int k = 0; k < 6; ++k) P.h[k] += f.h[k];
    }
    if constexpr (MODE == 3) {
        T h0, h1;
        if constexpr (Term::NRES > 0) {
            using S = D1<3, T>;
            const S q[3] = {var<S>(0, l), var<S>(1, 0.0), var<S>(2, 0.0)};
            S res[1];
            Term::template residual<S>(q, rest, A.prm, res);
            h0 = res[0].g[0] * res[0].g[0];
            h1 = res[0].g[1] * res[0].g[1];
        } else {
            using S = HD<3, T>;
            const S q[3] = {var<S>(0, l), var<S>(1, 0.0), var<S>(2, 0.0)};
            const S f = Term::template energy<S>(q, rest, A.prm);
            h0 = f.h[Packed<3>::at(0, 0)];
            h1 = f.h[Packed<3>::at(1, 1)];
        }
        // clamped in the orthonormal coordinate (x_1 - x_0) / sqrt(2), whose Hessian is twice this one; the
        // floor of the translations is added where the blocks are formed
        P.along += T(0.5) * fmax(T(2) * h0, te);
        P.across += T(0.5) * fmax(T(2) * h1, te);
    }
}

template <typename T, int MODE>
__device__ __forceinline__ void add_isotropic(RowPart<T, MODE>& P, T h, T te) {
    if constexpr (MODE == 2) {
#pragma unroll
        for (int c = 0; c < 3; ++c) P.h[Packed<3>::at(c, c)] += h;
    } else if constexpr (MODE == 3) {
        P.along += fmax(h, te);
        P.across += fmax(h, te);
    }
}

template <class Term, typename T, int MODE>
__device__ __forceinline__ void add_vertex(const RowTerm& A, const double (&in)[4], const double (&x)[3], T te,
                                           RowPart<T, MODE>& P) {
    static_assert(Term::NVD == 4 && Term::NS == 1 && Term::NREST == 0, "a vertex term");
    if constexpr (MODE == 0) {
        P.f += Term::template energy<double>(x, in, A.prm);
        return;
    } else if constexpr (Term::NRES > 0) {
        using S = D1<3, T>;
        const S q[3] = {var<S>(0, x[0]), var<S>(1, x[1]), var<S>(2, x[2])};
        S res[Term::NRES];
        Term::template residual<S>(q, in, A.prm, res);
        T h = T(0);
#pragma unroll
        for (int m = 0; m < Term::NRES; ++m) {
            P.f += 0.5 * res[m].v * res[m].v;
#pragma unroll
            for (int c = 0; c < 3; ++c) P.g[c] += T(res[m].v) * res[m].g[c];
            h += res[m].g[0] * res[m].g[0];
        }
        add_isotropic<T, MODE>(P, h, te);
    } else {
        using S = typename std::conditional<MODE == 1, D1<3, T>, HD<3, T>>::type;
        const S q[3] = {var<S>(0, x[0]), var<S>(1, x[1]), var<S>(2, x[2])};
        const S f = Term::template energy<S>(q, in, A.prm);
        P.f += f.v;
#pragma unroll
        for (int c = 0; c < 3; ++c) P.g[c] += f.g[c];
        if constexpr (MODE >= 2) add_isotropic<T, MODE>(P, f.h[0], te);
    }
}

// what an edge or vertex term reads per element: its rest data (edge), its vertex data (vertex)
__device__ __forceinline__ void edge_inputs(const RowTerm& A, int edge, double (&in)[4]) {
    in[0] = A.nrest > 0 ? A.rest[edge] : 0.0;
    in[1] = A.nrest > 1 ? A.rest[A.n + edge] : 0.0;
}
__device__ __forceinline__ void vertex_inputs(const RowTerm& A, int row, double (&in)[4]) {
#pragma unroll
    for (int k = 0; k < 4; ++k) in[k] = A.vdata[(int64_t)row * 4 + k];
}

__device__ __forceinline__ int2 uniform2(int2 v) {
    return int2{__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y)};
}

// HVP: the matrix-free product instead of the blocks (modes 2 and 3)
template <typename T, int MODE, bool HVP>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 5 : 3))) void k_eval_rows(RowLaunch L) {
    constexpr int kRowComps = row_comps(MODE, HVP), kGrad = row_grad(MODE, HVP);
    __shared__ __align__(16) T s_part[kRowWaves][64 * kRowComps];   // the lanes' contributions, then the unit's blocks
    __shared__ T s_sum[kRowWaves][64 * kRowComps];    // the rows' sums
    __shared__ int s_off[kRowWaves][65];              // first block of each row, from the unit's first
    __shared__ int s_dia[kRowWaves][64];              // diagonal block of each row (units longer than a wave)
    __shared__ unsigned char s_start[kRowWaves][64];  // a row starts at this lane
    __shared__ double s_energy[kRowWaves];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    // neighbouring chunks on one XCD, whose L2 then holds their part of x: workgroups go to the XCDs in turn
    const int per = (int)(gridDim.x >> 3), rest8 = (int)(gridDim.x & 7), xcd = (int)(blockIdx.x & 7);
    const int chunk = xcd * per + min(xcd, rest8) + (int)(blockIdx.x >> 3);
    T* part = s_part[w];
    T* sum = s_sum[w];
    int* off = s_off[w];
    const T te = T(L.eps > 0.0 ? L.eps : 0.0);
    double esum = 0.0;
    bool bad = false;
    // A unit's table entry, then its columns, edges and row starts are loaded while the unit before it is worked
    // on, so a unit waits for its vertices and element data only.
    const int u_end = L.chunk_unit[chunk + 1];
    int u = L.chunk_unit[chunk] + w;
    int2 at{0, 0}, to_at{0, 0};
    int col_l = 0, edge_l = -1, start_l = 0;
    auto fetch_unit = [&](int q, int2& a, int2& b) {
        a = L.unit[q];
        b = L.unit[q + 1];
    };
    auto fetch_lanes = [&](int2 a, int2 b, int& c, int& e, int& o) {
        if (lane < b.y - a.y) {
            c = L.colidx[a.y + lane];
            e = L.edge[a.y + lane];
        }
        if (lane < b.x - a.x) o = L.rowptr[a.x + lane] - a.y;
    };
    if (u < u_end) {
        fetch_unit(u, at, to_at);
        fetch_lanes(at, to_at, col_l, edge_l, start_l);
    }
    for (; u < u_end; u += kRowWaves) {
        const int row0 = __builtin_amdgcn_readfirstlane(at.x), nrows = __builtin_amdgcn_readfirstlane(to_at.x) - row0;
        const int k0 = __builtin_amdgcn_readfirstlane(at.y), nb = __builtin_amdgcn_readfirstlane(to_at.y) - k0;
        const bool single = nb <= 64;
        int2 next_at{0, 0}, next_to{0, 0};
        const bool more = __builtin_amdgcn_readfirstlane(u + kRowWaves) < u_end;
        if (more) fetch_unit(u + kRowWaves, next_at, next_to);
        if (lane < nrows) off[lane] = start_l;
        if (lane == 0) off[nrows] = nb;
        if (!single)
            for (int i = lane; i < nrows * kRowComps; i += 64) sum[i] = T(0);
        int next_col = 0, next_edge = -1, next_start = 0;
        for (int p0 = 0; p0 < nb; p0 += 64) {
            const bool have = p0 + lane < nb;
            int col = col_l, edge = edge_l;
            if (p0 > 0) {
                col = have ? L.colidx[k0 + p0 + lane] : 0;
                edge = have ? L.edge[k0 + p0 + lane] : -1;
            }
            const bool is_edge = have && edge >= 0;
            double xc[3] = {0.0, 0.0, 0.0}, xr[3] = {0.0, 0.0, 0.0};
            double in[4] = {0.0, 0.0, 0.0, 0.0};   // the element data of the lane's first term
            if (have) {
#pragma unroll
                for (int c = 0; c < 3; ++c) xc[c] = L.x[(int64_t)col * 3 + c];
            }
            if (is_edge && L.n_edge > 0) edge_inputs(L.edges[0], edge, in);
            // the row of every lane: row starts as bits of a mask
            s_start[w][lane] = 0;
            wave_sync();
            const int mine = lane < nrows ? off[lane] - p0 : 64;
            if (mine > 0 && mine < 64) s_start[w][mine] = 1;
            wave_sync();
            const unsigned long long starts = __ballot(s_start[w][lane] != 0);
            const int first = __popcll(__ballot(mine <= 0)) - 1;
            const int i = first + __popcll(starts & (~0ull >> (63 - lane)));
            const int row = row0 + i;
            const bool dia = have && col == row;
            if (have) {
#pragma unroll
                for (int c = 0; c < 3; ++c) xr[c] = L.x[(int64_t)row * 3 + c];
            }
            if (dia && L.n_vert > 0) vertex_inputs(L.verts[0], row, in);
            if (p0 == 0 && more) {
                next_at = uniform2(next_at);
                next_to = uniform2(next_to);
                fetch_lanes(next_at, next_to, next_col, next_edge, next_start);
            }
            RowPart<T, MODE> P{};
            T d[3] = {T(0), T(0), T(0)}, fl = T(0);   // clamped: u; floor of the translations, summed over the edge terms
            if (is_edge) {
                double r[3];   // from the row's vertex to the column's
#pragma unroll
                for (int c = 0; c < 3; ++c) r[c] = xc[c] - xr[c];
                double l = 0.0, il = 0.0;
                if constexpr (MODE == 3) {
                    const double rr = dot3(r, r);
                    il = rr > 0.0 ? frsq(rr) : 0.0;
                    l = length_of(rr, il);
#pragma unroll
                    for (int c = 0; c < 3; ++c) d[c] = rr > 0.0 ? T(r[c] * il) : T(c == 0 ? 1 : 0);
                }
                for (int t = 0; t < L.n_edge;) {
                    const RowTerm& A = L.edges[t];
                    if (A.kind == K_SPRING) add_edge<TermSpring, T, MODE>(A, in, r, l, il, te, P);
                    else if (A.kind == K_RES_EDGE) add_edge<TermResEdge, T, MODE>(A, in, r, l, il, te, P);
                    else add_edge<TermEdgeSqlen, T, MODE>(A, in, r, l, il, te, P);
                    if (MODE == 3) fl += T(0.5) * te;
                    if (++t < L.n_edge) edge_inputs(L.edges[t], edge, in);
                }
            } else if (dia) {
                for (int t = 0; t < L.n_vert;) {
                    const RowTerm& A = L.verts[t];
                    if (A.kind == K_INERTIA) add_vertex<TermInertia, T, MODE>(A, in, xr, te, P);
                    else add_vertex<TermResPosition, T, MODE>(A, in, xr, te, P);
                    if (++t < L.n_vert) vertex_inputs(L.verts[t], row, in);
                }
            }
            esum += row <= col ? P.f : 0.0;
            // a position that is not finite shows in the energy of every term that reads it (and a vertex that no
            // term reads may hold anything)
            bad = bad || !finite(P.f) || !finite(fabs(P.g[0]) + fabs(P.g[1]) + fabs(P.g[2]) + hess_size<T, MODE>(P));
            // the row's own part of the element: gradient, and diagonal block or product
            T* to = part + lane * kRowComps;
            if constexpr (MODE >= 1) {
                if (have && L.want_grad)
#pragma unroll
                    for (int c = 0; c < 3; ++c) to[kGrad + c] = dia ? P.g[c] : -P.g[c];
            }
            if constexpr (MODE >= 2) {
                if (have) {
                    if constexpr (HVP) {
                        T v[3], w[3], along = T(0);   // of the row's vertex; less the column's
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            v[c] = T(L.v[(int64_t)row * 3 + c]);
                            w[c] = v[c] - (dia ? T(0) : T(L.v[(int64_t)col * 3 + c]));
                            along += d[c] * w[c];
                        }
                        if constexpr (MODE == 3) along *= P.along - P.across;
#pragma unroll
                        for (int a = 0; a < 3; ++a) {
                            if constexpr (MODE == 2)
                                to[a] = P.h[Packed<3>::at(a, 0)] * w[0] + P.h[Packed<3>::at(a, 1)] * w[1] + P.h[Packed<3>::at(a, 2)] * w[2];
                            else
                                to[a] = P.across * w[a] + along * d[a] + fl * (T(2) * v[a] - w[a]);
                        }
                    } else {
#pragma unroll
                        for (int a = 0; a < 3; ++a)
#pragma unroll
                            for (int b = a; b < 3; ++b) {
                                const int k = Packed<3>::at(a, b);
                                if constexpr (MODE == 2) to[k] = P.h[k];
                                else to[k] = (P.along - P.across) * d[a] * d[b] + (a == b ? P.across + fl : T(0));
                            }
                    }
                }
            }
            if constexpr (MODE >= 1) {
                wave_sync();
                auto row_sums = [&](auto count, auto zero, int c0) {
                    using A = decltype(zero);
                    constexpr int NC = decltype(count)::value;
                    for (int k = lane; k < nrows * NC; k += 64) {
                        const int j = k / NC, c = c0 + k - j * NC;
                        const int b = max(off[j] - p0, 0), e = min(off[j + 1] - p0, 64);
                        A acc = single ? A(0) : A(sum[j * kRowComps + c]);
                        for (int l = b; l < e; l += 8) {   // eight reads in flight, added in order
                            T q[8];
#pragma unroll
                            for (int m = 0; m < 8; ++m) q[m] = part[min(l + m, e - 1) * kRowComps + c];
#pragma unroll
                            for (int m = 0; m < 8; ++m) acc += l + m < e ? A(q[m]) : A(0);
                        }
                        sum[j * kRowComps + c] = T(acc);
                    }
                };
                if constexpr (MODE >= 2) {
                    if constexpr (HVP) row_sums(std::integral_constant<int, 3>{}, T(0), 0);
                    else row_sums(std::integral_constant<int, 6>{}, T(0), 0);
                }
                if (L.want_grad) row_sums(std::integral_constant<int, 3>{}, 0.0, kGrad);
                wave_sync();
            }
            if constexpr (MODE >= 2) {
                if constexpr (!HVP) {
                    T* H = static_cast<T*>(L.hess) + (int64_t)(k0 + p0) * 9;
                    if (have) {
                        const T* q = sum + i * kRowComps;
                        T blk[9];
#pragma unroll
                        for (int a = 0; a < 3; ++a)
#pragma unroll
                            for (int b = 0; b < 3; ++b) {
                                T o;
                                if constexpr (MODE == 2) o = -P.h[Packed<3>::at(a, b)];
                                else o = (P.across - P.along) * d[a] * d[b] + (a == b ? fl - P.across : T(0));
                                blk[3 * a + b] = dia ? q[Packed<3>::at(a, b)] : o;
                            }
                        if (single) {
#pragma unroll
                            for (int k = 0; k < 9; ++k) part[lane * 9 + k] = blk[k];
                        } else if (dia) {
                            s_dia[w][i] = k0 + p0 + lane;
                        } else {
#pragma unroll
                            for (int k = 0; k < 9; ++k) H[lane * 9 + k] = blk[k];
                        }
                    }
                    if (single) {
                        wave_sync();
                        store_run(H, part, nb * 9, lane);
                    }
                }
            }
            wave_sync();   // part is read before the next pass writes it
        }
        wave_sync();
        if constexpr (MODE >= 2) {
            if constexpr (HVP) {
                for (int k = lane; k < nrows * 3; k += 64)
                    static_cast<T*>(L.y)[(int64_t)row0 * 3 + k] = sum[(k / 3) * kRowComps + k % 3];
            } else if (!single) {
                for (int k = lane; k < nrows * 9; k += 64) {
                    const int j = k / 9, q = k - j * 9;
                    static_cast<T*>(L.hess)[(int64_t)s_dia[w][j] * 9 + q] =
                        sum[j * kRowComps + Packed<3>::at(q / 3, q % 3)];
                }
            }
        }
        if constexpr (MODE >= 1) {
            if (L.want_grad)
                for (int k = lane; k < nrows * 3; k += 64)
                    static_cast<T*>(L.grad)[(int64_t)row0 * 3 + k] = sum[(k / 3) * kRowComps + kGrad + k % 3];
        }
        wave_sync();   // the sums are read before the next unit writes them
        at = next_at;
        to_at = next_to;
        col_l = next_col;
        edge_l = next_edge;
        start_l = next_start;
    }
    if (bad) atomicOr(L.flags, 1);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) esum += __shfl_down(esum, o);
    if (lane == 0) s_energy[w] = esum;
    __syncthreads();
    if (threadIdx.x == 0) {
        double e = s_energy[0];
        for (int k = 1; k < kRowWaves; ++k) e += s_energy[k];
        L.partial[chunk] = e;
    }
}

template <typename T>
hipError_t launch_rows(const RowLaunch& L, hipStream_t s) {
    const dim3 grid(L.n_chunks), block(kBlock);
    switch (L.mode) {
    case 0: hipLaunchKernelGGL((k_eval_rows<T, 0, false>), grid, block, 0, s, L); break;
    case 1: hipLaunchKernelGGL((k_eval_rows<T, 1, false>), grid, block, 0, s, L); break;
    case 2:
        if (L.hvp) hipLaunchKernelGGL((k_eval_rows<T, 2, true>), grid, block, 0, s, L);
        else hipLaunchKernelGGL((k_eval_rows<T, 2, false>), grid, block, 0, s, L);
        break;
    case 3:
        if (L.hvp) hipLaunchKernelGGL((k_eval_rows<T, 3, true>), grid, block, 0, s, L);
        else hipLaunchKernelGGL((k_eval_rows<T, 3, false>), grid, block, 0, s, L);
        break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

__device__ __forceinline__ int32_t block_of(const int32_t* rowptr, const int32_t* colidx, int32_t r, int32_t c) {
    int32_t lo = rowptr[r], hi = rowptr[r + 1] - 1;
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (colidx[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

__global__ void k_fill_i32(int32_t* a, int64_t n, int32_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a[i] = v;
}

__global__ void k_block_edges(const int32_t* edges, int64_t n, const int32_t* rowptr, const int32_t* colidx,
                              int32_t* edge, int32_t* flags) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int32_t a = edges[2 * e], b = edges[2 * e + 1];
    const int32_t k = block_of(rowptr, colidx, a, b), l = block_of(rowptr, colidx, b, a);
    if (colidx[k] != b || colidx[l] != a) {
        atomicOr(flags + 1, kFlagSlotMissing);
        return;
    }
    edge[k] = (int32_t)e;
    edge[l] = (int32_t)e;
}

__global__ void k_unit_blocks(const int32_t* rowptr, int2* unit, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) unit[i].y = rowptr[unit[i].x];
}

__global__ void k_move_edges(const int32_t* from, int64_t n, const int32_t* map, int32_t* to) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) to[map[i]] = from[i];
}

unsigned blocks_of(int64_t n) { return (unsigned)std::max<int64_t>(1, (n + 255) / 256); }

}  // namespace

hipError_t launch_eval_rows(const RowLaunch& L, hipStream_t s) {
    if (L.n_chunks <= 0) return hipSuccess;
    return L.prec == MAD_F32 ? launch_rows<float>(L, s) : launch_rows<double>(L, s);
}

hipError_t launch_block_edges(const int32_t* edges, int64_t n_edges, const int32_t* rowptr, const int32_t* colidx,
                              int64_t nnzb, int32_t* edge, int32_t* flags, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_of(nnzb)), dim3(256), 0, s, edge, nnzb, -1);
    if (n_edges > 0)
        hipLaunchKernelGGL(k_block_edges, dim3(blocks_of(n_edges)), dim3(256), 0, s, edges, n_edges, rowptr, colidx,
                           edge, flags);
    return hipGetLastError();
}

hipError_t launch_unit_blocks(const int32_t* rowptr, int32_t* unit, int64_t n_entries, hipStream_t s) {
    hipLaunchKernelGGL(k_unit_blocks, dim3(blocks_of(n_entries)), dim3(256), 0, s, rowptr,
                       reinterpret_cast<int2*>(unit), n_entries);
    return hipGetLastError();
}

hipError_t launch_move_edges(const int32_t* from, int64_t n, const int32_t* map, int32_t* to, int64_t n_to,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_of(n_to)), dim3(256), 0, s, to, n_to, -1);
    hipLaunchKernelGGL(k_move_edges, dim3(blocks_of(n)), dim3(256), 0, s, from, n, map, to);
    return hipGetLastError();
}

}  // namespace mad
