// Kernels of the learned per-triangle density (project-defined; no paper
// counterpart): passive vertex normals, the network pass that produces psi and
// its first and second derivatives with respect to the six features for every
// triangle, and the training pass (loss, gradient, Adam).
//
// Network pass. Forward mode is seeded on the six (scaled) features: layer 1's
// unit k carries, in closed form, sp(a1) and its first derivatives
// sigma(a1) W1[k,i] (second derivatives sigma'(a1) W1[k,i] W1[k,j]). Layer 2's
// value and first-order channels, the transposed contraction u = W2^T v that
// folds layer 2's second-order channels into one, and the layer-1 part of the
// second derivatives are contractions over the 64 units and run on the matrix
// cores (v_mfma_f32_16x16x32_bf16; see k_mlp_head). Weights and products of
// two weights are exact in one or two BF16 terms; every activation is split
// into three BF16 terms (hi + mid + lo carries all 24 bits of an FP32
// significand), so the MFMAs reproduce FP32 products with FP32 accumulation.
#include <hip/hip_runtime.h>

#include <cmath>

#include "mlp.hpp"
#include "terms.hpp"

namespace mad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short short8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {   // round to nearest even (finite inputs)
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float softplusf(float a) { return fmaxf(a, 0.0f) + log1pf(expf(-fabsf(a))); }
__device__ __forceinline__ float logisticf(float a) {
    const float e = expf(-fabsf(a));
    const float r = 1.0f / (1.0f + e);
    return a >= 0.0f ? r : e * r;
}

// softplus and logistic of a from one exponential, with the hardware exp2, log2 and reciprocal
// (about one ulp each; used by the network pass): e = exp(-|a|), with the product -|a| log2(e) carried
// to twice FP32 precision so that e keeps its relative accuracy for large |a|; sigma = 1/(1+e)
// (a >= 0) or e/(1+e); softplus = max(a, 0) + log1p(e), with log1p(e) = log(u) e / (u - 1),
// u = 1 + e rounded, and e itself where u rounds to 1: the method of D. Goldberg, "What every computer
// scientist should know about floating-point arithmetic" (ACM Computing Surveys, 1991), Theorem 4.
// Relative error within five FP32 ulps of FP64 log1p / exp over |a| <= 80 in an FP32 emulation with every
// hardware result rounded to nearest or one ulp off either way.
__device__ __forceinline__ void softplus_logistic(float a, float& sp, float& sg) {
    constexpr float kL2E = 1.44269502162933349609375f;          // log2(e) rounded to FP32
    constexpr float kL2ELo = 1.925963033500011079e-8f;          // log2(e) - kL2E
    constexpr float kLn2 = 0.693147180559945309f;
    const float x = -fabsf(a);
    const float t = x * kL2E;
    const float tl = fmaf(x, kL2E, -t) + x * kL2ELo;
    float e = __builtin_amdgcn_exp2f(t);
    e = fmaf(e, tl * kLn2, e);
    const float u = 1.0f + e;
    const float r = __builtin_amdgcn_rcpf(u);
    sg = a >= 0.0f ? r : e * r;
    const float um1 = u - 1.0f;
    const float l1p = um1 == 0.0f ? e : (__builtin_amdgcn_logf(u) * kLn2) * (e * __builtin_amdgcn_rcpf(um1));
    sp = fmaxf(a, 0.0f) + l1p;
}

// The workgroup's place in an order that keeps neighbours on one XCD, whose L2 then holds the part of x (and of the
// normals) that they share: workgroups go to the XCDs in turn. 708^2 cylinder: normals 11 us and features 3 us less
// (a pass 684 -> 670); more triangles in flight per vertex changed nothing.
__device__ __forceinline__ int64_t xcd_block() {
    const int per = (int)(gridDim.x >> 3), rest8 = (int)(gridDim.x & 7), xcd = (int)(blockIdx.x & 7);
    return xcd * per + min(xcd, rest8) + (int)(blockIdx.x >> 3);
}

// ---- vertex normals ------------------------------------------------------------------------------
__global__ void k_vertex_normals(const double* x, int64_t nv, const int32_t* vf_ptr, const int32_t* vf,
                                 const int32_t* tris, double* normals) {
    for (int64_t v = xcd_block() * blockDim.x + threadIdx.x; v < nv; v += (int64_t)gridDim.x * blockDim.x) {
        double n0 = 0.0, n1 = 0.0, n2 = 0.0;
        for (int32_t q = vf_ptr[v]; q < vf_ptr[v + 1]; ++q) {
            const int32_t* t = tris + 3 * (int64_t)vf[q];
            const double* a = x + 3 * (int64_t)t[0];
            const double* b = x + 3 * (int64_t)t[1];
            const double* c = x + 3 * (int64_t)t[2];
            const double e1x = b[0] - a[0], e1y = b[1] - a[1], e1z = b[2] - a[2];
            const double e2x = c[0] - a[0], e2y = c[1] - a[1], e2z = c[2] - a[2];
            n0 += e1y * e2z - e1z * e2y;
            n1 += e1z * e2x - e1x * e2z;
            n2 += e1x * e2y - e1y * e2x;
        }
        const double l = sqrt(n0 * n0 + n1 * n1 + n2 * n2);
        const double il = l > 0.0 ? 1.0 / l : 0.0;
        normals[3 * v] = n0 * il;
        normals[3 * v + 1] = n1 * il;
        normals[3 * v + 2] = n2 * il;
    }
}

hipError_t launch_vertex_normals(const double* x, int64_t nv, const int32_t* vf_ptr, const int32_t* vf,
                                 const int32_t* tris, double* normals, hipStream_t s) {
    if (nv <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((nv + 255) / 256, 16384);
    hipLaunchKernelGGL(k_vertex_normals, dim3((unsigned)blocks), dim3(256), 0, s, x, nv, vf_ptr, vf, tris, normals);
    return hipGetLastError();
}

// ---- network pass --------------------------------------------------------------------------------
// feature channel c >= 7: the packed upper pair (i, j) of Packed<6>
__host__ __device__ constexpr int pair_i(int q) { return q < 6 ? 0 : q < 11 ? 1 : q < 15 ? 2 : q < 18 ? 3 : q < 20 ? 4 : 5; }
__host__ __device__ constexpr int pair_j(int q) {
    return q < 6 ? q : q < 11 ? q - 5 : q < 15 ? q - 9 : q < 18 ? q - 12 : q < 20 ? q - 14 : 5;
}
static_assert(Packed<6>::at(pair_i(13), pair_j(13)) == 13 && Packed<6>::at(pair_i(20), pair_j(20)) == 20,
              "pair tables follow Packed<6>");

// features z of triangle e (FP64): same formulas as the element term's shell_features
__device__ __forceinline__ void features_at(const MlpHeadLaunch& L, int64_t e, double (&z)[6]) {
    const int32_t* st = L.stencil + 3 * e;
    double xs[9], in[17];
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            xs[3 * s + c] = L.x[3 * (int64_t)st[s] + c];
            in[8 + 3 * s + c] = L.normals[3 * (int64_t)st[s] + c];
        }
#pragma unroll
    for (int k = 0; k < 8; ++k) in[k] = L.rest[(int64_t)k * L.n + e];
    double r[6];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        r[i] = xs[3 + i] - xs[i];
        r[3 + i] = xs[6 + i] - xs[i];
    }
    shell_features<double>(r, in, z);
}

// wave-scope ordering of LDS accesses between the lanes of one wave
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// three BF16 terms of an FP32 value (hi + mid + lo reproduces its 24 significand bits), stored
// into element j of three operand vectors
__device__ __forceinline__ void split3(float v, bf16x8& h, bf16x8& m, bf16x8& l, int j) {
    const __bf16 a = (__bf16)v;
    const float r = v - (float)a;
    const __bf16 b = (__bf16)r;
    h[j] = a;
    m[j] = b;
    l[j] = (__bf16)(r - (float)b);
}

// One wave evaluates 16 triangles at a time (one per MFMA column). With v = w3 * sigma(a2) and
// u = W2^T v, the network's derivatives with respect to the scaled features xh are
//   dpsi/dxh_i        = sum_k u_k sigma(a1_k) W1[k,i]
//   d2psi/dxh_i dxh_j = sum_k u_k sigma'(a1_k) W1[k,i] W1[k,j] + sum_m w3_m sigma'(a2_m) g_mi g_mj,
// g_mi = sum_k W2[m,k] W1[k,i] sigma(a1_k) (layer 2's first-order channels). Four groups of contractions run
// on the matrix cores (v_mfma_f32_16x16x32_bf16):
//   a2 - b2 = W2 sp(a1)            W2 exact in BF16, sp(a1) in three BF16 terms;
//   g_i = G_i sigma(a1)            G_i[m,k] = W2[m,k] W1[k,i], a product of two BF16 values (16 significant
//                                  bits: exactly two BF16 terms); sigma(a1) in three terms, split once for the
//                                  six channels;
//   u = W2^T v                     v in three BF16 terms;
//   S1[t,q] = sum_k (u sigma') C[k,q]   C[k,q] = W1[k,i_q] W1[k,j_q] over the 21 packed pairs, two BF16 terms;
//                                  u sigma' in three: the layer-1 part of the second derivatives.
// A product of three-term by two-term operands drops only the lo x lo part (2^-24 relative), so every
// contraction reproduces FP32 products with FP32 accumulation. The layer-2 part of the second derivatives (a
// rank-6 sum per triangle) and the first derivatives are per-triangle VALU work.
//
// The constant operands (W2, W2^T, G, C) are built once per workgroup and fill the CU's LDS together with the
// waves' tiles, so that the forward channels need no operand of their own per triangle and a wave's state (one
// quarter of layer 2 at a time) fits half of a SIMD's registers: two waves per SIMD, one's vector instructions
// under the other's matrix instructions and latencies. 999,698 triangles: 569 us when each channel's activations
// were split on their own and one wave per SIMD held all of layer 2, 440 us now (2,110 vector and 308 matrix
// instructions a tile instead of 3,990 and 212): about 80% of the cycles issue a vector instruction. Unrolling the
// quarters of layer 2, or computing one quarter while another is finished, spilled or was slower.
// Layouts (16x16x32 MFMA): B operand lane l holds column l % 16 and k = 32 ks + 8 (l / 16) + j; A operand lane
// l holds row l % 16 and the same k; accumulators hold rows 4 (l / 16) + jj of column l % 16.
constexpr int kHeadWaves = 8;
constexpr int kTileRow = kHid + 1;   // floats of a tile's row in LDS

struct HeadSmem {   // byte offsets into the network pass's dynamic LDS
    static constexpr int w1 = 0;                                   // float [64][6]
    static constexpr int b1 = w1 + kHid * 6 * 4;                   // float [64]
    static constexpr int b2 = b1 + kHid * 4;
    static constexpr int w3 = b2 + kHid * 4;
    static constexpr int w2 = w3 + kHid * 4;                       // bf16 [m][64], rows swizzled (below)
    static constexpr int w2t = w2 + kHid * kHid * 2;               // bf16 [k][64]: W2 transposed
    static constexpr int c = w2t + kHid * kHid * 2;                // bf16 [2][32][64]: C hi, lo (q >= 21: 0)
    static constexpr int g = c + 2 * 32 * kHid * 2;                // bf16 [6][2][m][64]: G hi, lo
    static constexpr int t = g + 6 * 2 * kHid * kHid * 2;          // float [waves][16][kTileRow]
    static constexpr int bytes = t + kHeadWaves * 16 * kTileRow * 4;
};
static_assert(HeadSmem::w2 % 16 == 0 && HeadSmem::t % 16 == 0, "16-byte LDS operand reads");
static_assert(HeadSmem::bytes <= 160 * 1024, "network pass LDS fits a CU");

// element of (row, k) in an LDS table of 64-element BF16 rows: the row's eight 16-byte pieces are permuted by
// its number, so that the 16 rows a wave reads at one k lie in different banks
__device__ __forceinline__ int head_at(int row, int k) { return row * kHid + ((((k >> 3) ^ (row >> 1)) & 7) << 3) + (k & 7); }

__device__ __forceinline__ bf16x8 lds_bf16x8(const __bf16* p) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const short8*>(p));
}

// rows a, b, c, d of four per-lane values summed over the four 16-lane groups: group g gets the g-th value's sum
__device__ __forceinline__ float group_sums(float a, float b, float c, float d) {
    auto bits = [](float f) { return __float_as_uint(f); };
    const auto ab = __builtin_amdgcn_permlane16_swap(bits(a), bits(b), false, false);
    const auto cd = __builtin_amdgcn_permlane16_swap(bits(c), bits(d), false, false);
    const float p = __uint_as_float(ab[0]) + __uint_as_float(ab[1]);
    const float q = __uint_as_float(cd[0]) + __uint_as_float(cd[1]);
    const auto pq = __builtin_amdgcn_permlane32_swap(bits(p), bits(q), false, false);
    return __uint_as_float(pq[0]) + __uint_as_float(pq[1]);
}

#define MAD_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)

__global__ __launch_bounds__(kHeadWaves * 64) void k_mlp_head(MlpHeadLaunch L) {
    extern __shared__ __align__(16) unsigned char head_smem[];
    float* sW1 = reinterpret_cast<float*>(head_smem + HeadSmem::w1);
    float* sB1 = reinterpret_cast<float*>(head_smem + HeadSmem::b1);
    float* sB2 = reinterpret_cast<float*>(head_smem + HeadSmem::b2);
    float* sW3 = reinterpret_cast<float*>(head_smem + HeadSmem::w3);
    __bf16* sW2 = reinterpret_cast<__bf16*>(head_smem + HeadSmem::w2);
    __bf16* sW2T = reinterpret_cast<__bf16*>(head_smem + HeadSmem::w2t);
    __bf16* sC = reinterpret_cast<__bf16*>(head_smem + HeadSmem::c);
    __bf16* sG = reinterpret_cast<__bf16*>(head_smem + HeadSmem::g);
    for (int i = threadIdx.x; i < kHid * 6; i += blockDim.x) sW1[i] = bf2f(L.wbf[kOffW1 + i]);
    for (int i = threadIdx.x; i < kHid; i += blockDim.x) {
        sB1[i] = bf2f(L.wbf[kOffB1 + i]);
        sB2[i] = bf2f(L.wbf[kOffB2 + i]);
        sW3[i] = bf2f(L.wbf[kOffW3 + i]);
    }
    __syncthreads();
    // a product of two BF16 values, exact in FP32, is exactly two BF16 terms
    for (int idx = threadIdx.x; idx < kHid * kHid; idx += blockDim.x) {
        const int m = idx / kHid, k = idx % kHid, at = head_at(m, k);
        const float w2 = bf2f(L.wbf[kOffW2 + idx]);
        sW2[at] = (__bf16)w2;
        sW2T[head_at(k, m)] = (__bf16)w2;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const float p = w2 * sW1[k * 6 + i];
            const __bf16 hi = (__bf16)p;
            sG[(2 * i) * kHid * kHid + at] = hi;
            sG[(2 * i + 1) * kHid * kHid + at] = (__bf16)(p - (float)hi);
        }
    }
    for (int idx = threadIdx.x; idx < 32 * kHid; idx += blockDim.x) {
        const int q = idx / kHid, k = idx % kHid;
        const float p = q < 21 ? sW1[k * 6 + pair_i(q)] * sW1[k * 6 + pair_j(q)] : 0.0f;
        const __bf16 hi = (__bf16)p;
        sC[head_at(q, k)] = hi;
        sC[32 * kHid + head_at(q, k)] = (__bf16)(p - (float)hi);
    }
    __syncthreads();
    const float b3 = bf2f(L.wbf[kOffB3]);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, col = lane & 15;
    float (*T)[kTileRow] = reinterpret_cast<float (*)[kTileRow]>(head_smem + HeadSmem::t) + wave * 16;
    // back to z: psi scales by s_out, dpsi/dz_i by s_out s_in[i], the second derivatives by both inputs' scales;
    // this lane's outputs are 4 k + g of (psi, 6 first, 21 second derivatives)
    float sc[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) {
        const int o = 4 * k + g;
        float f = L.s_out;
        for (int i = 0; i < 6; ++i) {
            if (o == 1 + i) f *= L.s_in[i];
            for (int j = i; j < 6; ++j)
                if (o == 7 + Packed<6>::at(i, j)) f *= L.s_in[i] * L.s_in[j];
        }
        sc[k] = f;
    }
    const int64_t tiles = (L.n + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * kHeadWaves + wave; tile < tiles;
         tile += (int64_t)gridDim.x * kHeadWaves) {
        const int64_t e = tile * 16 + col;
        const bool valid = e < L.n;
        float xh[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) xh[i] = valid ? L.xh[(int64_t)i * L.n + e] : 0.0f;
        // layer 1 at this lane's 16 units (B layout): sp(a1) and sigma(a1), each split into three BF16 terms
        float s1[2][8];
        bf16x8 p0[2][3], sg[2][3];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = 32 * ks + 8 * g + j;
                float a = sB1[k];
#pragma unroll
                for (int i = 0; i < 6; ++i) a = fmaf(sW1[k * 6 + i], xh[i], a);
                float sp;
                softplus_logistic(a, sp, s1[ks][j]);
                split3(sp, p0[ks][0], p0[ks][1], p0[ks][2], j);
                split3(s1[ks][j], sg[ks][0], sg[ks][1], sg[ks][2], j);
            }
        // layer 2, 16 units at a time: the value and the six first-order channels, then everything that needs
        // them (v to LDS as [triangle][unit])
        float P[28];   // psi, first derivatives, packed second derivatives: this lane's part of the sums
#pragma unroll
        for (int q = 0; q < 28; ++q) P[q] = 0.0f;
#pragma unroll 1
        for (int mt = 0; mt < 4; ++mt) {
            const int row = 16 * mt + col;
            f32x4 val = {0.0f, 0.0f, 0.0f, 0.0f}, ch[6];
#pragma unroll
            for (int i = 0; i < 6; ++i) ch[i] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int at = head_at(row, 32 * ks + 8 * g);
                const bf16x8 a = lds_bf16x8(sW2 + at);
#pragma unroll
                for (int r = 0; r < 3; ++r) val = MAD_MFMA(a, p0[ks][r], val);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const bf16x8 hi = lds_bf16x8(sG + (2 * i) * kHid * kHid + at);
                    const bf16x8 lo = lds_bf16x8(sG + (2 * i + 1) * kHid * kHid + at);
                    ch[i] = MAD_MFMA(hi, sg[ks][0], ch[i]);
                    ch[i] = MAD_MFMA(hi, sg[ks][1], ch[i]);
                    ch[i] = MAD_MFMA(hi, sg[ks][2], ch[i]);
                    ch[i] = MAD_MFMA(lo, sg[ks][0], ch[i]);
                    ch[i] = MAD_MFMA(lo, sg[ks][1], ch[i]);
                }
            }
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int m = 16 * mt + 4 * g + jj;
                const float w3 = sW3[m];
                float sp, s2;
                softplus_logistic(val[jj] + sB2[m], sp, s2);
                const float v = w3 * s2;
                T[col][m] = v;
                P[0] = fmaf(w3, sp, P[0]);
                const float c2 = v * (1.0f - s2);
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    const float t = c2 * ch[i][jj];
#pragma unroll
                    for (int j = i; j < 6; ++j)
                        P[7 + Packed<6>::at(i, j)] = fmaf(t, ch[j][jj], P[7 + Packed<6>::at(i, j)]);
                }
            }
        }
        // u = W2^T v: v read back as the A operand (rows = triangles)
        wave_sync();
        bf16x8 vh[2], vm[2], vl[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) split3(T[col][32 * ks + 8 * g + j], vh[ks], vm[ks], vl[ks], j);
        f32x4 U[4];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
            U[nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                // B operand: W2[m][k], m = 32 ks + 8 g + j, k = 16 nt + col (a row of W2^T)
                const bf16x8 b = lds_bf16x8(sW2T + head_at(16 * nt + col, 32 * ks + 8 * g));
                U[nt] = MAD_MFMA(vh[ks], b, U[nt]);
                U[nt] = MAD_MFMA(vm[ks], b, U[nt]);
                U[nt] = MAD_MFMA(vl[ks], b, U[nt]);
            }
        }
        wave_sync();   // every lane has read v before u overwrites it
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) T[4 * g + jj][16 * nt + col] = U[nt][jj];
        wave_sync();
        // first derivatives over this lane's 16 units; u sigma' split as the A operand of the layer-1
        // second-order contraction (rows = triangles, the same lane distribution as the B layout)
        bf16x8 uh[2], um[2], ul[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = 32 * ks + 8 * g + j;
                const float us = T[col][k] * s1[ks][j];
#pragma unroll
                for (int i = 0; i < 6; ++i) P[1 + i] = fmaf(us, sW1[k * 6 + i], P[1 + i]);
                split3(us * (1.0f - s1[ks][j]), uh[ks], um[ks], ul[ks], j);
            }
        f32x4 S1[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            S1[nt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const int at = head_at(16 * nt + col, 32 * ks + 8 * g);
                const bf16x8 hi = lds_bf16x8(sC + at), lo = lds_bf16x8(sC + 32 * kHid + at);
                S1[nt] = MAD_MFMA(uh[ks], hi, S1[nt]);
                S1[nt] = MAD_MFMA(um[ks], hi, S1[nt]);
                S1[nt] = MAD_MFMA(ul[ks], hi, S1[nt]);
                S1[nt] = MAD_MFMA(uh[ks], lo, S1[nt]);
                S1[nt] = MAD_MFMA(um[ks], lo, S1[nt]);
            }
        }
        wave_sync();   // u is read before the layer-1 second derivatives overwrite it
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) T[4 * g + jj][16 * nt + col] = S1[nt][jj];
        wave_sync();
        // sums over the four lanes holding the same triangle; each writes seven of its 28 outputs
#pragma unroll
        for (int k = 0; k < 7; ++k) {
            const int o = 4 * k + g;
            float r = group_sums(P[4 * k], P[4 * k + 1], P[4 * k + 2], P[4 * k + 3]);
            r += o == 0 ? b3 : o >= 7 ? T[col][o - 7] : 0.0f;
            if (valid) L.psi[(int64_t)o * L.n + e] = sc[k] * r;
        }
        wave_sync();   // the layer-1 part is read before the next tile writes v
    }
}
#undef MAD_MFMA

__global__ __launch_bounds__(256) void k_mlp_features(MlpHeadLaunch L) {
    for (int64_t e = xcd_block() * blockDim.x + threadIdx.x; e < L.n; e += (int64_t)gridDim.x * blockDim.x) {
        double z[6];
        features_at(L, e, z);
#pragma unroll
        for (int i = 0; i < 6; ++i) L.xh[(int64_t)i * L.n + e] = float(z[i]) * L.s_in[i];
    }
}

hipError_t launch_mlp_head(const MlpHeadLaunch& L, hipStream_t s) {
    if (L.n <= 0) return hipSuccess;
    {
        const int64_t blocks = std::min<int64_t>((L.n + 255) / 256, 16384);
        hipLaunchKernelGGL(k_mlp_features, dim3((unsigned)blocks), dim3(256), 0, s, L);
    }
    const int64_t tiles = (L.n + 15) / 16;
    const int64_t blocks = std::min<int64_t>((tiles + kHeadWaves - 1) / kHeadWaves, std::max(L.n_cu, 1));
    hipLaunchKernelGGL(k_mlp_head, dim3((unsigned)blocks), dim3(kHeadWaves * 64), HeadSmem::bytes, s, L);
    return hipGetLastError();
}

// ---- training ------------------------------------------------------------------------------------
// One wave per sample, lane m = hidden unit m. Forward mode carries the six tangents
// d/dxh (xh = s_in * z) through both layers; reverse mode then differentiates
//   loss = (psi - W)^2 / (c_e B) + lam_g sum_i (dpsi/dz_i - dW_i)^2 / (c_g[i] B)   (B = batch size)
// with respect to every parameter. A workgroup takes four samples at a time; the gradient of W2, the sum of the
// samples' outer products, is shared out over its waves (16 columns each, summed over the four samples), so that a
// lane holds 16 of its sums and not 64 (which spilled). Each workgroup writes one partial row; the rows are summed
// in a fixed order afterwards. A minibatch of 512 is one sample per wave over 128 workgroups and bound by the
// latency of that sample's chain: 19 us, 132 us with eight samples after one another on each of 64 waves.
constexpr int kTrainWaves = 4, kTrainBlock = 64 * kTrainWaves;
constexpr int kW2Pad = kHid + 1;   // padded LDS rows: lane m reading row m is bank-conflict free

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ __launch_bounds__(kTrainBlock) void k_mlp_train(MlpTrainLaunch L) {
    __shared__ float sW2[kHid * kW2Pad];
    __shared__ __align__(16) float sX[kTrainWaves][kHid][8];    // per wave: h1, T1 (6), pad
    __shared__ __align__(16) float sD[kTrainWaves][kHid][8];    // per wave: delta2, G2a (6), pad
    constexpr int kCols = kHid / kTrainWaves;   // columns of W2 whose gradient a wave sums
    for (int i = threadIdx.x; i < kHid * kHid; i += blockDim.x)
        sW2[(i / kHid) * kW2Pad + i % kHid] = L.params[kOffW2 + i];
    const int m = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float w1[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) w1[i] = L.params[kOffW1 + m * 6 + i];
    const float b1 = L.params[kOffB1 + m], b2 = L.params[kOffB2 + m], w3 = L.params[kOffW3 + m];
    const float b3 = L.params[kOffB3];
    float gW2[kCols];
#pragma unroll
    for (int k = 0; k < kCols; ++k) gW2[k] = 0.0f;
    float gW1[6] = {0, 0, 0, 0, 0, 0};
    float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, loss = 0.0f;
    const float inv_b = 1.0f / float(L.count);
    // every wave runs the same number of rounds (the block barriers below need it); a wave past the
    // end of the batch evaluates sample 0 of the batch with zero weight
    const int64_t per_round = (int64_t)L.n_rows * kTrainWaves;
    for (int64_t q0 = 0; q0 < L.count; q0 += per_round) {
        const int64_t q = q0 + (int64_t)blockIdx.x * kTrainWaves + wv;
        const bool active = q < L.count;
        const int64_t qi = active ? q : 0;
        const int64_t smp = L.idx ? (int64_t)L.idx[L.base + qi] : L.base + qi;
        const float wgt = active ? inv_b : 0.0f;
        float xh[6], dWt[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            xh[i] = L.z[smp * 6 + i] * L.s_in[i];
            dWt[i] = L.dW[smp * 6 + i];
        }
        const float Wt = L.W[smp];
        // layer 1 (unit m)
        float a1 = b1;
#pragma unroll
        for (int i = 0; i < 6; ++i) a1 = fmaf(w1[i], xh[i], a1);
        const float h1 = softplusf(a1), d1 = logisticf(a1), d1p = d1 * (1.0f - d1);
        float4* x4 = reinterpret_cast<float4*>(sX[wv][m]);
        x4[0] = make_float4(h1, d1 * w1[0], d1 * w1[1], d1 * w1[2]);
        x4[1] = make_float4(d1 * w1[3], d1 * w1[4], d1 * w1[5], 0.0f);
        __syncthreads();   // the first round's W2 as well
        // layer 2 (unit m): a2 = W2[m, :] h1 + b2, T2a[m, i] = W2[m, :] T1[:, i]
        float a2 = b2, t2a[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 8
        for (int k = 0; k < kHid; ++k) {
            const float w = sW2[m * kW2Pad + k];
            const float4 p = reinterpret_cast<const float4*>(sX[wv][k])[0], r = reinterpret_cast<const float4*>(sX[wv][k])[1];
            a2 = fmaf(w, p.x, a2);
            t2a[0] = fmaf(w, p.y, t2a[0]);
            t2a[1] = fmaf(w, p.z, t2a[1]);
            t2a[2] = fmaf(w, p.w, t2a[2]);
            t2a[3] = fmaf(w, r.x, t2a[3]);
            t2a[4] = fmaf(w, r.y, t2a[4]);
            t2a[5] = fmaf(w, r.z, t2a[5]);
        }
        const float h2 = softplusf(a2), d2 = logisticf(a2), d2p = d2 * (1.0f - d2);
        // output: psi^ = w3 . h2 + b3, g^_i = w3 . (d2 T2a[:, i])
        const float ps = wave_sum(w3 * h2) + b3;
        float gh[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) gh[i] = wave_sum(w3 * d2 * t2a[i]);
        const float psi = L.s_out * ps;
        const float rr = 2.0f * (psi - Wt) * wgt / L.c_e * L.s_out;            // dloss / dpsi^
        float qq[6];
        float lg = 0.0f;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const float dz = L.s_out * L.s_in[i] * gh[i] - dWt[i];
            lg += dz * dz / L.c_g[i];
            qq[i] = 2.0f * L.lam_g * dz * wgt / L.c_g[i] * L.s_out * L.s_in[i];  // dloss / dg^_i
        }
        loss += ((psi - Wt) * (psi - Wt) / L.c_e + L.lam_g * lg) * wgt;
        // reverse through the output layer and layer 2's nonlinearity
        float qt = 0.0f, g2a[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            qt = fmaf(qq[i], t2a[i], qt);
            g2a[i] = d2 * w3 * qq[i];                 // dloss / dT2a[m, i]
        }
        gw3 += rr * h2 + d2 * qt;
        gb3 += rr;
        const float delta2 = d2p * w3 * qt + d2 * rr * w3;   // dloss / da2[m]
        gb2 += delta2;
        float4* d4 = reinterpret_cast<float4*>(sD[wv][m]);
        d4[0] = make_float4(delta2, g2a[0], g2a[1], g2a[2]);
        d4[1] = make_float4(g2a[3], g2a[4], g2a[5], 0.0f);
        __syncthreads();
        // dW2[m, k] += delta2[m] h1[k] + sum_i G2a[m, i] T1[k, i], over the workgroup's samples
#pragma unroll 1
        for (int s = 0; s < kTrainWaves; ++s) {
            const float4 a = reinterpret_cast<const float4*>(sD[s][m])[0], b = reinterpret_cast<const float4*>(sD[s][m])[1];
#pragma unroll
            for (int k = 0; k < kCols; ++k) {
                const float4* x = reinterpret_cast<const float4*>(sX[s][kCols * wv + k]);
                const float4 p = x[0], r = x[1];
                float acc = a.x * p.x;
                acc = fmaf(a.y, p.y, acc);
                acc = fmaf(a.z, p.z, acc);
                acc = fmaf(a.w, p.w, acc);
                acc = fmaf(b.x, r.x, acc);
                acc = fmaf(b.y, r.y, acc);
                gW2[k] += fmaf(b.z, r.z, acc);
            }
        }
        // unit k = m of layer 1: dh1[k] = sum_m W2[m, k] delta2[m], dT1[k, i] = sum_m W2[m, k] G2a[m, i]
        float dh1 = 0.0f, dT1[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll 8
        for (int mm = 0; mm < kHid; ++mm) {
            const float w = sW2[mm * kW2Pad + m];
            const float4 p = reinterpret_cast<const float4*>(sD[wv][mm])[0], r = reinterpret_cast<const float4*>(sD[wv][mm])[1];
            dh1 = fmaf(w, p.x, dh1);
            dT1[0] = fmaf(w, p.y, dT1[0]);
            dT1[1] = fmaf(w, p.z, dT1[1]);
            dT1[2] = fmaf(w, p.w, dT1[2]);
            dT1[3] = fmaf(w, r.x, dT1[3]);
            dT1[4] = fmaf(w, r.y, dT1[4]);
            dT1[5] = fmaf(w, r.z, dT1[5]);
        }
        float dd1 = 0.0f;
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            dd1 = fmaf(w1[i], dT1[i], dd1);
            gW1[i] += d1 * dT1[i];                      // through T1 = d1 W1
        }
        const float delta1 = d1p * dd1 + d1 * dh1;     // dloss / da1[m]
        gb1 += delta1;
#pragma unroll
        for (int i = 0; i < 6; ++i) gW1[i] += delta1 * xh[i];
        __syncthreads();   // sX / sD are rewritten by the next samples
    }
    // the workgroup's row: W2's part through LDS (coalesced), the units' other parameters summed over the waves
#pragma unroll
    for (int k = 0; k < kCols; ++k) sW2[m * kW2Pad + kCols * wv + k] = gW2[k];
#pragma unroll
    for (int i = 0; i < 6; ++i) sX[wv][m][i] = gW1[i];
    sX[wv][m][6] = gb1;
    sX[wv][m][7] = gb2;
    sD[wv][m][0] = gw3;
    if (m == 0) {
        sD[wv][0][1] = gb3;
        sD[wv][0][2] = loss;
    }
    __syncthreads();
    float* out = L.partial + (int64_t)blockIdx.x * (kMlpParams + 1);
    for (int i = threadIdx.x; i < kHid * kHid; i += blockDim.x) out[kOffW2 + i] = sW2[(i / kHid) * kW2Pad + i % kHid];
    auto over_waves = [&](const float* first) {   // the same place of every wave's array
        float acc = first[0];
#pragma unroll
        for (int w = 1; w < kTrainWaves; ++w) acc += first[w * kHid * 8];
        return acc;
    };
    for (int i = threadIdx.x; i < kHid * 6; i += blockDim.x) out[kOffW1 + i] = over_waves(&sX[0][i / 6][i % 6]);
    if (threadIdx.x < kHid) {
        out[kOffB1 + m] = over_waves(&sX[0][m][6]);
        out[kOffB2 + m] = over_waves(&sX[0][m][7]);
        out[kOffW3 + m] = over_waves(&sD[0][m][0]);
    }
    if (threadIdx.x == 0) {
        out[kOffB3] = over_waves(&sD[0][0][1]);
        out[kMlpParams] = over_waves(&sD[0][0][2]);
    }
}

hipError_t launch_mlp_train(const MlpTrainLaunch& L, hipStream_t s) {
    if (L.n_rows < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_mlp_train, dim3(L.n_rows), dim3(kTrainBlock), 0, s, L);
    return hipGetLastError();
}

// one lane per parameter in each of four waves, which take every fourth row (eight loads in flight); the four
// sums are added in order. 128 rows 4.9 us; one lane over all of 64 rows took 15.6 us.
__global__ __launch_bounds__(256) void k_mlp_reduce(const float* partial, int n_rows, float* grad, float* loss) {
    __shared__ float red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = blockIdx.x * 64 + lane;
    float acc = 0.0f;
    if (i <= kMlpParams) {
        const float* p = partial + i;
        int r = w;
        for (; r + 28 < n_rows; r += 32) {
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = p[(int64_t)(r + 4 * k) * (kMlpParams + 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += v[k];
        }
        for (; r < n_rows; r += 4) acc += p[(int64_t)r * (kMlpParams + 1)];
    }
    red[w][lane] = acc;
    __syncthreads();
    if (w != 0 || i > kMlpParams) return;
    acc = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    if (i < kMlpParams) grad[i] = acc;
    else *loss = acc;
}

hipError_t launch_mlp_reduce(const float* partial, int n_rows, float* grad, float* loss, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_reduce, dim3((kMlpParams + 1 + 63) / 64), dim3(256), 0, s, partial, n_rows, grad, loss);
    return hipGetLastError();
}

// every workgroup counts the steps in an entry of its own (all equal), so that none waits for another's reading
__global__ void k_mlp_adam(float* params, float* m, float* v, const float* grad, int64_t* steps, float lr,
                           float beta1, float beta2, float eps, uint16_t* wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t step = steps[blockIdx.x] + 1;
    __syncthreads();
    if (threadIdx.x == 0) steps[blockIdx.x] = step;
    if (i >= kMlpParams) return;
    const float t = float(step);
    const float g = grad[i];
    const float mi = beta1 * m[i] + (1.0f - beta1) * g;
    const float vi = beta2 * v[i] + (1.0f - beta2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float mh = mi / (1.0f - powf(beta1, t));
    const float vh = vi / (1.0f - powf(beta2, t));
    const float p = params[i] - lr * mh / (sqrtf(vh) + eps);
    params[i] = p;
    wbf[i] = f2bf(p);
}

hipError_t launch_mlp_adam(float* params, float* m, float* v, const float* grad, int64_t* steps, float lr,
                           float beta1, float beta2, float eps, uint16_t* wbf, hipStream_t s) {
    static_assert((kMlpParams + 255) / 256 == kAdamBlocks, "a step count for every workgroup");
    hipLaunchKernelGGL(k_mlp_adam, dim3(kAdamBlocks), dim3(256), 0, s, params, m, v, grad, steps, lr, beta1, beta2,
                       eps, wbf);
    return hipGetLastError();
}

__global__ void k_mlp_to_bf16(const float* params, uint16_t* wbf) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kMlpParams) wbf[i] = f2bf(params[i]);
}

hipError_t launch_mlp_to_bf16(const float* params, uint16_t* wbf, hipStream_t s) {
    hipLaunchKernelGGL(k_mlp_to_bf16, dim3((kMlpParams + 255) / 256), dim3(256), 0, s, params, wbf);
    return hipGetLastError();
}

}  // namespace mad
