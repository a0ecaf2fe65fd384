// The per-atom network of the NEP site energy (Sec. II.C of
// arXiv:2409.04430): the activation with its slope, and the matrix-core form
// of the network, shared by the descriptor kernels.
#pragma once

#include "nep_kernels.hpp"

namespace nep {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Orders this wavefront's LDS writes before its later LDS reads (LDS
// operations of one wavefront complete in issue order).
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Eight FP32 values as three BF16 vectors whose sum is exact: truncation
// keeps the top 8 significant bits, the remainder's top 8 bits follow, and
// the last remainder has at most 8 significant bits left.
__device__ __forceinline__ void split3(const float (&x)[8], bf16x8 &hi, bf16x8 &mid, bf16x8 &lo)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t u0 = __float_as_uint(x[e]) & 0xffff0000u;
        const float r1 = x[e] - __uint_as_float(u0);
        const uint32_t u1 = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(u1);
        hi[e] = __builtin_bit_cast(__bf16, (uint16_t)(u0 >> 16));
        mid[e] = __builtin_bit_cast(__bf16, (uint16_t)(u1 >> 16));
        lo[e] = __builtin_bit_cast(__bf16, (uint16_t)(__float_as_uint(r2) >> 16));
    }
}

// C += A B over the BF16 terms of both operands: A (weights) with WT terms,
// B (activations) with three.  WT = 1: the three products; WT = 3: the six
// products of term indices i + j <= 2 (a dropped product is below 2^-22 of
// the full one).
template <int WT>
__device__ __forceinline__ f32x4 mfma_terms(const bf16x8 (&a)[WT], const bf16x8 (&b)[3], f32x4 c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[0], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[1], c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[0], b[2], c, 0, 0, 0);
    if constexpr (WT == 3) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[1], b[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[2], b[0], c, 0, 0, 0);
    }
    return c;
}

// tanh and its slope, both to a few units in the last place over the whole
// range.  With a = |z| and r = 2 / (exp(2 a) + 1) in (0, 1]:
// |tanh z| = 1 - r and 1 - tanh^2 z = r (2 - r), free of cancellation for
// a >= 1/2 (r <= 0.54) and, for the slope, everywhere (exp saturates to inf
// for large a, so r = 0).  Below a = 1/2, tanh z = z f(z^2) with f the
// Maclaurin series of tanh(z) / z, whose coefficients are
// 2^2k (2^2k - 1) B_2k / (2k)! (B the Bernoulli numbers); through z^15 the
// series is exact to 1e-8 relative there.
__device__ __forceinline__ void tanh_and_slope(float z, float &h, float &dh)
{
#pragma clang fp contract(off)
    const float a = fabsf(z);
    const float r = 2.0f * __builtin_amdgcn_rcpf(__expf(2.0f * a) + 1.0f);
    dh = r * (2.0f - r);
    const float t = z * z;
    float f = -929569.0f / 638512875.0f;
    f = fmaf(f, t, 21844.0f / 6081075.0f);
    f = fmaf(f, t, -1382.0f / 155925.0f);
    f = fmaf(f, t, 62.0f / 2835.0f);
    f = fmaf(f, t, -17.0f / 315.0f);
    f = fmaf(f, t, 2.0f / 15.0f);
    f = fmaf(f, t, -1.0f / 3.0f);
    f = fmaf(f, t, 1.0f);
    h = a < 0.5f ? z * f : copysignf(1.0f - r, z);
}

// The network of the wavefront's 64 (atom, bead) rows on the matrix cores,
// as transposed products: Z^T = W0 Qh^T (A operand = weights, rows = hidden
// units; B operand = the scaled descriptors, columns = rows of the batch),
// h = tanh(Z - b0), U = w1 . h - b1, and G^T = W0^T (w1 (1 - h^2))^T.  The
// hidden units of a forward result tile sit in the lanes exactly where the
// adjoint product takes them as its B operand (its K order is permuted to
// match, in the weight fragments), so the hidden layer never leaves
// registers.  Qh is staged once in this wavefront's LDS tile X (64 rows of
// XS floats); each row's G and U are written back over it.  Zero rows for
// lanes outside the current species (mine = false).  Returns U of the
// lane's row and G (without the descriptor scale) in G[0..D).
// NJ: 16-row tiles of the batch that hold rows (4; 1 for a single row in lane 0).
template <int D, int WT, int NJ = 4>
__device__ float mlp_mf(const float (&qh)[D], bool mine, const uint16_t *__restrict__ frag, const float *b0,
                        const float *w1, float b1, int H, float *X, float (&G)[D])
{
    constexpr int DP = D <= 32 ? 32 : 64, KC = DP / 32, DT = DP / 16, XS = DP + 4;
    // batch tiles (16 rows each) per pass: every weight fragment is loaded
    // once per pass, and a pass keeps its tiles' operands and accumulators
    // in registers
    constexpr int JB = NJ == 1 ? 1 : (DP == 32 ? 4 : 2);
    const int HC = (H + 31) >> 5, HT = 2 * HC;
    const int l = threadIdx.x & 63, c = l & 15, g = l >> 4;
    if (NJ == 4 || l < 16 * NJ)
#pragma unroll
    for (int v4 = 0; v4 < DP / 4; ++v4) {
        float w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int v = 4 * v4 + e;
            w[e] = (mine && v < D) ? qh[v < D ? v : 0] : 0.0f;
        }
        *reinterpret_cast<float4 *>(X + l * XS + 4 * v4) = make_float4(w[0], w[1], w[2], w[3]);
    }
    wave_lds_sync();
    const bf16x8 *fw = reinterpret_cast<const bf16x8 *>(frag) + l;   // one 8-entry fragment per lane and block
    const int fwd = HT * KC, tstride = fwd + DT * HC;                 // blocks per term
    for (int j0 = 0; j0 < NJ; j0 += JB) {
        // B operands of the forward product: column c of tile j = batch row 16 j + c
        bf16x8 xb[JB][KC][3];
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            const float *xr = X + (16 * (j0 + jj) + c) * XS + 8 * g;
#pragma unroll
            for (int kc = 0; kc < KC; ++kc) {
                const float4 a0 = *reinterpret_cast<const float4 *>(xr + 32 * kc);
                const float4 a1 = *reinterpret_cast<const float4 *>(xr + 32 * kc + 4);
                const float x8[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
                split3(x8, xb[jj][kc][0], xb[jj][kc][1], xb[jj][kc][2]);
            }
        }
        f32x4 gacc[JB][DT];
        float uacc[JB];
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            uacc[jj] = 0.0f;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) gacc[jj][dt] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        for (int hc = 0; hc < HC; ++hc) {
            // this lane's eight hidden units of the chunk: 32 hc + 16 h2 + 4 g + e
            float bq[8], wq[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int mu = 32 * hc + 16 * (q >> 2) + 4 * g + (q & 3);
                bq[q] = mu < H ? b0[mu] : 0.0f;
                wq[q] = mu < H ? w1[mu] : 0.0f;
            }
            float gz[JB][8];
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
                const int ht = 2 * hc + h2;
                bf16x8 wa[KC][WT];
#pragma unroll
                for (int kc = 0; kc < KC; ++kc)
#pragma unroll
                    for (int t = 0; t < WT; ++t) wa[kc][t] = fw[(t * tstride + ht * KC + kc) * 64];
#pragma unroll
                for (int jj = 0; jj < JB; ++jj) {
                    f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int kc = 0; kc < KC; ++kc) z = mfma_terms<WT>(wa[kc], xb[jj][kc], z);
                    // z[e]: hidden unit 16 ht + 4 g + e of batch row 16 (j0 + jj) + c
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        float hh, dh;
                        tanh_and_slope(z[e] - bq[4 * h2 + e], hh, dh);
                        uacc[jj] = fmaf(wq[4 * h2 + e], hh, uacc[jj]);
                        gz[jj][4 * h2 + e] = wq[4 * h2 + e] * dh;
                    }
                }
            }
            // adjoint: B operand gz^T in K order (4 g + e, 16 + 4 g + e) as in the fragments
            bf16x8 wt[DT][WT];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int t = 0; t < WT; ++t) wt[dt][t] = fw[(t * tstride + fwd + dt * HC + hc) * 64];
#pragma unroll
            for (int jj = 0; jj < JB; ++jj) {
                bf16x8 gb[3];
                split3(gz[jj], gb[0], gb[1], gb[2]);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) gacc[jj][dt] = mfma_terms<WT>(wt[dt], gb, gacc[jj][dt]);
            }
        }
#pragma unroll
        for (int jj = 0; jj < JB; ++jj) {
            // U of column c: the four lane groups hold different hidden units
            float u = uacc[jj];
            u += __shfl_xor(u, 16, 64);
            u += __shfl_xor(u, 32, 64);
            // G^T (descriptor 16 dt + 4 g + e, column c) back over the row, which
            // this wavefront has finished reading (its LDS operations run in order)
            float *xo = X + (16 * (j0 + jj) + c) * XS;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
                *reinterpret_cast<float4 *>(xo + 16 * dt + 4 * g) =
                    make_float4(gacc[jj][dt][0], gacc[jj][dt][1], gacc[jj][dt][2], gacc[jj][dt][3]);
            if (g == 0) xo[DP] = u;
        }
    }
    wave_lds_sync();
    const int lr = NJ == 4 ? l : l & (16 * NJ - 1);
#pragma unroll
    for (int v = 0; v < D; ++v) G[v] = X[lr * XS + v];
    const float u = X[lr * XS + DP] - b1;
    wave_lds_sync();   // X is rewritten by the next species of this wavefront
    return u;
}

// LDS floats per wavefront of the matrix-core network.
template <int D>
constexpr int mf_lds_floats() { return 64 * ((D <= 32 ? 32 : 64) + 4); }

// Network arithmetic of k_descriptor: FP32 vector units with the weights
// read from global memory or staged in LDS; BF16 matrix cores with BF16
// weights (the student); or BF16 matrix cores with the FP32 weights as
// three exact BF16 terms (FP32 accuracy).  (FP32 operands on the matrix
// cores, 16 x 16 x 4 FP32 tiles, measured slower than the LDS-staged vector
// form: two wavefronts per SIMD cannot hide their dependent chains.)
constexpr int kNetGlobal = 0, kNetLds = 1, kNetBf16 = 2, kNetMf32 = 3;
constexpr int kNetRowRegs = 40;   // longest descriptor whose weight rows the LDS network holds in registers

}  // namespace nep
