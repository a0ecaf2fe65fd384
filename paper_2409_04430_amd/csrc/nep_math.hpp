// Device math shared by the NEP force kernels and the training kernels:
// the Chebyshev radial basis with its smooth cutoff, the real spherical
// harmonics l = 1..4 and their gradients, the adjoint contraction and the
// four-body helper (site-energy descriptors of Sec. II.C of arXiv:2409.04430).
#pragma once

#include "internal.hpp"

namespace nep {

constexpr float kPi = 3.14159265358979f;

// Squared length, in one fixed sequence of fused operations.
__device__ __forceinline__ float norm2(float x, float y, float z) { return fmaf(z, z, fmaf(y, y, x * x)); }

// The functions below fix every rounding (contraction off, fused operations
// written out): the kernels that share them give the same bits wherever the
// compiler inlines them.

// sin(pi w) and cos(pi w) for w in [-1/2, 1/2]: the Taylor series through
// x^13 (sin) and x^14 (cos) is accurate to ~2e-7 in FP32 for |pi w| <= pi/2.
__device__ __forceinline__ void sincospi_half(float w, float &sw, float &cw)
{
#pragma clang fp contract(off)
    const float x = kPi * w;
    const float x2 = x * x;
    float ps = (float)(-1.0 / 6227020800.0);
    ps = fmaf(ps, x2, (float)(1.0 / 39916800.0));
    ps = fmaf(ps, x2, (float)(-1.0 / 362880.0));
    ps = fmaf(ps, x2, (float)(1.0 / 5040.0));
    ps = fmaf(ps, x2, (float)(-1.0 / 120.0));
    ps = fmaf(ps, x2, (float)(1.0 / 6.0));
    sw = fmaf(-(x * x2), ps, x);
    float pc = (float)(-1.0 / 87178291200.0);
    pc = fmaf(pc, x2, (float)(1.0 / 479001600.0));
    pc = fmaf(pc, x2, (float)(-1.0 / 3628800.0));
    pc = fmaf(pc, x2, (float)(1.0 / 40320.0));
    pc = fmaf(pc, x2, (float)(-1.0 / 720.0));
    pc = fmaf(pc, x2, (float)(1.0 / 24.0));
    pc = fmaf(pc, x2, (float)(-1.0 / 2.0));
    cw = fmaf(x2, pc, 1.0f);
}

// The cutoff function and the Chebyshev polynomials:
// f_c(r) = (1 + cos(pi r/rc))/2 and T_k(x), x = 2 (r/rc - 1)^2 - 1, so that
// f_k = (T_k + 1)/2 f_c.  Sums of f_k then follow from sums of f_c T_k and
// of f_c.  With w = r/rc - 1/2, cos(pi r/rc) = -sin(pi w) and
// sin(pi r/rc) = cos(pi w).
template <int K1>
__device__ __forceinline__ void cheb_t(float r, float rcinv, float &fc, float *T)
{
#pragma clang fp contract(off)
    float sw, cw;
    sincospi_half(fmaf(r, rcinv, -0.5f), sw, cw);
    fc = fmaf(-0.5f, sw, 0.5f);
    const float y = fmaf(r, rcinv, -1.0f);
    const float x = fmaf(y + y, y, -1.0f);
    const float x2 = x + x;
    T[0] = 1.0f;
    if (K1 > 1) T[1] = x;
#pragma unroll
    for (int k = 2; k < K1; ++k) T[k] = fmaf(x2, T[k - 1], -T[k - 2]);
}

// f_c, df_c/dr, dx/dr, T_k(x) and T_k'(x) (T_{k+1}' = 2 T_k + 2x T_k' - T_{k-1}'),
// so that df_k/dr = (T_k' dx/dr f_c + (T_k + 1) df_c/dr) / 2.
template <int K1>
__device__ __forceinline__ void cheb_td(float r, float rcinv, float &fc, float &fcp, float &dxdr, float *T, float *Tp)
{
#pragma clang fp contract(off)
    float sw, cw;
    sincospi_half(fmaf(r, rcinv, -0.5f), sw, cw);
    fc = fmaf(-0.5f, sw, 0.5f);
    fcp = (-0.5f * kPi * rcinv) * cw;
    const float y = fmaf(r, rcinv, -1.0f);
    const float x = fmaf(y + y, y, -1.0f);
    dxdr = (4.0f * rcinv) * y;
    const float x2 = x + x;
    T[0] = 1.0f;
    Tp[0] = 0.0f;
    if (K1 > 1) {
        T[1] = x;
        Tp[1] = 1.0f;
    }
#pragma unroll
    for (int k = 2; k < K1; ++k) {
        T[k] = fmaf(x2, T[k - 1], -T[k - 2]);
        Tp[k] = fmaf(x2, Tp[k - 1], fmaf(2.0f, T[k - 1], -Tp[k - 2]));
    }
}

// f_k and df_k/dr.
template <int K1>
__device__ __forceinline__ void cheb_fd(float r, float rcinv, float *f, float *fp)
{
    float fc, fcp, dx, T[K1], Tp[K1];
    cheb_td<K1>(r, rcinv, fc, fcp, dx, T, Tp);
    const float hf = 0.5f * fc, hp = 0.5f * fcp, hd = hf * dx;
    f[0] = fc;
    fp[0] = fcp;
#pragma unroll
    for (int k = 1; k < K1; ++k) {
        const float t1 = T[k] + 1.0f;
        f[k] = t1 * hf;
        fp[k] = fmaf(Tp[k], hd, t1 * hp);
    }
}

// Normalisations of 1 for sh_eval / adjoint_contract: the bare polynomials
// p_m of Y_m = c_m p_m (the multiplications fold away), for sums that apply
// c_m once after the neighbour loop.
struct UnitNorm {
    __device__ constexpr float operator[](int) const { return 1.0f; }
};

// Real spherical harmonics l = 1..4 (m = -l..l) at unit vector (x, y, z);
// c holds the normalisations (a generic or constant-space pointer, or
// UnitNorm for the bare polynomials).
template <typename CP>
__device__ __forceinline__ void sh_eval(float x, float y, float z, CP c, float *Y)
{
#pragma clang fp contract(off)
    const float x2 = x * x, y2 = y * y, z2 = z * z;
    const float xy = x * y, yz = y * z, xz = x * z;
    const float d = x2 - y2, e = fmaf(3.0f, x2, -y2), f = fmaf(-3.0f, y2, x2);
    const float a5 = fmaf(5.0f, z2, -1.0f), b7 = fmaf(7.0f, z2, -1.0f), c7 = fmaf(7.0f, z2, -3.0f);
    Y[0] = c[0] * y;
    Y[1] = c[1] * z;
    Y[2] = c[2] * x;
    Y[3] = c[3] * xy;
    Y[4] = c[4] * yz;
    Y[5] = c[5] * fmaf(3.0f, z2, -1.0f);
    Y[6] = c[6] * xz;
    Y[7] = c[7] * d;
    Y[8] = c[8] * (y * e);
    Y[9] = c[9] * (xy * z);
    Y[10] = c[10] * (y * a5);
    Y[11] = c[11] * (z * fmaf(5.0f, z2, -3.0f));
    Y[12] = c[12] * (x * a5);
    Y[13] = c[13] * (z * d);
    Y[14] = c[14] * (x * f);
    Y[15] = c[15] * (xy * d);
    Y[16] = c[16] * (yz * e);
    Y[17] = c[17] * (xy * b7);
    Y[18] = c[18] * (yz * c7);
    Y[19] = c[19] * fmaf(fmaf(35.0f, z2, -30.0f), z2, 3.0f);
    Y[20] = c[20] * (xz * c7);
    Y[21] = c[21] * (d * b7);
    Y[22] = c[22] * (xz * f);
    Y[23] = c[23] * fmaf(x2, f, -(y2 * e));
}

// Contraction of the own adjoints (stored times the harmonics'
// normalisations, so with the bare polynomials p_m) with the harmonics of
// one pair at unit vector (x, y, z):
//   sY = sum_m b'_m p_m(u),  grad = sum_m b_m grad p_m(u),
//   b_m = sum_n B_nm g_n,  b'_m = sum_n B_nm g'_n
// (p_m differentiated on R^3).  The polynomials share factors, e.g.
// x y (w_3 + z w_9 + (7 z^2 - 1) w_17 + (x^2 - y^2) w_15), so they are summed
// in seven groups in nested form, at most four m at a time (about 85
// operations after the sums over n, where each p_m and its gradient on its
// own takes about 120).
template <int NA1>
__device__ __forceinline__ void adjoint_contract(float x, float y, float z, const float (*B)[kNumSH], const float *g,
                                                 const float *gp, float &sY, float &gx, float &gy, float &gz)
{
#pragma clang fp contract(off)
    const float x2 = x * x, y2 = y * y, z2 = z * z;
    const float xy = x * y;
    const float d = x2 - y2, e = fmaf(3.0f, x2, -y2), f = fmaf(-3.0f, y2, x2);
    const float b7 = fmaf(7.0f, z2, -1.0f), z14 = 14.0f * z;
    const float d3 = 3.0f * d, xy6 = 6.0f * xy, ye = y * e, xf = x * f;
    auto sums = [&](int m, float &b, float &bp) {
        b = B[0][m] * g[0];
        bp = B[0][m] * gp[0];
#pragma unroll
        for (int n = 1; n < NA1; ++n) {
            b = fmaf(B[n][m], g[n], b);
            bp = fmaf(B[n][m], gp[n], bp);
        }
    };
    {   // xy, xyz, xy (7z^2 - 1), xy (x^2 - y^2)
        float b0, p0, b1, p1, b2, p2, b3, p3;
        sums(3, b0, p0);
        sums(9, b1, p1);
        sums(17, b2, p2);
        sums(15, b3, p3);
        const float s = fmaf(b7, b2, fmaf(z, b1, b0));
        gx = y * fmaf(e, b3, s);
        gy = x * fmaf(f, b3, s);
        gz = xy * fmaf(z14, b2, b1);
        sY = xy * fmaf(d, p3, fmaf(b7, p2, fmaf(z, p1, p0)));
    }
    {   // x^2 - y^2, z (x^2 - y^2), (x^2 - y^2)(7z^2 - 1), x^4 - 6 x^2 y^2 + y^4
        float b0, p0, b1, p1, b2, p2, b3, p3;
        sums(7, b0, p0);
        sums(13, b1, p1);
        sums(21, b2, p2);
        sums(23, b3, p3);
        const float s = fmaf(b7, b2, fmaf(z, b1, b0)), q = b3 + b3;
        gx = fmaf(x + x, fmaf(f, q, s), gx);
        gy = fmaf(-(y + y), fmaf(e, q, s), gy);
        gz = fmaf(d, fmaf(z14, b2, b1), gz);
        sY = fmaf(d, fmaf(b7, p2, fmaf(z, p1, p0)), sY);
        sY = fmaf(fmaf(x2, f, -(y2 * e)), p3, sY);
    }
    {   // y (3x^2 - y^2), yz (3x^2 - y^2)
        float b0, p0, b1, p1;
        sums(8, b0, p0);
        sums(16, b1, p1);
        const float s = fmaf(z, b1, b0);
        gx = fmaf(xy6, s, gx);
        gy = fmaf(d3, s, gy);
        gz = fmaf(ye, b1, gz);
        sY = fmaf(ye, fmaf(z, p1, p0), sY);
    }
    {   // x (x^2 - 3y^2), xz (x^2 - 3y^2)
        float b0, p0, b1, p1;
        sums(14, b0, p0);
        sums(22, b1, p1);
        const float s = fmaf(z, b1, b0);
        gx = fmaf(d3, s, gx);
        gy = fmaf(-xy6, s, gy);
        gz = fmaf(xf, b1, gz);
        sY = fmaf(xf, fmaf(z, p1, p0), sY);
    }
    const float a5 = fmaf(5.0f, z2, -1.0f), c7 = fmaf(7.0f, z2, -3.0f), t21 = fmaf(21.0f, z2, -3.0f), z10 = 10.0f * z;
    {   // y, yz, y (5z^2 - 1), yz (7z^2 - 3)
        float b0, p0, b1, p1, b2, p2, b3, p3;
        sums(0, b0, p0);
        sums(4, b1, p1);
        sums(10, b2, p2);
        sums(18, b3, p3);
        gy += fmaf(z, fmaf(c7, b3, b1), fmaf(a5, b2, b0));
        gz = fmaf(y, fmaf(t21, b3, fmaf(z10, b2, b1)), gz);
        sY = fmaf(y, fmaf(z, fmaf(c7, p3, p1), fmaf(a5, p2, p0)), sY);
    }
    {   // x, xz, x (5z^2 - 1), xz (7z^2 - 3)
        float b0, p0, b1, p1, b2, p2, b3, p3;
        sums(2, b0, p0);
        sums(6, b1, p1);
        sums(12, b2, p2);
        sums(20, b3, p3);
        gx += fmaf(z, fmaf(c7, b3, b1), fmaf(a5, b2, b0));
        gz = fmaf(x, fmaf(t21, b3, fmaf(z10, b2, b1)), gz);
        sY = fmaf(x, fmaf(z, fmaf(c7, p3, p1), fmaf(a5, p2, p0)), sY);
    }
    {   // z, 3z^2 - 1, z (5z^2 - 3), 35z^4 - 30z^2 + 3
        float b0, p0, b1, p1, b2, p2, b3, p3;
        sums(1, b0, p0);
        sums(5, b1, p1);
        sums(11, b2, p2);
        sums(19, b3, p3);
        gz += fmaf(fmaf(15.0f, z2, -3.0f), b2, b0);
        gz = fmaf(z, fmaf(fmaf(140.0f, z2, -60.0f), b3, 6.0f * b1), gz);
        sY = fmaf(z, fmaf(fmaf(5.0f, z2, -3.0f), p2, p0), sY);
        sY = fmaf(fmaf(3.0f, z2, -1.0f), p1, sY);
        sY = fmaf(fmaf(fmaf(35.0f, z2, -30.0f), z2, 3.0f), p3, sY);
    }
}

// The angular pair term d_ij from the contracted adjoints (adjoint_contract)
// at unit vector u and inverse distance rinv.
__device__ __forceinline__ void pair_term(float ux, float uy, float uz, float rinv, float sY, float gx, float gy,
                                          float gz, float &px, float &py, float &pz)
{
#pragma clang fp contract(off)
    const float ug = fmaf(uz, gz, fmaf(uy, gy, ux * gx));
    px = fmaf(sY, ux, fmaf(-ux, ug, gx) * rinv);
    py = fmaf(sY, uy, fmaf(-uy, ug, gy) * rinv);
    pz = fmaf(sY, uz, fmaf(-uz, ug, gz) * rinv);
}

// Radial pair term over r: the force on i is w r_ij, w = sum_k A_k f_k'(r) / r with
// A_k = a^i_k(tj) + a^j_k(ti); ai and aj end in the sum of a_k over k >= 1.
//   sum_k A_k f_k' = (dx/dr f_c sum A_k T_k' + f_c' sum A_k (T_k + 1)) / 2,
//   sum_{k>0} A_k (T_k + 1) = sum_{k>0} A_k T_k + (the stored sums of a_k)
template <int KR1>
__device__ __forceinline__ float radial_pair_w(float r2, float rcinv, const float *ai, const float *aj)
{
#pragma clang fp contract(off)
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float r = r2 * rinv;
    float fc, fcp, dxdr, T[KR1], Tp[KR1];
    cheb_td<KR1>(r, rcinv, fc, fcp, dxdr, T, Tp);
    float s1 = fmaf(2.0f, ai[0] + aj[0], ai[KR1] + aj[KR1]), s2 = 0.0f;
#pragma unroll
    for (int k = 1; k < KR1; ++k) {
        const float A = ai[k] + aj[k];
        s1 = fmaf(A, T[k], s1);
        s2 = fmaf(A, Tp[k], s2);
    }
    return 0.5f * fmaf(dxdr * fc, s2, fcp * s1) * rinv;
}

// l of spherical-harmonic slot m (0..23).
__host__ __device__ constexpr int sh_l(int m) { return m < 3 ? 1 : (m < 8 ? 2 : (m < 15 ? 3 : 4)); }

template <int NR1, int NA1, bool FOUR>
struct Dims {
    static constexpr int D = NR1 + kLmax * NA1 + (FOUR ? NA1 : 0);
};

// Four-body helper: M_n = sum_j g_n (u u^T - I/3) rebuilt from the l = 2 sums
// (slots 3..7 hold m = -2..2): returns mxy, myz, mzz, mxz, d = mxx - myy.
__device__ __forceinline__ void m_from_l2(const float *A2, const float *shc, float *M)
{
#pragma clang fp contract(off)
    M[0] = A2[0] / shc[3];
    M[1] = A2[1] / shc[4];
    M[2] = A2[2] / (3.0f * shc[5]);
    M[3] = A2[3] / shc[6];
    M[4] = A2[4] / shc[7];
}

// tr(M_n^3) of the four-body invariant from radial function n's l = 2 sums.
__device__ __forceinline__ float four_body_tr3(const float *A2, const float *shc)
{
#pragma clang fp contract(off)
    float M[5];
    m_from_l2(A2, shc, M);
    const float mxy = M[0], myz = M[1], mzz = M[2], mxz = M[3], dd = M[4];
    const float mxx = 0.5f * (dd - mzz), myy = 0.5f * (-dd - mzz);
    const float qxy = mxy * mxy, qyz = myz * myz, qxz = mxz * mxz;
    float t = mxx * fmaf(3.0f, qxy + qxz, mxx * mxx);
    t = fmaf(myy, fmaf(3.0f, qxy + qyz, myy * myy), t);
    t = fmaf(mzz, fmaf(3.0f, qxz + qyz, mzz * mzz), t);
    return fmaf(6.0f * mxy * myz, mxz, t);
}

// Adjoint of one radial function n's angular sums, stored as B_nlm c_m:
// B_nlm = dU/dA_nlm = 2 (dU/dq_nl) A_nlm, plus for the four-body invariant
// q4_n = kappa tr(M_n^3) the derivative through M_n's l = 2 entries,
// 3 kappa (dU/dq4_n) d tr(M^3)/dM = 3 g4 M^2 mapped back onto m = -2..2.
// Gl[l - 1] = dU/dq_nl, g4 = kappa dU/dq4_n.  An and Bn may be the same
// array (M is formed before any entry is written).
template <bool FOUR>
__device__ __forceinline__ void form_adjoint(const float *An, const float (&Gl)[kLmax], float g4,
                                             const float *__restrict__ shc, float *Bn)
{
#pragma clang fp contract(off)
    float M[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (FOUR) m_from_l2(&An[3], shc, M);
#pragma unroll
    for (int m = 0; m < kNumSH; ++m) Bn[m] = 2.0f * Gl[sh_l(m) - 1] * An[m];
    if (FOUR) {
        const float mxy = M[0], myz = M[1], mzz = M[2], mxz = M[3], dd = M[4];
        const float mxx = 0.5f * (dd - mzz), myy = 0.5f * (-dd - mzz);
        // entries of M^2
        const float sxx = norm2(mxx, mxy, mxz);
        const float syy = norm2(mxy, myy, myz);
        const float szz = norm2(mxz, myz, mzz);
        const float sxy = fmaf(mxz, myz, mxy * (mxx + myy));
        const float syz = fmaf(mxy, mxz, myz * (myy + mzz));
        const float sxz = fmaf(mxy, myz, mxz * (mxx + mzz));
        Bn[3] += g4 * 6.0f * sxy / shc[3];
        Bn[4] += g4 * 6.0f * syz / shc[4];
        Bn[5] += g4 * 3.0f * (szz - 0.5f * sxx - 0.5f * syy) / (3.0f * shc[5]);
        Bn[6] += g4 * 6.0f * sxz / shc[6];
        Bn[7] += g4 * 1.5f * (sxx - syy) / shc[7];
    }
    // stored as B_nlm c_m, the factor the pair terms need with the bare polynomials
#pragma unroll
    for (int m = 0; m < kNumSH; ++m) Bn[m] *= shc[m];
}

// Directional derivatives D_m = c_m grad p_m(u) . v of the 24 harmonics
// (Y_m = c_m p_m) along v, p_m differentiated on R^3.
__device__ __forceinline__ void sh_dir(float x, float y, float z, float vx, float vy, float vz,
                                       const float *__restrict__ c, float *D)
{
    const float x2 = x * x, y2 = y * y, z2 = z * z;
    const float xy = x * y, yz = y * z, xz = x * z;
    D[0] = c[0] * (vy);
    D[1] = c[1] * (vz);
    D[2] = c[2] * (vx);
    D[3] = c[3] * (vx * (y) + vy * (x));
    D[4] = c[4] * (vy * (z) + vz * (y));
    D[5] = c[5] * (vz * (6.0f * z));
    D[6] = c[6] * (vx * (z) + vz * (x));
    D[7] = c[7] * (vx * (2.0f * x) - vy * (2.0f * y));
    D[8] = c[8] * (vx * (6.0f * xy) + vy * (3.0f * (x2 - y2)));
    D[9] = c[9] * (vx * (yz) + vy * (xz) + vz * (xy));
    D[10] = c[10] * (vy * ((5.0f * z2 - 1.0f)) + vz * (10.0f * yz));
    D[11] = c[11] * (vz * ((15.0f * z2 - 3.0f)));
    D[12] = c[12] * (vx * ((5.0f * z2 - 1.0f)) + vz * (10.0f * xz));
    D[13] = c[13] * (vx * (2.0f * xz) - vy * (2.0f * yz) + vz * ((x2 - y2)));
    D[14] = c[14] * (vx * (3.0f * (x2 - y2)) - vy * (6.0f * xy));
    D[15] = c[15] * (vx * ((3.0f * x2 * y - y2 * y)) + vy * ((x2 * x - 3.0f * x * y2)));
    D[16] = c[16] * (vx * (6.0f * xy * z) + vy * (3.0f * z * (x2 - y2)) + vz * ((3.0f * x2 * y - y2 * y)));
    D[17] = c[17] * (vx * (y * (7.0f * z2 - 1.0f)) + vy * (x * (7.0f * z2 - 1.0f)) + vz * (14.0f * xy * z));
    D[18] = c[18] * (vy * (z * (7.0f * z2 - 3.0f)) + vz * (y * (21.0f * z2 - 3.0f)));
    D[19] = c[19] * (vz * (z * (140.0f * z2 - 60.0f)));
    D[20] = c[20] * (vx * (z * (7.0f * z2 - 3.0f)) + vz * (x * (21.0f * z2 - 3.0f)));
    D[21] = c[21] * (vx * (2.0f * x * (7.0f * z2 - 1.0f)) - vy * (2.0f * y * (7.0f * z2 - 1.0f)) + vz * (14.0f * z * (x2 - y2)));
    D[22] = c[22] * (vx * (3.0f * z * (x2 - y2)) - vy * (6.0f * xy * z) + vz * (x * (x2 - 3.0f * y2)));
    D[23] = c[23] * (vx * ((4.0f * x2 * x - 12.0f * x * y2)) + vy * ((4.0f * y2 * y - 12.0f * x2 * y)));
}

}  // namespace nep
