// NEP energy, forces and virial of small systems on gfx950 (site-energy
// model of Sec. II.C, bead forces and virial of Sec. II.A of
// arXiv:2409.04430): one wavefront per (atom, bead), its lanes the
// neighbours.
//
// The kernels of nep.hip give every (atom, bead) one lane, which walks its
// neighbours one after another: with fewer rows than the chip has lanes to
// fill (65,536 for one wavefront per SIMD) they take the time of one such
// walk, however few rows there are.  Here a row's neighbours are evaluated
// side by side and their contributions left in LDS; each sum over
// neighbours (a basis sum, an A_nlm, a force or virial component) then has
// an owner lane that adds the contributions in list order.  Every number is
// thus formed by the same operations in the same order as in nep.hip, and
// the results agree bit for bit, so the choice between the two may follow
// the size of a call (takes_small).  Bound by latency at a few rows and by
// the LDS reads of the owner lanes as rows grow; 108 atoms x 4 beads: 125 ->
// 25 us for the kernels, 1,536 atoms x 1 bead 359 -> 40 us.
//   k_small_site  descriptor, network, adjoints and the angular pair terms
//                 (k_descriptor and k_force_ang in one: the adjoints B stay
//                 in LDS);
//   k_small_rad   radial pair terms and the reverse angular terms
//                 (k_force_rad).
// Energy and virial go out per row; the per-bead sums run over the same
// tiles of atoms in the same order as the partials of nep.hip.
#include "nep_net.hpp"
#include "nep_small.hpp"

namespace nep {

constexpr int kNetVector = 0;   // FP32 vector units (kNetBf16 and kNetMf32 as in nep.hip)
constexpr int kYPad = 25;       // row stride of the 24 harmonics in LDS (odd: no bank conflicts across lanes)

template <int NR1, int NA1, bool FOUR, int NET>
__global__ __launch_bounds__(64) void k_small_site(NepArgs a, const float *__restrict__ prm,
                                                   const int32_t *__restrict__ atom_sys, float *__restrict__ rowp)
{
    constexpr int KR1 = 9, KA1 = 9, D = Dims<NR1, NA1, FOUR>::D;
    constexpr bool MF = NET != kNetVector;
    constexpr int NACC = (NA1 * kNumSH + 63) / 64;   // angular sums owned by a lane
    // dynamic LDS: vector network, h and dU/dz of the hidden units; matrix-core network, its tile
    extern __shared__ float dyn[];
    __shared__ float sg[64 * NA1];                   // per neighbour: g_n, or fc and T_k
    __shared__ float sy[64 * kYPad];                 // per neighbour: harmonics, or pair term and vector
    __shared__ float ssk[kMaxSpecies * KR1];         // radial basis sums
    __shared__ float sq[D], sG[D];                   // descriptors (then scaled), their adjoints
    __shared__ float sA[NA1][kNumSH], sB[NA1][kNumSH];
    __shared__ float sc[kMaxSpecies * NA1 * KA1];    // angular coefficients of the centre's species
    __shared__ float scs[kMaxSpecies * NA1];
    static_assert(KR1 <= kYPad, "radial staging exceeds the harmonics' buffer");

    const int P = a.P, S = a.S, lane = threadIdx.x;
    const int i = blockIdx.x / P, b = blockIdx.x - i * P;
    const size_t PN = (size_t)P * a.N, at = (size_t)b * a.N + i;
    const int ti = a.types[i];
    const bool tok = ti >= 0 && ti < S;
    if (!tok) {   // whole wavefront
        if (lane == 0) {
            if (a.Eatom) a.Eatom[at] = 0.0f;
            atomicOr(a.flags, (uint32_t)NEP_FLAG_BAD_TYPE);
        }
        if (lane < 3) a.Fang[((size_t)i * P + b) * 3 + lane] = 0.0f;
        if (lane < 10) rowp[lane * PN + at] = 0.0f;
        if (a.Watom && lane < 9) a.Watom[at * 9 + lane] = 0.0f;
        return;
    }
    const LaneMap lm = row_map(a.geom[atom_sys[i]], i, b);
    const float4 *p4b = a.p4 + b;
    const uint32_t pstride = (uint32_t)P * sizeof(float4);
    const float4 pi = *row_at(p4b, i, pstride);
    const float *shc = prm + a.osh;
    const int32_t *uendR = a.uendR + (size_t)i * kMaxSpecies, *uendA = a.uendA + (size_t)i * kMaxSpecies;

    // ---- radial basis sums: owner lane 9 t + k adds f_c T_k (T_0 = 1) over species block t
    const int to = lane / KR1, ko = lane - to * KR1;
    const bool own = to < S;
    {
        const int32_t *uR = a.uniR + (size_t)i * a.capR;
        const uint64_t *mR = a.umR + (size_t)i * a.capR;
        const int n = uendR[S - 1];
        const int o0 = own && to ? uendR[to - 1] : 0, o1 = own ? uendR[to] : 0;
        float acc = 0.0f;
        for (int p0 = 0; p0 < n; p0 += 64) {
            const int e = p0 + lane;
            float fc = 0.0f, T[KR1];
#pragma unroll
            for (int k = 0; k < KR1; ++k) T[k] = 0.0f;
            if (e < n && ((mR[e] >> b) & 1u)) {
                float dx, dy, dz;
                pair_vec<kPosAny>(*row_at(p4b, uR[e], pstride), pi, lm, dx, dy, dz);
                cheb_t<KR1>(__builtin_amdgcn_sqrtf(norm2(dx, dy, dz)), a.rcRinv, fc, T);
            }
            sy[lane * kYPad] = fc;
#pragma unroll
            for (int k = 1; k < KR1; ++k) sy[lane * kYPad + k] = T[k];
            wave_lds_sync();
            const int hi = min(o1 - p0, 64);
#pragma unroll 4
            for (int x = max(o0 - p0, 0); x < hi; ++x)
                acc = fmaf(sy[x * kYPad], ko ? sy[x * kYPad + ko] : 1.0f, acc);
            wave_lds_sync();
        }
        const float s0 = __shfl(acc, min(to, kMaxSpecies - 1) * KR1, 64);
        if (own) ssk[lane] = ko ? 0.5f * (acc + s0) : acc;
    }
    // angular coefficients of this species pair row, and cs_n = c_n0 + sum_k c_nk
    {
        const float *c = prm + a.oA + ti * S * NA1 * KA1;
        for (int x = lane; x < S * NA1 * KA1; x += 64) sc[x] = c[x];
    }
    wave_lds_sync();
    if (lane < NR1) {
        float q = 0.0f;
        for (int t = 0; t < S; ++t) {
            const float *c = prm + a.oR + (ti * S + t) * NR1 * KR1 + lane * KR1;
#pragma unroll
            for (int k = 0; k < KR1; ++k) q = fmaf(c[k], ssk[t * KR1 + k], q);
        }
        sq[lane] = q;
    }
    if (lane < S * NA1) {
        float acc = sc[lane * KA1];
#pragma unroll
        for (int k = 0; k < KA1; ++k) acc += sc[lane * KA1 + k];
        scs[lane] = acc;
    }
    wave_lds_sync();

    // ---- angular sums: owner lane of entry (n, m) adds g_n p_m over the neighbours
    const int32_t *uW = a.uniW + (size_t)i * a.capA;
    const uint64_t *mA = a.umA + (size_t)i * a.capA;
    const int nA = uendA[S - 1];
    {
        float A[NACC];
        int on[NACC], om[NACC];
#pragma unroll
        for (int q = 0; q < NACC; ++q) {
            const int x = min(lane + 64 * q, NA1 * kNumSH - 1);
            A[q] = 0.0f;
            on[q] = x / kNumSH;
            om[q] = x - on[q] * kNumSH;
        }
        for (int p0 = 0; p0 < nA; p0 += 64) {
            const int e = p0 + lane;
            float g[NA1], Y[kNumSH];
#pragma unroll
            for (int n = 0; n < NA1; ++n) g[n] = 0.0f;
#pragma unroll
            for (int m = 0; m < kNumSH; ++m) Y[m] = 0.0f;
            if (e < nA && ((mA[e] >> b) & 1u)) {
                const int32_t w = uW[e];
                float dx, dy, dz;
                pair_vec<kPosAny>(*row_at(p4b, w >> 2, pstride), pi, lm, dx, dy, dz);
                const float r2 = norm2(dx, dy, dz);
                const float rinv = __builtin_amdgcn_rsqf(r2);
                const float r = r2 * rinv;
                float fc, T[KA1];
                cheb_t<KA1>(r, a.rcAinv, fc, T);
                const float hf = 0.5f * fc;
                sh_eval(dx * rinv, dy * rinv, dz * rinv, UnitNorm{}, Y);
                const int t = w & 3;
#pragma unroll
                for (int n = 0; n < NA1; ++n) {
                    float gn = scs[t * NA1 + n];
#pragma unroll
                    for (int k = 1; k < KA1; ++k) gn = fmaf(sc[(t * NA1 + n) * KA1 + k], T[k], gn);
                    g[n] = gn * hf;
                }
            }
#pragma unroll
            for (int n = 0; n < NA1; ++n) sg[lane * NA1 + n] = g[n];
#pragma unroll
            for (int m = 0; m < kNumSH; ++m) sy[lane * kYPad + m] = Y[m];
            wave_lds_sync();
            const int hi = min(nA - p0, 64);
#pragma unroll 4
            for (int x = 0; x < hi; ++x)
#pragma unroll
                for (int q = 0; q < NACC; ++q) A[q] = fmaf(sg[x * NA1 + on[q]], sy[x * kYPad + om[q]], A[q]);
            wave_lds_sync();
        }
#pragma unroll
        for (int q = 0; q < NACC; ++q)
            if (lane + 64 * q < NA1 * kNumSH) sA[on[q]][om[q]] = A[q] * shc[om[q]];   // A_nlm = c_m sum_j g_n p_m
    }
    wave_lds_sync();
    if (lane < NA1) {
#pragma unroll
        for (int l = 1; l <= kLmax; ++l) {
            float s2 = 0.0f;
#pragma unroll
            for (int m = 0; m < kNumSH; ++m)
                if (sh_l(m) == l) s2 = fmaf(sA[lane][m], sA[lane][m], s2);
            sq[NR1 + (l - 1) * NA1 + lane] = s2;
        }
        if (FOUR) {
            float A2[5];
#pragma unroll
            for (int m = 0; m < 5; ++m) A2[m] = sA[lane][3 + m];
            sq[NR1 + kLmax * NA1 + lane] = a.kappa4 * four_body_tr3(A2, shc);
        }
    }
    wave_lds_sync();
    const float *qs = prm + a.oq;
    const float qsl = qs[min(lane, D - 1)];
    static_assert(D < 64, "one lane per descriptor, and one for the energy");
    if (lane < D) sq[lane] *= qsl;
    wave_lds_sync();

    // ---- network: U and G_nu = dU/dq_nu
    const int H = a.H;
    const float *b0 = prm + a.ob0 + ti * H, *w1 = prm + a.ow1 + ti * H;
    float U;
    if constexpr (MF) {
        constexpr int WT = NET == kNetMf32 ? 3 : 1;
        float qh[D], G[D];
#pragma unroll
        for (int v = 0; v < D; ++v) qh[v] = sq[v];
        const MlpFrag fl = mlp_frag_layout(D, H, WT);
        // the row in lane 0 of the first batch tile
        U = mlp_mf<D, WT, 1>(qh, lane == 0, a.w0b + (size_t)ti * fl.species_stride, b0, w1, prm[a.ob1], H, dyn, G);
        if (lane == 0) {
#pragma unroll
            for (int v = 0; v < D; ++v) sG[v] = G[v];
        }
        U = __shfl(U, 0, 64);
        wave_lds_sync();
    } else {
        // a hidden unit per lane, then per lane one component of G (and, in
        // the last lane, U) summed over the hidden units in order
        const float *W0 = prm + a.oW0 + (size_t)ti * H * D;
        float *sh = dyn, *sz = dyn + H;
        for (int mu = lane; mu < H; mu += 64) {
            float z = -b0[mu];
#pragma unroll
            for (int v = 0; v < D; ++v) z = fmaf(W0[mu * D + v], sq[v], z);
            float h, dh;
            tanh_and_slope(z, h, dh);
            sh[mu] = h;
            sz[mu] = w1[mu] * dh;
        }
        wave_lds_sync();
        const bool last = lane == 63;
        const float *wp = last ? w1 : W0 + min(lane, D - 1);
        const float *xp = last ? sh : sz;
        const int ws = last ? 1 : D;
        float acc = last ? -prm[a.ob1] : 0.0f;
#pragma unroll 10
        for (int mu = 0; mu < H; ++mu) acc = fmaf(xp[mu], wp[mu * ws], acc);
        if (lane < D) sG[lane] = acc;
        U = __shfl(acc, 63, 64);
        wave_lds_sync();
    }
    if (lane < D) sG[lane] *= qsl;
    wave_lds_sync();

    // ---- adjoints: B_nlm c_m, one radial function per lane, and the radial a_k(t)
    if (lane < NA1) {
        float An[kNumSH];
#pragma unroll
        for (int m = 0; m < kNumSH; ++m) An[m] = sA[lane][m];
        const float Gl[kLmax] = {sG[NR1 + lane], sG[NR1 + NA1 + lane], sG[NR1 + 2 * NA1 + lane],
                                 sG[NR1 + 3 * NA1 + lane]};
        const float g4 = FOUR ? sG[NR1 + kLmax * NA1 + (FOUR ? lane : 0)] * a.kappa4 : 0.0f;
        float Bn[kNumSH];
        form_adjoint<FOUR>(An, Gl, g4, shc, Bn);
#pragma unroll
        for (int m = 0; m < kNumSH; ++m) sB[lane][m] = Bn[m];
    }
    if (own) {
        const float *c = prm + a.oR + (ti * S + to) * NR1 * KR1 + ko;
        float acc = 0.0f;
#pragma unroll
        for (int n = 0; n < NR1; ++n) acc = fmaf(sG[n], c[n * KR1], acc);
        ssk[lane] = acc;
    }
    wave_lds_sync();
    if (own) {
        float *ao = a.arad + (((size_t)i * S + to) * P + b) * kRadPad;
        ao[ko] = ssk[lane];
        if (ko == 0) {
            float s = 0.0f;
#pragma unroll
            for (int k = 1; k < KR1; ++k) s += ssk[to * KR1 + k];
            ao[KR1] = s;
        }
    }

    // ---- angular pair terms: per lane one neighbour, owner lanes 0..2 force, 3..11 virial
    const int32_t *uV = a.uniV + (size_t)i * a.capA;
    float4 *pairb = a.pairbuf + b;
    const int we = lane - 3, wa = we / 3, wb = we - 3 * wa;
    float acc = 0.0f, first = 0.0f;
    // entry where the second part of the sums begins (half_point)
    int mid = nA;
    if (two_parts(NA1, a.lg)) {
        const int hp = half_point(nA);
        for (int t = S - 1; t >= 0; --t) {
            const int s0 = t ? uendA[t - 1] : 0, s1 = uendA[t];
            const int m = s0 + split_batches(s0, s1, hp) * kBatchAng;
            if (m < s1) mid = m;
        }
    }
    for (int p0 = 0; p0 < nA; p0 += 64) {
        const int e = p0 + lane;
        const bool act = e < nA && ((mA[e < nA ? e : 0] >> b) & 1u);
        float px = 0.0f, py = 0.0f, pz = 0.0f, dx = 1.0f, dy = 0.0f, dz = 0.0f;
        if (act) {
            const int32_t w = uW[e];
            const int rk = uV[e], j = w >> 2, t = w & 3;
            pair_vec<kPosAny>(*row_at(p4b, j, pstride), pi, lm, dx, dy, dz);
            const float r2 = norm2(dx, dy, dz);
            const float rinv = __builtin_amdgcn_rsqf(r2);
            const float r = r2 * rinv;
            const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
            float gij[NA1], gpij[NA1];
            {
                float fc, fcp, dxdr, T[KA1], Tp[KA1];
                cheb_td<KA1>(r, a.rcAinv, fc, fcp, dxdr, T, Tp);
                const float hf = 0.5f * fc, hfp = 0.5f * fcp, hd = hf * dxdr;
#pragma unroll
                for (int n = 0; n < NA1; ++n) {
                    const float *cij = sc + (t * NA1 + n) * KA1;
                    float pn = 2.0f * cij[0], qn = 0.0f;
#pragma unroll
                    for (int k = 1; k < KA1; ++k) {
                        pn = fmaf(cij[k], T[k] + 1.0f, pn);
                        qn = fmaf(cij[k], Tp[k], qn);
                    }
                    gij[n] = hf * pn;
                    gpij[n] = fmaf(hd, qn, hfp * pn);
                }
            }
            float sY, gx, gy, gz;
            adjoint_contract<NA1>(ux, uy, uz, sB, gij, gpij, sY, gx, gy, gz);
            pair_term(ux, uy, uz, rinv, sY, gx, gy, gz, px, py, pz);
            if (rk >= 0)
                *const_cast<float4 *>(row_at(row_at(pairb, j, (uint32_t)a.capA * pstride), rk, pstride)) =
                    make_float4(px, py, pz, 0.0f);
        }
        float *o = sy + lane * kYPad;
        o[0] = px; o[1] = py; o[2] = pz;
        o[3] = dx; o[4] = dy; o[5] = dz;
        wave_lds_sync();
        const int hi = min(nA - p0, 64), xm = min(max(mid - p0, 0), hi);
        for (int h = 0; h < 2; ++h) {
            const int x0 = h ? xm : 0, x1 = h ? hi : xm;
            if (h && mid >= p0 && mid < p0 + 64) {
                first = acc;
                acc = 0.0f;
            }
            if (lane < 3) {
#pragma unroll 4
                for (int x = x0; x < x1; ++x) acc += sy[x * kYPad + lane];
            } else if (lane < 12) {
#pragma unroll 4
                for (int x = x0; x < x1; ++x) acc = fmaf(-sy[x * kYPad + 3 + wa], sy[x * kYPad + wb], acc);
            }
        }
        wave_lds_sync();
    }
    acc += first;
    if (lane < 3) {
        a.Fang[((size_t)i * P + b) * 3 + lane] = acc;
    } else if (lane < 12) {
        rowp[(size_t)(1 + we) * PN + at] = acc;
        if (a.Watom) a.Watom[at * 9 + we] = 0.5f * acc;   // own half of the per-atom split
    } else if (lane == 12) {
        rowp[at] = U;
        if (a.Eatom) a.Eatom[at] = U;
    }
}

__global__ __launch_bounds__(64) void k_small_rad(NepArgs a, const int32_t *__restrict__ atom_sys,
                                                  float *__restrict__ rowp)
{
    constexpr int KR1 = 9, kPad = 7;
    __shared__ float sv[64 * kPad];   // per neighbour: pair term and vector
    const int P = a.P, S = a.S, lane = threadIdx.x;
    const int i = blockIdx.x / P, b = blockIdx.x - i * P;
    const size_t PN = (size_t)P * a.N, at = (size_t)b * a.N + i;
    const int ti = a.types[i];
    const bool tok = ti >= 0 && ti < S;
    const LaneMap lm = row_map(a.geom[atom_sys[i]], i, b);
    const float4 *p4b = a.p4 + b;
    const uint32_t pstride = (uint32_t)P * sizeof(float4);
    const float4 pi = *row_at(p4b, i, pstride);
    // owner lanes: 0..2 force (FP64); 3..11 virial: radial entries (six of them summed, the
    // symmetric ones copied) and, for the per-atom virial, the reverse angular ones
    const int we = lane - 3, wa = (lane >= 3 ? we : 0) / 3, wb = (lane >= 3 ? we : 0) - 3 * wa;
    double Fd = 0.0;
    float Wf = 0.0f, Wa = 0.0f;
    if (tok) {
        const float *ab = a.arad + (size_t)b * kRadPad;
        const uint32_t trow = (uint32_t)P * kRadPad * sizeof(float), astride = (uint32_t)S * trow;
        const float *abt = row_at(ab, ti, trow);
        auto load_a = [&](const float *row, float (&out)[KR1 + 1]) {
            const float4 *p = reinterpret_cast<const float4 *>(row);
            const float4 v0 = p[0], v1 = p[1], v2 = p[2];
            out[0] = v0.x; out[1] = v0.y; out[2] = v0.z; out[3] = v0.w;
            out[4] = v1.x; out[5] = v1.y; out[6] = v1.z; out[7] = v1.w;
            out[8] = v2.x; out[9] = v2.y;
        };
        const int32_t *uR = a.uniR + (size_t)i * a.capR;
        const uint64_t *mR = a.umR + (size_t)i * a.capR;
        for (int t = 0; t < S; ++t) {
            int s0, s1;
            block_range(a.uendR, i, t, s0, s1);
            float ai[KR1 + 1];
            load_a(row_at(row_at(ab, t, trow), i, astride), ai);
            for (int p0 = s0; p0 < s1; p0 += 64) {
                const int e = p0 + lane;
                float w = 0.0f, dx = 1.0f, dy = 0.0f, dz = 0.0f;
                if (e < s1 && ((mR[e] >> b) & 1u)) {
                    const int j = uR[e];
                    float aj[KR1 + 1];
                    load_a(row_at(abt, j, astride), aj);
                    pair_vec<kPosAny>(*row_at(p4b, j, pstride), pi, lm, dx, dy, dz);
                    w = radial_pair_w<KR1>(norm2(dx, dy, dz), a.rcRinv, ai, aj);
                }
                float *o = sv + lane * kPad;
                o[0] = w * dx; o[1] = w * dy; o[2] = w * dz;
                o[3] = dx; o[4] = dy; o[5] = dz;
                o[6] = w;
                wave_lds_sync();
                const int cnt = min(s1 - p0, 64);
                if (lane < 3) {
                    // FP32 sums over batches of kBatch entries, each added to the FP64 force
                    for (int x0 = 0; x0 < cnt; x0 += kBatch) {
                        float f = 0.0f;
#pragma unroll
                        for (int u = 0; u < kBatch; ++u) {   // entries past the list's end hold zeros
                            const float *q = sv + (x0 + u) * kPad;
                            f = fmaf(q[6], q[3 + lane], f);
                        }
                        Fd += (double)f;
                    }
                } else if (lane < 12 && wb >= wa) {
#pragma unroll 4
                    for (int x = 0; x < cnt; ++x)
                        Wf = fmaf(-0.5f * sv[x * kPad + 3 + wa], sv[x * kPad + wb], Wf);
                }
                wave_lds_sync();
            }
        }
        // reverse angular terms, and their half of the per-atom virial
        const int32_t *uA = a.uniA + (size_t)i * a.capA;
        const uint64_t *mA = a.umA + (size_t)i * a.capA;
        const int32_t *uW = a.uniW + (size_t)i * a.capA;
        const float4 *pbuf = row_at(a.pairbuf + b, i, (uint32_t)a.capA * pstride);
        const int nA = a.uendA[(size_t)i * kMaxSpecies + S - 1];
        float g = 0.0f;
        for (int p0 = 0; p0 < nA; p0 += 64) {
            const int e = p0 + lane;
            float4 d = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            float dx = 0.0f, dy = 0.0f, dz = 0.0f;
            if (e < nA && ((mA[e] >> b) & 1u)) {
                const int slot = uA[e];
                d = *row_at(pbuf, slot, pstride);
                if (a.Watom) pair_vec<kPosAny>(*row_at(p4b, uW[e] >> 2, pstride), pi, lm, dx, dy, dz);
            }
            float *o = sv + lane * kPad;
            o[0] = d.x; o[1] = d.y; o[2] = d.z;
            o[3] = dx; o[4] = dy; o[5] = dz;
            wave_lds_sync();
            const int cnt = min(nA - p0, 64);
            if (lane < 3) {
#pragma unroll 4
                for (int x = 0; x < cnt; ++x) g -= sv[x * kPad + lane];
            } else if (lane < 12 && a.Watom) {
#pragma unroll 4
                for (int x = 0; x < cnt; ++x) Wa = fmaf(0.5f * sv[x * kPad + 3 + wa], sv[x * kPad + wb], Wa);
            }
            wave_lds_sync();
        }
        Fd += (double)g;
    }
    // the symmetric entries of the radial virial
    const int src = lane >= 3 && lane < 12 && wb < wa ? 3 + 3 * wb + wa : lane;
    Wf = __shfl(Wf, src, 64);
    if (lane < 3) {
        const double f = Fd + (double)a.Fang[((size_t)i * P + b) * 3 + lane];
        a.F[at * 3 + lane] = (float)f;
        if (!isfinite(f)) atomicOr(a.flags, (uint32_t)NEP_FLAG_NONFINITE);
    } else if (lane < 12) {
        rowp[(size_t)(10 + we) * PN + at] = Wf;
        if (a.Watom) {
            float *wo = a.Watom + at * 9 + we;
            *wo = (float)((double)Wf + (double)Wa + (double)*wo);
        }
    }
}

template <int NR1, int NA1, bool FOUR>
static void launch_site(const NepArgs &a, const nep_model *m, const int32_t *atom_sys, float *rowp, hipStream_t s)
{
    constexpr int D = Dims<NR1, NA1, FOUR>::D;
    const dim3 g((unsigned)(a.N * a.P));
    const size_t mf = sizeof(float) * (size_t)mf_lds_floats<D>() / 4;   // one 16-row tile
    ProfScope ps_(K_DESCRIPTOR, s);
    if (m->mlp == NEP_MLP_BF16_MFMA)
        hipLaunchKernelGGL((k_small_site<NR1, NA1, FOUR, kNetBf16>), g, dim3(64), mf, s, a, m->dev, atom_sys, rowp);
    else if (m->mlp == NEP_MLP_FP32_MFMA)
        hipLaunchKernelGGL((k_small_site<NR1, NA1, FOUR, kNetMf32>), g, dim3(64), mf, s, a, m->dev, atom_sys, rowp);
    else
        hipLaunchKernelGGL((k_small_site<NR1, NA1, FOUR, kNetVector>), g, dim3(64), sizeof(float) * 2 * a.H, s, a,
                           m->dev, atom_sys, rowp);
}

int32_t launch_small(const NepArgs &a, const nep_model *m, const int32_t *atom_sys, float *rowp, hipStream_t s)
{
    switch (m->hp.n_max_radial * 100 + m->hp.n_max_angular * 10 + m->hp.four_body) {
    case 440: launch_site<5, 5, false>(a, m, atom_sys, rowp, s); break;
    case 441: launch_site<5, 5, true>(a, m, atom_sys, rowp, s); break;
    case 640: launch_site<7, 5, false>(a, m, atom_sys, rowp, s); break;
    case 860: launch_site<9, 7, false>(a, m, atom_sys, rowp, s); break;
    case 881: launch_site<9, 9, true>(a, m, atom_sys, rowp, s); break;
    default: return fail(NEP_ERR_UNSUPPORTED, "nep_compute: unsupported model shape");
    }
    ProfScope ps_(K_FORCE, s);
    hipLaunchKernelGGL(k_small_rad, dim3((unsigned)(a.N * a.P)), dim3(64), 0, s, a, atom_sys, rowp);
    return NEP_OK;
}

}  // namespace nep
