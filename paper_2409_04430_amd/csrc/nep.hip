// NEP energy, forces and virial on gfx950 (site-energy model of Sec. II.C,
// bead forces and virial of Sec. II.A of arXiv:2409.04430).
//
// Four kernels per call, one lane per (bead, atom) (small systems: the
// kernels of nep_small.hip), neighbours taken from
// the per-bead compact lists built over the shared centroid candidate rows:
//   k_descriptor  radial sums, angular sums A_nlm = sum_j g_n(r_ij) Y_lm(u_ij)
//                 over real orthonormal spherical harmonics, q_nl = sum_m A_nlm^2
//                 (equal to the Legendre double sum by the addition theorem),
//                 the optional (2,2,2) four-body invariant, the tanh network,
//                 and the adjoints: B_nlm = dU_i/dA_nlm (stored times the
//                 harmonic's normalisation c_m) and the radial
//                 a_k(t) = sum_n dU_i/dq_n c^{ti t}_nk (with their sum over k > 0);
//   k_force_ang   angular pair terms d_ij = dU_i/dr_ij from the atom's own
//                 adjoints, kept per (bead, atom, candidate slot);
//   k_force_rad   radial pair terms (a^i_k(tj) + a^j_k(ti)) f'_k(r) u, the
//                 reverse angular terms d_ji gathered through the reverse
//                 slots, so that F_i = sum_j (dU_i/dr_ij - dU_j/dr_ji) needs no
//                 atomics; per-atom virial -1/2 sum_j r_ij (x) (d_ij - d_ji);
//   k_reduce      per-bead energy and virial from per-block partial sums in
//                 a fixed order (bitwise reproducible).
// The descriptor and angular-force passes run species-uniform groups of
// lanes, which makes every model-coefficient address wave-uniform (scalar
// loads, SGPR operands).  Neighbour loops keep several gathers in flight.
#include "internal.hpp"
#include "nep_kernels.hpp"
#include "nep_net.hpp"
#include "nep_small.hpp"

namespace nep {

// ----------------------------------------------------------- pass 1 ---

template <int NR1, int NA1, int KR1, int KA1, bool FOUR, int NET, int FORM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(2)))
void k_descriptor(NepArgs a, const float *__restrict__ prm)
{
    constexpr bool MF = NET == kNetBf16 || NET == kNetMf32;   // whole-wavefront network on the matrix cores
    constexpr bool NL = NET == kNetLds;
    // dynamic LDS: matrix-core network, one 64 x (32 or 64, + 4) tile per
    // wavefront; LDS weights, W0 [S][H][DP] (rows padded to DP = 4 ceil(D / 4)),
    // b0 [S][H], w1 [S][H]
    extern __shared__ float dyn[];
    constexpr int D = Dims<NR1, NA1, FOUR>::D;
    const LaneMap lm = lane_map(a, threadIdx.x);
    const int i = lm.i, b = lm.b, P = a.P, S = a.S;
    const bool valid = lm.valid;
    const int ti = a.types[i];
    const bool tok = ti >= 0 && ti < S;
    const float4 *p4b = a.p4 + b;   // this lane's bead of every atom
    const uint32_t pstride = (uint32_t)P * sizeof(float4);
    const uint64_t bit = 1ull << b;
    const float4 pi = *row_at(p4b, i, pstride);
    const float *shc = prm + a.osh;
    float U = 0.0f;

    constexpr int DP = (D + 3) & ~3;
    if constexpr (NL) {
        const int nw = S * a.H * DP, nb = S * a.H;
        for (int x = threadIdx.x; x < nw; x += blockDim.x) {
            const int row = x / DP, v = x - row * DP;
            dyn[x] = v < D ? prm[a.oW0 + row * D + v] : 0.0f;
        }
        for (int x = threadIdx.x; x < nb; x += blockDim.x) {
            dyn[nw + x] = prm[a.ob0 + x];
            dyn[nw + nb + x] = prm[a.ow1 + x];
        }
        __syncthreads();
    }

    uint64_t todo = __ballot(valid && tok);
    while (todo) {
        const int lead = __builtin_ctzll(todo);
        const int tc = __builtin_amdgcn_readlane(ti, lead);
        const bool mine = valid && tok && ti == tc;
        todo &= ~__ballot(mine);
        if constexpr (!MF) {
            if (!mine) continue;
        }

        float q[D];
#pragma unroll
        for (int v = 0; v < D; ++v) q[v] = 0.0f;
        // the wavefront's adjoint rows, interleaved (adj_rows): each float4
        // store or load of the wavefront covers 1 KiB contiguously
        const __amdgpu_buffer_rsrc_t Bo = adj_rows(a.B, NA1 * (kNumSH / 4), threadIdx.x, blockDim.x);
        // A stays in registers through the network for small angular sets;
        // otherwise it is parked in the lane's adjoint row, where the
        // angular force kernel reads it
        constexpr bool PARK = adj_parked(MF, NA1);
        float Ar[PARK ? 1 : NA1][kNumSH];
        if (MF ? mine : true) {

        // radial: per neighbour species, sum the basis, then contract with c
        const int32_t *uR = a.uniR + (size_t)i * a.capR;
        const uint64_t *mR = a.umR + (size_t)i * a.capR;
        for (int t = 0; t < S; ++t) {
            int s0, s1;
            block_range(a.uendR, i, t, s0, s1);
            float sk[KR1];
#pragma unroll
            for (int k = 0; k < KR1; ++k) sk[k] = 0.0f;
            for (int sb = s0; sb < s1; sb += kBatchR) {
                bool in[kBatchR];
                float4 pj[kBatchR];
                // every load unconditional (entries past the block end are
                // masked off) so that the batch's loads are in flight together
                const idx_run<kBatchR> jj = *reinterpret_cast<const idx_run<kBatchR> *>(uR + sb);
                const mask_run<kBatchR> mm = *reinterpret_cast<const mask_run<kBatchR> *>(mR + sb);
#pragma unroll
                for (int u = 0; u < kBatchR; ++u) in[u] = (sb + u < s1) & ((mm.v[u] & bit) != 0);
#pragma unroll
                for (int u = 0; u < kBatchR; ++u) pj[u] = *row_at(p4b, jj.v[u], pstride);
#pragma unroll
                for (int u = 0; u < kBatchR; ++u) keep(pj[u]);
#pragma unroll
                for (int u = 0; u < kBatchR; ++u) {
                    if (in[u]) {
                        float dx, dy, dz;
                        pair_vec<FORM>(pj[u], pi, lm, dx, dy, dz);
                        const float r2 = norm2(dx, dy, dz);
                        {
                            // sk[0] collects f_c, sk[k > 0] collects f_c T_k
                            const float r = __builtin_amdgcn_sqrtf(r2);
                            float fc, T[KR1];
                            cheb_t<KR1>(r, a.rcRinv, fc, T);
                            sk[0] += fc;
#pragma unroll
                            for (int q2 = 1; q2 < KR1; ++q2) sk[q2] = fmaf(fc, T[q2], sk[q2]);
                        }
                    }
                }
            }
            // sum_j f_k = (sum f_c T_k + sum f_c) / 2 for k > 0, sum f_c for k = 0
#pragma unroll
            for (int q2 = 1; q2 < KR1; ++q2) sk[q2] = 0.5f * (sk[q2] + sk[0]);
            const float *c = prm + a.oR + (tc * S + t) * NR1 * KR1;
#pragma unroll
            for (int n = 0; n < NR1; ++n) {
                float acc = q[n];
#pragma unroll
                for (int q2 = 0; q2 < KR1; ++q2) acc += c[n * KR1 + q2] * sk[q2];
                q[n] = acc;
            }
        }

        // angular: A_nlm = sum_j g_n(r_ij) Y_lm(u_ij), NG radial functions n
        // per pass over the neighbours: all of them up to five; in two
        // passes when more are parked, each pass's q entries formed (keep:
        // formed later, they would hold the pass's A in scratch) and its A
        // parked before the next.  32000 atoms x 32 with nine functions:
        // 1107 us with three passes and 120 spilled registers, 982 without
        // the spills, 905 with two passes (120 sums, as many as five
        // functions keep); 13824 x 64 with seven, 461 -> 452 us.
        constexpr int NG = NA1 > 5 ? (NA1 + 1) / 2 : NA1;
        const int32_t *uW = a.uniW + (size_t)i * a.capA;
        const uint64_t *mA = a.umA + (size_t)i * a.capA;
#pragma unroll
        for (int n0 = 0; n0 < NA1; n0 += NG) {
        float A[NG][kNumSH];
#pragma unroll
        for (int g = 0; g < NG; ++g)
#pragma unroll
            for (int m = 0; m < kNumSH; ++m) A[g][m] = 0.0f;
        for (int t = 0; t < S; ++t) {
            int s0, s1;
            block_range(a.uendA, i, t, s0, s1);
            const float *c = prm + __builtin_amdgcn_readfirstlane(a.oA + (tc * S + t) * NA1 * KA1);   // uniform
            // g_n = f_c / 2 (cs_n + sum_{k>0} c_nk T_k), cs_n = c_n0 + sum_k c_nk
            float cs[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int n = n0 + g < NA1 ? n0 + g : NA1 - 1;
                float acc = c[n * KA1];
#pragma unroll
                for (int q2 = 0; q2 < KA1; ++q2) acc += c[n * KA1 + q2];
                cs[g] = acc;
            }
            // batches of kBatch entries: partners, then their positions,
            // each level's loads in flight together (entries past the block
            // end masked off)
            for (int sb = s0; sb < s1; sb += kBatch) {
                // coefficients through scalar loads, which do not wait on the gathers
                const cf32p cl = launder(c);
                bool in[kBatch];
                float4 pj[kBatch];
                const idx_run<kBatch> jj = *reinterpret_cast<const idx_run<kBatch> *>(uW + sb);
                const mask_run<kBatch> mm = *reinterpret_cast<const mask_run<kBatch> *>(mA + sb);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) in[u] = (sb + u < s1) & ((mm.v[u] & bit) != 0);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) pj[u] = *row_at(p4b, jj.v[u] >> 2, pstride);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) keep(pj[u]);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if (!in[u]) continue;
                    float dx, dy, dz;
                    pair_vec<FORM>(pj[u], pi, lm, dx, dy, dz);
                    const float r2 = norm2(dx, dy, dz);
                    const float rinv = __builtin_amdgcn_rsqf(r2);
                    const float r = r2 * rinv;
                    float fc, T[KA1];
                    cheb_t<KA1>(r, a.rcAinv, fc, T);
                    const float hf = 0.5f * fc;
                    // bare polynomials: the normalisations c_m are applied to the sums below
                    float Y[kNumSH];
                    sh_eval(dx * rinv, dy * rinv, dz * rinv, UnitNorm{}, Y);
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        const int n = n0 + g;
                        if (n >= NA1) break;
                        float gn = cs[g];
#pragma unroll
                        for (int q2 = 1; q2 < KA1; ++q2) gn = fmaf(cl[n * KA1 + q2], T[q2], gn);
                        gn *= hf;
#pragma unroll
                        for (int m = 0; m < kNumSH; ++m) A[g][m] += gn * Y[m];
                    }
                }
            }
        }
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            const int n = n0 + g;
            if (n >= NA1) break;
#pragma unroll
            for (int m = 0; m < kNumSH; ++m) A[g][m] *= shc[m];   // A_nlm = c_m sum_j g_n p_m
#pragma unroll
            for (int l = 1; l <= kLmax; ++l) {
                float s2 = 0.0f;
#pragma unroll
                for (int m = 0; m < kNumSH; ++m)
                    if (sh_l(m) == l) s2 = fmaf(A[g][m], A[g][m], s2);
                q[NR1 + (l - 1) * NA1 + n] = s2;
                if constexpr (PARK) keep(q[NR1 + (l - 1) * NA1 + n]);
            }
            if (FOUR) {
                q[NR1 + kLmax * NA1 + n] = a.kappa4 * four_body_tr3(&A[g][3], shc);
                if constexpr (PARK) keep(q[NR1 + kLmax * NA1 + n]);
            }
            if constexpr (PARK) {
                // park A in this lane's adjoint row (the angular force kernel forms B from it)
#pragma unroll
                for (int q4 = 0; q4 < kNumSH / 4; ++q4)
                    adj_store(Bo, n * (kNumSH / 4) + q4,
                              make_float4(A[g][4 * q4], A[g][4 * q4 + 1], A[g][4 * q4 + 2], A[g][4 * q4 + 3]));
            } else {
#pragma unroll
                for (int m = 0; m < kNumSH; ++m) Ar[PARK ? 0 : n][m] = A[g][m];
            }
        }
        }   // angular passes
        }   // descriptors of the lanes of species tc

        // network: U = sum_mu w1 tanh(sum_nu W0 s_nu q_nu - b0) - b1;  G_nu = dU/dq_nu
        const float *qs = prm + a.oq;
        float qh[D], G[D];
#pragma unroll
        for (int v = 0; v < D; ++v) {
            qh[v] = qs[v] * q[v];
            G[v] = 0.0f;
        }
        if constexpr (MF) {
            constexpr int WT = NET == kNetMf32 ? 3 : 1;
            const float *b0 = prm + a.ob0 + tc * a.H;
            const float *w1 = prm + a.ow1 + tc * a.H;
            float *X = dyn + (threadIdx.x >> 6) * mf_lds_floats<D>();
            const MlpFrag fl = mlp_frag_layout(D, a.H, WT);
            const float u = mlp_mf<D, WT>(qh, mine, a.w0b + (size_t)tc * fl.species_stride, b0, w1, prm[a.ob1],
                                          a.H, X, G);
            if (mine) U = u;
        } else if constexpr (NL) {
            const int nw = S * a.H * DP, nb = S * a.H;
            const float *W0 = dyn + tc * a.H * DP;
            const float *b0 = dyn + nw + tc * a.H;
            const float *w1 = dyn + nw + nb + tc * a.H;
            float u = -prm[a.ob1];
            if constexpr (D <= kNetRowRegs) {
                for (int mu = 0; mu < a.H; ++mu) {
                    // the weight row in registers, read from LDS once for both products
                    const float4 *w4 = reinterpret_cast<const float4 *>(W0 + mu * DP);
                    float wr[DP];
#pragma unroll
                    for (int v4 = 0; v4 < DP / 4; ++v4) {
                        const float4 t4 = w4[v4];
                        wr[4 * v4] = t4.x; wr[4 * v4 + 1] = t4.y; wr[4 * v4 + 2] = t4.z; wr[4 * v4 + 3] = t4.w;
                    }
                    float z = -b0[mu];
#pragma unroll
                    for (int v = 0; v < D; ++v) z += wr[v] * qh[v];
                    float h, dh;
                    tanh_and_slope(z, h, dh);
                    u += w1[mu] * h;
                    const float gz = w1[mu] * dh;
#pragma unroll
                    for (int v = 0; v < D; ++v) G[v] += gz * wr[v];
                }
            } else {
                // long rows: read from LDS in 4-wide chunks for each product
                // (broadcast reads), so the row takes no registers; one hidden
                // unit per iteration (unrolling interleaves rows and spills)
#pragma unroll 1
                for (int mu = 0; mu < a.H; ++mu) {
                    const float4 *w4 = reinterpret_cast<const float4 *>(W0 + mu * DP);
                    float z = -b0[mu];
#pragma unroll
                    for (int v4 = 0; v4 < DP / 4; ++v4) {
                        const float4 t4 = w4[v4];
                        const float wq[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (4 * v4 + e < D) z += wq[e] * qh[4 * v4 + e < D ? 4 * v4 + e : 0];
                    }
                    float h, dh;
                    tanh_and_slope(z, h, dh);
                    u += w1[mu] * h;
                    const float gz = w1[mu] * dh;
#pragma unroll
                    for (int v4 = 0; v4 < DP / 4; ++v4) {
                        const float4 t4 = w4[v4];
                        const float wq[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (4 * v4 + e < D) G[4 * v4 + e < D ? 4 * v4 + e : 0] += gz * wq[e];
                    }
                }
            }
            U = u;
        } else {
            const float *W0 = prm + a.oW0 + tc * a.H * D;
            const float *b0 = prm + a.ob0 + tc * a.H;
            const float *w1 = prm + a.ow1 + tc * a.H;
            float u = -prm[a.ob1];
            for (int mu = 0; mu < a.H; ++mu) {
                float z = -b0[mu];
#pragma unroll
                for (int v = 0; v < D; ++v) z += W0[mu * D + v] * qh[v];
                float h, dh;
                tanh_and_slope(z, h, dh);
                u += w1[mu] * h;
                const float gz = w1[mu] * dh;
#pragma unroll
                for (int v = 0; v < D; ++v) G[v] += gz * W0[mu * D + v];
            }
            U = u;
        }
#pragma unroll
        for (int v = 0; v < D; ++v) G[v] *= qs[v];
        if (MF ? !mine : false) continue;

        // adjoints: B_nlm = dU/dA_nlm, formed here from the sums in
        // registers, or, with the sums parked in the adjoint rows, by the
        // angular force kernel from them and the descriptor adjoints stored
        // here (no read-back of the parked sums)
        if constexpr (PARK) {
            const __amdgpu_buffer_rsrc_t go = adj_rows(a.Gad, gad_q(NA1, FOUR), threadIdx.x, blockDim.x);
#pragma unroll
            for (int n = 0; n < NA1; ++n)
                adj_store(go, n, make_float4(G[NR1 + n], G[NR1 + NA1 + n], G[NR1 + 2 * NA1 + n], G[NR1 + 3 * NA1 + n]));
            if constexpr (FOUR) {
#pragma unroll
                for (int c4 = 0; c4 < (NA1 + 3) / 4; ++c4) {
                    float g4[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int n = 4 * c4 + e;
                        g4[e] = n < NA1 ? G[NR1 + kLmax * NA1 + (n < NA1 ? n : 0)] * a.kappa4 : 0.0f;
                    }
                    adj_store(go, NA1 + c4, make_float4(g4[0], g4[1], g4[2], g4[3]));
                }
            }
        } else {
#pragma unroll
            for (int n = 0; n < NA1; ++n) {
                const float Gl[kLmax] = {G[NR1 + n], G[NR1 + NA1 + n], G[NR1 + 2 * NA1 + n], G[NR1 + 3 * NA1 + n]};
                const float g4 = FOUR ? G[NR1 + kLmax * NA1 + n] * a.kappa4 : 0.0f;
                float Bn[kNumSH];
                form_adjoint<FOUR>(Ar[PARK ? 0 : n], Gl, g4, shc, Bn);
#pragma unroll
                for (int q4 = 0; q4 < kNumSH / 4; ++q4)
                    adj_store(Bo, n * (kNumSH / 4) + q4,
                              make_float4(Bn[4 * q4], Bn[4 * q4 + 1], Bn[4 * q4 + 2], Bn[4 * q4 + 3]));
            }
        }
        // radial adjoints a_k(t) = sum_n G_n c^{tc t}_nk, [atom][species][bead][12],
        // and in slot KR1 their sum over k >= 1 (the pair terms need it)
        static_assert(KR1 < kRadPad, "radial basis exceeds the padded adjoint row");
        for (int t = 0; t < S; ++t) {
            const float *c = prm + a.oR + (tc * S + t) * NR1 * KR1;
            float acc[kRadPad];
#pragma unroll
            for (int k = 0; k < kRadPad; ++k) {
                acc[k] = 0.0f;
                if (k < KR1) {
#pragma unroll
                    for (int n = 0; n < NR1; ++n) acc[k] += G[n] * c[n * KR1 + k];
                }
            }
#pragma unroll
            for (int k = 1; k < KR1; ++k) acc[KR1] += acc[k];
            float4 *ao = reinterpret_cast<float4 *>(a.arad + (((size_t)i * S + t) * P + b) * kRadPad);
#pragma unroll
            for (int q4 = 0; q4 < kRadPad / 4; ++q4)
                ao[q4] = make_float4(acc[4 * q4], acc[4 * q4 + 1], acc[4 * q4 + 2], acc[4 * q4 + 3]);
        }
    }

    if (valid && a.Eatom) a.Eatom[(size_t)b * a.N + i] = U;
    if (valid && !tok) atomicOr(a.flags, (uint32_t)NEP_FLAG_BAD_TYPE);
    __shared__ SumLds<1> lds;
    // partials bead-major, [P][workgroups]: the reduction reads them contiguously
    const float Us[1] = {U};
    bead_block_sums(Us, valid, lds, P, a.lg, a.partE + blockIdx.x, 0, gridDim.x, blockDim.x >> 6);
}

// ------------------------------------------------ pass 2: angular, own ---

// One lane per (atom i, bead): the angular pair terms d_ij = dU_i/dr_ij of
// the atom's own site energy, contracted with its own adjoints only:
//   d_ij = sum_n sum_lm B^i_nlm d/dr_ij [ g^{ij}_n(r) Y_lm(u) ],
// deposited where the partner j reads it back (its angular slot of i, same
// bead), and summed into the angular force part F_i += d_ij and the virial
// -r_ij (x) d_ij (the total needs no reverse terms).  B^i stays in
// registers for the whole neighbour walk; with more than five radial
// functions that takes the register file of one wavefront per SIMD
// (VGPRs and AGPRs): re-reading the row per neighbour instead streamed it
// from memory, the rows of a CU's wavefronts being larger than its caches.
// Control flow stays wave-uniform: lanes outside the current centre species,
// past their atom's last candidate or outside the cutoff compute on a dummy
// pair and contribute nothing; a candidate outside for every lane is
// skipped.
// How a row's own angular sums are taken: over the whole list, in two parts
// one after the other (systems of up to kTwoPartRows rows among the launch's),
// or in two parts by two lanes, in launches of up to kSplitWaves wavefronts,
// which leave each SIMD's place for a second one empty (all their systems are
// that small).  2048 atoms x 32 beads with five functions, whole call: 172 us
// by one lane, 161 by two; training on 8 x 256 atoms x 32, 606 and 596.  At
// twice the rows two lanes cost more than they give, the adjoint rows being
// read twice: 4096 x 32, 214 and 255 us.  In two parts by one lane the water
// boxes take 1478 us, as a whole 1470.
constexpr int kSumWhole = 0, kSumParts = 1, kSumLanes = 2;
constexpr int kSplitWaves = kTwoPartRows / 64;

// Wavefronts per SIMD of k_force_ang.
template <int NA1> constexpr int kAngWaves() { return NA1 > 5 ? 1 : 2; }
constexpr int kBatchRev = 8;   // reverse angular terms read together by the radial force kernel

template <int NA1, int KA1, bool FOUR, bool PARKED, int FORM, int SUM>
__global__ __launch_bounds__(SUM == kSumLanes ? 2 * kBlock : kBlock) __attribute__((amdgpu_waves_per_eu(kAngWaves<NA1>())))
void k_force_ang(NepArgs a, const float *__restrict__ prm)
{
    // this lane's row (thread of the descriptor's workgroup), and the part of
    // the list it takes with two lanes per row
    constexpr bool SPLIT = SUM == kSumLanes;
    const int thread = SPLIT ? (threadIdx.x >> 6) * 32 + (threadIdx.x & 31) : threadIdx.x;
    const int threads = SPLIT ? blockDim.x >> 1 : blockDim.x;
    const int part = SPLIT ? (threadIdx.x >> 5) & 1 : 0;
    const LaneMap lm = lane_map(a, thread);
    const int i = lm.i, b = lm.b, P = a.P, S = a.S;
    const bool valid = lm.valid;
    const int ti = a.types[i];
    const bool tok = ti >= 0 && ti < S;
    const float4 *p4b = a.p4 + b;
    const uint32_t pstride = (uint32_t)P * sizeof(float4);
    const uint64_t bit = 1ull << b;
    float4 *pairb = a.pairbuf + b;
    const float4 pi = *row_at(p4b, i, pstride);
    const float *shc = prm + a.osh;
    const int32_t *uW = a.uniW + (size_t)i * a.capA, *uV = a.uniV + (size_t)i * a.capA;
    const uint64_t *mA = a.umA + (size_t)i * a.capA;
    float Fx = 0.0f, Fy = 0.0f, Fz = 0.0f;
    float Wv[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) Wv[e] = 0.0f;
    __shared__ float first[SUM ? 12 : 1][SUM ? kBlock : 1];   // the first part's sums of each row
    bool parts = SPLIT;
    if constexpr (SUM == kSumParts) {
        const int sy = a.tile_sys[blockIdx.x];
        const int n = a.tile_atom1[a.sys_tile0[sy + 1] - 1] - a.tile_atom0[a.sys_tile0[sy]];
        parts = (int64_t)n * P <= kTwoPartRows;
    }
    __shared__ SumLds<9> lds;
    bool second = false;   // in the second part

    uint64_t todo = __ballot(valid && tok);
    while (todo) {
        const int lead = __builtin_ctzll(todo);
        const int tc = __builtin_amdgcn_readlane(ti, lead);
        const bool mine = valid && tok && ti == tc;
        todo &= ~__ballot(mine);

        // B^i from the adjoint rows, or formed from the parked sums A^i and
        // the descriptor adjoints (see the descriptor kernel): their loads
        // are issued after the first neighbour batch's, so that the wait for
        // them overlaps that batch's gathers
        float Bi[NA1][kNumSH];
        bool formed = false;   // wave-uniform
        auto get_adjoints = [&]() {
            const __amdgpu_buffer_rsrc_t bi4 = adj_rows(a.B, NA1 * (kNumSH / 4), thread, threads);
#pragma unroll
            for (int n = 0; n < NA1; ++n)
#pragma unroll
                for (int q4 = 0; q4 < kNumSH / 4; ++q4) {
                    const float4 v4 = adj_load(bi4, n * (kNumSH / 4) + q4, thread);
                    Bi[n][4 * q4] = v4.x; Bi[n][4 * q4 + 1] = v4.y;
                    Bi[n][4 * q4 + 2] = v4.z; Bi[n][4 * q4 + 3] = v4.w;
                }
            if constexpr (PARKED) {
                const __amdgpu_buffer_rsrc_t gi = adj_rows(a.Gad, gad_q(NA1, FOUR), thread, threads);
                const float *shc = prm + a.osh;
#pragma unroll
                for (int n = 0; n < NA1; ++n) {
                    const float4 gl = adj_load(gi, n, thread);
                    const float Gl[kLmax] = {gl.x, gl.y, gl.z, gl.w};
                    float g4 = 0.0f;
                    if constexpr (FOUR) {
                        const float4 q = adj_load(gi, NA1 + n / 4, thread);
                        g4 = (n & 3) == 0 ? q.x : (n & 3) == 1 ? q.y : (n & 3) == 2 ? q.z : q.w;
                    }
                    form_adjoint<FOUR>(Bi[n], Gl, g4, shc, Bi[n]);
                }
            }
            formed = true;
        };
        for (int t = 0; t < S; ++t) {
            int s0 = 0, s1 = 0, hp = 0;
            if (mine) {
                block_range(a.uendA, i, t, s0, s1);
                if (SUM) hp = half_point(a.uendA[(size_t)i * kMaxSpecies + S - 1]);
            }
            int cnt = s1 - s0;
            // where the second part begins in this block (-1: not here)
            int mid = -1;
            if constexpr (SUM != kSumWhole) mid = split_batches(s0, s1, hp) * kBatchAng;
            if constexpr (SPLIT) {   // this lane's part of the block
                s0 += part ? mid : 0;
                cnt = part ? cnt - mid : min(cnt, mid);
            } else if (!parts || second || mid >= cnt) {
                mid = -1;
            }
            int cmax = cnt;
            for (int o = 32; o > 0; o >>= 1) cmax = max(cmax, __shfl_xor(cmax, o));
            cmax = __builtin_amdgcn_readfirstlane(cmax);
            const float *cij = prm + a.oA + (tc * S + t) * NA1 * KA1;
            for (int sb = 0; sb < cmax; sb += kBatchAng) {
                // the batch's partners, reverse slots and positions, each
                // level's loads in flight together (a lane past the end
                // of its block reads entries that are valid but masked off;
                // its position stays below the longest block of the
                // wavefront, which the arrays' slack covers)
                bool aq[kBatchAng];
                float4 pq[kBatchAng];
                const idx_run<kBatchAng> jq = *reinterpret_cast<const idx_run<kBatchAng> *>(uW + s0 + sb);
                const idx_run<kBatchAng> rq = *reinterpret_cast<const idx_run<kBatchAng> *>(uV + s0 + sb);
                const mask_run<kBatchAng> mm = *reinterpret_cast<const mask_run<kBatchAng> *>(mA + s0 + sb);
#pragma unroll
                for (int u = 0; u < kBatchAng; ++u) aq[u] = (sb + u < cnt) & ((mm.v[u] & bit) != 0);
#pragma unroll
                for (int u = 0; u < kBatchAng; ++u) pq[u] = *row_at(p4b, jq.v[u] >> 2, pstride);
                if constexpr (SUM == kSumParts) {
                    if (sb == mid) {   // the first part ends here
                        second = true;
                        first[0][threadIdx.x] = Fx;
                        first[1][threadIdx.x] = Fy;
                        first[2][threadIdx.x] = Fz;
                        Fx = Fy = Fz = 0.0f;
#pragma unroll
                        for (int e = 0; e < 9; ++e) {
                            first[3 + e][threadIdx.x] = Wv[e];
                            Wv[e] = 0.0f;
                        }
                    }
                }
                if (!formed) get_adjoints();
#pragma unroll
                for (int u = 0; u < kBatchAng; ++u) keep(pq[u]);
#pragma unroll
                for (int u = 0; u < kBatchAng; ++u) {
                const cf32p cij_l = launder(cij);
                const int j = jq.v[u] >> 2;
                const bool act = aq[u];
                if (__ballot(act) == 0) continue;
                float dx, dy, dz;
                pair_vec<FORM>(pq[u], pi, lm, dx, dy, dz);
                if (!act) {
                    dx = 1.0f;
                    dy = 0.0f;
                    dz = 0.0f;
                }
                const float r2 = norm2(dx, dy, dz);
                const float rinv = __builtin_amdgcn_rsqf(r2);
                const float r = r2 * rinv;
                const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
                float gij[NA1], gpij[NA1];
                {
                    // g = f_c Pn / 2, g' = (dx/dr f_c Qn + f_c' Pn) / 2 with
                    // Pn = sum_k c_nk (T_k + 1), Qn = sum_k c_nk T_k'
                    float fc, fcp, dxdr, T[KA1], Tp[KA1];
                    cheb_td<KA1>(r, a.rcAinv, fc, fcp, dxdr, T, Tp);
                    const float hf = 0.5f * fc, hfp = 0.5f * fcp, hd = hf * dxdr;
#pragma unroll
                    for (int n = 0; n < NA1; ++n) {
                        float pn = 2.0f * cij_l[n * KA1], qn = 0.0f;
#pragma unroll
                        for (int q2 = 1; q2 < KA1; ++q2) {
                            pn = fmaf(cij_l[n * KA1 + q2], T[q2] + 1.0f, pn);
                            qn = fmaf(cij_l[n * KA1 + q2], Tp[q2], qn);
                        }
                        gij[n] = hf * pn;
                        gpij[n] = fmaf(hd, qn, hfp * pn);
                    }
                }
                float sY, gx, gy, gz;
                // B^i is stored as B_nlm c_m: bare polynomials here
                adjoint_contract<NA1>(ux, uy, uz, Bi, gij, gpij, sY, gx, gy, gz);
                float px, py, pz;
                pair_term(ux, uy, uz, rinv, sY, gx, gy, gz, px, py, pz);
                if (act) {
                    const int rk = rq.v[u];
                    if (rk >= 0)
                        *const_cast<float4 *>(row_at(row_at(pairb, j, (uint32_t)a.capA * pstride), rk, pstride)) =
                            make_float4(px, py, pz, 0.0f);
                    Fx += px; Fy += py; Fz += pz;
                    Wv[0] = fmaf(-dx, px, Wv[0]); Wv[1] = fmaf(-dx, py, Wv[1]); Wv[2] = fmaf(-dx, pz, Wv[2]);
                    Wv[3] = fmaf(-dy, px, Wv[3]); Wv[4] = fmaf(-dy, py, Wv[4]); Wv[5] = fmaf(-dy, pz, Wv[5]);
                    Wv[6] = fmaf(-dz, px, Wv[6]); Wv[7] = fmaf(-dz, py, Wv[7]); Wv[8] = fmaf(-dz, pz, Wv[8]);
                }
                }
            }
        }
    }

    // the two parts together
    if constexpr (SPLIT) {
        Fx += __shfl_xor(Fx, 32);
        Fy += __shfl_xor(Fy, 32);
        Fz += __shfl_xor(Fz, 32);
#pragma unroll
        for (int e = 0; e < 9; ++e) Wv[e] += __shfl_xor(Wv[e], 32);
    } else if (SUM == kSumParts && second) {
        Fx += first[0][threadIdx.x];
        Fy += first[1][threadIdx.x];
        Fz += first[2][threadIdx.x];
#pragma unroll
        for (int e = 0; e < 9; ++e) Wv[e] += first[3 + e][threadIdx.x];
    }
    if (valid && part == 0) {
        float *Fo = a.Fang + ((size_t)i * P + b) * 3;
        Fo[0] = Fx;
        Fo[1] = Fy;
        Fo[2] = Fz;
        if (a.Watom) {
            // own half of the per-atom split; the reverse half is added by the radial pass
            float *wo = a.Watom + ((size_t)b * a.N + i) * 9;
#pragma unroll
            for (int e = 0; e < 9; ++e) wo[e] = 0.5f * Wv[e];
        }
    }
    bool sum = valid;
    if constexpr (SPLIT) {   // back to the rows' own threads for the sums over atoms
        if (part == 0) {
#pragma unroll
            for (int e = 0; e < 9; ++e) first[e][thread] = valid ? Wv[e] : 0.0f;
        }
        __syncthreads();
        sum = (int)threadIdx.x < threads;
#pragma unroll
        for (int e = 0; e < 9; ++e) Wv[e] = first[e][sum ? threadIdx.x : 0];
    }
    bead_block_sums(Wv, sum, lds, P, a.lg, a.partWa + blockIdx.x, gridDim.x, 9 * gridDim.x, threads >> 6);
}

// ----------------------------------------- pass 3: radial + combination ---

// One lane per (atom i, bead): radial pair terms (a^i_k(tj) + a^j_k(ti))
// f'_k(r) u (both site energies at once, the partner's adjoints gathered
// bead-minor), then the reverse angular terms -dU_j/dr_ji that the angular
// pass deposited at this atom's slots, then the angular own part.  Force and
// per-atom virial sums are kept in FP64.
template <int KR1, int FORM>
__global__ __launch_bounds__(kBlock) void k_force_rad(NepArgs a)
{
    const LaneMap lm = lane_map(a, threadIdx.x);
    const int i = lm.i, b = lm.b, P = a.P, S = a.S;
    const bool valid = lm.valid;
    const int ti = a.types[i];
    const bool tok = ti >= 0 && ti < S;
    const float4 *p4b = a.p4 + b;
    const uint32_t pstride = (uint32_t)P * sizeof(float4);
    const uint64_t bit = 1ull << b;
    const float4 pi = *row_at(p4b, i, pstride);
    double Fx = 0.0, Fy = 0.0, Fz = 0.0;
    float Wf[9];   // radial pair virial of this (atom, bead), FP32 (a sum of like-signed terms)
#pragma unroll
    for (int e = 0; e < 9; ++e) Wf[e] = 0.0f;
    float Wa[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) Wa[e] = 0.0f;
    if (valid && tok) {
        // adjoint rows of this lane's bead: atom j's for species t at j * astride + t * P rows
        const float *ab = a.arad + (size_t)b * kRadPad;
        const uint32_t trow = (uint32_t)P * kRadPad * sizeof(float), astride = (uint32_t)S * trow;
        const float *abt = row_at(ab, ti, trow);
        auto load_a = [&](const float *row, float *out) {
            const float4 *p = reinterpret_cast<const float4 *>(row);
#pragma unroll
            for (int q4 = 0; q4 < kRadPad / 4; ++q4) {
                const float4 v = p[q4];
                if (4 * q4 <= KR1) out[4 * q4] = v.x;
                if (4 * q4 + 1 <= KR1) out[4 * q4 + 1] = v.y;
                if (4 * q4 + 2 <= KR1) out[4 * q4 + 2] = v.z;
                if (4 * q4 + 3 <= KR1) out[4 * q4 + 3] = v.w;
            }
        };
        const int32_t *uR = a.uniR + (size_t)i * a.capR;
        const uint64_t *mR = a.umR + (size_t)i * a.capR;
        for (int t = 0; t < S; ++t) {
            int s0, s1;
            block_range(a.uendR, i, t, s0, s1);
            float ai[KR1 + 1];   // a_k and, last, their sum over k >= 1
            load_a(row_at(row_at(ab, t, trow), i, astride), ai);
            for (int sb = s0; sb < s1; sb += kBatch) {
                bool in[kBatch];
                float4 pj[kBatch];
                float aj[kBatch][KR1 + 1];
                // unconditional loads, as in the descriptor's radial batches
                const idx_run<kBatch> jj = *reinterpret_cast<const idx_run<kBatch> *>(uR + sb);
                const mask_run<kBatch> mm = *reinterpret_cast<const mask_run<kBatch> *>(mR + sb);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) in[u] = (sb + u < s1) & ((mm.v[u] & bit) != 0);
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    pj[u] = *row_at(p4b, jj.v[u], pstride);
                    load_a(row_at(abt, jj.v[u], astride), aj[u]);
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) keep(pj[u]);
                float bx = 0.0f, by = 0.0f, bz = 0.0f;   // the batch's force, FP32, into the FP64 sum once
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    if (in[u]) {
                        float dx, dy, dz;
                        pair_vec<FORM>(pj[u], pi, lm, dx, dy, dz);
                        const float w = radial_pair_w<KR1>(norm2(dx, dy, dz), a.rcRinv, ai, aj[u]);
                        const float qx = w * dx, qy = w * dy, qz = w * dz;
                        bx = fmaf(w, dx, bx); by = fmaf(w, dy, by); bz = fmaf(w, dz, bz);
                        const float hx = -0.5f * dx, hy = -0.5f * dy, hz = -0.5f * dz;
                        // a central pair term: r (x) q is symmetric, six entries
                        Wf[0] = fmaf(hx, qx, Wf[0]); Wf[1] = fmaf(hx, qy, Wf[1]); Wf[2] = fmaf(hx, qz, Wf[2]);
                        Wf[4] = fmaf(hy, qy, Wf[4]); Wf[5] = fmaf(hy, qz, Wf[5]); Wf[8] = fmaf(hz, qz, Wf[8]);
                    }
                }
                Fx += (double)bx; Fy += (double)by; Fz += (double)bz;
            }
        }

        Wf[3] = Wf[1];
        Wf[6] = Wf[2];
        Wf[7] = Wf[5];

        // reverse angular terms: F_i -= dU_j/dr_ji for every angular neighbour j
        const int32_t *uA = a.uniA + (size_t)i * a.capA, *uW = a.uniW + (size_t)i * a.capA;
        const uint64_t *mA = a.umA + (size_t)i * a.capA;
        const float4 *pbuf = row_at(a.pairbuf + b, i, (uint32_t)a.capA * pstride);
        const int nA = a.uendA[(size_t)i * kMaxSpecies + S - 1];
        float gx = 0.0f, gy = 0.0f, gz = 0.0f;
        for (int sb = 0; sb < nA; sb += kBatchRev) {
            bool in[kBatchRev];
            float4 d[kBatchRev];
            // unconditional loads (values past the list end or outside the bead mask are dropped)
            const idx_run<kBatchRev> kk = *reinterpret_cast<const idx_run<kBatchRev> *>(uA + sb);
            const mask_run<kBatchRev> mm = *reinterpret_cast<const mask_run<kBatchRev> *>(mA + sb);
#pragma unroll
            for (int u = 0; u < kBatchRev; ++u) in[u] = (sb + u < nA) & ((mm.v[u] & bit) != 0);
#pragma unroll
            for (int u = 0; u < kBatchRev; ++u) d[u] = *row_at(pbuf, kk.v[u], pstride);
#pragma unroll
            for (int u = 0; u < kBatchRev; ++u) {
                keep(d[u]);
                if (!in[u]) d[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
#pragma unroll
            for (int u = 0; u < kBatchRev; ++u) {
                gx -= d[u].x; gy -= d[u].y; gz -= d[u].z;
            }
            if (a.Watom) {
#pragma unroll
                for (int u = 0; u < kBatchRev; ++u) {
                    if (!in[u]) continue;
                    float dx, dy, dz;
                    pair_vec<FORM>(*row_at(p4b, uW[sb + u] >> 2, pstride), pi, lm, dx, dy, dz);
                    const float4 dd = d[u];
                    // reverse half of the per-atom split: +1/2 r_ij (x) dU_j/dr_ji
                    const float hx = 0.5f * dx, hy = 0.5f * dy, hz = 0.5f * dz;
                    Wa[0] = fmaf(hx, dd.x, Wa[0]); Wa[1] = fmaf(hx, dd.y, Wa[1]); Wa[2] = fmaf(hx, dd.z, Wa[2]);
                    Wa[3] = fmaf(hy, dd.x, Wa[3]); Wa[4] = fmaf(hy, dd.y, Wa[4]); Wa[5] = fmaf(hy, dd.z, Wa[5]);
                    Wa[6] = fmaf(hz, dd.x, Wa[6]); Wa[7] = fmaf(hz, dd.y, Wa[7]); Wa[8] = fmaf(hz, dd.z, Wa[8]);
                }
            }
        }
        Fx += (double)gx;
        Fy += (double)gy;
        Fz += (double)gz;
    }
    if (valid) {
        const float *fa = a.Fang + ((size_t)i * P + b) * 3;
        const double gx = Fx + (double)fa[0], gy = Fy + (double)fa[1], gz = Fz + (double)fa[2];
        float *Fo = a.F + ((size_t)b * a.N + i) * 3;
        Fo[0] = (float)gx;
        Fo[1] = (float)gy;
        Fo[2] = (float)gz;
        if (a.Watom) {
            float *wo = a.Watom + ((size_t)b * a.N + i) * 9;
#pragma unroll
            for (int e = 0; e < 9; ++e) wo[e] = (float)((double)Wf[e] + (double)Wa[e] + (double)wo[e]);
        }
        if (!(isfinite(gx) && isfinite(gy) && isfinite(gz))) atomicOr(a.flags, (uint32_t)NEP_FLAG_NONFINITE);
    }
    __shared__ SumLds<9> lds;
    bead_block_sums(Wf, valid, lds, P, a.lg, a.partWr + blockIdx.x, gridDim.x, 9 * gridDim.x, blockDim.x >> 6);
}

// Per-(system, bead) energy and virial from the per-workgroup partial sums
// of the system's tiles, stored [P][nblk] (energy) and [P][9][nblk] (virial
// parts): one wavefront per (system, bead, component), in the fixed order of
// reduce_output.
__global__ __launch_bounds__(64) void k_reduce(PendingReduce r)
{
    reduce_output(r, blockIdx.x, threadIdx.x);
}

constexpr size_t kNetLdsMax = 60 * 1024;   // bytes of LDS for the staged network weights

// mlp: NEP_MLP_FP32 (vector units), NEP_MLP_BF16_MFMA or NEP_MLP_FP32_MFMA (matrix cores).
template <int NR1, int NA1, bool FOUR, int FORM>
static void launch_t(const NepArgs &a, const float *prm, int nblk, int wpb, int64_t min_rows, int mlp,
                     bool lds_net, hipStream_t s)
{
    const dim3 g(nblk);
    const dim3 blk(64 * wpb);
    {
        ProfScope ps_(K_DESCRIPTOR, s);
        constexpr int D = Dims<NR1, NA1, FOUR>::D, DP = (D + 3) & ~3;
        const size_t net = sizeof(float) * (size_t)a.S * a.H * (DP + 2);
        const size_t mf = sizeof(float) * (size_t)mf_lds_floats<D>() * wpb;
        if (mlp == NEP_MLP_BF16_MFMA)   // BF16 weights (the student)
            hipLaunchKernelGGL((k_descriptor<NR1, NA1, 9, 9, FOUR, kNetBf16, FORM>), g, blk, mf, s, a, prm);
        else if (mlp == NEP_MLP_FP32_MFMA)   // FP32 weights as three BF16 terms
            hipLaunchKernelGGL((k_descriptor<NR1, NA1, 9, 9, FOUR, kNetMf32, FORM>), g, blk, mf, s, a, prm);
        else if (lds_net && net <= kNetLdsMax)   // network weights staged in LDS
            hipLaunchKernelGGL((k_descriptor<NR1, NA1, 9, 9, FOUR, kNetLds, FORM>), g, blk, net, s, a, prm);
        else
            hipLaunchKernelGGL((k_descriptor<NR1, NA1, 9, 9, FOUR, kNetGlobal, FORM>), g, blk, 0, s, a, prm);
    }
    {
        ProfScope ps_(K_FORCE_ANG, s);
        const bool parked = adj_parked(mlp == NEP_MLP_BF16_MFMA || mlp == NEP_MLP_FP32_MFMA, NA1);
        if constexpr (adj_parked(false, NA1)) {   // wide sets are always parked
            hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, true, FORM, kSumWhole>), g, blk, 0, s, a, prm);
        } else if (two_parts(NA1, a.lg) && nblk * wpb <= kSplitWaves) {
            const dim3 b2(128 * wpb);
            if (parked) hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, true, FORM, kSumLanes>), g, b2, 0, s, a, prm);
            else hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, false, FORM, kSumLanes>), g, b2, 0, s, a, prm);
        } else if (two_parts(NA1, a.lg) && min_rows <= kTwoPartRows) {
            if (parked) hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, true, FORM, kSumParts>), g, blk, 0, s, a, prm);
            else hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, false, FORM, kSumParts>), g, blk, 0, s, a, prm);
        } else if (parked) {
            hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, true, FORM, kSumWhole>), g, blk, 0, s, a, prm);
        } else {
            hipLaunchKernelGGL((k_force_ang<NA1, 9, FOUR, false, FORM, kSumWhole>), g, blk, 0, s, a, prm);
        }
    }
    {
        ProfScope ps_(K_FORCE, s);
        hipLaunchKernelGGL((k_force_rad<9, FORM>), g, blk, 0, s, a);
    }
}

// form: the list's (what the launch carries code for).
template <int NR1, int NA1, bool FOUR>
static void launch(const NepArgs &a, const float *prm, int nblk, int wpb, int64_t min_rows, int form, int mlp,
                   bool lds_net, hipStream_t s)
{
    if (form == kPosFixed) launch_t<NR1, NA1, FOUR, kPosFixed>(a, prm, nblk, wpb, min_rows, mlp, lds_net, s);
    else if (form == kPosGrid) launch_t<NR1, NA1, FOUR, kPosGrid>(a, prm, nblk, wpb, min_rows, mlp, lds_net, s);
    else launch_t<NR1, NA1, FOUR, kPosAny>(a, prm, nblk, wpb, min_rows, mlp, lds_net, s);
}

}  // namespace nep

using namespace nep;

extern "C" int32_t nep_compute_batched(const nep_model *m, nep_nlist *nl, nep_ws *ws, const double *pos,
                                       const double *boxes, const int32_t *types, int32_t P, int32_t N, double *E,
                                       float *F, double *W, float *E_atom, float *W_atom, hipStream_t s)
{
    if (!m || !nl || !ws || !boxes) return fail(NEP_ERR_INVALID_ARG, "nep_compute: null argument");
    if (m->cutoffs_only) return fail(NEP_ERR_INVALID_ARG, "nep_compute: a list cutoff descriptor has no network");
    if (nl->P != P || nl->N != N || ws->P != P || ws->N != N || nl->S != m->hp.n_species || ws->S != m->hp.n_species ||
        ws->NA1 != m->hp.n_max_angular + 1 || nl->off != ws->off)
        return fail(NEP_ERR_INVALID_ARG, "nep_compute: P=%d N=%d do not match the list/workspace handles", P, N);
    // a deferral applies to this call only; a new call drops sums left pending
    const bool defer = ws->defer_next != 0;
    ws->defer_next = 0;
    ws->pending = PendingReduce{};
    if (P == 0) return NEP_OK;
    if (!E || !W) return fail(NEP_ERR_INVALID_ARG, "nep_compute: null E or W");
    const int nsys = nl->nsys;
    if (N == 0) {
        fill_u32(reinterpret_cast<uint32_t *>(E), 0u, (size_t)nsys * P * 2, s);
        fill_u32(reinterpret_cast<uint32_t *>(W), 0u, (size_t)nsys * P * 18, s);
        NEP_HIP(hipGetLastError());
        return NEP_OK;
    }
    if (!pos || !types || !F) return fail(NEP_ERR_INVALID_ARG, "nep_compute: null array");
    if (!nl->built) return fail(NEP_ERR_INVALID_ARG, "nep_compute: the neighbour lists were never built");
    if (nl->rc_built[0] != m->hp.rc_radial || nl->rc_built[1] != m->hp.rc_angular)
        return fail(NEP_ERR_INVALID_ARG, "nep_compute: the lists were built for cutoffs %g/%g, the model has %g/%g",
                    nl->rc_built[0], nl->rc_built[1], m->hp.rc_radial, m->hp.rc_angular);
    for (int sy = 0; sy < nsys; ++sy)
        for (int k = 0; k < 9; ++k)
            if (boxes[9 * sy + k] != nl->boxL[9 * sy + k])
                return fail(NEP_ERR_INVALID_ARG, "nep_compute: box of system %d differs from the last neighbor_build",
                            sy);
    const nep_hparams &h = m->hp;
    NepArgs a{};
    // packed positions of the last neighbor_build (the same positions, see the header)
    a.p4 = reinterpret_cast<const float4 *>(nl->pos4); a.types = types; a.N = N; a.S = h.n_species;
    a.H = h.hidden; a.P = P; a.lg = lanes_log2(P);
    a.geom = nl->geom; a.tile_atom0 = ws->tile_atom0; a.tile_atom1 = ws->tile_atom1; a.tile_sys = ws->tile_sys; a.sys_tile0 = ws->sys_tile0;
    a.rcRinv = (float)(1.0 / h.rc_radial); a.rcAinv = (float)(1.0 / h.rc_angular);
    a.kappa4 = (float)(-4.5 * std::sqrt(2.0 / 35.0) * std::pow(5.0 / (4.0 * M_PI), 1.5));
    a.uniR = nl->uniR; a.uendR = nl->uendR; a.uniA = nl->uniA;
    a.uniW = nl->uniW; a.uniV = nl->uniV;
    a.umR = nl->umR; a.umA = nl->umA;
    a.uendA = nl->uendA; a.capR = nl->capR; a.capA = nl->capA;
    a.pairbuf = reinterpret_cast<float4 *>(nl->pairbuf);
    a.B = ws->B; a.Gad = ws->Gad; a.arad = ws->arad; a.Fang = ws->Fang;
    a.partE = ws->partE; a.partWa = ws->partW; a.partWr = ws->partW + (size_t)P * ws->nblk * 9;
    a.flags = ws->flags;
    a.F = F; a.Eatom = E_atom; a.Watom = W_atom;
    a.oR = m->off.cR; a.oA = m->off.cA; a.oq = m->off.qs; a.oW0 = m->off.W0; a.ob0 = m->off.b0;
    a.ow1 = m->off.w1; a.ob1 = m->off.b1; a.osh = m->off.sh;
    a.w0b = m->w0b;
    const int mlp = m->mlp;
    PendingReduce r;
    r.sys_tile0 = ws->sys_tile0; r.P = P; r.nblk = ws->nblk; r.nout = nsys * P * 10; r.E = E; r.W = W;
    const bool small = ws->rowp && takes_small((int64_t)P * N, P, h, nl->capR + nl->capA, mlp);
    if (small) {   // one wavefront per (atom, bead)
        const int32_t rcs = launch_small(a, m, nl->atom_sys, ws->rowp, s);
        if (rcs != NEP_OK) return rcs;
        r.rowp = ws->rowp; r.tile_atom0 = ws->tile_atom0; r.tile_atom1 = ws->tile_atom1; r.N = N;
    } else {
        const int key = h.n_max_radial * 100 + h.n_max_angular * 10 + h.four_body;
        int64_t min_rows = INT64_MAX;   // the smallest (non-empty) system
        for (int sy = 0; sy < nsys; ++sy)
            if (ws->off[sy + 1] > ws->off[sy]) min_rows = std::min(min_rows, (int64_t)P * (ws->off[sy + 1] - ws->off[sy]));
        switch (key) {
        case 440: launch<5, 5, false>(a, m->dev, ws->nblk, ws->wpb, min_rows, nl->form, mlp, !ws->net_global, s); break;
        case 441: launch<5, 5, true>(a, m->dev, ws->nblk, ws->wpb, min_rows, nl->form, mlp, !ws->net_global, s); break;
        case 640: launch<7, 5, false>(a, m->dev, ws->nblk, ws->wpb, min_rows, nl->form, mlp, !ws->net_global, s); break;
        case 860: launch<9, 7, false>(a, m->dev, ws->nblk, ws->wpb, min_rows, nl->form, mlp, !ws->net_global, s); break;
        case 881: launch<9, 9, true>(a, m->dev, ws->nblk, ws->wpb, min_rows, nl->form, mlp, !ws->net_global, s); break;
        default: return fail(NEP_ERR_UNSUPPORTED, "nep_compute: unsupported model shape");
        }
        r.partE = ws->partE; r.partWa = a.partWa; r.partWr = a.partWr;
    }
    if (defer) {   // completed by the next integrator launch (trpmd_step_nep)
        ws->pending = r;
    } else {
        ProfScope ps_(K_REDUCE, s);
        hipLaunchKernelGGL(k_reduce, dim3(r.nout), dim3(64), 0, s, r);
    }
    NEP_HIP(hipGetLastError());
    return NEP_OK;
}

extern "C" int32_t nep_compute(const nep_model *m, nep_nlist *nl, nep_ws *ws, const double *pos,
                               const double box[9], const int32_t *types, int32_t P, int32_t N, double *E, float *F,
                               double *W, float *E_atom, float *W_atom, hipStream_t s)
{
    if (nl && nl->nsys != 1) return fail(NEP_ERR_INVALID_ARG, "nep_compute: the list holds a batch of systems");
    return nep_compute_batched(m, nl, ws, pos, box, types, P, N, E, F, W, E_atom, W_atom, s);
}

extern "C" int32_t nep_ws_defer_reduce(nep_ws *ws)
{
    if (!ws) return fail(NEP_ERR_INVALID_ARG, "nep_ws_defer_reduce: null workspace");
    ws->defer_next = 1;
    return NEP_OK;
}

extern "C" int32_t nep_autotune(const nep_model *m, nep_nlist *nl, nep_ws *ws, const double *pos, const double *boxes,
                                const int32_t *types, int32_t P, int32_t N, double *E, float *F, double *W,
                                int32_t reps, float *ms_out, int32_t *best_out, hipStream_t s)
{
    if (!m || !nl || !ws) return fail(NEP_ERR_INVALID_ARG, "nep_autotune: null argument");
    if (reps < 1 || reps > 100) return fail(NEP_ERR_INVALID_ARG, "nep_autotune: reps must be in 1..100");
    const int choices[3] = {1, 2, 4};
    // the staging knob exists for the vector-unit network whose weights fit LDS
    const nep_hparams &h = m->hp;
    const size_t net = sizeof(float) * (size_t)h.n_species * h.hidden * (((h.dim + 3) & ~3) + 2);
    const int nst = (m->mlp == NEP_MLP_FP32 && net <= kNetLdsMax) ? 2 : 1;
    float best_ms = 0.0f;
    int best = 4, best_st = NEP_WEIGHTS_LDS;
    if (ms_out)
        for (int k = 0; k < 6; ++k) ms_out[k] = -1.0f;
    hipEvent_t e0, e1;
    NEP_HIP(hipEventCreate(&e0));
    NEP_HIP(hipEventCreate(&e1));
    int32_t rc = NEP_OK;
    bool first = true;
    for (int c = 0; c < 3 && rc == NEP_OK; ++c)
        for (int st = 0; st < nst && rc == NEP_OK; ++st) {
            rc = nep_ws_set_tile(ws, choices[c]);
            if (rc == NEP_OK) rc = nep_ws_set_weight_staging(ws, st);
            if (rc != NEP_OK) break;
            rc = nep_compute_batched(m, nl, ws, pos, boxes, types, P, N, E, F, W, nullptr, nullptr, s);   // warm-up
            if (rc != NEP_OK) break;
            if (hipEventRecord(e0, s) != hipSuccess) rc = fail(NEP_ERR_HIP, "nep_autotune: event record failed");
            for (int r = 0; r < reps && rc == NEP_OK; ++r)
                rc = nep_compute_batched(m, nl, ws, pos, boxes, types, P, N, E, F, W, nullptr, nullptr, s);
            if (rc != NEP_OK) break;
            float ms = 0.0f;
            if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
                rc = fail(NEP_ERR_HIP, "nep_autotune: event timing failed");
                break;
            }
            ms /= (float)reps;
            if (ms_out) ms_out[2 * c + st] = ms;
            if (first || ms < best_ms) {
                best_ms = ms;
                best = choices[c];
                best_st = st;
                first = false;
            }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc != NEP_OK) return rc;
    if (best_out) {
        best_out[0] = best;
        best_out[1] = best_st;
    }
    rc = nep_ws_set_weight_staging(ws, best_st);
    return rc != NEP_OK ? rc : nep_ws_set_tile(ws, best);
}
