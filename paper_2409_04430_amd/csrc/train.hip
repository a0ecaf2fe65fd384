// Training of a NEP model on GPU: gradient of an energy / force / virial
// loss with respect to the network parameters (W0, b0, w1, b1) and the radial
// and angular descriptor coefficients c^R, c^A, and an Adam update (Kingma
// and Ba, ICLR 2015).
// The NEP site-energy model is that of Sec. II.C of arXiv:2409.04430; the
// paper fits its models by SNES, this library by gradients.
//
// For the P configurations of each system of one call (the beads of a
// neighbour handle, each with reference E, F, W; a batch of systems is a
// batch of independent snapshots) the loss is, summed over the systems,
//   L = sum_b [ lE (dE_b / N)^2 + lF sum_i |dF_bi|^2 / (3 N) + lW sum_ab (dW_b,ab / N)^2 ]
// with N the system's atom count.
// Force and virial terms are derivatives of E, so their parameter gradient
// is a mixed derivative.  With g_ij = dU_i/dr_ij and a per-pair field
//   d_ij = -(2 lF / 3N) (dF_j - dF_i) - (2 lW / N^2) dW_b^T r_ij
// one has dL_{F,W}/dtheta = d/dtheta sum_ij g_ij . d_ij  (d held fixed), and
// sum_ij g_ij . d_ij = sum_i G_i . qdot_i, G = dU/dq, qdot the derivative of
// the descriptor along d (a forward-mode pass).  The kernels therefore
// compute per (atom, bead): q, qdot, the network values and their forward
// derivatives, and write one row of factors; a reduction kernel forms the
// outer products that make up the gradient.
#include <algorithm>

#include "nep_net.hpp"

namespace nep {

struct TrainArgs {
    const float4 *dF;   // [N][P] scaled force residuals -2 lF/(3N) (F - F_ref), bead-minor
    const float *cW;    // [nsys][P][9] -2 lW/N^2 (W - W_ref)
    const float *eE;    // [nsys][P] 2 lE/N^2 (E - E_ref)
    float *rows;        // [N*P][RW] factor rows, row i * P + b (row[0] -1: species outside the model)
    int RW;
};

// Row layout (floats): type | u[H] | v[H] | gw1[H] | sq[D] | sqd[D] | gR[NR1] | GR[NR1] | sk[S][KR1] |
// skd[S][KR1] | eE | gA[S][NA1][KA1].
struct RowLayout {
    int u, v, gw1, sq, sqd, gR, GR, sk, skd, eE, gA, RW;
    __host__ __device__ RowLayout(int H, int D, int NR1, int S, int KR1, int NA1, int KA1)
    {
        u = 1; v = u + H; gw1 = v + H; sq = gw1 + H; sqd = sq + D; gR = sqd + D; GR = gR + NR1; sk = GR + NR1;
        skd = sk + S * KR1; eE = skd + S * KR1; gA = eE + 1; RW = gA + S * NA1 * KA1;
    }
};

// Residuals: scaled force residuals per (atom, bead) and per-(system, bead)
// energy and virial factors; the loss terms go out per workgroup (force) and
// per (system, bead) (energy, virial) in lossp and are added up by
// k_grad_final (same-address atomics of every workgroup serialised here:
// 17.5 us at 65,536 rows).  atom_sys [N] and sys_off [nsys+1] give each
// atom's system and the systems' atom counts.
__global__ __launch_bounds__(256) void k_residual(const float *__restrict__ F, const float *__restrict__ Fref,
                           const double *__restrict__ E,
                           const double *__restrict__ Eref, const double *__restrict__ W,
                           const double *__restrict__ Wref, int P, int N, int nsys,
                           const int32_t *__restrict__ atom_sys, const int32_t *__restrict__ sys_off, double lE,
                           double lF, double lW, float4 *__restrict__ dF, float *__restrict__ cW,
                           float *__restrict__ eE, double *__restrict__ lossp, int nfblk)
{
    if ((int)blockIdx.x >= nfblk) {   // energies and virials, one (system, bead) per lane
        const int x = ((int)blockIdx.x - nfblk) * 256 + threadIdx.x;
        if (x >= nsys * P) return;
        const int sy = x / P;
        const double Ns = (double)(sys_off[sy + 1] - sys_off[sy]);
        double le = 0.0, lw = 0.0;
        if (!(Ns > 0.0)) {
            eE[x] = 0.0f;
            for (int k = 0; k < 9; ++k) cW[9 * x + k] = 0.0f;
        } else {
            const double de = E[x] - Eref[x];
            eE[x] = (float)(2.0 * lE * de / (Ns * Ns));
            le = lE * (de / Ns) * (de / Ns);
            for (int k = 0; k < 9; ++k) {
                const double dw = W[9 * x + k] - Wref[9 * x + k];
                cW[9 * x + k] = (float)(-2.0 * lW * dw / (Ns * Ns));
                lw += lW * (dw / Ns) * (dw / Ns);
            }
        }
        lossp[nfblk + x] = le;
        lossp[nfblk + nsys * P + x] = lw;
        return;
    }
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    double lf = 0.0;
    if (e < (size_t)P * N) {
        const int b = (int)(e / (size_t)N), i = (int)(e - (size_t)b * N);
        const int sy = atom_sys[i];
        const double Ns = (double)(sys_off[sy + 1] - sys_off[sy]);
        const double dx = (double)F[3 * e] - Fref[3 * e], dy = (double)F[3 * e + 1] - Fref[3 * e + 1],
                     dz = (double)F[3 * e + 2] - Fref[3 * e + 2];
        lf = lF * (dx * dx + dy * dy + dz * dz) / (3.0 * Ns);
        const double cf = -2.0 * lF / (3.0 * Ns);
        dF[(size_t)i * P + b] = make_float4((float)(cf * dx), (float)(cf * dy), (float)(cf * dz), 0.0f);
    }
    __shared__ double red[4];
    lf = wave_sum(lf);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lf;
    __syncthreads();
    if (threadIdx.x == 0) lossp[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// One (atom, bead) per wavefront, its lanes the neighbours (owner lanes add
// the staged contributions in list order, as in nep_small.hip): descriptor q
// and its derivative along the pair field d, the network with its forward
// derivative, and the factor row of (atom, bead).
//
// Angular coefficients: with T_klm = sum_j f_k(r_ij) Y_lm(u_ij) (per
// neighbour species), A_nlm = sum_k c_nk T_klm and q_nl = sum_m A_nlm^2, the
// row's share of dL/dc_nk is sum_lm [X_nlm T_klm + B_nlm Tdot_klm] with
// B = 2 G_nl A_nlm (the energy adjoint), X = eE B + Bdot and Bdot = 2 (Gdot_nl
// A_nlm + G_nl Adot_nlm): per neighbour al_n = X.Y + B.Ydot and
// be_n = (u.d) B.Y, then sum_j al_n f_k + be_n f_k'.
//
// A lane per row instead walked the angular neighbours once for every two
// radial functions and once more for every coefficient row: 560 us for eight
// 256-atom snapshots of 32 beads (65,536 rows, one wavefront per SIMD) and as
// long for a single small snapshot; this kernel took 417 us there (three
// wavefronts per SIMD; at two 476), 375 since pair vectors are FP64 products,
// and falls with the rows.  The sums as 16 x 16 x 4 FP32 matrix-core tiles
// (mostly padding at 5 functions and 24 harmonics) measured slower, 427 us
// against the 417.
constexpr int kRowStage = 32;   // neighbours staged at a time (LDS)
template <int NR1, int NA1>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3)))
void k_train_row(NepArgs a, TrainArgs ta, const float *__restrict__ prm, const int32_t *__restrict__ atom_sys)
{
    constexpr int KR1 = 9, KA1 = 9, D = Dims<NR1, NA1, false>::D;
    constexpr int NACC = (NA1 * kNumSH + 63) / 64;
    constexpr int HP = 2 * kNumSH + 1, GP = 2 * NA1 + 1, RP = 2 * KR1 + 1;   // odd row strides
    extern __shared__ float dyn[];   // per hidden unit: u, udot
    __shared__ float sh[kRowStage * HP > 64 * RP ? kRowStage * HP : 64 * RP];   // Y, Ydot (then f, f'); radial staging before
    __shared__ float sg[kRowStage * GP];   // g, gdot; then al, be
    __shared__ float ssk[2 * 64];
    __shared__ float sq[D], sqd[D], sG[D], sGd[D];
    __shared__ float sA[NA1][kNumSH], sB[NA1][kNumSH];   // A, Adot, then X, B
    __shared__ float sc[kMaxSpecies * NA1 * KA1];

    const int P = a.P, S = a.S, H = a.H, lane = threadIdx.x;
    const int i = blockIdx.x / P, b = blockIdx.x - i * P;
    const RowLayout R(H, D, NR1, S, KR1, NA1, KA1);
    float *row = ta.rows + (size_t)blockIdx.x * ta.RW;
    const int ti = a.types[i];
    if (ti < 0 || ti >= S) {   // whole wavefront: a row outside every species
        if (lane == 0) row[0] = __int_as_float(-1);
        return;
    }
    const int sy = atom_sys[i];
    const LaneMap lm = row_map(a.geom[sy], i, b);
    const float4 *p4b = a.p4 + b, *dFb = ta.dF + b;
    const uint32_t pstride = (uint32_t)P * sizeof(float4);
    const float4 pi = *row_at(p4b, i, pstride), di = *row_at(dFb, i, pstride);
    const int sb = sy * P + b;   // (system, bead)
    float cw[9];
#pragma unroll
    for (int e = 0; e < 9; ++e) cw[e] = ta.cW[9 * sb + e];
    const float eEb = ta.eE[sb];
    const float *shc = prm + a.osh;
    const float *qs = prm + a.oq;
    // pair field along r_ij: d = (dF_j - dF_i) + cW^T r_ij
    auto field = [&](const float4 &dj, float dx, float dy, float dz, float &ex, float &ey, float &ez) {
        ex = dj.x - di.x + cw[0] * dx + cw[3] * dy + cw[6] * dz;
        ey = dj.y - di.y + cw[1] * dx + cw[4] * dy + cw[7] * dz;
        ez = dj.z - di.z + cw[2] * dx + cw[5] * dy + cw[8] * dz;
    };
    const int32_t *uendR = a.uendR + (size_t)i * kMaxSpecies, *uendA = a.uendA + (size_t)i * kMaxSpecies;

    // ---- radial basis sums and their derivatives: lane (group, species t,
    // k) adds every ng-th entry of block t, then the groups are added
    const int nk = S * KR1, ng = 64 / nk;
    const int gr = lane / nk, ok = lane - gr * nk, to = ok / KR1, ko = ok - to * KR1;
    {
        const int32_t *uR = a.uniR + (size_t)i * a.capR;
        const uint64_t *mR = a.umR + (size_t)i * a.capR;
        const int n = uendR[S - 1];
        const int o0 = to ? uendR[to - 1] : 0, o1 = gr < ng ? uendR[to] : 0;
        float s = 0.0f, sd = 0.0f;
        for (int p0 = 0; p0 < n; p0 += 64) {
            const int e = p0 + lane;
            float f[KR1], fd[KR1];
#pragma unroll
            for (int k = 0; k < KR1; ++k) {
                f[k] = 0.0f;
                fd[k] = 0.0f;
            }
            if (e < n && ((mR[e] >> b) & 1u)) {
                const int j = uR[e];
                const float4 dj = *row_at(dFb, j, pstride);
                float dx, dy, dz, ex, ey, ez;
                pair_vec<kPosAny>(*row_at(p4b, j, pstride), pi, lm, dx, dy, dz);
                const float r2 = norm2(dx, dy, dz);
                const float rinv = __builtin_amdgcn_rsqf(r2);
                field(dj, dx, dy, dz, ex, ey, ez);
                const float rdot = (dx * ex + dy * ey + dz * ez) * rinv;
                cheb_fd<KR1>(r2 * rinv, a.rcRinv, f, fd);
#pragma unroll
                for (int k = 0; k < KR1; ++k) fd[k] *= rdot;
            }
#pragma unroll
            for (int k = 0; k < KR1; ++k) {
                sh[lane * RP + k] = f[k];
                sh[lane * RP + KR1 + k] = fd[k];
            }
            wave_lds_sync();
            const int hi = min(o1 - p0, 64);
#pragma unroll 4
            for (int x = max(o0 - p0, 0) + gr; x < hi; x += ng) {
                s += sh[x * RP + ko];
                sd += sh[x * RP + KR1 + ko];
            }
            wave_lds_sync();
        }
        ssk[lane] = s;
        ssk[64 + lane] = sd;
        wave_lds_sync();
        if (gr == 0) {
            for (int g = 1; g < ng; ++g) {
                s += ssk[g * nk + lane];
                sd += ssk[64 + g * nk + lane];
            }
            row[R.sk + lane] = s;
            row[R.skd + lane] = sd;
        }
        wave_lds_sync();
        if (gr == 0) {
            ssk[lane] = s;
            ssk[64 + lane] = sd;
        }
    }
    {
        const float *c = prm + a.oA + ti * S * NA1 * KA1;
        for (int x = lane; x < S * NA1 * KA1; x += 64) sc[x] = c[x];
    }
    wave_lds_sync();
    if (lane < NR1) {
        float q = 0.0f, qd = 0.0f;
        for (int t = 0; t < S; ++t) {
            const float *c = prm + a.oR + (ti * S + t) * NR1 * KR1 + lane * KR1;
#pragma unroll
            for (int k = 0; k < KR1; ++k) {
                q = fmaf(c[k], ssk[t * KR1 + k], q);
                qd = fmaf(c[k], ssk[64 + t * KR1 + k], qd);
            }
        }
        sq[lane] = q;
        sqd[lane] = qd;
    }

    // ---- angular: per lane one neighbour's basis, harmonics and their derivatives along d
    const int32_t *uW = a.uniW + (size_t)i * a.capA;
    const uint64_t *mA = a.umA + (size_t)i * a.capA;
    const int nA = uendA[S - 1];
    float f[KA1], fp[KA1], Y[kNumSH], Dm[kNumSH], rdot = 0.0f;
    int tj = 0;
    auto eval = [&](int p0) {
        const int e = p0 + lane;
        rdot = 0.0f;
        tj = 0;
#pragma unroll
        for (int k = 0; k < KA1; ++k) {
            f[k] = 0.0f;
            fp[k] = 0.0f;
        }
#pragma unroll
        for (int m = 0; m < kNumSH; ++m) {
            Y[m] = 0.0f;
            Dm[m] = 0.0f;
        }
        if (e < nA && ((mA[e] >> b) & 1u)) {
            const int32_t w = uW[e];
            tj = w & 3;
            const float4 dj = *row_at(dFb, w >> 2, pstride);
            float dx, dy, dz, ex, ey, ez;
            pair_vec<kPosAny>(*row_at(p4b, w >> 2, pstride), pi, lm, dx, dy, dz);
            const float r2 = norm2(dx, dy, dz);
            const float rinv = __builtin_amdgcn_rsqf(r2);
            const float ux = dx * rinv, uy = dy * rinv, uz = dz * rinv;
            field(dj, dx, dy, dz, ex, ey, ez);
            rdot = ux * ex + uy * ey + uz * ez;
            cheb_fd<KA1>(r2 * rinv, a.rcAinv, f, fp);
            sh_eval(ux, uy, uz, shc, Y);
            // du/de = (d - u (u . d)) / r
            sh_dir(ux, uy, uz, (ex - ux * rdot) * rinv, (ey - uy * rdot) * rinv, (ez - uz * rdot) * rinv, shc, Dm);
        }
    };
    const int hl = lane / kRowStage, sl = lane & (kRowStage - 1);
    // owner lanes of the entries (n, m) of A and Adot
    float A[NACC], Ad[NACC];
    int on[NACC], om[NACC];
#pragma unroll
    for (int q = 0; q < NACC; ++q) {
        const int x = min(lane + 64 * q, NA1 * kNumSH - 1);
        A[q] = 0.0f;
        Ad[q] = 0.0f;
        on[q] = x / kNumSH;
        om[q] = x - on[q] * kNumSH;
    }
    for (int p0 = 0; p0 < nA; p0 += 64) {
        eval(p0);
        float g[NA1], gd[NA1];
#pragma unroll
        for (int n = 0; n < NA1; ++n) {
            const float *c = sc + (tj * NA1 + n) * KA1;
            float v = 0.0f, vp = 0.0f;
#pragma unroll
            for (int k = 0; k < KA1; ++k) {
                v = fmaf(c[k], f[k], v);
                vp = fmaf(c[k], fp[k], vp);
            }
            g[n] = v;
            gd[n] = vp * rdot;
        }
        for (int h = 0; h < 64 / kRowStage && p0 + h * kRowStage < nA; ++h) {
            wave_lds_sync();
            if (hl == h) {
#pragma unroll
                for (int m = 0; m < kNumSH; ++m) {
                    sh[sl * HP + m] = Y[m];
                    sh[sl * HP + kNumSH + m] = Dm[m];
                }
#pragma unroll
                for (int n = 0; n < NA1; ++n) {
                    sg[sl * GP + n] = g[n];
                    sg[sl * GP + NA1 + n] = gd[n];
                }
            }
            wave_lds_sync();
            const int hi = min(nA - p0 - h * kRowStage, kRowStage);
#pragma unroll 2
            for (int x = 0; x < hi; ++x)
#pragma unroll
                for (int q = 0; q < NACC; ++q) {
                    const float y = sh[x * HP + om[q]], gn = sg[x * GP + on[q]];
                    A[q] = fmaf(gn, y, A[q]);
                    Ad[q] = fmaf(sg[x * GP + NA1 + on[q]], y, fmaf(gn, sh[x * HP + kNumSH + om[q]], Ad[q]));
                }
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < NACC; ++q)
        if (lane + 64 * q < NA1 * kNumSH) {
            sA[on[q]][om[q]] = A[q];
            sB[on[q]][om[q]] = Ad[q];
        }
    wave_lds_sync();
    if (lane < NA1) {
#pragma unroll
        for (int l = 1; l <= kLmax; ++l) {
            float s2 = 0.0f, s2d = 0.0f;
#pragma unroll
            for (int m = 0; m < kNumSH; ++m)
                if (sh_l(m) == l) {
                    s2 = fmaf(sA[lane][m], sA[lane][m], s2);
                    s2d = fmaf(2.0f * sA[lane][m], sB[lane][m], s2d);
                }
            sq[NR1 + (l - 1) * NA1 + lane] = s2;
            sqd[NR1 + (l - 1) * NA1 + lane] = s2d;
        }
    }
    wave_lds_sync();
    const float qsl = qs[min(lane, D - 1)];
    if (lane < D) {
        const float v = qsl * sq[lane], vd = qsl * sqd[lane];
        sq[lane] = v;
        sqd[lane] = vd;
        row[R.sq + lane] = v;
        row[R.sqd + lane] = vd;
    }
    wave_lds_sync();

    // ---- network and its forward derivative: a hidden unit per lane, then G, Gdot per lane
    {
        const float *W0 = prm + a.oW0 + (size_t)ti * H * D;
        const float *b0 = prm + a.ob0 + ti * H, *w1 = prm + a.ow1 + ti * H;
        float *su = dyn, *sud = dyn + H;
        for (int mu = lane; mu < H; mu += 64) {
            float z = -b0[mu], zd = 0.0f;
#pragma unroll
            for (int v = 0; v < D; ++v) {
                const float w = W0[mu * D + v];
                z = fmaf(w, sq[v], z);
                zd = fmaf(w, sqd[v], zd);
            }
            float h, dh;
            tanh_and_slope(z, h, dh);
            const float u = w1[mu] * dh;                   // dU/dz
            const float ud = -2.0f * w1[mu] * h * dh * zd;  // its derivative along d
            su[mu] = u;
            sud[mu] = ud;
            row[R.u + mu] = u;
            row[R.v + mu] = eEb * u + ud;
            row[R.gw1 + mu] = eEb * h + dh * zd;
        }
        wave_lds_sync();
        const float *wv = W0 + min(lane, D - 1);
        float G = 0.0f, Gd = 0.0f;
#pragma unroll 10
        for (int mu = 0; mu < H; ++mu) {
            const float w = wv[mu * D];
            G = fmaf(su[mu], w, G);
            Gd = fmaf(sud[mu], w, Gd);
        }
        if (lane < D) {
            sG[lane] = qsl * G;
            sGd[lane] = qsl * Gd;
        }
    }
    if (lane == 0) {
        row[R.eE] = eEb;
        row[0] = __int_as_float(ti);
    }
    wave_lds_sync();
    if (lane < NR1) {
        row[R.gR + lane] = eEb * sG[lane] + sGd[lane];
        row[R.GR + lane] = sG[lane];
    }

    // ---- angular coefficients: X and B, then al, be per neighbour, then the sums over neighbours
#pragma unroll
    for (int q = 0; q < NACC; ++q)
        if (lane + 64 * q < NA1 * kNumSH) {
            const int l = om[q] < 3 ? 0 : om[q] < 8 ? 1 : om[q] < 15 ? 2 : 3, v = NR1 + l * NA1 + on[q];
            const float g = sG[v], gd = sGd[v], Bv = 2.0f * g * A[q];
            sA[on[q]][om[q]] = eEb * Bv + 2.0f * (gd * A[q] + g * Ad[q]);
            sB[on[q]][om[q]] = Bv;
        }
    const int nco = S * NA1 * KA1;
    constexpr int NC = (kMaxSpecies * NA1 * KA1 + 63) / 64;
    float acc[NC];   // owner lanes of the coefficients (t, n, k)
#pragma unroll
    for (int q = 0; q < NC; ++q) acc[q] = 0.0f;
    wave_lds_sync();
    for (int p0 = 0; p0 < nA; p0 += 64) {
        if (nA > 64) eval(p0);
        float al[NA1], be[NA1];
#pragma unroll
        for (int n = 0; n < NA1; ++n) {
            float x = 0.0f, y = 0.0f;
#pragma unroll
            for (int m = 0; m < kNumSH; ++m) {
                const float Bn = sB[n][m];
                x = fmaf(sA[n][m], Y[m], fmaf(Bn, Dm[m], x));
                y = fmaf(Bn, Y[m], y);
            }
            al[n] = x;
            be[n] = y * rdot;
        }
        for (int h = 0; h < 64 / kRowStage && p0 + h * kRowStage < nA; ++h) {
            const int q0 = p0 + h * kRowStage;
            wave_lds_sync();
            if (hl == h) {
#pragma unroll
                for (int n = 0; n < NA1; ++n) {
                    sg[sl * GP + n] = al[n];
                    sg[sl * GP + NA1 + n] = be[n];
                }
#pragma unroll
                for (int k = 0; k < KA1; ++k) {
                    sh[sl * HP + k] = f[k];
                    sh[sl * HP + KA1 + k] = fp[k];
                }
            }
            wave_lds_sync();
#pragma unroll
            for (int q = 0; q < NC; ++q) {
                if (64 * q >= nco) break;
                const int o = min(lane + 64 * q, nco - 1);
                const int t = o / (NA1 * KA1), n = (o - t * NA1 * KA1) / KA1, k = o % KA1;
                const int lo = max((t ? uendA[t - 1] : 0) - q0, 0), up = min(uendA[t] - q0, kRowStage);
                float v = acc[q];
#pragma unroll 2
                for (int x = lo; x < up; ++x)
                    v = fmaf(sg[x * GP + n], sh[x * HP + k], fmaf(sg[x * GP + NA1 + n], sh[x * HP + KA1 + k], v));
                acc[q] = v;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NC; ++q)
        if (lane + 64 * q < nco) row[R.gA + lane + 64 * q] = acc[q];
}

// Parameter-gradient partial sums over a block of rows, one species per
// grid.z.  Outputs of a species:
//   W0[mu][nu] += u_mu sqd_nu + v_mu sq_nu,  b0[mu] -= v_mu,  w1[mu] += gw1_mu,
//   cR[t][n][k] += gR_n sk_tk + GR_n skd_tk,  cA[t][n][k] += gA_tnk,
// and the last output of the call is b1 -= sum eE.  Workgroup y takes a tile
// of kTileH hidden units by all descriptors, an outer product per row with
// 2 x TD entries per thread (four LDS reads per four products), and 256 of
// the other outputs, so that the rows are read once where one tile and one
// slice hold all (60 MB at 65,536 rows; an output per thread, the rows
// streamed once per 256 outputs, took 152 us there).
constexpr int kRowChunk = 16;
constexpr int kTileH = 32;
template <int TD>
__global__ __launch_bounds__(256) void k_grad_partial(const float *__restrict__ rows, size_t nrow, int RW, int S,
                                                      int H, int D, int NR1, int KR1, int NA1, int KA1,
                                                      int rows_per_block, int chunk, int ntile,
                                                      float *__restrict__ part)
{
    extern __shared__ float sh[];   // [chunk][RW]
    const RowLayout R(H, D, NR1, S, KR1, NA1, KA1);
    const int per = H * D + 2 * H + S * NR1 * KR1 + S * NA1 * KA1;
    const int nout = S * per + 1;
    const int sp = blockIdx.z, tid = threadIdx.x;
    const size_t r0 = (size_t)blockIdx.x * rows_per_block;
    const size_t r1 = r0 + rows_per_block < nrow ? r0 + rows_per_block : nrow;
    const bool tile = (int)blockIdx.y < ntile;   // uniform
    // tile blocks: hidden units h0, h0 + 16 and descriptors td, td + 16, ...
    const int td = tid & 15, h0 = (int)blockIdx.y * kTileH + (tid >> 4);
    float w[2][TD];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int c = 0; c < TD; ++c) w[x][c] = 0.0f;
    int ou[2], od[TD];   // offsets into a row (clamped; only valid outputs are stored)
#pragma unroll
    for (int x = 0; x < 2; ++x) ou[x] = min(h0 + 16 * x, H - 1);
#pragma unroll
    for (int c = 0; c < TD; ++c) od[c] = min(td + 16 * c, D - 1);
    // other blocks: output q of the species (q == nrest: b1, by species 0)
    const int nrest = per - H * D;
    const int q = (int)blockIdx.y * 256 + tid;
    int kind = -1, i1 = 0, i2 = 0, t = 0;
    {
        if (q < H) {
            kind = 1; i1 = q;
        } else if (q < 2 * H) {
            kind = 2; i1 = q - H;
        } else if (q < 2 * H + S * NR1 * KR1) {
            const int c = q - 2 * H;   // [t][n][k]
            kind = 3; t = c / (NR1 * KR1);
            const int nk = c - t * NR1 * KR1;
            i1 = nk / KR1; i2 = nk - i1 * KR1;
        } else if (q < nrest) {
            kind = 5; i1 = q - 2 * H - S * NR1 * KR1;   // [t][n][k]
        } else if (q == nrest && sp == 0) {
            kind = 4;
        }
    }
    float acc = 0.0f;
    for (size_t c0 = r0; c0 < r1; c0 += chunk) {
        const int nr = (int)((r1 - c0) < (size_t)chunk ? (r1 - c0) : (size_t)chunk);
        // chunks without a row of this species are skipped (b1 takes the rows of every species)
        int ty = tid < nr ? __float_as_int(rows[(c0 + tid) * RW]) : -1;
        const bool any = __syncthreads_or(ty >= 0 && (ty == sp || sp == 0));
        if (!any) continue;
        const float *src = rows + c0 * RW;
#pragma unroll 8
        for (int x = tid; x < nr * RW; x += 256) sh[x] = src[x];
        __syncthreads();
        for (int r = 0; r < nr; ++r) {
            const float *rw = sh + r * RW;
            const int tr = __float_as_int(rw[0]);
            if (kind == 4 && tr >= 0) acc -= rw[R.eE];
            if (tr != sp) continue;   // uniform
            if (tile) {
                const float u0 = rw[R.u + ou[0]], u1 = rw[R.u + ou[1]], v0 = rw[R.v + ou[0]], v1 = rw[R.v + ou[1]];
#pragma unroll
                for (int c = 0; c < TD; ++c) {
                    const float s = rw[R.sq + od[c]], sd = rw[R.sqd + od[c]];
                    w[0][c] = fmaf(u0, sd, fmaf(v0, s, w[0][c]));
                    w[1][c] = fmaf(u1, sd, fmaf(v1, s, w[1][c]));
                }
            }
            if (kind == 1) {
                acc -= rw[R.v + i1];
            } else if (kind == 2) {
                acc += rw[R.gw1 + i1];
            } else if (kind == 5) {
                acc += rw[R.gA + i1];
            } else if (kind == 3) {
                acc = fmaf(rw[R.gR + i1], rw[R.sk + t * KR1 + i2], fmaf(rw[R.GR + i1], rw[R.skd + t * KR1 + i2], acc));
            }
        }
        __syncthreads();
    }
    float *out = part + (size_t)blockIdx.x * nout;
    if (tile) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int c = 0; c < TD; ++c)
                if (h0 + 16 * x < H && td + 16 * c < D) out[sp * per + (h0 + 16 * x) * D + td + 16 * c] = w[x][c];
    }
    if (kind == 4) {
        out[nout - 1] = acc;
    } else if (kind >= 0) {
        out[sp * per + H * D + q] = acc;
    }
}

// Sums the partials and scatters them to the parameter layout.  A
// workgroup takes 64 consecutive outputs (one per lane, coalesced reads);
// its kGradWaves wavefronts take every kGradWaves-th block in order, and
// the wavefronts' sums are added in wavefront order (fixed order).  The last
// workgroup adds the loss terms of k_residual, also in a fixed order.
constexpr int kGradWaves = 16;
__device__ double block_sum(const double *__restrict__ x, int n, double (*red)[64])
{
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += 64 * kGradWaves) s += x[k];
    s = wave_sum(s);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][0] = s;
    __syncthreads();
    double t = 0.0;
    for (int v = 0; v < kGradWaves; ++v) t += red[v][0];
    return t;
}

__global__ __launch_bounds__(64 * kGradWaves) void k_grad_final(const float *__restrict__ part, int nblk, int S, int H,
                                                                int D, int NR1, int KR1, int NA1, int KA1,
                                                                ParamLayout off, float *__restrict__ grad,
                                                                const double *__restrict__ lossp, int nfblk, int nsb,
                                                                double *__restrict__ loss)
{
    if (blockIdx.x == gridDim.x - 1) {
        __shared__ double lred[kGradWaves][64];
        const double lf = block_sum(lossp, nfblk, lred), le = block_sum(lossp + nfblk, nsb, lred),
                     lw = block_sum(lossp + nfblk + nsb, nsb, lred);
        if (threadIdx.x == 0) {
            loss[0] += le + lf + lw;
            loss[1] += le;
            loss[2] += lf;
            loss[3] += lw;
        }
        return;
    }
    const int per = H * D + 2 * H + S * NR1 * KR1 + S * NA1 * KA1;
    const int nout = S * per + 1;
    const int w = threadIdx.x >> 6;
    const int o = blockIdx.x * 64 + (threadIdx.x & 63);
    __shared__ double red[kGradWaves][64];
    double acc = 0.0;
    if (o < nout)
#pragma unroll 8
        for (int k = w; k < nblk; k += kGradWaves) acc += part[(size_t)k * nout + o];
    red[w][threadIdx.x & 63] = acc;
    __syncthreads();
    if (w != 0 || o >= nout) return;
    double s = 0.0;
    for (int v = 0; v < kGradWaves; ++v) s += red[v][threadIdx.x];
    int idx;
    if (o == nout - 1) {
        idx = off.b1;
    } else {
        const int sp = o / per, q = o - sp * per;
        if (q < H * D) idx = off.W0 + sp * H * D + q;
        else if (q < H * D + H) idx = off.b0 + sp * H + (q - H * D);
        else if (q < H * D + 2 * H) idx = off.w1 + sp * H + (q - H * D - H);
        else if (q < H * D + 2 * H + S * NR1 * KR1) idx = off.cR + sp * S * NR1 * KR1 + (q - H * D - 2 * H);
        else idx = off.cA + sp * S * NA1 * KA1 + (q - H * D - 2 * H - S * NR1 * KR1);
    }
    grad[idx] += (float)s;
}

// Adam with bias correction over the trainable parameter ranges.
__global__ void k_adam(float *__restrict__ th, const float *__restrict__ g, float *__restrict__ m1,
                       float *__restrict__ m2, int n, const int32_t *__restrict__ trainable, float lr, float b1,
                       float b2, float eps, float c1, float c2)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n || !trainable[k]) return;
    const float gk = g[k];
    const float a = b1 * m1[k] + (1.0f - b1) * gk;
    const float v = b2 * m2[k] + (1.0f - b2) * gk * gk;
    m1[k] = a;
    m2[k] = v;
    th[k] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
}

template <int NR1, int NA1>
static void launch_rows(const NepArgs &a, const TrainArgs &t, const float *prm, const int32_t *atom_sys, float *part,
                        int nblk, int rows_per_block, hipStream_t s)
{
    constexpr int D = Dims<NR1, NA1, false>::D;
    const unsigned nrow = (unsigned)a.N * (unsigned)a.P;
    hipLaunchKernelGGL((k_train_row<NR1, NA1>), dim3(nrow), dim3(64), sizeof(float) * 2 * a.H, s, a, t, prm, atom_sys);
    const int ntile = div_up(a.H, kTileH), nrest = 2 * a.H + a.S * (NR1 + NA1) * 9 + 1;
    // rows staged at a time: up to 60 KiB of LDS
    const int chunk = std::max(1, std::min(kRowChunk, (60 * 1024) / (int)(sizeof(float) * t.RW)));
    hipLaunchKernelGGL((k_grad_partial<(D + 15) / 16>), dim3(nblk, std::max(ntile, div_up(nrest, 256)), a.S), dim3(256),
                       sizeof(float) * chunk * t.RW, s, t.rows, (size_t)nrow, t.RW, a.S, a.H, D, NR1, 9, NA1, 9,
                       rows_per_block, chunk, ntile, part);
}

}  // namespace nep

using namespace nep;

struct nep_train_ws {
    int P = 0, N = 0, nsys = 1;
    std::vector<int> off;                // host [nsys+1]
    int32_t *atom_sys = nullptr;         // [N] system of each atom
    int32_t *sys_off = nullptr;          // [nsys+1]
    double *E = nullptr, *W = nullptr;   // [nsys][P], [nsys][P][9]
    float *F = nullptr;                  // [P][N][3]
    float4 *dF = nullptr;                // [N][P]
    float *cW = nullptr, *eE = nullptr;  // [nsys][P][9], [nsys][P]
    float *rows = nullptr;               // [N*P][RW]
    float *part = nullptr;               // [nblk][nout]
    double *lossp = nullptr;             // loss terms: force per workgroup of k_residual, energy and virial [nsys][P]
    int nfblk = 0;                       // workgroups of the force residuals
    int RW = 0, nout = 0, nblk = 0, rows_per_block = 0;
    int32_t *trainable = nullptr;        // [params] 0/1
    int ntrain_mask = -1;
};

extern "C" int32_t nep_train_ws_create_batched(const nep_model *m, int32_t P, int32_t nsys, const int32_t *off,
                                               nep_train_ws **out)
{
    if (!m || !out) return fail(NEP_ERR_INVALID_ARG, "nep_train_ws_create: null argument");
    if (m->cutoffs_only) return fail(NEP_ERR_INVALID_ARG, "nep_train_ws_create: a list cutoff descriptor has no network");
    if (m->embedded)
        return fail(NEP_ERR_UNSUPPORTED, "nep_train_ws_create: a model embedded in a larger kernel shape is not trainable");
    const int32_t rc0 = check_offsets(nsys, off, "nep_train_ws_create");
    if (rc0 != NEP_OK) return rc0;
    const int32_t N = off[nsys];
    if (P < 1 || P > kMaxBeads || N < 1) return fail(NEP_ERR_INVALID_ARG, "nep_train_ws_create: bad sizes");
    const nep_hparams &h = m->hp;
    if (h.four_body) return fail(NEP_ERR_UNSUPPORTED, "nep_train_ws_create: four-body models are not trainable");
    const int key = h.n_max_radial * 100 + h.n_max_angular * 10;
    if (key != 440 && key != 640 && key != 860)
        return fail(NEP_ERR_UNSUPPORTED, "nep_train_ws_create: unsupported model shape");
    const int S = h.n_species, H = h.hidden, D = h.dim, NR1 = h.n_max_radial + 1, KR1 = h.basis_radial + 1;
    const int NA1 = h.n_max_angular + 1, KA1 = h.basis_angular + 1;
    const RowLayout R(H, D, NR1, S, KR1, NA1, KA1);
    const int nout = S * (H * D + 2 * H + S * NR1 * KR1 + S * NA1 * KA1) + 1;
    if ((nout + 255) / 256 > 64) return fail(NEP_ERR_UNSUPPORTED, "nep_train_ws_create: model too large to train");
    *out = nullptr;
    nep_train_ws *w = new (std::nothrow) nep_train_ws;
    if (!w) return fail(NEP_ERR_NOMEM, "host allocation failed");
    w->P = P; w->N = N; w->RW = R.RW; w->nout = nout;
    w->nsys = nsys;
    w->off.assign(off, off + nsys + 1);
    std::vector<int32_t> asys((size_t)N);
    for (int sy = 0; sy < nsys; ++sy)
        for (int i = off[sy]; i < off[sy + 1]; ++i) asys[i] = sy;
    const size_t PN = (size_t)P * N;
    // about 1024 row blocks (times hidden-unit tiles and species), of 16 to 512 rows
    w->rows_per_block = (int)std::min<size_t>(512, std::max<size_t>(kRowChunk, (PN + 1023) / 1024));
    w->nfblk = (int)((PN + 255) / 256);
    w->nblk = (int)((PN + w->rows_per_block - 1) / w->rows_per_block);
    hipError_t e = hipSuccess;
    auto al = [&](void **p, size_t bytes) {
        if (e == hipSuccess) e = hipMalloc(p, bytes ? bytes : 4);
    };
    al((void **)&w->atom_sys, sizeof(int32_t) * N);
    al((void **)&w->sys_off, sizeof(int32_t) * (nsys + 1));
    if (e == hipSuccess) e = hipMemcpy(w->atom_sys, asys.data(), sizeof(int32_t) * N, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(w->sys_off, off, sizeof(int32_t) * (nsys + 1), hipMemcpyHostToDevice);
    al((void **)&w->E, sizeof(double) * nsys * P);
    al((void **)&w->W, sizeof(double) * 9 * nsys * P);
    al((void **)&w->F, sizeof(float) * 3 * PN);
    al((void **)&w->dF, sizeof(float4) * PN);
    al((void **)&w->cW, sizeof(float) * 9 * nsys * P);
    al((void **)&w->eE, sizeof(float) * nsys * P);
    al((void **)&w->rows, sizeof(float) * PN * R.RW);
    al((void **)&w->lossp, sizeof(double) * ((size_t)w->nfblk + 2 * (size_t)nsys * P));
    al((void **)&w->part, sizeof(float) * (size_t)w->nblk * nout);
    al((void **)&w->trainable, sizeof(int32_t) * m->off.total);
    if (e != hipSuccess) {
        nep_train_ws_destroy(w);
        return fail(e == hipErrorOutOfMemory ? NEP_ERR_NOMEM : NEP_ERR_HIP, "training workspace: %s",
                    hipGetErrorString(e));
    }
    *out = w;
    return NEP_OK;
}

extern "C" void nep_train_ws_destroy(nep_train_ws *w)
{
    if (!w) return;
    for (void *p : {(void *)w->atom_sys, (void *)w->sys_off, (void *)w->E, (void *)w->W, (void *)w->F, (void *)w->dF, (void *)w->cW, (void *)w->eE,
                    (void *)w->rows, (void *)w->lossp, (void *)w->part, (void *)w->trainable})
        if (p) (void)hipFree(p);
    delete w;
}

extern "C" int32_t nep_train_ws_create(const nep_model *m, int32_t P, int32_t N, nep_train_ws **out)
{
    if (N < 1) return fail(NEP_ERR_INVALID_ARG, "nep_train_ws_create: bad sizes");
    const int32_t off[2] = {0, N};
    return nep_train_ws_create_batched(m, P, 1, off, out);
}

extern "C" int32_t nep_param_grad_batched(const nep_model *m, nep_nlist *nl, nep_ws *ws, nep_train_ws *tw,
                                          const double *pos, const double *boxes, const int32_t *types, int32_t P,
                                          int32_t N, const double *E_ref, const float *F_ref, const double *W_ref,
                                          const double lambda[3], float *grad, double *loss, hipStream_t s)
{
    if (!m || !nl || !ws || !tw || !lambda || !grad || !loss || !E_ref || !F_ref || !W_ref)
        return fail(NEP_ERR_INVALID_ARG, "nep_param_grad: null argument");
    if (m->cutoffs_only) return fail(NEP_ERR_INVALID_ARG, "nep_param_grad: a list cutoff descriptor has no network");
    if (tw->P != P || tw->N != N || nl->nsys != tw->nsys || ws->nsys != tw->nsys || nl->off != tw->off ||
        ws->off != tw->off)
        return fail(NEP_ERR_INVALID_ARG, "nep_param_grad: sizes or systems do not match the training workspace");
    if (m->mlp == NEP_MLP_BF16_MFMA)
        return fail(NEP_ERR_INVALID_ARG, "nep_param_grad: training needs the FP32 weights (nep_model_set_mlp)");
    int32_t rc = nep_compute_batched(m, nl, ws, pos, boxes, types, P, N, tw->E, tw->F, tw->W, nullptr, nullptr, s);
    if (rc != NEP_OK) return rc;
    const size_t PN = (size_t)P * N;
    const int nsb = tw->nsys * P;
    hipLaunchKernelGGL(k_residual, dim3(tw->nfblk + div_up(nsb, 256)), dim3(256), 0, s, tw->F, F_ref, tw->E, E_ref,
                       tw->W, W_ref, P, N, tw->nsys, tw->atom_sys, tw->sys_off, lambda[0], lambda[1], lambda[2],
                       tw->dF, tw->cW, tw->eE, tw->lossp, tw->nfblk);
    const nep_hparams &h = m->hp;
    NepArgs a{};
    a.p4 = reinterpret_cast<const float4 *>(nl->pos4); a.types = types; a.N = N; a.S = h.n_species;
    a.H = h.hidden; a.P = P;
    a.geom = nl->geom;
    a.rcRinv = (float)(1.0 / h.rc_radial); a.rcAinv = (float)(1.0 / h.rc_angular);
    a.uniR = nl->uniR; a.uendR = nl->uendR; a.uniW = nl->uniW;
    a.umR = nl->umR; a.umA = nl->umA; a.uendA = nl->uendA; a.capR = nl->capR; a.capA = nl->capA;
    a.oR = m->off.cR; a.oA = m->off.cA; a.oq = m->off.qs; a.oW0 = m->off.W0; a.ob0 = m->off.b0;
    a.ow1 = m->off.w1; a.ob1 = m->off.b1; a.osh = m->off.sh;
    TrainArgs t{tw->dF, tw->cW, tw->eE, tw->rows, tw->RW};
    const int key = h.n_max_radial * 100 + h.n_max_angular * 10;
    switch (key) {
    case 440: launch_rows<5, 5>(a, t, m->dev, nl->atom_sys, tw->part, tw->nblk, tw->rows_per_block, s); break;
    case 640: launch_rows<7, 5>(a, t, m->dev, nl->atom_sys, tw->part, tw->nblk, tw->rows_per_block, s); break;
    case 860: launch_rows<9, 7>(a, t, m->dev, nl->atom_sys, tw->part, tw->nblk, tw->rows_per_block, s); break;
    default: return fail(NEP_ERR_UNSUPPORTED, "nep_param_grad: unsupported model shape");
    }
    const int S = h.n_species, H = h.hidden, D = h.dim, NR1 = h.n_max_radial + 1, KR1 = h.basis_radial + 1;
    const int NA1 = h.n_max_angular + 1, KA1 = h.basis_angular + 1;
    hipLaunchKernelGGL(k_grad_final, dim3((tw->nout + 63) / 64 + 1), dim3(64 * kGradWaves), 0, s, tw->part, tw->nblk,
                       S, H, D, NR1, KR1, NA1, KA1, m->off, grad, tw->lossp, tw->nfblk, nsb, loss);
    NEP_HIP(hipGetLastError());
    return NEP_OK;
}

extern "C" int32_t nep_param_grad(const nep_model *m, nep_nlist *nl, nep_ws *ws, nep_train_ws *tw, const double *pos,
                                  const double box[9], const int32_t *types, int32_t P, int32_t N,
                                  const double *E_ref, const float *F_ref, const double *W_ref,
                                  const double lambda[3], float *grad, double *loss, hipStream_t s)
{
    if ((nl && nl->nsys != 1) || (tw && tw->nsys != 1))
        return fail(NEP_ERR_INVALID_ARG, "nep_param_grad: the list or workspace holds a batch of systems");
    return nep_param_grad_batched(m, nl, ws, tw, pos, box, types, P, N, E_ref, F_ref, W_ref, lambda, grad, loss, s);
}

extern "C" int32_t nep_model_params(nep_model *m, float **params, int32_t *count, nep_param_offsets *off)
{
    if (!m || !params || !count) return fail(NEP_ERR_INVALID_ARG, "nep_model_params: null argument");
    if (m->cutoffs_only) return fail(NEP_ERR_INVALID_ARG, "nep_model_params: a list cutoff descriptor has no network");
    if (m->embedded)
        return fail(NEP_ERR_UNSUPPORTED, "nep_model_params: the parameters of a model embedded in a larger kernel "
                                         "shape are not exposed");
    *params = m->dev;
    *count = m->off.total;
    if (off) {
        off->c_radial = m->off.cR; off->c_angular = m->off.cA; off->q_scale = m->off.qs; off->W0 = m->off.W0;
        off->b0 = m->off.b0; off->w1 = m->off.w1; off->b1 = m->off.b1; off->sh = m->off.sh;
    }
    return NEP_OK;
}

extern "C" int32_t nep_adam_step(nep_model *m, nep_train_ws *tw, const float *grad, float *m1, float *m2,
                                 int64_t step, float lr, float beta1, float beta2, float eps, int32_t mask,
                                 hipStream_t s)
{
    if (!m || !tw || !grad || !m1 || !m2) return fail(NEP_ERR_INVALID_ARG, "nep_adam_step: null argument");
    if (step < 1 || !(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) ||
        !(eps > 0.0f) || mask < 1 || mask > 7)
        return fail(NEP_ERR_INVALID_ARG, "nep_adam_step: bad hyperparameters");
    const int n = m->off.total;
    if (tw->ntrain_mask != mask) {
        const nep_hparams &h = m->hp;
        std::vector<int32_t> tr(n, 0);
        if (mask & 1)
            for (int k = m->off.W0; k < m->off.b1 + 1; ++k) tr[k] = 1;   // W0, b0, w1, b1
        if (mask & 2) {
            const int nR = h.n_species * h.n_species * (h.n_max_radial + 1) * (h.basis_radial + 1);
            for (int k = m->off.cR; k < m->off.cR + nR; ++k) tr[k] = 1;
        }
        if (mask & 4) {
            const int nA = h.n_species * h.n_species * (h.n_max_angular + 1) * (h.basis_angular + 1);
            for (int k = m->off.cA; k < m->off.cA + nA; ++k) tr[k] = 1;
        }
        NEP_HIP(hipStreamSynchronize(s));
        NEP_HIP(hipMemcpy(tw->trainable, tr.data(), sizeof(int32_t) * n, hipMemcpyHostToDevice));
        tw->ntrain_mask = mask;
    }
    const double c1 = 1.0 - std::pow((double)beta1, (double)step), c2 = 1.0 - std::pow((double)beta2, (double)step);
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, m->dev, grad, m1, m2, n, tw->trainable, lr,
                       beta1, beta2, eps, (float)c1, (float)c2);
    NEP_HIP(hipGetLastError());
    return NEP_OK;
}

// ------------------------------------------------------- force judge ---

// Root-mean-square difference of two force arrays over every component,
// sqrt(sum (Fa - Fb)^2 / n): fixed-grid partial sums in FP64, then one
// block adds the partials in a fixed order (bitwise reproducible).
constexpr int kRmseBlocks = 1024;

__global__ __launch_bounds__(256) void k_rmse_partial(const float *__restrict__ Fa, const float *__restrict__ Fb,
                                                      int64_t n, double *__restrict__ part)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const double d = (double)Fa[e] - (double)Fb[e];
        acc += d * d;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = blockDim.x >> 1; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(256) void k_rmse_final(const double *__restrict__ part, int nblk, int64_t n,
                                                    double *__restrict__ out)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int k = threadIdx.x; k < nblk; k += blockDim.x) acc += part[k];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = blockDim.x >> 1; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = n > 0 ? sqrt(red[0] / (double)n) : 0.0;
}

extern "C" int32_t nep_force_rmse(const float *Fa, const float *Fb, int64_t n, double *work, hipStream_t s)
{
    if (!work) return fail(NEP_ERR_INVALID_ARG, "nep_force_rmse: null work array");
    if (n < 0) return fail(NEP_ERR_INVALID_ARG, "nep_force_rmse: negative length");
    if (n > 0 && (!Fa || !Fb)) return fail(NEP_ERR_INVALID_ARG, "nep_force_rmse: null force array");
    const int nblk = (int)std::min<int64_t>(kRmseBlocks, std::max<int64_t>(1, (n + 255) / 256));
    if (n > 0)
        hipLaunchKernelGGL(k_rmse_partial, dim3(nblk), dim3(256), 0, s, Fa, Fb, n, work + 1);
    hipLaunchKernelGGL(k_rmse_final, dim3(1), dim3(256), 0, s, work + 1, n > 0 ? nblk : 0, n, work);
    NEP_HIP(hipGetLastError());
    return NEP_OK;
}
