// Adjoint of the cosmic-shear likelihood (App. A of the paper), input
// gradients only.
//
// Reverse mode runs from logL back to the emulator table:
//   dense chi^2:   g_C = L^{-T} L^{-1} (d - C)  (two FP64-MFMA GEMMs, shear.hip)
//   Limber (A2):   C_pb = f_p sum_j W_a(j) W_b(j) P_bj wq_j,  f_p = (1+m_a)(1+m_b)
//                  -> g(P wq)_bj, g W_i(j), g wq_j, and g chi_j through k = (l+1/2)/chi_j
//   P lookup:      P = 10^{CR(t; Yhat_j(c))}, Yhat = the table carried to z_j
//                  (cubic spline or linear in z) -> scatter into g Y (and g M, the
//                  spline second derivatives, whose map M = S(Y) is then
//                  transposed by zspline_adjoint_kernel) -> emulator backward.
// Forward mode covers the per-walker background and windows, which depend on
// few parameters: shear_tangent_kernel stores, per a-node, chi, wq, W_i and
// their tangents in the directions (Om, h, w0, wa) and, per bin, (Dz_i,
// A_IA,i); limber_adjoint_kernel contracts them into the direct gradient
//   sum_j [ sum_i gW_i(j) dW_i(j) + g wq_j dwq_j + g chi_j dchi_j ].
// Every Limber-adjoint term belongs to one a-node, so a lane owns a node.
//
// The scatter into g Y (and g M) is accumulated in 64-bit fixed point, so that
// its result does not depend on the order in which the nodes of a walker
// reach a table entry: limber_adjoint_kernel computes and stores every
// g log10 P_bj of the walker and their largest magnitude G; then
// limber_scatter_kernel adds each contribution c w g log10 P (|c w| < 2:
// spline and Catmull-Rom weights) rounded to the grid 2^(e - FX_BITS),
// G < 2^e, as integers: slab by slab (runs of z rows that fit in LDS, each
// taking the parts of the contributions that fall on its rows) with LDS
// atomics, then each row once as a double.  At most
// n_a n_ell <= 2^16 contributions reach one entry, so every partial sum stays
// below 2^(FX_BITS + 17) < 2^63; the grid step is below G 2^-44 (about
// 6e-14 G), well under the FP64 gradient's error against the complex step.
// The spline-curvature table g M takes contributions smaller by the factor
// max |c2|, |c3| <= 0.385 h^2 / 6 (h the z-node spacing) and has a grid finer
// by 2^mshift, mshift = floor(log2(6 / (0.385 h^2))).
#include "devutil.h"
#include "nsmi.h"
#include "shear_common.h"

#include <type_traits>

namespace nsmi {

// ------------------------------------------------ background / window tangents
// Forward-mode tangents per node.  Directions 0..3 = (Om, h, w0, wa); per bin,
// Dz_i and A_IA,i.  One workgroup (256 threads) per (walker, group of BPG
// bins), nodes in chunks of 256.  Output record per node, structure of arrays
// tg[(w S + field) n_a + j]: for each of the n_grp groups the TG_FIXED fields
// below (every group forms them for itself, the adjoint reads group 0's),
// then at X = TG_FIXED n_grp: W_i at X + i, dW_i / d(Om, h, w0, wa)_q at
// X + nb + 4 i + q, dW_i / dDz_i at X + 5 nb + i, dW_i / dA_IA,i at
// X + 6 nb + i; S = X + 7 n_bins.
constexpr int TG_CHI = 0, TG_DCHI = 1, TG_WQ = 5, TG_DWQ = 6, TG_LND = 10, TG_DLND = 11, TG_LCHI = 15, TG_FIXED = 16;
//   (a) forward pass: Simpson increments of chi, -ln D and their tangents from
//       the background at the nodes and midpoints (powers of a from the
//       model's ln a table, one exponential each), prefix sums carried from
//       chunk to chunk;
//   (b) n(z) normalisations N_i and dN_i / dDz_i;
//   (c) reverse pass (last chunk first, threads from the last node down, so
//       that the reverse cumulative trapezoids are prefix sums): G0, G1 and
//       their Dz tangents, then the (Om, h, w0, wa) tangents of G1; windows
//       and their tangents.
// Bound by the serial chains of a workgroup.  Groups of two bins when the
// batch leaves CUs idle, of five (fewer copies of (a)) otherwise.  Eight bins,
// 700 nodes, 4 walkers: 34 us; 214 us with the library's pow, shuffled scans,
// three evaluations per interval and one workgroup per walker.

// Inclusive prefix sums over the block of NV per-thread values (buf: NV x 4).
template <int NV>
__device__ __forceinline__ void block_prefix(double (&v)[NV], double* buf) {
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = wave_scan(v[q]);
    if (lane == 63)
#pragma unroll
        for (int q = 0; q < NV; ++q) buf[q * 4 + wid] = v[q];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double pre = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k < wid) pre += buf[q * 4 + k];
        v[q] += pre;
    }
    __syncthreads();
}

struct Background { double f, g, E, dlnE[3]; };        // d ln E in the directions Om, w0, wa (0 in h)

template <int BPG>
__global__ __launch_bounds__(256) void shear_tangent_kernel(
    const double* __restrict__ theta, int64_t ld, int64_t B, ShearGeom G, const int* __restrict__ pidx,
    const double* __restrict__ pfix, const double* __restrict__ nz_mean, const double* __restrict__ agrid,
    const double* __restrict__ lna, double* __restrict__ tg) {
    constexpr int NV = 4 * BPG;
    __shared__ double buf[(NV > 10 ? NV : 10) * 4];
    __shared__ double nodev[5][257];            // f, g, d ln E of the chunk's nodes
    __shared__ double red[2 * BPG][4];
    __shared__ double carry[10];                // forward prefix sums of the chunks before
    __shared__ double nrm[2 * BPG];             // N_i, dN_i
    __shared__ double gcs[2][NV];               // reverse sums of the chunks above
    __shared__ double gnx[2][NV];               // integrands of the node above the chunk
    __shared__ double xw[4][NV];                // wave-boundary exchange
    const int64_t w = blockIdx.x;
    if (w >= B) return;
    const int grp = blockIdx.y, b0 = grp * BPG;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int na = G.n_a, nb = G.n_bins, nch = (na + 255) / 256, cnt = min(BPG, nb - b0);
    const int X = TG_FIXED * gridDim.y, S = X + 7 * nb;
    auto fix = [&](int f, int j) -> double& { return tg[((int64_t)w * S + TG_FIXED * grp + f) * na + j]; };
    auto bin = [&](int f, int j) -> double& { return tg[((int64_t)w * S + X + f) * na + j]; };
    auto phys = [&](int slot) { const int ix = pidx[slot]; return ix >= 0 ? theta[w * ld + ix] : pfix[slot]; };
    const double ob = phys(0), oc = phys(1), h = phys(2), w0 = phys(5), wa = phys(6);
    const double Om = (ob + oc) / (h * h), iOm = 1.0 / Om, ih = 1.0 / h;
    const double cH0 = C_KM_S / (100.0 * h), H0c = 1.0 / cH0;
    const double pde = -3.0 * (1.0 + w0 + wa);
    const double is2 = 1.0 / (G.nz_sigma * G.nz_sigma);
    // f = cH0/(a^2 E), g = (Om a^-3/E^2)^0.55 / a (when wanted) at scale factor a
    auto bg = [&](double a, double la, bool want_g) {
        Background r;
        const double ia = 1.0 / a, ia2 = ia * ia, ia3 = ia2 * ia;
        const double Xde = exp_of(pde * la - 3.0 * wa * (1.0 - a));
        const double E2 = Om * ia3 + (1.0 - Om) * Xde, i2 = 0.5 / E2;
        r.E = sqrt(E2);
        r.f = cH0 * ia2 / r.E;
        r.g = want_g ? exp_of(GROWTH_INDEX * log(Om * ia3 / E2)) * ia : 0.0;
        const double q = (1.0 - Om) * Xde * i2;
        r.dlnE[0] = (ia3 - Xde) * i2;
        r.dlnE[1] = q * (-3.0 * la);
        r.dlnE[2] = q * (-3.0 * la - 3.0 * (1.0 - a));
        return r;
    };
    // the ten quantities of (a): f, g, df(4), dg(4)
    auto ten = [&](double f, double g, const double* dl, double (&o)[10]) {
        const double dlnE[4] = {dl[0], 0.0, dl[1], dl[2]};
        o[0] = f;
        o[1] = g;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            o[2 + q] = -f * dlnE[q];
            o[6 + q] = -2.0 * GROWTH_INDEX * g * dlnE[q];
        }
        o[3] -= f * ih;
        o[6] += GROWTH_INDEX * g * iOm;
    };

    // (a) chi, ln D and tangents at every node
    if (t < 10) carry[t] = 0.0;
    if (t == 0) {
        fix(TG_CHI, 0) = fix(TG_LND, 0) = fix(TG_LCHI, 0) = 0.0;
        for (int q = 0; q < 4; ++q) fix(TG_DCHI + q, 0) = fix(TG_DLND + q, 0) = 0.0;
    }
    for (int c = 0; c < nch; ++c) {
        const int j = c * 256 + t;
        const bool seg = j < na - 1;
        auto put = [&](int place, int node) {
            if (node >= na) return;
            const Background b = bg(agrid[node], lna[node], true);
            nodev[0][place] = b.f;
            nodev[1][place] = b.g;
            for (int q = 0; q < 3; ++q) nodev[2 + q][place] = b.dlnE[q];
        };
        put(t, j);
        if (t == 255) put(256, j + 1);
        double inc[10] = {};
        double m10[10] = {};
        if (seg) {
            const Background b = bg(0.5 * (agrid[j] + agrid[j + 1]), lna[na + j], true);
            ten(b.f, b.g, b.dlnE, m10);
        }
        __syncthreads();
        if (seg) {
            double l10[10], r10[10];
            const double dl[3] = {nodev[2][t], nodev[3][t], nodev[4][t]};
            const double dr[3] = {nodev[2][t + 1], nodev[3][t + 1], nodev[4][t + 1]};
            ten(nodev[0][t], nodev[1][t], dl, l10);
            ten(nodev[0][t + 1], nodev[1][t + 1], dr, r10);
#pragma unroll
            for (int q = 0; q < 10; ++q) inc[q] = G.da / 6.0 * (l10[q] + 4.0 * m10[q] + r10[q]);
        }
        block_prefix<10>(inc, buf);
        if (seg) {                               // sums over intervals 0..j: values at node j + 1
            const double chi = carry[0] + inc[0];
            fix(TG_CHI, j + 1) = chi;
            fix(TG_LCHI, j + 1) = log10(chi);
            fix(TG_LND, j + 1) = -(carry[1] + inc[1]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                fix(TG_DCHI + q, j + 1) = carry[2 + q] + inc[2 + q];
                fix(TG_DLND + q, j + 1) = -(carry[6 + q] + inc[6 + q]);
            }
        }
        __syncthreads();
        if (t == 255)
#pragma unroll
            for (int q = 0; q < 10; ++q) carry[q] += inc[q];
    }

    // (b) normalisations of n_i(z) and their Dz tangents
    double mu[BPG], A[BPG];
#pragma unroll
    for (int cc = 0; cc < BPG; ++cc) {
        const int i = min(b0 + cc, nb - 1);
        mu[cc] = nz_mean[i] + phys(9 + nb + i);
        A[cc] = phys(9 + i);
    }
    {
        double sn[BPG] = {}, sd[BPG] = {};
        for (int c = 0; c < nch; ++c) {
            const int j = c * 256 + t;
            if (j <= 0 || j >= na) continue;
            const double ia = 1.0 / agrid[j], z = ia - 1.0;
            const double qw = (j == na - 1 ? 0.5 * G.da : G.da) * ia * ia;
#pragma unroll
            for (int cc = 0; cc < BPG; ++cc) {
                const double dz = z - mu[cc];
                const double raw = qw * exp_of(-0.5 * is2 * dz * dz);
                sn[cc] += raw;
                sd[cc] += raw * dz * is2;
            }
        }
#pragma unroll
        for (int cc = 0; cc < BPG; ++cc) {
            const double v0 = wave_total(sn[cc]), v1 = wave_total(sd[cc]);
            if (lane == 0) { red[2 * cc][wid] = v0; red[2 * cc + 1][wid] = v1; }
        }
        if (t < 2 * NV) { gcs[t / NV][t % NV] = 0.0; gnx[t / NV][t % NV] = 0.0; }
        __syncthreads();
        if (t < 2 * BPG) nrm[t] = red[t][0] + red[t][1] + red[t][2] + red[t][3];
        __syncthreads();
    }
    double iN[BPG], dlnN[BPG];
#pragma unroll
    for (int cc = 0; cc < BPG; ++cc) {
        iN[cc] = 1.0 / nrm[2 * cc];
        dlnN[cc] = nrm[2 * cc + 1] * iN[cc];
    }

    // (c) reverse pass: G sums, windows and tangents
    const double pref = 1.5 * Om * H0c * H0c;
    const double dpref[4] = {pref * iOm, 2.0 * pref * ih, 0.0, 0.0};
    for (int c = nch - 1; c >= 0; --c) {
        const int j = c * 256 + 255 - t;
        const bool node = j < na, live = node && j > 0, has = node && j < na - 1;
        const int jj = node ? j : 0;
        const double a = node ? agrid[j] : 1.0, ia = 1.0 / a, ia2 = ia * ia, z = ia - 1.0;
        const double chi = fix(TG_CHI, jj), ichi = live ? 1.0 / chi : 0.0;
        double dchi[4], dlnD[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dchi[q] = fix(TG_DCHI + q, jj);
            dlnD[q] = fix(TG_DLND + q, jj);
        }
        const double iD = exp_of(-fix(TG_LND, jj));
        const Background eb = bg(a, lna[jj], false);
        const double E = eb.E;
        const double dlnE[4] = {eb.dlnE[0], 0.0, eb.dlnE[1], eb.dlnE[2]};
        const double dlnf[4] = {-dlnE[0], -ih, -dlnE[2], -dlnE[3]};
        const double qw = (j == 0 || j == na - 1) ? 0.5 * G.da : G.da;
        if (node) {
            const double wq = qw * eb.f * ichi * ichi;
            fix(TG_WQ, j) = wq;
#pragma unroll
            for (int q = 0; q < 4; ++q) fix(TG_DWQ + q, j) = wq * (dlnf[q] - 2.0 * dchi[q] * ichi);
        }
        double n[BPG], dn[BPG];
#pragma unroll
        for (int cc = 0; cc < BPG; ++cc) {
            const double dz = z - mu[cc];
            n[cc] = live && cc < cnt ? exp_of(-0.5 * is2 * dz * dz) * iN[cc] : 0.0;
            dn[cc] = n[cc] * (dz * is2 - dlnN[cc]);
        }
        double Gs[NV], Gc[NV];
#pragma unroll
        for (int sc = 0; sc < 2; ++sc) {
            double v[NV];
#pragma unroll
            for (int cc = 0; cc < BPG; ++cc) {
                if (sc == 0) {
                    v[cc] = n[cc] * ia2;
                    v[BPG + cc] = n[cc] * ia2 * ichi;
                    v[2 * BPG + cc] = dn[cc] * ia2;
                    v[3 * BPG + cc] = dn[cc] * ia2 * ichi;
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[4 * cc + q] = -n[cc] * dchi[q] * ia2 * ichi * ichi;
                }
            }
            if (lane == 63)
#pragma unroll
                for (int k = 0; k < NV; ++k) xw[wid][k] = v[k];
            __syncthreads();
            double sg[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                double nv = __shfl_up(v[k], 1, 64);              // the node above: the thread before
                if (lane == 0) nv = wid > 0 ? xw[wid - 1][k] : gnx[sc][k];
                sg[k] = has ? 0.5 * G.da * (v[k] + nv) : 0.0;
            }
            __syncthreads();
            if (t == 255)
#pragma unroll
                for (int k = 0; k < NV; ++k) gnx[sc][k] = v[k];
            block_prefix<NV>(sg, buf);
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                sg[k] += gcs[sc][k];
                if (sc == 0) Gs[k] = sg[k];
                else Gc[k] = sg[k];
            }
            __syncthreads();
            if (t == 255)
#pragma unroll
                for (int k = 0; k < NV; ++k) gcs[sc][k] = sg[k];
        }
        if (node) {
#pragma unroll
            for (int cc = 0; cc < BPG; ++cc) {
                if (cc >= cnt) break;
                const int i = b0 + cc;
                const double G0 = Gs[cc], G1 = Gs[BPG + cc], G0z = Gs[2 * BPG + cc], G1z = Gs[3 * BPG + cc];
                const double Q = G0 - chi * G1;
                const double base = C1_RHOCR * Om * H0c * E * iD;     // W^I = -A n base
                const double WI = -A[cc] * n[cc] * base;
                bin(i, j) = pref * chi * ia * Q + WI;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double dQ = -dchi[q] * G1 - chi * Gc[4 * cc + q];
                    const double dWg = dpref[q] * chi * ia * Q + pref * dchi[q] * ia * Q + pref * chi * ia * dQ;
                    double dlnbase = dlnE[q] - dlnD[q];
                    if (q == 0) dlnbase += iOm;
                    if (q == 1) dlnbase += ih;
                    bin(nb + 4 * i + q, j) = dWg + WI * dlnbase;
                }
                bin(5 * nb + i, j) = pref * chi * ia * (G0z - chi * G1z) - A[cc] * dn[cc] * base;
                bin(6 * nb + i, j) = -n[cc] * base;
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------------- Limber adjoint
constexpr int FX_BITS = 45;
constexpr int LA_PART = 4 + 2 * MAXB;                  // sums per node chunk: directions, Dz_i, A_IA,i

// log10 k of a multipole at a node (log10(l + 1/2) - log10 chi) -> Catmull-Rom
// interval i0, its offset tt and the ghost flags at the ends of the k grid
// (one definition for both passes of the Limber adjoint)
struct KPos { int i0; double tt; bool lo_ghost, hi_ghost; };
__device__ __forceinline__ KPos k_position(double lk, const ShearGeom& G) {
    const double s = (lk - G.u0) / G.du;
    int i0 = (int)floor(s);
    i0 = i0 < 0 ? 0 : (i0 > G.n_k - 2 ? G.n_k - 2 : i0);
    return KPos{i0, s - i0, i0 == 0, i0 + 2 >= G.n_k};
}

// One workgroup per (walker, 64 nodes): lane = a-node j, wave = every fourth
// multipole.  g(P wq), g W_i(j), g wq_j and g chi_j (through k = (l+1/2)/chi_j)
// from the Limber sums: with H_ac = g_C (1 + m_a)(1 + m_c), twice that for
// a = c, v_a = sum_c H_ac W_c gives both g W_a = Pw v_a and g(P wq) =
// (1/2) sum_a W_a v_a.  g log10 P_bj goes to glp [B x n_ell x n_a] (every
// entry written; limber_scatter_kernel sums them into the tables g Y, g M)
// and the high word of the chunk's largest magnitude to gmx; the node terms,
// added over the four waves, are contracted with the tangents of
// shear_tangent_kernel into the chunk's sums part [B x chunks x LA_PART].
// NB: bins, padded to even.  Bound by FP64 issue and the table gathers'
// latency: 4 walkers of eight bins and 700 nodes 20 us, 512 walkers of five
// bins and 256 nodes 45 us (508 and 174 us with one workgroup per walker, its
// 256-node chunks in turn, run-time bin counts, so arrays in scratch memory,
// and a logarithm per lookup).
template <class T, bool LINZ, int NB>
__global__ __launch_bounds__(256) void limber_adjoint_kernel(
    const double* __restrict__ theta, int64_t ld, int64_t B, ShearGeom G, int n_grp, const int* __restrict__ pidx,
    const double* __restrict__ pfix, const int* __restrict__ zidx, const double* __restrict__ zcoef,
    const double* __restrict__ lell, const T* __restrict__ Ytab, const T* __restrict__ Mtab,
    const double* __restrict__ gC, const double* __restrict__ tg, double* __restrict__ glp_buf,
    int* __restrict__ gmx_out, double* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) double Hs[32 * NB * NB];   // [multipole][a][c]
    __shared__ double gsum[4][NB + 2][64];
    __shared__ double m1[NB];
    __shared__ int gmx[4];
    const int64_t w = blockIdx.x;
    if (w >= B) return;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int na = G.n_a, nb = G.n_bins, ne = G.n_ell, nout = G.n_pairs * ne;
    const int X = TG_FIXED * n_grp, S = X + 7 * nb;
    auto phys = [&](int slot) { const int ix = pidx[slot]; return ix >= 0 ? theta[w * ld + ix] : pfix[slot]; };
    const int j = blockIdx.y * 64 + lane;
    const bool node = j < na, live = node && j > 0;
    const int jj = node ? j : 0;
    const double* rec = tg + (int64_t)w * S * na + jj;                 // field f of this lane's node at rec[f na]
    if (t < NB) m1[t] = t < nb ? 1.0 + phys(9 + 2 * nb + t) : 0.0;
    __syncthreads();
    for (int e = t; e < ne * NB * NB; e += 256) {
        const int b = e / (NB * NB), a = e / NB % NB, c = e % NB;
        double v = 0.0;
        if (a < nb && c < nb) {
            const int lo = min(a, c), hi = max(a, c), p = lo * nb - lo * (lo - 1) / 2 + hi - lo;
            v = gC[w * nout + (int64_t)p * ne + b] * m1[a] * m1[c];
            if (a == c) v *= 2.0;
        }
        Hs[e] = v;
    }
    double W[NB], gW[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        W[i] = i < nb ? rec[(int64_t)(X + i) * na] : 0.0;
        gW[i] = 0.0;
    }
    const double chi = rec[(int64_t)TG_CHI * na], lchi = rec[(int64_t)TG_LCHI * na], wq = rec[(int64_t)TG_WQ * na];
    const double kchi = live ? -1.0 / (G.du * chi) : 0.0;
    double gwq = 0.0, gchi = 0.0;
    const int nn = zidx[jj];
    const double c0 = zcoef[4 * jj], c1 = zcoef[4 * jj + 1];
    const double c2 = LINZ ? 0.0 : zcoef[4 * jj + 2], c3 = LINZ ? 0.0 : zcoef[4 * jj + 3];
    const T* y0 = Ytab + (w * (int64_t)G.n_z + nn) * G.n_k;
    const T* mm0 = LINZ ? y0 : Mtab + (w * (int64_t)G.n_z + nn) * G.n_k;
    double* glw = glp_buf + w * (int64_t)ne * na;
    int gmax = 0;
    __syncthreads();
    // log10 P at z_j from rows nn, nn + 1 of Y (and of M for cubic z)
    auto zmix = [&](T ya, T yb, T ma, T mb) {
        if (LINZ) return c0 * (double)ya + c1 * (double)yb;
        return c0 * (double)ya + c1 * (double)yb + c2 * (double)ma + c3 * (double)mb;
    };
    auto Yz = [&](int col) {
        return zmix(y0[col], y0[col + G.n_k], LINZ ? T(0) : mm0[col], LINZ ? T(0) : mm0[col + G.n_k]);
    };
    for (int b = wid; b < ne; b += 4) {
        const double lk = lell[b] - lchi;
        double glp = 0.0;
        if (live && lk >= G.u0 && lk <= G.u1) {
            const KPos kp = k_position(lk, G);
            const int i0 = kp.i0;
            const double tt = kp.tt;
            double pm, p0, p1, p2;
            if (!kp.lo_ghost && !kp.hi_ghost) {
                // columns i0 - 1 .. i0 + 2 of each row in one (element-aligned) vector load
                struct Q4 { T v[4]; };
                auto row4 = [&](const T* q) { Q4 r; __builtin_memcpy(&r, q, sizeof(r)); return r; };
                const Q4 ya = row4(y0 + i0 - 1), yb = row4(y0 + G.n_k + i0 - 1);
                Q4 ma = {}, mb = {};
                if (!LINZ) {
                    ma = row4(mm0 + i0 - 1);
                    mb = row4(mm0 + G.n_k + i0 - 1);
                }
                pm = zmix(ya.v[0], yb.v[0], ma.v[0], mb.v[0]);
                p0 = zmix(ya.v[1], yb.v[1], ma.v[1], mb.v[1]);
                p1 = zmix(ya.v[2], yb.v[2], ma.v[2], mb.v[2]);
                p2 = zmix(ya.v[3], yb.v[3], ma.v[3], mb.v[3]);
            } else {
                p0 = Yz(i0);
                p1 = Yz(i0 + 1);
                pm = kp.lo_ghost ? 2.0 * p0 - p1 : Yz(i0 - 1);
                p2 = kp.hi_ghost ? 2.0 * p1 - p0 : Yz(i0 + 2);
            }
            const double k0 = 0.5 * (p1 - pm), k1 = 0.5 * (p2 - p0);
            const double t2 = tt * tt, t3 = t2 * tt;
            const double lp = (2 * t3 - 3 * t2 + 1) * p0 + (t3 - 2 * t2 + tt) * k0 + (-2 * t3 + 3 * t2) * p1 +
                              (t3 - t2) * k1;
            const double dlp_dt = (6 * t2 - 6 * tt) * p0 + (3 * t2 - 4 * tt + 1) * k0 + (-6 * t2 + 6 * tt) * p1 +
                                  (3 * t2 - 2 * tt) * k1;
            const double P = exp10_of<double>(lp);
            const double Pw = P * wq;
            const double* H = Hs + b * NB * NB;
            double gPw = 0.0;
#pragma unroll
            for (int a = 0; a < NB; ++a) {
                double v = 0.0;
#pragma unroll
                for (int c = 0; c < NB; ++c) v = fma(H[a * NB + c], W[c], v);
                gPw = fma(W[a], v, gPw);
                gW[a] = fma(Pw, v, gW[a]);
            }
            gPw *= 0.5;
            gwq += gPw * P;
            const double gP = gPw * wq;
            gchi += gP * P * dlp_dt * kchi;
            glp = gP * P * LN10;
        }
        if (node) glw[(int64_t)b * na + j] = glp;
        gmax = max(gmax, __double2hiint(glp) & 0x7fffffff);             // as integers: a NaN is the largest
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) gsum[wid][i][lane] = gW[i];
    gsum[wid][NB][lane] = gwq;
    gsum[wid][NB + 1][lane] = gchi;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) gmax = max(gmax, __shfl_xor(gmax, o, 64));
    if (lane == 0) gmx[wid] = gmax;
    __syncthreads();
    for (int i = wid; i < NB + 2; i += 4)
        gsum[0][i][lane] = gsum[0][i][lane] + gsum[1][i][lane] + gsum[2][i][lane] + gsum[3][i][lane];
    __syncthreads();
    if (t == 0) gmx_out[w * gridDim.y + blockIdx.y] = max(max(gmx[0], gmx[1]), max(gmx[2], gmx[3]));
    // contract with the tangents of the nodes
    double* out = part + (w * gridDim.y + blockIdx.y) * LA_PART;
    for (int q = wid; q < 4 + 2 * nb; q += 4) {
        double v = 0.0;
        if (live) {
            if (q < 4) {
                v = gsum[0][NB][lane] * rec[(int64_t)(TG_DWQ + q) * na] + gsum[0][NB + 1][lane] * rec[(int64_t)(TG_DCHI + q) * na];
#pragma unroll
                for (int i = 0; i < NB; ++i)
                    if (i < nb) v += gsum[0][i][lane] * rec[(int64_t)(X + nb + 4 * i + q) * na];
            } else {
                const int i = (q - 4) % nb;
                v = gsum[0][i][lane] * rec[(int64_t)(X + (q - 4 < nb ? 5 : 6) * nb + i) * na];
            }
        }
        v = wave_total(v);
        if (lane == 0) out[q] = v;
    }
}

// Fixed-point grid step of a walker from its chunks' largest |g log10 P| (high
// words): 2^(e - FX_BITS) with all below 2^e; NaN if one is not finite.
__device__ __forceinline__ double grid_step(const int* gmx, int n) {
    int m = 0;
    for (int c = threadIdx.x & 63; c < n; c += 64) m = max(m, gmx[c]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
    if (m >= 0x7ff00000) return __longlong_as_double(0x7ff8000000000000ll);
    return m == 0 ? ldexp(1.0, -FX_BITS) : ldexp(1.0, max((m >> 20) - 1022, -900) - FX_BITS);  // 1 / step stays finite
}

// Fixed-point scatter of g log10 P_bj (limber_adjoint_kernel's glp_buf, grid
// step from its gmx) into the tables gY (and gM for the cubic z-spline), one
// workgroup per (walker, slab).  Slab s = (first node, end node, first row,
// last row) of `slabs`: the z rows partitioned into runs, each with the nodes
// whose two rows meet it.  A slab adds the contributions of its nodes to its own rows
// only, as integers in LDS (atomics); every row's sum is then complete, and
// the slab writes its rows as doubles (integer x grid step, 2^-mshift finer
// for gM).  Every entry of the walker's tables is written.  A walker whose
// grid step is NaN (a non-finite gradient) gets NaN tables.
// SC_THREADS: a slab at low redshift holds most nodes, and each of its terms
// waits for a chain of loads (few walkers: 18 us, with 256 threads 29; 512
// walkers of 64 rows: 74 against 85).
constexpr int SC_THREADS = 1024;
template <bool LINZ>
__global__ __launch_bounds__(SC_THREADS) void limber_scatter_kernel(
    int64_t B, ShearGeom G, int n_grp, const int* __restrict__ zidx, const double* __restrict__ zcoef,
    const double* __restrict__ lell, const double* __restrict__ tg, const double* __restrict__ glp_buf,
    const int4* __restrict__ slabs, int rmax, const int* __restrict__ gmx, int n_chunk, int mshift,
    double* __restrict__ gY, double* __restrict__ gM) {
    extern __shared__ unsigned long long sl[];          // [tables][rmax][n_k]
    const int64_t w = blockIdx.x;
    if (w >= B) return;
    const int t = threadIdx.x;
    const int na = G.n_a, ne = G.n_ell, nk = G.n_k, nz = G.n_z;
    const int S = TG_FIXED * n_grp + 7 * G.n_bins;
    const double step = grid_step(gmx + w * n_chunk, n_chunk);
    const bool ok = !isnan(step);
    const double scale = 1.0 / step, mscale = ldexp(scale, mshift);     // powers of two: exact
    const double mstep = ldexp(step, -mshift);
    const int tab = rmax * nk;
    double* gYw = gY + w * (int64_t)nz * nk;
    double* gMw = LINZ ? gYw : gM + w * (int64_t)nz * nk;
    const double* glw = glp_buf + w * (int64_t)ne * na;
    const double* lchiw = tg + ((int64_t)w * S + TG_LCHI) * na;
    auto fx_add = [&](unsigned long long* p, double v, double sc) {
        if (v != 0.0) atomicAdd(p, (unsigned long long)llrint(v * sc));
    };
    {
        const int4 sb = slabs[blockIdx.y];
        const int lo = sb.z, nr = sb.w - sb.z + 1, nj = sb.y - sb.x;
        for (int e = t; e < nr * nk; e += SC_THREADS) {
            sl[e] = 0ull;
            if (!LINZ) sl[tab + e] = 0ull;
        }
        __syncthreads();
        if (ok)
            for (int it = t; it < nj * ne; it += SC_THREADS) {
                const int j = sb.x + it % nj, b = it / nj;
                const double glp = glw[(int64_t)b * na + j];
                if (glp == 0.0) continue;                    // as outside the emulated k range
                // the node's rows zi[j], zi[j] + 1 as rows of this slab (either may lie outside it)
                const int r0 = zidx[j] - lo, r1 = r0 + 1;
                const bool in0 = r0 >= 0, in1 = r1 < nr;
                const double c0 = zcoef[4 * j], c1 = zcoef[4 * j + 1];
                const double c2 = LINZ ? 0.0 : zcoef[4 * j + 2], c3 = LINZ ? 0.0 : zcoef[4 * j + 3];
                const KPos kp = k_position(lell[b] - lchiw[j], G);
                const double tt = kp.tt, t2 = tt * tt, t3 = t2 * tt;
                const double h00 = 2 * t3 - 3 * t2 + 1, h10 = t3 - 2 * t2 + tt, h01 = -2 * t3 + 3 * t2,
                             h11 = t3 - t2;
                // d lp / d (pm, p0, p1, p2), ghosts folded into the real columns
                double wm = -0.5 * h10, w0c = h00 - 0.5 * h11, w1c = h01 + 0.5 * h10, w2 = 0.5 * h11;
                if (kp.lo_ghost) { w0c += 2.0 * wm; w1c -= wm; wm = 0.0; }
                if (kp.hi_ghost) { w1c += 2.0 * w2; w0c -= w2; w2 = 0.0; }
                auto scatter = [&](int col, double wgt) {
                    const double gy = glp * wgt;
                    if (in0) {
                        fx_add(&sl[r0 * nk + col], c0 * gy, scale);
                        if (!LINZ) fx_add(&sl[tab + r0 * nk + col], c2 * gy, mscale);
                    }
                    if (in1) {
                        fx_add(&sl[r1 * nk + col], c1 * gy, scale);
                        if (!LINZ) fx_add(&sl[tab + r1 * nk + col], c3 * gy, mscale);
                    }
                };
                if (!kp.lo_ghost) scatter(kp.i0 - 1, wm);
                scatter(kp.i0, w0c);
                scatter(kp.i0 + 1, w1c);
                if (!kp.hi_ghost) scatter(kp.i0 + 2, w2);
            }
        __syncthreads();
        const int64_t g0 = (int64_t)lo * nk;
        for (int e = t; e < nr * nk; e += SC_THREADS) {
            gYw[g0 + e] = ok ? (double)(long long)sl[e] * step : NAN;
            if (!LINZ) gMw[g0 + e] = ok ? (double)(long long)sl[tab + e] * mstep : NAN;
        }
    }
}

// ------------------------------------------------------------ spline adjoint
// gY, gM (doubles, from limber_scatter_kernel): gY += S^T gM for the
// not-a-knot spline of each (walker, k) column, and
// delta_out[row = w n_z + n][c] = gY[n][c] sigma_out[c] (padded to n_pad).
template <class T>
__global__ __launch_bounds__(256) void zspline_adjoint_kernel(double* __restrict__ gY, double* __restrict__ gM,
                                                              int64_t B, int nz, int nk, double h,
                                                              const double* __restrict__ sigma_out, int n_pad,
                                                              T* __restrict__ delta) {
    __shared__ double cps[256];
    if (threadIdx.x == 0) {
        double c = 0.0;
        for (int n = 2; n <= nz - 3 && n < 256; ++n) {
            c = 1.0 / (4.0 - (n == 2 ? 0.0 : c));
            cps[n] = c;
        }
    }
    __syncthreads();
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= B * n_pad) return;
    const int64_t w = g / n_pad;
    const int c = (int)(g % n_pad);
    if (c >= nk) {
        for (int n = 0; n < nz; ++n) delta[(w * nz + n) * n_pad + c] = T(0);
        return;
    }
    double* gy = gY + w * nz * nk + c;
    double* gm = gM + w * nz * nk + c;
    auto Y = [&](int n) -> double& { return gy[(int64_t)n * nk]; };
    auto Mg = [&](int n) -> double& { return gm[(int64_t)n * nk]; };
    const double ih2 = 1.0 / (h * h);
    // M_0 = 2 M_1 - M_2 and M_{N-1} = 2 M_{N-2} - M_{N-3}: fold their adjoints
    // into the other nodes first (valid for every nz >= 4)
    const double g0 = Mg(0), gl = Mg(nz - 1);
    Mg(1) += 2.0 * g0;
    Mg(2) -= g0;
    Mg(nz - 2) += 2.0 * gl;
    Mg(nz - 3) -= gl;
    double gM1 = Mg(1);
    double gMb = Mg(nz - 2);
    if (nz > 4) {
        // interior (1,4,1) system is symmetric: g_rhs = T^{-1} gM_interior (same Thomas sweep)
        double dp = 0.0;
        for (int n = 2; n <= nz - 3; ++n) {
            dp = (Mg(n) - (n == 2 ? 0.0 : dp)) * cps[n];
            Mg(n) = dp;
        }
        double next = dp;
        for (int n = nz - 4; n >= 2; --n) {
            next = Mg(n) - cps[n] * next;
            Mg(n) = next;
        }
        // rhs_n = 6 d2Y_n / h^2 - [n == 2] M_1 - [n == nz-3] M_{N-2}
        gM1 -= Mg(2);
        gMb -= Mg(nz - 3);
        for (int n = 2; n <= nz - 3; ++n) {
            const double gr = 6.0 * ih2 * Mg(n);
            Y(n + 1) += gr;
            Y(n) -= 2.0 * gr;
            Y(n - 1) += gr;
        }
    }
    // M_1 = d2Y_1 / h^2, M_{N-2} = d2Y_{N-2} / h^2
    Y(2) += gM1 * ih2; Y(1) -= 2.0 * gM1 * ih2; Y(0) += gM1 * ih2;
    Y(nz - 1) += gMb * ih2; Y(nz - 2) -= 2.0 * gMb * ih2; Y(nz - 3) += gMb * ih2;
    const double sg = sigma_out[c];
    for (int n = 0; n < nz; ++n) delta[(w * nz + n) * n_pad + c] = (T)(Y(n) * sg);
}

// The same for 4 <= n_z <= NZ with the column of g M in registers: both tables
// are read once and only delta is written (the kernel above sweeps over memory).
// The tridiagonal system's ratios are compile-time constants, and the end rows'
// second differences are those of entries 1 and n_z - 2 of one vector g with
// delta_n = g Y_n + g_{n-1} - 2 g_n + g_{n+1}.  512 walkers of 64 rows: 117 us,
// swept 253; its bytes alone take 67 at the rate of a large copy.
struct SplineRatios {                           // c_2 = 1/4, c_n = 1 / (4 - c_{n-1})
    double c[64];
    constexpr SplineRatios() : c{} {
        double v = 0.0;
        for (int n = 2; n < 64; ++n) c[n] = v = 1.0 / (4.0 - v);
    }
};
template <class T, int NZ>
__global__ __launch_bounds__(256) void zspline_adjoint_reg_kernel(const double* __restrict__ gY,
                                                                  const double* __restrict__ gM, int64_t B, int nz,
                                                                  int nk, double h,
                                                                  const double* __restrict__ sigma_out, int n_pad,
                                                                  T* __restrict__ delta) {
    constexpr SplineRatios R{};
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= B * n_pad) return;
    const int64_t w = g / n_pad;
    const int c = (int)(g % n_pad);
    T* out = delta + w * nz * n_pad + c;
    if (c >= nk) {
        for (int n = 0; n < nz; ++n) out[(int64_t)n * n_pad] = T(0);
        return;
    }
    const double* gm = gM + w * nz * nk + c;
    const double* gy = gY + w * nz * nk + c;
    // the last row's index, opaque so that the loops' comparisons are not kept
    // across them (hundreds of scalar registers)
    auto last = [&]() {
        int v = nz - 1;
        asm volatile("" : "+s"(v));
        return v;
    };
    const double ih2 = 1.0 / (h * h), sg = sigma_out[c];
    // M_0 = 2 M_1 - M_2 and M_{N-1} = 2 M_{N-2} - M_{N-3}, folded into the other nodes
    const double m0 = gm[0], ml = gm[(int64_t)(nz - 1) * nk];
    double gM1 = gm[nk] + 2.0 * m0, gMb = gm[(int64_t)(nz - 2) * nk] + 2.0 * ml;
    if (nz == 4) {
        gM1 -= ml;
        gMb -= m0;
    }
    double m[NZ];
    {
        const int e = last();
#pragma unroll
        for (int n = 2; n < NZ - 2; ++n) m[n] = n <= e - 2 ? gm[(int64_t)n * nk] : 0.0;
    }
    m[2] -= nz > 4 ? m0 : 0.0;
    // the symmetric interior system (1, 4, 1): g_rhs, times 6 / h^2, in m[2 .. nz-3]
    // (rows above with ratio and value 0)
    {
        const int e = last();
        double dp = 0.0;
#pragma unroll
        for (int n = 2; n < NZ - 2; ++n) {
            const bool end = n == e - 2;
            dp = (m[n] - (end ? ml : 0.0) - dp) * (n <= e - 2 ? R.c[n] : 0.0);
            m[n] = dp;
            gMb -= end ? dp : 0.0;
        }
    }
    {
        const int e = last();
        double next = 0.0;
#pragma unroll
        for (int n = NZ - 3; n >= 2; --n) {
            next = m[n] - (n <= e - 2 ? R.c[n] : 0.0) * next;
            m[n] = 6.0 * ih2 * next;
        }
        gM1 -= next;
    }
    const double e1 = gM1 * ih2, eb = gMb * ih2;
    const int e = last();
    double below = 0.0, here = 0.0;
#pragma unroll
    for (int n = 0; n < NZ; ++n) {
        const double inner = n == 0 ? e1 : n < NZ - 3 ? m[n < NZ - 3 ? n + 1 : 0] : 0.0;
        const double above = n + 2 == e ? eb : inner;          // entry n + 1 of g
        if (n <= e) {
            const double v = gy[(int64_t)n * nk] + (below - 2.0 * here + above);
            out[(int64_t)n * n_pad] = (T)(v * sg);
        }
        below = here;
        here = above;
    }
}

// Linear z: delta = g Y sigma_out, entry by entry.
template <class T>
__global__ __launch_bounds__(256) void zlinear_adjoint_kernel(const double* __restrict__ gY, int64_t rows, int nk,
                                                              const double* __restrict__ sigma_out, int n_pad,
                                                              T* __restrict__ delta) {
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    for (int c = threadIdx.x & 63; c < n_pad; c += 64)
        delta[r * n_pad + c] = c < nk ? (T)(gY[r * nk + c] * sigma_out[c]) : T(0);
}

// Gradient of a walker (one workgroup): the emulator's input gradients summed
// over its redshift rows, the direct terms from the Limber adjoint's chunk
// sums, and the multiplicative biases dC_pb/dm_i = C_pb [(i==a) + (i==b)] /
// (1 + m_i).  Sums in fixed strided parts, so repeated calls agree bitwise.
__global__ __launch_bounds__(256) void shear_assemble_kernel(
    const double* __restrict__ theta, int64_t ld, int d, ShearGeom G, const int* __restrict__ pidx,
    const double* __restrict__ pfix, const int* __restrict__ src, int n_in, const double* __restrict__ gx,
    const double* __restrict__ part, int n_chunk, const double* __restrict__ gC, const double* __restrict__ Cv,
    const double* __restrict__ logl, double* __restrict__ grad) {
    __shared__ double em[16][17];
    __shared__ double tot[LA_PART], mb[MAXB];
    __shared__ double gd[64];
    const int64_t w = blockIdx.x;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int nb = G.n_bins, ne = G.n_ell, nout = G.n_pairs * ne, nz = G.n_z;
    auto phys = [&](int slot) { const int ix = pidx[slot]; return ix >= 0 ? theta[w * ld + ix] : pfix[slot]; };
    {
        const int k = t & 15, z0 = t >> 4;                 // input k, rows z0, z0 + 16, ...
        double v = 0.0;
        if (k < n_in)
            for (int z = z0; z < nz; z += 16) v += gx[((int64_t)w * nz + z) * n_in + k];
        em[z0][k] = v;
    }
    if (t < 4 + 2 * nb) {
        double v = 0.0;
        for (int c = 0; c < n_chunk; ++c) v += part[((int64_t)w * n_chunk + c) * LA_PART + t];
        tot[t] = v;
    }
    for (int i = wid; i < nb; i += 4) {
        double v = 0.0;
        for (int c = 0; c < nb; ++c) {                     // pairs (i, c); twice for c = i
            const int lo = min(i, c), hi = max(i, c), p = lo * nb - lo * (lo - 1) / 2 + hi - lo;
            for (int b = lane; b < ne; b += 64) {
                const int64_t o = w * nout + (int64_t)p * ne + b;
                v += (c == i ? 2.0 : 1.0) * gC[o] * Cv[o];
            }
        }
        v = wave_total(v);
        if (lane == 0) mb[i] = v / (1.0 + phys(9 + 2 * nb + i));
    }
    if (t < 64) gd[t] = 0.0;
    __syncthreads();
    if (t < n_in) {
        double v = 0.0;
        for (int z = 0; z < 16; ++z) v += em[z][t];
        em[0][t] = v;
    }
    if (t == 64) {
        // (Om, h) -> (omega_b, omega_cdm, h)
        const double h = phys(2), Om = (phys(0) + phys(1)) / (h * h), dOm = tot[0];
        auto add = [&](int slot, double v) { if (pidx[slot] >= 0) gd[pidx[slot]] += v; };
        add(0, dOm / (h * h));
        add(1, dOm / (h * h));
        add(2, tot[1] - 2.0 * Om / h * dOm);
        add(5, tot[2]);
        add(6, tot[3]);
        for (int i = 0; i < nb; ++i) {
            add(9 + nb + i, tot[4 + i]);
            add(9 + i, tot[4 + nb + i]);
            add(9 + 2 * nb + i, mb[i]);
        }
    }
    __syncthreads();
    if (t < d) {
        double v = gd[t];
        for (int k = 0; k < n_in; ++k)
            if (src[k] == t) v += em[0][k];
        grad[w * d + t] = logl[w] == -INFINITY ? 0.0 : v;
    }
}

// ------------------------------------------------------------------ driver
void shear_grad(ns_model* m, const double* theta, int64_t ld, int64_t B, double* logl, double* grad, int prec,
                hipStream_t s) {
    const bool f64 = prec == NS_FP64, lin = m->z_linear;
    const size_t elem = f64 ? 8 : 4;
    const int nk = m->n_k, nz = m->n_z, n = m->n_data, d = m->d, na = m->n_a, nb = m->n_bins;
    const int64_t rows = B * nz;
    // forward: emulator table (with pre-activation saves), spline, spectra
    m->ws_out.ensure((size_t)B * nz * nk * elem);
    const int id0 = 0, no_log = 0;
    void* out0 = m->ws_out.p;
    emulator_forward(m, &id0, 1, theta, ld, B, &out0, nk, &no_log, prec, nullptr, s, true);
    const double* Cv = shear_spectra_from_table(m, theta, ld, B, prec, nullptr, s);
    const void* Mtab = m->ws_aux.p;
    // node chunks of the Limber adjoint, bin groups of the tangents: two bins
    // each while a workgroup per walker and five bins would leave CUs idle
    const int n_chunk = (na + 63) / 64;
    const int bpg = B * ((nb + 4) / 5) < 2 * (int64_t)device_cus(m->device) ? 2 : 5, n_grp = (nb + bpg - 1) / bpg;
    // adjoint scratch: gC, R [B n], chi^2 partial sums [n_ct B], gY (and gM) [B nz nk],
    // tangents [B S n_a], g log10 P [B n_ell n_a], chunk sums and maxima [B n_chunk]
    const size_t ntab = (size_t)B * nz * nk, n_ct = (n + 63) / 64;
    const size_t S = TG_FIXED * (size_t)n_grp + 7 * (size_t)nb;
    m->ws_grad.ensure(((size_t)B * (2 * n + n_ct) + (lin ? 1 : 2) * ntab + (size_t)B * S * na +
                       (size_t)B * m->n_ell * na + (size_t)B * n_chunk * (LA_PART + 1)) *
                      sizeof(double));
    double* gC = m->ws_grad.as<double>();
    double* R = gC + (size_t)B * n;
    double* part = R + (size_t)B * n;
    double* gY = part + (size_t)B * n_ct;
    double* gM = lin ? gY : gY + ntab;          // spline second derivatives: cubic z only
    double* tg = gY + (lin ? 1 : 2) * ntab;
    double* glp = tg + (size_t)B * S * na;
    double* sums = glp + (size_t)B * m->n_ell * na;
    int* gmx = reinterpret_cast<int*>(sums + (size_t)B * n_chunk * LA_PART);
    // finer fixed-point grid of g M: its coefficients are at most 0.385 h^2 / 6
    const double hz = (1.0 / m->a_min - 1.0) / (nz - 1);
    const int mshift = lin ? 0 : std::max(0, std::min(40, (int)std::floor(std::log2(6.0 / (0.385 * hz * hz)))));
    {
        TraceScope ts(m, s, "adj_dense_chi2");
        dense_chi2_adjoint(m, theta, ld, B, Cv, R, part, logl, gC, s);
    }
    const ShearGeom G = shear_geom(m);
    {
        TraceScope ts(m, s, "adj_tangents");
        const auto kern = bpg == 2 ? shear_tangent_kernel<2> : shear_tangent_kernel<5>;
        hipLaunchKernelGGL(kern, dim3((unsigned)B, (unsigned)n_grp), dim3(256), 0, s, theta, ld, B, G,
                           m->pidx_d.as<int>(), m->pfix_d.as<double>(), m->nz_mean_d.as<double>(),
                           m->agrid_d.as<double>(), m->lna_d.as<double>(), tg);
        NS_HIP(hipGetLastError());
    }
    {
        TraceScope ts(m, s, "adj_limber");
        auto launch = [&](auto kern, const auto* Y) {
            hipLaunchKernelGGL(kern, dim3((unsigned)B, (unsigned)n_chunk), dim3(256), 0, s, theta, ld, B, G, n_grp,
                               m->pidx_d.as<int>(), m->pfix_d.as<double>(), m->zsp_idx_d.as<int>(),
                               m->zsp_coef_d.as<double>(), m->lell_d.as<double>(), Y, (decltype(Y))Mtab, gC, tg, glp,
                               gmx, sums);
        };
        const bool few = nb <= 6;
        if (f64) {
            const double* Y = m->ws_out.as<double>();
            if (lin) few ? launch(limber_adjoint_kernel<double, true, 6>, Y) : launch(limber_adjoint_kernel<double, true, 10>, Y);
            else few ? launch(limber_adjoint_kernel<double, false, 6>, Y) : launch(limber_adjoint_kernel<double, false, 10>, Y);
        } else {
            const float* Y = m->ws_out.as<float>();
            if (lin) few ? launch(limber_adjoint_kernel<float, true, 6>, Y) : launch(limber_adjoint_kernel<float, true, 10>, Y);
            else few ? launch(limber_adjoint_kernel<float, false, 6>, Y) : launch(limber_adjoint_kernel<float, false, 10>, Y);
        }
        NS_HIP(hipGetLastError());
    }
    {
        TraceScope ts(m, s, "adj_limber_scatter");
        const size_t smem = (size_t)(lin ? 1 : 2) * m->lslab_rows * nk * sizeof(unsigned long long);
        const auto kern = lin ? limber_scatter_kernel<true> : limber_scatter_kernel<false>;
        if (smem > 64 * 1024)
            NS_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
        hipLaunchKernelGGL(kern, dim3((unsigned)B, (unsigned)m->n_lslab), dim3(SC_THREADS), smem, s, B, G, n_grp,
                           m->zsp_idx_d.as<int>(), m->zsp_coef_d.as<double>(), m->lell_d.as<double>(), tg, glp,
                           m->lslab_d.as<int4>(), m->lslab_rows, gmx, n_chunk, mshift, gY, gM);
        NS_HIP(hipGetLastError());
    }
    // spline adjoint -> delta for the emulator's raw outputs
    const Net& net = *m->nets[0];
    const int n_pad = net.layers[net.n_layers - 1]->n_pad;
    size_t max_w = 0;
    for (int l = 1; l < net.n_layers; ++l) max_w = std::max(max_w, (size_t)net.dims[l]);
    const size_t gstride = (size_t)rows * std::max(max_w, (size_t)n_pad);
    m->ws_gact[0].ensure(gstride * elem);
    m->ws_gact[1].ensure(gstride * elem);
    {
        TraceScope ts(m, s, "adj_zspline");
        const dim3 gz((unsigned)((B * n_pad + 255) / 256));
        const double* so = net.out_sigma64.as<double>();
        auto spline = [&](auto* delta) {
            using T = std::remove_pointer_t<decltype(delta)>;
            if (lin)
                hipLaunchKernelGGL(zlinear_adjoint_kernel<T>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, gY,
                                   rows, nk, so, n_pad, delta);
            else if (nz <= 16)
                hipLaunchKernelGGL((zspline_adjoint_reg_kernel<T, 16>), gz, dim3(256), 0, s, gY, gM, B, nz, nk, hz, so,
                                   n_pad, delta);
            else if (nz <= 32)
                hipLaunchKernelGGL((zspline_adjoint_reg_kernel<T, 32>), gz, dim3(256), 0, s, gY, gM, B, nz, nk, hz, so,
                                   n_pad, delta);
            else if (nz <= 64)
                hipLaunchKernelGGL((zspline_adjoint_reg_kernel<T, 64>), gz, dim3(256), 0, s, gY, gM, B, nz, nk, hz, so,
                                   n_pad, delta);
            else
                hipLaunchKernelGGL(zspline_adjoint_kernel<T>, gz, dim3(256), 0, s, gY, gM, B, nz, nk, hz, so, n_pad,
                                   delta);
        };
        if (f64) spline(m->ws_gact[0].as<double>());
        else spline(m->ws_gact[0].as<float>());
        NS_HIP(hipGetLastError());
    }
    emulator_backward(m, &id0, 1, B, f64 ? NS_FP64 : NS_FP32, s);
    TraceScope ts(m, s, "adj_assemble");
    hipLaunchKernelGGL(shear_assemble_kernel, dim3((unsigned)B), dim3(256), 0, s, theta, ld, d, G, m->pidx_d.as<int>(),
                       m->pfix_d.as<double>(), m->emu_src_d.as<int>(), net.dims[0], m->ws_gx.as<double>(), sums, n_chunk,
                       gC, Cv, logl, grad);
    NS_HIP(hipGetLastError());
}

}  // namespace nsmi
