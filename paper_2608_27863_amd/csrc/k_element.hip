// Element residuals and Jacobian blocks of the HDG discretisation.
//
// Two stages (the quadrature-point kernels feed the assembly kernel through a
// workspace, as in the paper's split of pointwise kernels and assembly
// kernels that look like batched linear algebra):
//   k_qp_volume / k_qp_face : interpolate (u, u^n, q, nu) to the Gauss points,
//       evaluate the fluxes of eqs. convective-flux, viscous-flux, stress-heat,
//       av-total and the numerical flux of eq. num-flux-hdg, and their exact
//       Jacobians (derived by hand below), already multiplied by quadrature
//       weights, the geometric factors and dt / alpha;
//   k_conserved_blocks, k_conserved_trace, k_grad_rows, k_trace_rows : contract the point
//       coefficients with the basis (phi_i, reference derivatives of phi_i,
//       phi_k, trace basis mu_a) into the rows of the element system
//       E^K = [[A B R_qu],[C D R_uh]], by sum factorisation over the tensor
//       Gauss points.  A chunk's systems (21.7 GB for 256 elements at p = 4) are
//       far larger than any cache: the gradient rows, most of them, are stored
//       nontemporally.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "hdg_internal.h"

namespace hdg {
namespace {

typedef double v2d __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------ physics
// Intermediates at one point for state w and conservative gradient q.
struct PState {
    double rho, v[3], E, mus, kap, dmus[5];
    double dv[3][3], dE[3], de[3], S[3][3];
    double vv;  // |v|^2
};

__device__ inline void pstate(const double *w, const double *q, const Phys &P, PState &s) {
    const double rho = w[0], ir = 1.0 / rho;
    s.rho = rho;
    for (int i = 0; i < 3; ++i) s.v[i] = w[1 + i] * ir;
    s.E = w[4] * ir;
    s.vv = s.v[0] * s.v[0] + s.v[1] * s.v[1] + s.v[2] * s.v[2];
    const double e = s.E - 0.5 * s.vv;
    const double cT = P.gamma * (P.gamma - 1.0) * P.mach * P.mach;
    double mu = 1.0, dmu = 0.0;
    if (P.visc_law == 1) {
        const double T = cT * e, sq = sqrt(T), den = 1.0 / (T + 0.40417);
        mu = 1.4042 * T * sq * den;
        // d/dT [c1 T^{3/2} / (T + c2)] = c1 sqrt(T) (T/2 + 3 c2 / 2) / (T + c2)^2
        dmu = 1.4042 * sq * (0.5 * T + 1.5 * 0.40417) * den * den;
    }
    s.mus = mu / P.reynolds;
    s.kap = P.gamma * s.mus / P.prandtl;
    // de/dw = ((|v|^2 - E)/rho, -v/rho, 1/rho)
    const double dedw[5] = {(s.vv - s.E) * ir, -s.v[0] * ir, -s.v[1] * ir, -s.v[2] * ir, ir};
    for (int c = 0; c < 5; ++c) s.dmus[c] = dmu * cT * dedw[c] / P.reynolds;
    for (int j = 0; j < 3; ++j) {
        for (int i = 0; i < 3; ++i) s.dv[i][j] = (q[3 * (1 + i) + j] - s.v[i] * q[j]) * ir;
        s.dE[j] = (q[12 + j] - s.E * q[j]) * ir;
        s.de[j] = s.dE[j] - (s.v[0] * s.dv[0][j] + s.v[1] * s.dv[1][j] + s.v[2] * s.dv[2][j]);
    }
    const double div = s.dv[0][0] + s.dv[1][1] + s.dv[2][2];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) s.S[i][j] = s.dv[i][j] + s.dv[j][i] - (i == j ? (2.0 / 3.0) * div : 0.0);
}

// F = F^c(w) - F^v(w, q) - nu q   (total flux entering the residuals)
__device__ inline void total_flux(const double *w, const double *q, double nu, const Phys &P,
                                  const PState &s, double F[5][3]) {
    const double p = (P.gamma - 1.0) * (w[4] - 0.5 * s.rho * s.vv);
    for (int j = 0; j < 3; ++j) {
        F[0][j] = w[1 + j];
        double tv = 0.0;
        for (int i = 0; i < 3; ++i) {
            const double tau = s.mus * s.S[i][j];
            F[1 + i][j] = w[1 + i] * s.v[j] + (i == j ? p : 0.0) - tau;
            tv += s.v[i] * tau;
        }
        F[4][j] = (w[4] + p) * s.v[j] - tv - s.kap * s.de[j];
        for (int c = 0; c < 5; ++c) F[c][j] -= nu * q[3 * c + j];
    }
}

// dF/dw_cp (q fixed) of F = F^c - F^v; nu q does not depend on w.
__device__ inline void dflux_dw(const double *w, const double *q, const Phys &P, const PState &s,
                                int cp, double dF[5][3]) {
    const double ir = 1.0 / s.rho, gm1 = P.gamma - 1.0;
    const double p = gm1 * (w[4] - 0.5 * s.rho * s.vv);
    double dp, dvel[3];
    if (cp == 0) {
        dp = gm1 * 0.5 * s.vv;
        for (int i = 0; i < 3; ++i) dvel[i] = -s.v[i] * ir;
    } else if (cp < 4) {
        dp = -gm1 * s.v[cp - 1];
        for (int i = 0; i < 3; ++i) dvel[i] = (i == cp - 1) ? ir : 0.0;
    } else {
        dp = gm1;
        for (int i = 0; i < 3; ++i) dvel[i] = 0.0;
    }
    // derivatives of the primitive gradients
    double ddv[3][3], ddE[3], dde[3];
    for (int j = 0; j < 3; ++j) {
        const double q0 = q[j];
        for (int i = 0; i < 3; ++i) {
            if (cp == 0) ddv[i][j] = (s.v[i] * q0 * ir - s.dv[i][j]) * ir;
            else if (cp == 1 + i) ddv[i][j] = -q0 * ir * ir;
            else ddv[i][j] = 0.0;
        }
        if (cp == 0) ddE[j] = (s.E * q0 * ir - s.dE[j]) * ir;
        else if (cp == 4) ddE[j] = -q0 * ir * ir;
        else ddE[j] = 0.0;
        dde[j] = ddE[j];
        for (int i = 0; i < 3; ++i) dde[j] -= dvel[i] * s.dv[i][j] + s.v[i] * ddv[i][j];
    }
    const double ddiv = ddv[0][0] + ddv[1][1] + ddv[2][2];
    const double dmus = s.dmus[cp], dkap = P.gamma * dmus / P.prandtl;
    for (int j = 0; j < 3; ++j) {
        // convective part
        dF[0][j] = (cp == 1 + j) ? 1.0 : 0.0;
        for (int i = 0; i < 3; ++i)
            dF[1 + i][j] = ((cp == 1 + i) ? s.v[j] : 0.0) + s.rho * s.v[i] * dvel[j] + (i == j ? dp : 0.0);
        dF[4][j] = ((cp == 4 ? 1.0 : 0.0) + dp) * s.v[j] + (w[4] + p) * dvel[j];
        // viscous part
        double dvt = 0.0;
        for (int i = 0; i < 3; ++i) {
            const double dS = ddv[i][j] + ddv[j][i] - (i == j ? (2.0 / 3.0) * ddiv : 0.0);
            const double dtau = dmus * s.S[i][j] + s.mus * dS;
            dF[1 + i][j] -= dtau;
            dvt += dvel[i] * s.mus * s.S[i][j] + s.v[i] * dtau;
        }
        dF[4][j] -= dvt + dkap * s.de[j] + s.kap * dde[j];
    }
}

// dF^v/dq_{cpp,l} including nu q (F^v is linear in q).
__device__ inline void dfv_dq(const PState &s, double nu, int cpp, int l, double dF[5][3]) {
    const double ir = 1.0 / s.rho;
    double b[3];
    for (int i = 0; i < 3; ++i) b[i] = (((cpp == 1 + i) ? 1.0 : 0.0) - (cpp == 0 ? s.v[i] : 0.0)) * ir;
    double a = 0.0;
    if (cpp == 4) a = ir;
    else if (cpp == 0) a = (s.vv - s.E) * ir;
    else a = -s.v[cpp - 1] * ir;
    const double vb = s.v[0] * b[0] + s.v[1] * b[1] + s.v[2] * b[2];
    for (int j = 0; j < 3; ++j) {
        const double djl = (j == l) ? 1.0 : 0.0;
        dF[0][j] = (cpp == 0) ? nu * djl : 0.0;
        for (int i = 0; i < 3; ++i)
            dF[1 + i][j] = s.mus * (djl * b[i] + (i == l ? b[j] : 0.0) - (i == j ? (2.0 / 3.0) * b[l] : 0.0)) +
                           ((cpp == 1 + i) ? nu * djl : 0.0);
        dF[4][j] = s.mus * (djl * vb + s.v[l] * b[j] - (2.0 / 3.0) * s.v[j] * b[l]) + s.kap * djl * a +
                   ((cpp == 4) ? nu * djl : 0.0);
    }
}

__device__ inline int64_t qp_face_base(const DevMesh &dm, int e, int lf, int Nq) {
    int64_t off = dm.qp_off[e] + (int64_t)(kVJac + kVRes) * Nq;
    for (int l = 0; l < lf; ++l) {
        const int pf = dm.face_p[dm.elem_face[6 * e + l]];
        off += (int64_t)kFPer * (pf + 2) * (pf + 2);
    }
    return off;
}

// ------------------------------------------------------- point kernel: volume
__global__ void __launch_bounds__(256) k_qp_volume(DevMesh dm, Phys P, int e0, const double *__restrict__ Qg,
                                                   const double *__restrict__ Ug, const double *__restrict__ Ung,
                                                   const double *__restrict__ nug, double *__restrict__ qp) {
    const int e = e0 + blockIdx.x;
    const int p = dm.elem_p[e], p1 = p + 1, Np = p1 * p1 * p1, nq = p + 2, Nq = nq * nq * nq;
    __shared__ double sU[5 * 125], sUn[5 * 125], sQ[15 * 125], sNu[125], sL[5 * 6];
    const int64_t no = dm.node_off[e];
    for (int t = threadIdx.x; t < 5 * Np; t += blockDim.x) {
        sU[t] = Ug[5 * no + t];
        sUn[t] = Ung[5 * no + t];
    }
    for (int t = threadIdx.x; t < 15 * Np; t += blockDim.x) sQ[t] = Qg[15 * no + t];
    for (int t = threadIdx.x; t < Np; t += blockDim.x) sNu[t] = nug[no + t];
    for (int t = threadIdx.x; t < p1 * nq; t += blockDim.x) sL[t] = dm.tbl[tbl_L(p, p, t / nq, t % nq)];
    __syncthreads();
    const double *vg = dm.vgeo + dm.vgeo_off[e];
    double *out = qp + (dm.qp_off[e] - dm.qp_off[e0]);
    for (int g = threadIdx.x; g < Nq; g += blockDim.x) {
        const int g0 = g % nq, g1 = (g / nq) % nq, g2 = g / (nq * nq);
        double u[5] = {0, 0, 0, 0, 0}, un[5] = {0, 0, 0, 0, 0}, q[15], nu = 0.0;
        for (int m = 0; m < 15; ++m) q[m] = 0.0;
        for (int i2 = 0; i2 < p1; ++i2)
            for (int i1 = 0; i1 < p1; ++i1) {
                const double l12 = sL[i1 * nq + g1] * sL[i2 * nq + g2];
                for (int i0 = 0; i0 < p1; ++i0) {
                    const double ph = sL[i0 * nq + g0] * l12;
                    const int i = i0 + p1 * (i1 + p1 * i2);
                    for (int c = 0; c < 5; ++c) {
                        u[c] += ph * sU[c * Np + i];
                        un[c] += ph * sUn[c * Np + i];
                    }
                    for (int m = 0; m < 15; ++m) q[m] += ph * sQ[m * Np + i];
                    nu += ph * sNu[i];
                }
            }
        const double W = vg[g];
        double G[3][3];
        for (int d = 0; d < 3; ++d)
            for (int j = 0; j < 3; ++j) G[d][j] = vg[(1 + 3 * d + j) * Nq + g];
        PState s;
        pstate(u, q, P, s);
        double F[5][3];
        total_flux(u, q, nu, P, s, F);
        double *vres = out + (int64_t)kVJac * Nq;
        // residual coefficients of the conservation rows (the gradient rows' residuals are
        // formed from their blocks, k_grad_rows)
        for (int c = 0; c < 5; ++c) {
            vres[(4 * c + 0) * Nq + g] = P.alpha * W * (u[c] - un[c]);
            for (int d = 0; d < 3; ++d)
                vres[(4 * c + 1 + d) * Nq + g] = -P.dt * W * (G[d][0] * F[c][0] + G[d][1] * F[c][1] + G[d][2] * F[c][2]);
        }
        // Jacobian coefficients of the conservation rows
        for (int cp = 0; cp < 5; ++cp) {
            double dF[5][3];
            dflux_dw(u, q, P, s, cp, dF);
            for (int c = 0; c < 5; ++c) {
                const int sidx = 15 + cp;
                double *o = out + (int64_t)(4 * (20 * c + sidx)) * Nq + g;
                o[0] = (c == cp) ? P.alpha * W : 0.0;
                for (int d = 0; d < 3; ++d)
                    o[(1 + d) * Nq] = -P.dt * W * (G[d][0] * dF[c][0] + G[d][1] * dF[c][1] + G[d][2] * dF[c][2]);
            }
        }
        for (int m = 0; m < 15; ++m) {
            double dF[5][3];
            dfv_dq(s, nu, m / 3, m % 3, dF);
            for (int c = 0; c < 5; ++c) {
                double *o = out + (int64_t)(4 * (20 * c + m)) * Nq + g;
                o[0] = 0.0;
                for (int d = 0; d < 3; ++d)
                    o[(1 + d) * Nq] = P.dt * W * (G[d][0] * dF[c][0] + G[d][1] * dF[c][1] + G[d][2] * dF[c][2]);
            }
        }
    }
}

// --------------------------------------------------------- point kernel: face
__global__ void __launch_bounds__(64) k_qp_face(DevMesh dm, Phys P, int e0, const double *__restrict__ Qg,
                                                const double *__restrict__ Ug, const double *__restrict__ Uhg,
                                                const double *__restrict__ nug, const double *__restrict__ Ubg,
                                                double *__restrict__ qp) {
    const int lf = blockIdx.x, e = e0 + blockIdx.y;
    const int p = dm.elem_p[e], p1 = p + 1, Np = p1 * p1 * p1, nq = p + 2, Nq = nq * nq * nq;
    const int F = dm.elem_face[6 * e + lf], pf = dm.face_p[F], pf1 = pf + 1, nqf1 = pf + 2, Nqf = nqf1 * nqf1;
    const int Nfp = pf1 * pf1, bc = dm.face_bc[F];
    const int d = lf / 2, side = lf & 1, t0 = (d == 0) ? 1 : 0, t1 = (d == 2) ? 1 : 2;
    const int64_t no = dm.node_off[e];
    const double *fg = dm.fgeo + dm.fgeo_off[6 * e + lf];
    double *out = qp + (qp_face_base(dm, e, lf, Nq) - dm.qp_off[e0]);
    const double *uh_g = Uhg + dm.face_off[F];
    const bool has_ub = (bc == 1 || bc == 3);  // boundary types that read prescribed data
    const double *ub_g = has_ub ? Ubg + dm.face_off[F] : nullptr;
    for (int s = threadIdx.x; s < Nqf; s += blockDim.x) {
        const int s0 = s % nqf1, s1 = s / nqf1;
        double u[5] = {0, 0, 0, 0, 0}, q[15], nu = 0.0, uh[5] = {0, 0, 0, 0, 0}, ub[5] = {0, 0, 0, 0, 0};
        for (int m = 0; m < 15; ++m) q[m] = 0.0;
        // element fields: only the nodes on this face are nonzero there
        for (int a1 = 0; a1 < p1; ++a1)
            for (int a0 = 0; a0 < p1; ++a0) {
                const double ph = dm.tbl[tbl_L(p, pf, a0, s0)] * dm.tbl[tbl_L(p, pf, a1, s1)];
                int idx[3];
                idx[d] = side ? p : 0;
                idx[t0] = a0;
                idx[t1] = a1;
                const int i = idx[0] + p1 * (idx[1] + p1 * idx[2]);
                for (int c = 0; c < 5; ++c) u[c] += ph * Ug[5 * no + c * Np + i];
                for (int m = 0; m < 15; ++m) q[m] += ph * Qg[15 * no + m * Np + i];
                nu += ph * nug[no + i];
            }
        for (int b1 = 0; b1 < pf1; ++b1)
            for (int b0 = 0; b0 < pf1; ++b0) {
                const double mu = dm.tbl[tbl_L(pf, pf, b0, s0)] * dm.tbl[tbl_L(pf, pf, b1, s1)];
                const int b = b0 + pf1 * b1;
                for (int c = 0; c < 5; ++c) {
                    uh[c] += mu * uh_g[c * Nfp + b];
                    if (has_ub) ub[c] += mu * ub_g[c * Nfp + b];
                }
            }
        const double wN[3] = {fg[s], fg[Nqf + s], fg[2 * Nqf + s]}, wA = fg[3 * Nqf + s];
        PState st;
        pstate(uh, q, P, st);
        double Fl[5][3];
        total_flux(uh, q, nu, P, st, Fl);
        for (int c = 0; c < 5; ++c)
            out[(kFRes + c) * Nqf + s] = Fl[c][0] * wN[0] + Fl[c][1] * wN[1] + Fl[c][2] * wN[2] + P.tau * wA * (u[c] - uh[c]);
        // d fh / d u (element trace): tau |N| I
        for (int c = 0; c < 5; ++c)
            for (int cp = 0; cp < 5; ++cp) out[(25 * c + cp) * Nqf + s] = (c == cp) ? P.tau * wA : 0.0;
        // d fh / d q
        for (int m = 0; m < 15; ++m) {
            double dF[5][3];
            dfv_dq(st, nu, m / 3, m % 3, dF);
            for (int c = 0; c < 5; ++c)
                out[(25 * c + 5 + m) * Nqf + s] = -(dF[c][0] * wN[0] + dF[c][1] * wN[1] + dF[c][2] * wN[2]);
        }
        // d fh / d uh
        for (int cp = 0; cp < 5; ++cp) {
            double dF[5][3];
            dflux_dw(uh, q, P, st, cp, dF);
            for (int c = 0; c < 5; ++c)
                out[(25 * c + 20 + cp) * Nqf + s] =
                    dF[c][0] * wN[0] + dF[c][1] * wN[1] + dF[c][2] * wN[2] - ((c == cp) ? P.tau * wA : 0.0);
        }
        if (bc) {
            // boundary residual b^ of eq. hdg-trace (weighted by w |N|) into slots kFBRes + c, its
            // derivatives d b^_c / d(u 0..4, q 5..19, uh 20..24) into kFBJac + 25 c + slot:
            //  1 prescribed state uh - ub; 2 extrapolated state uh - u;
            //  3 no-slip isothermal wall (rho^ - rho, m^, rho^E^ - rho^ e_w), e_w the internal
            //    energy of the prescribed state; 4 no-slip adiabatic wall (rho^ - rho, m^, the
            //    energy component of the numerical flux); 5 symmetry (rho^ - rho,
            //    m^ - (I - n n^T) m, rho^E^ - rhoE)
            double *bj = out + (int64_t)kFBJac * Nqf + s;
            for (int k = 0; k < 125; ++k) bj[(int64_t)k * Nqf] = 0.0;
            auto J = [&](int c, int slot) -> double & { return bj[(int64_t)(25 * c + slot) * Nqf]; };
            double br[5];
            if (bc == 1 || bc == 2) {
                for (int c = 0; c < 5; ++c) {
                    br[c] = wA * (uh[c] - (bc == 1 ? ub[c] : u[c]));
                    J(c, 20 + c) = wA;
                    if (bc == 2) J(c, c) = -wA;
                }
            } else if (bc == 3 || bc == 4) {
                br[0] = wA * (uh[0] - u[0]);
                J(0, 20) = wA;
                J(0, 0) = -wA;
                for (int i = 1; i < 4; ++i) {
                    br[i] = wA * uh[i];
                    J(i, 20 + i) = wA;
                }
                if (bc == 3) {
                    const double ew = ub[4] / ub[0] - 0.5 * (ub[1] * ub[1] + ub[2] * ub[2] + ub[3] * ub[3]) / (ub[0] * ub[0]);
                    br[4] = wA * (uh[4] - ew * uh[0]);
                    J(4, 24) = wA;
                    J(4, 20) = -wA * ew;
                } else {
                    br[4] = out[(kFRes + 4) * Nqf + s];
                    for (int k = 0; k < 25; ++k) J(4, k) = out[(25 * 4 + k) * Nqf + s];
                }
            } else {
                const double nn[3] = {wN[0] / wA, wN[1] / wA, wN[2] / wA};
                br[0] = wA * (uh[0] - u[0]);
                J(0, 20) = wA;
                J(0, 0) = -wA;
                for (int i = 0; i < 3; ++i) {
                    double t = uh[1 + i];
                    for (int j = 0; j < 3; ++j) {
                        const double pij = (i == j ? 1.0 : 0.0) - nn[i] * nn[j];
                        t -= pij * u[1 + j];
                        J(1 + i, 1 + j) = -wA * pij;
                    }
                    br[1 + i] = wA * t;
                    J(1 + i, 21 + i) = wA;
                }
                br[4] = wA * (uh[4] - u[4]);
                J(4, 24) = wA;
                J(4, 4) = -wA;
            }
            for (int c = 0; c < 5; ++c) out[(kFBRes + c) * Nqf + s] = br[c];
        }
    }
}

// --------------------------------------------------------- assembly kernel
// Face of an element: is volume node i on local face lf, and its face indices.
__device__ inline bool on_face(int i, int p1, int lf, int &a0, int &a1) {
    const int d = lf / 2, side = lf & 1;
    int idx[3] = {i % p1, (i / p1) % p1, i / (p1 * p1)};
    if (idx[d] != (side ? p1 - 1 : 0)) return false;
    const int t0 = (d == 0) ? 1 : 0, t1 = (d == 2) ? 1 : 2;
    a0 = idx[t0];
    a1 = idx[t1];
    return true;
}



// Face tables of the element-row kernels: the element's 1-D basis and each
// face's trace basis at the face's Gauss points, face quadrature bases in the
// point workspace.
__device__ inline void load_face_tables(const DevMesh &dm, int e, int p, int Nq, double (*sLf)[30],
                                        double (*sMf)[30], int *sPf, int *sNqf, int64_t *sFbase) {
    const int tid = threadIdx.x;
    if (tid < 6) {
        const int pf = dm.face_p[dm.elem_face[6 * e + tid]];
        sPf[tid] = pf;
        sNqf[tid] = (pf + 2) * (pf + 2);
        sFbase[tid] = qp_face_base(dm, e, tid, Nq) - dm.qp_off[e];
    }
    __syncthreads();
    for (int t = tid; t < 6 * 30; t += blockDim.x) {
        const int lf = t / 30, r = t % 30, pf = sPf[lf], nqf1 = pf + 2;
        const int a = r / nqf1, s = r % nqf1;
        sLf[lf][r] = (r < (p + 1) * nqf1) ? dm.tbl[tbl_L(p, pf, a, s)] : 0.0;
        sMf[lf][r] = (r < (pf + 1) * nqf1) ? dm.tbl[tbl_L(pf, pf, a, s)] : 0.0;
    }
}

// Gradient and conserved rows of the element system, by sum factorisation: every
// N_p x N_p block sum_g phi_k(g) [c0 phi_i + sum_d c_d dref_d phi_i](g) is contracted
// one direction at a time over the tensor Gauss points:
//   x:  T0 = sum_g1 (L_i1 c0 + D_i1 c1) L_k1,  T1 = sum_g1 L_i1 c2 L_k1,  T2 = sum_g1 L_i1 c3 L_k1
//   y:  VL = sum_g2 (L_i2 T0 + D_i2 T1) L_k2,   VD = sum_g2 L_i2 T2 L_k2
//   z:  A  = sum_g3 (L_i3 VL + D_i3 VD) L_k3
// (L, D: the 1-D basis and its derivative at the Gauss points).  The face terms
// and the trace columns are 2-D contractions over each face's Gauss points.
// Instantiated per degree PT (LDS sized for it, loop bounds and index arithmetic
// known at compile time); workgroups of elements of another degree return.
//
// Bound by LDS reads: in every stage a thread holds its operands of the contracted
// direction in registers and forms all p+1 (x, y) or (p+1)^2 (z) outputs that share
// them; the whole block goes through each stage at once (three barriers a block;
// one i1 slice at a time and one output per thread took 15 barriers and, at p = 4,
// 30 LDS reads an output instead of 2).  T and V are laid out so that consecutive
// lanes read consecutive entries.  256 elements at p = 4: 5.09 -> 1.56 ms for the
// conserved rows' blocks.
constexpr int kP1 = kMaxP + 1, kNQ = kMaxP + 2;

template <int PT> struct Block {
    static constexpr int p1 = PT + 1, Np = p1 * p1 * p1, nq = PT + 2, Nq = nq * nq * nq;
    static constexpr int P2 = p1 * p1, P4 = P2 * P2, Q2 = nq * nq;
    static constexpr int NT = (P4 + 63) / 64 * 64;  // threads: one per (i1, i2, k1, k2)
    double L[p1][nq], D[p1][nq];
    double C[4][nq][Q2];         // coefficient fields of one block, [g1][g2 + nq g3]
    double T[3][nq][nq * P2];    // x stage, [g2][(g3 p1 + i1) p1 + k1]
    double V[2][nq][P4];         // y stage, [g3][(i2 p1 + i1) p1^2 + k2 p1 + k1]

    __device__ void load_basis(const DevMesh &dm) {
        for (int t = threadIdx.x; t < p1 * nq; t += blockDim.x) {
            L[t / nq][t % nq] = dm.tbl[tbl_L(PT, PT, t / nq, t % nq)];
            D[t / nq][t % nq] = dm.tbl[tbl_D(PT, t / nq, t % nq)];
        }
    }
    // place of the coefficient d at Gauss point g
    __device__ double &coef(int d, int g) { return C[d][g % nq][g / nq]; }
    // The block of the coefficients C: emit(z) on every thread t < P4 of the last stage,
    // z[i3][k3] its entries; i1, i2, k1, k2 of a thread by split().  Begins and
    // ends without a barrier: C is read until the first one, V after the last.
    __device__ static void split(int t, int &i1, int &i2, int &k1, int &k2) {
        k1 = t % p1;
        k2 = (t / p1) % p1;
        i1 = (t / P2) % p1;
        i2 = t / (P2 * p1);
    }
    template <class Emit> __device__ void contract(Emit emit) {
        const int tid = threadIdx.x;
        __syncthreads();
        for (int t = tid; t < p1 * Q2; t += NT) {
            const int i1 = t / Q2, g23 = t % Q2;
            double u[3][nq];
#pragma unroll
            for (int g1 = 0; g1 < nq; ++g1) {
                const double l = L[i1][g1];
                u[0][g1] = l * C[0][g1][g23] + D[i1][g1] * C[1][g1][g23];
                u[1][g1] = l * C[2][g1][g23];
                u[2][g1] = l * C[3][g1][g23];
            }
            const int g2 = g23 % nq, at = ((g23 / nq) * p1 + i1) * p1;
#pragma unroll
            for (int k1 = 0; k1 < p1; ++k1) {
                double a[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int g1 = 0; g1 < nq; ++g1)
#pragma unroll
                    for (int d = 0; d < 3; ++d) a[d] += u[d][g1] * L[k1][g1];
#pragma unroll
                for (int d = 0; d < 3; ++d) T[d][g2][at + k1] = a[d];
            }
        }
        __syncthreads();
        for (int t = tid; t < p1 * nq * P2; t += NT) {
            const int q = t % (nq * P2), i2 = t / (nq * P2);  // q = (g3 p1 + i1) p1 + k1
            double u[nq], d[nq];
#pragma unroll
            for (int g2 = 0; g2 < nq; ++g2) {
                const double l = L[i2][g2];
                u[g2] = l * T[0][g2][q] + D[i2][g2] * T[1][g2][q];
                d[g2] = l * T[2][g2][q];
            }
            const int g3 = q / P2, at = (i2 * p1 + (q / p1) % p1) * P2 + q % p1;
#pragma unroll
            for (int k2 = 0; k2 < p1; ++k2) {
                double vl = 0.0, vd = 0.0;
#pragma unroll
                for (int g2 = 0; g2 < nq; ++g2) {
                    vl += u[g2] * L[k2][g2];
                    vd += d[g2] * L[k2][g2];
                }
                V[0][g3][at + k2 * p1] = vl;
                V[1][g3][at + k2 * p1] = vd;
            }
        }
        __syncthreads();
        if (tid < P4) {
            double vl[nq], vd[nq];
#pragma unroll
            for (int g3 = 0; g3 < nq; ++g3) {
                vl[g3] = V[0][g3][tid];
                vd[g3] = V[1][g3][tid];
            }
            double z[p1][p1];
#pragma unroll
            for (int i3 = 0; i3 < p1; ++i3) {
                double u[nq];
#pragma unroll
                for (int g3 = 0; g3 < nq; ++g3) u[g3] = L[i3][g3] * vl[g3] + D[i3][g3] * vd[g3];
#pragma unroll
                for (int k3 = 0; k3 < p1; ++k3) {
                    double v = 0.0;
#pragma unroll
                    for (int g3 = 0; g3 < nq; ++g3) v += u[g3] * L[k3][g3];
                    z[i3][k3] = v;
                }
            }
            emit(z);
        }
    }
};

// Scalar blocks of one element, in its part of the point workspace (read by
// k_grad_rows): the mass matrix M, G_j = int phi_k d_j phi_i (j = 0..2), each
// [N_p][N_p], then per face H_j[a][b] = -int_F phi_a mu_b n_j, [j][p1^2][N_fp] (a, b
// face-local).  They are the same for every component, so the gradient rows are
// copies of them; formed per row field as before they took 30 blocks an element
// instead of four.  kind: 0 M, 1..3 G_j, 4 the faces.
__device__ inline double *scalar_blocks(const DevMesh &dm, int e, int e0, double *qp, int Np, int p1) {
    const int w = dm.toff[7 * e + 6] / 5;
    return qp + (dm.qp_off[e + 1] - dm.qp_off[e0]) - scal_size(Np, p1, w);
}
template <int PT> struct BlockShared {
    Block<PT> sb;
    double Lf[6][30], Mf[6][30];
    int Pf[6], Nqf[6];
    int64_t Fbase[6];
    double F[6 * Block<PT>::P4];                     // face terms [lf][a0 a1][b0 b1]
    double G[std::max(6 * Block<PT>::P2 * kNQ, 3 * (PT + 1) * kP1 * kNQ)];  // first stage of the face contractions
    double Cf[6][kNQ * kNQ];                         // one block's face coefficients
};
template <int PT> __device__ void scalar_block(const DevMesh &dm, int e, int e0, int kind, double *qp, BlockShared<PT> &sh) {
    typedef Block<PT> B;
    constexpr int p1 = B::p1, Np = B::Np, Nq = B::Nq, NT = B::NT;
    const int tid = threadIdx.x;
    double *out = scalar_blocks(dm, e, e0, qp, Np, p1);
    if (kind < 4) {
        const double *vg = dm.vgeo + dm.vgeo_off[e];
        sh.sb.load_basis(dm);
        for (int t = tid; t < 4 * Nq; t += NT) {
            const int d = t / Nq, g = t % Nq;
            double v;
            if (kind == 0) v = (d == 0) ? vg[g] : 0.0;
            else v = (d == 0) ? 0.0 : vg[g] * vg[(1 + 3 * (d - 1) + kind - 1) * Nq + g];
            sh.sb.coef(d, g) = v;
        }
        double *dst = out + (int64_t)kind * Np * Np;
        sh.sb.contract([&](const double (&z)[p1][p1]) {
            int i1, i2, k1, k2;
            B::split(tid, i1, i2, k1, k2);
#pragma unroll
            for (int i3 = 0; i3 < p1; ++i3)
#pragma unroll
                for (int k3 = 0; k3 < p1; ++k3)
                    dst[(i1 + p1 * (i2 + p1 * i3)) * Np + k1 + p1 * (k2 + p1 * k3)] = z[i3][k3];
        });
        return;
    }
    load_face_tables(dm, e, PT, Nq, sh.Lf, sh.Mf, sh.Pf, sh.Nqf, sh.Fbase);
    out += (int64_t)4 * Np * Np;
    for (int lf = 0; lf < 6; ++lf) {
        const int pf1 = sh.Pf[lf] + 1, nqf1 = sh.Pf[lf] + 2, Nqf = sh.Nqf[lf], Nfp = pf1 * pf1;
        const double *fg = dm.fgeo + dm.fgeo_off[6 * e + lf];
        __syncthreads();
        for (int t = tid; t < 3 * p1 * pf1 * nqf1; t += NT) {
            const int j = t / (p1 * pf1 * nqf1), rem = t % (p1 * pf1 * nqf1);
            const int a0 = rem / (pf1 * nqf1), b0 = (rem / nqf1) % pf1, s1 = rem % nqf1;
            double v = 0.0;
            for (int s0 = 0; s0 < nqf1; ++s0)
                v += sh.Lf[lf][a0 * nqf1 + s0] * sh.Mf[lf][b0 * nqf1 + s0] * fg[j * Nqf + s0 + nqf1 * s1];
            sh.G[t] = -v;
        }
        __syncthreads();
        for (int t = tid; t < 3 * p1 * p1 * Nfp; t += NT) {
            const int j = t / (p1 * p1 * Nfp), rem = t % (p1 * p1 * Nfp);
            const int a = rem / Nfp, b = rem % Nfp;  // a = a0 + p1 a1, b = b0 + pf1 b1
            const int a0 = a % p1, a1 = a / p1, b0 = b % pf1, b1 = b / pf1;
            const double *gg = sh.G + ((j * p1 + a0) * pf1 + b0) * nqf1;
            double v = 0.0;
            for (int s1 = 0; s1 < nqf1; ++s1) v += sh.Lf[lf][a1 * nqf1 + s1] * sh.Mf[lf][b1 * nqf1 + s1] * gg[s1];
            out[t] = v;
        }
        out += 3 * p1 * p1 * Nfp;
    }
}

// Gradient rows (three quarters of A and B): row (c, j, node i) holds M's row i in
// its own field, G_j's in u_c, H_j's in the trace of component c and zeros elsewhere;
// its residual is M q_(c,j) + G_j u_c + H_j uh_c, the same integrals.  Bound by the
// writes: one workgroup takes `nodes` nodes, holds the scalar rows of a node in LDS and
// streams its 15 rows with 16-byte nontemporal stores, each thread's column pair
// classified once for all of them (12.5 GB at p = 4 in 2.40 ms, 2.82 with plain
// stores).
template <int PT>
__global__ void __launch_bounds__(256) k_grad_rows(DevMesh dm, int e0, int nodes, const double *__restrict__ Qg,
                                                   const double *__restrict__ Ug, const double *__restrict__ Uhg,
                                                   double *__restrict__ qp, double *__restrict__ Ebase) {
    constexpr int p = PT, p1 = p + 1, Np = p1 * p1 * p1, n = 20 * Np;
    constexpr int kW = 6 * kP1 * kP1;  // trace unknowns of a component, at most
    const int e = e0 + blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (dm.elem_p[e] != PT) return;
    const int *toff = dm.toff + 7 * e;
    const int f = toff[6], w = f / 5;
    const int64_t ld = e_ld(n, f), no = dm.node_off[e];
    double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]);
    const double *sc = scalar_blocks(dm, e, e0, qp, Np, p1);
    constexpr int oG = Np, oH = 4 * Np, oR = oH + 3 * kW;
    __shared__ double sv[oR + 15];  // a node's rows of M | G_0..2 | H_0..2 | its 15 residuals
    __shared__ int sTf[kW];  // trace unknown t of a component -> its entry in Uhat (component 0)
    __shared__ int sTn[kW];  // and the face's N_fp
    __shared__ signed char sTl[kW];  // and the local face
    for (int t = tid; t < w; t += 256) {
        int lf = 0;
        while (5 * t >= toff[lf + 1]) ++lf;
        sTn[t] = (toff[lf + 1] - toff[lf]) / 5;
        sTl[t] = (signed char)lf;
        sTf[t] = (int)(dm.face_off[dm.elem_face[6 * e + lf]] - dm.face_off[dm.elem_face[6 * e]]) + t - toff[lf] / 5;
    }
    const double *uh = Uhg + dm.face_off[dm.elem_face[6 * e]];
    for (int i = blockIdx.x * nodes; i < min((int)(blockIdx.x + 1) * nodes, Np); ++i) {
        __syncthreads();
        for (int t = tid; t < 4 * Np; t += 256) {
            sv[t] = sc[((int64_t)(t / Np) * Np + i) * Np + t % Np];
        }
        for (int t = tid; t < 3 * w; t += 256) {
            const int j = t / w, tt = t % w, lf = sTl[tt];
            const int nfp = sTn[tt], b = tt - toff[lf] / 5;
            int a0, a1;
            double v = 0.0;
            if (on_face(i, p1, lf, a0, a1))
                v = sc[(int64_t)4 * Np * Np + 3 * p1 * p1 * (toff[lf] / 5) + ((int64_t)j * p1 * p1 + a0 + p1 * a1) * nfp + b];
            sv[oH + j * kW + tt] = v;
        }
        __syncthreads();
        // the faces the node lies on: the trace of the others has no part in its residuals
        // (not even as a product with zero: it may not be finite)
        unsigned faces = 0;
        for (int lf = 0, a0, a1; lf < 6; ++lf) faces |= (unsigned)on_face(i, p1, lf, a0, a1) << lf;
        for (int r = wave; r < 15; r += 4) {
            const int c = r / 3, j = r % 3;
            double a = 0.0;
            for (int k = lane; k < Np; k += 64)
                a += sv[k] * Qg[15 * no + (int64_t)r * Np + k] + sv[oG + j * Np + k] * Ug[5 * no + (int64_t)c * Np + k];
            for (int t = lane; t < w; t += 64)
                if ((faces >> sTl[t]) & 1u) a += sv[oH + j * kW + t] * uh[sTf[t] + c * sTn[t]];
            for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off);
            if (lane == 0) sv[oR + r] = a;
        }
        __syncthreads();
        for (int c2 = tid; c2 < ld / 2; c2 += 256) {  // ld and the row starts are multiples of 8
            // rows of this column pair's entries that are not zero, and where row j's value is
            unsigned rows[2];
            int src[2], step[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int col = 2 * c2 + h;
                rows[h] = 0;
                src[h] = step[h] = 0;
                if (col < 15 * Np) {
                    const int fld = col / Np;
                    rows[h] = 1u << fld;
                    src[h] = col - fld * Np;
                } else if (col < n) {
                    const int k = col - 15 * Np, cu = k / Np;
                    rows[h] = 7u << (3 * cu);
                    src[h] = oG + k - cu * Np;
                    step[h] = Np;
                } else if (col < n + f) {
                    const int tc = col - n;
                    int lf = 0;
                    while (tc >= toff[lf + 1]) ++lf;
                    const int nfp = (toff[lf + 1] - toff[lf]) / 5, q = tc - toff[lf], ct = q / nfp;
                    rows[h] = 7u << (3 * ct);
                    src[h] = oH + toff[lf] / 5 + q - ct * nfp;
                    step[h] = kW;
                } else if (col == n + f) {
                    rows[h] = 0x7FFFu;
                    src[h] = oR;
                    step[h] = -1;
                }
            }
            double *dst = E + (int64_t)i * ld + 2 * c2;
#pragma unroll
            for (int r = 0; r < 15; ++r) {
                v2d v = {0.0, 0.0};
                if ((rows[0] >> r) & 1u) v.x = sv[src[0] + (step[0] < 0 ? r : (r % 3) * step[0])];
                if ((rows[1] >> r) & 1u) v.y = sv[src[1] + (step[1] < 0 ? r : (r % 3) * step[1])];
                __builtin_nontemporal_store(v, (v2d *)(dst + (int64_t)r * Np * ld));
            }
        }
    }
}

// Conserved rows, row field c: its 20 column-field blocks (volume and face terms)
// over kUG workgroups, its trace columns, residual column and padding in one more.
// The blocks of gradient fields that the fluxes of row c do not read are zero:
// they are written as such (21 of the 100 blocks).  blockIdx.x from 5 kUG on: the
// scalar blocks of the gradient rows.
constexpr int kUG = 4;
template <int PT>
__global__ void __launch_bounds__(Block<PT>::NT) k_conserved_blocks(DevMesh dm, Phys P, int e0,
                                                                    double *qp, double *__restrict__ Ebase) {
    const int e = e0 + blockIdx.y, c = blockIdx.x / kUG, ug = blockIdx.x % kUG;
    if (dm.elem_p[e] != PT) return;
    __shared__ BlockShared<PT> sh;
    if (blockIdx.x >= 5 * kUG) {
        scalar_block<PT>(dm, e, e0, blockIdx.x - 5 * kUG, qp, sh);
        return;
    }
    typedef Block<PT> B;
    constexpr int p = PT, p1 = B::p1, Np = B::Np, nq = B::nq, Nq = B::Nq, NT = B::NT, P2 = B::P2, P4 = B::P4;
    const int *toff = dm.toff + 7 * e;
    const int n = 20 * Np, f = toff[6];
    const int64_t ld = e_ld(n, f);
    double *Er = Ebase + (dm.E_off[e] - dm.E_off[e0]) + (int64_t)(15 + c) * Np * ld;
    const double *qpe = qp + (dm.qp_off[e] - dm.qp_off[e0]);
    const int tid = threadIdx.x;
    constexpr int kNqfFace = kNQ * kNQ;          // Gauss points of a face, at most
    B &sb = sh.sb;
    auto &sLf = sh.Lf;
    auto &sPf = sh.Pf, &sNqf = sh.Nqf;
    auto &sFbase = sh.Fbase;
    auto &sF = sh.F;
    auto &sG = sh.G;
    auto &sCf = sh.Cf;
    sb.load_basis(dm);
    load_face_tables(dm, e, PT, Nq, sLf, sh.Mf, sPf, sNqf, sFbase);
    __syncthreads();
    int i1, i2, k1, k2;
    B::split(min(tid, P4 - 1), i1, i2, k1, k2);
    // the x and y faces that both (i1, i2, .) and (k1, k2, .) lie on, or -1
    const int fx = (i1 == k1) ? (i1 == 0 ? 0 : i1 == p ? 1 : -1) : -1;
    const int fy = (i2 == k2) ? (i2 == 0 ? 2 : i2 == p ? 3 : -1) : -1;
    double *dst = Er + (int64_t)(i1 + p1 * i2) * ld + k1 + p1 * k2;
    // gradient fields that row c reads: the first 3 of them (mass), 12 (momentum), 15 (energy)
    const int nread = (c == 0) ? 3 : (c == 4) ? 15 : 12;
    constexpr int kLC = (4 * Nq + NT - 1) / NT, kLF = (6 * kNqfFace + NT - 1) / NT;
    double rc[kLC], rf[kLF];  // the next block's coefficients, in flight during this one's stages
    auto load = [&](int sblk) {
        const int slot = (sblk < 15) ? 5 + sblk : sblk - 15;
#pragma unroll
        for (int q = 0; q < kLC; ++q) {
            const int t = tid + NT * q;
            if (t < 4 * Nq) rc[q] = qpe[(int64_t)(4 * (20 * c + sblk)) * Nq + t];
        }
#pragma unroll
        for (int q = 0; q < kLF; ++q) {
            const int t = tid + NT * q, lf = t / kNqfFace, sq = t % kNqfFace;
            if (lf < 6 && sq < sNqf[lf]) rf[q] = qpe[sFbase[lf] + (int64_t)(25 * c + slot) * sNqf[lf] + sq];
        }
    };
    // the columns in the order zero fields last: nread gradient fields, 5 conserved, the rest
    auto field = [&](int o) { return o < nread ? o : (o < nread + 5 ? 15 + o - nread : o - 5); };
    const int o1 = (ug + 1) * (nread + 5) / kUG;
    int o = ug * (nread + 5) / kUG;
    if (o < o1) load(field(o));
    for (; o < o1; ++o) {
        const int sblk = field(o);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kLC; ++q) {
            const int t = tid + NT * q;
            if (t < 4 * Nq) sb.coef(t / Nq, t % Nq) = rc[q];
        }
#pragma unroll
        for (int q = 0; q < kLF; ++q) {
            const int t = tid + NT * q;
            if (t < 6 * kNqfFace) sCf[t / kNqfFace][t % kNqfFace] = rf[q];
        }
        __syncthreads();
        if (o + 1 < o1) load(field(o + 1));
        // face terms: F[a0 a1][b0 b1] = sum_s c(s) phi_a(s) phi_b(s) per face, two 1-D stages
        for (int t = tid; t < 6 * p1 * kNQ; t += NT) {
            const int lf = t / (p1 * kNQ), a0 = t % p1, s1 = (t / p1) % kNQ;
            const int nqf1 = sPf[lf] + 2;
            double g[p1];
#pragma unroll
            for (int b0 = 0; b0 < p1; ++b0) g[b0] = 0.0;
            if (s1 < nqf1)
                for (int s0 = 0; s0 < nqf1; ++s0) {
                    const double u = P.dt * sLf[lf][a0 * nqf1 + s0] * sCf[lf][s0 + nqf1 * s1];
#pragma unroll
                    for (int b0 = 0; b0 < p1; ++b0) g[b0] += u * sLf[lf][b0 * nqf1 + s0];
                }
#pragma unroll
            for (int b0 = 0; b0 < p1; ++b0) sG[(lf * kNQ + s1) * P2 + a0 * p1 + b0] = g[b0];
        }
        __syncthreads();
        for (int t = tid; t < 6 * P2 * p1; t += NT) {
            const int lf = t / (P2 * p1), b0 = t % p1, a1 = (t / p1) % p1, a0 = (t / P2) % p1;
            const int nqf1 = sPf[lf] + 2;
            double g[p1];
#pragma unroll
            for (int b1 = 0; b1 < p1; ++b1) g[b1] = 0.0;
            for (int s1 = 0; s1 < nqf1; ++s1) {
                const double u = sLf[lf][a1 * nqf1 + s1] * sG[(lf * kNQ + s1) * P2 + a0 * p1 + b0];
#pragma unroll
                for (int b1 = 0; b1 < p1; ++b1) g[b1] += u * sLf[lf][b1 * nqf1 + s1];
            }
#pragma unroll
            for (int b1 = 0; b1 < p1; ++b1) sF[lf * P4 + (a0 * p1 + a1) * P2 + b0 * p1 + b1] = g[b1];
        }
        sb.contract([&](double (&z)[p1][p1]) {
#pragma unroll
            for (int i3 = 0; i3 < p1; ++i3)
#pragma unroll
                for (int k3 = 0; k3 < p1; ++k3) {
                    double v = z[i3][k3];
                    if (fx >= 0) v += sF[fx * P4 + (i2 * p1 + i3) * P2 + k2 * p1 + k3];
                    if (fy >= 0) v += sF[fy * P4 + (i1 * p1 + i3) * P2 + k1 * p1 + k3];
                    if (i3 == 0 && k3 == 0) v += sF[4 * P4 + (i1 * p1 + i2) * P2 + k1 * p1 + k2];
                    if (i3 == p && k3 == p) v += sF[5 * P4 + (i1 * p1 + i2) * P2 + k1 * p1 + k2];
                    dst[(int64_t)P2 * i3 * ld + sblk * Np + P2 * k3] = v;
                }
        });
    }
    // the fields that row c does not read (gradient fields nread .. 14), spread over the groups
    const int z0 = nread * Np, zn = (15 - nread) * Np;
    for (int t = ug * NT + tid; t < zn * Np; t += kUG * NT)
        __builtin_nontemporal_store(0.0, Er + (int64_t)(t / zn) * ld + z0 + t % zn);
}

// Conserved rows, row field c = blockIdx.x: trace columns, residual column, padding.
template <int PT> struct ConservedTraceShared {
    static constexpr int p1 = PT + 1, Np = p1 * p1 * p1, nq = PT + 2, Nq = nq * nq * nq;
    double L[p1][nq], D[p1][nq], C[4][Nq];
    double Lf[6][30], Mf[6][30];
    int Pf[6], Nqf[6];
    int64_t Fbase[6];
    double F[5 * p1 * p1 * kP1 * kP1];               // trace-column blocks (face degree up to kMaxP)
    double G[std::max(5 * p1 * kP1 * kNQ, 2 * Np)];  // their first stage
    signed char Na[Np];                              // each node's index a0 p1 + a1 on the face, or -1
};
template <int PT>
__global__ void __launch_bounds__(256) k_conserved_trace(DevMesh dm, Phys P, int e0, const double *__restrict__ qp,
                                                         double *__restrict__ Ebase) {
    const int e = e0 + blockIdx.y, c = blockIdx.x, r = 15 + c;
    if (dm.elem_p[e] != PT) return;
    __shared__ ConservedTraceShared<PT> sh;
    constexpr int NT = 256;
    constexpr int p1 = PT + 1, Np = p1 * p1 * p1, nq = PT + 2, Nq = nq * nq * nq;
    const int *toff = dm.toff + 7 * e;
    const int n = 20 * Np, f = toff[6];
    const int64_t ld = e_ld(n, f);
    double *Er = Ebase + (dm.E_off[e] - dm.E_off[e0]) + (int64_t)r * Np * ld;
    const double *qpe = qp + (dm.qp_off[e] - dm.qp_off[e0]);
    const int tid = threadIdx.x;
    auto &sL = sh.L, &sD = sh.D;
    auto &sC = sh.C;
    auto &sLf = sh.Lf, &sMf = sh.Mf;
    auto &sPf = sh.Pf, &sNqf = sh.Nqf;
    auto &sFbase = sh.Fbase;
    auto &sF = sh.F;
    auto &sG = sh.G;
    auto &sNa = sh.Na;
    for (int t = tid; t < p1 * nq; t += NT) {
        sL[t / nq][t % nq] = dm.tbl[tbl_L(PT, PT, t / nq, t % nq)];
        sD[t / nq][t % nq] = dm.tbl[tbl_D(PT, t / nq, t % nq)];
    }
    load_face_tables(dm, e, PT, Nq, sLf, sMf, sPf, sNqf, sFbase);
    // ---- trace columns B: face by face, B_lf[cp][a0 a1][b0 b1] = sum_s c_cp(s) phi_a(s) mu_b(s)
    for (int lf = 0; lf < 6; ++lf) {
        const int pf1 = sPf[lf] + 1, nqf1 = sPf[lf] + 2, Nqf = sNqf[lf], Nfp = pf1 * pf1;
        __syncthreads();
        for (int i = tid; i < Np; i += NT) {
            int a0, a1;
            sNa[i] = (signed char)(on_face(i, p1, lf, a0, a1) ? a0 * p1 + a1 : -1);
        }
        for (int t = tid; t < 5 * p1 * pf1 * nqf1; t += NT) {
            const int cp = t / (p1 * pf1 * nqf1), rem = t % (p1 * pf1 * nqf1);
            const int a0 = rem / (pf1 * nqf1), b0 = (rem / nqf1) % pf1, s1 = rem % nqf1;
            const double *cf = qpe + sFbase[lf] + (int64_t)(25 * c + 20 + cp) * Nqf;
            double v = 0.0;
            for (int s0 = 0; s0 < nqf1; ++s0)
                v += sLf[lf][a0 * nqf1 + s0] * sMf[lf][b0 * nqf1 + s0] * cf[s0 + nqf1 * s1];
            sG[t] = P.dt * v;
        }
        __syncthreads();
        for (int t = tid; t < 5 * p1 * p1 * Nfp; t += NT) {
            const int cp = t / (p1 * p1 * Nfp), rem = t % (p1 * p1 * Nfp);
            const int a = rem / Nfp, b = rem % Nfp;
            const int a0 = a / p1, a1 = a % p1, b0 = b % pf1, b1 = b / pf1;
            const double *gg = sG + (cp * p1 * pf1 + a0 * pf1 + b0) * nqf1;
            double v = 0.0;
            for (int s1 = 0; s1 < nqf1; ++s1) v += sLf[lf][a1 * nqf1 + s1] * sMf[lf][b1 * nqf1 + s1] * gg[s1];
            sF[t] = v;
        }
        __syncthreads();
        // a thread keeps one column (ncol = 5 N_fp <= 125) and walks rows; a row
        // off the face is zero, a row on it reads its face-local index a0 p1 + a1
        const int ncol = 5 * Nfp, groups = NT / ncol;
        if (tid < groups * ncol) {
            const int col = tid % ncol, cp = col / Nfp, b = col % Nfp;
            const double *fc = sF + cp * p1 * p1 * Nfp + b;
            double *dst = Er + n + toff[lf] + col;
            for (int i = tid / ncol; i < Np; i += groups)
                __builtin_nontemporal_store(sNa[i] >= 0 ? fc[sNa[i] * Nfp] : 0.0, dst + (int64_t)i * ld);
        }
    }
    __syncthreads();
    // ---- residual column and padding: the residual's point coefficients in LDS,
    // the sum over the Gauss points split over two halves of the threads
    {
        const double *rc = qpe + (int64_t)kVJac * Nq + (int64_t)(4 * c) * Nq;
        for (int t = tid; t < 4 * Nq; t += NT) sC[t / Nq][t % Nq] = rc[t];
    }
    __syncthreads();
    static_assert(2 * Np <= 256, "two threads per row");
    if (tid < 2 * Np) {
        const int i = tid % Np, h = tid / Np;
        const int i1 = i % p1, i2 = (i / p1) % p1, i3 = i / (p1 * p1);
        double v = 0.0;
        for (int g = h * (Nq / 2); g < (h + 1) * (Nq / 2) + h * (Nq % 2); ++g) {
            const int g1 = g % nq, g2 = (g / nq) % nq, g3 = g / (nq * nq);
            const double l0 = sL[i1][g1], l1 = sL[i2][g2], l2 = sL[i3][g3];
            v += sC[0][g] * l0 * l1 * l2 + sC[1][g] * sD[i1][g1] * l1 * l2 + sC[2][g] * l0 * sD[i2][g2] * l2 +
                 sC[3][g] * l0 * l1 * sD[i3][g3];
        }
        sG[tid] = v;
    }
    __syncthreads();
    for (int i = tid; i < Np; i += NT) {
        double v = sG[i] + sG[Np + i];
        for (int lf = 0; lf < 6; ++lf) {
            int a0, a1;
            if (!on_face(i, p1, lf, a0, a1)) continue;
            const int Nqf = sNqf[lf], nqf1 = sPf[lf] + 2;
            const double *fb = qpe + sFbase[lf];
            for (int s = 0; s < Nqf; ++s)
                v += P.dt * fb[(kFRes + c) * Nqf + s] * sLf[lf][a0 * nqf1 + s % nqf1] * sLf[lf][a1 * nqf1 + s / nqf1];
        }
        Er[(int64_t)i * ld + n + f] = v;
        for (int64_t col = n + f + 1; col < ld; ++col) Er[(int64_t)i * ld + col] = 0.0;
    }
}

// Trace rows of local face lf: [C | D | R_uh] rows of this element's side, kTC of
// the five components per workgroup: the numerical flux on an interior face, the
// boundary residual on a boundary face.  Only the columns of the face's own
// nodes (C), of the face's trace block (D) and the residual column are nonzero.
// Entry (a, k) of a slot (0..19: C by column field, u then q; 20..24: D by trace
// component) is sum_s coef(s) mu_a(s) phi_k(s), contracted one direction at a time:
// all slots' first stage G[s1][a0][k0] in LDS, then per a1 the entries of the rows
// a = (a0, a1) into compact LDS rows; a column map then writes those rows in one
// coalesced sweep, zeros included, each thread's column pair looked up once for
// all of them.  Bound by the writes: the rows are consecutive and start on 64
// bytes, so half lines of neighbouring stores meet in L2, and plain stores are
// faster than nontemporal ones (5.0 GB at p = 4 in 1.14 against 2.30 ms; dot products
// over all Gauss points of the face, five times the multiplications, took 2.29).
constexpr int kNqfMax = kNQ * kNQ, kNfpMax = kP1 * kP1;
template <int PT> struct TraceCfg {
    static constexpr int p1 = PT + 1, Np = p1 * p1 * p1;
    static constexpr int TC = PT <= 2 ? 5 : 1;                                // components per workgroup
    static constexpr int GS = kP1 * (20 * p1 + 5 * kP1);                      // G entries per s1, at most
    static constexpr int RO = 20 * p1 * p1 + 5 * kNfpMax + 1;                 // nonzero entries of a row, at most
    static constexpr int LD = (20 * Np + 30 * kNfpMax + 1 + 7) / 8 * 8;       // columns, at most
};
template <int PT> struct TraceShared {
    typedef TraceCfg<PT> Cfg;
    double L[30], M[30];             // element and trace basis at the face's Gauss points
    double K[26][kNqfMax];           // coefficients of the component
    double G[kNQ][Cfg::GS];          // first stage: [s1][C: (slot, a0, k0) | D: (cp, a0, b0)]
    double R[kNQ][kP1];              // first stage of the residual: [s1][a0]
    double Out[kP1][Cfg::RO];        // the nonzero entries of the pass's rows
    short Map[Cfg::LD];              // column -> index into a row of Out, or -1
};
template <int PT>
__global__ void __launch_bounds__(256) k_trace_rows(DevMesh dm, int e0, const double *__restrict__ qp,
                                                    double *__restrict__ Ebase) {
    typedef TraceCfg<PT> Cfg;
    __shared__ TraceShared<PT> sh;
    if (dm.elem_p[e0 + blockIdx.y] != PT) return;
    constexpr int p1 = Cfg::p1, Np = Cfg::Np, n = 20 * Np, nq = PT + 2, Nq = nq * nq * nq, nC = 20 * p1 * p1;
    const int e = e0 + blockIdx.y, lf = blockIdx.x % 6, c0 = blockIdx.x / 6 * Cfg::TC;
    const int *toff = dm.toff + 7 * e;
    const int f = toff[6], ld = (int)e_ld(n, f);
    double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]);
    const int tid = threadIdx.x;
    const int F = dm.elem_face[6 * e + lf], bc = dm.face_bc[F], pf = dm.face_p[F];
    const int pf1 = pf + 1, nqf1 = pf + 2, Nfp = pf1 * pf1, Nqf = nqf1 * nqf1;
    const double *fb = qp + (qp_face_base(dm, e, lf, Nq) - dm.qp_off[e0]);
    double *Et = E + (int64_t)(n + toff[lf]) * ld;
    auto &sL = sh.L, &sM = sh.M;
    auto &sK = sh.K;
    auto &sG = sh.G;
    auto &sR = sh.R;
    auto &sOut = sh.Out;
    auto &sMap = sh.Map;
    for (int t = tid; t < 30; t += 256) {
        const int a = t / nqf1, q = t % nqf1;
        sL[t] = (a < p1) ? dm.tbl[tbl_L(PT, pf, a, q)] : 0.0;
        sM[t] = (a < pf1) ? dm.tbl[tbl_L(pf, pf, a, q)] : 0.0;
    }
    for (int col = tid; col < ld; col += 256) {
        int idx = -1;
        if (col < n) {
            const int sblk = col / Np, k = col - sblk * Np;
            int ka0, ka1;
            if (on_face(k, p1, lf, ka0, ka1)) idx = ((sblk < 15) ? 5 + sblk : sblk - 15) * p1 * p1 + ka0 + p1 * ka1;
        } else if (col < n + f) {
            const int cc = col - n;
            if (cc >= toff[lf] && cc < toff[lf + 1]) idx = nC + (cc - toff[lf]);
        } else if (col == n + f) {
            idx = nC + 5 * Nfp;
        }
        sMap[col] = (short)idx;
    }
    const int gC = 20 * pf1 * p1, gD = 5 * pf1 * pf1;
    for (int c = c0; c < c0 + Cfg::TC; ++c) {
        __syncthreads();
        for (int t = tid; t < 26 * Nqf; t += 256) {
            const int slot = t / Nqf, sq = t % Nqf;
            sK[slot][sq] = (slot == 25) ? fb[(int64_t)((bc ? kFBRes : kFRes) + c) * Nqf + sq]
                                        : fb[(int64_t)((bc ? kFBJac : 0) + 25 * c + slot) * Nqf + sq];
        }
        __syncthreads();
        for (int t = tid; t < 26 * pf1 * nqf1; t += 256) {
            const int a0 = t % pf1, s1 = (t / pf1) % nqf1, slot = t / (pf1 * nqf1);
            double g[kP1];
#pragma unroll
            for (int k = 0; k < kP1; ++k) g[k] = 0.0;
            const double *tab = slot < 20 ? sL : sM;
            for (int s0 = 0; s0 < nqf1; ++s0) {
                const double u = sK[slot][s0 + nqf1 * s1] * sM[a0 * nqf1 + s0];
                if (slot == 25) {
                    g[0] += u;
                } else {
#pragma unroll
                    for (int k = 0; k < kP1; ++k)
                        if (k < (slot < 20 ? p1 : pf1)) g[k] += u * tab[k * nqf1 + s0];
                }
            }
            if (slot == 25) {
                sR[s1][a0] = g[0];
            } else {
                const int nk = slot < 20 ? p1 : pf1;
                double *o = sG[s1] + (slot < 20 ? (slot * pf1 + a0) * p1 : gC + ((slot - 20) * pf1 + a0) * pf1);
#pragma unroll
                for (int k = 0; k < kP1; ++k)
                    if (k < nk) o[k] = g[k];
            }
        }
        for (int a1 = 0; a1 < pf1; ++a1) {
            __syncthreads();  // the first stage (or the previous sweep) is done
            for (int t = tid; t < gC + gD + pf1; t += 256) {
                const bool isC = t < gC;
                double v[kP1];
#pragma unroll
                for (int k = 0; k < kP1; ++k) v[k] = 0.0;
                if (t < gC + gD) {
                    const int nk = isC ? p1 : pf1, q = isC ? t : t - gC;
                    const double *tab = isC ? sL : sM;
                    for (int s1 = 0; s1 < nqf1; ++s1) {
                        const double u = sG[s1][t] * sM[a1 * nqf1 + s1];
#pragma unroll
                        for (int k = 0; k < kP1; ++k)
                            if (k < nk) v[k] += u * tab[k * nqf1 + s1];
                    }
                    const int k0 = q % nk, a0 = (q / nk) % pf1, sl = q / (nk * pf1);
                    double *o = sOut[a0] + (isC ? sl * p1 * p1 : nC + sl * Nfp) + k0;
#pragma unroll
                    for (int k = 0; k < kP1; ++k)
                        if (k < nk) o[k * nk] = v[k];
                } else {
                    const int a0 = t - gC - gD;
                    for (int s1 = 0; s1 < nqf1; ++s1) v[0] += sR[s1][a0] * sM[a1 * nqf1 + s1];
                    sOut[a0][nC + 5 * Nfp] = v[0];
                }
            }
            __syncthreads();
            double *row = Et + (int64_t)(c * Nfp + a1 * pf1) * ld;
            for (int c2 = tid; c2 < ld / 2; c2 += 256) {  // ld and the row starts are multiples of 8
                const int i0 = sMap[2 * c2], i1 = sMap[2 * c2 + 1];
                double *dst = row + 2 * c2;
                if (i0 < 0 && i1 < 0) {
                    const v2d zero = {0.0, 0.0};
                    for (int a0 = 0; a0 < pf1; ++a0) *(v2d *)(dst + (int64_t)a0 * ld) = zero;
                } else {
                    for (int a0 = 0; a0 < pf1; ++a0) {
                        const v2d v = {i0 >= 0 ? sOut[a0][i0] : 0.0, i1 >= 0 ? sOut[a0][i1] : 0.0};
                        *(v2d *)(dst + (int64_t)a0 * ld) = v;
                    }
                }
            }
        }
    }
}

}  // namespace

int launch_element_system(const hdg_ctx *ctx, int e0, int ne, const double *Q, const double *U,
                          const double *Un, const double *Uhat, const double *nu, const double *Ub,
                          double *E, double *qp, hipStream_t s) {
    const DevMesh &dm = ctx->dm;
    const Phys P = ctx->phys;
    hipLaunchKernelGGL(k_qp_volume, dim3(ne), dim3(256), 0, s, dm, P, e0, Q, U, Un, nu, qp);
    hipLaunchKernelGGL(k_qp_face, dim3(6, ne), dim3(64), 0, s, dm, P, e0, Q, U, Uhat, nu, Ub, qp);
    const double *qpc = qp;
    unsigned degrees = 0;
    for (int e = e0; e < e0 + ne; ++e) degrees |= 1u << ctx->elem_p[e];
    auto rows = [&](auto degree) {
        constexpr int PT = decltype(degree)::value, Np = (PT + 1) * (PT + 1) * (PT + 1);
        // k_grad_rows: at least 200 KB a workgroup where that leaves four workgroups per CU
        const int nodes = (PT > 2 || ne * Np < 4 * 256 * 8) ? 1 : (PT == 1) ? 8 : 3;
        if (!(degrees & (1u << PT))) return;
        hipLaunchKernelGGL(k_conserved_blocks<PT>, dim3(5 * kUG + 5, ne), dim3(Block<PT>::NT), 0, s, dm, P, e0, qp, E);
        hipLaunchKernelGGL(k_grad_rows<PT>, dim3((Np + nodes - 1) / nodes, ne), dim3(256), 0, s, dm, e0, nodes, Q, U, Uhat, qp, E);
        hipLaunchKernelGGL(k_conserved_trace<PT>, dim3(5, ne), dim3(256), 0, s, dm, P, e0, qpc, E);
        hipLaunchKernelGGL(k_trace_rows<PT>, dim3(30 / TraceCfg<PT>::TC, ne), dim3(256), 0, s, dm, e0, qpc, E);
    };
    rows(std::integral_constant<int, 1>{});
    rows(std::integral_constant<int, 2>{});
    rows(std::integral_constant<int, 3>{});
    rows(std::integral_constant<int, 4>{});
    return (int)hipGetLastError();
}

}  // namespace hdg
