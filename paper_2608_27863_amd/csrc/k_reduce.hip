// Block elimination of the gradient unknowns ahead of the dense condensation
// (eqs. newton-local-block, local-elimination, schur-trace).
//
// In the element system E^K = [[A B R_qu],[C D R_uh]] the gradient equations
// (eq. hdg-grad) couple q_(c,j) to itself through the mass matrix M, to u_c
// through G_j and to the trace of component c through H_j, the same M, G_j, H_j
// for every c and nothing else:
//   M q_(c,j) + G_j u_c + H_j uh_c = -R_(c,j).
// With Y_j = M^{-1} [G_j | H_j] and r_(c,j) = M^{-1} R_(c,j) the other rows (the
// conserved fields' and the trace's) become
//   K' = K - sum_(c,j) K_(., q_cj) [Y_j at (u_c, uh_c) | r_(c,j)],
// a system of 5 N_p + f rows whose first 5 N_p columns (padded to a multiple of 4)
// are then eliminated by the dense blocked LU (k_condense.hip).  At p = 4 the LU has 625 pivot columns
// instead of 2500, and the whole condensation takes 2.4e9 flop per element
// instead of 2.26e10.  In the products, a row field's blocks that the fluxes
// make zero are skipped (54 of the 75 couplings of conserved to gradient fields
// remain), and a trace row meets only the nodes of its own face.
//
// None of this is assumed of a system that a caller hands in: k_check compares
// every entry of E that the elimination relies on, k_minv looks at how well M is
// conditioned, and an element that fails either takes the dense LU of all its n columns.  The one-call Newton
// step forms the systems itself in the same call and does without the check.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "hdg_internal.h"
#include "lanes.h"

namespace hdg {
namespace {

typedef double acc_t __attribute__((ext_vector_type(4)));

__device__ inline acc_t mfma64(double a, double b, acc_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline int rowof(int lane, int j) { return 4 * j + (lane >> 4); }

// An element's tiles share an XCD (its Y and Minv stay in one L2).
__device__ inline bool xcd_item(int ne, int tiles, int &el, int &t) {
    const int xcd = blockIdx.x % 8, idx = blockIdx.x / 8;
    el = 8 * (idx / tiles) + xcd;
    t = idx % tiles;
    return el < ne;
}
inline int xcd_grid(int ne, int tiles) { return 8 * ((ne + 7) / 8) * tiles; }

// Components of q that the fluxes of row component c read (bit c'): the
// artificial viscosity's for the mass row, the velocity gradients' for the
// momentum rows, all for the energy row.  Boundary residuals read a subset.
__device__ inline unsigned group_mask(int c) { return c == 0 ? 0x1u : (c == 4 ? 0x1Fu : 0xFu); }

__device__ inline bool on_face(int node, int p1, int lf) {
    const int d = lf >> 1, end = (lf & 1) ? p1 - 1 : 0;
    const int x = (d == 0) ? node % p1 : (d == 1) ? (node / p1) % p1 : node / (p1 * p1);
    return x == end;
}
// t-th node of face lf (t < p1^2)
__device__ inline int face_node(int t, int p1, int lf) {
    const int d = lf >> 1, end = (lf & 1) ? p1 - 1 : 0;
    const int a = t % p1, b = t / p1;
    return (d == 0) ? end + p1 * (a + p1 * b) : (d == 1) ? a + p1 * (end + p1 * b) : a + p1 * (b + p1 * end);
}

// Pointers of one element's part of the auxiliary region: Y [3 Np][ldy] (column
// blocks G: Np, H: w, r: one column per c), M^{-1} [Np][ldm] zero-padded, and the
// residual contributions [5][red_n + f] of the five gradient components.
struct Aux {
    double *Y, *Minv, *part;
    int ldy, ldm;
};
__device__ inline Aux aux_of(const RedBuf &rb, int e, int e0, int Np, int w) {
    Aux a;
    a.ldy = red_ldy(Np, w);
    a.ldm = red_ldm(Np);
    a.Y = rb.aux + (rb.aux_off[e] - rb.aux_off[e0]);
    a.Minv = a.Y + (int64_t)3 * Np * a.ldy;
    a.part = a.Minv + (int64_t)Np * a.ldm;
    return a;
}

// Trace column index t of one component (t < w: the faces in order, their nodes)
// -> column of E relative to the first trace column, for component 0; the
// component's stride on that face in *nfp.
__device__ inline int trace_col(const int *to, int t, int *nfp) {
    int lf = 0;
    while (lf < 5 && 5 * t >= to[lf + 1]) ++lf;
    const int n = (to[lf + 1] - to[lf]) / 5;
    *nfp = n;
    return to[lf] + t - to[lf] / 5;
}

// ------------------------------------------------------------------- check
__global__ void k_red_init(int ne, int structured, int *__restrict__ info, int *__restrict__ sel) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ne) {
        info[i] = 0;
        sel[i] = structured;
    }
}

// sel[el] = 0 unless the element's system has the structure above, entry by
// entry (a NaN differs from everything).  Bound by HBM: the gradient rows are
// three quarters of A and B.  Part q < nq of an element: kCN nodes of the gradient rows
// (all 15 fields, against the rows of component 0); the later ones: kCR rows of the other
// equations (the entries in gradient columns that have to be zero).  Elements one after
// another, `rest` parts each, an odd number, so that every XCD gets parts of both kinds (with
// 32 parts at p = 2 the gradient rows fell to 6 of the 8 XCDs: 512 elements 836 us, now 380).
// From p = 2 on the first parts of all elements come before that: where they find a
// difference, the others return at once (512 elements at p = 2 that all differ there: 136 us;
// at p = 1, where an element has two gradient parts, it costs more than it gives: 1000
// elements 130 us, with leading parts 152).
constexpr int kCN = 5, kCR = 16;
template <int P> constexpr int kLead = P > 1 ? 1 : 0;  // leading parts per element
template <int P>
__global__ void __launch_bounds__(256) k_check(DevMesh dm, int e0, int ne, int nq, int rest,
                                               const double *__restrict__ Ebase, int *__restrict__ sel) {
    constexpr int p1 = P + 1, Np = p1 * p1 * p1;
    const int i = (int)blockIdx.x - kLead<P> * ne, el = i < 0 ? i + ne : i / rest, part = i < 0 ? 0 : kLead<P> + i % rest;
    const int e = e0 + el;
    if (dm.elem_p[e] != P || __hip_atomic_load(sel + el, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) return;
    const int *to = dm.toff + 7 * e;
    const int f = to[6], n = 20 * Np;
    const int64_t ld = e_ld(n, f);
    const double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]);
    bool bad = false;
    if (part < nq) {
        const int i0 = part * kCN;
        for (int col = threadIdx.x; col < n + f; col += 256) {
            // the field (or trace component) of this column and where component 0's
            // rows hold the value that belongs there
            int fld, ref;
            if (col < n) {
                fld = col / Np;
                ref = col - fld * Np;
                if (fld >= 15) ref += 15 * Np;
            } else {
                int lf = 0;
                while (col - n >= to[lf + 1]) ++lf;
                const int nfp = (to[lf + 1] - to[lf]) / 5, t = col - n - to[lf];
                fld = 20 + t / nfp;
                ref = n + to[lf] + t % nfp;
            }
            for (int i = i0; i < min(i0 + kCN, Np); ++i) {
                const double m = (fld < 15) ? E[(int64_t)i * ld + ref] : 0.0;
                double g[3];
#pragma unroll
                for (int j = 0; j < 3; ++j) g[j] = (fld < 15) ? 0.0 : E[(int64_t)(j * Np + i) * ld + ref];
                double v[15];
#pragma unroll
                for (int r = 0; r < 15; ++r) v[r] = E[(int64_t)(r * Np + i) * ld + col];
#pragma unroll
                for (int r = 0; r < 15; ++r) {
                    const int c = r / 3, j = r % 3;
                    const double want = (fld < 15) ? (fld == r ? m : 0.0) : ((fld - 15) % 5 == c ? g[j] : 0.0);
                    bad |= !(v[r] == want);
                }
            }
        }
    } else {
        const int r0 = (part - nq) * kCR;
        const int rows = 5 * Np + f;
        for (int r = r0; r < min(r0 + kCR, rows); ++r) {
            int c, lf = -1;
            if (r < 5 * Np) {
                c = r / Np;
            } else {
                const int t = r - 5 * Np;
                lf = 0;
                while (t >= to[lf + 1]) ++lf;
                c = (t - to[lf]) / ((to[lf + 1] - to[lf]) / 5);
            }
            const unsigned mask = group_mask(c);
            const double *row = E + (int64_t)(15 * Np + r) * ld;
            // conserved rows: only the groups outside the mask (the columns from 3 c' Np of the first one on)
            const int first = (lf >= 0) ? 0 : 3 * Np * __popc(mask);
            for (int col = first + threadIdx.x; col < 15 * Np; col += 256) {
                const bool may = ((mask >> (col / (3 * Np))) & 1u) && (lf < 0 || on_face(col % Np, p1, lf));
                if (!may) bad |= !(row[col] == 0.0);
            }
        }
    }
    if (bad) __hip_atomic_store(sel + el, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------ mass matrix
// M^{-1} by Gauss-Jordan elimination with partial pivoting, one workgroup per element,
// the matrix in registers: thread (rg, cg) of 32 x 16 holds rows rg + 32 i and
// columns cg + 16 j, which move round by one j after every 16 steps so that the
// step's column is in register 0.  Rows are not exchanged; the inverse's rows and
// columns are put in place when it is written.  Bound by the latency of its N_p
// dependent steps (two barriers, the search by every wave, one division).  256 elements
// at p = 4: 277 us (70 elements: 199); with the matrix in LDS, read and written in
// every step, 584 (438).  A zero or non-finite k-th pivot sends the element to the dense LU (sel = 0), or is
// reported as info[e] = k+1 in a call that runs without it (checked).  A matrix whose
// |M| |M^{-1}| (Frobenius norms) is over kMassCond goes there too: the elimination through
// M cannot pivot out of it, and loses up to the cube of that factor in systems where the LU
// of all columns loses none (random couplings of order 1 at p = 2: S within 1e-12 at a factor
// of 7e2, within 6e-7 at 2e4).  The bound is 16 times an affine element's 37, 536, 2112, 5831;
// vertices moved by 0.4 of the spacing give at most 1.6 times those, a Jacobian that varies a
// hundredfold in an element ten times.  In systems that the same call forms (checked) the
// couplings are graded as M is, and this route is the more accurate one (a Jacobian varying
// 10^4-fold, p = 3: S within 1e-15 to 2e-13, by all columns 1e-15 to 1e-10).
// With `unit` the 15 diagonal blocks of the gradient rows of E become identities (the block
// factor M is divided out of those rows).
template <int P> constexpr double kMassCond = 16 * (P == 1 ? 37 : P == 2 ? 536 : P == 3 ? 2112 : 5831);
template <int P>
__global__ void __launch_bounds__(512) k_minv(DevMesh dm, RedBuf rb, int e0, int checked, int unit,
                                              double *__restrict__ Ebase, int *__restrict__ info) {
    constexpr int p1 = P + 1, Np = p1 * p1 * p1, NT = 512, RI = (Np + 31) / 32, CJ = (Np + 15) / 16;
    const int e = e0 + blockIdx.x;
    if (dm.elem_p[e] != P || !rb.sel[blockIdx.x]) return;
    const int f = dm.toff[7 * e + 6], n = 20 * Np;
    const int64_t ld = e_ld(n, f);
    double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]);
    const Aux ax = aux_of(rb, e, e0, Np, f / 5);
    __shared__ double sfac[2][128], srow[16 * CJ];  // the step's column; its scaled pivot row
    __shared__ int sstep[128], spiv[16 * CJ];       // step of a pivot row; pivot row of a step
    __shared__ double snorm[2][NT / 64];            // squares of M's and of the inverse's entries, by wave
    const int tid = threadIdx.x, lane = tid & 63, cg = tid & 15, rg = tid >> 4;
    double a[RI][CJ];
#pragma unroll
    for (int i = 0; i < RI; ++i)
#pragma unroll
        for (int j = 0; j < CJ; ++j) {
            const int r = rg + 32 * i, c = cg + 16 * j;
            a[i][j] = (r < Np && c < Np) ? E[(int64_t)r * ld + c] : 0.0;
        }
    auto squares = [&](double *out) {
        double v = 0.0;
#pragma unroll
        for (int i = 0; i < RI; ++i)
#pragma unroll
            for (int j = 0; j < CJ; ++j) v += a[i][j] * a[i][j];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) out[tid >> 6] = v;
    };
    if (!checked) squares(snorm[0]);
    if (tid < 256) sfac[tid >> 7][tid & 127] = 0.0;
    __syncthreads();
    if (cg == 0)
#pragma unroll
        for (int i = 0; i < RI; ++i) sfac[0][rg + 32 * i] = a[i][0];
    bool free0 = lane < Np, free1 = 64 + lane < Np;  // rows lane and 64 + lane, not pivots yet
    int bad = 0;
#pragma unroll 1
    for (int jb = 0; jb < CJ; ++jb) {
#pragma unroll 1
        for (int kc = 0; kc < 16; ++kc) {
            const int k = 16 * jb + kc, buf = k & 1;
            if (k >= Np) break;  // uniform
            __syncthreads();
            // pivot: largest |a| over the rows left (smallest row on ties, NaN wins), by the
            // upper words and, where two of those agree, the values
            double best = free0 ? fabs(sfac[buf][lane]) : -1.0;
            if (!(best == best)) best = INFINITY;
            int p = lane;
            if (Np > 64) {
                double v = free1 ? fabs(sfac[buf][64 + lane]) : -1.0;
                if (!(v == v)) v = INFINITY;
                if (v > best) { best = v; p = 64 + lane; }
            }
            const unsigned key = best >= 0.0 ? upper_word(best) : 0u, top = lanes_max<64>(key);
            const unsigned long long tie = __ballot(key == top);
            if ((tie & (tie - 1)) != 0)
                for (int off = 32; off > 0; off >>= 1) {
                    const double ov = __shfl_xor(best, off);
                    const int op = __shfl_xor(p, off);
                    if (ov > best || (ov == best && op < p)) { best = ov; p = op; }
                }
            else
                p = __builtin_amdgcn_readlane(p, __ffsll((long long)tie) - 1);
            p = __builtin_amdgcn_readfirstlane(p);
            const double d = sfac[buf][p], pinv = (d != 0.0) ? 1.0 / d : 0.0;
            if (bad == 0 && !(fabs(d) > 0.0 && fabs(d) < INFINITY)) bad = k + 1;
            free0 &= lane != p;
            free1 &= 64 + lane != p;
            if (rg == (p & 31))
#pragma unroll
                for (int i = 0; i < RI; ++i)
                    if (i == p >> 5)
#pragma unroll
                        for (int j = 0; j < CJ; ++j) srow[16 * j + cg] = (j == 0 && cg == kc) ? pinv : a[i][j] * pinv;
            if (tid == 0) {
                sstep[p] = k;
                spiv[k] = p;
            }
            __syncthreads();
            double s[CJ];
#pragma unroll
            for (int j = 0; j < CJ; ++j) s[j] = srow[16 * j + cg];
#pragma unroll
            for (int i = 0; i < RI; ++i) {
                const int r = rg + 32 * i;
                const double fct = sfac[buf][r];
                if (cg == kc) a[i][0] = 0.0;
#pragma unroll
                for (int j = 0; j < CJ; ++j) a[i][j] = (r == p) ? s[j] : a[i][j] - fct * s[j];
            }
            if (cg == ((kc + 1) & 15))  // the next step's column
#pragma unroll
                for (int i = 0; i < RI; ++i) sfac[buf ^ 1][rg + 32 * i] = (kc == 15) ? a[i][CJ > 1 ? 1 : 0] : a[i][0];
        }
#pragma unroll
        for (int i = 0; i < RI; ++i) {
            const double t = a[i][0];
#pragma unroll
            for (int j = 0; j < CJ - 1; ++j) a[i][j] = a[i][j + 1];
            a[i][CJ - 1] = t;
        }
    }
    if (bad) {  // uniform: a singular block leaves the element to the dense LU where that follows
        if (tid == 0) {
            if (checked) info[e] = bad;
            else rb.sel[blockIdx.x] = 0;
        }
        if (!checked) return;
    }
    if (!checked) squares(snorm[1]);
    __syncthreads();
    if (!checked) {
        double m = 0.0, v = 0.0;
        for (int q = 0; q < NT / 64; ++q) {
            m += snorm[0][q];
            v += snorm[1][q];
        }
        if (!(m * v <= kMassCond<P> * kMassCond<P>)) {  // uniform; also where a square leaves the range
            if (tid == 0) rb.sel[blockIdx.x] = 0;
            return;
        }
    }
    // entry (p_k, j) of the result is entry (k, p_j) of the inverse
#pragma unroll
    for (int i = 0; i < RI; ++i) {
        const int r = rg + 32 * i;
        if (r >= Np) continue;
        double *out = ax.Minv + (int64_t)sstep[r] * ax.ldm;
#pragma unroll
        for (int j = 0; j < CJ; ++j)
            if (cg + 16 * j < Np) out[spiv[cg + 16 * j]] = a[i][j];
        for (int c = Np + cg; c < ax.ldm; c += 16) out[c] = 0.0;
    }
    if (unit)
        for (int m = 0; m < 15; ++m)
            for (int t = tid; t < Np * Np; t += NT) {
                const int r = t / Np, c = t % Np;
                E[(int64_t)(m * Np + r) * ld + m * Np + c] = (r == c) ? 1.0 : 0.0;
            }
}

// Y_j = M^{-1} [G_j | H_j | R_(0..4,j)], one workgroup per (element, j, 64
// columns): the columns' N_p rows in LDS, M^{-1} from the cache in matrix-core
// operand order.  With `write` the result also replaces those columns of E's
// gradient rows (all five components).
template <int P>
__global__ void __launch_bounds__(256) k_ysolve(DevMesh dm, RedBuf rb, int e0, int ne, int tiles, int write,
                                                double *__restrict__ Ebase) {
    constexpr int p1 = P + 1, Np = p1 * p1 * p1, NB = (Np + 15) / 16, RB = (NB + 3) / 4, TC = 64;
    int el, t;
    if (!xcd_item(ne, 3 * tiles, el, t)) return;
    const int e = e0 + el;
    if (dm.elem_p[e] != P || !rb.sel[el]) return;
    const int *to = dm.toff + 7 * e;
    const int f = to[6], w = f / 5, n = 20 * Np, ncol = Np + w + 5;
    const int j = t / tiles, c0 = (t % tiles) * TC;
    if (c0 >= ncol) return;
    const int64_t ld = e_ld(n, f);
    double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]);
    const Aux ax = aux_of(rb, e, e0, Np, w);
    __shared__ double sX[16 * NB][TC + 1];
    __shared__ int scol[TC], snfp[TC];  // column of E (component 0), component stride (0: the residual column)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < TC) {
        const int c = c0 + tid;
        int col = -1, st = 0;
        if (c < Np) {
            col = 15 * Np + c;
            st = Np;
        } else if (c < Np + w) {
            col = n + trace_col(to, c - Np, &st);
        } else if (c < ncol) {
            col = n + f;
        }
        scol[tid] = col;
        snfp[tid] = st;
    }
    __syncthreads();
    for (int q = tid; q < 16 * NB * TC; q += 256) {
        const int r = q / TC, c = q % TC, col = scol[c];
        const int rr = (snfp[c] == 0) ? 3 * (c0 + c - Np - w) + j : j;  // residual columns: field (c', j)
        sX[r][c] = (r < Np && col >= 0) ? E[(int64_t)(rr * Np + r) * ld + col] : 0.0;
    }
    __syncthreads();
    const int kq = lane >> 4, cl = lane & 15;
    acc_t acc[RB][4];
#pragma unroll
    for (int h = 0; h < RB; ++h) {
        const int blk = wave + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[h][q] = (acc_t){0.0, 0.0, 0.0, 0.0};
        if (blk >= NB) continue;  // uniform per wave
        const double *arow = ax.Minv + (int64_t)min(16 * blk + cl, Np - 1) * ax.ldm + kq;
        for (int kb = 0; kb < 16 * NB; kb += 16) {
            double a[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = arow[kb + 4 * q];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int b = 0; b < 4; ++b) acc[h][b] = mfma64(a[q], sX[kb + 4 * q + kq][16 * b + cl], acc[h][b]);
        }
    }
#pragma unroll
    for (int h = 0; h < RB; ++h)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int c = 16 * b + cl, col = scol[c], st = snfp[c];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = 16 * (wave + 4 * h) + rowof(lane, q);
                if (r >= Np || col < 0) continue;
                const double v = acc[h][b][q];
                ax.Y[(int64_t)(j * Np + r) * ax.ldy + c0 + c] = v;
                if (write) {
                    if (st == 0) {
                        E[(int64_t)((3 * (c0 + c - Np - w) + j) * Np + r) * ld + col] = v;
                    } else {
#pragma unroll
                        for (int cc = 0; cc < 5; ++cc) E[(int64_t)((3 * cc + j) * Np + r) * ld + col + cc * st] = v;
                    }
                }
            }
        }
}

// ------------------------------------------------------- tile product core
// acc += A B over K, A(r, k) and B(k, c) through pointers from the functors
// (valid addresses for every r, k, c; okA / okB say which entries count), K in
// chunks of 16 double-buffered through LDS, the next chunk's loads in flight
// during the current one's products.  Four waves, WR x WC of them, each BR x BC
// blocks of 16 x 16.  use: bit b of a wave = its row block b takes the products.
template <int WR, int WC, int BR, int BC> struct Tile {
    static constexpr int TM = 16 * WR * BR, TN = 16 * WC * BC, KC = 16;
    static constexpr int SA = KC + 2, SB = TN + 16;
    static_assert(WR * WC == 4, "four waves");
    static constexpr int LA = TM / 16, LB = TN / 16;  // loads per thread and chunk
    struct Smem {
        double A[2][TM][SA];
        double B[2][KC][SB];
    };
    template <class PA, class OA, class PB, class OB>
    __device__ static void product(int K, PA pa, OA okA, PB pb, OB okB, unsigned use, bool negate, Smem &s,
                                   acc_t (&acc)[BR][BC]) {
        const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
        const int wr = (wave / WC) * 16 * BR, wc = (wave % WC) * 16 * BC;
        const int ak = tid & 15, ar = tid >> 4;
        double ra[LA], rb[LB];
        auto load = [&](int kc) {
#pragma unroll
            for (int q = 0; q < LA; ++q) ra[q] = *pa(ar + 16 * q, min(kc + ak, K - 1));
#pragma unroll
            for (int q = 0; q < LB; ++q) {
                const int i = tid + 256 * q;
                rb[q] = *pb(min(kc + i / TN, K - 1), i % TN);
            }
        };
        auto store = [&](int buf, int kc) {
#pragma unroll
            for (int q = 0; q < LA; ++q) {
                const double v = (kc + ak < K && okA(ar + 16 * q)) ? ra[q] : 0.0;
                s.A[buf][ar + 16 * q][ak] = negate ? -v : v;
            }
#pragma unroll
            for (int q = 0; q < LB; ++q) {
                const int i = tid + 256 * q;
                s.B[buf][i / TN][i % TN] = (kc + i / TN < K && okB(i % TN)) ? rb[q] : 0.0;
            }
        };
        load(0);
        store(0, 0);
        __syncthreads();
        const int nch = (K + KC - 1) / KC;
        for (int ch = 0; ch < nch; ++ch) {
            const int buf = ch & 1;
            if (ch + 1 < nch) load((ch + 1) * KC);
            if (use) {
#pragma unroll
                for (int kk = 0; kk < KC; kk += 4) {
                    double av[BR], bv[BC];
#pragma unroll
                    for (int b = 0; b < BR; ++b) av[b] = s.A[buf][wr + 16 * b + (lane & 15)][kk + (lane >> 4)];
#pragma unroll
                    for (int b = 0; b < BC; ++b) bv[b] = s.B[buf][kk + (lane >> 4)][wc + 16 * b + (lane & 15)];
#pragma unroll
                    for (int b = 0; b < BR; ++b)
                        if ((use >> b) & 1u)
#pragma unroll
                            for (int c = 0; c < BC; ++c) acc[b][c] = mfma64(av[b], bv[c], acc[b][c]);
                }
            }
            if (ch + 1 < nch) {
                store(buf ^ 1, (ch + 1) * KC);
                __syncthreads();
            }
        }
    }
};

// K' (rows of the conserved fields, or of the trace) in the columns of
// component c', one tile per workgroup.  A conserved tile is one row field
// (N_p rows); a trace tile lies in one face's rows and its K runs over the
// nodes of that face only.  The last column is the residual's contribution of
// this c' (the five are summed by k_rescol).
template <int P, bool TRACE, int WR, int WC, int BR, int BC>
__global__ void __launch_bounds__(256, 2) k_reduce(DevMesh dm, RedBuf rb, int e0, int ne, int tiles_r, int tiles_n,
                                                   const double *__restrict__ Ebase) {
    constexpr int p1 = P + 1, Np = p1 * p1 * p1, nu = (5 * Np + 3) & ~3, KN = TRACE ? 3 * p1 * p1 : 3 * Np;
    typedef Tile<WR, WC, BR, BC> T;
    static_assert(TRACE || T::TM >= Np, "a conserved tile holds a whole row field");
    int el, t;
    if (!xcd_item(ne, tiles_r * 5 * tiles_n, el, t)) return;
    const int e = e0 + el;
    if (dm.elem_p[e] != P || !rb.sel[el]) return;
    const int *to = dm.toff + 7 * e;
    const int f = to[6], w = f / 5, n = 20 * Np, N = Np + w + 1;
    const int n0 = (t % tiles_n) * T::TN, cp = (t / tiles_n) % 5, rt = t / tiles_n / 5;
    // rows of K' [r0, r1) and the row component of r0's tile (or its face)
    int r0, r1, lf = 0;
    if (TRACE) {
        lf = rt % 6;
        r0 = nu + to[lf] + (rt / 6) * T::TM;
        r1 = min(r0 + T::TM, nu + to[lf + 1]);
    } else {
        r0 = rt * Np;
        r1 = r0 + Np;
    }
    if (n0 >= N || r0 >= r1) return;  // uniform per block
    const int64_t ld = e_ld(n, f), ldk = e_ld(nu, f);
    // rows and columns of K' before nu are E's from 15 Np on, those from nu on E's from n on
    const double *Er = Ebase + (dm.E_off[e] - dm.E_off[e0]) + (int64_t)(TRACE ? n - nu : 15 * Np) * ld;
    double *Kr = rb.K + (rb.k_off[e] - rb.k_off[e0]);
    const Aux ax = aux_of(rb, e, e0, Np, w);
    __shared__ __attribute__((aligned(16))) typename T::Smem sm;
    __shared__ int skc[TRACE ? KN : 1];  // gradient columns of a trace tile's product: j Np + node
    __shared__ int scol[T::TN];   // column of K' of each tile column (-1: the residual, -2: none)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (TRACE)
        for (int k = tid; k < KN; k += 256) skc[k] = (k / (p1 * p1)) * Np + face_node(k % (p1 * p1), p1, lf);
    for (int i = tid; i < T::TN; i += 256) {
        const int c = n0 + i;
        int col = -2;
        if (c < Np) {
            col = cp * Np + c;
        } else if (c < Np + w) {
            int st;
            col = nu + trace_col(to, c - Np, &st);
            col += cp * st;
        } else if (c == Np + w) {
            col = -1;
        }
        scol[i] = col;
    }
    __syncthreads();
    const int wr = (wave / WC) * 16 * BR, wc = (wave % WC) * 16 * BC;
    acc_t acc[BR][BC];
#pragma unroll
    for (int b = 0; b < BR; ++b)
#pragma unroll
        for (int c = 0; c < BC; ++c) {
            const int col = scol[wc + 16 * c + (lane & 15)];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + wr + 16 * b + rowof(lane, q);
                acc[b][c][q] = (col >= 0 && r < r1) ? Er[(int64_t)r * ld + col + (col < nu ? 15 * Np : n - nu)] : 0.0;
            }
        }
    unsigned use = 0, any = 0;
    if (TRACE) {
        const int nfp = (to[lf + 1] - to[lf]) / 5;
#pragma unroll
        for (int b = 0; b < BR; ++b) {
            const int lo = r0 + wr + 16 * b, hi = min(lo + 15, r1 - 1);
            if (lo >= r1) continue;
            for (int c = (lo - nu - to[lf]) / nfp; c <= (hi - nu - to[lf]) / nfp; ++c)
                if ((group_mask(c) >> cp) & 1u) use |= 1u << b;
        }
        any = 1u;
    } else {
        any = (group_mask(rt) >> cp) & 1u;
        if (any)
#pragma unroll
            for (int b = 0; b < BR; ++b)
                if (r0 + wr + 16 * b < r1) use |= 1u << b;
    }
    if (any) {
        const double *A0 = Er + (int64_t)r0 * ld + (int64_t)3 * cp * Np;
        const int rl = r1 - 1 - r0;
        T::product(
            KN, [&](int r, int k) { return A0 + (int64_t)min(r, rl) * ld + (TRACE ? skc[k] : k); }, [&](int r) { return r <= rl; },
            [&](int k, int c) {
                const int col = n0 + c;
                return ax.Y + (int64_t)(TRACE ? skc[k] : k) * ax.ldy + (col < Np + w ? col : Np + w + cp);
            },
            [&](int c) { return n0 + c < N; }, use, true, sm, acc);
    }
#pragma unroll
    for (int b = 0; b < BR; ++b)
#pragma unroll
        for (int c = 0; c < BC; ++c) {
            const int col = scol[wc + 16 * c + (lane & 15)];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + wr + 16 * b + rowof(lane, q);
                if (r >= r1) continue;
                if (col >= 0) Kr[(int64_t)r * ldk + col] = acc[b][c][q];
                else if (col == -1) ax.part[(int64_t)cp * (nu + f) + r] = acc[b][c][q];
            }
        }
}

// The residual column of K', the decoupled unknowns and the padding columns.
__global__ void __launch_bounds__(256) k_rescol(DevMesh dm, RedBuf rb, int e0, const double *__restrict__ Ebase) {
    const int el = blockIdx.y, e = e0 + el;
    if (!rb.sel[el]) return;
    const int p = dm.elem_p[e], Np = (p + 1) * (p + 1) * (p + 1), nu = red_n(Np), f = dm.toff[7 * e + 6];
    const int r = blockIdx.x * 256 + threadIdx.x;
    if (r >= nu + f) return;
    const int64_t ld = e_ld(20 * Np, f), ldk = e_ld(nu, f);
    const double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]);
    double *row = rb.K + (rb.k_off[e] - rb.k_off[e0]) + (int64_t)r * ldk;
    const Aux ax = aux_of(rb, e, e0, Np, f / 5);
    const bool pad = r >= 5 * Np && r < nu;
    double v = 0.0;
    if (pad) {
        for (int c = 0; c < ldk; ++c) row[c] = 0.0;
    } else {
        v = E[(int64_t)(r < nu ? 15 * Np + r : 20 * Np + r - nu) * ld + 20 * Np + f];
#pragma unroll
        for (int c = 0; c < 5; ++c) v += ax.part[(int64_t)c * (nu + f) + r];
    }
    for (int c = 5 * Np; c < nu; ++c) row[c] = (c == r) ? 1.0 : 0.0;
    row[nu + f] = v;
    for (int c = nu + f + 1; c < ldk; ++c) row[c] = 0.0;
}

// -------------------------------------------------------------- write back
// The factored rows of the conserved fields return to E (U, from the row's 64-column
// block on, and L^{-1} P [B | R]; the recovery reads nothing to the left).  256
// elements at p = 4: 0.59 ms (all columns 0.95; nontemporal stores, whose rows share
// lines, 0.76).
__global__ void __launch_bounds__(256) k_wb_rows(DevMesh dm, RedBuf rb, int e0, double *__restrict__ Ebase) {
    const int el = blockIdx.y, e = e0 + el;
    if (!rb.sel[el]) return;
    const int p = dm.elem_p[e], Np = (p + 1) * (p + 1) * (p + 1), nu = red_n(Np), f = dm.toff[7 * e + 6];
    const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= 5 * Np) return;
    const int64_t ld = e_ld(20 * Np, f), ldk = e_ld(nu, f);
    const double *src = rb.K + (rb.k_off[e] - rb.k_off[e0]) + (int64_t)r * ldk;
    double *dst = Ebase + (dm.E_off[e] - dm.E_off[e0]) + (int64_t)(15 * Np + r) * ld + 15 * Np;
    for (int c = (r & ~63) + lane; c < 5 * Np; c += 64) dst[c] = src[c];
    for (int c = lane; c <= f; c += 64) dst[5 * Np + c] = src[nu + c];
}

// [S^K | -g^K] from K' into E's trace rows, and [S^K | g^K] column-major into SK,
// one 64 x 64 tile per workgroup; the element's first tile leaves the mark by
// which the recovery knows the gradient rows' form.  256 elements at p = 4: 1.00 ms
// (1.13 with 32 x 32 tiles, whose segments are two lines; 0.65 at the copy rate).
constexpr int kWbTile = 64;
__global__ void __launch_bounds__(256) k_wb_trace(DevMesh dm, RedBuf rb, int e0, double *__restrict__ Ebase,
                                                  double *__restrict__ SK) {
    const int el = blockIdx.z, e = e0 + el;
    if (!rb.sel[el]) return;
    const int p = dm.elem_p[e], Np = (p + 1) * (p + 1) * (p + 1), nu = red_n(Np), f = dm.toff[7 * e + 6];
    const int i0 = blockIdx.y * kWbTile, j0 = blockIdx.x * kWbTile;
    if (i0 >= f || j0 > f) return;
    const int64_t ld = e_ld(20 * Np, f), ldk = e_ld(nu, f);
    const double *Kr = rb.K + (rb.k_off[e] - rb.k_off[e0]) + (int64_t)nu * ldk + nu;
    double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]) + (int64_t)20 * Np * ld;
    double *out = SK + dm.SK_off[e];
    __shared__ double tile[kWbTile][kWbTile + 1];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    {
        const int j = j0 + tx;
        double v[kWbTile / 4];
#pragma unroll
        for (int q = 0; q < kWbTile / 4; ++q) v[q] = Kr[(int64_t)min(i0 + ty + 4 * q, f - 1) * ldk + min(j, f)];
#pragma unroll
        for (int q = 0; q < kWbTile / 4; ++q) {
            const int i = i0 + ty + 4 * q;
            if (i < f && j <= f) __builtin_nontemporal_store(v[q], E + (int64_t)i * ld + 20 * Np + j);
            tile[ty + 4 * q][tx] = j == f ? -v[q] : v[q];
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int c = ty; c < kWbTile; c += 4) {
        const int j = j0 + c, i = i0 + tx;
        if (i < f && j <= f) out[(int64_t)j * f + i] = tile[tx][c];
    }
    if (i0 == 0 && j0 == 0 && threadIdx.x < kRedMarkN)
        E[threadIdx.x] = __longlong_as_double((long long)red_mark(threadIdx.x));
}

// Gradient rows of X = A^{-1} [B | R] from the conserved ones (mixed path), into
// the right-hand columns of E: X_(c,j) = [H part of Y_j at uh_c | r] - Y_j,G X_u_c.
// Tiles over the 3 N_p rows of one component c and the f + 1 columns.  Xu: the
// conserved rows, stride x_ld, element e at x_off[e].
template <int P, int WR, int WC, int BR, int BC>
__global__ void __launch_bounds__(256, 2) k_xq(DevMesh dm, RedBuf rb, int e0, int ne, int tiles_r, int tiles_n,
                                               const double *__restrict__ Xbase, double *__restrict__ Ebase) {
    constexpr int p1 = P + 1, Np = p1 * p1 * p1;
    typedef Tile<WR, WC, BR, BC> T;
    int el, t;
    if (!xcd_item(ne, 5 * tiles_r * tiles_n, el, t)) return;
    const int e = e0 + el;
    if (dm.elem_p[e] != P || !rb.sel[el]) return;
    const int *to = dm.toff + 7 * e;
    const int f = to[6], w = f / 5, n = 20 * Np;
    const int c0 = (t % tiles_n) * T::TN, r0 = (t / tiles_n) % tiles_r * T::TM, c = t / tiles_n / tiles_r;
    if (c0 > f || r0 >= 3 * Np) return;  // uniform per block
    const int64_t ld = e_ld(n, f), ldx = x_ld(f);
    double *E = Ebase + (dm.E_off[e] - dm.E_off[e0]) + (int64_t)3 * c * Np * ld + n;
    const double *X = Xbase + (dm.x_off[e] - dm.x_off[e0]) + (int64_t)c * Np * ldx;
    const Aux ax = aux_of(rb, e, e0, Np, w);
    __shared__ __attribute__((aligned(16))) typename T::Smem sm;
    __shared__ int scol[T::TN];  // column of Y that each column starts from (-1: none)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < T::TN; i += 256) {
        const int col = c0 + i;
        int y = -1;
        if (col == f) {
            y = Np + w + c;
        } else if (col < f) {
            int lf = 0;
            while (col >= to[lf + 1]) ++lf;
            const int nfp = (to[lf + 1] - to[lf]) / 5, k = col - to[lf] - c * nfp;
            if (k >= 0 && k < nfp) y = Np + to[lf] / 5 + k;
        }
        scol[i] = y;
    }
    __syncthreads();
    const int wr = (wave / WC) * 16 * BR, wc = (wave % WC) * 16 * BC;
    acc_t acc[BR][BC];
#pragma unroll
    for (int b = 0; b < BR; ++b)
#pragma unroll
        for (int h = 0; h < BC; ++h) {
            const int y = scol[wc + 16 * h + (lane & 15)];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + wr + 16 * b + rowof(lane, q);
                acc[b][h][q] = (y >= 0 && r < 3 * Np) ? ax.Y[(int64_t)r * ax.ldy + y] : 0.0;
            }
        }
    const int rl = 3 * Np - 1 - r0;
    T::product(
        Np, [&](int r, int k) { return ax.Y + (int64_t)(r0 + min(r, rl)) * ax.ldy + k; },
        [&](int r) { return r <= rl; }, [&](int k, int h) { return X + (int64_t)k * ldx + min(c0 + h, f); },
        [&](int h) { return c0 + h <= f; }, (1u << BR) - 1u, true, sm, acc);
#pragma unroll
    for (int b = 0; b < BR; ++b)
#pragma unroll
        for (int h = 0; h < BC; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = r0 + wr + 16 * b + rowof(lane, q), col = c0 + wc + 16 * h + (lane & 15);
                if (r < 3 * Np && col <= f) __builtin_nontemporal_store(acc[b][h][q], E + (int64_t)r * ld + col);
            }
}

// A densely factored element (every element without sel) must not carry the mark.
__global__ void __launch_bounds__(256) k_clear_mark(DevMesh dm, int e0, int ne, const int *__restrict__ sel,
                                                    double *__restrict__ Ebase) {
    const int el = blockIdx.x * 256 + threadIdx.x;
    if (el >= ne || (sel && sel[el])) return;
    const int e = e0 + el, p = dm.elem_p[e], n = 20 * (p + 1) * (p + 1) * (p + 1);
    Ebase[(dm.E_off[e] - dm.E_off[e0]) + (int64_t)n * e_ld(n, dm.toff[7 * e + 6])] = 0.0;
}

// Degrees present among e0 .. e0+ne-1 (bit p), their largest trace sizes and
// largest single faces.
unsigned degrees_of(const hdg_ctx *ctx, int e0, int ne, int *maxf, int *maxb) {
    unsigned d = 0;
    for (int p = 0; p <= kMaxP; ++p) maxf[p] = maxb[p] = 0;
    for (int e = e0; e < e0 + ne; ++e) {
        const int p = ctx->elem_p[e];
        d |= 1u << p;
        maxf[p] = std::max(maxf[p], ctx->elem_f[e]);
        for (int lf = 0; lf < 6; ++lf) maxb[p] = std::max(maxb[p], ctx->toff[7 * e + lf + 1] - ctx->toff[7 * e + lf]);
    }
    return d;
}

template <int P>
void eliminate(const hdg_ctx *ctx, const RedBuf &rb, int e0, int ne, int maxf, int maxb, bool checked, bool write,
               double *E, int *info, hipStream_t s) {
    constexpr int p1 = P + 1, Np = p1 * p1 * p1;
    const DevMesh &dm = ctx->dm;
    const int w = maxf / 5;
    if (!checked) {
        const int nq = (Np + kCN - 1) / kCN, nr = (5 * Np + maxf + kCR - 1) / kCR;
        const int rest = (nq + nr - kLead<P>) | 1;
        hipLaunchKernelGGL(k_check<P>, dim3(ne * (kLead<P> + rest)), dim3(256), 0, s, dm, e0, ne, nq, rest, (const double *)E, rb.sel);
    }
    hipLaunchKernelGGL(k_minv<P>, dim3(ne), dim3(512), 0, s, dm, rb, e0, checked ? 1 : 0, write ? 1 : 0, E, info);
    const int yt = (Np + w + 5 + 63) / 64;
    hipLaunchKernelGGL(k_ysolve<P>, dim3(xcd_grid(ne, 3 * yt)), dim3(256), 0, s, dm, rb, e0, ne, yt, write ? 1 : 0, E);
    // tile shapes: a conserved tile's rows are N_p rounded up to 16, a trace
    // tile's (part of) a face's 5 (p+1)^2; the
    // columns (N_p + w + 1: 33, 82, 161, 276 for p = 1 .. 4) go in the fewest
    // tiles of a multiple of 32, the stride that keeps LDS reads off one bank
    auto go = [&](auto kernel, int TM, int TN, bool trace) {
        const int tr = trace ? 6 * ((maxb + TM - 1) / TM) : 5;
        const int tn = (Np + w + 1 + TN - 1) / TN;
        hipLaunchKernelGGL(kernel, dim3(xcd_grid(ne, tr * 5 * tn)), dim3(256), 0, s, dm, rb, e0, ne, tr, tn,
                           (const double *)E);
    };
    if constexpr (P == 4) {
        go(k_reduce<P, false, 2, 2, 4, 3>, 128, 96, false);
        go(k_reduce<P, true, 2, 2, 4, 3>, 128, 96, true);
    } else if constexpr (P == 3) {
        go(k_reduce<P, false, 1, 4, 4, 3>, 64, 192, false);
        go(k_reduce<P, true, 1, 4, 3, 3>, 48, 192, true);
    } else if constexpr (P == 2) {
        go(k_reduce<P, false, 2, 2, 1, 3>, 32, 96, false);
        go(k_reduce<P, true, 1, 4, 3, 2>, 48, 128, true);
    } else {
        go(k_reduce<P, false, 1, 4, 1, 1>, 16, 64, false);
        go(k_reduce<P, true, 1, 4, 2, 1>, 32, 64, true);
    }
}

}  // namespace

void launch_red_init(int ne, bool structured, int *info, int *sel, hipStream_t s) {
    hipLaunchKernelGGL(k_red_init, dim3((ne + 255) / 256), dim3(256), 0, s, ne, structured ? 1 : 0, info, sel);
}

// K' of every element with sel = 1 (set to 0 here, unless `checked`, where an
// element lacks the structure).  write: the gradient rows of E become
// [I | Y_j | r] (the FP64 path's factored form).
int launch_red_eliminate(const hdg_ctx *ctx, const RedBuf &rb, int e0, int ne, bool checked, bool write, double *E,
                         int *info, hipStream_t s) {
    int maxf[kMaxP + 1], maxb[kMaxP + 1];
    const unsigned deg = degrees_of(ctx, e0, ne, maxf, maxb);
    if (deg & 2u) eliminate<1>(ctx, rb, e0, ne, maxf[1], maxb[1], checked, write, E, info, s);
    if (deg & 4u) eliminate<2>(ctx, rb, e0, ne, maxf[2], maxb[2], checked, write, E, info, s);
    if (deg & 8u) eliminate<3>(ctx, rb, e0, ne, maxf[3], maxb[3], checked, write, E, info, s);
    if (deg & 16u) eliminate<4>(ctx, rb, e0, ne, maxf[4], maxb[4], checked, write, E, info, s);
    int rows = 0;
    for (int e = e0; e < e0 + ne; ++e) rows = std::max(rows, red_n(ctx->elem_n[e] / 20) + ctx->elem_f[e]);
    hipLaunchKernelGGL(k_rescol, dim3((rows + 255) / 256, ne), dim3(256), 0, s, ctx->dm, rb, e0, (const double *)E);
    return (int)hipGetLastError();
}

int launch_red_writeback(const hdg_ctx *ctx, const RedBuf &rb, int e0, int ne, double *E, double *SK, hipStream_t s) {
    int nu = 0, f = 0;
    for (int e = e0; e < e0 + ne; ++e) {
        nu = std::max(nu, ctx->elem_n[e] / 4);
        f = std::max(f, ctx->elem_f[e]);
    }
    hipLaunchKernelGGL(k_wb_rows, dim3((nu + 3) / 4, ne), dim3(256), 0, s, ctx->dm, rb, e0, E);
    hipLaunchKernelGGL(k_wb_trace, dim3(f / kWbTile + 1, (f + kWbTile - 1) / kWbTile, ne), dim3(256), 0, s, ctx->dm, rb, e0, E, SK);
    return (int)hipGetLastError();
}

int launch_red_xq(const hdg_ctx *ctx, const RedBuf &rb, int e0, int ne, const double *Xu, double *E, hipStream_t s) {
    int maxf[kMaxP + 1], maxb[kMaxP + 1];
    const unsigned deg = degrees_of(ctx, e0, ne, maxf, maxb);
    auto go = [&](auto kernel, int p, int TM) {
        const int Np = (p + 1) * (p + 1) * (p + 1), tr = (3 * Np + TM - 1) / TM, tn = (maxf[p] + 1 + 127) / 128;
        hipLaunchKernelGGL(kernel, dim3(xcd_grid(ne, 5 * tr * tn)), dim3(256), 0, s, ctx->dm, rb, e0, ne, tr, tn, Xu, E);
    };
    // 128 columns; rows: 24, 81, 192, 375 for p = 1 .. 4
    if (deg & 2u) go(k_xq<1, 1, 4, 2, 2>, 1, 32);
    if (deg & 4u) go(k_xq<2, 2, 2, 3, 4>, 2, 96);
    if (deg & 8u) go(k_xq<3, 1, 4, 4, 2>, 3, 64);
    if (deg & 16u) go(k_xq<4, 2, 2, 4, 4>, 4, 128);
    return (int)hipGetLastError();
}

int launch_red_clear_mark(const hdg_ctx *ctx, int e0, int ne, const int *sel, double *E, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_mark, dim3((ne + 255) / 256), dim3(256), 0, s, ctx->dm, e0, ne, sel, E);
    return (int)hipGetLastError();
}

}  // namespace hdg
