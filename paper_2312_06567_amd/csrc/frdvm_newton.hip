// Conservative discrete equilibrium (FP64 Newton), stand-alone collision,
// moment output and global totals (gfx950).
//
// Paper, Section "Numerical method", eq. (discrete_compatibility): the
// modified equilibrium g' must have exactly the discrete moments of f,
// M.(g' psi) = M.(f psi).  Following Mieussens it is the analytic
// equilibrium at a modified state Q', i.e. an exponential of a quadratic in
// u, found per solution point by a small nonlinear solve (Newton).  Section
// "Governing equations": tau = mu/(Pr P), ES-BGK tensor
// T = theta/Pr I + (1 - 1/Pr) Pi/rho.
//
// Formulation (the same reading as the CPU oracle): in the frame
// c = (u - U)/sqrt(theta) with weights wt = w theta^-3/2 the five equations
// are sum_k wt_k (1, c_k, |c_k|^2/2) exp(z0 + z.c_k - z4 q(c_k)/2) =
// (1, 0, 0, 0, 3/2), q = |c|^2 (BGK) or c^T A c with A = theta T^-1 (ES-BGK),
// and g' = rho wt exp(...).
//
// BGK kernel: one to eight lanes per point (by the number of points; the
// result is the same for all).  On a tensor velocity grid the BGK exponential
// factorises per axis, so each Newton iteration costs 3 n_v exponentials and
// 1-D power sums instead of n_v^3 terms.
// ES kernel: a wave per point for the sums, one thread per point for the
// iteration around them; the state the two share lives in LDS.  The sums come
// in three forms, chosen per evaluation by the range of its exponents.
// Starting points: cold (continuous equilibrium of the moments), warm (the
// previous solution at the point) or learned (cold + a correction predicted
// by the MLP kernels; the start with the smaller residual is kept, so the
// learned start never costs more than one extra evaluation).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "frdvm_common.h"
#include "frdvm_dev.h"

namespace frdvm {

namespace {

struct NewtonArgs {
    VGrid vg;
    int64_t npts;
    int nmom;
    const double *wax;   // [3][64]
    const double *Q;     // [npts][nmom]
    const double *Qpart; // nparts > 1: [nparts][npts][nmom], the moments as parts to be added in order
    int nparts;
    double *eq;          // [npts][kEqW]
    double *z;           // [npts][5]
    double *prim;        // [npts][5]
    unsigned long long *stats;  // [kHist] histogram, [kHist] fallback, [kHist+1] ES guard
    unsigned long long *maxres;
    int32_t *pt_iters;   // optional per-point outputs
    int32_t *pt_evals;
    int32_t *pt_status;
    double *pt_resid;
    double Pr, mu_ref, theta_ref, omega, theta_s;
    int visc_law;
    double tol;
    int max_iter;
    int guess;
    const float *dz_guess;  // [npts][5] learned correction (guess == MLP)
    int use_fact;           // ES: factorised sums
    int nph, nrow, es_pts;  // ES: lanes that share an x node, y nodes padded to them, points per workgroup
    double delta;           // internal degrees of freedom (the reduced pair)
    double *gfp;            // [npts] delta theta / 2 per point (pair only, else null)
};

// Total energy of a moment record: E (BGK), half the trace of the raw second
// moments (ES), plus the integral of G in the last slot for the reduced pair
// (records of 6 / 11 values).
__device__ __forceinline__ double record_energy(const double *q, int nmom) {
    switch (nmom) {
        case 5: return q[4];
        case 6: return q[4] + q[5];
        case 10: return 0.5 * (q[4] + q[5] + q[6]);
        default: return 0.5 * (q[4] + q[5] + q[6]) + q[10];
    }
}

constexpr double kTwoPi = 6.283185307179586476925286766559;
// Line search: the step is halved after each rejected trial point (z4 <= 0 or
// too little decrease of |r|_2); a solve may reject at most this many trial
// points in total, then it stops (fallback unless at the rounding floor).
constexpr int kRejectBudget = 40;

// Velocity node umin + i du, rounded as two separate operations (no FMA
// contraction) so that every kernel sees the node values the host sees.
__device__ __forceinline__ double gridu(const VGrid &vg, int d, int i) {
    return __dadd_rn(vg.umin[d], __dmul_rn((double)i, vg.du[d]));
}

__device__ double viscosity(const NewtonArgs &A, double th) {
    if (A.visc_law == 1)
        return A.mu_ref * pow(th / A.theta_ref, 1.5) * (A.theta_ref + A.theta_s) / (th + A.theta_s);
    return A.mu_ref * pow(th / A.theta_ref, A.omega);
}

// Gaussian elimination with partial pivoting on a 5x5 system.  Every loop is
// unrolled so the row exchange is a set of selects on registers.
__device__ __forceinline__ bool solve5(const double J[5][5], const double b[5], double x[5]) {
    double M[5][6];
#pragma unroll
    for (int i = 0; i < 5; ++i) {
#pragma unroll
        for (int j = 0; j < 5; ++j) M[i][j] = J[i][j];
        M[i][5] = b[i];
    }
    bool ok = true;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        double best = fabs(M[c][c]);
        int piv = c;
#pragma unroll
        for (int r = c + 1; r < 5; ++r)
            if (fabs(M[r][c]) > best) { best = fabs(M[r][c]); piv = r; }
        ok = ok && (best > 0.0);
#pragma unroll
        for (int r = c + 1; r < 5; ++r) {
            const bool sw = (r == piv);
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                double a = M[c][j], bb = M[r][j];
                M[c][j] = sw ? bb : a;
                M[r][j] = sw ? a : bb;
            }
        }
        const double inv = 1.0 / M[c][c];
#pragma unroll
        for (int r = c + 1; r < 5; ++r) {
            const double fct = M[r][c] * inv;
#pragma unroll
            for (int j = c; j < 6; ++j) M[r][j] -= fct * M[c][j];
        }
    }
#pragma unroll
    for (int i = 4; i >= 0; --i) {
        double s = M[i][5];
#pragma unroll
        for (int j = i + 1; j < 5; ++j) s -= M[i][j] * x[j];
        x[i] = s / M[i][i];
    }
    return ok;
}

__device__ __forceinline__ double norm2_5(const double r[5]) {
    return sqrt(r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + r[3] * r[3] + r[4] * r[4]);
}
__device__ __forceinline__ double normi_5(const double r[5]) {
    double m = 0;
#pragma unroll
    for (int a = 0; a < 5; ++a) m = fmax(m, fabs(r[a]));
    return m;
}

// Raw sums over the velocity grid:
//   S0 = sum wt e, Sc_i = sum wt c_i e, Scc (xx yy zz xy xz yz), Sq = sum wt q e,
//   Scq_i = sum wt c_i q e, Sc2c_i = sum wt |c|^2 c_i e, Sc2q = sum wt |c|^2 q e.
struct Sums {
    double S0, Sc[3], Scc[6], Sq, Scq[3], Sc2c[3], Sc2q;
};

// Residual and Jacobian; rows psi = (1, c, |c|^2/2), columns d/dz = (1, c, -q/2).
__device__ __forceinline__ void assemble(const Sums &s, double r[5], double J[5][5]) {
    const double c2 = s.Scc[0] + s.Scc[1] + s.Scc[2];
    r[0] = s.S0 - 1.0;
    r[1] = s.Sc[0];
    r[2] = s.Sc[1];
    r[3] = s.Sc[2];
    r[4] = 0.5 * c2 - 1.5;
    J[0][0] = s.S0; J[0][1] = s.Sc[0]; J[0][2] = s.Sc[1]; J[0][3] = s.Sc[2]; J[0][4] = -0.5 * s.Sq;
    J[1][0] = s.Sc[0]; J[1][1] = s.Scc[0]; J[1][2] = s.Scc[3]; J[1][3] = s.Scc[4]; J[1][4] = -0.5 * s.Scq[0];
    J[2][0] = s.Sc[1]; J[2][1] = s.Scc[3]; J[2][2] = s.Scc[1]; J[2][3] = s.Scc[5]; J[2][4] = -0.5 * s.Scq[1];
    J[3][0] = s.Sc[2]; J[3][1] = s.Scc[4]; J[3][2] = s.Scc[5]; J[3][3] = s.Scc[2]; J[3][4] = -0.5 * s.Scq[2];
    J[4][0] = 0.5 * c2; J[4][1] = 0.5 * s.Sc2c[0]; J[4][2] = 0.5 * s.Sc2c[1]; J[4][3] = 0.5 * s.Sc2c[2];
    J[4][4] = -0.25 * s.Sc2q;
}

// BGK sums by axis factorisation: e = exp(z0) prod_d exp(z_d c_d - z4 c_d^2 / 2).
// LPP lanes share a point.  Whatever LPP is, the nodes of an axis are summed in
// eight classes (i mod 8), and the classes p0 .. p7 added as ((p0 + p1) +
// (p2 + p3)) + ((p4 + p5) + (p6 + p7)): a lane adds those of its own classes,
// 8 / LPP consecutive ones, a butterfly over the lanes the rest (every lane
// gets the same bits).  So a point's result does not depend on the batch it is
// solved in.  Up to four classes are walked side by side: an exponential is a
// chain of its own.
template <int LPP>
__device__ void sums_bgk(const NewtonArgs &A, int lane, const double U[3], double ist, const double z[5], Sums &s) {
    constexpr int NC = 8 / LPP, W = NC < 4 ? NC : 4;  // classes of a lane, and those it walks side by side
    double m[3][5];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int nv = A.vg.nv[d];
        const double zd = z[1 + d], hz = 0.5 * z[4];
        // (a node past the end has weight zero and the last node's velocity)
#pragma unroll 1
        for (int pass = 0; pass < NC / W; ++pass) {
            double a[W][5] = {};
            for (int i0 = NC * lane + W * pass; i0 < nv; i0 += 8)
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const int i = i0 + w;
                    const double c = (gridu(A.vg, d, W == 1 || i < nv ? i : nv - 1) - U[d]) * ist;
                    double t = A.wax[64 * d + i] * ist * exp(c * (zd - hz * c));
#pragma unroll
                    for (int e = 0; e < 5; ++e) {
                        a[w][e] += t;
                        t *= c;
                    }
                }
#pragma unroll
            for (int o = 1; o < W; o *= 2)
#pragma unroll
                for (int w = 0; w < W; w += 2 * o)
#pragma unroll
                    for (int e = 0; e < 5; ++e) a[w][e] += a[w + o][e];
#pragma unroll
            for (int e = 0; e < 5; ++e) m[d][e] = pass ? m[d][e] + a[0][e] : a[0][e];
        }
    }
#pragma unroll
    for (int o = 1; o < LPP; o *= 2)
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int a = 0; a < 5; ++a) m[d][a] += __shfl_xor(m[d][a], o, LPP);
    const double K = exp(z[0]) * m[0][0] * m[1][0] * m[2][0];
    double Pn[3][5];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double inv = 1.0 / m[d][0];
#pragma unroll
        for (int a = 0; a < 5; ++a) Pn[d][a] = m[d][a] * inv;
    }
    s.S0 = K;
#pragma unroll
    for (int i = 0; i < 3; ++i) s.Sc[i] = K * Pn[i][1];
    s.Scc[0] = K * Pn[0][2]; s.Scc[1] = K * Pn[1][2]; s.Scc[2] = K * Pn[2][2];
    s.Scc[3] = K * Pn[0][1] * Pn[1][1];
    s.Scc[4] = K * Pn[0][1] * Pn[2][1];
    s.Scc[5] = K * Pn[1][1] * Pn[2][1];
    s.Sq = s.Scc[0] + s.Scc[1] + s.Scc[2];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double t = 0;
#pragma unroll
        for (int mm = 0; mm < 3; ++mm) t += (mm == i) ? Pn[i][3] : Pn[i][1] * Pn[mm][2];
        s.Scq[i] = K * t;
        s.Sc2c[i] = K * t;
    }
    double t4 = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) t4 += (a == b) ? Pn[a][4] : Pn[a][2] * Pn[b][2];
    s.Sc2q = K * t4;
}

// ---- ES sums: one wave per solution point --------------------------------
// The state of a point's iteration that its wave and its owner thread share
// (see k_newton_es): the frame (U, theta^-1/2, A = theta T^-1 as xx yy zz xy
// xz yz), the point z under evaluation, and two sets of sums.
struct EsPoint {
    double U[3], ist, A[6], z[5];
    Sums s[2];
    int req, tgt;  // requested evaluation (kReq*; 0: none) and the set it goes to
};
// kReqJac: all 18 sums, not the residual's 5 only; kReqWide, kReqDirect: the form of the sums (sums_form)
constexpr int kReqSums = 1, kReqJac = 2, kReqWide = 4, kReqDirect = 8;

// Sums over the 64 lanes of N values each, value k left with one lane of the
// wave: each step halves the values a lane carries (it keeps one half and
// sends the other to its partner), 21 exchanges for 18 values instead of the
// 108 of a butterfly per value.  Returns the lane's sum; `slot` is the index
// of its value (lanes without one: -1).
template <int N, int O>
__device__ __forceinline__ double spread_sum(const double *v, int lane, int base, int n_valid, int &slot) {
    const bool up = (lane & O) != 0;
    constexpr int H = (N + 1) / 2;  // values kept (an odd count is padded with a zero)
    double w[H];
    if constexpr (N == 1) {
        w[0] = v[0] + __shfl_xor(v[0], O);
    } else {
#pragma unroll
        for (int k = 0; k < H; ++k) {
            const double lo = v[k], hi = k + H < N ? v[k + H] : 0.0;
            w[k] = (up ? hi : lo) + __shfl_xor(up ? lo : hi, O);
        }
        base += up ? H : 0;
        n_valid = up ? (n_valid - H < H ? n_valid - H : H) : (n_valid < H ? n_valid : H);
    }
    if constexpr (O == 1) {
        slot = n_valid > 0 ? base : -1;
        return w[0];
    } else {
        return spread_sum<H, O / 2>(w, lane, base, n_valid, slot);
    }
}
template <int N>
__device__ __forceinline__ void store_sums(const double *v, int lane, double *out) {
    int slot;
    const double t = spread_sum<N, 32>(v, lane, 0, N, slot);
    if (slot >= 0) out[slot] = t;  // (lanes that share a value write the same bits)
}

// Sums over all velocity nodes, lane-strided, without factorisation.  With
// JAC == false only the residual sums S0, Sc and the trace of Scc (stored in
// Scc[0], the other diagonal entries zero) are formed.
template <bool JAC>
__device__ void sums_es(const NewtonArgs &A, int lane, const EsPoint &p, double *out) {
    double acc[18];
#pragma unroll
    for (int a = 0; a < 18; ++a) acc[a] = 0.0;
    const VGrid &vg = A.vg;
    const double ist = p.ist, wscale = ist * ist * ist;
    for (int k = lane; k < vg.nu; k += 64) {
        const int i = k % vg.nv[0], j = (k / vg.nv[0]) % vg.nv[1], l = k / (vg.nv[0] * vg.nv[1]);
        const double c0 = (gridu(vg, 0, i) - p.U[0]) * ist;
        const double c1 = (gridu(vg, 1, j) - p.U[1]) * ist;
        const double c2 = (gridu(vg, 2, l) - p.U[2]) * ist;
        const double q = p.A[0] * c0 * c0 + p.A[1] * c1 * c1 + p.A[2] * c2 * c2 +
                         2.0 * (p.A[3] * c0 * c1 + p.A[4] * c0 * c2 + p.A[5] * c1 * c2);
        const double w = A.wax[i] * A.wax[64 + j] * A.wax[128 + l] * wscale;
        const double ev = w * exp(p.z[0] + p.z[1] * c0 + p.z[2] * c1 + p.z[3] * c2 - 0.5 * p.z[4] * q);
        const double cc = c0 * c0 + c1 * c1 + c2 * c2;
        acc[0] += ev;
        acc[1] += ev * c0; acc[2] += ev * c1; acc[3] += ev * c2;
        if (!JAC) {
            acc[4] += ev * cc;
            continue;
        }
        const double eq_ = ev * q, ec = ev * cc;
        acc[4] += ev * c0 * c0; acc[5] += ev * c1 * c1; acc[6] += ev * c2 * c2;
        acc[7] += ev * c0 * c1; acc[8] += ev * c0 * c2; acc[9] += ev * c1 * c2;
        acc[10] += eq_;
        acc[11] += eq_ * c0; acc[12] += eq_ * c1; acc[13] += eq_ * c2;
        acc[14] += ec * c0; acc[15] += ec * c1; acc[16] += ec * c2;
        acc[17] += ec * q;
    }
    store_sums<JAC ? 18 : 5>(acc, lane, out);
    if (!JAC && lane == 0) out[5] = out[6] = 0.0;
}

// ---- factorised sums ----
// On a tensor grid the exponent z0 + z.c - z4 c^T A c / 2 splits into one-axis
// factors and the cross factors exp(k01 c0 c1), exp(k02 c0 c2), exp(k12 c1 c2)
// (k_ab = -z4 A_ab).  Each lane keeps one x node (row) i and walks every
// nph-th y node j (nph = 64 / n0 lanes share a row).  Along l the two factors
// with c2 are geometric on a uniform grid, with ratio Ra(i) Rb(j), so
//   T_e(i,j) = sum_l Z(l) c2_l^e (Ra Rb)^l
// are polynomials in the ratio: one multiply-add per (pair, node, e) by
// Horner's rule on the table Z c2^e, shared by the pairs a lane works on
// together.  Along j the factor of c0 c1 is geometric too (no table), and the
// T_e are collected with powers of c1 into the row's sums over j of c1^b c2^e,
// b + e <= 4 (15; residual: b + e <= 2, 6), from which the lane's c0 gives its
// share of the 18 (5) sums once per evaluation.  What this bounds: FP64
// multiply-adds, 5 (3) n0 n1 n2 / 64 of them per lane; a pair-by-pair finish
// with two-axis tables cost as much again, and its tables (5.6 KB per point
// at 20^3, now 1.6) held the occupancy.

// Doubles of one wave's tables: per y node factor with weight, Rb, c1 (padded
// with zero weights to the same number of nodes for every lane); Z c2^e.
__host__ __device__ inline int es_table_doubles(const NewtonArgs &A) { return 3 * A.nrow + 5 * A.vg.nv[2]; }

__device__ __forceinline__ void lds_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Index of the row sum of c1^b c2^e: for e = 0..D, b = 0..D-e.
template <int D>
__device__ __forceinline__ constexpr int row_sum(int b, int e) {
    int o = 0;
    for (int x = 0; x < e; ++x) o += D + 1 - x;
    return o + b;
}

// A y node's T_e times its factor w, with the powers of its c1, into the row sums.
template <int D>
__device__ __forceinline__ void collect_node(double w, double c1, const double (&T)[D + 1], double *M) {
#pragma unroll
    for (int e = 0; e <= D; ++e) {
        double t = w * T[e];
#pragma unroll
        for (int x = 0; x <= D - e; ++x) {
            M[row_sum<D>(x, e)] += t;
            if (x < D - e) t *= c1;
        }
    }
}

// B y nodes j0, j0 + nph, ... of a lane's row.  W: the row's factor at j0
// (times Pr per node); D: degree of the sums (4 or 2).
template <int B, int D>
__device__ __forceinline__ void row_block(const double *tb, int np, int n2, int j0, int nph, double Ra, double Pr,
                                          double &W, double *M) {
    const double *yj = tb + j0, *zc = tb + 3 * np;
    double r[B], T[B][D + 1];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        r[b] = Ra * yj[np + b * nph];
#pragma unroll
        for (int e = 0; e <= D; ++e) T[b][e] = 0.0;
    }
#pragma unroll 2
    for (int l = n2 - 1; l >= 0; --l) {
#pragma unroll
        for (int e = 0; e <= D; ++e) {
            const double z = zc[5 * l + e];
#pragma unroll
            for (int b = 0; b < B; ++b) T[b][e] = fma(T[b][e], r[b], z);
        }
    }
#pragma unroll
    for (int b = 0; b < B; ++b) {
        const double w = W * yj[b * nph], c1 = yj[2 * np + b * nph];
        W *= Pr;
        collect_node<D>(w, c1, T[b], M);
    }
}

// The same for the y nodes j[b] in the wide form: the powers of the ratio
// count from node lc, Horner's rule from either end of the z axis.
template <int B, int D>
__device__ __forceinline__ void row_block_wide(const double *tb, int np, int n2, int lc, const int (&j)[B], double Ra,
                                               double Pr, double &W, double *M) {
    const double *zc = tb + 3 * np;
    double r[B], T[B][D + 1], L[B][D + 1];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        r[b] = Ra * tb[np + j[b]];
#pragma unroll
        for (int e = 0; e <= D; ++e) T[b][e] = L[b][e] = 0.0;
    }
    for (int l = n2 - 1; l >= lc; --l)
#pragma unroll
        for (int e = 0; e <= D; ++e) {
            const double z = zc[5 * l + e];
#pragma unroll
            for (int b = 0; b < B; ++b) T[b][e] = fma(T[b][e], r[b], z);
        }
#pragma unroll
    for (int b = 0; b < B; ++b) r[b] = 1.0 / r[b];
    for (int l = 0; l < lc; ++l)
#pragma unroll
        for (int e = 0; e <= D; ++e) {
            const double z = zc[5 * l + e];
#pragma unroll
            for (int b = 0; b < B; ++b) L[b][e] = fma(L[b][e], r[b], z);
        }
#pragma unroll
    for (int b = 0; b < B; ++b) {
#pragma unroll
        for (int e = 0; e <= D; ++e) T[b][e] = fma(L[b][e], r[b], T[b][e]);
        const double w = W * tb[j[b]], c1 = tb[2 * np + j[b]];
        W *= Pr;
        collect_node<D>(w, c1, T[b], M);
    }
}

// z node the wide form's powers count from: the one nearest the mean.
__device__ __forceinline__ int wide_centre(const VGrid &vg, const EsPoint &p) {
    if (vg.nv[2] == 1) return 0;
    return (int)fmin(fmax(rint((p.U[2] - vg.umin[2]) / vg.du[2]), 0.0), (double)(vg.nv[2] - 1));
}

template <bool JAC, bool WIDE>
__device__ __forceinline__ void sums_es_fact(const NewtonArgs &A, int lane, double *tb, const EsPoint &p, double *out) {
    constexpr int D = JAC ? 4 : 2, NM = (D + 1) * (D + 2) / 2;
    // nothing derived from the lane is kept in registers between evaluations
    asm volatile("" : "+v"(lane));
    const VGrid &vg = A.vg;
    const int n0 = vg.nv[0], n1 = vg.nv[1], n2 = vg.nv[2], nph = A.nph;
    const double ist = p.ist, z4 = p.z[4], hz = 0.5 * z4;
    const double k01 = -z4 * p.A[3], k02 = -z4 * p.A[4], k12 = -z4 * p.A[5];
    const int lc = WIDE ? __builtin_amdgcn_readfirstlane(wide_centre(vg, p)) : 0;  // the node the ratio's powers count from
    const double c2a = (gridu(vg, 2, lc) - p.U[2]) * ist, dl2 = vg.du[2] * ist, dl1 = vg.du[1] * ist;
    lds_wave_sync();  // previous evaluation's readers are done with the tables
    // the y and z tables: one exponential per entry, the entries of all three
    // tables dealt to the lanes together
    const int np = A.nrow;
    for (int t = lane; t < np - n1; t += 64) {
        tb[n1 + t] = tb[2 * np + n1 + t] = 0.0;
        tb[np + n1 + t] = WIDE ? 1.0 : 0.0;  // (the wide form divides by it)
    }
    for (int t = lane; t < 2 * n1 + n2; t += 64) {
        const bool isz = t >= 2 * n1, isr = !isz && t >= n1;
        const int i = isz ? t - 2 * n1 : (isr ? t - n1 : t);
        const double c = isz ? (gridu(vg, 2, i) - p.U[2]) * ist : (gridu(vg, 1, i) - p.U[1]) * ist;
        const double own = isz ? c * (p.z[3] - hz * p.A[2] * c) : c * (p.z[2] - hz * p.A[1] * c) + k12 * c * c2a;
        const double v = exp(isr ? k12 * c * dl2 : own);
        if (isz) {
            double q = A.wax[128 + i] * ist * v;
#pragma unroll
            for (int e = 0; e <= D; ++e) {
                tb[3 * np + 5 * i + e] = q;
                q *= c;
            }
        } else if (isr) {
            tb[np + i] = v;
        } else {
            tb[i] = A.wax[64 + i] * ist * v;
            tb[2 * np + i] = c;
        }
    }
    // the lane's row: x node i, y nodes ph, ph + nph, ...
    const int ph = lane / n0, i = lane - ph * n0;
    const bool live = ph < nph;  // (other lanes follow along with weight zero)
    const int j0 = live ? ph : 0;
    const double c0 = (gridu(vg, 0, i) - p.U[0]) * ist;
    // (wide: from the end of the lane's nodes where the row's factor is largest)
    const int cv = (n1 - j0 + nph - 1) / nph;
    const bool down = WIDE && k01 * c0 > 0.0;
    const double c1p = (gridu(vg, 1, down ? j0 + nph * (cv - 1) : j0) - p.U[1]) * ist;
    const double Ra = exp(k02 * c0 * dl2);
    const double Pr = exp(WIDE ? -fabs(k01 * c0 * dl1) * nph : k01 * c0 * dl1 * nph);
    double W = A.wax[i] * ist * exp(p.z[0] + c0 * (p.z[1] - hz * p.A[0] * c0) + k02 * c0 * c2a + k01 * c0 * c1p);
    W = live ? W : 0.0;
    double M[NM];
#pragma unroll
    for (int a = 0; a < NM; ++a) M[a] = 0.0;
    lds_wave_sync();
    const int cnt = np / nph;
    int m = 0;
    if constexpr (WIDE) {
        // the lane's m-th node (past its last one: a padded node)
        auto node = [&](int q) { return q < cv ? j0 + nph * (down ? cv - 1 - q : q) : np - 1; };
        for (; m + 2 <= cnt; m += 2) row_block_wide<2, D>(tb, np, n2, lc, {node(m), node(m + 1)}, Ra, Pr, W, M);
        if (m < cnt) row_block_wide<1, D>(tb, np, n2, lc, {node(m)}, Ra, Pr, W, M);
    } else {
        for (; m + 4 <= cnt; m += 4) row_block<4, D>(tb, np, n2, j0 + nph * m, nph, Ra, Pr, W, M);
        if (cnt - m == 3) row_block<3, D>(tb, np, n2, j0 + nph * m, nph, Ra, Pr, W, M);
        else if (cnt - m == 2) row_block<2, D>(tb, np, n2, j0 + nph * m, nph, Ra, Pr, W, M);
        else if (cnt - m == 1) row_block<1, D>(tb, np, n2, j0 + nph * m, nph, Ra, Pr, W, M);
    }
    auto m_ = [&](int b, int e) { return M[row_sum<D>(b, e)]; };
    const double cc = c0 * c0;
    if constexpr (!JAC) {
        const double v[5] = {m_(0, 0), c0 * m_(0, 0), m_(1, 0), m_(0, 1), fma(cc, m_(0, 0), m_(2, 0) + m_(0, 2))};
        store_sums<5>(v, lane, out);
        if (lane == 0) out[5] = out[6] = 0.0;
    } else {
        const double a00 = p.A[0] * cc, t01 = 2.0 * p.A[3] * c0, t02 = 2.0 * p.A[4] * c0, t12 = 2.0 * p.A[5];
        // sum of q c1^b c2^e, and of |c|^2 c1^b c2^e
        auto q_ = [&](int b, int e) {
            double t = a00 * m_(b, e);
            t = fma(t01, m_(b + 1, e), t);
            t = fma(p.A[1], m_(b + 2, e), t);
            t = fma(t02, m_(b, e + 1), t);
            t = fma(t12, m_(b + 1, e + 1), t);
            return fma(p.A[2], m_(b, e + 2), t);
        };
        auto s_ = [&](int b, int e) { return fma(cc, m_(b, e), m_(b + 2, e) + m_(b, e + 2)); };
        const double q0 = q_(0, 0);
        const double v[18] = {m_(0, 0), c0 * m_(0, 0), m_(1, 0), m_(0, 1),                                 // S0, Sc
                              cc * m_(0, 0), m_(2, 0), m_(0, 2), c0 * m_(1, 0), c0 * m_(0, 1), m_(1, 1),   // Scc
                              q0, c0 * q0, q_(1, 0), q_(0, 1),                                             // Sq, Scq
                              c0 * s_(0, 0), s_(1, 0), s_(0, 1), fma(cc, q0, q_(2, 0) + q_(0, 2))};        // Sc2c, Sc2q
        store_sums<18>(v, lane, out);
    }
}

// The form of an evaluation's sums, by how far its factors reach in the FP64
// range (0: factorised; kReqWide, kReqDirect).
// Factorised: the largest |exponents| of the cross factors over the grid
// (their sum bounds the lanes' start values, twice it the range of a geometric
// factor), the peaks of the one-axis factors, and the largest value W of a row
// can take in the padded y nodes: it goes on growing there, and only a finite
// W times their zero weight is zero (8 x 9 nodes have 7 padded ones, 2.75 times
// as far from the mean as the last node).
// Wide: a row's W only falls from its largest value, and the ratio's powers
// reach to either side of the node nearest the mean, so that the exponents of
// each cross factor may be twice as large.  Half the nodes at a time and their
// z tables read twice: 1.4 times the time of the factorised form, where the
// direct sums take 10 times (cold solves of 64,000 sheared states, 24^3
// velocities, three evaluations: 1.10, 1.52 and 10.7 ms).
// Any other evaluation sums over the nodes one by one.
__device__ __forceinline__ int sums_form(const NewtonArgs &A, const EsPoint &p) {
    if (!A.use_fact) return kReqDirect;
    const VGrid &vg = A.vg;
    const double z4 = p.z[4];
    double lo[3], hi[3], cm[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[d] = (gridu(vg, d, 0) - p.U[d]) * p.ist;
        hi[d] = (gridu(vg, d, vg.nv[d] - 1) - p.U[d]) * p.ist;
        cm[d] = fmax(fabs(lo[d]), fabs(hi[d]));
    }
    double peak = fabs(p.z[0]);
#pragma unroll
    for (int d = 0; d < 3; ++d) peak = fmax(peak, p.z[1 + d] * p.z[1 + d] / (2.0 * z4 * p.A[d]));
    const double a01 = z4 * fabs(p.A[3]), a02 = z4 * fabs(p.A[4]), a12 = z4 * fabs(p.A[5]);
    const double cross = a01 * cm[0] * cm[1] + a02 * cm[0] * cm[2] + a12 * cm[1] * cm[2];
    const double c1p = fmax(cm[1], fabs(gridu(vg, 1, A.nrow - 1) - p.U[1]) * p.ist);
    const double row = cm[0] * (a01 * c1p + a02 * cm[2]);
    if (cross <= 300.0 && row <= 650.0 && peak <= 25.0) return 0;  // (false for NaN)
    // the largest exponent of the c0 c1 factor, that of a ratio over its reach,
    // and that of both at the centre node
    const double k01 = -z4 * p.A[3], k02 = -z4 * p.A[4], k12 = -z4 * p.A[5];
    const double up01 = fmax(fmax(k01 * lo[0] * lo[1], k01 * lo[0] * hi[1]), fmax(k01 * hi[0] * lo[1], k01 * hi[0] * hi[1]));
    const double kap = fmax(fmax(fabs(k02 * lo[0] + k12 * lo[1]), fabs(k02 * lo[0] + k12 * hi[1])),
                            fmax(fabs(k02 * hi[0] + k12 * lo[1]), fabs(k02 * hi[0] + k12 * hi[1])));
    const double cc = (gridu(vg, 2, wide_centre(vg, p)) - p.U[2]) * p.ist;
    const double reach = kap * fmax(cc - lo[2], hi[2] - cc), start = up01 + (a02 * cm[0] + a12 * cm[1]) * fabs(cc);
    return start <= 640.0 && reach <= 640.0 && peak <= 30.0 ? kReqWide : kReqDirect;
}

// Smallest eigenvalue of a symmetric 3x3 matrix (closed form, trigonometric).
__device__ double sym3_min_eig(const double T[3][3]) {
    const double p1 = T[0][1] * T[0][1] + T[0][2] * T[0][2] + T[1][2] * T[1][2];
    const double q = (T[0][0] + T[1][1] + T[2][2]) / 3.0;
    if (p1 == 0.0) return fmin(T[0][0], fmin(T[1][1], T[2][2]));
    const double p2 = (T[0][0] - q) * (T[0][0] - q) + (T[1][1] - q) * (T[1][1] - q) +
                      (T[2][2] - q) * (T[2][2] - q) + 2.0 * p1;
    const double p = sqrt(p2 / 6.0);
    double B[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) B[i][j] = (T[i][j] - (i == j ? q : 0.0)) / p;
    const double detB = B[0][0] * (B[1][1] * B[2][2] - B[1][2] * B[2][1]) -
                        B[0][1] * (B[1][0] * B[2][2] - B[1][2] * B[2][0]) +
                        B[0][2] * (B[1][0] * B[2][1] - B[1][1] * B[2][0]);
    const double r = fmin(1.0, fmax(-1.0, 0.5 * detB));
    const double phi = acos(r) / 3.0;
    return q + 2.0 * p * cos(phi + kTwoPi / 3.0);
}

__device__ __forceinline__ double det3(const double M[3][3]) {
    return M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) - M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
           M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]);
}

__device__ __forceinline__ void inv3(const double M[3][3], double R[3][3]) {
    const double d = 1.0 / det3(M);
    R[0][0] = (M[1][1] * M[2][2] - M[1][2] * M[2][1]) * d;
    R[0][1] = (M[0][2] * M[2][1] - M[0][1] * M[2][2]) * d;
    R[0][2] = (M[0][1] * M[1][2] - M[0][2] * M[1][1]) * d;
    R[1][0] = (M[1][2] * M[2][0] - M[1][0] * M[2][2]) * d;
    R[1][1] = (M[0][0] * M[2][2] - M[0][2] * M[2][0]) * d;
    R[1][2] = (M[0][2] * M[1][0] - M[0][0] * M[1][2]) * d;
    R[2][0] = (M[1][0] * M[2][1] - M[1][1] * M[2][0]) * d;
    R[2][1] = (M[0][1] * M[2][0] - M[0][0] * M[2][1]) * d;
    R[2][2] = (M[0][0] * M[1][1] - M[0][1] * M[1][0]) * d;
}

// Equilibrium record and primitive output from the converged parameters.
__device__ void write_point(const NewtonArgs &A, int64_t pt, double rho, const double U[3], double th,
                            const double Am[3][3], const double z[5], double inv_tau, double res) {
    double Ai[3][3];
    inv3(Am, Ai);
    double m[3], mAm = 0;
#pragma unroll
    for (int i = 0; i < 3; ++i) m[i] = (Ai[i][0] * z[1] + Ai[i][1] * z[2] + Ai[i][2] * z[3]) / z[4];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) mAm += m[i] * Am[i][j] * m[j];
#pragma unroll
    for (int a = 0; a < 5; ++a)
        if (A.z) A.z[pt * 5 + a] = z[a];
    if (!A.eq) return;  // moment vectors of the caller: no record
    const double st = sqrt(th);
    double *eq = A.eq + pt * kEqW;
    eq[EQ_C0] = log(rho) - 1.5 * log(th) + z[0] + 0.5 * z[4] * mAm;
#pragma unroll
    for (int d = 0; d < 3; ++d) eq[EQ_V + d] = U[d] + st * m[d];
    const double sc = z[4] / th;
    eq[EQ_B] = sc * Am[0][0]; eq[EQ_B + 1] = sc * Am[1][1]; eq[EQ_B + 2] = sc * Am[2][2];
    eq[EQ_B + 3] = sc * Am[0][1]; eq[EQ_B + 4] = sc * Am[0][2]; eq[EQ_B + 5] = sc * Am[1][2];
    eq[EQ_INVTAU] = inv_tau;
    eq[EQ_RES] = res;
    double *pp = A.prim + pt * 5;
    pp[0] = rho * exp(z[0] + 0.5 * z[4] * mAm) * pow(kTwoPi / z[4], 1.5) / sqrt(det3(Am));
#pragma unroll
    for (int d = 0; d < 3; ++d) pp[1 + d] = eq[EQ_V + d];
    pp[4] = th / z[4];
}

__device__ void write_nonreal(const NewtonArgs &A, int64_t pt) {
    for (int a = 0; a < 5; ++a)
        if (A.z) A.z[pt * 5 + a] = 0.0;
    if (!A.eq) return;
    double *eq = A.eq + pt * kEqW;
    eq[EQ_C0] = -INFINITY;
    for (int a = 1; a < kEqW; ++a) eq[a] = 0.0;
    for (int a = 0; a < 5; ++a) A.prim[pt * 5 + a] = 0.0;
}

// Moment a of point pt from its parts.
__device__ __forceinline__ double moment_part_sum(const NewtonArgs &A, int64_t pt, int a) {
    const double *q = A.Qpart + pt * A.nmom + a;
    const int64_t step = A.npts * A.nmom;
    double t = q[0];
#pragma unroll 4
    for (int s = 1; s < A.nparts; ++s) t += q[s * step];
    return t;
}

// Per-point outcome; the counters are aggregated afterwards by k_stats_reduce
// (per-point atomics on a handful of counters would serialise the kernel,
// also on small solves: 1620 points 31 -> 46 us for the 5 us of that launch).
__device__ void record_stats(const NewtonArgs &A, int64_t pt, int iters, int evals, int status, double res) {
    if (A.pt_iters) A.pt_iters[pt] = iters;
    if (A.pt_evals) A.pt_evals[pt] = evals;
    if (A.pt_status) A.pt_status[pt] = status;
    if (A.pt_resid) A.pt_resid[pt] = res;
}

// Histogram of iterations, fallback / ES-guard counts, total evaluations and
// the largest final residual, aggregated per workgroup in LDS and then added
// to the handle's counters with one atomic per non-empty bin.  Nearly every
// point takes the same number of iterations, so one LDS atomic per point
// would queue a whole wave on one bin (50 us for 262,144 points): each wave
// counts its points of one iteration number with a ballot and adds that
// once (7 us), four points per thread with their loads together.
constexpr int kStatPts = 4;
__global__ __launch_bounds__(256) void k_stats_reduce(int64_t npts, const int32_t *__restrict__ iters,
                                                      const int32_t *__restrict__ evals,
                                                      const int32_t *__restrict__ status,
                                                      const double *__restrict__ resid, unsigned long long *stats,
                                                      unsigned long long *maxres) {
    __shared__ unsigned int hist[kHist + 3];
    __shared__ double rmax[4];
    for (int i = threadIdx.x; i < kHist + 3; i += 256) hist[i] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t step = (int64_t)gridDim.x * 256;
    double m = 0.0;
    unsigned int ev = 0u;
    int64_t pt = (int64_t)blockIdx.x * 256 + threadIdx.x;
    for (int64_t base = 0; base < npts; base += kStatPts * step) {
        int it[kStatPts], st[kStatPts];
#pragma unroll
        for (int a = 0; a < kStatPts; ++a) {
            const int64_t q = pt + base + a * step;
            const bool in = q < npts;
            it[a] = in ? iters[q] : -1;
            st[a] = in ? status[q] : -1;
            ev += in ? (unsigned int)evals[q] : 0u;
            const double r = in ? resid[q] : 0.0;
            if (in) it[a] = it[a] < kHist ? (it[a] < 0 ? 0 : it[a]) : kHist - 1;
            if (r >= 0.0 && isfinite(r)) m = fmax(m, r);
        }
#pragma unroll
        for (int a = 0; a < kStatPts; ++a) {
            unsigned long long todo = __ballot(it[a] >= 0);
            while (todo) {
                const int v = __shfl(it[a], __ffsll(todo) - 1);
                const unsigned long long same = __ballot(it[a] == v);
                if (lane == 0) atomicAdd(&hist[v], (unsigned int)__popcll(same));
                todo &= ~same;
            }
            const unsigned long long fb = __ballot(st[a] == FR_DVM_NEWTON_FALLBACK);
            const unsigned long long eg = __ballot(st[a] == FR_DVM_NEWTON_ESGUARD);
            if (lane == 0 && fb) atomicAdd(&hist[kHist], (unsigned int)__popcll(fb));
            if (lane == 0 && eg) atomicAdd(&hist[kHist + 1], (unsigned int)__popcll(eg));
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        ev += __shfl_xor(ev, o);
        m = fmax(m, __shfl_xor(m, o));
    }
    if (lane == 0) {
        if (ev) atomicAdd(&hist[kHist + 2], ev);
        rmax[threadIdx.x >> 6] = m;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kHist + 3; i += 256)
        if (hist[i]) atomicAdd(&stats[i], (unsigned long long)hist[i]);
    if (threadIdx.x == 0) {
        m = fmax(fmax(rmax[0], rmax[1]), fmax(rmax[2], rmax[3]));
        if (m > 0.0) atomicMax(maxres, (unsigned long long)__double_as_longlong(m));
    }
}

// Second starting point besides the cold one (warm or learned), if any.
__device__ bool alt_start(const NewtonArgs &A, int64_t pt, const double zc[5], double z[5]) {
    bool ok = false;
    if (A.guess == FR_DVM_GUESS_WARM) {
        ok = true;
#pragma unroll
        for (int a = 0; a < 5; ++a) { z[a] = A.z[pt * 5 + a]; ok = ok && isfinite(z[a]); }
    } else if (A.guess == FR_DVM_GUESS_MLP && A.dz_guess) {
        ok = true;
#pragma unroll
        for (int a = 0; a < 5; ++a) { z[a] = zc[a] + (double)A.dz_guess[pt * 5 + a]; ok = ok && isfinite(z[a]); }
    }
    return ok && z[4] > 0.0;
}

// Residual rows psi = (1, c, |c|^2/2) against the targets (1, 0, 0, 0, 3/2).
__device__ __forceinline__ void residual(const Sums &s, double r[5]) {
    r[0] = s.S0 - 1.0;
    r[1] = s.Sc[0];
    r[2] = s.Sc[1];
    r[3] = s.Sc[2];
    r[4] = 0.5 * (s.Scc[0] + s.Scc[1] + s.Scc[2]) - 1.5;
}

// Below this residual norm the iteration keeps its Jacobian (chord steps)
// and evaluates only the residual sums; from a start this close the chord
// contraction factor is of the order of the distance to the root.
constexpr double kChord = 1e-5;

// Damped Newton from the better of the cold start and the alternative start.
// Returns 1 on convergence; z, res, iterations (linear solves) and evals
// (sum passes) are outputs.
template <typename SumsFn>
__device__ int newton_solve(const NewtonArgs &A, SumsFn sums, int64_t pt, const double zc[5], double z[5],
                            double &res, int &iters, int &evals) {
    // s: full sums at the point of the current Jacobian (assembled right
    // before each solve, to keep register pressure low); r: residual at z.
    double r[5], J[5][5];
    Sums s;
    // the alternative start is tried first; the cold start is evaluated too
    // only when the alternative is not already close (scaled residual > 1e-2)
    const bool have_alt = A.guess != FR_DVM_GUESS_COLD && alt_start(A, pt, zc, z);
    if (!have_alt) {
#pragma unroll
        for (int a = 0; a < 5; ++a) z[a] = zc[a];
    }
    sums(z, s, true);
    residual(s, r);
    evals = 1;
    if (have_alt && !(norm2_5(r) <= 1e-2)) {
        Sums sc;
        double rc[5];
        sums(zc, sc, true);
        residual(sc, rc);
        ++evals;
        if (!(norm2_5(r) <= norm2_5(rc))) {
            s = sc;
#pragma unroll
            for (int a = 0; a < 5; ++a) { z[a] = zc[a]; r[a] = rc[a]; }
        }
    }
    int conv = 0, it, rej = 0;  // rej: rejected line-search trials over the whole solve
    for (it = 0; it < A.max_iter; ++it) {
        const double rn = norm2_5(r), ri = normi_5(r);
        double rhs[5] = {-r[0], -r[1], -r[2], -r[3], -r[4]}, dz[5], rdum[5];
        assemble(s, rdum, J);
        const bool ok = solve5(J, rhs, dz);
        if (ok && ri <= A.tol) {
            // converged: one extra step makes the result path independent
#pragma unroll
            for (int a = 0; a < 5; ++a) z[a] += dz[a];
            res = ri;
            conv = 1;
            ++it;
            break;
        }
        if (!ok) break;
        const bool chord = rn <= kChord;
        double alpha = 1.0, zt[5], rt[5];
        Sums st;
        bool acc = false;
        while (rej < kRejectBudget) {
#pragma unroll
            for (int a = 0; a < 5; ++a) zt[a] = z[a] + alpha * dz[a];
            if (zt[4] > 0.0) {
                sums(zt, st, !chord);
                ++evals;
                residual(st, rt);
                if (norm2_5(rt) < (1.0 - 1e-4 * alpha) * rn) { acc = true; break; }
            }
            alpha *= 0.5;
            ++rej;
        }
        if (!acc) {
            // stagnation at the rounding floor of the FP64 sums
            if (ri <= 100.0 * A.tol) { res = ri; conv = 1; ++it; }
            break;
        }
#pragma unroll
        for (int a = 0; a < 5; ++a) { z[a] = zt[a]; r[a] = rt[a]; }
        if (!chord) {
            s = st;
        } else if (norm2_5(rt) > 1e-2 * rn) {
            // slow chord contraction: refresh the Jacobian at the new point
            sums(z, s, true);
            ++evals;
            residual(s, r);
        }
    }
    iters = it;
    if (!conv) {
        res = normi_5(r);
#pragma unroll
        for (int a = 0; a < 5; ++a) z[a] = zc[a];
    }
    return conv;
}

// The iteration of newton_solve for one point, written as a state machine
// that is advanced after every evaluation of the sums: advance() takes the
// sums the last request asked for and makes the next request, or ends.
// Every point's iteration is the same as newton_solve's.  It lives in LDS:
// the sums need the registers of every wave.
struct EsIter {
    enum Phase { kStart, kCold, kTrial, kRefresh };
    double z[5], r[5], dz[5], zc0;
    double alpha, rn, ri, res;
    double rho, th, inv_tau;  // of the point, for its record
    int phase, it, hh, conv, evals, cur;  // cur: the set of sums of the current Jacobian
    int status, chord, have_alt;

    __device__ __forceinline__ void request(const NewtonArgs &A, EsPoint &p, bool jac, int tgt) {
        p.tgt = tgt;
        p.req = kReqSums | (jac ? kReqJac : 0) | sums_form(A, p);
        ++evals;
    }
    __device__ __forceinline__ void point(EsPoint &p, double al) const {
#pragma unroll
        for (int a = 0; a < 5; ++a) p.z[a] = z[a] + al * dz[a];
    }
    __device__ void start(const NewtonArgs &A, int64_t pt, EsPoint &p, double zc0_) {
        zc0 = zc0_;
        const double zc[5] = {zc0, 0.0, 0.0, 0.0, 1.0};
        double za[5];
        have_alt = A.guess != FR_DVM_GUESS_COLD && alt_start(A, pt, zc, za);
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            z[a] = have_alt ? za[a] : zc[a];
            r[a] = dz[a] = 0.0;
        }
        alpha = 1.0;
        rn = ri = res = 0.0;
        phase = kStart;
        it = hh = conv = evals = cur = 0;
        chord = false;
        point(p, 0.0);
        request(A, p, true, 0);
    }
    // Returns false when the iteration has ended (p.req cleared).
    __device__ bool advance(const NewtonArgs &A, EsPoint &p) {
        p.req = 0;
        double re[5];
        residual(p.s[p.tgt], re);
        if (phase == kStart) {
#pragma unroll
            for (int a = 0; a < 5; ++a) r[a] = re[a];
            if (have_alt && !(norm2_5(r) <= 1e-2)) {
                // the alternative start is not already close: evaluate the
                // cold start too and keep the better one
                phase = kCold;
                p.z[0] = zc0;
                p.z[1] = p.z[2] = p.z[3] = 0.0;
                p.z[4] = 1.0;
                request(A, p, true, cur ^ 1);
                return true;
            }
        } else if (phase == kCold) {
            if (!(norm2_5(r) <= norm2_5(re))) {
                cur = p.tgt;
#pragma unroll
                for (int a = 0; a < 5; ++a) { z[a] = p.z[a]; r[a] = re[a]; }
            }
        } else if (phase == kTrial) {
            const double rt = norm2_5(re);
            if (rt < (1.0 - 1e-4 * alpha) * rn) {
#pragma unroll
                for (int a = 0; a < 5; ++a) { z[a] = p.z[a]; r[a] = re[a]; }
                if (!chord) {
                    cur = p.tgt;
                } else if (rt > 1e-2 * rn) {
                    // slow chord contraction: refresh the Jacobian at z
                    phase = kRefresh;
                    request(A, p, true, cur);
                    return true;
                }
                ++it;
            } else {
                // rejected: halve the step until the trial is admissible
                do {
                    alpha *= 0.5;
                    ++hh;
                    point(p, alpha);
                } while (hh < kRejectBudget && !(p.z[4] > 0.0));
                if (hh < kRejectBudget) {
                    request(A, p, !chord, cur ^ 1);
                    return true;
                }
                // stagnation at the rounding floor of the FP64 sums
                if (ri <= 100.0 * A.tol) { res = ri; conv = 1; ++it; }
                return false;
            }
        } else {  // kRefresh
#pragma unroll
            for (int a = 0; a < 5; ++a) r[a] = re[a];
            ++it;
        }
        // Newton step from z with the Jacobian of the current sums
        if (it >= A.max_iter) return false;
        rn = norm2_5(r);
        ri = normi_5(r);
        double J[5][5], rdum[5];
        const double rhs[5] = {-r[0], -r[1], -r[2], -r[3], -r[4]};
        assemble(p.s[cur], rdum, J);
        const bool ok = solve5(J, rhs, dz);
        if (ok && ri <= A.tol) {
            // converged: one extra step makes the result path independent
#pragma unroll
            for (int a = 0; a < 5; ++a) z[a] += dz[a];
            res = ri;
            conv = 1;
            ++it;
            return false;
        }
        if (!ok) return false;
        chord = rn <= kChord;
        alpha = 1.0;
        // hh counts the rejected trials of the whole solve (not reset here)
        point(p, alpha);
        while (hh < kRejectBudget && !(p.z[4] > 0.0)) {
            alpha *= 0.5;
            ++hh;
            point(p, alpha);
        }
        if (hh >= kRejectBudget) {
            if (ri <= 100.0 * A.tol) { res = ri; conv = 1; ++it; }
            return false;
        }
        phase = kTrial;
        request(A, p, !chord, cur ^ 1);
        return true;
    }
    __device__ __forceinline__ void finish() {
        if (conv) return;
        res = normi_5(r);
        z[0] = zc0;
        z[1] = z[2] = z[3] = 0.0;
        z[4] = 1.0;
    }
};

constexpr int kBgkBlock = 64;
// One solution point per LPP lanes; the iteration runs alike in all of them
// and the first writes the point (launch_bgk chooses LPP).
template <int LPP>
__global__ __launch_bounds__(kBgkBlock) void k_newton_bgk(const NewtonArgs A) {
    const int64_t pt = ((int64_t)blockIdx.x * kBgkBlock + threadIdx.x) / LPP;
    const int lane = threadIdx.x % LPP;
    if (pt >= A.npts) return;  // a point's lanes leave together
    const bool first = lane == 0;
    double Q[6];  // (records of 5 or 6 values)
    if (A.nparts > 1) {
        // lane a of the point adds the parts of moment a, a + LPP, ...
#pragma unroll
        for (int a0 = 0; a0 < 6; a0 += LPP) {
            const int a = a0 + lane;
            const double t = a < A.nmom ? moment_part_sum(A, pt, a) : 0.0;
#pragma unroll
            for (int b = 0; b < LPP && a0 + b < 6; ++b) Q[a0 + b] = __shfl(t, b, LPP);
        }
    } else {
#pragma unroll
        for (int a = 0; a < 6; ++a) Q[a] = a < A.nmom ? A.Q[pt * A.nmom + a] : 0.0;
    }
    const double rho = Q[0];
    const double irho = 1.0 / rho;
    double U[3] = {Q[1] * irho, Q[2] * irho, Q[3] * irho};
    // E - rho |U|^2 / 2 = (3 + delta)/2 rho theta
    const double E = record_energy(Q, A.nmom);
    const double th = (2.0 / (3.0 + A.delta)) * (E * irho - 0.5 * (U[0] * U[0] + U[1] * U[1] + U[2] * U[2]));
    if (!(rho > 0.0) || !(th > 0.0) || !isfinite(rho) || !isfinite(th)) {
        if (first) {
            write_nonreal(A, pt);
            if (A.gfp) A.gfp[pt] = 0.0;
            record_stats(A, pt, 0, 0, FR_DVM_NEWTON_NONREAL, -1.0);
        }
        return;
    }
    if (A.gfp && first) A.gfp[pt] = 0.5 * A.delta * th;
    const double inv_tau = rho * th / viscosity(A, th);
    const double ist = 1.0 / sqrt(th);
    const double zc[5] = {-1.5 * log(kTwoPi), 0.0, 0.0, 0.0, 1.0};
    double z[5];
    auto fn = [&](const double zz[5], Sums &s, bool) { sums_bgk<LPP>(A, lane, U, ist, zz, s); };
    double res;
    int iters, evals;
    const int conv = newton_solve(A, fn, pt, zc, z, res, iters, evals);
    if (!first) return;
    const double Am[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
    write_point(A, pt, rho, U, th, Am, z, inv_tau, res);
    record_stats(A, pt, iters, evals, conv ? FR_DVM_NEWTON_OK : FR_DVM_NEWTON_FALLBACK, res);
}

// ES Newton.  The sums over the velocity grid need a wave per point, the rest
// of the iteration (moments to frame, 5 x 5 solves, step control, equilibrium
// record) is scalar work per point that a wave would do 64 times over.  So a
// workgroup takes A.es_pts points: in each round its waves evaluate the sums
// that the points request, one point per wave after the other, and then one
// thread per point (the first es_pts threads) advances the point's iteration
// and makes its next request, until no point has one.  Every wave reaches
// every barrier, and a point makes at most 2 max_iter + kRejectBudget + 1
// requests after its first (an accepted trial and its refresh per iteration,
// the rejected trials, the cold start).
// Warm solves (two evaluations a point), 32 lanes per point running the whole
// iteration and two-axis tables -> this form: 262,144 points of a 20^3 grid
// 2.89 -> 1.73 ms, 62,208 of 24^3 1.19 -> 0.78, 51,200 of 24^3 0.97 -> 0.66;
// the multiply-adds of the sums alone are 0.5 ms of the first.  Register
// targets of 2 and 4 waves per SIMD: 1.97 and 1.71 ms.
#ifndef FRDVM_WAVES_ES
#define FRDVM_WAVES_ES 3
#endif
constexpr int kEsBlock = 256;
constexpr int kEsPointD = (int)((sizeof(EsPoint) + sizeof(EsIter)) / sizeof(double));
static_assert(sizeof(EsPoint) % 8 == 0 && sizeof(EsIter) % 8 == 0, "LDS records of whole doubles");
constexpr int kEsMaxPts = 64;  // points of a workgroup: at most one per lane of its first wave

__global__ __launch_bounds__(kEsBlock) __attribute__((amdgpu_waves_per_eu(FRDVM_WAVES_ES))) void k_newton_es(
    const NewtonArgs A) {
    extern __shared__ double es_lds[];
    const int npw = A.es_pts;  // <= kEsMaxPts
    EsPoint *const P = reinterpret_cast<EsPoint *>(es_lds);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double *const tb = es_lds + npw * kEsPointD + wave * es_table_doubles(A);
    const int64_t p0 = (int64_t)blockIdx.x * npw;
    const bool owner = (int)threadIdx.x < npw && p0 + threadIdx.x < A.npts;
    const int64_t pt = p0 + threadIdx.x;
    EsIter &I = reinterpret_cast<EsIter *>(P + npw)[threadIdx.x < npw ? threadIdx.x : 0];
    bool active = false;
    if ((int)threadIdx.x < npw) P[threadIdx.x].req = 0;
    if (A.nparts > 1) {
        // the points' moments from their parts, into the space of their sums
        for (int t = threadIdx.x; t < npw * A.nmom; t += kEsBlock) {
            const int q = t / A.nmom, a = t - q * A.nmom;
            if (p0 + q < A.npts) reinterpret_cast<double *>(&P[q].s[0])[a] = moment_part_sum(A, p0 + q, a);
        }
        __syncthreads();
    }
    if (owner) {
        EsPoint &p = P[threadIdx.x];
        const double *Q = A.nparts > 1 ? reinterpret_cast<const double *>(&p.s[0]) : A.Q + pt * A.nmom;
        const double rho = Q[0];
        const double irho = 1.0 / rho;
        const double U[3] = {Q[1] * irho, Q[2] * irho, Q[3] * irho};
        // raw second moments -> pressure tensor Pi = M2 - rho U U^T
        const double Pi[6] = {Q[4] - rho * U[0] * U[0], Q[5] - rho * U[1] * U[1], Q[6] - rho * U[2] * U[2],
                              Q[7] - rho * U[0] * U[1], Q[8] - rho * U[0] * U[2], Q[9] - rho * U[1] * U[2]};
        // (3 + delta) rho theta = tr Pi + 2 (integral of G)
        const double th = (Pi[0] + Pi[1] + Pi[2] + (A.nmom == 11 ? 2.0 * Q[10] : 0.0)) / ((3.0 + A.delta) * rho);
        if (!(rho > 0.0) || !(th > 0.0) || !isfinite(rho) || !isfinite(th)) {
            write_nonreal(A, pt);
            if (A.gfp) A.gfp[pt] = 0.0;
            record_stats(A, pt, 0, 0, FR_DVM_NEWTON_NONREAL, -1.0);
        } else {
            if (A.gfp) A.gfp[pt] = 0.5 * A.delta * th;
            const double Pr = A.Pr;
            I.rho = rho;
            I.th = th;
            I.inv_tau = Pr * rho * th / viscosity(A, th);
            I.status = FR_DVM_NEWTON_OK;
            double Am[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
            const double a1 = th / Pr, a2 = (1.0 - 1.0 / Pr) * irho;
            const double T[3][3] = {{a1 + a2 * Pi[0], a2 * Pi[3], a2 * Pi[4]},
                                    {a2 * Pi[3], a1 + a2 * Pi[1], a2 * Pi[5]},
                                    {a2 * Pi[4], a2 * Pi[5], a1 + a2 * Pi[2]}};
            if (sym3_min_eig(T) <= 1e-8 * th) {
                I.status = FR_DVM_NEWTON_ESGUARD;
            } else {
                double Ti[3][3];
                inv3(T, Ti);
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) Am[i][j] = th * Ti[i][j];
            }
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                p.U[d] = U[d];
                p.A[d] = Am[d][d];
            }
            p.A[3] = Am[0][1];
            p.A[4] = Am[0][2];
            p.A[5] = Am[1][2];
            p.ist = 1.0 / sqrt(th);
            I.start(A, pt, p, -1.5 * log(kTwoPi) + 0.5 * log(det3(Am)));
            active = true;
        }
    }
    while (__syncthreads_or(active)) {
        for (int s = wave; s < npw; s += kEsBlock / 64) {
            EsPoint &p = P[s];
            const int req = __builtin_amdgcn_readfirstlane(p.req);
            if (!req) continue;
            double *out = reinterpret_cast<double *>(&p.s[__builtin_amdgcn_readfirstlane(p.tgt)]);
            if (req & kReqJac) {
                if (req & kReqDirect) sums_es<true>(A, lane, p, out);
                else if (req & kReqWide) sums_es_fact<true, true>(A, lane, tb, p, out);
                else sums_es_fact<true, false>(A, lane, tb, p, out);
            } else {
                if (req & kReqDirect) sums_es<false>(A, lane, p, out);
                else if (req & kReqWide) sums_es_fact<false, true>(A, lane, tb, p, out);
                else sums_es_fact<false, false>(A, lane, tb, p, out);
            }
        }
        __syncthreads();
        if (active) {
            EsPoint &p = P[threadIdx.x];
            active = I.advance(A, p);
            if (!active) {
                I.finish();
                const double Am[3][3] = {{p.A[0], p.A[3], p.A[4]}, {p.A[3], p.A[1], p.A[5]}, {p.A[4], p.A[5], p.A[2]}};
                write_point(A, pt, I.rho, p.U, I.th, Am, I.z, I.inv_tau, I.res);
                record_stats(A, pt, I.it, I.evals, I.conv ? I.status : FR_DVM_NEWTON_FALLBACK, I.res);
            }
        }
    }
}

// Size of the discrete-velocity error of the continuous equilibrium, which
// scales the learned correction: trapezoid aliasing exp(-2 pi^2 theta/du^2)
// plus truncation by the velocity box exp(-(u_max - |U_d|)^2 / (2 theta)).
__device__ __forceinline__ double guess_envelope(const double U[3], double th, double umax, double du) {
    double tr = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double g = fmax(umax - fabs(U[d]), 0.0);
        tr = fmax(tr, exp(-g * g / (2.0 * th)));
    }
    const double s = exp(-0.5 * kTwoPi * kTwoPi * th / (du * du)) + tr;
    return fmin(fmax(s, 1e-10), 1.0);  // below 1e-10 the correction is Newton round-off
}

// Features of the learned guess from the moments: [ln rho, U/u_max, ln theta,
// u_max/10, n_v/32, sin and cos of the grid phase 2 pi (U - umin)/du] (FP32)
// and the correction envelope; non-realizable
// points get zeros (Newton marks them).
__global__ void k_mlp_features(int64_t npts, int nmom, const double *__restrict__ Q, const VGrid vg, double umax,
                               double du, float *__restrict__ X, float *__restrict__ env) {
    const int64_t pt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pt >= npts) return;
    const double *q = Q + pt * nmom;
    const double rho = q[0];
    const double U[3] = {q[1] / rho, q[2] / rho, q[3] / rho};
    const double E = nmom == 5 ? q[4] : 0.5 * (q[4] + q[5] + q[6]);
    const double th = (2.0 / 3.0) * (E / rho - 0.5 * (U[0] * U[0] + U[1] * U[1] + U[2] * U[2]));
    float *x = X + pt * FR_MLP_INPUTS;
    if (!(rho > 0.0) || !(th > 0.0)) {
        for (int a = 0; a < FR_MLP_INPUTS; ++a) x[a] = 0.f;
        env[pt] = 0.f;
        return;
    }
    env[pt] = (float)guess_envelope(U, th, umax, du);
    x[0] = (float)log(rho);
    x[1] = (float)(U[0] / umax);
    x[2] = (float)(U[1] / umax);
    x[3] = (float)(U[2] / umax);
    x[4] = (float)log(th);
    x[5] = (float)(umax / 10.0);
    x[6] = (float)(vg.nv[0] / 32.0);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double ph = vg.du[d] > 0.0 ? kTwoPi * (U[d] - vg.umin[d]) / vg.du[d] : 0.0;
        x[7 + d] = (float)sin(ph);
        x[10 + d] = (float)cos(ph);
    }
}

__global__ void k_collide(const VGrid vg, const double *__restrict__ eqs, const void *fv, void *Sv, int accumulate,
                          int fp64, int ncomp, const double *__restrict__ gfp) {
    const int64_t pt = blockIdx.x;
    const double *eqp = eqs + pt * kEqW;
    double eq[kEqW];
#pragma unroll
    for (int a = 0; a < kEqW; ++a) eq[a] = eqp[a];
    // the pair's G relaxes to delta theta / 2 times the equilibrium of F:
    // its exponent is shifted by the logarithm of that factor
    const double lg = ncomp == 2 ? (gfp[pt] > 0.0 ? log(gfp[pt]) : -1000.0) : 0.0;
    const int nut = vg.nu * ncomp;
    for (int kk = threadIdx.x; kk < nut; kk += blockDim.x) {
        const int comp = kk >= vg.nu, k = kk - comp * vg.nu;
        const int i = k % vg.nv[0], j = (k / vg.nv[0]) % vg.nv[1], l = k / (vg.nv[0] * vg.nv[1]);
        const double u[3] = {gridu(vg, 0, i), gridu(vg, 1, j), gridu(vg, 2, l)};
        const int64_t idx = pt * nut + kk;
        const double c0g = eq[EQ_C0] + (comp ? lg : 0.0);
        if (fp64) {
            const double c0 = u[0] - eq[EQ_V], c1 = u[1] - eq[EQ_V + 1], c2 = u[2] - eq[EQ_V + 2];
            const double q = eq[EQ_B] * c0 * c0 + eq[EQ_B + 1] * c1 * c1 + eq[EQ_B + 2] * c2 * c2 +
                             2.0 * (eq[EQ_B + 3] * c0 * c1 + eq[EQ_B + 4] * c0 * c2 + eq[EQ_B + 5] * c1 * c2);
            const double g = exp(c0g - 0.5 * q);
            const double f = ((const double *)fv)[idx];
            const double S = (g - f) * eq[EQ_INVTAU];
            double *So = (double *)Sv;
            So[idx] = accumulate ? So[idx] + S : S;
        } else {
            // the exponent in FP64 and the exponential rounded once to FP32,
            // as in the fused stage
            const double c0 = u[0] - eq[EQ_V], c1 = u[1] - eq[EQ_V + 1], c2 = u[2] - eq[EQ_V + 2];
            const double q = eq[EQ_B] * c0 * c0 + eq[EQ_B + 1] * c1 * c1 + eq[EQ_B + 2] * c2 * c2 +
                             2.0 * (eq[EQ_B + 3] * c0 * c1 + eq[EQ_B + 4] * c0 * c2 + eq[EQ_B + 5] * c1 * c2);
            const float g = exp_to_f32(c0g - 0.5 * q);
            const float f = ((const float *)fv)[idx];
            const float S = (g - f) * (float)eq[EQ_INVTAU];
            float *So = (float *)Sv;
            So[idx] = accumulate ? So[idx] + S : S;
        }
    }
}

__global__ void k_moments_out(int64_t npts, int nmom, const double *__restrict__ Q, double *__restrict__ out) {
    const int64_t pt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (pt >= npts) return;
    const double *q = Q + pt * nmom;
    double *o = out + pt * 5;
    o[0] = q[0]; o[1] = q[1]; o[2] = q[2]; o[3] = q[3];
    o[4] = record_energy(q, nmom);
}

// Gradient-length local Knudsen number (Section "Results"):
// Kn = lambda |grad rho| / rho with the hard-sphere-type mean free path
// lambda = mu(theta)/rho sqrt(pi/(2 theta)).  grad rho is the derivative of
// the element's solution polynomial of rho (the FR interpolant, no interface
// correction); on an axis-aligned box d/dx_d = (2/h_d) d/dxi_d, on a general
// element grad = (1/|J|) sum_d a^d d/dxi_d.  One wave per
// element (ns <= 64 points), the density of the element staged in LDS.
// Points with rho <= 0 or theta <= 0 get 0.
constexpr int kKnElems = 4;

__global__ __launch_bounds__(64 * kKnElems) void k_kn_gll(NewtonArgs A, Ops1D ops, int n, int64_t ne,
                                                          const double *__restrict__ gfac, const double *__restrict__ S,
                                                          const double *__restrict__ ijac, double *__restrict__ kn) {
    __shared__ double srho[kKnElems][64];
    const int w = threadIdx.x >> 6, s = threadIdx.x & 63;
    const int64_t e = (int64_t)blockIdx.x * kKnElems + w;
    const int ns = n * n * n;
    const bool live = e < ne && s < ns;
    const int64_t pt = e * ns + s;
    if (live) srho[w][s] = A.Q[pt * A.nmom];
    __syncthreads();
    if (!live) return;
    const int i = s % n, j = (s / n) % n, l = s / (n * n);
    double d0 = 0, d1 = 0, d2 = 0;
    for (int m = 0; m < n; ++m) {
        d0 += ops.D[i * n + m] * srho[w][m + n * (j + n * l)];
        d1 += ops.D[j * n + m] * srho[w][i + n * (m + n * l)];
        d2 += ops.D[l * n + m] * srho[w][i + n * (j + n * m)];
    }
    if (S) {  // general element: grad = (1/|J|) sum_d a^d d/dxi_d
        // (stored line by line of each direction)
        const double *a = S + (e * 3 * ns + (j + n * l) * n + i) * 3;
        const double *b = S + ((e * 3 + 1) * ns + (i + n * l) * n + j) * 3;
        const double *c = S + ((e * 3 + 2) * ns + (i + n * j) * n + l) * 3;
        const double g0 = ijac[pt] * (a[0] * d0 + b[0] * d1 + c[0] * d2);
        const double g1 = ijac[pt] * (a[1] * d0 + b[1] * d1 + c[1] * d2);
        const double g2 = ijac[pt] * (a[2] * d0 + b[2] * d1 + c[2] * d2);
        d0 = g0;
        d1 = g1;
        d2 = g2;
    } else {
        d0 *= gfac[e * 3 + 0];
        d1 *= gfac[e * 3 + 1];
        d2 *= gfac[e * 3 + 2];
    }
    const double *q = A.Q + pt * A.nmom;
    const double rho = q[0];
    const double ux = q[1] / rho, uy = q[2] / rho, uz = q[3] / rho;
    const double E = record_energy(q, A.nmom);
    const double th = (2.0 / (3.0 + A.delta)) * (E / rho - 0.5 * (ux * ux + uy * uy + uz * uz));
    double out = 0.0;
    if (rho > 0.0 && th > 0.0) {
        const double lam = viscosity(A, th) / rho * sqrt(kTwoPi / (4.0 * th));
        out = lam * sqrt(d0 * d0 + d1 * d1 + d2 * d2) / rho;
    }
    kn[pt] = out;
}

// Domain totals in two passes of fixed order: each workgroup sums a strided
// share of the points, the last pass adds the workgroups.  (One workgroup over
// all points waits on its own loads: 179 us at 262,144 points, now 11.)
__device__ __forceinline__ void block_totals(const double a[5], double *__restrict__ out) {
    __shared__ double red[5][256];
#pragma unroll
    for (int c = 0; c < 5; ++c) red[c][threadIdx.x] = a[c];
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o)
#pragma unroll
            for (int c = 0; c < 5; ++c) red[c][threadIdx.x] += red[c][threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x < 5) out[threadIdx.x] = red[threadIdx.x][0];
}
__global__ __launch_bounds__(256) void k_totals(int64_t npts, int nmom, const double *__restrict__ Q,
                                                const double *__restrict__ wJ, double *__restrict__ part) {
    double a[5] = {0, 0, 0, 0, 0};
#pragma unroll 4
    for (int64_t pt = (int64_t)blockIdx.x * 256 + threadIdx.x; pt < npts; pt += (int64_t)gridDim.x * 256) {
        const double *q = Q + pt * nmom;
        const double w = wJ[pt];
        a[0] += w * q[0]; a[1] += w * q[1]; a[2] += w * q[2]; a[3] += w * q[3];
        a[4] += w * record_energy(q, nmom);
    }
    block_totals(a, part + 5 * blockIdx.x);
}
__global__ __launch_bounds__(256) void k_totals_sum(int n, const double *__restrict__ part, double *__restrict__ out) {
    double a[5] = {0, 0, 0, 0, 0};
    if ((int)threadIdx.x < n)  // (n <= kTotBlocks = 256)
#pragma unroll
        for (int c = 0; c < 5; ++c) a[c] = part[5 * threadIdx.x + c];
    block_totals(a, out);
}

int check(fr_dvm *h, const char *what) {
    hipError_t st = hipGetLastError();
    if (st != hipSuccess) return h->fail(FR_DVM_EHIP, std::string(what) + ": " + hipGetErrorString(st));
    return FR_DVM_OK;
}

NewtonArgs newton_args(fr_dvm *h, int guess) {
    NewtonArgs A;
    std::memset(&A, 0, sizeof(A));
    A.vg = h->vg;
    A.npts = h->ne * h->ns;
    A.nmom = h->nmom;
    A.wax = h->d_wax;
    A.Q = h->d_Q;
    A.Qpart = h->d_Qpart;
    A.nparts = h->q_parts;
    A.eq = h->d_eq;
    A.z = h->d_z;
    A.prim = h->d_prim;
    A.stats = reinterpret_cast<unsigned long long *>(h->d_stats);
    A.maxres = reinterpret_cast<unsigned long long *>(h->d_maxres);
    A.Pr = h->prm.prandtl;
    A.mu_ref = h->prm.mu_ref;
    A.theta_ref = h->prm.theta_ref;
    A.omega = h->prm.omega;
    A.theta_s = h->prm.theta_s;
    A.visc_law = h->prm.visc_law;
    A.tol = h->prm.newton_tol;
    A.max_iter = h->prm.newton_max_iter;
    A.guess = (guess == FR_DVM_GUESS_WARM && !h->zvalid) ? FR_DVM_GUESS_COLD : guess;
    // the learned start is trained on monatomic states: cold start for the pair
    if (A.guess == FR_DVM_GUESS_MLP && (!h->d_mlp || h->ncomp == 2)) A.guess = FR_DVM_GUESS_COLD;
    A.delta = h->ncomp == 2 ? h->delta : 0.0;
    A.gfp = h->d_gfp;
    return A;
}

double grid_umax(const VGrid &vg) {
    double m = 0;
    for (int d = 0; d < 3; ++d)
        m = std::fmax(m, std::fmax(std::fabs(vg.umin[d]), std::fabs(vg.umin[d] + (vg.nv[d] - 1) * vg.du[d])));
    return m;
}

// Learned correction dz[n][5] (float) for moment vectors Q[n][nmom], batched
// through the MLP forward kernels.
int mlp_predict(fr_dvm *h, const double *Q, int64_t n, int nmom, float *dz) {
    const int64_t batch = 65536;
    const int64_t nb = n < batch ? n : batch;
    const size_t need_x = (size_t)nb * (FR_MLP_INPUTS + 1);
    if (h->mlp_x_n < need_x) {
        if (h->d_mlp_x) (void)hipFree(h->d_mlp_x);
        h->d_mlp_x = nullptr;
        h->mlp_x_n = 0;
        if (hipMalloc(&h->d_mlp_x, need_x * sizeof(float)) != hipSuccess) {
            h->d_mlp_x = nullptr;
            return h->fail(FR_DVM_ENOMEM, "MLP features");
        }
        h->mlp_x_n = need_x;
    }
    const double umax = grid_umax(h->vg);
    const double du = std::fmax(h->vg.du[0], std::fmax(h->vg.du[1], h->vg.du[2]));
    float *env = h->d_mlp_x + (size_t)nb * FR_MLP_INPUTS;
    for (int64_t b0 = 0; b0 < n; b0 += batch) {
        const int64_t m = (n - b0) < batch ? (n - b0) : batch;
        hipLaunchKernelGGL(k_mlp_features, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, h->stream, m, nmom,
                           Q + b0 * nmom, h->vg, umax, du, h->d_mlp_x, env);
        int rc = mlp_forward_scaled(h->mlp_hidden, h->d_mlp, h->d_mlp_x, m, env, dz + b0 * 5, h->stream);
        if (rc) return h->fail(rc, "MLP forward");
    }
    return check(h, "MLP features");
}

int ensure_dz(fr_dvm *h, int64_t n) {
    if (h->dz_n >= (size_t)n) return FR_DVM_OK;
    if (h->d_mlp_dz) (void)hipFree(h->d_mlp_dz);
    h->d_mlp_dz = nullptr;
    h->dz_n = 0;
    if (hipMalloc(&h->d_mlp_dz, sizeof(float) * 5 * n) != hipSuccess) {
        h->d_mlp_dz = nullptr;
        return h->fail(FR_DVM_ENOMEM, "MLP output");
    }
    h->dz_n = n;
    return FR_DVM_OK;
}

}  // namespace

namespace {

template <int LPP>
void launch_bgk_lanes(const NewtonArgs &A, hipStream_t s) {
    constexpr int per = kBgkBlock / LPP;
    hipLaunchKernelGGL(k_newton_bgk<LPP>, dim3((unsigned)((A.npts + per - 1) / per)), dim3(kBgkBlock), 0, s, A);
}
// Lanes per point: one where the points alone fill the chip (the sums are a
// part of the work, the 5 x 5 solves are repeated by every lane: at 262,144
// points of a 32^3 grid 1, 2, 4, 8 lanes take 269, 282, 369, 571 us), more
// on small batches, where one lane's chain over the nodes is the time (4096
// points: 90, 59, 47, 45 us; 512 points of an 8^3 grid 54, 45, 42, 41 us, of
// which 30 are the call).  The lines lie where the measured times cross:
// with the axis length, since the shared part grows with it.  A point's sums
// have one order for every number of lanes.
void launch_bgk(const NewtonArgs &A, hipStream_t s) {
    const int64_t nv = std::max(A.vg.nv[0], std::max(A.vg.nv[1], A.vg.nv[2]));
    if (A.npts <= 128 * nv) launch_bgk_lanes<8>(A, s);
    else if (A.npts <= 512 * nv) launch_bgk_lanes<4>(A, s);
    else if (A.npts <= 2048 * nv) launch_bgk_lanes<2>(A, s);
    else launch_bgk_lanes<1>(A, s);
}

// Points per workgroup: 64 on large solves (a full wave of owner threads),
// fewer where that would leave fewer than four workgroups per CU.
void launch_es(const fr_dvm *h, NewtonArgs &A, hipStream_t s) {
    A.use_fact = !h->es_direct;
    A.nph = std::max(1, std::min(64 / A.vg.nv[0], A.vg.nv[1]));
    A.nrow = (A.vg.nv[1] + A.nph - 1) / A.nph * A.nph;
    int pts = kEsMaxPts;
    while (pts > 4 && A.npts < (int64_t)pts * 1024) pts /= 2;
    A.es_pts = pts;
    const size_t shm = sizeof(double) * (size_t)(pts * kEsPointD + (kEsBlock / 64) * es_table_doubles(A));
    hipLaunchKernelGGL(k_newton_es, dim3((unsigned)((A.npts + pts - 1) / pts)), dim3(kEsBlock), shm, s, A);
}

// The Newton kernel and its statistics over the points [p0, p0 + np) on
// stream s: every per-point array of A is offset to p0, so the kernels see a
// contiguous range starting at their point 0.
int newton_run(fr_dvm *h, NewtonArgs A, int64_t p0, int64_t np, hipStream_t s) {
    A.npts = np;
    A.Q += p0 * A.nmom;
    A.eq += p0 * kEqW;
    A.z += p0 * 5;
    A.prim += p0 * 5;
    if (A.dz_guess) A.dz_guess += p0 * 5;
    if (A.gfp) A.gfp += p0;
    A.pt_iters = h->d_pt_iters + p0;
    A.pt_evals = h->d_pt_evals + p0;
    A.pt_status = h->d_pt_status + p0;
    A.pt_resid = h->d_pt_resid + p0;
    ProfScope ps(h, 1, s);
    if (h->prm.model == FR_DVM_ESBGK) {
        launch_es(h, A, s);
    } else {
        launch_bgk(A, s);
    }
    int64_t nb = (A.npts + 256 * kStatPts - 1) / (256 * kStatPts);
    if (nb > 1024) nb = 1024;
    hipLaunchKernelGGL(k_stats_reduce, dim3((unsigned)nb), dim3(256), 0, s, A.npts, A.pt_iters, A.pt_evals,
                       A.pt_status, A.pt_resid, A.stats, A.maxres);
    const int rc = check(h, "newton kernel");
    if (!rc) h->newton_done = true;
    return rc;
}

}  // namespace

int launch_newton(fr_dvm *h, int guess) {
    // learned start where no previous solution exists, warm start afterwards
    if (guess == FR_DVM_GUESS_MLP_WARM) guess = h->zvalid ? FR_DVM_GUESS_WARM : FR_DVM_GUESS_MLP;
    NewtonArgs A = newton_args(h, guess);
    if (A.guess == FR_DVM_GUESS_MLP) {
        ProfScope ps(h, 3);
        int rc = ensure_dz(h, A.npts);
        if (!rc) rc = mlp_predict(h, h->d_Q, A.npts, h->nmom, h->d_mlp_dz);
        if (rc) return rc;
        A.dz_guess = h->d_mlp_dz;
    }
    const int rc = newton_run(h, A, 0, A.npts, h->stream);
    if (!rc) h->zvalid = 1;
    return rc;
}

int newton_part_ok(fr_dvm *h, int guess) {
    if (guess == FR_DVM_GUESS_MLP_WARM) guess = h->zvalid ? FR_DVM_GUESS_WARM : FR_DVM_GUESS_MLP;
    return newton_args(h, guess).guess != FR_DVM_GUESS_MLP;
}

int launch_newton_part(fr_dvm *h, int guess, int64_t p0, int64_t np, hipStream_t s) {
    if (guess == FR_DVM_GUESS_MLP_WARM) guess = h->zvalid ? FR_DVM_GUESS_WARM : FR_DVM_GUESS_MLP;
    NewtonArgs A = newton_args(h, guess);
    if (A.guess == FR_DVM_GUESS_MLP) return h->fail(FR_DVM_EINVAL, "learned start needs all points");
    if (p0 < 0 || np < 0 || p0 + np > A.npts) return h->fail(FR_DVM_EINVAL, "point range");
    return newton_run(h, A, p0, np, s);
}

// Newton on caller-supplied moment vectors (BGK form), for training targets
// and guess evaluation: the per-point outputs only, no equilibrium records.
int launch_newton_points(fr_dvm *h, const double *Q, int64_t n, int guess, double *z, int32_t *iters,
                         int32_t *evals, int32_t *status, double *resid) {
    if (n <= 0) return FR_DVM_OK;
    if (guess == FR_DVM_GUESS_MLP && !h->d_mlp) return h->fail(FR_DVM_EINVAL, "no MLP weights set");
    NewtonArgs A = newton_args(h, guess == FR_DVM_GUESS_MLP ? FR_DVM_GUESS_MLP : FR_DVM_GUESS_COLD);
    int rc = FR_DVM_OK;
    if (A.guess == FR_DVM_GUESS_MLP) {
        rc = ensure_dz(h, n);
        if (!rc) rc = mlp_predict(h, Q, n, 5, h->d_mlp_dz);
        A.dz_guess = h->d_mlp_dz;
    }
    if (!rc) {
        A.npts = n;
        A.nmom = 5;
        A.Q = Q;
        A.nparts = 0;
        A.eq = nullptr;
        A.prim = nullptr;
        A.z = z;
        A.pt_iters = iters;
        A.pt_evals = evals;
        A.pt_status = status;
        A.pt_resid = resid;
        A.delta = 0.0;  // monatomic moment vectors
        A.gfp = nullptr;
        if (!(A.mu_ref > 0)) A.mu_ref = 1.0;  // tau is not an output here
        launch_bgk(A, h->stream);
        rc = check(h, "newton kernel");
    }
    (void)hipStreamSynchronize(h->stream);
    return rc;
}

int launch_collide(fr_dvm *h, const void *f, void *S, int accumulate) {
    hipLaunchKernelGGL(k_collide, dim3((unsigned)(h->ne * h->ns)), dim3(256), 0, h->stream, h->vg, h->d_eq, f, S,
                       accumulate, h->prm.precision == FR_DVM_FP64 ? 1 : 0, h->ncomp, h->d_gfp);
    return check(h, "collide kernel");
}

int launch_prim_out(fr_dvm *h, double *Qp) {
    if (hipMemcpyAsync(Qp, h->d_prim, sizeof(double) * 5 * h->ne * h->ns, hipMemcpyDeviceToDevice, h->stream) !=
        hipSuccess)
        return h->fail(FR_DVM_EHIP, "copy of Q'");
    return FR_DVM_OK;
}

int launch_moments_out(fr_dvm *h, double *Q) {
    const int64_t npts = h->ne * h->ns;
    hipLaunchKernelGGL(k_moments_out, dim3((unsigned)((npts + 255) / 256)), dim3(256), 0, h->stream, npts, h->nmom,
                       h->d_Q, Q);
    return check(h, "moments output kernel");
}

int launch_kn_gll(fr_dvm *h, double *kn) {
    NewtonArgs A = newton_args(h, FR_DVM_GUESS_COLD);
    hipLaunchKernelGGL(k_kn_gll, dim3((unsigned)((h->ne + kKnElems - 1) / kKnElems)), dim3(64 * kKnElems), 0,
                       h->stream, A, h->ops, h->n, h->ne, h->axis_mode ? h->d_gfac : nullptr,
                       h->axis_mode ? nullptr : h->d_S, h->d_ijac, kn);
    return check(h, "Knudsen number kernel");
}

int launch_totals(fr_dvm *h, double *host_tot) {
    const int64_t npts = h->ne * h->ns;
    const int64_t nb = (npts + 255) / 256;
    const int n = (int)(nb < kTotBlocks ? nb : kTotBlocks);
    hipLaunchKernelGGL(k_totals, dim3(n), dim3(256), 0, h->stream, npts, h->nmom, h->d_Q, h->d_wq3J, h->d_tot + 5);
    hipLaunchKernelGGL(k_totals_sum, dim3(1), dim3(256), 0, h->stream, n, h->d_tot + 5, h->d_tot);
    int rc = check(h, "totals kernel");
    if (rc) return rc;
    if (hipMemcpyAsync(host_tot, h->d_tot, 5 * sizeof(double), hipMemcpyDeviceToHost, h->stream) != hipSuccess)
        return h->fail(FR_DVM_EHIP, "totals copy");
    if (hipStreamSynchronize(h->stream) != hipSuccess) return h->fail(FR_DVM_EHIP, "stream synchronise");
    return FR_DVM_OK;
}

}  // namespace frdvm
