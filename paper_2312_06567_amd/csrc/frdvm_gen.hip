// FR residual + collision + Runge-Kutta stage on general hexahedral meshes
// (gfx950): curved 27-node elements, faces met under any orientation,
// farfield and diffuse isothermal wall boundaries.
//
// Paper, Section "Numerical method": per velocity node the transformed flux
// F~_d = (a^d . u) f with the area-scaled contravariant vectors
// a^d = |J| grad xi_d, its divergence along the element's tensor lines, and
// at every flux point the upwind common flux F^I = u_n f- (u_n > 0) or
// u_n f+ (otherwise), u_n = u . n with the area-scaled outward normal; the
// jump F^I - u_n f- enters through the DG-recovering correction.  Exterior
// states (Section "Implementation & problem setup"): the neighbour's trace, the freestream Maxwellian (farfield),
// rho_w M(0, theta_w) (diffuse wall at rest) with rho_w chosen so that no
// mass crosses the wall, or the element's own trace at the mirrored velocity
// (specular symmetry wall).  The collision source (g(Q') - f)/tau and the RK
// combination are those of the box kernel.
//
// Work decomposition: one wave per (element, 64 velocities), one lane per
// velocity; the element's metrics and normals are read through the scalar
// cache, its equilibrium records staged in LDS.  A lane keeps its velocity's
// N^3 values in registers and their residual in a private LDS column; the derivative and
// the face terms are formed line by line, direction by direction.  Every access to f, the
// RK registers and the traces is a run of consecutive velocities.  Traces
// have a place for every velocity at every flux point, [e][face][point][k]; a
// wave stores its row of a point where one of its velocities leaves the element
// there (within a margin for rounding, on specular faces for the mirror image
// too), which is where the neighbour, the wall and the mirror image read it;
// the first pass over a small state stores every row (kGenAllBytes).
// The per-point moments are a separate reduction over the velocity axis.
#include <hip/hip_runtime.h>

#include <cstring>

#include "frdvm_common.h"
#include "frdvm_dev.h"
#include "frdvm_simplex.h"

namespace frdvm {

namespace {

constexpr int GMODE_STAGE = 1, GMODE_RESID = 2;
constexpr int kGBlock = 256;  // velocities per workgroup (traces, moments, wall sums)
constexpr int kGWave = 64;    // velocities per workgroup of the stage kernel

template <typename Real>
struct GOps {
    Real D[kMaxN * kMaxN];
    Real lam[2][kMaxN];
    Real corr[2][kMaxN];
};

struct GenArgs {
    GOps<float> of;
    GOps<double> od;
    VGrid vg;
    int nu, nut, ncomp;  // velocities; state values per point (ncomp components of nu)
    int nvb, nvw;        // blocks of 256 and of 64 state values per element
    double gwall;        // the pair's G wall factor delta theta_w / 2
    const double *gfp;   // [npts] the pair's G equilibrium factor delta theta / 2
    const double *wax;   // [3][64] 1-D trapezoid weights
    const double *wJ;    // [ne][ns] Gauss weight x |J| (positivity limiter)
    const double *S;     // [ne][3][nfp][n][3] a^d at the points of each line of direction d
    const double *ijac;  // [ne][ns]
    const double *nf;    // [ne][6]: normals [nfp][3], margins of u.n [nfp]
    const double *nm;    // [ne][6][nfp][4]: each normal with its margin
    const float *Sf, *ijacf, *nff, *nmf;  // the same in FP32
    const int32_t *conn; // [ne][6][4]
    const int32_t *wall; // [nwall]
    double *rw;          // [ne*6][nfp]
    const double *mw;    // [nu]
    const double *finf;  // [nu]
    StageArgs sa;
    int do_traces;
};

template <typename Real>
__device__ __forceinline__ const GOps<Real> &gops(const GenArgs &A);
template <>
__device__ __forceinline__ const GOps<float> &gops<float>(const GenArgs &A) { return A.of; }
template <>
__device__ __forceinline__ const GOps<double> &gops<double>(const GenArgs &A) { return A.od; }

// Metric tables in the working precision, read through the scalar cache
// (the indices are uniform over the workgroup).
template <typename Real>
using cptr = const __attribute__((address_space(4))) Real *;
template <typename Real>
struct Metrics {
    cptr<Real> S, ijac, nf, nm;
};
__device__ __forceinline__ Metrics<float> metrics(const GenArgs &A, float) {
    return {(cptr<float>)A.Sf, (cptr<float>)A.ijacf, (cptr<float>)A.nff, (cptr<float>)A.nmf};
}
__device__ __forceinline__ Metrics<double> metrics(const GenArgs &A, double) {
    return {(cptr<double>)A.S, (cptr<double>)A.ijac, (cptr<double>)A.nf, (cptr<double>)A.nm};
}

// exp of W exponents, side by side
template <int W>
__device__ __forceinline__ void gexp(const double (&E)[W], float (&g)[W]) { exp_to_f32<W>(E, g); }
template <int W>
__device__ __forceinline__ void gexp(const double (&E)[W], double (&g)[W]) {
#pragma unroll
    for (int w = 0; w < W; ++w) g[w] = exp(E[w]);
}

// Uniform base + the lane's byte offset (a run of consecutive velocities).
template <typename T>
__device__ __forceinline__ T ldo(const T *base, uint32_t boff) {
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + boff);
}
template <typename T>
__device__ __forceinline__ void sto(T *base, uint32_t boff, T v) {
    *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + boff) = v;
}

// Velocity node umin + i du (two roundings, as on the host).
__device__ __forceinline__ double node_u(const VGrid &vg, int d, int i) {
    return __dadd_rn(vg.umin[d], __dmul_rn((double)i, vg.du[d]));
}

// Velocity node k = i + n0 (j + n1 l) -> (i, j, l).  The quotients are taken
// in FP32 from (k + 1/2) times the reciprocal, exact for k < 2^22 (a grid
// has at most 64^3 nodes), instead of integer divisions.
__device__ __forceinline__ void split_k(const VGrid &vg, int k, int iv[3]) {
    const int n0 = vg.nv[0], n01 = vg.nv[0] * vg.nv[1];
    const int q2 = (int)(((float)k + 0.5f) * (1.0f / (float)n01));
    const int r = k - q2 * n01;
    const int q1 = (int)(((float)r + 0.5f) * (1.0f / (float)n0));
    iv[0] = r - q1 * n0;
    iv[1] = q1;
    iv[2] = q2;
}

template <int N>
__device__ __forceinline__ constexpr int spt(int i, int j, int l) { return i + N * (j + N * l); }

// m-th point of the line along axis d through face point (a, b); (a, b) run
// along the two other axes in increasing order.
template <int N>
__device__ __forceinline__ constexpr int line_pt(int d, int a, int b, int m) {
    return d == 0 ? spt<N>(m, a, b) : (d == 1 ? spt<N>(a, m, b) : spt<N>(a, b, m));
}

// Own face point (a, b) -> neighbour face point under orientation code o.
template <int N>
__device__ __forceinline__ int nbr_point(int o, int a, int b) {
    int x = (o & 1) ? b : a, y = (o & 1) ? a : b;
    if (o & 2) x = N - 1 - x;
    if (o & 4) y = N - 1 - y;
    return x + N * y;
}

// Value at a line's end from its N points.  The order of the operations is
// spelled out: the trace a neighbour stored and the own one it is compared with
// come from different kernels, and a compiler free to contract either product
// of a sum rounds them differently, which turns a continuous field's jump into
// noise (p = 1, FP32: 6 % on the residual's error).
template <typename Real, int N>
__device__ __forceinline__ Real face_value(const Real *lam, const Real (&line)[N]) {
    Real t = lam[0] * line[0];
#pragma unroll
    for (int m = 1; m < N; ++m) t = fma(lam[m], line[m], t);
    return t;
}

// Traces of f, stored at the flux points where one of the wave's velocities
// leaves the element (u.n above minus the margin).  The decision is the
// wave's, since a row stored in part costs more than a whole one: with every
// value stored the prime pass of the Mach-8 O-grid (p = 2, FP32) takes 1.82
// ms, with each lane storing for itself 2.66, so 1.57.
// ALL: every row, for states of up to kGenAllBytes, where the decisions' loads
// and ballots take longer than the rows: residual in FP64, decided / all, of 216
// elements p = 2, 120 velocities (6 MB) 32.3 / 28.8 us, 24 elements p = 3, 12^3
// (21 MB) 68.7 / 60.9, 216 elements p = 1, 12^3 (24 MB) 37.0 / 39.1, p = 2 (81 MB)
// 112 / 128.
constexpr int64_t kGenAllBytes = 22 << 20;
template <typename Real, int P, bool ALL>
__global__ __launch_bounds__(kGBlock) void k_gen_traces(const GenArgs A, const Real *__restrict__ f,
                                                         Real *__restrict__ tr) {
    constexpr int N = P + 1, NS = N * N * N, NFP = N * N;
    const int64_t e = blockIdx.x / A.nvb;
    const int k = (int)(blockIdx.x % A.nvb) * kGBlock + threadIdx.x;
    if (k >= A.nut) return;
    const int64_t nu = A.nut;  // stride of a solution point
    const GOps<Real> &op = gops<Real>(A);
    const uint32_t ko = (uint32_t)k * (uint32_t)sizeof(Real);
    const Real *fe = f + e * NS * nu;
    Real v[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) v[s] = ldo(fe + s * nu, ko);
    int iv[3];
    split_k(A.vg, k >= A.nu ? k - A.nu : k, iv);
    const Real u0 = (Real)node_u(A.vg, 0, iv[0]), u1 = (Real)node_u(A.vg, 1, iv[1]), u2 = (Real)node_u(A.vg, 2, iv[2]);
    const Real ul1 = (u0 < 0 ? -u0 : u0) + (u1 < 0 ? -u1 : u1) + (u2 < 0 ? -u2 : u2);
    const cptr<Real> gN = metrics(A, Real(0)).nf + e * 6 * NFP * 4;
    Real *te = tr + e * 6 * NFP * nu;
#pragma unroll
    for (int face = 0; face < 6; ++face) {
        const int d = face / 2, side = face & 1;
        // (the decisions of a face first: a branch around each value would
        // wait for its own scalar loads)
        uint32_t kept = 0;
        Real t[NFP];
#pragma unroll
        for (int q = 0; q < NFP; ++q) {
            const cptr<Real> nf = gN + 4 * face * NFP, n = nf + 3 * q;
            if constexpr (ALL) kept |= 1u << q;
            else kept |= __ballot(n[0] * u0 + n[1] * u1 + n[2] * u2 + nf[3 * NFP + q] * ul1 > Real(0)) ? 1u << q : 0u;
            Real line[N];
#pragma unroll
            for (int m = 0; m < N; ++m) line[m] = v[line_pt<N>(d, q % N, q / N, m)];
            t[q] = face_value<Real, N>(op.lam[side], line);
        }
#pragma unroll
        for (int q = 0; q < NFP; ++q)
            if ((kept >> q) & 1) sto(te + (face * NFP + q) * nu, ko, t[q]);
    }
}

// Moments of one solution point over the velocity grid (FP64, fixed order),
// one wave per point and kMomPts points per workgroup.  Lane t of the wave
// takes the (x, y) nodes t, t + 64, ... and walks each one's z column: the
// nodes of a z step are consecutive over the lanes (coalesced), and along
// the column only the z weight and u_z vary, so the column is summed as
// (sum w_z f, sum w_z u_z f, sum w_z u_z^2 f): three multiply-adds per value
// with wave-uniform coefficients; the (x, y) weight and velocity close the
// column into the moments, and a wave butterfly sums the lanes.  (A
// workgroup per point, its threads over the columns, spent most of its time
// starting workgroups and reducing across waves.)  BGK: rho, rho U, E; ES:
// rho, rho U and the raw second moments xx yy zz xy xz yz; the pair's G adds
// its integral (last slot).
constexpr int kMomMaxZ = 64;
constexpr int kMomPts = 4;  // points (waves) per workgroup
template <typename Real, int NMOM>
__global__ __launch_bounds__(64 * kMomPts) void k_gen_moments(const GenArgs A, const Real *__restrict__ f,
                                                              double *__restrict__ Q, int64_t npts) {
    constexpr bool PAIR = NMOM == 6 || NMOM == 11;
    __shared__ double tz[kMomMaxZ][3];  // w_z, w_z u_z, w_z u_z^2
    const int nx = A.vg.nv[0], ny = A.vg.nv[1], nz = A.vg.nv[2], nxy = nx * ny;
    for (int iz = threadIdx.x; iz < nz; iz += blockDim.x) {
        const double w = A.wax[128 + iz], u = node_u(A.vg, 2, iz);
        tz[iz][0] = w;
        tz[iz][1] = w * u;
        tz[iz][2] = (w * u) * u;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int64_t pt = (int64_t)blockIdx.x * kMomPts + (threadIdx.x >> 6);
    if (pt >= npts) return;  // (no barrier follows)
    const Real *fp = f + pt * A.nut;
    double M[NMOM];
#pragma unroll
    for (int a = 0; a < NMOM; ++a) M[a] = 0.0;
    for (int t = lane; t < nxy; t += 64) {
        const int iy = t / nx, ix = t - iy * nx;
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, g0 = 0.0;
#pragma unroll 4
        for (int iz = 0; iz < nz; ++iz) {
            const double x = (double)fp[t + iz * nxy];
            s0 = fma(tz[iz][0], x, s0);
            s1 = fma(tz[iz][1], x, s1);
            s2 = fma(tz[iz][2], x, s2);
            if constexpr (PAIR) g0 = fma(tz[iz][0], (double)fp[A.nu + t + iz * nxy], g0);
        }
        const double W = A.wax[ix] * A.wax[64 + iy];
        const double ux = node_u(A.vg, 0, ix), uy = node_u(A.vg, 1, iy);
        const double a0 = W * s0, a1 = W * s1, a2 = W * s2;
        M[0] += a0;
        M[1] = fma(ux, a0, M[1]);
        M[2] = fma(uy, a0, M[2]);
        M[3] += a1;
        if constexpr (NMOM == 5 || NMOM == 6) {
            M[4] = fma(0.5, fma(ux * ux + uy * uy, a0, a2), M[4]);
        } else {
            M[4] = fma(ux * ux, a0, M[4]);
            M[5] = fma(uy * uy, a0, M[5]);
            M[6] += a2;
            M[7] = fma(ux * uy, a0, M[7]);
            M[8] = fma(ux, a1, M[8]);
            M[9] = fma(uy, a1, M[9]);
        }
        if constexpr (PAIR) M[NMOM - 1] = fma(W, g0, M[NMOM - 1]);
    }
#pragma unroll
    for (int a = 0; a < NMOM; ++a) {
        double v = M[a];
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
        if (lane == a) Q[pt * NMOM + a] = v;
    }
}
inline unsigned gen_moment_grid(int64_t npts) { return (unsigned)((npts + kMomPts - 1) / kMomPts); }

// Wall density at each flux point of the diffuse-wall faces: the outflow
// mass flux of the interior trace over the inflow flux of the unit wall
// Maxwellian, rho_w = sum_{u_n>0} w u_n f- / sum_{u_n<0} w |u_n| M_w.
template <typename Real, int P>
__global__ __launch_bounds__(kGBlock) void k_gen_wall(const GenArgs A, const Real *__restrict__ tr) {
    constexpr int N = P + 1, NFP = N * N;
    __shared__ double red[kGBlock / 64][2];
    const int64_t fid = A.wall[blockIdx.x / NFP];
    const int fp = blockIdx.x % NFP;
    const double *nv = A.nf + fid * NFP * 4 + fp * 3;
    const double n0 = nv[0], n1 = nv[1], n2 = nv[2];
    const Real *t = tr + (fid * NFP + fp) * (int64_t)A.nut;  // F part of the trace
    double out = 0.0, in = 0.0;
    for (int k = threadIdx.x; k < A.nu; k += kGBlock) {
        int iv[3];
        split_k(A.vg, k, iv);
        const double w = A.wax[iv[0]] * A.wax[64 + iv[1]] * A.wax[128 + iv[2]];
        const double un = node_u(A.vg, 0, iv[0]) * n0 + node_u(A.vg, 1, iv[1]) * n1 + node_u(A.vg, 2, iv[2]) * n2;
        if (un > 0.0)
            out += w * un * (double)t[k];
        else
            in -= w * un * A.mw[k];
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        out += __shfl_xor(out, o);
        in += __shfl_xor(in, o);
    }
    if (lane == 0) {
        red[wv][0] = out;
        red[wv][1] = in;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double so = red[0][0], si = red[0][1];
#pragma unroll
        for (int q = 1; q < kGBlock / 64; ++q) {
            so += red[q][0];
            si += red[q][1];
        }
        A.rw[fid * NFP + fp] = si > 0.0 ? so / si : 0.0;
    }
}

// What a lane needs to find its exterior values (load_ext).
template <typename Real>
struct ExtArgs {
    cptr<int32_t> conn;   // the element's [6][4]
    int32_t cn[24];       // the same, read
    cptr<double> rwall;   // wall densities of its faces [6][nfp]
    cptr<Real> gN;        // its normals
    const double *finf, *mwall;
    const Real *tin;
    double gw;            // wall factor of the lane's component
    int64_t e, nu;
    uint32_t ko, k8, kv8;
    Real u0, u1, u2, ul1;
};

// u.n and the exterior values of both faces of axis d, requested together
// (the connectivity through the scalar cache: a vector load of it would put
// its latency before every direction's requests).  km0..2: the node mirrored
// in each axis (passed by value: a choice between members of X would keep X in
// scratch memory).  KEEP: kept gets the (wave-uniform) bits of the flux points
// whose traces the wave has to store.
template <typename Real, int N, bool KEEP, bool CONN, bool PAIRS>
__device__ __forceinline__ void load_ext(const ExtArgs<Real> &X, int d, int km0, int km1, int km2,
                                         Real (&un)[2][N * N], Real (&ext)[2][N * N], uint64_t (&kept)[2]) {
    constexpr int NFP = N * N, NW = PAIRS ? 4 : 3;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int face = 2 * d + side;
        int32_t c[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) c[i] = CONN ? X.cn[4 * face + i] : X.conn[4 * face + i];
        const int32_t nb = c[0], nface = c[1], orient = c[2], bc = c[3];
        const cptr<Real> nv = X.gN + face * NFP * 4;
#pragma unroll
        for (int q = 0; q < NFP; ++q)
            un[side][q] = nv[NW * q] * X.u0 + nv[NW * q + 1] * X.u1 + nv[NW * q + 2] * X.u2;
        if constexpr (KEEP) {
#pragma unroll
            for (int q = 0; q < NFP; ++q) {
                const int b = face * NFP + q;
                const uint64_t bit = __ballot(un[side][q] + nv[PAIRS ? 4 * q + 3 : 3 * NFP + q] * X.ul1 > Real(0)) ? 1ull << (b & 63) : 0ull;
                if (b < 64) kept[0] |= bit;
                else kept[1] |= bit;
            }
        }
        if (nb >= 0) {
            const Real *tn = X.tin + ((int64_t)nb * 6 + nface) * NFP * X.nu;
#pragma unroll
            for (int q = 0; q < NFP; ++q)
                ext[side][q] =
                    un[side][q] < Real(0) ? ldo(tn + nbr_point<N>(orient, q % N, q / N) * X.nu, X.ko) : Real(0);
        } else if (bc == 1) {
            const Real fi = (Real)ldo(X.finf, X.k8);
#pragma unroll
            for (int q = 0; q < NFP; ++q) ext[side][q] = fi;
        } else if (bc == 3) {
            // specular: the own trace at the velocity mirrored in the face's
            // axis (orient holds the axis), same component
            const uint32_t kmo = (uint32_t)(orient == 0 ? km0 : (orient == 1 ? km1 : km2)) * (uint32_t)sizeof(Real);
            const Real *to = X.tin + (X.e * 6 + face) * NFP * X.nu;
#pragma unroll
            for (int q = 0; q < NFP; ++q) ext[side][q] = un[side][q] < Real(0) ? ldo(to + q * X.nu, kmo) : Real(0);
        } else {
            const double mw = ldo(X.mwall, X.kv8) * X.gw;
            const cptr<double> rw = X.rwall + face * NFP;
#pragma unroll
            for (int q = 0; q < NFP; ++q) ext[side][q] = (Real)(rw[q] * mw);
        }
    }
}

// One wave per (element, 64 velocities).  Each lane keeps its velocity's N^3
// stage values in registers (all loops over directions, lines and flux points
// unrolled, so every value has a fixed register) and its N^3 residual
// accumulators in its own LDS column (lane-private: no barrier between the
// phases; in registers too, p = 2 would need 175 in FP32).  The register
// targets are what LDS admits, 3 (FP32) / 2 (FP64) waves per SIMD at p = 2,
// 2 / 1 at p = 3, and at p = 1 what measured best (FP32 6: 596 us, 5: 647;
// p = 2 FP32 at 4 spills: 5.39 for 5.22 ms).  (With the values of p = 3 in a
// second LDS column, loops rolled, LDS held 4 / 2 waves per CU: 3.07 / 6.60 ms
// per stage at 256 elements, 20^3 velocities, against 1.15 / 2.30.)  What
// bounds it: half VALU issue, half HBM (3.4-4.2 TB/s); p = 2 FP32, 2304
// elements, 24^3, limiter on: 5.99 -> 5.34 ms per stage with the exterior
// values requested a direction ahead, the connectivity and the metrics of
// whole lines through the scalar cache, one random-number hash per lane
// instead of per value, and the traces of waves that only enter left out;
// 5.22 with the points of the collision in pairs (p = 3 FP32 1.32 -> 1.14, and
// 63 registers fewer); 5.08 with the normals and margins as laid out below.
template <typename Real, int P>
constexpr int gen_waves() {
    if (sizeof(Real) == 8) return P == 3 ? 1 : 2;
    return P == 3 ? 2 : (P == 2 ? 3 : 6);
}
// Whether the next direction's exterior values are requested ahead: where
// that costs no wave per SIMD (at p = 2 it does in FP64 and for the residual
// alone: 1.44 -> 1.46 and 0.79 -> 0.84 ms at 1024 elements, 20^3).
template <typename Real, int P, int MODE>
constexpr bool gen_ahead() {
    return P == 1 || (P == 2 && sizeof(Real) == 4 && MODE == GMODE_STAGE);
}
// Whether a stage reads each margin with its normal.  The residual reads no
// margins: consecutive normals are fewer scalar loads (384 elements, 20^3, FP64,
// pairs / apart: p = 1 344 / 328 us, p = 2 912 / 850, p = 3 2998 / 2603).  The stage
// reads both; which is better is a matter of its registers: low-storage steps
// at that size p = 1 no difference, p = 2 FP64 2909 / 3055, FP32 1564 / 1561, p = 3
// FP64 9522 / 8713, FP32 4144 / 4258 us.
template <typename Real, int P, int MODE>
constexpr bool gen_pairs() {
    return MODE == GMODE_STAGE && P == (sizeof(Real) == 8 ? 2 : 3);
}
template <typename Real, int P, int MODE>
__global__ __launch_bounds__(kGWave) __attribute__((amdgpu_waves_per_eu(gen_waves<Real, P>()))) void
k_gen_stage(const GenArgs A) {
    constexpr int N = P + 1, NS = N * N * N, NFP = N * N;
    constexpr bool STAGE = MODE == GMODE_STAGE, PAIRS = gen_pairs<Real, P, MODE>();
    Real fv[NS];  // the lane's stage value
    __shared__ Real sa[NS][kGWave];
    __shared__ double sEb[STAGE ? NS * 8 : 1];
    __shared__ double sEv[STAGE ? NS * 3 : 1];
    __shared__ double sLg[STAGE ? NS : 1];  // log of the pair's G factor per point
    const int64_t e = blockIdx.x / A.nvw;
    const int lane = threadIdx.x;
    const int k = (int)(blockIdx.x % A.nvw) * kGWave + lane;
    const bool collide = STAGE && A.sa.collide;
    if (collide) {
        for (int s = lane; s < NS; s += kGWave) {
            const double *q = A.sa.eq + (e * NS + s) * kEqW;
            double *b = &sEb[s * 8];
            b[0] = -0.5 * q[EQ_B];
            b[1] = -0.5 * q[EQ_B + 1];
            b[2] = -0.5 * q[EQ_B + 2];
            b[3] = -q[EQ_B + 3];
            b[4] = -q[EQ_B + 4];
            b[5] = -q[EQ_B + 5];
            b[6] = q[EQ_C0];
            b[7] = q[EQ_INVTAU];
            sEv[s * 3] = q[EQ_V];
            sEv[s * 3 + 1] = q[EQ_V + 1];
            sEv[s * 3 + 2] = q[EQ_V + 2];
            if (A.ncomp == 2) {
                const double gf = A.gfp[e * NS + s];
                sLg[s] = gf > 0.0 ? log(gf) : -1000.0;
            }
        }
    }
    __syncthreads();
    if (k >= A.nut) return;

    const GOps<Real> &op = gops<Real>(A);
    const Metrics<Real> G = metrics(A, Real(0));
    const cptr<Real> gS = G.S + e * NS * 9, gJ = G.ijac + e * NS, gN = (PAIRS ? G.nm : G.nf) + e * 6 * NFP * 4;
    const int64_t nu = A.nut;  // stride of a solution point
    const int comp = k >= A.nu, kv = k - comp * A.nu;  // component, velocity node
    int iv[3];
    split_k(A.vg, kv, iv);
    const double ud[3] = {node_u(A.vg, 0, iv[0]), node_u(A.vg, 1, iv[1]), node_u(A.vg, 2, iv[2])};
    const Real u0 = (Real)ud[0], u1 = (Real)ud[1], u2 = (Real)ud[2];
    const int64_t eoff = e * NS * nu;
    const uint32_t ko = (uint32_t)k * (uint32_t)sizeof(Real), k8 = (uint32_t)k * 8u, kv8 = (uint32_t)kv * 8u;
    const Real *fe = reinterpret_cast<const Real *>(A.sa.f) + eoff;
#pragma unroll
    for (int s = 0; s < NS; ++s) fv[s] = ldo(fe + s * nu, ko);
    // the second RK register of the stage
    const bool useX = STAGE && (A.sa.scheme == 0 ? A.sa.alpha != 0.0 : A.sa.lsA != 0.0);
    const Real *XE = reinterpret_cast<const Real *>(A.sa.fn) + eoff;
    // Divergence and interface corrections, direction by direction: along
    // each line of direction d the transformed flux F_d = (a^d . u) f, its
    // derivative, and the corrections of the line's two flux points on the
    // faces 2d and 2d+1 are formed in registers; each point's accumulator
    // is then written once per direction (the first direction initialises
    // it), so no accumulator waits on another update of itself.
    const Real *tin = reinterpret_cast<const Real *>(A.sa.tr_in);
    const Real ul1 = (u0 < 0 ? -u0 : u0) + (u1 < 0 ? -u1 : u1) + (u2 < 0 ? -u2 : u2);
    uint64_t kept[2] = {0, 0};  // flux points (face * NFP + q) whose traces the wave stores
    ExtArgs<Real> X = {(cptr<int32_t>)A.conn + e * 24, {}, (cptr<double>)A.rw + e * 6 * NFP, gN, A.finf, A.mw, tin,
                       comp ? A.gwall : 1.0, e, nu, ko, k8, kv8, u0, u1, u2, ul1};
    // the connectivity of all faces now: face by face, each direction's
    // requests would wait for it (at p = 1 the registers cost more than that)
    constexpr bool CONN = P > 1;
    if constexpr (CONN) {
#pragma unroll
        for (int i = 0; i < 24; ++i) X.cn[i] = X.conn[i];
    }
    const int km0 = k + A.vg.nv[0] - 1 - 2 * iv[0], km1 = k + (A.vg.nv[1] - 1 - 2 * iv[1]) * A.vg.nv[0],
              km2 = k + (A.vg.nv[2] - 1 - 2 * iv[2]) * (A.vg.nv[0] * A.vg.nv[1]);
    // the next direction's exterior values, and before the last direction the
    // first layer's second-register values, are requested while a direction
    // is computed
    constexpr bool AHEAD = gen_ahead<Real, P, MODE>();
    Real unx[2][2][NFP], exx[2][2][NFP];
    if constexpr (AHEAD) load_ext<Real, N, STAGE, CONN, PAIRS>(X, 0, km0, km1, km2, unx[0], exx[0], kept);
    Real xv[2][NFP];
    auto load_x = [&](int s0, Real(&x)[NFP]) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < NFP; ++r) x[r] = useX ? ldo(XE + (s0 + r) * nu, ko) : Real(0);
    };
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        Real un[2][NFP], ext[2][NFP];
        // one direction's exterior values (and the next one's) in registers at a time
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (AHEAD) {
            if (d < 2) load_ext<Real, N, STAGE, CONN, PAIRS>(X, d + 1, km0, km1, km2, unx[(d + 1) & 1], exx[(d + 1) & 1], kept);
            else if (STAGE) load_x(0, xv[0]);
#pragma unroll
            for (int side = 0; side < 2; ++side)
#pragma unroll
                for (int q = 0; q < NFP; ++q) {
                    un[side][q] = unx[d & 1][side][q];
                    ext[side][q] = exx[d & 1][side][q];
                }
        } else {
            load_ext<Real, N, STAGE, CONN, PAIRS>(X, d, km0, km1, km2, un, ext, kept);
        }
#pragma unroll
        for (int q = 0; q < NFP; ++q) {
            const int a = q % N, b = q / N;
            int pts[N];
            Real fl[N], Fd[N];
            const cptr<Real> Sq = gS + (d * NFP + q) * N * 3;
#pragma unroll
            for (int m = 0; m < N; ++m) {
                pts[m] = line_pt<N>(d, a, b, m);
                fl[m] = fv[pts[m]];
                const cptr<Real> Sm = Sq + m * 3;
                Fd[m] = (Sm[0] * u0 + Sm[1] * u1 + Sm[2] * u2) * fl[m];
            }
            Real acc[N];
#pragma unroll
            for (int r = 0; r < N; ++r) {
                Real t = Real(0);
#pragma unroll
                for (int m = 0; m < N; ++m) t += op.D[r * N + m] * Fd[m];
                acc[r] = t;
            }
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                if (un[side][q] < Real(0)) {
                    const Real jump = un[side][q] * (ext[side][q] - face_value<Real, N>(op.lam[side], fl));
#pragma unroll
                    for (int r = 0; r < N; ++r) acc[r] += op.corr[side][r] * jump;
                }
            }
#pragma unroll
            for (int r = 0; r < N; ++r) sa[pts[r]][lane] = d == 0 ? acc[r] : sa[pts[r]][lane] + acc[r];
        }
    }
    if (MODE == GMODE_RESID) {
        Real *R = reinterpret_cast<Real *>(A.sa.fout) + eoff;
#pragma unroll 4
        for (int s = 0; s < NS; ++s) sto(R + s * nu, ko, -sa[s][lane] * gJ[s]);
        return;
    }
    // collision source and the Runge-Kutta combination
    const Real dt = (Real)A.sa.dt;
    Real *outE = reinterpret_cast<Real *>(A.sa.fout) + eoff;
    Real *dFE = reinterpret_cast<Real *>(A.sa.dF) + eoff;
    // positivity limiter: the result is held in the value registers (fv)
    // until its element mean and smallest value are known
    const bool limit = A.sa.positivity != 0;
    const cptr<double> gW = (cptr<double>)A.wJ + e * NS;
    Real lim_min = Real(0);
    // random bits of the stochastic rounding: one hash per lane, a xorshift
    // step per value
    uint32_t rs = sizeof(Real) == 4 ? round_bits(A.sa.seed, (uint32_t)(e * NS), (uint32_t)k) | 1u : 0u;
    // One loop per combination of the launch-uniform switches (the collision,
    // the RK scheme, whether dF is kept): no branch splits the points, and two
    // chains run side by side.
    auto points = [&](auto coll_c, auto lsrk_c, auto keep_c) __attribute__((always_inline)) {
        constexpr bool COLL = decltype(coll_c)::value, LSRK = decltype(lsrk_c)::value;
        constexpr bool KEEP = decltype(keep_c)::value;
        auto group = [&](auto width, int s0, const Real *x) __attribute__((always_inline)) {
            constexpr int W = decltype(width)::value;
            Real g[W];
            if constexpr (COLL) {
                double E[W];
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    const int s = s0 + i;
                    const double *bq = &sEb[s * 8];
                    const double c0 = ud[0] - sEv[s * 3], c1 = ud[1] - sEv[s * 3 + 1], c2 = ud[2] - sEv[s * 3 + 2];
                    double t0 = bq[0] * c0;
                    t0 = fma(bq[3], c1, t0);
                    t0 = fma(bq[4], c2, t0);
                    double t1 = bq[1] * c1;
                    t1 = fma(bq[5], c2, t1);
                    const double t2 = bq[2] * c2;
                    E[i] = fma(c0, t0, comp ? bq[6] + sLg[s] : bq[6]);
                    E[i] = fma(c1, t1, E[i]);
                    E[i] = fma(c2, t2, E[i]);
                }
                gexp<W>(E, g);
            }
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const int s = s0 + i;
                const Real fq = fv[s];
                Real L = -sa[s][lane] * gJ[s];
                if constexpr (COLL) L += (g[i] - fq) * (Real)sEb[s * 8 + 7];
                // the result, in FP64 for the stochastic rounding of the FP32 state
                double fod;
                if constexpr (!LSRK) {
                    fod = A.sa.beta * ((double)fq + (double)(dt * L));
                    fod = fma(A.sa.alpha, (double)x[i], fod);  // (0 when not read)
                } else {
                    Real dd = dt * L;
                    dd += (Real)A.sa.lsA * x[i];
                    if constexpr (KEEP) sto(dFE + s * nu, ko, dd);
                    fod = fma(A.sa.lsB, (double)dd, (double)fq);
                }
                Real fo;
                if constexpr (sizeof(Real) == 4) {
                    rs = xorshift32(rs);
                    fo = round_stochastic(fod, rs);
                } else {
                    fo = (Real)fod;
                }
                fv[s] = fo;
                lim_min = s == 0 ? fo : (fo < lim_min ? fo : lim_min);
                sto(outE + s * nu, ko, fo);
            }
            // (the fences bound the chains in flight at once)
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int s0 = 0; s0 < NS; s0 += NFP) {
            // a layer's second-register values requested together
            if constexpr (AHEAD) {
                if (s0 + NFP < NS) load_x(s0 + NFP, xv[(s0 / NFP + 1) & 1]);
            } else {
                load_x(s0, xv[(s0 / NFP) & 1]);
            }
            const Real *x = xv[(s0 / NFP) & 1];
#pragma unroll
            for (int r = 0; r + 2 <= NFP; r += 2) group(IntC<2>{}, s0 + r, x + r);
            if constexpr (NFP % 2) group(IntC<1>{}, s0 + NFP - 1, x + NFP - 1);
        }
    };
    if constexpr (STAGE) {
        if (A.sa.scheme == 0) {
            if (collide) points(BoolC<true>{}, BoolC<false>{}, BoolC<false>{});
            else points(BoolC<false>{}, BoolC<false>{}, BoolC<false>{});
        } else if (A.sa.keep_dF) {
            if (collide) points(BoolC<true>{}, BoolC<true>{}, BoolC<true>{});
            else points(BoolC<false>{}, BoolC<true>{}, BoolC<true>{});
        } else {
            if (collide) points(BoolC<true>{}, BoolC<true>{}, BoolC<false>{});
            else points(BoolC<false>{}, BoolC<true>{}, BoolC<false>{});
        }
    }
    // Traces of the result where the velocity leaves; with the positivity limiter
    // the same pass (over every flux point) finds the smallest value of the element polynomial at its
    // solution and flux points.  Where that is negative (rare: f is positive
    // almost everywhere) the lane scales its polynomial about the element mean
    // (weights Gauss x |J|), so that the smallest value becomes zero and the
    // element integral of the value, hence every moment, is kept, and stores
    // the values and traces again.
    Real *te = reinterpret_cast<Real *>(A.sa.tr_out) + e * 6 * NFP * nu;
    auto trace_pass = [&](bool store, bool find_min) {
#pragma unroll
        for (int face = 0; face < 6; ++face) {
            const int d = face / 2, side = face & 1;
            // one face's traces in registers at a time
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < NFP; ++q) {
                const int a = q % N, b = q / N;
                Real line[N];
#pragma unroll
                for (int m = 0; m < N; ++m) line[m] = fv[line_pt<N>(d, a, b, m)];
                const Real t = face_value<Real, N>(op.lam[side], line);
                const int pt = face * NFP + q;
                if (store && ((kept[pt >> 6] >> (pt & 63)) & 1)) sto(te + pt * nu, ko, t);
                if (find_min) lim_min = t < lim_min ? t : lim_min;
            }
        }
    };
    if (A.do_traces || limit) trace_pass(A.do_traces, limit);
    if (limit && lim_min < Real(0)) {
        double lim_int = 0.0, lim_w = 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            lim_int = fma(gW[s], (double)fv[s], lim_int);
            lim_w += gW[s];
        }
        const double mean = lim_int / lim_w;
        const double th = mean > 0.0 ? mean / (mean - (double)lim_min) : 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const Real v = (Real)fma(th, (double)fv[s] - mean, mean);
            fv[s] = v;
            sto(outE + s * nu, ko, v);
        }
        if (A.do_traces) trace_pass(true, false);
    }
}

int gcheck(fr_dvm *h, const char *what) {
    hipError_t st = hipGetLastError();
    if (st != hipSuccess) return h->fail(FR_DVM_EHIP, std::string(what) + ": " + hipGetErrorString(st));
    return FR_DVM_OK;
}

template <typename Real, int P>
int gen_run(fr_dvm *h, int mode, const GenArgs &A, int do_moments) {
    const unsigned blocks = (unsigned)(h->ne * A.nvb);
    const int64_t npts = h->ne * h->ns;
    auto moments = [&](const void *src) {
        const Real *fs = reinterpret_cast<const Real *>(src);
        switch (h->nmom) {
            case 5: hipLaunchKernelGGL((k_gen_moments<Real, 5>), dim3(gen_moment_grid(npts)), dim3(64 * kMomPts), 0, h->stream, A, fs, A.sa.Q, (int64_t)npts); break;
            case 6: hipLaunchKernelGGL((k_gen_moments<Real, 6>), dim3(gen_moment_grid(npts)), dim3(64 * kMomPts), 0, h->stream, A, fs, A.sa.Q, (int64_t)npts); break;
            case 10: hipLaunchKernelGGL((k_gen_moments<Real, 10>), dim3(gen_moment_grid(npts)), dim3(64 * kMomPts), 0, h->stream, A, fs, A.sa.Q, (int64_t)npts); break;
            default: hipLaunchKernelGGL((k_gen_moments<Real, 11>), dim3(gen_moment_grid(npts)), dim3(64 * kMomPts), 0, h->stream, A, fs, A.sa.Q, (int64_t)npts);
        }
        return gcheck(h, "moment kernel");
    };
    int rc;
    if (mode == 0) {
        if (A.do_traces) {
            const Real *f = reinterpret_cast<const Real *>(A.sa.f);
            Real *tr = reinterpret_cast<Real *>(A.sa.tr_out);
            if (npts * A.nut * (int64_t)sizeof(Real) <= kGenAllBytes)
                hipLaunchKernelGGL((k_gen_traces<Real, P, true>), dim3(blocks), dim3(kGBlock), 0, h->stream, A, f, tr);
            else
                hipLaunchKernelGGL((k_gen_traces<Real, P, false>), dim3(blocks), dim3(kGBlock), 0, h->stream, A, f, tr);
            if ((rc = gcheck(h, "trace kernel"))) return rc;
        }
        return do_moments ? moments(A.sa.f) : FR_DVM_OK;
    }
    if (h->nwall) {
        hipLaunchKernelGGL((k_gen_wall<Real, P>), dim3((unsigned)(h->nwall * h->nfp)), dim3(kGBlock), 0, h->stream,
                           A, reinterpret_cast<const Real *>(A.sa.tr_in));
        if ((rc = gcheck(h, "wall kernel"))) return rc;
    }
    const unsigned wblocks = (unsigned)(h->ne * A.nvw);
    if (mode == GMODE_RESID)
        hipLaunchKernelGGL((k_gen_stage<Real, P, GMODE_RESID>), dim3(wblocks), dim3(kGWave), 0, h->stream, A);
    else
        hipLaunchKernelGGL((k_gen_stage<Real, P, GMODE_STAGE>), dim3(wblocks), dim3(kGWave), 0, h->stream, A);
    if ((rc = gcheck(h, "general stage kernel"))) return rc;
    return (mode == GMODE_STAGE && do_moments) ? moments(A.sa.fout) : FR_DVM_OK;
}

template <typename Real>
int gen_p(fr_dvm *h, int mode, const GenArgs &A, int do_moments) {
    switch (h->p) {
        case 1: return gen_run<Real, 1>(h, mode, A, do_moments);
        case 2: return gen_run<Real, 2>(h, mode, A, do_moments);
        case 3: return gen_run<Real, 3>(h, mode, A, do_moments);
    }
    return h->fail(FR_DVM_EUNSUPPORTED, "order");
}

// ---- mixed meshes of straight hexahedra, prisms and tetrahedra ----
//
// Nodal FR with the DG-recovering correction on each element (Section
// "Numerical method"): with f the element's values at its solution points,
//   R_i = -sum_j (sum_a c_a D_a[i][j]) f_j
//         - sum_t lift[i][t] s_f min(u.n_f, 0) (f_nb,t - f_node(t)),
// c_a = u . grad xi_a (constant on a straight element), t running over the
// face points (the solution points on each face, faces in order), f_nb,t the
// neighbour's value at the same position, s_f = |J_face| / |J|.  The flux
// points are solution points, so the neighbours' traces are read from the
// stage value itself; no trace is stored (a stage never writes over the value
// it reads).  One wave per (element, 64 velocities), one lane per velocity,
// the operators read through the scalar cache.  The collision source and the
// RK combination are those of the hexahedral kernels.
struct MixArgs {
    VGrid vg;
    int nu, nvw;
    const int32_t *elems;                 // elements of the launched type
    const int64_t *poff, *toff, *pnb;     // first point / face point of each element; the neighbour's point at each face point
    const double *geo;                    // [ne][kMixGeo]
    const float *geof;
    const double *D, *lift, *stream;      // the type's operators: hexahedra D [3][ns][ns], lift [nft][ns]; others the stream
    const float *Df, *liftf, *streamf;
    const int32_t *fnode, *ffac;          // hexahedra: [nft] solution point and face of each face point
    StageArgs sa;
};

template <typename Real>
struct MixOps {
    cptr<Real> geo, D, lift, stream;
};
__device__ __forceinline__ MixOps<float> mix_ops(const MixArgs &A, float) {
    return {(cptr<float>)A.geof, (cptr<float>)A.Df, (cptr<float>)A.liftf, (cptr<float>)A.streamf};
}
__device__ __forceinline__ MixOps<double> mix_ops(const MixArgs &A, double) {
    return {(cptr<double>)A.geo, (cptr<double>)A.D, (cptr<double>)A.lift, (cptr<double>)A.stream};
}

// The wave's element, its lane's velocity and the velocity's contravariant
// components; a lane past the last node does and stores exactly what the lane
// of the last node (of the same wave) does.
template <typename Real>
struct MixLane {
    int64_t e, p0, t0, nu;
    int k;
    uint32_t ko;
    double ud[3];
    Real u0, u1, u2, c[3];
    cptr<Real> g;
    __device__ __forceinline__ MixLane(const MixArgs &A, const MixOps<Real> &op) {
        e = A.elems[blockIdx.x / A.nvw];
        k = (int)(blockIdx.x % A.nvw) * kGWave + threadIdx.x;
        k = k < A.nu ? k : A.nu - 1;
        nu = A.nu;
        ko = (uint32_t)k * (uint32_t)sizeof(Real);
        p0 = A.poff[e];
        t0 = A.toff[e];
        g = op.geo + e * kMixGeo;
        int iv[3];
        split_k(A.vg, k, iv);
#pragma unroll
        for (int d = 0; d < 3; ++d) ud[d] = node_u(A.vg, d, iv[d]);
        u0 = (Real)ud[0];
        u1 = (Real)ud[1];
        u2 = (Real)ud[2];
#pragma unroll
        for (int a = 0; a < 3; ++a) c[a] = u0 * g[3 * a] + u1 * g[3 * a + 1] + u2 * g[3 * a + 2];
    }
    __device__ __forceinline__ Real un(int f) const { return u0 * g[9 + 3 * f] + u1 * g[10 + 3 * f] + u2 * g[11 + 3 * f]; }
};

// Collision source and Runge-Kutta combination of an element's points with
// values val(i) and advective residuals res(i); stores the results.  One loop
// per combination of the launch-uniform switches (the collision, the RK
// scheme, whether dF is kept), XB second-register values requested together
// and two points' chains side by side.
template <typename Real, int NS, int XB, typename Val, typename Res>
__device__ __forceinline__ void mix_points(const MixArgs &A, const MixLane<Real> &v, Val val, Res res) {
    const bool useX = A.sa.scheme == 0 ? A.sa.alpha != 0.0 : A.sa.lsA != 0.0;
    const Real *XE = reinterpret_cast<const Real *>(A.sa.fn) + v.p0 * v.nu;
    Real *dFE = reinterpret_cast<Real *>(A.sa.dF) + v.p0 * v.nu;
    Real *outE = reinterpret_cast<Real *>(A.sa.fout) + v.p0 * v.nu;
    const Real dt = (Real)A.sa.dt;
    // the lane's stream of random bits, one xorshift step per value
    uint32_t rs = sizeof(Real) == 4 ? round_bits(A.sa.seed, (uint32_t)v.p0, (uint32_t)v.k) | 1u : 0u;
    auto points = [&](auto coll_c, auto lsrk_c, auto keep_c) __attribute__((always_inline)) {
        constexpr bool COLL = decltype(coll_c)::value, LSRK = decltype(lsrk_c)::value;
        constexpr bool KEEP = decltype(keep_c)::value;
        auto group = [&](auto width, int i0, const Real *x) __attribute__((always_inline)) {
            constexpr int W = decltype(width)::value;
            Real g[W], it[W];
            if constexpr (COLL) {
                double E[W];
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const cptr<double> q = (cptr<double>)A.sa.eq + (v.p0 + i0 + w) * kEqW;
                    const double c0 = v.ud[0] - q[EQ_V], c1 = v.ud[1] - q[EQ_V + 1], c2 = v.ud[2] - q[EQ_V + 2];
                    double t0 = -0.5 * q[EQ_B] * c0;
                    t0 = fma(-q[EQ_B + 3], c1, t0);
                    t0 = fma(-q[EQ_B + 4], c2, t0);
                    double t1 = -0.5 * q[EQ_B + 1] * c1;
                    t1 = fma(-q[EQ_B + 5], c2, t1);
                    const double t2 = -0.5 * q[EQ_B + 2] * c2;
                    E[w] = fma(c0, t0, q[EQ_C0]);
                    E[w] = fma(c1, t1, E[w]);
                    E[w] = fma(c2, t2, E[w]);
                    it[w] = (Real)q[EQ_INVTAU];
                }
                gexp<W>(E, g);
            }
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int i = i0 + w;
                const Real fq = val(i);
                Real L = res(i);
                if constexpr (COLL) L += (g[w] - fq) * it[w];
                double fod;
                if constexpr (!LSRK) {
                    fod = A.sa.beta * ((double)fq + (double)(dt * L));
                    fod = fma(A.sa.alpha, (double)x[w], fod);  // (0 when not read)
                } else {
                    Real dd = dt * L;
                    dd += (Real)A.sa.lsA * x[w];
                    if constexpr (KEEP) sto(dFE + i * v.nu, v.ko, dd);
                    fod = fma(A.sa.lsB, (double)dd, (double)fq);
                }
                Real fo;
                if constexpr (sizeof(Real) == 4) {
                    rs = xorshift32(rs);
                    fo = round_stochastic(fod, rs);
                } else {
                    fo = (Real)fod;
                }
                sto(outE + i * v.nu, v.ko, fo);
            }
        };
#pragma unroll
        for (int i0 = 0; i0 < NS; i0 += XB) {
            Real xv[XB];
#pragma unroll
            for (int x = 0; x < XB; ++x)
                if (i0 + x < NS) xv[x] = useX ? ldo(XE + (i0 + x) * v.nu, v.ko) : Real(0);
#pragma unroll
            for (int x = 0; x < XB; x += 2) {
                if (x + 2 <= XB && i0 + x + 2 <= NS) group(IntC<2>{}, i0 + x, &xv[x]);
                else if (i0 + x < NS) group(IntC<1>{}, i0 + x, &xv[x]);
            }
        }
    };
    if (A.sa.scheme == 0) {
        if (A.sa.collide) points(BoolC<true>{}, BoolC<false>{}, BoolC<false>{});
        else points(BoolC<false>{}, BoolC<false>{}, BoolC<false>{});
    } else if (A.sa.keep_dF) {
        if (A.sa.collide) points(BoolC<true>{}, BoolC<true>{}, BoolC<true>{});
        else points(BoolC<false>{}, BoolC<true>{}, BoolC<true>{});
    } else {
        if (A.sa.collide) points(BoolC<true>{}, BoolC<true>{}, BoolC<false>{});
        else points(BoolC<false>{}, BoolC<true>{}, BoolC<false>{});
    }
}

// Hexahedra: dense operators; up to 27 points the values and residuals in
// registers, above in LDS columns.
template <typename Real, int NS, int NFT, int MODE>
__global__ __launch_bounds__(kGWave) void k_mix_hex(const MixArgs A) {
    constexpr bool REG = NS <= 27;
    __shared__ Real sf[NS][kGWave];
    __shared__ Real sa[REG ? 1 : NS][kGWave];
    const MixOps<Real> op = mix_ops(A, Real(0));
    const MixLane<Real> v(A, op);
    const int lane = threadIdx.x;
    const int64_t nu = v.nu;
    const cptr<int32_t> fnode = (cptr<int32_t>)A.fnode, ffac = (cptr<int32_t>)A.ffac;
    const cptr<int64_t> pnb = (cptr<int64_t>)A.pnb + v.t0;
    const Real *fin = reinterpret_cast<const Real *>(A.sa.f);
    const Real *fE = fin + v.p0 * nu;
    // the upwind jump at face point t, scaled (0 where the velocity leaves)
    auto jump_at = [&](int t) {
        const int f = ffac[t];
        const Real un = v.un(f);
        Real jump = Real(0);
        if (un < Real(0)) jump = un * v.g[27 + f] * (ldo(fin + pnb[t] * nu, v.ko) - sf[fnode[t]][lane]);
        return jump;
    };
    Real fv[REG ? NS : 1], r[REG ? NS : 1];
    if constexpr (REG) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            fv[i] = ldo(fE + i * nu, v.ko);
            sf[i][lane] = fv[i];
            r[i] = Real(0);
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                Real gi = Real(0);
#pragma unroll
                for (int j = 0; j < NS; ++j) gi = fma(op.D[(a * NS + i) * NS + j], fv[j], gi);
                r[i] = fma(-v.c[a], gi, r[i]);
            }
        }
#pragma unroll 1
        for (int t = 0; t < NFT; ++t) {
            const Real jump = jump_at(t);
#pragma unroll
            for (int i = 0; i < NS; ++i) r[i] = fma(-op.lift[t * NS + i], jump, r[i]);
        }
    } else {
#pragma unroll 4
        for (int i = 0; i < NS; ++i) sf[i][lane] = ldo(fE + i * nu, v.ko);
#pragma unroll 1
        for (int i = 0; i < NS; ++i) {
            Real acc = Real(0);
#pragma unroll 4
            for (int j = 0; j < NS; ++j) {
                const Real w = v.c[0] * op.D[i * NS + j] + v.c[1] * op.D[(NS + i) * NS + j] + v.c[2] * op.D[(2 * NS + i) * NS + j];
                acc = fma(w, sf[j][lane], acc);
            }
            sa[i][lane] = -acc;
        }
#pragma unroll 1
        for (int t = 0; t < NFT; ++t) {
            const Real jump = jump_at(t);
#pragma unroll 4
            for (int i = 0; i < NS; ++i) sa[i][lane] -= op.lift[t * NS + i] * jump;
        }
    }
    auto res = [&](int i) -> Real {
        if constexpr (REG) return r[i];
        else return sa[i][lane];
    };
    auto val = [&](int i) -> Real {
        if constexpr (REG) return fv[i];
        else return sf[i][lane];
    };
    if (MODE == GMODE_RESID) {
        Real *R = reinterpret_cast<Real *>(A.sa.fout) + v.p0 * nu;
#pragma unroll
        for (int i = 0; i < NS; ++i) sto(R + i * nu, v.ko, res(i));
        return;
    }
    if constexpr (MODE == GMODE_STAGE) mix_points<Real, NS, 2>(A, v, val, res);
}

// Prisms (DIM 2: the triangle's points on the PL = p + 1 Gauss-Lobatto layers
// of a line) and tetrahedra (DIM 3): values and residuals in registers, the
// operators as scalar operands from one stream in the order of use, only
// their nonzero entries (frdvm_simplex.h); a prism's entry serves all layers
// (columns) at once.  A face's normal is constant, so whether a velocity
// enters is decided once per face: a wave none of whose velocities enter
// skips the face, and the neighbour's values of a face are requested
// together.  What bounds it: HBM (f, the neighbours' face values, the result,
// the second register) and, for tetrahedra, VALU issue.  A stage of 51,200
// points at p = 3, 24^3 velocities, FP32 low-storage: tetrahedra 3.44 -> 1.64 ms
// (4.2 TB/s), prisms 2.70 -> 1.22 ms (3.7 TB/s); before, with dense
// tetrahedral products, the face points one after the other through LDS and
// their traces stored and read back, VALU issue and load latency bound it.
// Points in pairs without branches (mix_points; before, each point waited
// for its record and branched on the collision, the scheme, the register and
// the idle lanes): tetrahedra 1.64 -> 1.53 ms, prisms 1.22 -> 1.13 ms, FP64
// tetrahedra 0.63 -> 0.59 ms, prisms 0.55 -> 0.50 ms at 21,600 points, 20^3.
// Waves per SIMD the registers are held to: what the kernel needs by itself,
// and where a few registers stand in the way of one more wave (p = 3: prisms
// FP32, tetrahedra FP64) that wave: 1.25 / 1.05 ms and 0.69 / 0.59 ms per
// stage without / with it.  (6 waves for FP32 tetrahedra leave arrays in
// scratch memory: 34 ms.)
template <typename Real, int DIM, int P>
constexpr int mix_waves() {
    if (DIM == 2) return P == 1 ? 8 : (P == 2 ? (sizeof(Real) == 4 ? 5 : 4) : (sizeof(Real) == 4 ? 4 : 2));
    return P == 1 ? 8 : (P == 2 ? (sizeof(Real) == 4 ? 6 : 5) : (sizeof(Real) == 4 ? 5 : 4));
}
template <typename Real, int DIM, int P, int MODE>
__global__ __launch_bounds__(kGWave) __attribute__((amdgpu_waves_per_eu(mix_waves<Real, DIM, P>()))) void
k_mix_simplex(const MixArgs A) {
    using S = Simplex<DIM, P>;
    constexpr auto tb = S::table();
    constexpr auto rest = S::rest();
    constexpr auto face = S::faces();
    constexpr int NT = S::NP, NM = S::NM, PL = DIM == 2 ? P + 1 : 1, NS = NT * PL;
    const MixOps<Real> op = mix_ops(A, Real(0));
    const MixLane<Real> v(A, op);
    const int64_t nu = v.nu;
    const cptr<int64_t> pnb = (cptr<int64_t>)A.pnb + v.t0;
    const Real *fin = reinterpret_cast<const Real *>(A.sa.f);
    const Real *fE = fin + v.p0 * nu;
    Real fv[NS], r[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) fv[i] = ldo(fE + i * nu, v.ko);
    int o = 0;  // position in the stream (a constant everywhere once unrolled)
    // volume: r = -sum_a c_a D_a f at the sub points, then interpolated
#pragma unroll
    for (int m = 0; m < NM; ++m) {
        Real gm[PL];
#pragma unroll
        for (int k = 0; k < PL; ++k) gm[k] = Real(0);
#pragma unroll
        for (int a = 0; a < DIM; ++a) {
            Real s[PL];
#pragma unroll
            for (int k = 0; k < PL; ++k) s[k] = Real(0);
#pragma unroll
            for (int j = 0; j < NT; ++j)
                if ((tb.d[a][m] >> j) & 1) {
                    const Real w = op.stream[o++];
#pragma unroll
                    for (int k = 0; k < PL; ++k) s[k] = fma(w, fv[j + NT * k], s[k]);
                }
#pragma unroll
            for (int k = 0; k < PL; ++k) gm[k] = fma(-v.c[a], s[k], gm[k]);
        }
#pragma unroll
        for (int k = 0; k < PL; ++k) r[tb.sub[m] + NT * k] = gm[k];
    }
#pragma unroll
    for (int q = 0; q < NT - NM; ++q) {
        Real s[PL];
#pragma unroll
        for (int k = 0; k < PL; ++k) s[k] = Real(0);
#pragma unroll
        for (int m = 0; m < NM; ++m)
            if ((tb.e[q] >> m) & 1) {
                const Real w = op.stream[o++];
#pragma unroll
                for (int k = 0; k < PL; ++k) s[k] = fma(w, r[tb.sub[m] + NT * k], s[k]);
            }
#pragma unroll
        for (int k = 0; k < PL; ++k) r[rest.i[q] + NT * k] = s[k];
    }
    if constexpr (DIM == 3) {
#pragma unroll
        for (int f = 0; f < S::NFACE; ++f) {
            const Real un = v.un(f);
            if (un < Real(0)) {
                const Real sc = un * v.g[27 + f];
                Real ext[S::NF];
#pragma unroll
                for (int t = 0; t < S::NF; ++t) ext[t] = ldo(fin + pnb[f * S::NF + t] * nu, v.ko);
#pragma unroll
                for (int t = 0; t < S::NF; ++t) {
                    const Real jump = sc * (ext[t] - fv[face.n[f][t]]);
#pragma unroll
                    for (int i = 0; i < NS; ++i)
                        r[i] = fma(-op.stream[o + (f * S::NF + t) * NS + i], jump, r[i]);
                }
            }
        }
    } else {
        // axial derivative, column by column
#pragma unroll
        for (int i = 0; i < PL; ++i)
#pragma unroll
            for (int m = 0; m < NT; ++m) {
                Real s = Real(0);
#pragma unroll
                for (int k = 0; k < PL; ++k) s = fma(op.stream[o + i * PL + k], fv[m + NT * k], s);
                r[m + NT * i] = fma(-v.c[2], s, r[m + NT * i]);
            }
        o += PL * PL;
        // bottom and top: point m lifts onto its column
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const Real un = v.un(f);
            if (un < Real(0)) {
                const Real sc = un * v.g[27 + f];
                Real ext[NT];
#pragma unroll
                for (int m = 0; m < NT; ++m) ext[m] = ldo(fin + pnb[f * NT + m] * nu, v.ko);
#pragma unroll
                for (int m = 0; m < NT; ++m) {
                    const Real jump = sc * (ext[m] - fv[m + (f ? NT * (PL - 1) : 0)]);
#pragma unroll
                    for (int k = 0; k < PL; ++k) r[m + NT * k] = fma(-op.stream[o + f * PL + k], jump, r[m + NT * k]);
                }
            }
        }
        o += 2 * PL;
        // sides: edge point e on layer k lifts onto the layer; the points of
        // EB edge points requested together
        constexpr int EB = sizeof(Real) == 4 || PL < 3 ? PL : 2;
#pragma unroll
        for (int f = 0; f < 3; ++f) {
            const Real un = v.un(2 + f);
            if (un < Real(0)) {
                const Real sc = un * v.g[29 + f];
#pragma unroll
                for (int e0 = 0; e0 < PL; e0 += EB) {
                    Real ext[EB][PL];
#pragma unroll
                    for (int x = 0; x < EB; ++x)
                        if (e0 + x < PL)
#pragma unroll
                            for (int k = 0; k < PL; ++k)
                                ext[x][k] = ldo(fin + pnb[2 * NT + f * PL * PL + e0 + x + PL * k] * nu, v.ko);
#pragma unroll
                    for (int x = 0; x < EB; ++x)
                        if (e0 + x < PL) {
                            Real jump[PL];
#pragma unroll
                            for (int k = 0; k < PL; ++k) jump[k] = sc * (ext[x][k] - fv[face.n[f][e0 + x] + NT * k]);
#pragma unroll
                            for (int m = 0; m < NT; ++m) {
                                const Real w = -op.stream[o + (f * PL + e0 + x) * NT + m];
#pragma unroll
                                for (int k = 0; k < PL; ++k) r[m + NT * k] = fma(w, jump[k], r[m + NT * k]);
                            }
                        }
                }
            }
        }
    }
    if (MODE == GMODE_RESID) {
        Real *R = reinterpret_cast<Real *>(A.sa.fout) + v.p0 * nu;
#pragma unroll
        for (int i = 0; i < NS; ++i) sto(R + i * nu, v.ko, r[i]);
        return;
    }
    // a layer's (the tetrahedron: ten points') second-register values together
    if constexpr (MODE == GMODE_STAGE)
        mix_points<Real, NS, DIM == 2 ? NT : (NS < 10 ? NS : 10)>(
            A, v, [&](int i) __attribute__((always_inline)) { return fv[i]; },
            [&](int i) __attribute__((always_inline)) { return r[i]; });
}

template <typename Real, int NS, int NFT>
int mix_hex(fr_dvm *h, int mode, const MixArgs &A, unsigned blocks) {
    if (mode == GMODE_RESID)
        hipLaunchKernelGGL((k_mix_hex<Real, NS, NFT, GMODE_RESID>), dim3(blocks), dim3(kGWave), 0, h->stream, A);
    else
        hipLaunchKernelGGL((k_mix_hex<Real, NS, NFT, GMODE_STAGE>), dim3(blocks), dim3(kGWave), 0, h->stream, A);
    return gcheck(h, "mixed-mesh kernel");
}
template <typename Real, int DIM, int P>
int mix_simplex(fr_dvm *h, int mode, const MixArgs &A, unsigned blocks) {
    if (mode == GMODE_RESID)
        hipLaunchKernelGGL((k_mix_simplex<Real, DIM, P, GMODE_RESID>), dim3(blocks), dim3(kGWave), 0, h->stream, A);
    else
        hipLaunchKernelGGL((k_mix_simplex<Real, DIM, P, GMODE_STAGE>), dim3(blocks), dim3(kGWave), 0, h->stream, A);
    return gcheck(h, "mixed-mesh kernel");
}

// (type, order) -> the kernel instantiation for its point counts
template <typename Real>
int mix_dispatch(fr_dvm *h, int mode, const MixArgs &A, int t, unsigned blocks) {
    switch (10 * t + h->p) {
        case 1: return mix_hex<Real, 8, 24>(h, mode, A, blocks);
        case 2: return mix_hex<Real, 27, 54>(h, mode, A, blocks);
        case 3: return mix_hex<Real, 64, 96>(h, mode, A, blocks);
        case 11: return mix_simplex<Real, 2, 1>(h, mode, A, blocks);
        case 12: return mix_simplex<Real, 2, 2>(h, mode, A, blocks);
        case 13: return mix_simplex<Real, 2, 3>(h, mode, A, blocks);
        case 21: return mix_simplex<Real, 3, 1>(h, mode, A, blocks);
        case 22: return mix_simplex<Real, 3, 2>(h, mode, A, blocks);
        case 23: return mix_simplex<Real, 3, 3>(h, mode, A, blocks);
    }
    return h->fail(FR_DVM_EUNSUPPORTED, "mixed-mesh element type / order");
}

template <typename Real>
int mix_run(fr_dvm *h, int mode, const StageArgs &sa, int do_moments) {
    const Mixed &mx = *h->mx;
    MixArgs A;
    std::memset(&A, 0, sizeof(A));
    A.vg = h->vg;
    A.nu = h->vg.nu;
    A.nvw = (A.nu + kGWave - 1) / kGWave;
    A.poff = mx.d_poff;
    A.toff = mx.d_toff;
    A.pnb = mx.d_pnb;
    A.geo = mx.d_geo;
    A.geof = mx.d_geof;
    A.sa = sa;
    int rc;
    if (mode != 0) {  // (the incoming f needs no pass for its traces)
        for (int t = 0; t < 3; ++t) {
            const MixType &T = mx.t[t];
            if (T.elems.empty()) continue;
            const int key_ns[3][4] = {{0, 8, 27, 64}, {0, 6, 18, 40}, {0, 4, 10, 20}};
            if (T.ns != key_ns[t][h->p]) return h->fail(FR_DVM_EINVAL, "mixed-mesh operator size");
            A.elems = T.d_elems;
            A.D = T.d_D;
            A.lift = T.d_lift;
            A.Df = T.d_Df;
            A.liftf = T.d_liftf;
            A.stream = T.d_stream;
            A.streamf = T.d_streamf;
            A.fnode = T.d_fnode;
            A.ffac = T.d_ffac;
            if ((rc = mix_dispatch<Real>(h, mode, A, t, (unsigned)(T.elems.size() * A.nvw)))) return rc;
        }
    }
    const bool moments = (mode == 0 || mode == GMODE_STAGE) && do_moments;
    if (!moments) return FR_DVM_OK;
    // moments of every point: the general-mesh reduction over the velocity axis
    GenArgs G;
    std::memset(&G, 0, sizeof(G));
    G.vg = h->vg;
    G.nu = h->vg.nu;
    G.ncomp = 1;
    G.nut = G.nu;
    G.wax = h->d_wax;
    const Real *src = reinterpret_cast<const Real *>(mode == 0 ? sa.f : sa.fout);
    const unsigned npts = (unsigned)mx.npts;
    if (h->nmom == 5)
        hipLaunchKernelGGL((k_gen_moments<Real, 5>), dim3(gen_moment_grid(npts)), dim3(64 * kMomPts), 0, h->stream, G, src, sa.Q, (int64_t)npts);
    else if (h->nmom == 10)
        hipLaunchKernelGGL((k_gen_moments<Real, 10>), dim3(gen_moment_grid(npts)), dim3(64 * kMomPts), 0, h->stream, G, src, sa.Q, (int64_t)npts);
    else
        return h->fail(FR_DVM_EUNSUPPORTED, "mixed meshes need a monatomic gas");
    return gcheck(h, "moment kernel");
}

}  // namespace

int launch_fr_mixed(fr_dvm *h, int mode, const StageArgs &sa, int do_moments) {
    if (sa.e0 != 0 || sa.ecount != 0) return h->fail(FR_DVM_EINVAL, "element ranges need an axis-aligned box mesh");
    return h->prm.precision == FR_DVM_FP64 ? mix_run<double>(h, mode, sa, do_moments)
                                           : mix_run<float>(h, mode, sa, do_moments);
}

int launch_fr_gen(fr_dvm *h, int mode, const StageArgs &sa, int do_traces, int do_moments) {
    if (sa.e0 != 0 || sa.ecount != 0) return h->fail(FR_DVM_EINVAL, "element ranges need an axis-aligned box mesh");
    GenArgs A;
    std::memset(&A, 0, sizeof(A));
    for (int i = 0; i < kMaxN * kMaxN; ++i) {
        A.od.D[i] = h->ops.D[i];
        A.of.D[i] = (float)h->ops.D[i];
    }
    for (int s = 0; s < 2; ++s)
        for (int m = 0; m < kMaxN; ++m) {
            A.od.lam[s][m] = h->ops.lam[s][m];
            A.of.lam[s][m] = (float)h->ops.lam[s][m];
            A.od.corr[s][m] = h->ops.corr[s][m];
            A.of.corr[s][m] = (float)h->ops.corr[s][m];
        }
    A.vg = h->vg;
    A.nu = h->vg.nu;
    A.ncomp = h->ncomp;
    A.nut = A.nu * A.ncomp;
    A.nvb = (A.nut + kGBlock - 1) / kGBlock;
    A.nvw = (A.nut + kGWave - 1) / kGWave;
    A.gwall = 0.5 * h->delta * h->prm.theta_wall;
    A.gfp = h->d_gfp;
    A.wax = h->d_wax;
    A.wJ = h->d_wq3J;
    A.S = h->d_S;
    A.ijac = h->d_ijac;
    A.nf = h->d_nf;
    A.Sf = h->d_Sf;
    A.ijacf = h->d_ijacf;
    A.nff = h->d_nff;
    A.nm = h->d_nm;
    A.nmf = h->d_nmf;
    A.conn = h->d_conn;
    A.wall = h->d_wall;
    A.rw = h->d_rw;
    A.mw = h->d_mw;
    A.finf = h->d_finf;
    A.sa = sa;
    A.do_traces = do_traces;
    return h->prm.precision == FR_DVM_FP64 ? gen_p<double>(h, mode, A, do_moments)
                                           : gen_p<float>(h, mode, A, do_moments);
}

}  // namespace frdvm
