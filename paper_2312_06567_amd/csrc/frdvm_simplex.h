// Structure of the nodal operators on the simplex point sets (warp & blend
// points for p <= 3), shared by the set-up that fills the operator stream of
// a mixed mesh's prisms and tetrahedra and by the kernel that reads it.
//
// The derivatives of a degree-p polynomial lie in P_(p-1), so they are formed
// at NM = dim P_(p-1) of the NP points (`sub`, chosen for the smallest
// interpolation constant, 2.4 at p = 3) and interpolated to the others; and
// the points lie on lines of the barycentric lattice, so most entries of the
// derivative rows and of the interpolation vanish.  The masks below mark the
// entries that do not: bit j of d[a][m], entry j of the derivative along xi_a
// at point sub[m]; bit m of e[q], the weight of point sub[m] at the q-th
// other point.  On the tetrahedron at p = 3 this is 297 multiply-adds per
// velocity instead of the 1260 of three dense 20 x 20 products.  Set-up checks
// every mask and the interpolation against the dense operators.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

namespace frdvm {

template <int NP_, int NM_, int DIM_>
struct SimplexTable {
    int sub[NM_];
    uint32_t d[DIM_][NM_];
    uint32_t e[NP_ - NM_];
};

template <int DIM, int P>
struct Simplex {
    static constexpr int NP = DIM == 3 ? (P + 1) * (P + 2) * (P + 3) / 6 : (P + 1) * (P + 2) / 2;
    static constexpr int NM = DIM == 3 ? P * (P + 1) * (P + 2) / 6 : P * (P + 1) / 2;
    using Table = SimplexTable<NP, NM, DIM>;
    __host__ __device__ static constexpr Table table() {
        if constexpr (DIM == 2 && P == 1) {
            return {{0}, {{0x3}, {0x5}}, {0x1, 0x1}};
        } else if constexpr (DIM == 2 && P == 2) {
            return {{0, 2, 5}, {{0x7, 0x7, 0x1d}, {0x29, 0x33, 0x29}}, {0x3, 0x5, 0x6}};
        } else if constexpr (DIM == 2 && P == 3) {
            return {{0, 1, 3, 6, 7, 9},
                    {{0xf, 0xd, 0xf, 0x3ff, 0x3ff, 0x1d9}, {0x291, 0x3ff, 0x347, 0x3ff, 0x211, 0x291}},
                    {0x7, 0x31, 0x3f, 0x2c}};
        } else if constexpr (DIM == 3 && P == 1) {
            return {{0}, {{0x3}, {0x5}, {0x9}}, {0x1, 0x1, 0x1}};
        } else if constexpr (DIM == 3 && P == 2) {
            return {{0, 2, 5, 9},
                    {{0x7, 0x7, 0x1d, 0xc5}, {0x29, 0x33, 0x29, 0x161}, {0x241, 0x283, 0x309, 0x241}},
                    {0x3, 0x5, 0x6, 0x9, 0xa, 0xc}};
        } else {
            static_assert(DIM == 3 && P == 3, "orders 1..3");
            return {{0, 1, 3, 4, 6, 9, 12, 15, 16, 19},
                    {{0xf, 0xd, 0xf, 0x3ff, 0x3ff, 0x1d9, 0xb1c0f, 0x375d9, 0xb1c0f, 0x31409},
                     {0x291, 0x3ff, 0x347, 0x281, 0x3ff, 0x291, 0x5cf47, 0xda691, 0xda691, 0x58601},
                     {0x90401, 0xb1c0f, 0xa1007, 0xda691, 0xed0b7, 0xc8091, 0xb1c0f, 0xda691, 0x80401, 0x90401}},
                    {0x7, 0x3f, 0x29, 0x34, 0x301, 0x347, 0x3a9, 0x2f4, 0x244, 0x2a0}};
        }
    }
    // the points outside `sub`, in order
    struct Rest {
        int i[NP - NM];
    };
    __host__ __device__ static constexpr Rest rest() {
        constexpr Table t = table();
        Rest r{};
        int c = 0;
        for (int i = 0; i < NP; ++i) {
            bool in = false;
            for (int m = 0; m < NM; ++m) in = in || t.sub[m] == i;
            if (!in) r.i[c++] = i;
        }
        return r;
    }
    // Solution points on each face (edge of the triangle), ascending, in the
    // face order of the ABI: tetrahedron {0,1,2} {0,1,3} {1,2,3} {0,2,3}, the
    // triangle's edges {0,1} {1,2} {2,0}; points are indexed by barycentric
    // (i, j[, k]) with i fastest.
    static constexpr int NFACE = DIM == 3 ? 4 : 3;
    static constexpr int NF = DIM == 3 ? (P + 1) * (P + 2) / 2 : P + 1;
    struct Faces {
        int n[NFACE][NF];
    };
    __host__ __device__ static constexpr Faces faces() {
        Faces r{};
        int c[NFACE] = {}, s = 0;
        for (int k = 0; k <= (DIM == 3 ? P : 0); ++k)
            for (int j = 0; j + k <= P; ++j)
                for (int i = 0; i + j + k <= P; ++i, ++s) {
                    if (DIM == 3) {
                        const bool on[4] = {k == 0, j == 0, i + j + k == P, i == 0};
                        for (int f = 0; f < 4; ++f)
                            if (on[f]) r.n[f][c[f]++] = s;
                    } else {
                        const bool on[3] = {j == 0, i + j == P, i == 0};
                        for (int f = 0; f < 3; ++f)
                            if (on[f]) r.n[f][c[f]++] = s;
                    }
                }
        return r;
    }
    // Entries of the derivative and interpolation part of the stream.
    __host__ __device__ static constexpr int volume_entries() {
        constexpr Table t = table();
        int c = 0;
        for (int m = 0; m < NM; ++m)
            for (int a = 0; a < DIM; ++a)
                for (int j = 0; j < NP; ++j) c += (t.d[a][m] >> j) & 1;
        for (int q = 0; q < NP - NM; ++q)
            for (int m = 0; m < NM; ++m) c += (t.e[q] >> m) & 1;
        return c;
    }
};

// Operator stream of one element type, in the order the kernel reads it:
//   per sub point m, direction a: the marked derivative entries;
//   per other point: the marked interpolation weights;
//   tetrahedron: lift[f][t][i], a unit jump at face point t onto point i;
//   prism (triangle x line, PL = p + 1 layers): the axial derivative [PL][PL],
//   the lifting of a bottom and of a top face point onto its column [2][PL],
//   and of edge point e of side f on a layer onto that layer [3][PL][NT].
template <int P>
constexpr int tet_stream() {
    using S = Simplex<3, P>;
    return S::volume_entries() + S::NFACE * S::NF * S::NP;
}
template <int P>
constexpr int prism_stream() {
    using S = Simplex<2, P>;
    return S::volume_entries() + (P + 1) * (P + 1) + 2 * (P + 1) + 3 * (P + 1) * S::NP;
}

}  // namespace frdvm
