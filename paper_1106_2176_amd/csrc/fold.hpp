// fold.hpp -- the M2L offsets and coefficients grouped by reflections (FP64
// form; device and host).
//
// Every coefficient of the real basis is even or odd under each of the
// reflections x -> -x, y -> -y, z -> -z (fold_parity: one bit per axis, 1 =
// odd), and the M2L matrix of a reflected offset is the matrix of the offset
// with signs on both sides, F_{sd}[r][c] = chi_r(s) F_d[r][c] chi_c(s),
// chi_c(s) = -1 when an odd number of the axes s flips are odd in c.  The
// sources of a target at the offsets {s d} of one orbit therefore share the
// matrix entries of one offset,
//     sum_s F_{sd}[r][c] M_s[c] = F_d[r][c] (sum_s chi_r(s) chi_c(s) M_s[c]),
// and the sum in brackets, for the eight parities of r, is a Walsh-Hadamard
// transform of the orbit's (signed) sources: one product per matrix entry
// serves up to eight sources.
//
// Orbits: seen from class 0 (the target's low octant of its parent) an
// offset's component per axis is one of -2 .. 3: 0 and 3 alone, +-1 and +-2
// in pairs, hence 4^3 - 2^3 = 56 orbits (a, b, c), components 0 .. 3, with a
// mask T of the paired axes; the source of pair mask m (a subset of T) lies
// at (a, b, c) with the axes of m negated.  A target of class k sees the
// same picture reflected in the axes of k.  An entry F_d[r][c] vanishes
// where d is zero along an axis in which r and c differ in parity (mask z).
//
// Coefficients are reordered (K order) in pairs of opposite parity in all
// three axes where possible.  Along a zero axis a row then meets exactly one
// of a pair's two coefficients, so that an orbit with a zero axis takes half
// the matrix products on those chunks.  Rows are grouped by parity in quads
// padded with zero rows.
#pragma once
#include "common.hpp"

namespace fmm {

constexpr int kFoldOrbits = 56;

__host__ __device__ constexpr int fold_parity(int c) {
    int n = 0;
    while ((n + 1) * (n + 1) <= c) ++n;
    const int r = c - n * n, m = (r + 1) / 2, sine = r > 0 && r % 2 == 0;
    return ((m + sine) & 1) | (sine << 1) | (((n + m) & 1) << 2);
}

// The orbits, sorted by pair mask T and, within it, by the first zero axis
// (none, x, y, z).
struct FoldOrbit {
    int8_t a[3], T, za;         // components, pair mask, 0 or 1 + the first zero axis
};
struct FoldOrbits {
    FoldOrbit o[kFoldOrbits];
    int t0[8][5];               // first orbit of each (T, za); [T][4]: the end
    int src0[kFoldOrbits + 1];  // first source of each orbit, 189 in all
};
__host__ __device__ constexpr FoldOrbits fold_orbits() {
    FoldOrbits f{};
    int n = 0, s = 0;
    for (int T = 0; T < 8; ++T) {
        for (int zw = 0; zw < 4; ++zw) {
            f.t0[T][zw] = n;
            for (int i = 0; i < 64; ++i) {
                const int a[3] = {i & 3, (i >> 2) & 3, i >> 4};
                int t = 0, za = 0, far = 0;
                for (int d = 2; d >= 0; --d) {
                    if (a[d] == 1 || a[d] == 2) t |= 1 << d;
                    if (a[d] == 0) za = 1 + d;
                    if (a[d] >= 2) far = 1;
                }
                if (t != T || za != zw || !far) continue;
                for (int d = 0; d < 3; ++d) f.o[n].a[d] = (int8_t)a[d];
                f.o[n].T = (int8_t)T;
                f.o[n].za = (int8_t)za;
                f.src0[n++] = s;
                s += 1 << ((T & 1) + ((T >> 1) & 1) + (T >> 2));
            }
        }
        f.t0[T][4] = n;
    }
    f.src0[n] = s;
    return f;
}
static_assert(fold_orbits().t0[7][4] == kFoldOrbits, "orbits");
static_assert(fold_orbits().src0[kFoldOrbits] == kOffsetsPerClass, "sources");

// position of the source of pair mask m among those of pair mask T's subsets
__host__ __device__ constexpr int fold_rank(int T, int m) {
    int r = 0, w = 1;
    for (int d = 0; d < 3; ++d)
        if ((T >> d) & 1) {
            if ((m >> d) & 1) r += w;
            w *= 2;
        }
    return r;
}

// The K order and the row quads of order P.  Position i of the K order lies
// in chunk i / 8; positions 2 i and 2 i + 1 are a pair.
template <int P>
struct FoldTab {
    static constexpr int P2 = P * P, S = coef_stride(P), NCH = S / 8;
    int16_t kperm[S];   // coefficient of each position, -1 past p^2
    uint8_t kap[S];     // its parity
    int npair;          // first chunks, of opposite pairs only
    int rq0[9];         // first row quad of each parity, rq0[8] = all
};
template <int P>
__host__ __device__ constexpr FoldTab<P> fold_tab() {
    using F = FoldTab<P>;
    FoldTab<P> f{};
    int16_t list[8][F::P2 + 1] = {};
    int cnt[8] = {}, used[8] = {};
    for (int c = 0; c < F::P2; ++c) {
        const int k = fold_parity(c);
        list[k][cnt[k]++] = (int16_t)c;
    }
    int n = 0;
    for (int k = 0; k < 4; ++k)
        while (used[k] < cnt[k] && used[7 - k] < cnt[7 - k]) {
            f.kperm[n++] = list[k][used[k]++];
            f.kperm[n++] = list[7 - k][used[7 - k]++];
        }
    f.npair = n / 8;
    for (int k = 0; k < 8; ++k)
        while (used[k] < cnt[k]) f.kperm[n++] = list[k][used[k]++];
    for (; n < F::S; ++n) f.kperm[n] = -1;
    for (int i = 0; i < F::S; ++i) f.kap[i] = f.kperm[i] < 0 ? 0 : (uint8_t)fold_parity(f.kperm[i]);
    for (int k = 0; k < 8; ++k) f.rq0[k + 1] = f.rq0[k] + (cnt[k] + 3) / 4;
    return f;
}
// row quads of order P
__host__ __device__ constexpr int fold_row_quads(int P) {
    int cnt[8] = {};
    for (int c = 0; c < P * P; ++c) ++cnt[fold_parity(c)];
    int n = 0;
    for (int k = 0; k < 8; ++k) n += (cnt[k] + 3) / 4;
    return n;
}
// Groups of four row quads (one 16 x 16 x 4 matrix product) of the parities
// below rho; the quads left over in a parity take products of their own.
__host__ __device__ constexpr int fold_bigs(int P, int rho) {
    int cnt[8] = {};
    for (int c = 0; c < P * P; ++c) ++cnt[fold_parity(c)];
    int n = 0;
    for (int k = 0; k < rho; ++k) n += (cnt[k] + 3) / 4 / 4;
    return n;
}
// Doubles of the operator table: per chunk and orbit, the four K pairs q of
// the rows: [q][row][2] for each group of four quads, then each single one.
__host__ __device__ constexpr size_t fold_table_size(int P) {
    return (size_t)kFoldOrbits * (coef_stride(P) / 8) * fold_row_quads(P) * 32;
}

}  // namespace fmm
