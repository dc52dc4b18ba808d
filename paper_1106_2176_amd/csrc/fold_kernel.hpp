// fold_kernel.hpp -- the folded M2L of a tile of targets (FP64 form): the
// device core shared by the uniform tree (m2l_fold.hip) and the adaptive one
// (m2l_fold_ad.hip), which differ in where a target's sources lie.
//
// A target box receives L = sum over the 56 orbits of its offsets of
// F_d W, where W, for the rows of each of the eight parities, is the sum of
// the orbit's sources with signs: the rows of parity rho take
// W_rho[c] = sum_m (-1)^(|rho & m| + |kappa_c & m|) M_m[c] over the pair
// masks m of the orbit, kappa_c the parity of coefficient c.  With the
// sources' signs (-1)^|kappa_c & m| put on first, that is a Walsh-Hadamard
// transform in up to three butterfly stages.  A target of class k sees its
// offsets reflected in the axes of k, which is one more sign per
// coefficient, |kappa_c & k|, and one per row, |rho & k|; the operators are
// those of class 0, so that targets of every class and level share them and
// are taken in one list, 16 to a wave.
//
// What bounds it: the FP64 matrix cores.  While an FP64 matrix product runs
// its SIMD issues no vector instruction (8 products and 48 FMAs took the sum
// of their times, in one wave and in two), so the butterflies, the signs and
// the address arithmetic add to it.  Direct products over the 189 offsets
// (v_mfma_f64_16x16x4_f64, 112 rows) took 2.2e6 matrix cycles per 16 targets
// at p = 10; folded they take 0.52e6: 56 products in place of 189, those of
// an orbit with a zero axis halved, and rows padded to 4 within a parity.
// Rows in fours use v_mfma_f64_4x4x4_f64, whose four blocks take the same
// operator rows and four columns each, at the same 32 FLOP per cycle and
// SIMD as the 16 x 16 x 4 instruction (75 and 78 TFLOP/s measured), and
// groups of four quads of a parity the latter, which reads a quarter of the
// operators from LDS.
// Measured, N = 1e6 uniform particles at p = 10 (32768 leaves): 0.99 ms, the
// direct kernel 3.83 ms; at p = 12, 4096 leaves: 0.27 against 1.25 ms; at
// p = 8, 4096 leaves: 0.085 against 0.25 ms.
// Lane layouts (measured on gfx950), 4 x 4 x 4: A lane l holds row l % 4 of
// K index l / 16 (the same for the four blocks), B lane l column l % 16 of
// K index l / 16, the result lane l row l / 16 of column l % 16; 16 x 16 x 4:
// A lane l row l % 16 of K index l / 16, B alike, the result's item i in
// lane l row l / 16 + 4 i.
#pragma once
#include "fold.hpp"
#include "kernels.hpp"

namespace fmm {

// A block is a tile of 16 targets per wave: eight waves (two per SIMD) up to
// p = 12, where the accumulators (one double per row quad), the transformed
// sources and the sources a step ahead fit 256 registers; four waves (one
// per SIMD, 512 registers) above, where they would spill.  The operators of
// a step (8 K positions of an orbit) pass through LDS for all waves.
__host__ __device__ constexpr int fold_waves(int P) { return P <= 12 ? 8 : 4; }
__host__ __device__ constexpr int fold_tile(int P) { return 16 * fold_waves(P); }

// Native vectors: arrays of the HIP vector structs are copied through memory.
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double flip(double v, uint32_t sign) {
    uint64_t u = __builtin_bit_cast(uint64_t, v);
    u ^= (uint64_t)sign << 32;
    return __builtin_bit_cast(double, u);
}

// A lane's sums: rows q of each row quad, four quads in one accumulator of
// the 16 x 16 instruction, and the single ones.
template <int P>
struct FoldAcc {
    static constexpr int RQ = fold_row_quads(P), NBIG = fold_bigs(P, 8);
    f64x4 big[NBIG + 1];
    double one[RQ - 4 * NBIG + 1];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int r = 0; r < NBIG; ++r) big[r] = f64x4{0, 0, 0, 0};
#pragma unroll
        for (int r = 0; r < RQ - 4 * NBIG; ++r) one[r] = 0.0;
    }
    // f(coefficient, value) for the lane's valid rows, signs of class k put on
    template <typename Fn>
    __device__ __forceinline__ void each(int k, int q, const int16_t *__restrict__ rows, Fn &&f) {
        constexpr FoldTab<P> F = fold_tab<P>();
        static_for<0, 8>([&](auto rc) __attribute__((always_inline)) {
            constexpr int rho = decltype(rc)::value, R0 = F.rq0[rho], NR = F.rq0[rho + 1] - R0;
            constexpr int NB = NR / 4, B0 = fold_bigs(P, rho);
            const uint32_t sign = (uint32_t)__popc(rho & k) << 31;
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const int c = rows[4 * (R0 + r) + q];
                const double v = r < 4 * NB ? big[B0 + r / 4][r % 4] : one[R0 + r - 4 * (B0 + NB)];
                if (c >= 0) f(c, flip(v, sign));
            }
        });
    }
};

// block -> tile and its range of steps: whole tiles first (part -1; each XCD
// takes a contiguous run of them), then the parts of the rest
__device__ __forceinline__ void fold_unit(const FoldPlan &pl, int nch, int64_t &tile, int &part, int &sbeg, int &send) {
    const int64_t b = blockIdx.x;
    part = -1;
    sbeg = 0;
    send = nch * kFoldOrbits;
    if (b < pl.nfull) {
        const int64_t per = pl.nfull >> 3;
        tile = b < 8 * per ? (b & 7) * per + (b >> 3) : b;
    } else {
        const int64_t r = b - pl.nfull;
        part = (int)(r / pl.nrest);
        tile = pl.nfull + (r - (int64_t)part * pl.nrest);
        sbeg = pl.cut[part];
        send = pl.cut[part + 1];
    }
}

// pieces (16 bytes) of a step's operators
template <int P>
constexpr int kFoldPieces = fold_row_quads(P) * 16;

// The steps [sbeg, send) (chunk j and orbit o, 56 j + o) of this lane's
// target, of class k, added to acc.  As: 4 kFoldPieces LDS pieces.  Src:
//   chunk(j)        the sources of chunk j from now on (all threads; a
//                   barrier follows)
//   fetch<T>(o, e)  the places of orbit o's sources (e: its components)
//   load<T, HALF>(sw, nx)  the pairs there, their elements swapped if sw
template <int P, typename Src>
__device__ __forceinline__ void fold_run(Src &src, int k, int sbeg, int send, const double *__restrict__ A,
                                         const uint32_t *__restrict__ orbits, const uint16_t *__restrict__ kap,
                                         f64x2 *As, FoldAcc<P> &acc) {
    constexpr FoldTab<P> F = fold_tab<P>();
    constexpr FoldOrbits O = fold_orbits();
    constexpr int NT = 64 * fold_waves(P);
    // a step's operators: NPC 16-byte pieces, fetched by the waves of one of
    // four groups
    constexpr int NPC = kFoldPieces<P>, GT = NT / 4, EPT = (NPC + GT - 1) / GT;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4;
    // The operators are one stream for every block, which each XCD's L2 misses
    // on the way: each of four groups of waves fetches every fourth step's,
    // and stores them a pair of steps ahead, so that a barrier every second
    // step is enough (the two waves of a SIMD then drift apart and one's
    // transform runs beside the other's products).
    const int grp = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
    const int gt = (tid >> 8) * 64 + lane;  // thread within its group
    f64x2 ar[EPT];
    auto load_a = [&](int s) __attribute__((always_inline)) {
        const f64x2 *a = (const f64x2 *)A + (size_t)min(s, send - 1) * NPC;
#pragma unroll
        for (int i = 0; i < EPT; ++i) ar[i] = a[min(gt + GT * i, NPC - 1)];
    };
    auto store_a = [&](int s) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = gt + GT * i;
            if (NPC % GT == 0 || e < NPC) As[(s & 3) * NPC + e] = ar[i];
        }
    };
    int step = sbeg;
    const int pair0 = sbeg & ~1;
    int fetched = pair0 + ((grp - pair0) & 3);  // the step whose operators are in ar
    load_a(fetched);
    if (fetched < pair0 + 2) {
        store_a(fetched);
        load_a(fetched += 4);
    }
    for (int j = sbeg / kFoldOrbits; j * kFoldOrbits < send; ++j) {
        src.chunk(j);  // every wave is past the last chunk
        lds_barrier();
        const int obeg = max(sbeg - j * kFoldOrbits, 0), oend = min(send - j * kFoldOrbits, kFoldOrbits);
        const uint32_t kk = kap[4 * j + q];  // parities of the lane's two positions
        const bool paired = j < F.npair;
        // The orbits [o0, o1) of pair mask T.  HALF = 0: every row with both
        // positions of each pair; HALF = 1 + axis (opposite pairs, zero
        // axis): element 0 is the one that is even along the axis, which the
        // even rows meet, element 1 the odd one.
        auto orbit_loop = [&](auto Tc, auto Hc, int o0, int o1) __attribute__((always_inline)) {
            constexpr int T = decltype(Tc)::value, HALF = decltype(Hc)::value;
            if (o0 >= o1) return;
            const int sw = HALF ? (int)((kk >> (HALF ? HALF - 1 : 0)) & 1) : 0;  // the lane's elements swapped
            uint32_t sg[2][4];  // signs of the elements: class, then each axis
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const uint32_t kp = (kk >> (8 * (e ^ sw))) & 7;
                sg[e][0] = (uint32_t)__popc(kp & (uint32_t)k) << 31;
                sg[e][1] = kp << 31;
                sg[e][2] = (kp >> 1) << 31;
                sg[e][3] = (kp >> 2) << 31;
            }
            double nx[8][2], w[8][2];
            src.template fetch<T>(o0, orbits[o0]);
            src.template load<T, HALF>(sw, nx);
            src.template fetch<T>(min(o0 + 1, o1 - 1), orbits[min(o0 + 1, o1 - 1)]);
            uint32_t en = orbits[min(o0 + 2, o1 - 1)];  // the orbit after the next
            for (int o = o0; o < o1; ++o, ++step) {
                // the next pair of steps' operators into the buffers that
                // every wave finished reading before the last barrier
                if ((!(step & 1) || step == sbeg) && fetched < (step & ~1) + 4) {
                    store_a(fetched);
                    load_a(fetched += 4);
                }
                // transform of the sources
#pragma unroll
                for (int e = 0; e < 2; ++e) {
#pragma unroll
                    for (int mm = 0; mm < 8; ++mm)
                        if ((mm & ~T) == 0)
                            w[mm][e] = flip(nx[mm][e], sg[e][0] ^ (mm & 1 ? sg[e][1] : 0u) ^ (mm & 2 ? sg[e][2] : 0u) ^
                                                           (mm & 4 ? sg[e][3] : 0u));
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        const int bit = 1 << d;
                        if (!(T & bit)) continue;
#pragma unroll
                        for (int mm = 0; mm < 8; ++mm)
                            if ((mm & ~T) == 0 && !(mm & bit)) {
                                const double u = w[mm][e], v = w[mm | bit][e];
                                w[mm][e] = u + v;
                                w[mm | bit][e] = u - v;
                            }
                    }
                }
                src.template load<T, HALF>(sw, nx);
                src.template fetch<T>(min(o + 2, o1 - 1), en);
                en = orbits[min(o + 3, o1 - 1)];
                // products: four row quads of a parity at a time, then the
                // single ones
                const f64x2 *ab = As + (step & 3) * NPC + lane, *as = As + (step & 3) * NPC + (q * 4 + (lane & 3));
                static_for<0, 8>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int rho = decltype(rc)::value, R0 = F.rq0[rho], NR = F.rq0[rho + 1] - R0;
                    constexpr int NB = NR / 4, N1 = NR - 4 * NB, B0 = fold_bigs(P, rho), R1 = R0 + 4 * NB;
                    constexpr int e = HALF ? (rho >> (HALF ? HALF - 1 : 0)) & 1 : 0;
                    const int off = e ? 1 - sw : sw;
                    f64x2 g[NB + 1], a[N1 + 1];
#pragma unroll
                    for (int r = 0; r < NB; ++r) {
                        if (HALF) g[r].x = ((const double *)(ab + 16 * (R0 + 4 * r)))[off];
                        else g[r] = ab[16 * (R0 + 4 * r)];
                    }
#pragma unroll
                    for (int r = 0; r < N1; ++r) {
                        if (HALF) a[r].x = ((const double *)(as + 16 * (R1 + r)))[off];
                        else a[r] = as[16 * (R1 + r)];
                    }
#pragma unroll
                    for (int h = 0; h < (HALF ? 1 : 2); ++h) {
                        const double v = w[rho & T][HALF ? e : h];
#pragma unroll
                        for (int r = 0; r < NB; ++r)
                            acc.big[B0 + r] = __builtin_amdgcn_mfma_f64_16x16x4f64(h ? g[r].y : g[r].x, v, acc.big[B0 + r], 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < N1; ++r)
                            acc.one[R1 - 4 * (B0 + NB) + r] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                h ? a[r].y : a[r].x, v, acc.one[R1 - 4 * (B0 + NB) + r], 0, 0, 0);
                    }
                });
                if (step & 1) lds_barrier();
            }
        };
        static_for<0, 8>([&](auto Tc) __attribute__((always_inline)) {
            constexpr int T = decltype(Tc)::value;
            // without a zero axis, or all of them where pairs are not opposite
            orbit_loop(Tc, std::integral_constant<int, 0>{}, max(obeg, O.t0[T][0]), min(oend, O.t0[T][paired ? 1 : 4]));
            if (paired)
                static_for<1, 4>([&](auto Hc) __attribute__((always_inline)) {
                    constexpr int H = decltype(Hc)::value;
                    if constexpr (O.t0[T][H + 1] > O.t0[T][H])
                        orbit_loop(Tc, Hc, max(obeg, O.t0[T][H]), min(oend, O.t0[T][H + 1]));
                });
        });
    }
}

}  // namespace fmm
