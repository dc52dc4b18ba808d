// m2l_fold.hip -- the FP64 form's multipole-to-local translation on the
// matrix cores, its offsets folded by reflections (fold.hpp).
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
#include "fold.hpp"
#include "kernels.hpp"

namespace fmm {

namespace {

// A block is a tile of 16 targets per wave: eight waves (two per SIMD) up to
// p = 12, where the accumulators (one double per row quad), the transformed
// sources and the sources a chunk ahead fit 256 registers; four waves (one
// per SIMD, 512 registers) above, where they would spill.  The operators of
// a chunk (8 K positions) pass through LDS, double buffered, for all waves.
__host__ __device__ constexpr int fold_waves(int P) { return P <= 12 ? 8 : 4; }
__host__ __device__ constexpr int fold_tile(int P) { return 16 * fold_waves(P); }

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double flip(double v, uint32_t sign) {
    uint64_t u = __builtin_bit_cast(uint64_t, v);
    u ^= (uint64_t)sign << 32;
    return __builtin_bit_cast(double, u);
}

// The sources of a tile: the children of its parents (4 x 2 x 2 of them, 2 x
// 2 x 2 in a four-wave tile) and of their neighbours, 12 x 8 x 8 boxes.  The
// 8 K positions of a chunk of all of them are held in LDS as four planes of
// 16-byte pairs, box (x, y, z) at x + 12 y + 104 z: the 16 targets of a wave
// are 4 x 2 x 2 boxes, whose places differ modulo 16 (16 pairs are the 64
// banks).  From global memory each source would be read by its up to 189
// targets (5.2 GB at p = 10, 32768 boxes: the kernel took 1.45 ms).
constexpr int kRegY = 12, kRegZ = 104, kRegPlane = 8 * kRegZ;

}  // namespace

// Tile of the flat list: its level's index, the level, its first target
// (Morton) and its column's target
__device__ __forceinline__ void fold_place_of(const FoldPlan &pl, int64_t tile, int &li, int &l, int64_t &m0) {
    li = 0;
#pragma unroll
    for (int j = 1; j < kFoldMaxLev; ++j)
        if (j < pl.nlev && tile >= pl.tile0[j]) li = j;
    l = pick(pl.level, li);
    m0 = (tile - pick(pl.tile0, li)) * pl.tile;
}

// Multipoles of every level into its padded grid [(2^l + 6)^3][S], a halo of
// 3 zero boxes, in K order: a block per row of boxes, two positions a thread.
__global__ __launch_bounds__(256) void k_fold_pack(int P, PackPlan pl, const int16_t *__restrict__ kperm) {
    const int64_t b = blockIdx.x;
    int li = 0;
#pragma unroll
    for (int j = 1; j < kMaxPackLev; ++j)
        if (j < pl.nlev && b >= pl.row0[j]) li = j;
    const int n = 1 << pick(pl.level, li), g = n + 6, S2 = coef_stride(P) / 2;
    const double *__restrict__ in = (const double *)pick(pl.in, li);
    f64x2 *__restrict__ out = (f64x2 *)pick(pl.out, li);
    const int row = (int)(b - pick(pl.row0, li)), y = row % g - 3, z = row / g - 3;
    const bool yz = y >= 0 && z >= 0 && y < n && z < n;
    for (int e = threadIdx.x; e < g * S2; e += 256) {
        const int bx = e / S2, c = 2 * (e - bx * S2), x = bx - 3;
        f64x2 v = {0.0, 0.0};
        if (yz && x >= 0 && x < n) {
            const double *src = in + ((size_t)x + (size_t)n * ((size_t)y + (size_t)n * z)) * (2 * S2);
            const int c0 = kperm[c], c1 = kperm[c + 1];
            if (c0 >= 0) v.x = src[c0];
            if (c1 >= 0) v.y = src[c1];
        }
        out[(size_t)row * g * S2 + e] = v;
    }
}

template <int P>
__global__ __launch_bounds__(64 * fold_waves(P))
__attribute__((amdgpu_waves_per_eu(fold_waves(P) / 4, fold_waves(P) / 4))) void k_m2l_fold(
    FoldPlan pl, const double *__restrict__ A, const uint32_t *__restrict__ orbits, const uint16_t *__restrict__ kap, const int16_t *__restrict__ rows,
    double *__restrict__ partial) {
    constexpr FoldTab<P> F = fold_tab<P>();
    constexpr FoldOrbits O = fold_orbits();
    constexpr int P2 = P * P, S = coef_stride(P), RQ = fold_row_quads(P), NCH = FoldTab<P>::NCH;
    constexpr int NT = 64 * fold_waves(P);
    // a step's operators: NPC 16-byte pieces, fetched by the waves of one of
    // four groups
    constexpr int NPC = RQ * 16, GT = NT / 4, EPT = (NPC + GT - 1) / GT;
    constexpr int RX = fold_waves(P) == 8 ? 12 : 8;          // region boxes along x
    constexpr int REG = RX * 8 * 8 * 4 / NT;                 // region pieces per thread
    static_assert(RX * 8 * 8 * 4 % NT == 0, "region pieces");
    __shared__ __align__(16) f64x2 As[4 * NPC];
    __shared__ __align__(16) f64x2 reg[4 * kRegPlane];

    // block -> tile and its range of steps (chunk, orbit): whole tiles first,
    // each XCD a contiguous run of them, then the parts of the rest
    const int64_t b = blockIdx.x;
    int64_t tile;
    int part = -1, sbeg = 0, send = NCH * kFoldOrbits;
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
    int li, l;
    int64_t m0;
    fold_place_of(pl, tile, li, l, m0);
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, slot = (tid >> 6) * 16 + (lane & 15);
    const int n = 1 << l, G = n + 6;
    const int64_t m = m0 + slot;
    const bool valid = m < ((int64_t)1 << (3 * l));
    const int k = slot & 7;
    // tile origin, and this lane's place in the region
    const int ox = (int)compact3((uint32_t)m0), oy = (int)compact3((uint32_t)m0 >> 1), oz = (int)compact3((uint32_t)m0 >> 2);
    const int x = (int)compact3((uint32_t)slot), y = (int)compact3((uint32_t)slot >> 1), z = (int)compact3((uint32_t)slot >> 2);
    const int here = (x + 2) + kRegY * (y + 2) + kRegZ * (z + 2) + q * kRegPlane;
    const int st[3] = {k & 1 ? -1 : 1, k & 2 ? -kRegY : kRegY, k & 4 ? -kRegZ : kRegZ};
    // region pieces of this thread: box e / 4, pair e % 4; boxes past the
    // grid's halo (a tile wider than its level) read the halo
    const double *__restrict__ B = pick(pl.B, li);
    int64_t gsrc[REG];
    int gdst[REG];
#pragma unroll
    for (int i = 0; i < REG; ++i) {
        const int e = tid + NT * i, bx = e >> 2, rx = bx % RX, ry = bx / RX % 8, rz = bx / (RX * 8);
        gsrc[i] = ((int64_t)min(ox + rx + 1, G - 1) + G * ((int64_t)min(oy + ry + 1, G - 1) +
                                                          (int64_t)G * min(oz + rz + 1, G - 1))) * S + 2 * (e & 3);
        gdst[i] = (e & 3) * kRegPlane + rx + kRegY * ry + kRegZ * rz;
    }
    // sums of the lane's rows q of each row quad: of four quads in one
    // accumulator of the 16 x 16 instruction, and of the single ones
    constexpr int NBIG = fold_bigs(P, 8);
    f64x4 big[NBIG + 1];
    double one[RQ - 4 * NBIG + 1];
#pragma unroll
    for (int r = 0; r < NBIG; ++r) big[r] = f64x4{0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < RQ - 4 * NBIG; ++r) one[r] = 0.0;

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
        // the chunk's region (every wave is past the last one's)
        {
            f64x2 v[REG];
#pragma unroll
            for (int i = 0; i < REG; ++i) v[i] = *(const f64x2 *)(B + gsrc[i] + 8 * j);
#pragma unroll
            for (int i = 0; i < REG; ++i) reg[gdst[i]] = v[i];
        }
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
            const double *const r0 = (const double *)(reg + here) + sw, *const r1 = (const double *)(reg + here) + (1 - sw);
            double nx[8][2], w[8][2];
            auto load_b = [&](uint32_t e) __attribute__((always_inline)) {
                const int d0 = __mul24((int)(e & 3), st[0]), d1 = __mul24((int)((e >> 2) & 3), st[1]),
                          d2 = __mul24((int)((e >> 4) & 3), st[2]);
#pragma unroll
                for (int mm = 0; mm < 8; ++mm)
                    if ((mm & ~T) == 0) {
                        const int at = (mm & 1 ? -d0 : d0) + (mm & 2 ? -d1 : d1) + (mm & 4 ? -d2 : d2);
                        if (HALF) {
                            nx[mm][0] = r0[2 * at];
                            nx[mm][1] = r1[2 * at];
                        } else {
                            const f64x2 v = reg[here + at];
                            nx[mm][0] = v.x;
                            nx[mm][1] = v.y;
                        }
                    }
            };
            load_b(orbits[o0]);
            uint32_t en = orbits[min(o0 + 1, o1 - 1)];  // the next orbit
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
                load_b(en);
                en = orbits[min(o + 2, o1 - 1)];
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
                            big[B0 + r] = __builtin_amdgcn_mfma_f64_16x16x4f64(h ? g[r].y : g[r].x, v, big[B0 + r], 0, 0, 0);
#pragma unroll
                        for (int r = 0; r < N1; ++r)
                            one[R1 - 4 * (B0 + NB) + r] = __builtin_amdgcn_mfma_f64_4x4x4f64(
                                h ? a[r].y : a[r].x, v, one[R1 - 4 * (B0 + NB) + r], 0, 0, 0);
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
    double *dst = part < 0
                      ? pick(pl.L, li) + ((int64_t)(ox + x) + (int64_t)n * ((oy + y) + (int64_t)n * (oz + z))) * S
                      : partial + (((int64_t)part * pl.nrest + (tile - pl.nfull)) * (NT / 4) + slot) * P2;
    static_for<0, 8>([&](auto rc) __attribute__((always_inline)) {
        constexpr int rho = decltype(rc)::value, R0 = F.rq0[rho], NR = F.rq0[rho + 1] - R0;
        constexpr int NB = NR / 4, B0 = fold_bigs(P, rho);
        const uint32_t sign = (uint32_t)__popc(rho & k) << 31;
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int c = rows[4 * (R0 + r) + q];
            const double v = r < 4 * NB ? big[B0 + r / 4][r % 4] : one[R0 + r - 4 * (B0 + NB)];
            if (valid && c >= 0) dst[c] = flip(v, sign);
        }
    });
}

// Sum of the parts of the rest tiles, in part order; one thread per target
// and coefficient.
__global__ __launch_bounds__(256) void k_m2l_fold_sum(int P, FoldPlan pl, const double *__restrict__ partial) {
    const int P2 = P * P, S = coef_stride(P);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t step = (int64_t)pl.nrest * pl.tile * P2;
    if (i >= step) return;
    const int64_t t = i / P2, rt = t / pl.tile;
    int li, l;
    int64_t m;
    fold_place_of(pl, pl.nfull + rt, li, l, m);
    m += t - rt * pl.tile;
    if (m >= (int64_t)1 << (3 * l)) return;
    double v = 0.0;
    for (int s = 0; s < pl.nsplit; ++s) v += partial[s * step + i];
    const int64_t n = (int64_t)1 << l;
    const int64_t x = compact3((uint32_t)m), y = compact3((uint32_t)m >> 1), z = compact3((uint32_t)m >> 2);
    pick(pl.L, li)[(x + n * (y + n * z)) * S + (i - t * P2)] = v;
}

// ------------------------------------------------------------ host side
// Tiles to compute units: as many whole rounds of one tile per unit as there
// are, then the rest in s parts of their steps, s the count that takes the
// least time among those whose FP64 partial sums fit `cap` bytes.
static FoldPlan fold_plan(int P, int L, int ncu, size_t cap) {
    constexpr FoldOrbits O = fold_orbits();
    FoldPlan pl{};
    pl.tile = fold_tile(P);
    pl.nlev = L - 1;
    int64_t tiles = 0;
    for (int i = 0; i < pl.nlev; ++i) {
        pl.level[i] = L - i;
        pl.tile0[i] = tiles;
        tiles += (((int64_t)1 << (3 * (L - i))) + pl.tile - 1) / pl.tile;
    }
    pl.nfull = tiles / ncu * ncu;
    pl.nrest = (int)(tiles - pl.nfull);
    pl.nsplit = 1;
    // costs of an orbit's step: a zero axis halves its products
    int cost[kFoldOrbits + 1] = {};
    for (int o = 0; o < kFoldOrbits; ++o) cost[o + 1] = cost[o] + (O.o[o].za ? 1 : 2);
    if (pl.nrest) {
        const size_t unit = sizeof(double) * (size_t)pl.nrest * pl.tile * P * P;
        double best = 1e300;
        for (int s = 1; s <= kFoldParts; ++s) {
            if (s > 1 && s * unit > cap) break;
            const double rounds = (double)(((int64_t)pl.nrest * s + ncu - 1) / ncu);
            const double t = rounds * (1.0 / s + 0.01) + (s > 1 ? 0.01 : 0.0);
            if (t < best - 1e-9) {
                best = t;
                pl.nsplit = s;
            }
        }
        if (pl.nsplit == 1) {  // nothing to add up: whole tiles
            pl.nfull = tiles;
            pl.nrest = 0;
        }
    }
    const int nch = coef_stride(P) / 8;
    const int64_t total = (int64_t)nch * cost[kFoldOrbits];
    int at = 0;
    for (int s = 0; s <= pl.nsplit; ++s) {
        while (at < nch * kFoldOrbits &&
               ((int64_t)(at / kFoldOrbits) * cost[kFoldOrbits] + cost[at % kFoldOrbits]) * pl.nsplit < total * s)
            ++at;
        pl.cut[s] = (uint16_t)at;
    }
    return pl;
}

static size_t plan_partial_bytes(const FoldPlan &pl, int P) {
    return pl.nrest ? sizeof(double) * (size_t)pl.nsplit * pl.nrest * pl.tile * P * P : 0;
}

size_t m2l_fold_partial_bytes(int P, int L, int ncu, size_t cap) {
    return L < 2 ? 0 : plan_partial_bytes(fold_plan(P, L, ncu, cap), P);
}

template <int P>
static void fold_fill(FoldHost &h) {
    constexpr FoldTab<P> F = fold_tab<P>();
    constexpr int RQ = fold_row_quads(P);
    h.kperm.assign(F.kperm, F.kperm + FoldTab<P>::S);
    h.kap.clear();
    for (int i = 0; i < FoldTab<P>::S; i += 2) h.kap.push_back((uint16_t)(F.kap[i] | F.kap[i + 1] << 8));
    h.rows.assign(4 * RQ, -1);
    int at[8];
    for (int k = 0; k < 8; ++k) at[k] = 4 * F.rq0[k];
    for (int c = 0; c < P * P; ++c) h.rows[at[fold_parity(c)]++] = (int16_t)c;
    // place of each row position in a step's operators, and its K stride
    h.row_place.clear();
    for (int rp = 0; rp < 4 * RQ; ++rp) {
        int k = 0;
        while (rp >= 4 * F.rq0[k + 1]) ++k;
        const int i = rp - 4 * F.rq0[k], nb = (F.rq0[k + 1] - F.rq0[k]) / 4;
        h.row_place.push_back(i < 16 * nb ? int2{32 * F.rq0[k] + 128 * (i / 16) + 2 * (i % 16), 32}
                                          : int2{32 * (rp / 4) + 2 * (rp % 4), 8});
    }
}

void fold_host(int P, FoldHost &h) {
    constexpr FoldOrbits O = fold_orbits();
    switch (P) {
#define CASE(PP) \
    case PP: fold_fill<PP>(h); break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
        CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14) CASE(15) CASE(16)
#undef CASE
    }
    h.orbits.clear();
    for (int o = 0; o < kFoldOrbits; ++o)
        h.orbits.push_back(O.o[o].a[0] | O.o[o].a[1] << 2 | O.o[o].a[2] << 4);
    h.table.assign(fold_table_size(P), 0.0);
}

size_t fold_place(int P, const FoldHost &h, int o, int rowpos, int kpos) {
    const int2 r = h.row_place[rowpos];
    return ((size_t)(kpos / 8) * kFoldOrbits + o) * fold_row_quads(P) * 32 + r.x + (size_t)((kpos % 8) / 2) * r.y +
           (kpos & 1);
}

hipError_t launch_fold_pack(int P, const PackPlan &pl, const FoldDev &fd, hipStream_t st) {
    if (pl.nlev <= 0) return hipSuccess;
    k_fold_pack<<<(unsigned)pl.row0[pl.nlev], 256, 0, st>>>(P, pl, fd.kperm);
    return hipGetLastError();
}

hipError_t launch_m2l_fold(int P, int L, void *const *B, void *const *Lc, const double *A, const FoldDev &fd,
                           double *partial, size_t partial_bytes, int ncu, size_t cap, hipStream_t st) {
    if (L < 2) return hipSuccess;
    FoldPlan pl = fold_plan(P, L, ncu, cap);
    if (plan_partial_bytes(pl, P) > 0 && (!partial || partial_bytes < plan_partial_bytes(pl, P)))
        return hipErrorInvalidValue;
    for (int i = 0; i < pl.nlev; ++i) {
        pl.B[i] = (const double *)B[pl.level[i]];
        pl.L[i] = (double *)Lc[pl.level[i]];
    }
    const unsigned nb = (unsigned)(pl.nfull + (int64_t)pl.nrest * pl.nsplit);
    switch (P) {
#define CASE(PP) \
    case PP: k_m2l_fold<PP><<<nb, 64 * fold_waves(PP), 0, st>>>(pl, A, fd.orbits, fd.kap, fd.rows, partial); break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
        CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14) CASE(15) CASE(16)
#undef CASE
        default: return hipErrorInvalidValue;
    }
    if (pl.nrest)
        k_m2l_fold_sum<<<(unsigned)(((int64_t)pl.nrest * pl.tile * P * P + 255) / 256), 256, 0, st>>>(P, pl, partial);
    return hipGetLastError();
}

}  // namespace fmm
