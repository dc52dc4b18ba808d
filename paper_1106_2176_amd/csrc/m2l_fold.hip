// m2l_fold.hip -- the FP64 form's multipole-to-local translation on the
// matrix cores, its offsets folded by reflections (fold.hpp, fold_kernel.hpp):
// the uniform tree's kernels and the tables' host side.
#include "fold_kernel.hpp"

namespace fmm {

// The sources of a tile: the children of its parents (4 x 2 x 2 of them, 2 x
// 2 x 2 in a four-wave tile) and of their neighbours, 12 x 8 x 8 boxes.  The
// 8 K positions of a chunk of all of them are held in LDS as four planes of
// 16-byte pairs, box (x, y, z) at x + 12 y + 104 z: the 16 targets of a wave
// are 4 x 2 x 2 boxes, whose places differ modulo 16 (16 pairs are the 64
// banks).  From global memory each source would be read by its up to 189
// targets (5.2 GB at p = 10, 32768 boxes: the kernel took 1.45 ms).
constexpr int kRegY = 12, kRegZ = 104, kRegPlane = 8 * kRegZ;

template <int P>
struct GridSource {
    static constexpr int S = coef_stride(P), NT = 64 * fold_waves(P);
    static constexpr int RX = fold_waves(P) == 8 ? 12 : 8;  // region boxes along x
    static constexpr int REG = RX * 8 * 8 * 4 / NT;         // region pieces per thread
    static_assert(RX * 8 * 8 * 4 % NT == 0, "region pieces");
    const double *__restrict__ B;  // the level's padded grid
    int G, ox, oy, oz;             // its pitch, the tile's origin
    f64x2 *reg;
    int here, st[3];               // the lane's target in the region, strides signed by its class
    int d[3];
    __device__ __forceinline__ void chunk(int j) {
        // boxes past the grid's halo (a tile wider than its level) read the halo
        f64x2 v[REG];
#pragma unroll
        for (int i = 0; i < REG; ++i) {
            const int e = threadIdx.x + NT * i, bx = e >> 2, rx = bx % RX, ry = bx / RX % 8, rz = bx / (RX * 8);
            const int64_t at = (int64_t)min(ox + rx + 1, G - 1) +
                               G * ((int64_t)min(oy + ry + 1, G - 1) + (int64_t)G * min(oz + rz + 1, G - 1));
            v[i] = *(const f64x2 *)(B + at * S + 8 * j + 2 * (e & 3));
        }
#pragma unroll
        for (int i = 0; i < REG; ++i) {
            const int e = threadIdx.x + NT * i, bx = e >> 2, rx = bx % RX, ry = bx / RX % 8, rz = bx / (RX * 8);
            reg[(e & 3) * kRegPlane + rx + kRegY * ry + kRegZ * rz] = v[i];
        }
    }
    template <int T>
    __device__ __forceinline__ void fetch(int, uint32_t e) {
        d[0] = __mul24((int)(e & 3), st[0]);
        d[1] = __mul24((int)((e >> 2) & 3), st[1]);
        d[2] = __mul24((int)((e >> 4) & 3), st[2]);
    }
    template <int T, int HALF>
    __device__ __forceinline__ void load(int sw, double (&nx)[8][2]) {
#pragma unroll
        for (int m = 0; m < 8; ++m)
            if ((m & ~T) == 0) {
                const int at = here + (m & 1 ? -d[0] : d[0]) + (m & 2 ? -d[1] : d[1]) + (m & 4 ? -d[2] : d[2]);
                if (HALF) {
                    nx[m][0] = ((const double *)(reg + at))[sw];
                    nx[m][1] = ((const double *)(reg + at))[1 - sw];
                } else {
                    const f64x2 v = reg[at];
                    nx[m][0] = v.x;
                    nx[m][1] = v.y;
                }
            }
    }
};

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
    FoldPlan pl, const double *__restrict__ A, const uint32_t *__restrict__ orbits, const uint16_t *__restrict__ kap,
    const int16_t *__restrict__ rows, double *__restrict__ partial) {
    constexpr int P2 = P * P, S = coef_stride(P);
    __shared__ __align__(16) f64x2 As[4 * kFoldPieces<P>];
    __shared__ __align__(16) f64x2 reg[4 * kRegPlane];
    int64_t tile;
    int part, sbeg, send;
    fold_unit(pl, coef_stride(P) / 8, tile, part, sbeg, send);
    int li, l;
    int64_t m0;
    fold_place_of(pl, tile, li, l, m0);
    const int lane = threadIdx.x & 63, q = lane >> 4, slot = (threadIdx.x >> 6) * 16 + (lane & 15), k = slot & 7;
    const int n = 1 << l;
    const int x = (int)compact3((uint32_t)slot), y = (int)compact3((uint32_t)slot >> 1), z = (int)compact3((uint32_t)slot >> 2);
    GridSource<P> src;
    src.B = pick(pl.B, li);
    src.G = n + 6;
    src.ox = (int)compact3((uint32_t)m0);
    src.oy = (int)compact3((uint32_t)m0 >> 1);
    src.oz = (int)compact3((uint32_t)m0 >> 2);
    src.reg = reg;
    src.here = (x + 2) + kRegY * (y + 2) + kRegZ * (z + 2) + q * kRegPlane;
    src.st[0] = k & 1 ? -1 : 1;
    src.st[1] = k & 2 ? -kRegY : kRegY;
    src.st[2] = k & 4 ? -kRegZ : kRegZ;
    FoldAcc<P> acc;
    acc.clear();
    fold_run<P>(src, k, sbeg, send, A, orbits, kap, As, acc);
    if (m0 + slot >= (int64_t)1 << (3 * l)) return;
    double *dst = part < 0 ? pick(pl.L, li) + ((int64_t)(src.ox + x) +
                                               (int64_t)n * ((src.oy + y) + (int64_t)n * (src.oz + z))) * S
                           : partial + (((int64_t)part * pl.nrest + (tile - pl.nfull)) * fold_tile(P) + slot) * P2;
    acc.each(k, q, rows, [&](int c, double v) __attribute__((always_inline)) { dst[c] = v; });
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
int fold_tile_targets(int P) { return fold_tile(P); }

// Tiles to compute units: as many whole rounds of one tile per unit as there
// are, then the rest in s parts of their steps, s the count that takes the
// least time among those whose FP64 partial sums fit `cap` bytes.
FoldPlan fold_plan(int P, int64_t tiles, int ncu, size_t cap) {
    constexpr FoldOrbits O = fold_orbits();
    FoldPlan pl{};
    pl.tile = fold_tile(P);
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

// the uniform tree's tiles, the largest level first
static FoldPlan grid_plan(int P, int L, int ncu, size_t cap) {
    int64_t tiles = 0, tile0[kFoldMaxLev] = {};
    for (int i = 0; i < L - 1; ++i) {
        tile0[i] = tiles;
        tiles += (((int64_t)1 << (3 * (L - i))) + fold_tile(P) - 1) / fold_tile(P);
    }
    FoldPlan pl = fold_plan(P, tiles, ncu, cap);
    pl.nlev = L - 1;
    for (int i = 0; i < L - 1; ++i) {
        pl.level[i] = L - i;
        pl.tile0[i] = tile0[i];
    }
    return pl;
}

size_t fold_partial_bytes(const FoldPlan &pl, int P) {
    return pl.nrest ? sizeof(double) * (size_t)pl.nsplit * pl.nrest * pl.tile * P * P : 0;
}

size_t m2l_fold_partial_bytes(int P, int L, int ncu, size_t cap) {
    return L < 2 ? 0 : fold_partial_bytes(grid_plan(P, L, ncu, cap), P);
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
    // slots of each class: its offsets are class 0's with the axes of k negated
    h.cls.assign((size_t)8 * kOffsetsPerClass, int2{0, 0});
    for (int k = 0; k < 8; ++k)
        for (int o = 0; o < kFoldOrbits; ++o)
            for (int m = 0; m < 8; ++m) {
                if (m & ~O.o[o].T) continue;
                int d[3];
                for (int a = 0; a < 3; ++a) d[a] = (((m ^ k) >> a) & 1 ? -O.o[o].a[a] : O.o[o].a[a]) + 4;
                h.cls[(size_t)k * kOffsetsPerClass + O.src0[o] + fold_rank(O.o[o].T, m)].x = d[0] | d[1] << 4 | d[2] << 8;
            }
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
    FoldPlan pl = grid_plan(P, L, ncu, cap);
    if (fold_partial_bytes(pl, P) > 0 && (!partial || partial_bytes < fold_partial_bytes(pl, P)))
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
