// m2l_fold_ad.hip -- the folded FP64 M2L (fold.hpp, fold_kernel.hpp) on the
// adaptive tree: the boxes of levels >= 2 are one list of targets, their
// sources the rows that their V slots name.  Targets need no grouping by
// level or class (the operators serve all of them).
// Measured, 1e6 particles in Gaussian blobs, p = 8 (60,559 boxes): 1.07
// ms against 2.92 ms of the direct products (v_mfma_f64_16x16x4_f64, 189
// slots); the matrix products alone would take 0.31 ms, the rest is the signs,
// butterflies and addresses, which do not run beside them, and waiting for
// the sources (with every source read left out, 28% less).
#include "fold_kernel.hpp"

namespace fmm {

// The slots of a tile's boxes lie in LDS (slot-major, an odd pitch so that
// they are stored without bank conflicts), as places of the source rows in
// units of 64 bytes; the rows' pairs are read from memory a step ahead.  Chunk by chunk, a tile and
// its neighbours' tiles on the same XCD read one 64-byte line of each row at
// a time, which the L2 then holds for its up to 189 readers.
template <int P>
struct SlotSource {
    static constexpr int S = coef_stride(P), NT = 64 * fold_waves(P), PITCH = fold_tile(P) + 1;
    const f64x2 *__restrict__ M;   // rows in K order, at the lane's pair
    const f64x2 *mj;               // the same at the chunk
    const uint32_t *slots;         // LDS, at the lane's box
    uint32_t row[8];
    __device__ __forceinline__ void chunk(int j) { mj = M + 4 * j; }
    template <int T>
    __device__ __forceinline__ void fetch(int o, uint32_t) {
        constexpr FoldOrbits O = fold_orbits();
        constexpr int o0 = O.t0[T][0], NS = 1 << ((T & 1) + ((T >> 1) & 1) + (T >> 2));
        const uint32_t *s = slots + (O.src0[o0] + (o - o0) * NS) * PITCH;
#pragma unroll
        for (int m = 0; m < 8; ++m)
            if ((m & ~T) == 0) row[m] = s[fold_rank(T, m) * PITCH];
    }
    template <int T, int HALF>
    __device__ __forceinline__ void load(int sw, double (&nx)[8][2]) {
#pragma unroll
        for (int m = 0; m < 8; ++m)
            if ((m & ~T) == 0) {
                const f64x2 v = mj[(uint64_t)row[m] * 4];
                nx[m][0] = HALF && sw ? v.y : v.x;
                nx[m][1] = HALF && sw ? v.x : v.y;
            }
    }
};

template <int P>
__global__ __launch_bounds__(64 * fold_waves(P))
__attribute__((amdgpu_waves_per_eu(fold_waves(P) / 4, fold_waves(P) / 4))) void k_ad_m2l_fold(
    FoldPlan pl, const double *__restrict__ A, const uint32_t *__restrict__ orbits, const uint16_t *__restrict__ kap,
    const int16_t *__restrict__ rows, const double *__restrict__ M, const int *__restrict__ vidx,
    const uint32_t *__restrict__ code, int64_t box2, int64_t nv, int64_t zero_row, double *__restrict__ Lc,
    double *__restrict__ partial) {
    constexpr int P2 = P * P, S = coef_stride(P), TILE = fold_tile(P), PITCH = SlotSource<P>::PITCH;
    __shared__ __align__(16) f64x2 As[4 * kFoldPieces<P>];
    __shared__ uint32_t sl[kOffsetsPerClass * PITCH];
    int64_t tile;
    int part, sbeg, send;
    fold_unit(pl, coef_stride(P) / 8, tile, part, sbeg, send);
    const int lane = threadIdx.x & 63, q = lane >> 4, slot = (threadIdx.x >> 6) * 16 + (lane & 15);
    const int64_t b0 = tile * TILE;
    const int nb = (int)min((int64_t)TILE, nv - b0);
    const int *v0 = vidx + b0 * kOffsetsPerClass;
#pragma unroll 8
    for (int e = threadIdx.x; e < TILE * kOffsetsPerClass; e += SlotSource<P>::NT) {
        const int c = e / kOffsetsPerClass, s = e - c * kOffsetsPerClass;
        const int r = c < nb ? v0[e] : -1;
        sl[s * PITCH + c] = (uint32_t)((r >= 0 ? (int64_t)r : zero_row) * (S / 8));
    }
    const int64_t g = box2 + b0 + min(slot, nb - 1);
    const int k = (int)(code[g] & 7u);
    SlotSource<P> src;
    src.M = (const f64x2 *)M + q;
    src.slots = sl + slot;
    FoldAcc<P> acc;
    acc.clear();
    fold_run<P>(src, k, sbeg, send, A, orbits, kap, As, acc);
    if (slot >= nb) return;
    if (part < 0) {
        double *dst = Lc + g * S;
        acc.each(k, q, rows, [&](int c, double v) __attribute__((always_inline)) { dst[c] += v; });
    } else {
        double *dst = partial + (((int64_t)part * pl.nrest + (tile - pl.nfull)) * TILE + slot) * P2;
        acc.each(k, q, rows, [&](int c, double v) __attribute__((always_inline)) { dst[c] = v; });
    }
}

// the parts of the rest tiles added into the locals, in part order
__global__ __launch_bounds__(256) void k_ad_m2l_fold_sum(int P, FoldPlan pl, int64_t box2, int64_t nv,
                                                         const double *__restrict__ partial, double *__restrict__ Lc) {
    const int P2 = P * P, S = coef_stride(P);
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t step = (int64_t)pl.nrest * pl.tile * P2;
    const int64_t t = i / P2, b = pl.nfull * pl.tile + t;
    if (i >= step || b >= nv) return;
    double v = 0.0;
    for (int s = 0; s < pl.nsplit; ++s) v += partial[s * step + i];
    Lc[(box2 + b) * S + (i - t * P2)] += v;
}

// Rows 0 .. nrow - 1 into K order, the last one zero; two positions a thread.
__global__ __launch_bounds__(256) void k_ad_fold_pack(int P, int64_t nrow, const int16_t *__restrict__ kperm,
                                                      const double *__restrict__ M, f64x2 *__restrict__ out) {
    const int S2 = coef_stride(P) / 2;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x, r = i / S2;
    if (r >= nrow) return;
    const int c = 2 * (int)(i - r * S2);
    f64x2 v = {0.0, 0.0};
    if (r + 1 < nrow) {
        const double *src = M + r * 2 * S2;
        const int c0 = kperm[c], c1 = kperm[c + 1];
        if (c0 >= 0) v.x = src[c0];
        if (c1 >= 0) v.y = src[c1];
    }
    out[i] = v;
}

// The rows 0 .. nrow - 1 of M into K order in their place (BACK: into the
// coefficients' own order again), the last row zero: a block reads and writes
// reorder_rows(P) rows, four elements a thread.  Where the operands have no
// room of their own: two passes over M in place of k_ad_fold_pack's one
// (206,000 boxes at p = 4: 9.9 and 10.8 us against 9.4; 24,000 at p = 14: 14.1
// and 15.7 against 14.5).
constexpr int kReorder = 4;  // elements per thread
static int reorder_rows(int P) { return 256 * kReorder / coef_stride(P); }
static_assert(kMaxStride <= 256 * kReorder, "a row per block");
template <bool BACK>
__global__ __launch_bounds__(256) void k_ad_fold_reorder(int P, int rows, int64_t nrow,
                                                         const int16_t *__restrict__ kperm, double *M) {
    const int S = coef_stride(P);
    const int64_t r0 = (int64_t)blockIdx.x * rows;
    double *row[kReorder], v[kReorder];
    int to[kReorder];  // where the thread's elements go, -1: none
#pragma unroll
    for (int k = 0; k < kReorder; ++k) {
        const int e = threadIdx.x + 256 * k, lr = e / S, i = e - lr * S;
        const int64_t r = r0 + lr;
        const bool in = lr < rows && r < nrow;
        const int c = in ? kperm[i] : -1;  // no coefficient past p^2, in either order
        row[k] = M + r * S;
        to[k] = in ? (BACK && c >= 0 ? c : i) : -1;
        v[k] = r + 1 < nrow && c >= 0 ? row[k][BACK ? i : c] : 0.0;
    }
    __syncthreads();  // the rows have been read
#pragma unroll
    for (int k = 0; k < kReorder; ++k)
        if (to[k] >= 0) row[k][to[k]] = v[k];
}

hipError_t ad_launch_m2l_fold(int P, const FoldPlan &pl, const double *A, const FoldDev &fd, double *M,
                              const int *vidx, const uint32_t *code, int64_t box2, int64_t nbox, double *Lc,
                              double *pack, double *partial, hipStream_t st) {
    const int64_t nv = nbox - box2;
    if (nv <= 0) return hipSuccess;
    const int64_t np = (nbox + 1) * (coef_stride(P) / 2);
    const int rows = reorder_rows(P);
    const unsigned nr = (unsigned)((nbox + rows) / rows);
    if (pack == M)
        k_ad_fold_reorder<false><<<nr, 256, 0, st>>>(P, rows, nbox + 1, fd.kperm, M);
    else
        k_ad_fold_pack<<<(unsigned)((np + 255) / 256), 256, 0, st>>>(P, nbox + 1, fd.kperm, M, (f64x2 *)pack);
    const unsigned nb = (unsigned)(pl.nfull + (int64_t)pl.nrest * pl.nsplit);
    switch (P) {
#define CASE(PP)                                                                                                   \
    case PP:                                                                                                       \
        k_ad_m2l_fold<PP><<<nb, 64 * fold_waves(PP), 0, st>>>(pl, A, fd.orbits, fd.kap, fd.rows, pack, vidx, code, \
                                                              box2, nv, nbox, Lc, partial);                        \
        break;
        CASE(1) CASE(2) CASE(3) CASE(4) CASE(5) CASE(6) CASE(7) CASE(8)
        CASE(9) CASE(10) CASE(11) CASE(12) CASE(13) CASE(14) CASE(15) CASE(16)
#undef CASE
        default: return hipErrorInvalidValue;
    }
    if (pl.nrest)
        k_ad_m2l_fold_sum<<<(unsigned)(((int64_t)pl.nrest * pl.tile * P * P + 255) / 256), 256, 0, st>>>(
            P, pl, box2, nv, partial, Lc);
    if (pack == M) k_ad_fold_reorder<true><<<nr, 256, 0, st>>>(P, rows, nbox + 1, fd.kperm, M);
    return hipGetLastError();
}

}  // namespace fmm
