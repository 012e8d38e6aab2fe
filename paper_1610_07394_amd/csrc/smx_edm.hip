// Packed Euclidean distance matrix, FP32 difference form (paper Sec. I and
// II: the EDM is a 2-simplex problem; only the upper triangle is computed and
// stored).
//
// One block of 256 threads owns a T x T tile (X, Y), X <= Y, of the packed
// upper triangle, T = 16 MT (MT = 4 or 8).  The map (lambda2, bounding box or
// linear) only decides which tile a block gets; the body is the same, so
// results are bit-identical across maps.  Per block:
//   * the two T x d row panels of X are staged through LDS in K chunks of 32
//     (row-major, row stride 36 floats: the 16 distinct rows a wave reads with
//     ds_read_b128 land in 16 distinct 16-byte bank groups);
//   * thread (tx, ty) accumulates rows ty + 16 r and columns tx + 16 c
//     (r, c < MT) with one subtract and one FMA per element and dimension --
//     the difference form costs 2 VALU operations per element-dimension, and
//     each ds_read_b128 feeds 4 MT such operations;
//   * stores go to p(i, j) = i n - i (i - 1) / 2 + (j - i): for fixed (r, c) the
//     16 lanes of a row write 16 consecutive floats.
// Larger sets take the matrix form of smx_gram.hip, which falls back on this tile.
#include "smx_device.h"
#include "smx_edm_tile.h"
#include "smx_internal.h"

namespace smx {

// TILED: the tile-contiguous layout (tile (X, Y) at rank Y(Y+1)/2 + X times T^2,
// element (i, j) at (i mod T) T + (j mod T), entries outside i <= j < n zero).
template <int MAP, int MT, bool VEC, bool STATS, bool TILED>
__global__ __launch_bounds__(kEdmThreads, 3) void edm_diff_kernel(MapGeom g, const float *__restrict__ X,
                                                               int64_t n, int64_t d, int64_t ldx,
                                                               float *__restrict__ D,
                                                               unsigned long long *slots) {
    constexpr int T = 16 * MT;
    uint64_t lin;
    int TX, TY;
    if (!tile2_of<MAP, true>(g, lin, TX, TY)) return;

    __shared__ __attribute__((aligned(16))) float As[T * kEdmLd];
    __shared__ __attribute__((aligned(16))) float Bs[T * kEdmLd];

    edm_diff_tile<MT, VEC, TILED>(As, Bs, TX, TY, X, n, d, ldx, D);
    if (STATS) {
        __shared__ unsigned long long red[2][kEdmThreads / kWave];
        unsigned long long cnt, cs;
        tile_pairs_le_stats<kEdmThreads>(int64_t(TX) * T, int64_t(TY) * T, T, T, n, cnt, cs);
        const unsigned long long c = block_sum<unsigned long long, kEdmThreads>(cnt, red[0]);
        const unsigned long long h = block_sum<unsigned long long, kEdmThreads>(cs, red[1]);
        if (threadIdx.x == 0) stats_add(slots, lin, c, h);
    }
}

template <int MAP, int MT, bool VEC, bool TILED>
static void go_edm(const MapGeom &g, const float *X, int64_t n, int64_t d, int64_t ldx, float *D,
                   unsigned long long *slots, hipStream_t s) {
    const dim3 grid = MAP == MAP_BBOX ? dim3(g.nb, g.nb, 1) : grid_for(g.G, kEdmThreads);
    if (slots)
        hipLaunchKernelGGL((edm_diff_kernel<MAP, MT, VEC, true, TILED>), grid, dim3(kEdmThreads), 0, s, g, X, n,
                           d, ldx, D, slots);
    else
        hipLaunchKernelGGL((edm_diff_kernel<MAP, MT, VEC, false, TILED>), grid, dim3(kEdmThreads), 0, s, g, X, n,
                           d, ldx, D, slots);
}

template <int MAP>
static void go_edm_map(const MapGeom &g, int tile, bool vec, bool tiled, const float *X, int64_t n, int64_t d,
                       int64_t ldx, float *D, unsigned long long *slots, hipStream_t s) {
    if (tiled) {  // the tile-contiguous layout uses 128-wide tiles at every n
        if (vec) go_edm<MAP, 8, true, true>(g, X, n, d, ldx, D, slots, s);
        else go_edm<MAP, 8, false, true>(g, X, n, d, ldx, D, slots, s);
    } else if (tile == 128) {
        if (vec) go_edm<MAP, 8, true, false>(g, X, n, d, ldx, D, slots, s);
        else go_edm<MAP, 8, false, false>(g, X, n, d, ldx, D, slots, s);
    } else {
        if (vec) go_edm<MAP, 4, true, false>(g, X, n, d, ldx, D, slots, s);
        else go_edm<MAP, 4, false, false>(g, X, n, d, ldx, D, slots, s);
    }
}

int launch_edm_diff(const MapGeom &g, int tile, const float *X, int64_t n, int64_t d, int64_t ldx, float *D,
                    unsigned long long *slots, bool tiled, hipStream_t s) {
    const bool vec = (ldx % 4 == 0) && (d % kEdmKc == 0) && ((reinterpret_cast<uintptr_t>(X) & 15) == 0);
    prof_begin(K_EDM_DIFF, s);
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        go_edm_map<decltype(M)::value>(gg, tile, vec, tiled, X, n, d, ldx, D, slots, s);
    });
    prof_end(K_EDM_DIFF, s);
    return check_launch("edm_packed (fp32 diff)");
}

SMX_CHECK_READER(check_flags_edm)

}  // namespace smx
