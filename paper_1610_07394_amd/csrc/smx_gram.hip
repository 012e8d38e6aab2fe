// Packed Euclidean distance matrix, Gram form on the BF16 matrix cores.
//
//   D_ij = |x_i|^2 + |x_j|^2 - 2 G_ij,  G = X X^T on the tile pair (I, J),
//
// with G from v_mfma_f32_32x32x16_bf16 (FP32 accumulation) and the norms in
// FP32 from the FP32 input.  Plain BF16: G = hi hi^T.  Split BF16 (hi =
// bf16(x), lo = bf16(x - hi), both round-to-nearest-even): G = hi hi^T +
// hi lo^T + lo hi^T, dropping lo lo^T (relative size 2^-16).  D is clamped
// at 0 and the diagonal is set to exactly 0 (the Gram form cancels there).
//
// Block: 256 threads (4 waves as 2 x 2), tile 128 x 128 of the packed upper
// triangle, each wave 64 x 64 in MFMA tiles of 32 x 32.  K advances in steps
// of 16 BF16 through a 32 KB ring of LDS slots filled directly from global
// memory in MFMA fragment order (see the staging notes below), so the loads
// of the next steps are in flight while the matrix cores run the current one.
#include <type_traits>

#include "smx_device.h"
#include "smx_edm_tile.h"
#include "smx_internal.h"

namespace smx {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kGramThreads = 256;

__device__ __forceinline__ uint16_t bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return uint16_t((u >> 16) | 0x40u);  // quiet NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return uint16_t(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }

// Operand layout in HBM ("fragment order").  hi and lo are stored as 1 KB
// blocks, one per (32-row block rb, 16-wide k block kb), at uint4 index
// (rb * KB + kb) * 64 + s, KB = dpad / 16, where slot s holds row
// 32 rb + (s & 31), k = 16 kb + 8 (s >> 5) .. +7: exactly the operand a lane
// s of v_mfma_f32_32x32x16_bf16 reads.  So a staging load is one contiguous
// 1 KB run.  Rows are padded with zeros to npad = 32 ceil(n / 32), k to dpad.
//
// One wave per row: each lane converts 8 consecutive k (one 16-byte slot of
// hi and of lo) and adds their squares to an FP32 norm (lane-ordered FMA
// sums, then a fixed wave tree).
__global__ __launch_bounds__(256) void gram_prep_kernel(const float *__restrict__ X, int64_t n,
                                                        int64_t d, int64_t ldx, int64_t dpad,
                                                        int64_t npad, uint4 *__restrict__ hi,
                                                        uint4 *__restrict__ lo,
                                                        float *__restrict__ norms) {
    const int lane = threadIdx.x & 63;
    const int64_t row = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (row >= npad) return;
    const int64_t KB = dpad / 16;
    float acc = 0.f;
    for (int64_t q = lane; q < dpad / 8; q += 64) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t k = 8 * q + e;
            x[e] = (row < n && k < d) ? X[row * ldx + k] : 0.f;
            acc = __builtin_fmaf(x[e], x[e], acc);
        }
        uint32_t h[4], l[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint16_t h0 = bf16_rne(x[2 * e]), h1 = bf16_rne(x[2 * e + 1]);
            h[e] = uint32_t(h0) | (uint32_t(h1) << 16);
            const uint16_t l0 = bf16_rne(x[2 * e] - bf16_to_f32(h0));
            const uint16_t l1 = bf16_rne(x[2 * e + 1] - bf16_to_f32(h1));
            l[e] = uint32_t(l0) | (uint32_t(l1) << 16);
        }
        const int64_t slot = ((row >> 5) * KB + (q >> 1)) * 64 + (row & 31) + 32 * (q & 1);
        hi[slot] = make_uint4(h[0], h[1], h[2], h[3]);
        if (lo != nullptr) lo[slot] = make_uint4(l[0], l[1], l[2], l[3]);
    }
    acc = wave_sum(acc);
    if (lane == 0 && row < n) norms[row] = acc;
}

int launch_gram_prep(const float *X, int64_t n, int64_t d, int64_t ldx, int64_t dpad, uint16_t *hi,
                     uint16_t *lo, float *norms, bool split, hipStream_t s) {
    const int64_t npad = gram_rows(n);
    prof_begin(K_GRAM_PREP, s);
    hipLaunchKernelGGL(gram_prep_kernel, dim3(uint32_t(npad / 4)), dim3(256), 0, s, X, n, d, ldx, dpad,
                       npad, reinterpret_cast<uint4 *>(hi), split ? reinterpret_cast<uint4 *>(lo) : nullptr,
                       norms);
    prof_end(K_GRAM_PREP, s);
    return check_launch("gram prep");
}

// Staging.  Every MFMA operand fragment travels from global memory straight
// into LDS with global_load_lds_dwordx4: one wave load moves one contiguous
// 1 KB block of the fragment-ordered operand, lane s writing the 16 bytes it
// later reads back as its operand (rows mb*32 + (s & 31), k = 8*(s >> 5) .. +7
// of one 16-wide k step), so an operand read is base + 16*lane (no bank
// conflicts) and staging costs no VGPRs.
//
// Pipeline.  One stage = one 16-wide k step of both panels.  A ring of S
// stages keeps S - 1 steps of loads in flight: at step s a wave waits until
// only the loads of steps s+1 .. s+S-2 are outstanding (loads complete in
// issue order), the block synchronises, the loads of step s+S-1 go into the
// slot step s-1 used, and the MFMAs of step s run.
//
// WT = wave tile: the block tile is T = 2 WT, each wave owns WT / 32 x WT / 32
// MFMA tiles.  T = 128 (WT = 64) with a 32 KB ring (4 slots of 8 KB plain, 2
// of 16 KB split): at most 128 registers per lane and 33 KB of LDS, so four
// blocks share a CU and the store-heavy epilogue of one overlaps the others'
// k loops.  Measured on MI355X against 2 blocks per CU with 64 KB rings and
// against wider slots (2 or 4 k steps each, 32-64 KB): those were 4-20%
// slower; so were persistent grids that overlap each tile's stores with the
// next tile's k loop inside one block.
template <bool SPLIT, int WT>
struct GramCfg {
    static constexpr int NARR = SPLIT ? 4 : 2;     // A_hi, B_hi, (A_lo, B_lo)
    static constexpr int T = 2 * WT;               // block tile edge
    static constexpr int MT = WT / 32;             // MFMA tiles per wave edge
    static constexpr int RB = T / 32;              // 32-row blocks per panel
    static constexpr int KS = 1;                   // 16-wide k blocks per stage
    static constexpr int STAGE = NARR * RB * KS;   // 1 KB blocks per stage
    static constexpr int LPW = STAGE / 4;          // loads per wave per stage
    static constexpr int S = SPLIT ? 2 : 4;         // ring depth: 32 KB either way
};

// One 16-byte store of four packed distances, ordinary or marked non-temporal.
// The distances are written once and never read back by the kernel; streaming
// them past the caches keeps the L2 for the operand panels, which pays once the
// k loop is long.  Measured on MI355X at n = 32768 (ms, ordinary / streaming):
// plain d = 32 0.58 / 0.77, d = 128 0.64 / 0.76, d = 256 0.77 / 0.76, d = 512
// 1.02 / 0.80; split d = 64 0.67 / 0.79, d = 128 0.81 / 0.80, d = 512 1.71 /
// 1.69.  The streaming stores hold about 2.8 TB/s whatever d; the ordinary
// ones reach 3.7 TB/s alone but slow the k loop down as d grows.  The
// tile-contiguous layout (aligned 64 KB runs) follows the same rule: plain
// d = 32 0.37 / 0.37, d = 512 0.83 / 0.74.  (A HIP float4 assignment here
// compiled to a 12-byte and a 4-byte store, hence the vector type.)
template <bool NT>
__device__ __forceinline__ void store4(float *p, float4 v) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const f4 w = {v.x, v.y, v.z, v.w};
    if constexpr (NT)
        __builtin_nontemporal_store(w, reinterpret_cast<f4 *>(p));
    else
        *reinterpret_cast<f4 *>(p) = w;
}

// One stage's loads into buf ([narr][rb_n][64] uint4); the counts are
// compile-time constants at every (inlined) call.  Row blocks past the padded
// operand (a ragged last tile) load its last block; their outputs are never
// stored.
__device__ __forceinline__ void gram_issue(uint4 *buf, int narr, int rb_n, int ks, const uint4 *__restrict__ hi,
                                           const uint4 *__restrict__ lo, int64_t I0, int64_t J0, int64_t rbmax,
                                           int64_t KB, int64_t kb, int wave, int lane) {
#pragma unroll
    for (int t = 0; t < narr * rb_n * ks / 4; ++t) {
        const int gb = wave + 4 * t;  // 0 .. narr * rb_n * ks - 1: [array][row block][k block]
        const int arr = gb / (rb_n * ks), rem = gb % (rb_n * ks), mb = rem / ks, kk = rem % ks;
        const uint4 *src = (arr & 2) ? lo : hi;
        int64_t rb = (((arr & 1) ? J0 : I0) >> 5) + mb;
        rb = rb < rbmax ? rb : rbmax;
        __builtin_amdgcn_global_load_lds(src + (rb * KB + kb + kk) * 64 + lane, buf + gb * 64, 16, 0, 0);
    }
}

// s_waitcnt with vmcnt <= N (N < 64) and no wait on the other counters.
template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
template <int LPW, int A>
__device__ __forceinline__ void wait_vm_ahead(int ahead) {
    if constexpr (A < 0) {
        return;
    } else {
        if (ahead == A) wait_vm<A * LPW>();
        else wait_vm_ahead<LPW, A - 1>(ahead);
    }
}

// Operand fragments are read from the ring with ds_read_b128 written out as
// inline assembly: the compiler does not model the LDS writes of the
// global-to-LDS loads, so it would either wait for every load in flight
// before each LDS read or treat the ring as never written.  The reads are
// waited for explicitly (lds_wait), and that wait names the fragment
// registers so no use can move above it.
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ bf16x8_t lds_frag(uint32_t addr) {
    bf16x8_t v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr) : "memory");
    return v;
}
template <int NP, int MT>
__device__ __forceinline__ void lds_wait(bf16x8_t (&a)[NP][MT], bf16x8_t (&b)[NP][MT]) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int m = 0; m < MT; ++m) asm volatile("" : "+v"(a[p][m]), "+v"(b[p][m]));
}

// TILED: the tile-contiguous layout (tile (X, Y) at rank Y(Y+1)/2 + X times T^2,
// element (i, j) at (i mod T) T + (j mod T), entries outside i <= j < n zero).
// NT: the output stores are streaming (non-temporal); chosen at compile time,
// since the compiler merges the two arms of a run-time choice into one ordinary
// store.
template <int MAP, bool SPLIT, bool STATS, int WT, bool TILED, bool NT>
__global__ __launch_bounds__(kGramThreads, 4) void edm_gram_kernel(MapGeom g, const uint16_t *__restrict__ hi,
                                                               const uint16_t *__restrict__ lo,
                                                               const float *__restrict__ norms,
                                                               int64_t n, int64_t dpad,
                                                               float *__restrict__ D,
                                                               unsigned long long *slots) {
    using C = GramCfg<SPLIT, WT>;
    constexpr int T = C::T, MT = C::MT, NP = SPLIT ? 2 : 1, S = C::S;
    constexpr int BUF = C::STAGE * 64;  // uint4 per ring slot
    static_assert(S * BUF * 16 >= 2 * 32 * T * 4, "the epilogue stages 64 tile rows in the ring");
    uint64_t lin;
    int TX, TY;
    if (MAP == MAP_LAMBDA) {
        // Each XCD takes one contiguous range of Pi2, walked in patches (w_x by
        // w_y ids: 8 x 16 plain, 16 x 8 split) so that its L2 keeps the row and
        // column panels of the tiles it runs at once: operands fetched from
        // beyond L2 4.2 -> 0.8 GB plain, 8.6 -> 2.8 GB split.  Column-major order
        // (w_y fastest, whose concurrent tiles extend the same packed rows) is
        // the faster one for the stores alone, but with the non-temporal stores
        // the patches took 5-10% less time at d = 512.  Where nb is no power of two the
        // filtered ids lie in stretches that would empty some XCDs' ranges, and runs of 16
        // ids are dealt in turn instead, us: n = 16484, d = 300 268 -> 227 plain, 536 -> 333
        // split; n = 20000, d = 64 250 -> 235 and 300 -> 247; n = 5000, d = 32 28 -> 20 and
        // 34 -> 22.
        lin = launch_index();
        if (lin >= g.G) return;
        const uint32_t id = (g.nb & (g.nb - 1)) == 0 ? xcd_remap(uint32_t(lin), uint32_t(g.G))
                                                     : xcd_deal(uint32_t(lin), uint32_t(g.G), 4);
        if (!lambda2(SPLIT ? lambda2_patch_to_xfast(id, g.lg, 4, 3) : lambda2_patch_to_xfast(id, g.lg, 3, 4), g.lg,
                     g.nb, TX, TY))
            return;
        if (SMX_CHECKED && !smx_check(0 <= TX && TX <= TY && TY < g.nb, kCheckMap)) return;
    } else if (!tile2_of<MAP, true>(g, lin, TX, TY)) {
        return;
    }
    __shared__ __attribute__((aligned(16))) uint4 Lb[S * BUF];
    __shared__ __attribute__((aligned(16))) float nA[T], nB[T];

    const int t = threadIdx.x;
    const int lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
    const int64_t I0 = int64_t(TX) * T, J0 = int64_t(TY) * T;
    const bool diag = TX == TY;

    for (int x = t; x < 2 * T; x += kGramThreads) {
        const int64_t r = (x < T ? I0 : J0) + (x & (T - 1));
        (x < T ? nA : nB)[x & (T - 1)] = r < n ? norms[r] : 0.f;
    }

    f32x16_t acc[MT][MT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int c = 0; c < MT; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][c][e] = 0.f;

    constexpr int KS = C::KS;
    const int nst = int(dpad / (16 * KS));  // stages of KS 16-wide k blocks
    const int64_t KB = dpad / 16, rbmax = gram_rows(n) / 32 - 1;
    const uint4 *hi4 = reinterpret_cast<const uint4 *>(hi), *lo4 = reinterpret_cast<const uint4 *>(lo);
    for (int p = 0; p < S - 1 && p < nst; ++p)
        gram_issue(Lb + p * BUF, C::NARR, C::RB, KS, hi4, lo4, I0, J0, rbmax, KB, int64_t(p) * KS, w, lane);
    const uint32_t ring = lds_addr(Lb);
    bf16x8_t a[2][NP][MT], b[2][NP][MT];  // [k block parity][hi, lo][sub-tile]
    for (int st = 0; st < nst; ++st) {
        const int ahead = nst - 1 - st < S - 2 ? nst - 1 - st : S - 2;
        wait_vm_ahead<C::LPW, S - 2>(ahead);  // this wave's loads of stage st have landed
        __builtin_amdgcn_s_barrier();           // ... and every wave's; stage st - 1 is consumed
        if (st + S - 1 < nst)
            gram_issue(Lb + ((st + S - 1) % S) * BUF, C::NARR, C::RB, KS, hi4, lo4, I0, J0, rbmax, KB,
                       int64_t(st + S - 1) * KS, w, lane);
        const uint32_t cur = ring + uint32_t((st % S) * BUF) * 16u + uint32_t(lane) * 16u;
        // k blocks of the stage, the fragments of block kk + 1 read while block kk multiplies
        auto rd = [&](int kk, bf16x8_t(&fa)[NP][MT], bf16x8_t(&fb)[NP][MT]) {
#pragma unroll
            for (int p = 0; p < NP; ++p)
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    fa[p][m] = lds_frag(cur + uint32_t((((2 * p) * C::RB + wm * MT + m) * KS + kk) * 64 * 16));
                    fb[p][m] = lds_frag(cur + uint32_t((((2 * p + 1) * C::RB + wn * MT + m) * KS + kk) * 64 * 16));
                }
        };
        rd(0, a[0], b[0]);
        lds_wait<NP, MT>(a[0], b[0]);
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const int q = kk & 1;
            if (kk + 1 < KS) rd(kk + 1, a[q ^ 1], b[q ^ 1]);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int c = 0; c < MT; ++c) {
                    acc[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q][0][m], b[q][0][c], acc[m][c], 0, 0, 0);
                    if (SPLIT) {
                        acc[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q][0][m], b[q][NP - 1][c], acc[m][c], 0,
                                                                            0, 0);
                        acc[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[q][NP - 1][m], b[q][0][c], acc[m][c], 0,
                                                                            0, 0);
                    }
                }
            if (kk + 1 < KS) lds_wait<NP, MT>(a[q ^ 1], b[q ^ 1]);
        }
    }

    // Epilogue.  32 x 32 accumulator layout: lane l, element e holds row
    // (e & 3) + 4 (l >> 5) + 8 (e >> 2) and column l & 31 of the MFMA tile.
    // Per pass m the four waves stage 64 whole rows of the tile (32 from each
    // row half) in the (now idle) ring; then each wave writes 16 of them, two
    // 512-byte tile rows per store instruction, so that only the two ends of a
    // tile row share a 128-byte line with the neighbouring tiles (half-row
    // pieces per wave: 0.995 against 0.938 ms plain, 1.855 against 1.829 split).
    // Tiles off the diagonal and inside n (all but a thin fringe) store
    // unmasked.
    static_assert(T == 128 && kGramThreads == 256, "the store loop assumes 4 waves and 128-wide tile rows");
    float *St = reinterpret_cast<float *>(Lb);  // [2 * 32 rows][T], the rows of one pass
    const bool interior = !diag && I0 + T <= n && J0 + T <= n;
    __syncthreads();  // nA and nB are other threads' work (the k loop's barriers order no LDS writes)
    float nb[MT];
#pragma unroll
    for (int c = 0; c < MT; ++c) nb[c] = nB[wn * WT + c * 32 + (lane & 31)];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        __syncthreads();  // the ring (k loop) or the previous pass's rows are consumed
        float na[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 r4 = *reinterpret_cast<const float4 *>(&nA[wm * WT + m * 32 + 8 * q + 4 * (lane >> 5)]);
            na[4 * q + 0] = r4.x; na[4 * q + 1] = r4.y; na[4 * q + 2] = r4.z; na[4 * q + 3] = r4.w;
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int rl = (e & 3) + 4 * (lane >> 5) + 8 * (e >> 2);
#pragma unroll
            for (int c = 0; c < MT; ++c) {
                float v = fmaxf(__builtin_fmaf(-2.f, acc[m][c][e], na[e] + nb[c]), 0.f);
                // on a diagonal tile, element (il, il) is the diagonal: exactly 0
                v = (diag && wm * WT + m * 32 + rl == wn * WT + c * 32 + (lane & 31)) ? 0.f : v;
                St[(wm * 32 + rl) * T + wn * WT + c * 32 + (lane & 31)] = v;
            }
        }
        __syncthreads();
        // each wave writes 16 whole tile rows, two per instruction
#pragma unroll
        for (int it = 0; it < 8; ++it) {
            const int r = w * 16 + 2 * it + (lane >> 5), cl = 4 * (lane & 31);
            const int64_t i = I0 + (r >> 5) * WT + m * 32 + (r & 31), j = J0 + cl;
            const float4 v = *reinterpret_cast<const float4 *>(St + r * T + cl);
            if (TILED) {
                const uint64_t rank = uint64_t(TY) * (uint64_t(TY) + 1) / 2 + uint64_t(TX);
                float *tdst = D + rank * uint64_t(T * T) + uint64_t(i - I0) * T + uint64_t(j - J0);
                float4 o = v;
                if (!interior) {
                    o.x = (i < n && j + 0 < n && j + 0 >= i) ? v.x : 0.f;
                    o.y = (i < n && j + 1 < n && j + 1 >= i) ? v.y : 0.f;
                    o.z = (i < n && j + 2 < n && j + 2 >= i) ? v.z : 0.f;
                    o.w = (i < n && j + 3 < n && j + 3 >= i) ? v.w : 0.f;
                }
                store4<NT>(tdst, o);  // 16-byte aligned: tiles start at multiples of T^2
                continue;
            }
            float *dst = D + (i * n - (i * (i - 1)) / 2 - i) + j;
            if (interior) {
                if (smx_check(i < n && j >= i && j + 3 < n, kCheckStore))
                    store4<NT>(dst, v);  // 4-byte aligned: the packed rows start anywhere
            } else if (i < n) {
                const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (j + q < n && j + q >= i) dst[q] = vv[q];
            }
        }
    }
    if (STATS) {
        __shared__ unsigned long long red[2][kGramThreads / kWave];
        unsigned long long cnt, cs;
        tile_pairs_le_stats<kGramThreads>(I0, J0, T, T, n, cnt, cs);
        const unsigned long long c = block_sum<unsigned long long, kGramThreads>(cnt, red[0]);
        const unsigned long long h = block_sum<unsigned long long, kGramThreads>(cs, red[1]);
        if (t == 0) stats_add(slots, lin, c, h);
    }
}


template <int MAP, bool SPLIT, int WT, bool TILED, bool NT>
static void go_gram(const MapGeom &g, const uint16_t *hi, const uint16_t *lo, const float *norms,
                    int64_t n, int64_t dpad, float *D, unsigned long long *slots, hipStream_t s) {
    const dim3 grid = MAP == MAP_BBOX ? dim3(g.nb, g.nb, 1) : grid_for(g.G, kGramThreads);
    if (slots)
        hipLaunchKernelGGL((edm_gram_kernel<MAP, SPLIT, true, WT, TILED, NT>), grid, dim3(kGramThreads), 0, s, g,
                           hi, lo, norms, n, dpad, D, slots);
    else
        hipLaunchKernelGGL((edm_gram_kernel<MAP, SPLIT, false, WT, TILED, NT>), grid, dim3(kGramThreads), 0, s, g,
                           hi, lo, norms, n, dpad, D, slots);
}

// Streaming stores once the k loop is long enough for the operand panels' L2
// residency to matter more than the stores' own rate (see store4).
static bool gram_streaming(int64_t dpad, bool split) { return (split ? 2 : 1) * dpad >= 256; }

int launch_edm_gram(const MapGeom &g, int tile, const uint16_t *hi, const uint16_t *lo, const float *norms,
                    int64_t n, int64_t dpad, bool split, float *D, unsigned long long *slots, bool tiled,
                    hipStream_t s) {
    prof_begin(K_EDM_GRAM, s);
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        constexpr int MAPK = decltype(M)::value;
        constexpr int WT = kGramTile / 2;
        (void)tile;  // kGramTile
        const bool nt = gram_streaming(dpad, split);
        if (tiled && nt) {
            if (split) go_gram<MAPK, true, WT, true, true>(gg, hi, lo, norms, n, dpad, D, slots, s);
            else go_gram<MAPK, false, WT, true, true>(gg, hi, lo, norms, n, dpad, D, slots, s);
        } else if (tiled) {
            if (split) go_gram<MAPK, true, WT, true, false>(gg, hi, lo, norms, n, dpad, D, slots, s);
            else go_gram<MAPK, false, WT, true, false>(gg, hi, lo, norms, n, dpad, D, slots, s);
        } else if (nt) {
            if (split) go_gram<MAPK, true, WT, false, true>(gg, hi, lo, norms, n, dpad, D, slots, s);
            else go_gram<MAPK, false, WT, false, true>(gg, hi, lo, norms, n, dpad, D, slots, s);
        } else {
            if (split) go_gram<MAPK, true, WT, false, false>(gg, hi, lo, norms, n, dpad, D, slots, s);
            else go_gram<MAPK, false, WT, false, false>(gg, hi, lo, norms, n, dpad, D, slots, s);
        }
    });
    prof_end(K_EDM_GRAM, s);
    return check_launch("edm_packed (gram)");
}


// ---------------------------------------------------------------- FP32, matrix form
// The difference form costs two vector operations per element and dimension (n =
// 65536, d = 64: 6.3 ms, of which the stores need 2).  This form keeps its FP32
// accuracy on the matrix cores.  Coordinates less a common centre are held as FP16
// pairs hi + lo (2^-23, each row scaled by a power of two); G = hi hi^T + hi lo^T + lo
// hi^T in exact products and FP32 sums; D = (|x_i|^2 - 2 G_ij) + |x_j|^2 with norms
// summed in FP64.  A pair's value stands where it is as exact as the difference
// form's: D >= 5/16 (|x_i|^2 + |x_j|^2) and finite.  Any other pair (near points, NaN,
// infinities, overflow) is summed as the difference form does, in its order, from the
// FP32 input: one thread a pair where a pass of 64 rows has few, else all of the
// pass's through LDS.  Its value does not depend on the tile that holds it.  Where more
// than one of 4096 sampled pairs in 128 is such a pair (kEdmGate), every block takes the
// difference form's tile.  2-norm error, n = 5200 to 8200, normal points, d = 36 / 64 /
// 130 / 512 / 2000 / 8192: 4.5 / 4.4 / 4.5 / 5.1 / 6.2 / 11e-8 against 9.4 / 12 / 17 / 31 / 60 /
// 124e-8 (uniform, offset and unevenly scaled points alike).
//
// Stores.  Packed rows (i, .) start at any 4-byte offset.  A block's row i is shifted
// left by s_i < 32 columns to where its piece starts a 128-byte line: rows of tile (X,
// Y) hold the columns J0 - s_i .. J0 + 127 - s_i (the last tile's to n, the first
// tile's from i), the block computes one 32-column block more on the left (5 / 4 of
// the products), and all stores but those at the ends of a packed row are whole
// lines, streaming.
//
// n = 65536, d = 64: 6.3 -> 2.6 ms (3.3 TB/s of stores); 20000, 100: 1.1 -> 0.37; 9001,
// 37: 0.12 -> 0.09.
constexpr int kLineCols = 160;           // 32 + 128 columns of a tile row
constexpr int kLineLd = kLineCols + 4;   // LDS row: shifted by s_i mod 4 floats
constexpr int kLineList = 128;
// share of |x_i|^2 + |x_j|^2 from which a pair's Gram value is kept
constexpr float kEdmNear = 0.3125f;
// kEdmSampleBlocks blocks of the preparation sample 16 pairs each; the share of near ones,
// 1 / kEdmGate, above which every block takes the difference tile.  A pass lists up to kLineList pairs, 1.25% of its 10240, and with more
// sums all of them as differences; that many passes overflow, so close to a share of 1%,
// cost more than the difference tile does.  Never / always that tile, ms, n = 65536, d = 64, tight
// clusters of equal size in random order: 128 (0.8% near) 3.5 / 6.3, 100 3.7 / 6.3, 90 4.3 /
// 6.2, 80 7.2 / 6.3, 64 10.7 / 6.3; a single one of a tenth of the points (1%) 5.9 / 6.3; n
// = 9001, d = 64, the same: 0.115 0.118 0.136 0.183 0.243 and 0.178, against 0.120.
constexpr int kEdmSamples = kEdmSampleBlocks * 16;
constexpr unsigned kEdmGate = 128;
static_assert(kEdmSampleBlocks == 4 * kWave, "four counts a lane");

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x16_t line_mfma(bf16x8_t a, bf16x8_t b, f32x16_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0,
                                                  0, 0);
}

// sum_k (x_ik - x_jk)^2 in the difference form's order
__device__ __forceinline__ float edm_pair(const float *__restrict__ xi, const float *__restrict__ xj, int64_t d) {
    float acc = 0.f;
#pragma unroll 8
    for (int64_t k = 0; k < d; ++k) {
        const float u = xi[k] - xj[k];
        acc = __builtin_fmaf(u, u, acc);
    }
    return acc;
}

// Names a fragment register, so that no use of it moves above the wait before this.
__device__ __forceinline__ void asm_use(bf16x8_t &v) { asm volatile("" : "+v"(v)); }

// Keeps memory accesses in program order here.
__device__ __forceinline__ void mem_order() { asm volatile("" ::: "memory"); }
__device__ __forceinline__ void line_load(const uint4 *src, uint4 *lds) {
    __builtin_amdgcn_global_load_lds(src, lds, 16, 0, 0);
}


// One stage: a 16-wide k block of both panels, [part][row panel 4, column panel 4 + EX]
// 1 KB blocks, five loads a wave (two waves' last repeats their one before).
template <int NP, int CB>
__device__ __forceinline__ void line_issue(uint4 *buf, const uint4 *__restrict__ hi, const uint4 *__restrict__ lo,
                                           int64_t ra, int64_t rc, int64_t rbmax, int64_t KB, int64_t kb, int wave,
                                           int lane) {
    constexpr int PER = 4 + CB, TOT = NP * PER, LPW = (TOT + 3) / 4;
#pragma unroll
    for (int t = 0; t < LPW; ++t) {
        int g = wave + 4 * t;
        g = g < TOT ? g : g - 4;
        const int part = g / PER, b = g % PER;
        int64_t rb = b < 4 ? ra + b : rc + (b - 4);
        rb = rb < 0 ? 0 : rb < rbmax ? rb : rbmax;  // blocks outside the operand: never used
        line_load((part ? lo : hi) + (rb * KB + kb) * 64 + lane, buf + g * 64);
    }
}

// The pairs of one pass (64 rows x 160 columns in LDS) that are marked -1, summed as
// differences: thread (t & 31, t >> 5) takes 5 columns by 8 rows.  Four coordinates of
// the pass's rows and columns at a time go through LDS, a row of X a thread, the next
// four loading meanwhile.
constexpr int kPassRows = 64, kPassStage = kPassRows + kLineCols;
static_assert(kPassStage <= kGramThreads, "a thread stages one row");
__device__ __forceinline__ void edm_pass_diff(float *St, float4 *Cs, const float4 *rowinfo, const float *__restrict__ X,
                                              int64_t n, int64_t d, int64_t ldx, int64_t I0, int64_t J0, int m, int c0,
                                              int t) {
    const int tx = t & 31, ty = t >> 5;
    const bool stage = t < kPassStage;
    int64_t row = t < kPassRows ? I0 + (t >> 5) * 64 + m * 32 + (t & 31) : J0 - 32 + (t - kPassRows);
    row = row < 0 ? 0 : row < n ? row : n - 1;  // rows outside: their pairs are never marked
    const float *src = X + row * ldx;
    auto fetch = [&](int64_t k) {
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (k + 4 <= d) {
            __builtin_memcpy(&v, src + k, 16);  // rows begin at any 4-byte offset
        } else {
            v.x = src[k];
            if (k + 1 < d) v.y = src[k + 1];
            if (k + 2 < d) v.z = src[k + 2];
        }
        return v;
    };
    float acc[8][5];
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 5; ++c) acc[r][c] = 0.f;
    float4 next = make_float4(0.f, 0.f, 0.f, 0.f);
    if (stage) next = fetch(0);
#pragma unroll 1
    for (int64_t k = 0; k < d; k += 4) {
        __syncthreads();
        if (stage) Cs[t] = next;
        __syncthreads();
        if (stage && k + 4 < d) next = fetch(k + 4);
        float4 b[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) b[c] = Cs[kPassRows + tx + 32 * c];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const float4 a = Cs[ty + 8 * r];
#pragma unroll
            for (int c = 0; c < 5; ++c) {
                float u;
                u = a.x - b[c].x; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                u = a.y - b[c].y; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                u = a.z - b[c].z; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                u = a.w - b[c].w; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
            }
        }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int c = 0; c < 5; ++c) {
            const int rr = ty + 8 * r, il = (rr >> 5) * 64 + m * 32 + (rr & 31);
            float *p = St + rr * kLineLd + tx + 32 * c + (__float_as_int(rowinfo[il].w) & 3);
            if (c >= c0 && *p == -1.f) *p = acc[r][c];
        }
}

template <int MAP, bool STATS, bool TILED>
__global__ __launch_bounds__(kGramThreads, 3) void edm_matrix_kernel(MapGeom g, const uint16_t *__restrict__ hi,
                                                                 const uint16_t *__restrict__ lo,
                                                                 const float *__restrict__ norms,
                                                                 const float *__restrict__ inv,
                                                                 const unsigned *__restrict__ near, int64_t n,
                                                                 int64_t dpad, const float *__restrict__ X, int64_t d, int64_t ldx,
                                                                 float *__restrict__ D, unsigned long long *slots) {
    constexpr int T = 128, NP = 2, S = 2, EX = TILED ? 0 : 1, CB = 4 + EX;
    constexpr int PER = 4 + CB, TOT = NP * PER, LPW = (TOT + 3) / 4, BUF = TOT * 64;
    constexpr size_t LDS = S * BUF * 16 > 64 * kLineLd * 4 ? S * BUF * 16 : 64 * kLineLd * 4;
    uint64_t lin;
    int TX, TY;
    if (MAP == MAP_LAMBDA) {
        lin = launch_index();
        if (lin >= g.G) return;
        const uint32_t id = xcd_remap(uint32_t(lin), uint32_t(g.G));
        if (!lambda2(lambda2_patch_to_xfast(id, g.lg, 3, 4), g.lg, g.nb, TX, TY)) return;
        if (SMX_CHECKED && !smx_check(0 <= TX && TX <= TY && TY < g.nb, kCheckMap)) return;
    } else if (!tile2_of<MAP, true>(g, lin, TX, TY)) {
        return;
    }
    __shared__ __attribute__((aligned(16))) uint4 Lb[LDS / 16];
    // per row: norm, -2 / scale, LDS offset of column 0 in its pass, s_i
    __shared__ __attribute__((aligned(16))) float4 rowinfo[T];
    // ... and where its piece begins: in D, and in its LDS row (floats)
    struct __attribute__((aligned(16))) RowOut {
        float *to;
        int from, pad;
    };
    __shared__ RowOut rowout[T];
    __shared__ float nB[kLineCols], iB[kLineCols];
    __shared__ int nflag, flag[kLineList];
    __shared__ float4 Cs[kPassStage];
    auto shift = [&](int il) { return __float_as_int(rowinfo[il].w); };

    const int t = threadIdx.x;
    const int lane = t & 63, w = t >> 6, wm = w >> 1, wn = w & 1;
    const int64_t I0 = int64_t(TX) * T, J0 = int64_t(TY) * T;
    const bool diag = TX == TY;

    auto stats = [&]() {
        if (!STATS) return;
        __shared__ unsigned long long red[2][kGramThreads / kWave];
        unsigned long long cnt, cs;
        tile_pairs_le_stats<kGramThreads>(I0, J0, T, T, n, cnt, cs);
        const unsigned long long c = block_sum<unsigned long long, kGramThreads>(cnt, red[0]);
        const unsigned long long h = block_sum<unsigned long long, kGramThreads>(cs, red[1]);
        if (t == 0) stats_add(slots, lin, c, h);
    };
    const int nst = int(dpad / 16);
    const int64_t KB = dpad / 16, rbmax = gram_rows(n) / 32 - 1;
    const uint4 *hi4 = reinterpret_cast<const uint4 *>(hi), *lo4 = reinterpret_cast<const uint4 *>(lo);
    const int64_t ra = I0 / 32, rc = J0 / 32 - EX;
    auto issue = [&](int st) {
        line_issue<NP, CB>(Lb + (st % S) * BUF, hi4, lo4, ra, rc, rbmax, KB, st, w, lane);
    };
    {
        // the gate, before the ring is touched: its wait costs what the products run no
        // time (n = 65536, d = 64 2.71 / 2.75 ms, gate first / behind the first loads), and the
        // difference tile starts without 36 KB of loads that it drops (6.24 / 6.8)
        const uint4 c4 = reinterpret_cast<const uint4 *>(near)[lane];
        const unsigned c = wave_sum(c4.x + c4.y + c4.z + c4.w);
        if (kEdmGate * c > unsigned(kEdmSamples)) {
            float *As = reinterpret_cast<float *>(Lb);
            static_assert(LDS >= 2 * 128 * kEdmLd * 4, "the difference form's panels fit");
            if ((ldx & 3) == 0 && d % kEdmKc == 0 && (reinterpret_cast<uintptr_t>(X) & 15) == 0)
                edm_diff_tile<8, true, TILED>(As, As + 128 * kEdmLd, TX, TY, X, n, d, ldx, D);
            else
                edm_diff_tile<8, false, TILED>(As, As + 128 * kEdmLd, TX, TY, X, n, d, ldx, D);
            stats();
            return;
        }
    }
    issue(0);
    issue(1);  // d > 16: two stages at least
    const int eoff = int((reinterpret_cast<uintptr_t>(D) >> 2) & 31);
    for (int x = t; x < T; x += kGramThreads) {
        const int64_t i = I0 + x;
        const int64_t a = i * n - (i * (i - 1)) / 2 - i + J0;  // element of column J0
        const int s = TILED ? 0 : int(a + eoff) & 31, r = (x >> 6) * 32 + (x & 31);
        rowinfo[x] = make_float4(i < n ? norms[i] : 0.f, i < n ? -2.f * inv[i] : 0.f,
                                 __int_as_float(r * kLineLd + (s & 3)), __int_as_float(s));
        rowout[x] = {D + (a - s), 32 - (s & ~3), 0};
    }
    for (int x = t; x < kLineCols; x += kGramThreads) {
        const int64_t j = J0 - 32 + x;
        nB[x] = j >= 0 && j < n ? norms[j] : 0.f;
        iB[x] = j >= 0 && j < n ? inv[j] : 0.f;
    }

    // wave (wm, wn): rows 64 wm .., columns 64 wn .. as 2 x 2 products, and of the extra
    // column block the 32 rows 64 wm + 32 wn ..
    f32x16_t acc[2][2], ext;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        ext[e] = 0.f;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int c = 0; c < 2; ++c) acc[m][c][e] = 0.f;
    }
    const uint32_t ring = lds_addr(Lb);
    // a stage's slot is filled again as soon as every wave has its fragments
    for (int st = 0; st < nst; ++st) {
        if (st + 1 < nst) wait_vm<LPW>();
        else wait_vm<0>();
        __builtin_amdgcn_s_barrier();
        const uint32_t cur = ring + uint32_t((st % S) * BUF) * 16u + uint32_t(lane) * 16u;
        bf16x8_t a[NP][2], b[NP][2], x[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const uint32_t at0 = cur + uint32_t(p * PER) * 1024u;
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                a[p][m] = lds_frag(at0 + uint32_t(wm * 2 + m) * 1024u);
                b[p][m] = lds_frag(at0 + uint32_t(4 + EX + wn * 2 + m) * 1024u);
            }
            if constexpr (EX != 0) x[p] = lds_frag(at0 + 4u * 1024u);
        }
        lds_wait<NP, 2>(a, b);
        if constexpr (EX != 0) {
#pragma unroll
            for (int p = 0; p < NP; ++p) asm_use(x[p]);
        }
        __builtin_amdgcn_s_barrier();
        if (st + 2 < nst) issue(st + 2);
#pragma unroll
        for (int q = 0; q < 3; ++q) {  // hi hi, hi lo, lo hi
            const int pa = q == 2, pb = q == 1;
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int c = 0; c < 2; ++c) acc[m][c] = line_mfma(a[pa][m], b[pb][c], acc[m][c]);
            if constexpr (EX != 0) ext = line_mfma(wn ? a[pa][1] : a[pa][0], x[pb], ext);
        }
    }

    // Epilogue, two passes of 64 rows (32 of each half) staged in the idle ring at
    // LDS column 32 + (j - J0) + (s_i mod 4), so that a row's line starts are 16-byte
    // aligned there too.
    float *St = reinterpret_cast<float *>(Lb);
    const bool edge = TILED || TX + 1 >= TY || J0 + T >= n || I0 + T > n;
    // pairs i < j < n: column - row > -dIJ, column below `past`
    const int dIJ = (TY - TX > 1 ? 2 : TY - TX) * T - 32, past = n - J0 < T ? int(n - J0) + 32 : kLineCols;
    __syncthreads();     // rowinfo, nB, iB and at are other threads' work (the k loop's barriers order no LDS writes)
    float nb[3], ib[3];  // this lane's columns: two of the wave's 64, one of the extra block
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int col = c < 2 ? 32 + wn * 64 + c * 32 + (lane & 31) : lane & 31;
        nb[c] = nB[col];
        ib[c] = iB[col];
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        __syncthreads();
        if (t == 0) nflag = 0;
        __syncthreads();
        // FULL: every element is a pair of the tile
        auto rows = [&](auto full) {
            constexpr bool FULL = decltype(full)::value;
            uint32_t left = 0;  // bit e: this lane's row e holds a pair for the list
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int il = wm * 64 + m * 32 + (e & 3) + 4 * (lane >> 5) + 8 * (e >> 2);
                const float4 ri = rowinfo[il];
                float *row = St + __float_as_int(ri.z);
                auto put = [&](int c, int col, float gv) {
                    const float sum = ri.x + nb[c];
                    float v;
                    // (x_i - 2 g) + x_j: one rounding at the sum's size less than the sum first
                    v = __builtin_fmaf(gv * ri.y, ib[c], ri.x) + nb[c];
                    // v >= kEdmNear sum and finite, as one comparison of the difference's bits
                    const uint32_t far = __float_as_uint(__builtin_fmaf(-kEdmNear, sum, v));
                    bool bad = far >= 0x7f800000u;
                    if (!FULL) {
                        const int ij = col - il + dIJ;  // j - i, or above 0 with it
                        v = ij > 0 && col < past ? v : 0.f;
                        bad = bad && ij > 0 && col < past;
                        // the diagonal: exactly 0, or what a point that is not finite gives
                        bad = bad || (ij == 0 && col < past && !(sum < __builtin_inff()));
                    }
                    v = bad ? -1.f : v;  // to be summed as differences
                    left |= uint32_t(bad) << e;
                    row[col] = v;
                };
#pragma unroll
                for (int c = 0; c < 2; ++c) put(c, 32 + wn * 64 + c * 32 + (lane & 31), acc[m][c][e]);
                if (EX && wn == m) put(2, lane & 31, ext[e]);
                mem_order();  // one row's LDS operands at a time
            }
            while (left != 0) {
                const int e = __builtin_ctz(left);
                left &= left - 1;
                const int rl = (e & 3) + 4 * (lane >> 5) + 8 * (e >> 2);
                const int at = __float_as_int(rowinfo[wm * 64 + m * 32 + rl].z);
                for (int c = 0; c < 2 + (EX && wn == m); ++c) {
                    const int col = c < 2 ? 32 + wn * 64 + c * 32 + (lane & 31) : lane & 31;
                    if (St[at + col] == -1.f) {
                        const int f = atomicAdd(&nflag, 1);
                        if (f < kLineList) flag[f] = (wm * 32 + rl) << 8 | col;
                    }
                }
            }
        };
        if (edge) rows(std::false_type{});
        else rows(std::true_type{});
        __syncthreads();
        if (nflag != 0) {
            // pairs to be summed as differences: listed, or too many for the list
            if (nflag <= kLineList) {
                if (t < nflag) {
                    const int r = flag[t] >> 8, col = flag[t] & 255, il = (r >> 5) * 64 + m * 32 + (r & 31);
                    St[r * kLineLd + col + (shift(il) & 3)] = edm_pair(X + (I0 + il) * ldx, X + (J0 - 32 + col) * ldx, d);
                }
            } else {
                edm_pass_diff(St, Cs, rowinfo, X, n, d, ldx, I0, J0, m, 1 - EX, t);
            }
            __syncthreads();
        }
        if (TILED) {
            const uint64_t rank = uint64_t(TY) * (uint64_t(TY) + 1) / 2 + uint64_t(TX);
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const int r = w * 16 + 2 * it + (lane >> 5), cl = 4 * (lane & 31), il = (r >> 5) * 64 + m * 32 + (r & 31);
                float4 v = *reinterpret_cast<const float4 *>(St + r * kLineLd + 32 + cl);
                const int64_t i = I0 + il, j = J0 + cl;
                v.x = i < n && j + 0 < n && j + 0 >= i ? v.x : 0.f;
                v.y = i < n && j + 1 < n && j + 1 >= i ? v.y : 0.f;
                v.z = i < n && j + 2 < n && j + 2 >= i ? v.z : 0.f;
                v.w = i < n && j + 3 < n && j + 3 >= i ? v.w : 0.f;
                store4<true>(D + rank * uint64_t(T * T) + uint64_t(il * T + cl), v);
            }
        } else if (!edge) {
            // a wave writes two rows, four whole lines each, per instruction
            const RowOut *out = rowout + (w >> 1) * 64 + m * 32 + (w & 1) * 16 + (lane >> 5);
            const float *sr = St + (w * 16 + (lane >> 5)) * kLineLd + 4 * (lane & 31);
#pragma unroll
            for (int it = 0; it < 8; ++it) {
                const RowOut o = out[2 * it];
                const float4 v = *reinterpret_cast<const float4 *>(sr + 2 * it * kLineLd + o.from);
                const int il = (w >> 1) * 64 + m * 32 + (w & 1) * 16 + (lane >> 5) + 2 * it;
                const int64_t i = I0 + il, j = J0 - shift(il) + 4 * (lane & 31);
                if (smx_check(i <= j && j + 3 < n, kCheckStore)) store4<true>(o.to + 4 * (lane & 31), v);
            }
        } else {
            for (int q = 0; q < 16; ++q) {
                const int r = w * 16 + q, il = (r >> 5) * 64 + m * 32 + (r & 31), s = shift(il);
                const int64_t i = I0 + il;
                if (i >= n) continue;
                const int64_t first = diag || J0 - s < i ? i : J0 - s, last = J0 + T >= n ? n : J0 + T - s;
                for (int col = lane; col < kLineCols; col += 64) {
                    const int64_t j = J0 - 32 + col;
                    if (j >= first && j < last) rowout[il].to[j - (J0 - s)] = St[r * kLineLd + col + (s & 3)];
                }
            }
        }
    }
    stats();
}

// FP32 operands.  The centre is the mean of eight rows (0 where that is not finite):
// it cancels in every pair, and removes what the points have in common.  Per row the
// centred norm (summed in FP64), the power-of-two scale and the scaled coordinates
// as FP16 hi + lo in fragment order.  2^lgl lanes share a row, eight coordinates a
// lane at a time (in registers between the two uses while d <= 512); a block makes
// 256 >> lgl rows.  The blocks also look at kEdmSampleBlocks x 16 pairs and count those
// that the Gram form would have to leave to differences.
__global__ __launch_bounds__(256) void edm_prep_kernel(const float *__restrict__ X, int64_t n, int64_t d, int64_t ldx,
                                                      int64_t dpad, int64_t npad, int lgl, uint4 *__restrict__ hi,
                                                      uint4 *__restrict__ lo, float *__restrict__ norms,
                                                      float *__restrict__ inv, unsigned *__restrict__ near) {
    extern __shared__ float centre[];  // [d]
    __shared__ unsigned found[16];
    for (int64_t k = threadIdx.x; k < d; k += 256) {
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < 8; ++q) s += X[(q * n / 8) * ldx + k];
        s *= 0.125f;
        centre[k] = __builtin_fabsf(s) < __builtin_inff() ? s : 0.f;
    }
    __syncthreads();
    const int64_t KB = dpad / 16, nq = dpad / 8;
    const int lanes = 1 << lgl, l = int(threadIdx.x) & (lanes - 1);
    const int64_t row = (int64_t(blockIdx.x) << (8 - lgl)) + (threadIdx.x >> lgl);
    const bool in = row < n;
    double x[8];
    auto load8 = [&](int64_t q) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int64_t k = 8 * q + e;
            x[e] = in && k < d ? double(X[row * ldx + k]) - double(centre[k]) : 0.0;
        }
    };
    double acc = 0.0, big = 0.0;
    for (int64_t q = l; q < nq; q += lanes) {
        load8(q);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            acc = __builtin_fma(x[e], x[e], acc);
            const double a = __builtin_fabs(x[e]);
            big = a > big || a != a ? a : big;
        }
    }
    for (int o = lanes / 2; o > 0; o >>= 1) {
        acc += __shfl_xor(acc, o, kWave);
        const double v = __shfl_xor(big, o, kWave);
        big = v > big || v != v ? v : big;
    }
    // c big in [2^13, 2^14): FP16 ends at 2^16.  Not a number where the row is not.
    int ex = 0;
    (void)__builtin_frexp(big, &ex);
    const double c = !(big < double(__builtin_inff())) ? __builtin_nan("") : big == 0.0 ? 1.0 : __builtin_ldexp(1.0, 14 - ex);
    if (row < npad)
        for (int64_t q = l; q < nq; q += lanes) {
            if (nq > lanes) load8(q);
            uint32_t h[4], w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x0 = in ? float(x[2 * e] * c) : 0.f, x1 = in ? float(x[2 * e + 1] * c) : 0.f;
                const _Float16 h0 = _Float16(x0), h1 = _Float16(x1);
                const _Float16 l0 = _Float16(x0 - float(h0)), l1 = _Float16(x1 - float(h1));
                h[e] = uint32_t(__builtin_bit_cast(uint16_t, h0)) | uint32_t(__builtin_bit_cast(uint16_t, h1)) << 16;
                w[e] = uint32_t(__builtin_bit_cast(uint16_t, l0)) | uint32_t(__builtin_bit_cast(uint16_t, l1)) << 16;
            }
            const int64_t slot = ((row >> 5) * KB + (q >> 1)) * 64 + (row & 31) + 32 * (q & 1);
            hi[slot] = make_uint4(h[0], h[1], h[2], h[3]);
            lo[slot] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    if (l == 0 && in) {
        norms[row] = float(acc);
        inv[row] = float(1.0 / c);
    }
    // 16 lanes a sampled pair
    for (int sb = int(blockIdx.x); sb < kEdmSampleBlocks; sb += int(gridDim.x)) {
        const uint64_t z = mix64(uint64_t(sb) * 16 + (threadIdx.x >> 4));
        const int64_t i = int64_t(uint32_t(z) % uint64_t(n)), j = int64_t(uint32_t(z >> 32) % uint64_t(n));
        double s = 0.0, g = 0.0;
        for (int64_t k = threadIdx.x & 15; k < d; k += 16) {
            const double m = centre[k], a = double(X[i * ldx + k]) - m, b = double(X[j * ldx + k]) - m;
            s += a * a + b * b;
            g += (a - b) * (a - b);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            s += __shfl_xor(s, o, kWave);
            g += __shfl_xor(g, o, kWave);
        }
        if ((threadIdx.x & 15) == 0) found[threadIdx.x >> 4] = i != j && !(g >= double(kEdmNear) * s) ? 1u : 0u;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned f = 0;
            for (int q = 0; q < 16; ++q) f += found[q];
            near[sb] = f;
        }
        __syncthreads();
    }
}

int launch_edm_prep(const float *X, int64_t n, int64_t d, int64_t ldx, int64_t dpad, unsigned *near, uint16_t *hi,
                    uint16_t *lo, float *norms, float *inv, hipStream_t s) {
    const int64_t npad = gram_rows(n);
    int lgl = 2;  // lanes a row: one per eight coordinates, 4 to 64
    while (lgl < 6 && (int64_t(1) << lgl) < dpad / 8) ++lgl;
    const int64_t rows = 256 >> lgl;
    prof_begin(K_GRAM_PREP, s);
    hipLaunchKernelGGL(edm_prep_kernel, dim3(uint32_t((npad + rows - 1) / rows)), dim3(256), size_t(d) * 4, s, X, n, d, ldx,
                       dpad, npad, lgl, reinterpret_cast<uint4 *>(hi), reinterpret_cast<uint4 *>(lo), norms, inv, near);
    prof_end(K_GRAM_PREP, s);
    return check_launch("edm prep");
}

template <int MAP, bool TILED>
static void go_lines(const MapGeom &g, const uint16_t *hi, const uint16_t *lo, const float *norms, const float *inv,
                     const unsigned *near, int64_t n, int64_t dpad, const float *X, int64_t d, int64_t ldx, float *D, unsigned long long *slots,
                     hipStream_t s) {
    const dim3 grid = MAP == MAP_BBOX ? dim3(g.nb, g.nb, 1) : grid_for(g.G, kGramThreads);
    if (slots)
        hipLaunchKernelGGL((edm_matrix_kernel<MAP, true, TILED>), grid, dim3(kGramThreads), 0, s, g, hi, lo, norms,
                           inv, near, n, dpad, X, d, ldx, D, slots);
    else
        hipLaunchKernelGGL((edm_matrix_kernel<MAP, false, TILED>), grid, dim3(kGramThreads), 0, s, g, hi, lo, norms,
                           inv, near, n, dpad, X, d, ldx, D, slots);
}

int launch_edm_matrix(const MapGeom &g, const uint16_t *hi, const uint16_t *lo, const float *norms, const float *inv,
                      const unsigned *near, int64_t n, int64_t dpad, const float *X, int64_t d, int64_t ldx, float *D,
                      unsigned long long *slots, bool tiled, hipStream_t s) {
    prof_begin(K_EDM_DIFF, s);
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        constexpr int MAPK = decltype(M)::value;
        if (tiled) go_lines<MAPK, true>(gg, hi, lo, norms, inv, near, n, dpad, X, d, ldx, D, slots, s);
        else go_lines<MAPK, false>(gg, hi, lo, norms, inv, near, n, dpad, X, d, ldx, D, slots, s);
    });
    prof_end(K_EDM_DIFF, s);
    return check_launch("edm_packed (fp32, matrix form)");
}

SMX_CHECK_READER(check_flags_gram)

}  // namespace smx
