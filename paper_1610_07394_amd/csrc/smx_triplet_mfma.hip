// Axilrod-Teller energy and gradient as matrix products (paper Sec. I: the
// triple-interaction n-body problem), for the matrix cores.
//
// With the dipole tensors of the pairs, T_ij = 3 x x^T / r^5 - 1 / r^3 with
// x = x_i - x_j (symmetric, traceless), a triplet's energy is
//   E_t = nu (1 + 3 cos cos cos) / (r r r)^3 = -(nu / 3) tr(T_ij T_jk T_ki):
// expand the product of unit vectors, and use cos^2 A + cos^2 B + cos^2 C =
// 1 - 2 cos A cos B cos C for the angles of a triangle.  tr(ABC) is symmetric
// in three symmetric matrices, so it is the polarised form of the cubic
// tr(A^3), and a way to write that cubic on traceless A as a sum of cubes of
// linear forms, tr(A^3) = sum_r l_r(A)^3, splits the trace into scalars:
//   tr(T_ij T_jk T_ki) = sum_r l_r(T_ij) l_r(T_jk) l_r(T_ki).
// With L_r the symmetric n x n matrix of l_r(T_ij) (zero diagonal) and
// S_r = L_r L_r^T, everything about triplets is in the ten S_r:
//   E        = -(nu / 9) sum_{i<j} sum_r l_r(T_ij) S_r,ij
//   dE/dx_i  = -(nu / 3) sum_{j != i} sum_r S_r,ij grad l_r(T_ij).
// The energy alone takes each triplet once: with the strictly upper part U_r of
// L_r, E = -(nu / 3) sum_{i<j} sum_r l_r(T_ij) (U_r U_r^T)_ij, a third of the
// products.
//
// Precision.  l_r(T) is evaluated in FP64 and held as an FP16 pair hi + lo (22
// bits and the sign of lo: 2^-23), each row scaled by a power of two so that its
// nearest neighbour's T is near 2^13.  FP16 ends at 2^-24 below, so entries of a row at
// more than about 30 times the distance of its nearest are held to some 2^-38 (r / r_min)^3
// instead: what a very close pair gets from the rest (its mutual S) loses that much.
// S = hi hi^T + hi lo^T + lo hi^T with exact products and FP32 accumulation in one or two
// levels (at_pair_kernel), and the forces of the pairs are formed in FP64.
// Relative error of the Axilrod-Teller gradient alone (2-norm), particles at 0.8 to 1
// apart: n = 800 3.2e-7, 2051 3.4e-7, 8192 1.3e-6, of the FP32 triplet loop 9.5e-7,
// 1.2e-6, 1.6e-6; its energy 1e-8 against 1e-7.  One pair at 0.1 / 0.01 / 0.003 of the
// spacing, n = 1100: 1.8e-6, 1.2e-5, 2.0e-4 against 1.9e-4, 5.2e-3, 0.13.
#include <type_traits>
#include <utility>

#include "smx_at_forms.h"
#include "smx_device.h"
#include "smx_internal.h"

namespace smx {

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// The least r^2 of each row (the nearest neighbour), kept as the complement of the
// float's bits so that an integer maximum over zeroed words finds it.  64 columns
// a block, so that small n fill the chip.
constexpr int kNearThreads = 256, kNearCols = 64;
__global__ __launch_bounds__(kNearThreads) void at_nearest_kernel(const float *__restrict__ X, int64_t n, int64_t ldx,
                                                                  unsigned *__restrict__ near) {
    __shared__ float4 P[kNearCols];
    const int t = threadIdx.x;
    const int64_t i = int64_t(blockIdx.x) * kNearThreads + t, k0 = int64_t(blockIdx.y) * kNearCols;
    if (t < kNearCols && k0 + t < n)
        P[t] = make_float4(X[(k0 + t) * ldx], X[(k0 + t) * ldx + 1], X[(k0 + t) * ldx + 2], 0.f);
    const int64_t ii = i < n ? i : n - 1;
    const float x = X[ii * ldx], y = X[ii * ldx + 1], z = X[ii * ldx + 2];
    __syncthreads();
    if (i >= n) return;
    const int m = int(n - k0 < kNearCols ? n - k0 : kNearCols);
    unsigned best = 0;
#pragma unroll 8
    for (int k = 0; k < m; ++k) {
        const float4 p = P[k];
        const float dx = p.x - x, dy = p.y - y, dz = p.z - z;
        const float s = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
        const unsigned b = k0 + k == i ? 0u : ~__float_as_uint(s);
        best = b > best ? b : best;
    }
    atomicMax(near + i, best);
}

// How many of 256 rows have a neighbour much nearer than the rest: 1 / r_min^3 above a
// fifth of sum_k 1 / r^3.  (A liquid's rows, the nearest other at 0.8 of the spacing, have
// 0.05 to 0.15, a bond of half the spacing 0.2, of 0.3 of it 0.45.)  A wave a row, kShortBlocks
// counts.
constexpr int kShortBlocks = kWave, kShortRows = kShortBlocks * 4, kShortMax = 2;
__global__ __launch_bounds__(256) void at_short_kernel(const float *__restrict__ X, int64_t n, int64_t ldx,
                                                      unsigned *__restrict__ found) {
    __shared__ unsigned red[4];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t i = int64_t(mix64(uint64_t(blockIdx.x) * 4 + uint64_t(w)) % uint64_t(n));
    const float x = X[i * ldx], y = X[i * ldx + 1], z = X[i * ldx + 2];
    float most = 0.f, sum = 0.f;
#pragma unroll 4
    for (int64_t k = lane; k < n; k += kWave) {
        const float dx = X[k * ldx] - x, dy = X[k * ldx + 1] - y, dz = X[k * ldx + 2] - z;
        const float d = __builtin_amdgcn_rsqf(__builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)));
        const float d3 = k == i ? 0.f : d * d * d;
        most = d3 > most ? d3 : most;
        sum += d3;
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
        const float m = __shfl_xor(most, o, kWave);
        most = m > most ? m : most;
        sum += __shfl_xor(sum, o, kWave);
    }
    if (lane == 0) red[w] = most <= 0.2f * sum ? 0u : 1u;
    __syncthreads();
    if (threadIdx.x == 0) found[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Row scale c, a power of two with c / r_min^3 in (2^12, 2^14] (a form is at
// most 2.8 / r^3 and FP16 ends at 2^16).  NaN where a pair coincides or the row's
// position is no number: every result that the row takes part in is then NaN.
__device__ __forceinline__ double at_row_scale(unsigned near) {
    const float s = __uint_as_float(~near);
    if (near == 0u || s == __builtin_inff()) return 1.0;  // no neighbour within FP32's range
    if (!(s > 0.f)) return __builtin_nan("");
    int e;
    (void)__builtin_frexpf(s, &e);  // s >= 2^(e - 1), so 1 / r^3 <= 2^(-3 (e - 1) / 2)
    const int h = 3 * (e - 1);
    return __builtin_ldexp(1.0, 14 + (h >= 0 ? h / 2 : -((1 - h) / 2)));
}

// 1 / sqrt(s) to 2^-43: the FP32 instruction and one Newton step.
__device__ __forceinline__ double rsqrt_f64(double s) {
    double y = double(__builtin_amdgcn_rsqf(float(s)));
    const double h = 0.5 * s;
    return y * __builtin_fma(-h * y, y, 1.5);
}

// Operand panels in matrix-core order: panel (r, part) of the rows of all
// particles and the k of one chunk, 1 KB blocks of 32 rows x 16 k, slot s of a
// block = row 32 rb + (s & 31), k = 16 kb + 8 (s >> 5) .. + 7 (what lane s of
// v_mfma_f32_32x32x16_f16 reads).  One wave makes one block of every panel of the
// launch's forms.  upper: entries with k <= row are 0, and blocks left of their
// row's tile (tmask + 1 rows), which are not read, are left out.
template <int NR>
__global__ __launch_bounds__(256) void at_forms_kernel(const float *__restrict__ X, int64_t n, int64_t ldx,
                                                      const unsigned *__restrict__ near, int r0, int64_t k0, int KB,
                                                      int RB, int upper, int tmask, uint4 *__restrict__ ops) {
    const int lane = threadIdx.x & 63;
    const int kb = int(blockIdx.x) * 4 + int(threadIdx.x >> 6), rb = int(blockIdx.y);
    if (kb >= KB) return;
    const int64_t i = int64_t(rb) * 32 + (lane & 31), kf = k0 + 16 * int64_t(kb) + 8 * (lane >> 5);
    if (upper && k0 + 16 * int64_t(kb) + 15 < ((int64_t(rb) * 32) & ~int64_t(tmask))) return;
    const bool row = i < n;
    double x = 0, y = 0, z = 0, c3 = 0;
    if (row) {
        x = X[i * ldx];
        y = X[i * ldx + 1];
        z = X[i * ldx + 2];
        c3 = 3.0 * at_row_scale(near[i]);
    }
    uint32_t hi[NR][4], lo[NR][4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float f[NR][2];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int64_t k = kf + 2 * q + p;
            const bool on = row && k < n && (upper ? k > i : k != i);
            const int64_t kk = k < n ? k : n - 1;
            const double dx = x - double(X[kk * ldx]), dy = y - double(X[kk * ldx + 1]),
                         dz = z - double(X[kk * ldx + 2]);
            const double xx = dx * dx, yy = dy * dy, zz = dz * dz, s = xx + yy + zz;
            const double d = rsqrt_f64(on ? s : 1.0), d2 = d * d, w = on ? (d2 * d2) * (d * c3) : 0.0;
            const double Z = w * (zz - s * (1.0 / 3.0)), u = w * (0.5 * (xx - yy)), v = w * (dx * dy),
                         sxz = w * (dx * dz), t = w * (dy * dz);
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const double *m = kAtForm[r0 + r];
                const double l = __builtin_fma(m[0], Z, __builtin_fma(m[1], u, __builtin_fma(m[2], v, __builtin_fma(m[3], sxz, m[4] * t))));
                f[r][p] = on ? float(l) : 0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const _Float16 h0 = _Float16(f[r][0]), h1 = _Float16(f[r][1]);
            const _Float16 l0 = _Float16(f[r][0] - float(h0)), l1 = _Float16(f[r][1] - float(h1));
            hi[r][q] = uint32_t(__builtin_bit_cast(uint16_t, h0)) | uint32_t(__builtin_bit_cast(uint16_t, h1)) << 16;
            lo[r][q] = uint32_t(__builtin_bit_cast(uint16_t, l0)) | uint32_t(__builtin_bit_cast(uint16_t, l1)) << 16;
        }
    }
    const size_t panel = size_t(RB) * size_t(KB) * 64, at = (size_t(rb) * size_t(KB) + size_t(kb)) * 64 + size_t(lane);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        ops[(2 * r) * panel + at] = make_uint4(hi[r][0], hi[r][1], hi[r][2], hi[r][3]);
        ops[(2 * r + 1) * panel + at] = make_uint4(lo[r][0], lo[r][1], lo[r][2], lo[r][3]);
    }
}

// s_waitcnt with vmcnt <= N and no wait on the other counters; the ring's loads
// complete in issue order.
template <int N>
__device__ __forceinline__ void wait_loads() {
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
// One wave moves 1 KB from global memory to LDS, 16 bytes a lane.
__device__ __forceinline__ void load_block(const uint4 *src, uint4 *lds) {
    __builtin_amdgcn_global_load_lds(src, lds, 16, 0, 0);
}

// An operand fragment from the ring.  Written out, because the compiler does not
// model the LDS writes of the global-to-LDS loads; frags_wait waits for it and
// names the registers, so that no use moves above the wait.
template <int OFF>
__device__ __forceinline__ f16x8_t frag(uint32_t addr) {
    static_assert(OFF >= 0 && OFF < 65536, "16-bit offset");
    f16x8_t v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
    return v;
}

template <int MR, int MC>
struct Frags {
    f16x8_t a[2][MR], b[2][MC];
};
// Fragment K of a step: the hi fragments first, then the lo ones.
template <int K, int MR, int MC, int RB>
__device__ __forceinline__ void read_frag(uint32_t a, uint32_t b, Frags<MR, MC> &f) {
    constexpr int p = K / (MR + MC), i = K % (MR + MC);
    if constexpr (i < MC) f.b[p][i] = frag<((2 + p) * RB + i) * 1024>(b);
    else f.a[p][i - MC] = frag<(p * RB + i - MC) * 1024>(a);
}
template <int MR, int MC, int RB, int... K>
__device__ __forceinline__ void read_frags(uint32_t a, uint32_t b, Frags<MR, MC> &f, std::integer_sequence<int, K...>) {
    (read_frag<K, MR, MC, RB>(a, b, f), ...);
}
// Product K of a step (hi hi, hi lo, lo hi over the wave's MR x MC tiles), and
// behind it one of the next step's fragment reads: issued in one go the reads
// would hold the products back until the LDS had taken them all.
template <int K, int MR, int MC, int RB>
__device__ __forceinline__ void product(const Frags<MR, MC> &f, f32x16_t (&acc)[MR][MC], uint32_t a, uint32_t b,
                                        Frags<MR, MC> &nxt) {
    constexpr int q = K / (MR * MC), m = K / MC % MR, c = K % MC;
    acc[m][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(f.a[q == 2][m], f.b[q == 1][c], acc[m][c], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (K < 2 * (MR + MC)) {
        read_frag<K, MR, MC, RB>(a, b, nxt);
        __builtin_amdgcn_sched_barrier(0);
    }
}
template <int MR, int MC, int RB, int... K>
__device__ __forceinline__ void products(const Frags<MR, MC> &f, f32x16_t (&acc)[MR][MC], uint32_t a, uint32_t b,
                                         Frags<MR, MC> &nxt, std::integer_sequence<int, K...>) {
    (product<K, MR, MC, RB>(f, acc, a, b, nxt), ...);
}
template <int MR, int MC>
__device__ __forceinline__ void frags_wait(Frags<MR, MC> &f) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int m = 0; m < MR; ++m) asm volatile("" : "+v"(f.a[p][m]));
#pragma unroll
        for (int c = 0; c < MC; ++c) asm volatile("" : "+v"(f.b[p][c]));
    }
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
// Sum over the 16 lanes of a row; every lane gets it.
__device__ __forceinline__ float row16_sum(float v) {
    v += dpp<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp<0x124>(v);  // row_ror:4
    v += dpp<0x128>(v);  // row_ror:8
    return v;
}

// Keep v's value and the memory accesses around here in program order.
__device__ __forceinline__ void pin(double &v) { asm volatile("" : "+v"(v) : : "memory"); }

// One particle of a tile as the epilogue reads it: position, M_r x, 1 / row scale.
struct AtSide {
    double x, y, z, qx, qy, qz, ic, pad;
};

// WR x WC waves of MR x MC products of 32 x 32 each: T x T pairs a block.
// T = 256 (8 waves, 128 accumulators a lane, one block a CU): per 16-wide k step a
// CU reads 96 KB of fragments and writes 32 KB of staging in LDS against 1536
// cycles of products on each SIMD, 65% of what LDS moves in that time.  T = 128 (4
// waves, 64 accumulators, two blocks a CU) needs 95% of it but makes four times as
// many blocks, which fill the chip at smaller n.  Gradient, ms, T = 256 / 128: n =
// 2051 0.40 / 0.37, 3000 1.02 / 0.94, 4096 2.07 / 2.09, 8192 13.8 / 15.9; energy:
// 3000 0.45 / 0.39, 6000 2.41 / 2.30, 8192 6.0 / 6.5.  256 x 128 (two blocks a CU,
// 3 slots) 16.1 and 128 x 128 of two waves 18.9 at n = 8192; a barrier every other
// step changed nothing.  At n = 8192 the matrix cores are busy 0.74 of the time,
// at a clock (1.6 GHz) that the board's power sets: a plain library product of
// 8192^3 reaches 1.5 PFLOP/s here, this kernel 1.2 with its epilogue.
template <int WR, int WC, int MR, int MC>
struct AtTile {
    static constexpr int NW = WR * WC, NT = 64 * NW, T = 32 * WR * MR, RB = T / 32;
    static constexpr int S = 4;             // ring slots
    // sums in two levels (see at_pair_kernel): where the registers hold a second set
    static constexpr bool TWO = MR * MC <= 4;
    static constexpr int STAGE = 4 * RB;    // 1 KB blocks per slot: row panel hi, lo, column panel hi, lo
    static constexpr int LPW = STAGE / NW;  // loads per wave per slot
    static_assert(T == 32 * WC * MC && STAGE % NW == 0, "square tiles");
    static_assert(size_t(S) * STAGE * 1024 >= size_t(2 * T) * sizeof(AtSide) + size_t(2 * WC + 2 * WR) * T * 12,
                  "the epilogue's data fit the ring");
};

// One block: form r of the pairs of one T x T tile (I, J), all k of the chunk;
// then the pairs' share of the energy and of the gradient.  The map orders the
// pair tiles; blocks are dealt to the XCDs in runs (xcd_deal), whose blocks share
// row and column panels in one L2 (0.75 of the reads hit it at n = 8192).
//
// The FP32 sums over k.  Where one term is far above the others, as two particles much
// nearer to each other than to the rest make it (a bond), the many small products of one
// sign that come after it fall below half an ulp of the sum and are lost, and the energy,
// in which the bonds' own terms largely cancel, collects that loss: n = 8192, pairs at
// 0.3 / 0.2 of the spacing, 7.9e-6 / 2.2e-5 of E against 8.7e-7 / 2.3e-6 by the triplet
// loop.  Tiles of 128 therefore sum 512 k at a time and add those up, for which they
// have the registers (n = 2051 0.350 ms, without 0.346).  Tiles of 256 have not: found
// (given when both sizes are launched) counts sampled rows with such a neighbour, and
// more than kShortMax of 256 send the call to the smaller tiles, which then sum 128 k at
// a time (3.8e-7 / 8.0e-7, with 512 k 7.0e-7 / 2.1e-6; 16.2 and 15.8 ms instead of 13.9,
// the loop 52.7).
template <int MAP, int WR, int WC, int MR, int MC, bool GRAD>
__global__ __launch_bounds__(64 * WR * WC, 2) void at_pair_kernel(
    MapGeom g, int nr, int r0, const uint4 *__restrict__ ops, int KB, int RB, int64_t k0, const float *__restrict__ X,
    int64_t n, int64_t ldx, const unsigned *__restrict__ near, const unsigned *__restrict__ found, double nu,
    double *__restrict__ G64, double *__restrict__ eslots) {
    using C = AtTile<WR, WC, MR, MC>;
    constexpr int T = C::T, S = C::S, LPW = C::LPW;
    if (found != nullptr && (wave_sum(found[threadIdx.x & (kWave - 1)]) > unsigned(kShortMax)) != C::TWO) return;
    const uint64_t task0 = launch_index(), ntask = g.G * uint64_t(nr);
    if (task0 >= ntask) return;
    // the energy's tiles differ in depth, so its runs are shorter (n = 8192: 6.3 -> 6.0 ms)
    const uint32_t task = xcd_deal(uint32_t(task0), uint32_t(ntask), GRAD ? 5 : 3);
    const uint32_t r = task / uint32_t(g.G), id = task - r * uint32_t(g.G);
    int TX, TY;
    if (MAP == MAP_LAMBDA) {
        if (!lambda2(lambda2_patch_to_xfast(id, g.lg, 2, 3), g.lg, g.nb, TX, TY)) return;
        if (SMX_CHECKED && !smx_check(0 <= TX && TX <= TY && TY < g.nb, kCheckMap)) return;
    } else {
        uint64_t lin;
        if (!tile2_of_id<MAP>(g, id, lin, TX, TY)) return;
    }
    const int64_t I0 = int64_t(TX) * T, J0 = int64_t(TY) * T;
    // the energy's operand is 0 for k <= j: its k loop starts at the column tile
    int kb0 = 0;
    if (!GRAD) {
        if (J0 > k0) kb0 = int((J0 - k0) / 16 < KB ? (J0 - k0) / 16 : KB);
        if (kb0 >= KB) return;
    }
    const int nst = KB - kb0;

    __shared__ __attribute__((aligned(16))) uint4 ring[S * C::STAGE * 64];
    __shared__ double red[C::NW];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = w / WC, wn = w % WC;

    // this wave's share of a slot: LPW blocks, each one contiguous 1 KB per k step
    const size_t panel = size_t(RB) * size_t(KB) * 64;
    const uint4 *src[LPW];
#pragma unroll
    for (int q = 0; q < LPW; ++q) {
        const int b = w + C::NW * q, side = b / (2 * C::RB), lo = (b / C::RB) & 1;
        int64_t rb = (side ? J0 : I0) / 32 + b % C::RB;
        rb = rb < RB ? rb : RB - 1;  // past the last row block of a ragged tile: never used
        src[q] = ops + size_t(2 * r + lo) * panel + (size_t(rb) * KB + kb0) * 64 + lane;
    }
    auto issue = [&](int st) {
#pragma unroll
        for (int q = 0; q < LPW; ++q)
            load_block(src[q] + size_t(st) * 64, ring + size_t(st % S) * (C::STAGE * 64) + (w + C::NW * q) * 64);
    };
    // this wave's fragments: A rows from block wm MR, B rows from block wn MC
    const uint32_t baseA = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ring)) + uint32_t(wm * MR * 1024 + lane * 16);
    const uint32_t baseB = baseA + uint32_t((wn * MC - wm * MR) * 1024);
    f32x16_t acc[MR][MC];
#pragma unroll
    for (int m = 0; m < MR; ++m)
#pragma unroll
        for (int c = 0; c < MC; ++c)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[m][c][e] = 0.f;
    f32x16_t sum[C::TWO ? MR : 1][C::TWO ? MC : 1];
    const int chunk = found != nullptr ? 8 : 32;  // k steps
    if constexpr (C::TWO) {
#pragma unroll
        for (int m = 0; m < MR; ++m)
#pragma unroll
            for (int c = 0; c < MC; ++c) sum[m][c] = acc[m][c];
    }
    // Ring: slots st .. st + S - 1 are filled or in flight.  A step multiplies the
    // fragments of step st from registers while it reads those of st + 1 (the last
    // one reads a stale slot that nothing uses).  At its barrier every wave holds st
    // in registers, so that st's slot is free for st + S, and has seen its own loads
    // of st + 1 land.
    for (int p = 0; p < S && p < nst; ++p) issue(p);
    Frags<MR, MC> f0, f1;
    if (nst >= S) wait_loads<(S - 1) * LPW>();
    else wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    read_frags<MR, MC, C::RB>(baseA, baseB, f0, std::make_integer_sequence<int, 2 * (MR + MC)>{});
    frags_wait(f0);
    auto step = [&](int st, const Frags<MR, MC> &cur, Frags<MR, MC> &nxt) {
        if (st + S <= nst) wait_loads<(S - 2) * LPW>();
        else wait_loads<0>();
        __builtin_amdgcn_s_barrier();
        if (st + S < nst) issue(st + S);
        const uint32_t at = uint32_t((st + 1) % S) * uint32_t(C::STAGE * 1024);
        products<MR, MC, C::RB>(cur, acc, baseA + at, baseB + at, nxt, std::make_integer_sequence<int, 3 * MR * MC>{});
        frags_wait(nxt);
    };
    for (int st = 0; st < nst; st += 2) {  // nst is even
        step(st, f0, f1);
        step(st + 1, f1, f0);
        if constexpr (C::TWO) {
            if (st + 2 == nst || ((st + 2) & (chunk - 1)) == 0) {
#pragma unroll
                for (int m = 0; m < MR; ++m)
#pragma unroll
                    for (int c = 0; c < MC; ++c)
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            sum[m][c][e] += acc[m][c][e];
                            acc[m][c][e] = 0.f;
                        }
            }
        }
    }
    if constexpr (C::TWO) {
#pragma unroll
        for (int m = 0; m < MR; ++m)
#pragma unroll
            for (int c = 0; c < MC; ++c) acc[m][c] = sum[m][c];
    }
    __syncthreads();

    // ---- the pairs of the tile
    AtSide *side = reinterpret_cast<AtSide *>(ring);
    float *Frow = reinterpret_cast<float *>(side + 2 * T);  // [2 WC][T][3]
    float *Fcol = Frow + 2 * WC * T * 3;                    // [2 WR][T][3]
    const double *m = kAtForm[r0 + int(r)];
    const double mxx = 0.5 * m[1] - m[0] * (1.0 / 3.0), myy = -0.5 * m[1] - m[0] * (1.0 / 3.0),
                 mzz = m[0] * (2.0 / 3.0), mxy = 0.5 * m[2], mxz = 0.5 * m[3], myz = 0.5 * m[4];
    for (int q = t; q < 2 * T; q += C::NT) {
        const int64_t p = (q < T ? I0 : J0) + (q & (T - 1));
        AtSide v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (p < n) {
            v.x = X[p * ldx];
            v.y = X[p * ldx + 1];
            v.z = X[p * ldx + 2];
            v.ic = 1.0 / at_row_scale(near[p]);
            v.qx = mxx * v.x + mxy * v.y + mxz * v.z;
            v.qy = mxy * v.x + myy * v.y + myz * v.z;
            v.qz = mxz * v.x + myz * v.y + mzz * v.z;
        }
        side[q] = v;
    }
    __syncthreads();
    const int half = lane >> 5, cl = lane & 31;
    const uint32_t i0 = uint32_t(I0), j0 = uint32_t(J0), un = uint32_t(n);  // below 2^31
    double e = 0.0;
    double fj[MC][3];
    AtSide B[MC];
#pragma unroll
    for (int c = 0; c < MC; ++c) {
        B[c] = side[T + wn * (32 * MC) + c * 32 + cl];
        fj[c][0] = fj[c][1] = fj[c][2] = 0.0;
    }
    auto pairs = [&](auto full) {
    constexpr bool FULL = decltype(full)::value;
#pragma unroll
    for (int mm = 0; mm < MR; ++mm) {
#pragma unroll
        for (int el = 0; el < 16; ++el) {
            const int il = wm * (32 * MR) + mm * 32 + (el & 3) + 8 * (el >> 2) + 4 * half;
            const AtSide A = side[il];
            double gx = 0, gy = 0, gz = 0;
#pragma unroll
            for (int c = 0; c < MC; ++c) {
                const int jl = wn * (32 * MC) + c * 32 + cl;
                const bool on = FULL || (i0 + il < j0 + jl && j0 + jl < un);
                const double dx = A.x - B[c].x, dy = A.y - B[c].y, dz = A.z - B[c].z;
                const double s2 = on ? __builtin_fma(dx, dx, __builtin_fma(dy, dy, dz * dz)) : 1.0;
                const double sv = on ? double(acc[mm][c][el]) * (A.ic * B[c].ic) : 0.0;
                const double d = rsqrt_f64(s2), d2 = d * d;
                const double qx = A.qx - B[c].qx, qy = A.qy - B[c].qy, qz = A.qz - B[c].qz;
                const double xq = __builtin_fma(dx, qx, __builtin_fma(dy, qy, dz * qz));
                const double w5 = 3.0 * sv * (d2 * d2 * d);  // l = 3 d^5 x.Mx
                e = __builtin_fma(w5, xq, e);
                if (GRAD) {
                    // grad l = 6 d^5 Mx - 15 d^7 (x.Mx) x
                    const double a = 2.0 * w5, b = -5.0 * w5 * (xq * d2);
                    const double hx = __builtin_fma(a, qx, b * dx), hy = __builtin_fma(a, qy, b * dy),
                                 hz = __builtin_fma(a, qz, b * dz);
                    gx += hx;
                    gy += hy;
                    gz += hz;
                    fj[c][0] += hx;
                    fj[c][1] += hy;
                    fj[c][2] += hz;
                }
            }
            if (GRAD) {
                const float sx = row16_sum(float(gx)), sy = row16_sum(float(gy)), sz = row16_sum(float(gz));
                const int l16 = lane & 15;
                const float v = l16 == 0 ? sx : l16 == 1 ? sy : sz;
                if (l16 < 3) Frow[((2 * wn + ((lane >> 4) & 1)) * T + il) * 3 + l16] = v;
            }
            // one row at a time: without this the compiler loads all 16 MR rows first and spills
            pin(e);
            if (GRAD) {
#pragma unroll
                for (int c = 0; c < MC; ++c)
#pragma unroll
                    for (int q = 0; q < 3; ++q) pin(fj[c][q]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    };
    // every pair of a tile off the diagonal and inside n is one
    if (TX < TY && J0 + T <= n) pairs(std::true_type{});
    else pairs(std::false_type{});
    if (GRAD) {
#pragma unroll
        for (int c = 0; c < MC; ++c)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                Fcol[((2 * wm + half) * T + wn * (32 * MC) + c * 32 + cl) * 3 + q] = float(fj[c][q]);
    }
    const double eb = block_sum<double, C::NT>(e, red);  // synchronises the block
    if (t == 0) atomicAdd(eslots + (task0 % kSlots) * kSlotStride + 0, eb * (GRAD ? -nu / 9.0 : -nu / 3.0));
    if (GRAD) {
        const double sc = -nu / 3.0;
        for (int q = t; q < 3 * T; q += C::NT) {
            double a = 0.0, b = 0.0;
#pragma unroll
            for (int p = 0; p < 2 * WC; ++p) a += double(Frow[p * T * 3 + q]);
#pragma unroll
            for (int p = 0; p < 2 * WR; ++p) b += double(Fcol[p * T * 3 + q]);
            if (I0 + q / 3 < n) atomicAdd(G64 + 3 * I0 + q, sc * a);
            if (J0 + q / 3 < n) atomicAdd(G64 + 3 * J0 + q, -sc * b);
        }
    }
}

template <int MAP, int WR, int WC, int MR, int MC, bool GRAD>
static void go_pairs(const MapGeom &g, int nr, int r0, const uint4 *ops, int KB, int RB, int64_t k0, const float *X,
                     int64_t n, int64_t ldx, const unsigned *near, const unsigned *found, double nu, double *G64,
                     double *eslots, hipStream_t s) {
    using C = AtTile<WR, WC, MR, MC>;
    hipLaunchKernelGGL((at_pair_kernel<MAP, WR, WC, MR, MC, GRAD>), grid_for(g.G * uint64_t(nr), C::NT), dim3(C::NT),
                       0, s, g, nr, r0, ops, KB, RB, k0, X, n, ldx, near, found, nu, G64, eslots);
}

template <int NR>
static void go_forms(const float *X, int64_t n, int64_t ldx, const unsigned *near, int r0, int64_t k0, int KB, int RB,
                     bool upper, int tile, uint4 *ops, hipStream_t s) {
    hipLaunchKernelGGL(at_forms_kernel<NR>, dim3(uint32_t((KB + 3) / 4), uint32_t(RB)), dim3(256), 0, s, X, n, ldx,
                       near, r0, k0, KB, RB, int(upper), tile - 1, ops);
}

// The pair tiles of edge TILE, of every form in ops.
template <int TILE, bool GRAD, typename... Args>
static void go_tiles(const MapGeom &g, Args... args) {
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        constexpr int MAPK = decltype(M)::value;
        if constexpr (TILE == 256) go_pairs<MAPK, 2, 4, 4, 2, GRAD>(gg, args...);
        else go_pairs<MAPK, 2, 2, 2, 2, GRAD>(gg, args...);
    });
}

int launch_triplet_mfma(const MapGeom &g, const MapGeom *g256, const AtPlan &plan, const float *X, int64_t n, int64_t ldx,
                        float nu, bool grad, double *G64, double *eslots, unsigned *near, unsigned *found, void *ops_,
                        hipStream_t s) {
    uint4 *ops = reinterpret_cast<uint4 *>(ops_);
    const int kid = grad ? K_TRIP_GRAD : K_TRIP_ENERGY;
    const int RB = int((n + 31) / 32), tile = g256 != nullptr ? 256 : 128;
    prof_begin(kid, s);
    hipLaunchKernelGGL(at_nearest_kernel,
                       dim3(uint32_t((n + kNearThreads - 1) / kNearThreads), uint32_t((n + kNearCols - 1) / kNearCols)),
                       dim3(kNearThreads), 0, s, X, n, ldx, near);
    if (g256 != nullptr) hipLaunchKernelGGL(at_short_kernel, dim3(kShortBlocks), dim3(256), 0, s, X, n, ldx, found);
    else found = nullptr;
    for (int64_t k0 = 0; k0 < n; k0 += plan.kc) {
        const int64_t kn = n - k0 < plan.kc ? n - k0 : plan.kc;
        const int KB = int((kn + 31) / 32) * 2;
        for (int r0 = 0; r0 < kAtForms; r0 += plan.nr) {
            const int nr = plan.nr;
            if (nr == 10) go_forms<10>(X, n, ldx, near, r0, k0, KB, RB, !grad, tile, ops, s);
            else if (nr == 5) go_forms<5>(X, n, ldx, near, r0, k0, KB, RB, !grad, tile, ops, s);
            else if (nr == 2) go_forms<2>(X, n, ldx, near, r0, k0, KB, RB, !grad, tile, ops, s);
            else go_forms<1>(X, n, ldx, near, r0, k0, KB, RB, !grad, tile, ops, s);
            if (grad) {
                if (g256 != nullptr) go_tiles<256, true>(*g256, nr, r0, ops, KB, RB, k0, X, n, ldx, near, found, nu, G64, eslots, s);
                go_tiles<128, true>(g, nr, r0, ops, KB, RB, k0, X, n, ldx, near, found, nu, G64, eslots, s);
            } else {
                if (g256 != nullptr) go_tiles<256, false>(*g256, nr, r0, ops, KB, RB, k0, X, n, ldx, near, found, nu, G64, eslots, s);
                go_tiles<128, false>(g, nr, r0, ops, KB, RB, k0, X, n, ldx, near, found, nu, G64, eslots, s);
            }
        }
    }
    prof_end(kid, s);
    return check_launch(grad ? "triplet energy+grad (matrix form)" : "triplet energy (matrix form)");
}

SMX_CHECK_READER(check_flags_triplet_mfma)

}  // namespace smx
