// Packed per-triplet Axilrod-Teller energies on the 3-simplex: the tetrahedral
// analogue of the packed EDM (paper Sec. I: the triple-interaction n-body
// problem and the simplex-shaped outputs of pair problems).  Output E[p] for
// every triplet i < j < k < n, p the lexicographic rank
//   p(i,j,k) = C(n,3) - C(n-i,3) + T2(i,j) + (k - j - 1),
//   T2(i,j)  = (j-i-1)(n-1) - (j(j-1)/2 - i(i+1)/2)      (pairs (j', k) of row i
//              with j' < j), so T2(i, j+1) = T2(i, j) + (n - 1 - j).
// The energy of one triplet is written in the angle form itself,
//   E_t = nu (1 + 3 cos g_i cos g_j cos g_k) / (r1 r2 r3)^3
//       = nu (1 - 3 (a.b)(b.c)(c.a)) d1^3 d2^3 d3^3,   d = 1 / r,
// a, b, c the unit vectors of x_j - x_i, x_k - x_j, x_i - x_k (cos g_i = -(a.c), ...),
// with the cosines taken from their dot products: each element is then accurate to
// a few units of FP32 rounding relative to its scale nu d^9.  (The squared-distance
// form used by the reductions forms 16 x squared area by cancellation, whose error
// grows with a triangle's aspect ratio; it is harmless in sums, not per element.)
// 15 FP32 operations per 4-byte store, the unit vectors and cubes being the pairs',
// and a 2-norm error of 1.5e-7 (norms divided out per element: 19 operations,
// 2.6e-7).  The kernels are bound by the stores.
//
// Two kernels for the packed layout: whole runs per block from n = 704 (below, at
// at_packed_rows_kernel), and the tile kernel for smaller n, statistics and the
// tile-contiguous layout.
//
// Tile kernel: a block of 256 threads owns the 32^3 triplets of tile (X, Y, Z), X <= Y <= Z.
// (A second, tile-contiguous output layout is described at the kernel.)
//   1. positions of the three tiles -> LDS;
//   2. per pair of the sets (i,j), (i,k), (j,k) the unit vector and d^3 -> LDS as
//      one float4, stored [i][j], [i][k], [j][k]; 0 for a pair out of order or past
//      n (an invalid triplet computes 0; it is also never stored);
//   3. lane kl of a half wave takes k = Z 32 + kl; half wave h takes i = X 32 +
//      h + 8 m (m < 4) and sweeps j over the Y tile: the 32 lanes store 32
//      consecutive k of one (i, j), one contiguous 128-byte run.
#include "smx_device.h"
#include "smx_internal.h"

namespace smx {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kPackThreads = 256;

// nu as the elements use it: nu = m e, e a power of two.  m and 2^kPackShift go into the
// pairs (i, k) and 2^-kPackShift into the pairs (i, j), so that the products of an element
// stay in range where the element does: with k far from i and j (1 / r_ik^3 1 / r_jk^3
// is 1e-42 at r = 1e7) and with a large nu and a close pair (i, k).
struct PackNu {
    double m;
    float e;
};
constexpr double kPackShift = 0x1p40;
static PackNu pack_nu(float nu) {
    int x = 0;
    (void)__builtin_frexpf(nu, &x);
    if (!(__builtin_fabsf(nu) <= __FLT_MAX__) || nu == 0.f) x = 0;  // inf and NaN stay in m
    x = x < -100 ? -100 : x > 100 ? 100 : x;
    return {__builtin_ldexp(double(nu), -x) * kPackShift, __builtin_ldexpf(1.f, x)};
}

// A pair a, b as the elements use it: the unit vector from a to b and f / r^3 (0
// vectors for a pair that is not `on`).  The pairs (i, j) and (i, k), which serve
// many elements, are formed in FP64 and rounded once; 1 / r there to 2^-43, the FP32
// instruction and one Newton step.
__device__ __forceinline__ float4 pack_pair(float4 pa, float4 pb, bool on) {
    const float dx = pb.x - pa.x, dy = pb.y - pa.y, dz = pb.z - pa.z;
    const float sv = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
    const float d = on ? __builtin_amdgcn_rsqf(sv) : 0.f;
    return make_float4(dx * d, dy * d, dz * d, (d * d) * d);
}
__device__ __forceinline__ float4 pack_pair64(float4 pa, float4 pb, bool on, double f) {
    const double dx = double(pb.x) - double(pa.x), dy = double(pb.y) - double(pa.y), dz = double(pb.z) - double(pa.z);
    const double sv = __builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx));
    const double d0 = double(__builtin_amdgcn_rsqf(float(sv)));
    const double d = d0 * __builtin_fma(-0.5 * sv * d0, d0, 1.5);
    return on ? make_float4(float(dx * d), float(dy * d), float(dz * d), float(f * (d * d * d)))
              : make_float4(0.f, 0.f, 0.f, 0.f);
}
// Element (i, j, k) from its pairs (i, j), (j, k) and (i, k), with PackNu's factors.
__device__ __forceinline__ float pack_element(float4 a, float4 b, float4 c, float e) {
    const float ab = __builtin_fmaf(a.z, b.z, __builtin_fmaf(a.y, b.y, a.x * b.x));
    const float bc = __builtin_fmaf(b.z, c.z, __builtin_fmaf(b.y, c.y, b.x * c.x));
    const float ca = __builtin_fmaf(c.z, a.z, __builtin_fmaf(c.y, a.y, c.x * a.x));
    // cos cos cos = -(a.b)(b.c)(c.a) with the third side k -> i; c here is i -> k, which flips two signs
    return __builtin_fmaf(-3.f * e, (ab * bc) * ca, e) * (a.w * (b.w * c.w));
}

// TILED: the tile-contiguous layout instead of the lexicographic one.  Tile
// (X, Y, Z) of T3 owns the 32^3 floats starting at rank(X, Y, Z) * 32^3, rank =
// Z(Z+1)(Z+2)/6 + Y(Y+1)/2 + X (the tile's place in the listing by Z, Y, X);
// element (i, j, k) sits at offset 1024 (i mod 32) + 32 (j mod 32) + (k mod 32)
// inside it, and the tile's entries that are not triplets i < j < k < n hold
// 0.  Every tile is then one contiguous 128 KB run, written in full.
template <int MAP, bool STATS, bool TILED>
__global__ __launch_bounds__(kPackThreads) void at_packed_kernel(MapGeom g, const float *__restrict__ Xp,
                                                                 int64_t n, int64_t ldx, PackNu nu,
                                                                 float *__restrict__ E,
                                                                 unsigned long long *sslots) {
    uint64_t lin;
    int TX, TY, TZ;
    if (!tile3_of<MAP, true>(g, lin, TX, TY, TZ)) return;
    constexpr int T = kTripTile, PS = T * T;
    __shared__ float4 Pos[3][T];
    // pair terms, sets 0 (i,j), 1 (i,k), both with PackNu's factors, 2 (j,k)
    __shared__ float4 Vp[3][PS];
    __shared__ unsigned long long sred[2][kPackThreads / kWave];

    const int t = threadIdx.x;
    const int64_t base[3] = {int64_t(TX) * T, int64_t(TY) * T, int64_t(TZ) * T};
    if (t < 3 * T) {
        const int tile = t >> 5, a = t & 31;
        const int64_t p = base[tile] + a;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p < n) {
            v.x = Xp[p * ldx + 0];
            v.y = Xp[p * ldx + 1];
            v.z = Xp[p * ldx + 2];
        }
        Pos[tile][a] = v;
    }
    __syncthreads();

    // a tile with X < Y < Z wholly below n holds only valid triplets
    const bool interior = TX < TY && TY < TZ && base[2] + T <= n;
    {
        const int c = t & 31, r0 = t >> 5;
#pragma unroll
        for (int set = 0; set < 3; ++set) {
            const int ta = set == 2 ? 1 : 0, tb = set == 0 ? 1 : 2;  // row tile, column tile
            const float4 pb = Pos[tb][c];
            const int64_t gb = base[tb] + c;
#pragma unroll
            for (int it = 0; it < 4; ++it) {
                const int r = r0 + 8 * it;
                const float4 pa = Pos[ta][r];
                const int64_t ga = base[ta] + r;
                const bool valid = interior || (ga < gb && gb < n);
                Vp[set][r * T + c] = set == 2 ? pack_pair(pa, pb, valid) : pack_pair64(pa, pb, valid, set == 1 ? nu.m : 1.0 / kPackShift);
            }
        }
    }
    __syncthreads();

    const int kl = t & 31, h = t >> 5;
    const int64_t k = base[2] + kl;
    const int64_t c3 = n * (n - 1) * (n - 2) / 6;
    unsigned long long cnt = 0, cs = 0;
#pragma unroll 1
    for (int m = 0; m < 4; ++m) {
        const int il = h + 8 * m;
        const int64_t i = base[0] + il;
        const float4 vc = Vp[1][il * T + kl];
        // element index of (i, j, k) minus k, at j = Y 32, advanced per j
        const int64_t ni = n - i, j0 = base[1];
        int64_t rowj = c3 - ni * (ni - 1) * (ni - 2) / 6 + (j0 - i - 1) * (n - 1) - (j0 * (j0 - 1) / 2 - i * (i + 1) / 2) -
                       j0 - 1;
        float *out = E + k;
        if (TILED) {
            const uint64_t Z = uint64_t(TZ), Y = uint64_t(TY);
            const uint64_t rank = Z * (Z + 1) * (Z + 2) / 6 + Y * (Y + 1) / 2 + uint64_t(TX);
            out = E + rank * uint64_t(T * T * T) + uint64_t(il * T * T + kl);
        }
#pragma unroll 4
        for (int jl = 0; jl < T; ++jl) {
            const int64_t j = j0 + jl;
            const float4 va = Vp[0][il * T + jl];
            const float4 vb = Vp[2][jl * T + kl];
            const float e = pack_element(va, vb, vc, nu.e);
            const bool ok = TILED ? (i < j && j < k && k < n)
                          : interior ? smx_check(i < j && j < k && k < n, kCheckStore) : (i < j && j < k && k < n);
            if (TILED)
                out[jl * T] = ok ? e : 0.f;
            else if (ok)
                out[rowj - jl] = e;
            if (STATS && ok) {
                ++cnt;
                cs += mix64(id_trip_lt(uint64_t(i), uint64_t(j), uint64_t(k)));
            }
            rowj += n - 1 - j;
        }
    }
    if (STATS) {
        const unsigned long long c = block_sum<unsigned long long, kPackThreads>(cnt, sred[0]);
        const unsigned long long hs = block_sum<unsigned long long, kPackThreads>(cs, sred[1]);
        if (t == 0) stats_add(sslots, lin, c, hs);
    }
}

// Rows form of the packed layout.  The elements (i, j, .) of a pair are one
// contiguous run of n - 1 - j floats at any 4-byte offset.  A block writes whole runs:
// kPackI particles i and the 32 j of one pair tile (X, Y) of the 2-simplex, all k, 256
// at a time (thread t computes k = k0 + t; x_k - x_j and 1 / r_jk serve the block's
// kPackI particles).  kPackJ x kPackI pieces of runs are staged in LDS, each at its
// run's offset inside a 128-byte line, and leave as whole lines, 16 bytes a lane and
// streaming; only a run's two ends are partial.  What each of these gives at n = 2048
// (5.72 GB): the tile kernel (128-byte runs in pieces of two blocks) 3.76 ms; whole
// runs in 4-byte stores 2.36 (the texture-address unit busy 0.8 of the time); 16-byte
// aligned stores 1.97; whole lines 1.73; and streaming 1.34 ms = 4.3 TB/s, where a fill
// of the buffer reaches 6.9 (streaming without whole lines 1.92; per-XCD ranges of
// blocks 1.80 against 1.73).
constexpr int kPackI = 4, kPackJ = 4;
constexpr int kPackLine = 32;                         // floats per 128-byte line
constexpr int kPackPiece = kPackThreads + kPackLine;  // LDS floats per piece: offset 0..31, 256 elements
// Pieces overlap by a line, so that a piece stores whole lines and only a run's own
// ends go element by element: at any offset the lines of one piece end where the
// next piece's begin.
constexpr int kPackStride = kPackThreads - kPackLine;

template <int MAP>
__global__ __launch_bounds__(kPackThreads) void at_packed_rows_kernel(MapGeom g, const float *__restrict__ Xp, int64_t n,
                                                                      int64_t ldx, PackNu nu, float *__restrict__ E) {
    constexpr int T = kTripTile, PARTS = T / kPackI, PIECES = kPackI * kPackJ, NW = kPackThreads / kWave;
    static_assert(NW == kPackI && kPackThreads == 4 * kWave, "a wave stores one i's pieces, a group a lane");
    const uint64_t b = launch_index();
    if (b >= g.G * PARTS) return;
    const uint32_t task = uint32_t(b);
    uint64_t lin;
    int TX, TY;
    if (!tile2_of_id<MAP>(g, task / PARTS, lin, TX, TY)) return;
    __shared__ float4 Pj[T];          // positions of the tile's j
    __shared__ float4 Va[T][kPackI];  // pair terms (i, j)
    __shared__ __attribute__((aligned(16))) float St[PIECES][kPackPiece];
    const int t = threadIdx.x, lane = t & (kWave - 1), w = __builtin_amdgcn_readfirstlane(t / kWave);
    const int64_t i0 = int64_t(TX) * T + (task % PARTS) * kPackI, j0 = int64_t(TY) * T;
    auto pos = [&](int64_t p) {
        return p < n ? make_float4(Xp[p * ldx], Xp[p * ldx + 1], Xp[p * ldx + 2], 0.f) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    if (t < T) Pj[t] = pos(j0 + t);
    if (t < T * kPackI) Va[t / kPackI][t % kPackI] = pack_pair64(pos(i0 + t % kPackI), pos(j0 + t / kPackI), true, 1.0 / kPackShift);
    __syncthreads();
    // element (i, j, k) at start(i) + step(j) + k, step(j + 1) = step(j) + n - 2 - j
    const int64_t c3 = n * (n - 1) * (n - 2) / 6;
    auto start = [&](int64_t i) {
        const int64_t ni = n - i;
        return c3 - ni * (ni - 1) * (ni - 2) / 6 - (i + 1) * (n - 1) + i * (i + 1) / 2;
    };
    const int64_t step0 = j0 * (n - 1) - j0 * (j0 - 1) / 2 - j0 - 1;
    const int eoff = int((reinterpret_cast<uintptr_t>(E) >> 2) & (kPackLine - 1));  // E is 4-byte aligned
    // offsets of the pieces modulo a line: those of (i0 + u, j0, k = 0)
    uint32_t si[kPackI];
    float4 pi[kPackI];
#pragma unroll
    for (int u = 0; u < kPackI; ++u) {
        si[u] = uint32_t(start(i0 + u)) + uint32_t(step0) + uint32_t(eoff);
        pi[u] = pos(i0 + u);
    }
    const int64_t iw = i0 + w, sw = start(iw) + step0;  // the particle whose pieces this wave stores
    const int jn = int(n - j0 < T ? n - j0 : T), dn = int(n - 2 - j0);
    const uint32_t lane16 = uint32_t(lane) * 16u;
    for (int64_t k0 = j0; k0 < n; k0 += kPackStride) {
        const float4 pk = pos(k0 + t);
        float4 vc[kPackI];
#pragma unroll
        for (int u = 0; u < kPackI; ++u) vc[u] = pack_pair64(pi[u], pk, true, nu.m);
        const int hi = int(n - k0 < kPackThreads ? n - k0 : kPackThreads);
        const int dk = int(k0 - j0);
        int64_t at0 = sw + k0;  // element t = 0 of the piece of (iw, j0 + jb)
        uint32_t sj0 = uint32_t(k0);  // its offset without si
        for (int jb = 0; jb < jn; jb += kPackJ) {
            uint32_t sj = sj0;
            if (w * kWave < hi)  // (a wave past the last k has nothing to compute)
#pragma unroll
            for (int jj = 0; jj < kPackJ; ++jj) {
                const int jl = jb + jj;
                const float4 vb = pack_pair(Pj[jl], pk, true);
#pragma unroll
                for (int u = 0; u < kPackI; ++u) {
                    St[jj * kPackI + u][((sj + si[u]) & (kPackLine - 1)) + t] = pack_element(Va[jl][u], vb, vc[u], nu.e);
                }
                sj += uint32_t(dn - jl);
            }
            __syncthreads();
            // wave w stores the pieces of particle i0 + w: the lines that are all in
            // [lo, hi), 16 bytes a lane
            int64_t at = at0;
#pragma unroll
            for (int m = 0; m < kPackJ; ++m) {
                const int jl = jb + m, lo = jl >= dk ? jl + 1 - dk : 0;
                if (jl < jn && iw < j0 + jl && lo < hi) {
                    const int ph = int(at + eoff) & (kPackLine - 1);
                    const int la = (lo + ph + kPackLine - 1) / kPackLine, lb = (hi + ph) / kPackLine;
                    char *row = reinterpret_cast<char *>(E + (at - ph));  // at a line
                    const float *st = St[m * kPackI + w];
                    if (lane >= 8 * la && lane < 8 * lb && smx_check(k0 + 4 * lane - ph + 3 < n, kCheckStore))
                        __builtin_nontemporal_store(*reinterpret_cast<const f32x4_t *>(st + 4 * lane),
                                                    reinterpret_cast<f32x4_t *>(row + lane16));
                    // a run's first and last elements outside those lines
                    if (lo > 0 || hi < kPackThreads) {
                        const int le = lane & (kPackLine - 1);
                        const bool head = lane < kPackLine;
                        const int e = kPackLine * (head ? la - 1 : lb) - ph + le;
                        const bool mine = head ? lo > 0 : hi < kPackThreads && lb >= la;
                        if (mine && e >= lo && e < hi) reinterpret_cast<float *>(row)[e + ph] = st[e + ph];
                    }
                }
                at += dn - jl;
            }
            at0 = at;
            sj0 += uint32_t(kPackJ * dn - kPackJ * jb - kPackJ * (kPackJ - 1) / 2);
            __syncthreads();
        }
    }
}

template <int MAP, bool TILED>
static void go_packed(const MapGeom &g, const float *X, int64_t n, int64_t ldx, PackNu nu, float *E,
                      unsigned long long *sslots, hipStream_t s) {
    const dim3 grid = MAP == MAP_BBOX ? dim3(g.nb, g.nb, g.nb) : grid_for(g.G, kPackThreads);
    if (sslots)
        hipLaunchKernelGGL((at_packed_kernel<MAP, true, TILED>), grid, dim3(kPackThreads), 0, s, g, X, n, ldx, nu,
                           E, sslots);
    else
        hipLaunchKernelGGL((at_packed_kernel<MAP, false, TILED>), grid, dim3(kPackThreads), 0, s, g, X, n, ldx, nu,
                           E, sslots);
}

int launch_triplet_packed(const MapGeom &g, const float *X, int64_t n, int64_t ldx, float nu, float *E,
                          unsigned long long *sslots, bool tiled, bool rows, hipStream_t s) {
    const int kid = tiled ? K_TRIP_TILED : K_TRIP_PACKED;
    const PackNu pn = pack_nu(nu);
    prof_begin(kid, s);
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        constexpr int MAPK = decltype(M)::value;
        if (rows)
            hipLaunchKernelGGL((at_packed_rows_kernel<MAPK>), grid_for(gg.G * (kTripTile / kPackI), kPackThreads),
                               dim3(kPackThreads), 0, s, gg, X, n, ldx, pn, E);
        else if (tiled) go_packed<MAPK, true>(gg, X, n, ldx, pn, E, sslots, s);
        else go_packed<MAPK, false>(gg, X, n, ldx, pn, E, sslots, s);
    });
    prof_end(kid, s);
    return check_launch("triplet packed");
}

SMX_CHECK_READER(check_flags_tripack)

}  // namespace smx
