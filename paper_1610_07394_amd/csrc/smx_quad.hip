// 4-point contacts on the 4-simplex: the number of quadruplets i < j < k < l
// whose six pairs all lie within a contact radius (the 4-cliques of the
// contact graph) -- a 4-body count over the discrete orthogonal 4-simplex
// (paper Sec. I lists correlation counts among simplex-shaped problems; the
// 4-simplex parallel space is the lambda4 map built on the recursive set of
// Sec. III-D).
//
// Two passes, both over simplex tiles of 64 elements per dimension:
//   1. contact words (2-simplex, one 64-thread block per tile (X, Y), X <= Y):
//      W[Y][64 X + p] bit q = contact(i, j), i = 64 X + p < j = 64 Y + q < n,
//      decided on the FP32 squared distance fl(fma(dz,dz, fma(dy,dy, dx*dx))),
//      d* = fl(x_j* - x_i*), below fl(rc*rc).  Column-tile-major, so the 64
//      words of one tile pair are contiguous.
//   2. cliques (4-simplex, tiles X1 <= X2 <= X3 <= X4, each counted by one
//      wave): lane p1 holds words p1 of the six 64-word blocks of the tile's
//      index sets, and for every contact (p1, p2) and every common neighbour p3
//      (bits of W13[p1] & W23[p2]) adds popcount(W14[p1] & W24[p2] & W34[p3]).
//      The ordering i < j < k < l within equal tiles and the bound n are
//      already in the words.
// Contacts are sparse, so a tile needs little arithmetic: this form is bound by
// each wave's chain of per-tile word loads (3 KB per tile, from L2) and LDS
// exchange.  Calls without statistics count from the contacts instead while the
// graph is sparse (clique_rows_kernel), and take the tiles when it is not.
#include "smx_device.h"
#include "smx_internal.h"

namespace smx {

constexpr int kQuadWordThreads = 64;
constexpr int kQuadThreads = 256;

// What the calls that count from the contacts keep in the count slots (zeroed with
// them): beside each slot's count the length of its list of work items and the counter
// that deals the tile form's ids; in slot 0, one line for a scalar load, whether a list
// overflowed, kCostWords shares of the cost and how many blocks are done with the tiles.
constexpr int kSlotItems = 1, kSlotWalk = 2, kSlotDone = 3, kSlotFull = 4, kSlotCost = 8, kCostWords = 8;

// The gate: true when the tile form is to count.  Final once quad_cost_kernel is done.
__device__ __forceinline__ bool quad_dense(const unsigned long long *cslots, unsigned long long limit) {
    unsigned long long cost = 0;
#pragma unroll
    for (int q = 0; q < kCostWords; ++q) cost += cslots[kSlotCost + q];
    return cost > limit || cslots[kSlotFull] != 0;
}

// out = sum of the slots' counts, by the kSlots threads of one block.
__device__ __forceinline__ void write_count(const unsigned long long *cslots, int64_t *out) {
    __shared__ unsigned long long red[kSlots / kWave];
    const unsigned long long v = block_sum<unsigned long long, kSlots>(
        __hip_atomic_load(cslots + threadIdx.x * kSlotStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), red);
    if (threadIdx.x == 0) out[0] = int64_t(v);
}
// Whether this block is the last of the launch to get here; what the others have added
// to the slots is then there.  Every thread of the block calls it.
__device__ __forceinline__ bool last_block(unsigned long long *done) {
    __shared__ bool last;
    __threadfence();
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(done, 1ull) == (unsigned long long)(gridDim.x) * gridDim.y - 1;
    __syncthreads();
    if (last) __threadfence();
    return last;
}

// A work item of the rows form: tile (X, Y) of the contact words and one of 2^lgparts
// parts of its contacts, by rows (row mod 2^min(lgparts, 6)), then by columns.
constexpr int kItemLgMax = 8;
__device__ __forceinline__ uint32_t item_pack(int X, int Y, int part, int lgparts) {
    return uint32_t(X) | uint32_t(Y) << 8 | uint32_t(part) << 16 | uint32_t(lgparts) << 24;
}

// ROWS: row-major words (row i, column tile Y at i nb + Y), and the tile's contacts as
// work items of about `fill` in the list of one slot (given items; `cap` a list, past
// that the graph is taken to be dense); else column-tile-major.  WALK: for a launch that
// the gate may leave nothing to do, few blocks that walk the tiles.
template <int MAP, bool ROWS, bool WALK>
__global__ __launch_bounds__(kQuadWordThreads) void contact_words_kernel(MapGeom g, const float *__restrict__ Xp,
                                                                        int64_t n, int64_t ldx, float rc2,
                                                                        uint64_t *__restrict__ W, int64_t npad,
                                                                        unsigned long long *cslots,
                                                                        uint32_t *__restrict__ items, uint32_t cap,
                                                                        uint32_t fill, unsigned long long limit) {
    if (WALK && !quad_dense(cslots, limit)) return;
    for (uint64_t b = launch_index(); !WALK || b < g.G; b += uint64_t(gridDim.x) * gridDim.y) {
        uint64_t lin;
        int TX, TY;
        const bool tile = WALK ? tile2_of_id<MAP>(g, uint32_t(b), lin, TX, TY) : tile2_of<MAP, true>(g, lin, TX, TY);
        if (!tile) {
            if (WALK) continue;
            return;
        }
        __shared__ float4 Pc[kQuadTile];
        const int p = threadIdx.x;
        const int64_t i = int64_t(TX) * kQuadTile + p, jc = int64_t(TY) * kQuadTile + p;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (jc < n) v = make_float4(Xp[jc * ldx + 0], Xp[jc * ldx + 1], Xp[jc * ldx + 2], 0.f);
        Pc[p] = v;
        float xi = 0.f, yi = 0.f, zi = 0.f;
        if (i < n) {
            xi = Xp[i * ldx + 0];
            yi = Xp[i * ldx + 1];
            zi = Xp[i * ldx + 2];
        }
        __syncthreads();
        uint64_t word = 0;
        if (i < n) {
            const int64_t jbase = int64_t(TY) * kQuadTile;
            const int q0 = TX == TY ? p + 1 : 0;
            for (int q = q0; q < kQuadTile; ++q) {
                const float4 c = Pc[q];
                const float dx = c.x - xi, dy = c.y - yi, dz = c.z - zi;
                const float s = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
                if (jbase + q < n && s < rc2) word |= uint64_t(1) << q;
            }
        }
        if (ROWS) {
            W[i * g.nb + TY] = word;
            const unsigned c = items != nullptr ? wave_sum(uint32_t(__builtin_popcountll(word))) : 0;
            if (c != 0) {
                int lg = 0;
                while (lg < kItemLgMax && (c >> lg) > fill) ++lg;
                const uint32_t parts = 1u << lg, slot = uint32_t(16 * TX + TY) % kSlots;
                uint32_t at = 0;
                if (p == 0) at = uint32_t(atomicAdd(cslots + slot * kSlotStride + kSlotItems, (unsigned long long)parts));
                at = __builtin_amdgcn_readfirstlane(at);
                for (uint32_t e = p; e < parts; e += kQuadTile)
                    if (at + e < cap) items[slot * cap + at + e] = item_pack(TX, TY, int(e), lg);
                if (p == 0 && at + parts > cap) atomicOr(cslots + kSlotFull, 1ull);
            }
        } else {
            W[int64_t(TY) * npad + i] = word;
        }
        if (!WALK) return;
        __syncthreads();  // Pc is free for the next tile
    }
}

// The cost of counting from the contacts, which the gate goes by.  Its work is the
// triangles; what bounds them, and is near them where points in space make the
// contacts (0.47 of it for even points, 1 for a cluster in contact), are the pairs of
// forward contacts of each row, sum_i C(f_i, 2).
constexpr int kCostRows = 8;  // per wave
__global__ __launch_bounds__(kQuadThreads) void quad_cost_kernel(const uint64_t *__restrict__ R, int64_t n, int nb,
                                                                 unsigned long long *cslots) {
    __shared__ unsigned long long red[kQuadThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int64_t r0 = (int64_t(blockIdx.x) * (kQuadThreads / kWave) + w) * kCostRows;
    unsigned long long cost = 0;
#pragma unroll
    for (int r = 0; r < kCostRows; ++r) {
        const int64_t i = r0 + r;
        uint32_t f = 0;
        if (i < n)
            for (int c = int(i / kQuadTile) + lane; c < nb; c += kWave) f += uint32_t(__builtin_popcountll(R[i * nb + c]));
        f = wave_sum(f);
        cost += (unsigned long long)(f) * (f > 0 ? f - 1 : 0) / 2;
    }
    if (lane == 0) red[w] = cost;
    __syncthreads();
    if (threadIdx.x == 0) {
        cost = 0;
#pragma unroll
        for (int q = 0; q < kQuadThreads / kWave; ++q) cost += red[q];
        if (cost != 0) atomicAdd(cslots + kSlotCost + blockIdx.x % kCostWords, cost);
    }
}

// Cliques from neighbours, for sparse contacts.  Row i of the contact graph is a
// bit string of nb words (column tiles below its own are not written and are
// masked).  A wave takes the work items of one slot's list in turn (LISTED), or one row
// of a tile of T2 (n <= 2048: 64 waves for each of few tiles; n = 1500, rc = 2 50 us, by
// lists 56); for every contact
// i < j of an item the common neighbours m = row i & row j (a word a lane, NQ words
// when nb > 64), and for every k in m the count of m & row k: what is left are the l >
// k in contact with all three.  So the work follows the contacts (n = 8192, 34
// contacts a particle: 1.4e5 pairs, 1.2e6 triangles) and not the 1.2e7 tiles of the
// 4-simplex, whose 3 KB of words each the tile form reads whether they hold a
// clique or not; and the items spread the contacts of a cluster that lies in a few
// tiles.  The rows of k are read four at a time: the pass is bound by their latency.
// Tiles / this form, ms a call: n = 8192, even, rc = 2 1.92 / 0.146, rc = 4 5.3 / 2.7;
// 300 of the particles in one cluster, consecutive 18.2 / 2.7 (58 with the rows of a tile
// dealt to a fixed number of waves), at random 2.8 / 0.85; 700 19.5 / 11.9 and 9.3 / 6.1.
template <int NQ, bool LISTED>
__global__ __launch_bounds__(kQuadThreads) void clique_rows_kernel(int nb, const uint64_t *__restrict__ R,
                                                                  const uint32_t *__restrict__ items, uint32_t cap,
                                                                  unsigned long long limit, unsigned long long *cslots) {
    if (limit != 0 && quad_dense(cslots, limit)) return;
    const int lane = threadIdx.x & (kWave - 1);
    const uint32_t wv = blockIdx.x * (kQuadThreads / kWave) + uint32_t(__builtin_amdgcn_readfirstlane(threadIdx.x / kWave));
    // wave q0 of a list, the lists turned by 37 from one q0 to the next: with equal places
    // the waves of one list would meet on four CUs
    const uint32_t q0 = LISTED ? wv / kSlots : 0, slot = (wv + 37u * q0) % kSlots;
    const uint32_t step = LISTED ? gridDim.x * (kQuadThreads / kWave) / kSlots : 1;
    uint32_t len = 1;
    if (LISTED) {
        const unsigned long long listed = cslots[slot * kSlotStride + kSlotItems];
        len = listed < cap ? uint32_t(listed) : cap;
    }
    auto lane64 = [](uint64_t v, int l) -> uint64_t {
        return uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v)), l))) |
               uint64_t(uint32_t(__builtin_amdgcn_readlane(int(uint32_t(v >> 32)), l))) << 32;
    };
    // words q of a row from column tile `from` on
    auto row = [&](int64_t i, int from, int q) -> uint64_t {
        const int w = lane + 64 * q;
        return w >= from && w < nb ? R[i * nb + w] : 0;
    };
    unsigned long long cnt = 0;
    for (uint32_t e = q0; e < len; e += step) {
        int X, Y, part, lg;
        if (LISTED) {
            const uint32_t item = __builtin_amdgcn_readfirstlane(items[slot * cap + e]);
            X = int(item & 255u), Y = int(item >> 8 & 255u), part = int(item >> 16 & 255u), lg = int(item >> 24);
        } else {
            linear2(wv >> 6, X, Y);
            if (Y >= nb) return;
            part = int(wv & 63u), lg = 6;
        }
        const int64_t i0 = int64_t(X) * kQuadTile;
        const int lgrow = lg < 6 ? lg : 6, lgcol = lg - lgrow;
        const bool mine = (lane & ((1 << lgrow) - 1)) == (part & ((1 << lgrow) - 1));
        const uint64_t cols = (lgcol == 0 ? ~0ull : lgcol == 1 ? 0x5555555555555555ull : 0x1111111111111111ull) << (part >> lgrow);
        const uint64_t word = mine ? R[(i0 + lane) * nb + Y] & cols : 0;
        uint64_t act = __ballot(word != 0);
        while (act != 0) {
            const int p = __builtin_ctzll(act);
            act &= act - 1;
            uint64_t mi[NQ];
#pragma unroll
            for (int q = 0; q < NQ; ++q) mi[q] = row(i0 + p, Y, q);
            uint64_t js = lane64(word, p);
            while (js != 0) {
                const int64_t j = int64_t(Y) * kQuadTile + __builtin_ctzll(js);
                js &= js - 1;
                uint64_t m[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) m[q] = mi[q] & row(j, Y, q);
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    uint64_t nz = __ballot(m[q] != 0);
                    int wl = 0;
                    uint64_t ks = 0;
                    while (ks != 0 || nz != 0) {
                        int64_t k[4];
                        int have = 0;
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            if (ks == 0 && nz != 0) {
                                wl = __builtin_ctzll(nz);
                                nz &= nz - 1;
                                ks = lane64(m[q], wl);
                            }
                            k[u] = -1;
                            if (ks != 0) {
                                k[u] = int64_t(wl + 64 * q) * kQuadTile + __builtin_ctzll(ks);
                                ks &= ks - 1;
                                ++have;
                            }
                        }
                        uint64_t r[4][NQ];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int v = q; v < NQ; ++v)
                                r[u][v] = u < have && m[v] != 0 ? row(k[u], int(k[u] >> 6), v) : 0;
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int v = q; v < NQ; ++v) cnt += unsigned(__builtin_popcountll(m[v] & r[u][v]));
                    }
                }
            }
        }
    }
    const unsigned long long c = wave_sum(cnt);
    if (lane == 0 && c != 0) atomicAdd(cslots + slot * kSlotStride, c);
}

// Quadruplets i < j < k < l of a 4-simplex tile, in closed form (edge lengths
// below n; runs of equal tile coordinates hold C(t, r) strict r-tuples).
__device__ __forceinline__ uint64_t quad_tile_volume(const int T[4], int64_t n) {
    uint64_t cnt = 1;
    int d = 0;
    while (d < 4) {
        int r = 1;
        while (d + r < 4 && T[d + r] == T[d]) ++r;
        const int64_t rem = n - int64_t(T[d]) * kQuadTile;
        const uint64_t t = rem <= 0 ? 0 : (rem < kQuadTile ? uint64_t(rem) : uint64_t(kQuadTile));
        uint64_t v = 1;
        for (int q = 0; q < r; ++q) v = t < uint64_t(q) ? 0 : v * (t - uint64_t(q)) / uint64_t(q + 1);
        cnt *= v;
        d += r;
    }
    return cnt;
}

// One wave per 64 logical block ids, one tile at a time.  Lane q evaluates the
// map for id 64 (4 b + w) + q, so a wave decodes its 64 ids in one pass and an
// id outside the simplex costs one lane of that pass; the wave then walks the
// mapped tiles (a ballot of the lanes' results) with each tile's coordinates
// read from the lane that decoded it, loading the next tile's words while it
// counts the current one.  Per tile, lane p holds word p of the six 64-word
// blocks of the index sets, keeps its own three in registers, shares the other
// three through the wave's 1.5 KB of LDS, and walks its 64 p2 bits.  A launch
// has G / 256 hardware blocks.  A gated launch that walks the ids also writes the count.
template <int MAP, bool STATS>
__global__ __launch_bounds__(kQuadThreads) void quad_kernel(MapGeom g, const uint64_t *__restrict__ W, int64_t npad,
                                                           int64_t n, uint32_t grab, unsigned long long limit,
                                                           unsigned long long *cslots, unsigned long long *sslots,
                                                           int64_t *out) {
    // pair sets s = (a, b): 0 (0,1), 1 (0,2), 2 (0,3), 3 (1,2), 4 (1,3), 5 (2,3);
    // sets 3..5 are read across lanes
    __shared__ uint64_t A[kQuadThreads / kWave][3][kQuadTile];
    const int w = threadIdx.x / kWave, p = threadIdx.x & (kWave - 1);
    uint64_t (*Aw)[kQuadTile] = A[w];
    const uint64_t wave = launch_index() * (kQuadThreads / kWave) + uint64_t(w);
    // 64 ids a wave; gated (grab > 0), runs of `grab` times 64 ids, the waves of a slot
    // taking the next of its runs from its counter (one counter for all would serialise
    // their atomics; not for the launches per cube, which would share them).  (The next round's first LDS writes stay behind this
    // round's reads: the wave barriers of the tile loop order them.)
    const bool gated = !STATS && grab != 0, walk = gated && MAP != MAP_CUBE;
    if (gated && !quad_dense(cslots, limit)) {
        if (walk && launch_index() == 0) write_count(cslots, out);  // an earlier launch has counted
        return;
    }
    for (bool more_ids = true; more_ids;) {
        uint64_t chunk = wave, end = wave + 1;
        if (walk) {
            uint32_t k = 0;
            if (p == 0) k = uint32_t(atomicAdd(cslots + (wave % kSlots) * kSlotStride + kSlotWalk, 1ull));
            chunk = (uint64_t(__builtin_amdgcn_readfirstlane(k)) * kSlots + wave % kSlots) * grab;
            end = chunk + grab;
        }
        more_ids = walk && end * kWave < g.G;
        for (; chunk < end && chunk * kWave < g.G; ++chunk) {
            const uint64_t base = chunk * kWave;

            uint64_t mylin = 0;
            int Tq[4] = {0, 0, 0, 0};
            bool ok = false;
            if (base + uint64_t(p) < g.G) ok = tile4_of_id<MAP>(g, uint32_t(base + uint64_t(p)), mylin, Tq);
            uint64_t mask = __ballot(ok);

            // coordinates of the tile decoded by lane q (q uniform), and its words
            auto coords = [&](int q, int T[4]) {
#pragma unroll
                for (int d = 0; d < 4; ++d) T[d] = __builtin_amdgcn_readlane(Tq[d], q);
            };
            auto load = [&](const int T[4], uint64_t a[6]) {
#pragma unroll
                for (int s = 0; s < 6; ++s) {
                    const int64_t ra = s < 3 ? T[0] : (s < 5 ? T[1] : T[2]);
                    const int64_t cb = s == 0 ? T[1] : (s == 1 || s == 3) ? T[2] : T[3];
                    a[s] = W[cb * npad + ra * kQuadTile + p];
                }
            };

            uint32_t cnt = 0;
            if (mask != 0) {
                int q = __builtin_ctzll(mask);
                mask &= mask - 1;
                int T[4];
                uint64_t a[6];
                coords(q, T);
                load(T, a);
                while (true) {
                    const bool more = mask != 0;
                    int qn = 0, Tn[4] = {0, 0, 0, 0};
                    uint64_t an[6] = {0, 0, 0, 0, 0, 0};
                    if (more) {
                        qn = __builtin_ctzll(mask);
                        mask &= mask - 1;
                        coords(qn, Tn);
                        load(Tn, an);
                    }
                    // the previous tile's reads of this wave's LDS are done before it is
                    // overwritten, and the writes land before other lanes read them
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int s = 0; s < 3; ++s) Aw[s][p] = a[3 + s];
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                    uint64_t bits = a[0];
                    while (bits != 0) {
                        const int p2 = __builtin_ctzll(bits);
                        bits &= bits - 1;
                        uint64_t m3 = a[1] & Aw[0][p2];
                        const uint64_t wv = a[2] & Aw[1][p2];
                        while (m3 != 0) {
                            const int p3 = __builtin_ctzll(m3);
                            m3 &= m3 - 1;
                            cnt += uint32_t(__builtin_popcountll(wv & Aw[2][p3]));
                        }
                    }
                    if (STATS && p == 0) {
                        const uint64_t lin = uint64_t(__builtin_amdgcn_readlane(uint32_t(mylin), q)) |
                                             (uint64_t(__builtin_amdgcn_readlane(uint32_t(mylin >> 32), q)) << 32);
                        stats_add(sslots, lin, quad_tile_volume(T, n), 0);
                    }
                    if (!more) break;
                    q = qn;
#pragma unroll
                    for (int d = 0; d < 4; ++d) T[d] = Tn[d];
#pragma unroll
                    for (int s = 0; s < 6; ++s) a[s] = an[s];
                }
            }
            const unsigned c = wave_sum(cnt);
            if (p == 0 && c != 0) atomicAdd(cslots + (base / kWave % kSlots) * kSlotStride, (unsigned long long)c);
        }
    }
    if (walk && last_block(cslots + kSlotDone)) write_count(cslots, out);
}

__global__ void count_finalize_kernel(const unsigned long long *slots, int64_t *out) {
    __shared__ unsigned long long red[kSlots / kWave];
    const unsigned long long v = block_sum<unsigned long long, kSlots>(slots[threadIdx.x * kSlotStride], red);
    if (threadIdx.x == 0) out[0] = int64_t(v);
}

template <bool ROWS>
static void go_words(const MapGeom &g, const float *X, int64_t n, int64_t ldx, float rc2, uint64_t *W, int64_t npad,
                     unsigned long long *cslots, uint32_t *items, uint32_t cap, uint32_t fill, uint64_t limit, hipStream_t s) {
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        constexpr int MAPK = decltype(M)::value;
        if (!ROWS && cslots != nullptr) {
            const dim3 grid = grid_for(gg.G < 2048 ? gg.G : 2048, kQuadWordThreads);
            hipLaunchKernelGGL((contact_words_kernel<MAPK, false, true>), grid, dim3(kQuadWordThreads), 0, s, gg, X, n,
                               ldx, rc2, W, npad, cslots, items, cap, fill, (unsigned long long)limit);
        } else {
            const dim3 grid = MAPK == MAP_BBOX ? dim3(gg.nb, gg.nb, 1) : grid_for(gg.G, kQuadWordThreads);
            hipLaunchKernelGGL((contact_words_kernel<MAPK, ROWS, false>), grid, dim3(kQuadWordThreads), 0, s, gg, X, n,
                               ldx, rc2, W, npad, cslots, items, cap, fill, (unsigned long long)limit);
        }
    });
}

int launch_contact_words(const MapGeom &g, const float *X, int64_t n, int64_t ldx, float rc2, uint64_t *W,
                         int64_t npad, unsigned long long *cslots, bool rows, uint32_t *items, uint32_t cap,
                         uint64_t limit, hipStream_t s) {
    // contacts an item: the fewer, the more waves share the work (us, 1 / 4 / 16: n = 3000,
    // rc = 2 76 75 90, rc = 3 269 260 284; n = 8192, rc = 3 650 655 717); 8 at larger n for
    // half the list
    const uint32_t fill = n <= 4096 ? 4 : 8;
    prof_begin(K_QUAD_WORDS, s);
    if (rows) go_words<true>(g, X, n, ldx, rc2, W, npad, cslots, items, cap, fill, 0, s);
    else go_words<false>(g, X, n, ldx, rc2, W, npad, cslots, nullptr, 0, 0, limit, s);
    prof_end(K_QUAD_WORDS, s);
    return check_launch("contact words");
}

int launch_quad_rows(int nb, const uint64_t *R, int64_t n, const uint32_t *items, uint32_t cap, uint64_t limit,
                     unsigned long long *cslots, hipStream_t s) {
    constexpr int waves = kQuadThreads / kWave;
    const unsigned long long lim = limit;
    prof_begin(K_QUAD, s);
    if (limit != 0) {
        constexpr int rows = waves * kCostRows;
        hipLaunchKernelGGL(quad_cost_kernel, dim3(uint32_t((n + rows - 1) / rows)), dim3(kQuadThreads), 0, s, R, n, nb,
                           cslots);
    }
    // listed: 16384 waves, a full chip twice, in equal shares of the lists
    static_assert(16384 % kSlots == 0, "equal shares");
    const dim3 grid(items != nullptr ? 16384 / waves : uint32_t(nb * (nb + 1) / 2 * kWave / waves));
    if (items == nullptr) hipLaunchKernelGGL((clique_rows_kernel<1, false>), grid, dim3(kQuadThreads), 0, s, nb, R, items, cap, lim, cslots);  // nb <= 64
    else if (nb <= 64) hipLaunchKernelGGL((clique_rows_kernel<1, true>), grid, dim3(kQuadThreads), 0, s, nb, R, items, cap, lim, cslots);
    else if (nb <= 128) hipLaunchKernelGGL((clique_rows_kernel<2, true>), grid, dim3(kQuadThreads), 0, s, nb, R, items, cap, lim, cslots);
    else hipLaunchKernelGGL((clique_rows_kernel<4, true>), grid, dim3(kQuadThreads), 0, s, nb, R, items, cap, lim, cslots);
    prof_end(K_QUAD, s);
    return check_launch("quad contacts (rows)");
}

int launch_quad(const MapGeom &g, const uint64_t *W, int64_t npad, int64_t n, bool gated, uint64_t limit, unsigned long long *cslots,
                unsigned long long *sslots, int64_t *out, hipStream_t s) {
    prof_begin(K_QUAD, s);
    for_each_launch(g, [&](auto M, const MapGeom &gg) {
        constexpr int MAPK = decltype(M)::value;
        const uint64_t chunks = (gg.G + kWave - 1) / kWave;  // 64 ids a wave
        const uint64_t blocks = (chunks + kQuadThreads / kWave - 1) / (kQuadThreads / kWave);
        // a launch that may find nothing to do keeps few blocks, which then walk the ids:
        // equal shares took 10% longer than a block per 256 ids where heavy tiles lie together,
        // runs dealt on demand take as long (n = 8192, 1400 in a cluster 35.4, 32.0, 32.2 ms)
        const dim3 grid = grid_for(gated && MAPK != MAP_CUBE && blocks > 2048 ? 2048 : blocks, kQuadThreads);
        const uint32_t grab = gated ? uint32_t(1 + (chunks >> 23)) : 0;
        if (sslots)
            hipLaunchKernelGGL((quad_kernel<MAPK, true>), grid, dim3(kQuadThreads), 0, s, gg, W, npad, n, grab,
                               (unsigned long long)limit, cslots, sslots, out);
        else
            hipLaunchKernelGGL((quad_kernel<MAPK, false>), grid, dim3(kQuadThreads), 0, s, gg, W, npad, n, grab,
                               (unsigned long long)limit, cslots, sslots, out);
    });
    prof_end(K_QUAD, s);
    return check_launch("quad contacts");
}

int launch_count_finalize(const unsigned long long *slots, int64_t *out, hipStream_t s) {
    prof_begin(K_FINALIZE, s);
    hipLaunchKernelGGL(count_finalize_kernel, dim3(1), dim3(kSlots), 0, s, slots, out);
    prof_end(K_FINALIZE, s);
    return check_launch("count finalize");
}

SMX_CHECK_READER(check_flags_quad)

}  // namespace smx
