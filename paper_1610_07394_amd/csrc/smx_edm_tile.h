// One tile of the packed distance matrix in the FP32 difference form (see
// smx_edm.hip), shared by the kernel of that form and by the matrix form's kernel,
// which takes it for inputs whose pairs mostly cancel.
#pragma once
#include "smx_device.h"

namespace smx {

constexpr int kEdmThreads = 256;
constexpr int kEdmKc = 32;
constexpr int kEdmLd = kEdmKc + 4;

// Stage rows [r0, r0 + 16 MT) x dims [k0, k0 + 32) of X into LDS (zero outside):
// slot (row, q) = 8 floats, 4 slots per row, MT / 4 ... MT / 2 slots per thread.
template <int MT, bool VEC>
__device__ __forceinline__ void edm_stage(float *__restrict__ sm, const float *__restrict__ X,
                                          int64_t n, int64_t d, int64_t ldx, int64_t r0, int64_t k0) {
    constexpr int T = 16 * MT;
#pragma unroll
    for (int h = 0; h < T * 4 / kEdmThreads; ++h) {
        const int slot = threadIdx.x + h * kEdmThreads;
        const int row = slot >> 2, q = slot & 3;
        const int64_t gr = r0 + row;
        float v[8];
        if (VEC) {
            // ldx % 4 == 0, 16-byte aligned base, d % 32 == 0: whole chunk in range per row
            if (gr < n) {
                const float4 *src = reinterpret_cast<const float4 *>(X + gr * ldx + k0 + 8 * q);
                const float4 a = src[0], b = src[1];
                v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
                v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = 0.f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t k = k0 + 8 * q + e;
                v[e] = (gr < n && k < d) ? X[gr * ldx + k] : 0.f;
            }
        }
        float4 *dst = reinterpret_cast<float4 *>(sm + row * kEdmLd + 8 * q);
        dst[0] = make_float4(v[0], v[1], v[2], v[3]);
        dst[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
}

// TILED: the tile-contiguous layout (tile (X, Y) at rank Y(Y+1)/2 + X times T^2,
// element (i, j) at (i mod T) T + (j mod T), entries outside i <= j < n zero).  As and
// Bs: 16 MT rows of kEdmLd floats each, 16-byte aligned.
template <int MT, bool VEC, bool TILED>
__device__ __forceinline__ void edm_diff_tile(float *As, float *Bs, int TX, int TY, const float *__restrict__ X, int64_t n,
                                              int64_t d, int64_t ldx, float *__restrict__ D) {
    constexpr int T = 16 * MT;
    const int t = threadIdx.x;
    const int tx = t & 15, ty = t >> 4;
    const int64_t r0 = int64_t(TX) * T, c0 = int64_t(TY) * T;
    const bool diag = TX == TY;

    float acc[MT][MT];
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int c = 0; c < MT; ++c) acc[r][c] = 0.f;

    for (int64_t k0 = 0; k0 < d; k0 += kEdmKc) {
        edm_stage<MT, VEC>(As, X, n, d, ldx, r0, k0);
        if (!diag) edm_stage<MT, VEC>(Bs, X, n, d, ldx, c0, k0);
        __syncthreads();
        const float *Bp = diag ? As : Bs;
#pragma unroll
        for (int kk = 0; kk < kEdmKc; kk += 4) {
            float4 a[MT], b[MT];
#pragma unroll
            for (int r = 0; r < MT; ++r) a[r] = *reinterpret_cast<const float4 *>(As + (ty + 16 * r) * kEdmLd + kk);
#pragma unroll
            for (int c = 0; c < MT; ++c) b[c] = *reinterpret_cast<const float4 *>(Bp + (tx + 16 * c) * kEdmLd + kk);
#pragma unroll
            for (int r = 0; r < MT; ++r)
#pragma unroll
                for (int c = 0; c < MT; ++c) {
                    float u;
                    u = a[r].x - b[c].x; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                    u = a[r].y - b[c].y; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                    u = a[r].z - b[c].z; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                    u = a[r].w - b[c].w; acc[r][c] = __builtin_fmaf(u, u, acc[r][c]);
                }
        }
        __syncthreads();
    }

    // a tile off the diagonal and inside n (nearly every block) stores unmasked
    const bool interior = !diag && r0 + T <= n && c0 + T <= n;
    if (TILED) {
        const uint64_t rank = uint64_t(TY) * (uint64_t(TY) + 1) / 2 + uint64_t(TX);
        float *tileD = D + rank * uint64_t(T * T) + tx;
#pragma unroll
        for (int r = 0; r < MT; ++r) {
            const int64_t i = r0 + ty + 16 * r;
            float *row = tileD + (ty + 16 * r) * T;
#pragma unroll
            for (int c = 0; c < MT; ++c) {
                const int64_t j = c0 + tx + 16 * c;
                row[16 * c] = (interior || (i < n && j < n && j >= i)) ? acc[r][c] : 0.f;
            }
        }
    } else {
#pragma unroll
    for (int r = 0; r < MT; ++r) {
        const int64_t i = r0 + ty + 16 * r;
        if (!interior && i >= n) continue;
        float *row = D + (i * n - (i * (i - 1)) / 2 - i) + c0 + tx;  // p(i, j) = i n - i(i-1)/2 + (j - i)
#pragma unroll
        for (int c = 0; c < MT; ++c) {
            const int64_t j = c0 + tx + 16 * c;
            // plain stores: measured faster than non-temporal ones here
            if (interior ? smx_check(i < n && j < n && j >= i, kCheckStore) : (j < n && (!diag || j >= i)))
                row[16 * c] = acc[r][c];
        }
    }
    }
}

}  // namespace smx
