// One pass over the lower triangle of a [T, T] float32 matrix: column sums
// and diagonal sums (i - j = const) of its entries, every entry read once.
//
// Workgroup = a block of 256 rows x 256 columns, wavefront w its rows
// 64 w .. 64 w + 63, lane l its columns 4 l .. 4 l + 3 (one 16-byte load per
// row, 1 KB a wavefront).  A lane sums its four columns down the rows.  The
// diagonal sums move with the rows: a register holds the running sum of the
// diagonal that meets the lane's column k in the current row, and from one row
// to the next it belongs to column k + 1, so the four registers rotate and the
// last one passes to the next lane (one DPP shift of the wavefront a row).
// The sum that leaves the block on the right in row r is kept in lane r.  The
// bound is memory: the first version walked each column and each diagonal of
// a block separately, reading every entry twice from unaligned rows.
#pragma once

#include "saf_common.h"

namespace saf {

// Row r and column c of entry k of a lower triangle counted row by row (row r
// starts at r (r + 1) / 2).
__device__ __forceinline__ void tri_entry(int k, int& r, int& c) {
    r = (int)((sqrtf(8.0f * (float)k + 1.0f) - 1.0f) * 0.5f);
    while (r * (r + 1) / 2 > k) --r;
    while ((r + 1) * (r + 2) / 2 <= k) ++r;
    c = k - r * (r + 1) / 2;
}

// Blocks of a triangle of n x n blocks for each of H heads, spread over the 8
// XCDs (to which workgroups are dealt in turn): each XCD takes a run of
// consecutive blocks, row by row, so the blocks it has in flight cover whole
// rows.  Dealing the blocks themselves in turn gives an XCD every eighth piece
// of a row, and where T is a multiple of 1024 these pieces meet a part of its
// L2 channels only (calibration call at T = 4096, 512-byte pieces: 0.350 ms so,
// 0.203 ms in runs).
__host__ __device__ inline int tri_per_xcd(int H, int blocks) { return (H * blocks + 7) / 8; }
__host__ __device__ inline int tri_lower(int n) { return n * (n + 1) / 2; }

// Block of workgroup blk in a grid of 8 tri_per_xcd(H, tri_lower(n)); false past the end.
__device__ __forceinline__ bool tri_block_of(unsigned blk, int H, int n, int& h, int& k, int& r, int& c) {
    const int lower = tri_lower(n);
    k = (int)(blk & 7) * tri_per_xcd(H, lower) + (int)(blk >> 3);
    if (k >= H * lower) return false;
    h = k / lower;
    tri_entry(k - h * lower, r, c);
    return true;
}

constexpr int TRI_COLS = 256;
constexpr int TRI_ROWS = 256;
constexpr int TRI_WROWS = TRI_ROWS / 4;  // rows of a wavefront
constexpr int TRI_STEP = 8;              // rows loaded ahead

// 16 bytes at any 4-byte boundary (rows start at multiples of T entries).
struct __attribute__((packed, aligned(4))) TriQuad {
    float x[4];
};

// LDS of a workgroup: sums of the block's columns, and of its diagonals (entry
// i - j + TRI_COLS - 1 of block-local row i and column j).
struct TriShared {
    float col[TRI_COLS];
    float dia[TRI_ROWS + TRI_COLS];
};

// Adds the sums of block (rows i0 .., columns j0 ..) of M's lower triangle to
// col[j] and dia[i - j] by float32 atomics.  value(m, i): the term an entry m
// of row i adds (called for j <= i only).  Block wholly above the diagonal:
// not to be called.  Every thread of the workgroup calls it.
template <typename Value>
__device__ __forceinline__ void tri_block(const float* __restrict__ M, int T, int i0, int j0, TriShared& sh,
                                          float* col, float* dia, Value value) {
    const int tid = (int)threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    sh.col[tid] = 0.0f;
    sh.dia[tid] = 0.0f;
    sh.dia[tid + 256] = 0.0f;
    __syncthreads();
    const int r0 = i0 + TRI_WROWS * w;             // the wavefront's first row
    const int r1 = min(r0 + TRI_WROWS, T);         // and the end of its rows
    const int j = j0 + 4 * lane;
    if (r0 < r1 && j0 <= r1 - 1) {
        float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float d[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        float out = 0.0f;  // lane r: the diagonal sum that left after row r0 + r
        const bool whole = j0 + TRI_COLS - 1 <= r0 && r1 == r0 + TRI_WROWS;  // no entry above the diagonal, no row missing
        auto row = [&](int i, const float (&m)[4], bool masked) {
            float v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = (!masked || j + k <= i) ? value(m[k], i) : 0.0f;
                c[k] += v[k];
                d[k] += v[k];
            }
            // Hand the diagonals on: column k's sum belongs to column k + 1 in the next row.
            const int last = __builtin_amdgcn_readlane(__float_as_int(d[3]), 63);
            out = lane == i - r0 ? __int_as_float(last) : out;
            const int in = __builtin_amdgcn_update_dpp(0, __float_as_int(d[3]), 0x138, 0xf, 0xf, true);  // wave_shr:1
            d[3] = d[2];
            d[2] = d[1];
            d[1] = d[0];
            d[0] = __int_as_float(in);
        };
        if (whole) {
            const float* p = M + (size_t)r0 * T + j;
            float m[2][TRI_STEP][4];
            auto load = [&](int s, int r) {
#pragma unroll
                for (int u = 0; u < TRI_STEP; ++u) {
                    const TriQuad q = *reinterpret_cast<const TriQuad*>(p + (size_t)(r + u) * T);
#pragma unroll
                    for (int k = 0; k < 4; ++k) m[s][u][k] = q.x[k];
                }
            };
            load(0, 0);
#pragma unroll
            for (int r = 0; r < TRI_WROWS; r += 2 * TRI_STEP) {
                load(1, r + TRI_STEP);
#pragma unroll
                for (int u = 0; u < TRI_STEP; ++u) row(r0 + r + u, m[0][u], false);
                if (r + 2 * TRI_STEP < TRI_WROWS) load(0, r + 2 * TRI_STEP);
#pragma unroll
                for (int u = 0; u < TRI_STEP; ++u) row(r0 + r + TRI_STEP + u, m[1][u], false);
            }
        } else {
            // Blocks that meet the diagonal or the last rows: entries above
            // the diagonal are neither read nor added.
            for (int i = r0; i < r1; i += TRI_STEP) {
                float m[TRI_STEP][4];
#pragma unroll
                for (int u = 0; u < TRI_STEP; ++u) {
                    const float* q = M + (size_t)(i + u) * T + j;
#pragma unroll
                    for (int k = 0; k < 4; ++k) m[u][k] = (i + u < r1 && j + k <= i + u) ? q[k] : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < TRI_STEP; ++u)
                    if (i + u < r1) row(i + u, m[u], true);
            }
        }
        // The sums still in the block meet row r1 at columns j + k (column 0 of
        // lane 0 holds nothing yet), the others left in rows r0 .. r1 - 1.
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            atomicAdd(&sh.col[4 * lane + k], c[k]);
            const int at = (r1 - i0) - (4 * lane + k) + TRI_COLS - 1;
            if (4 * lane + k > 0) atomicAdd(&sh.dia[at], d[k]);
        }
        if (lane < r1 - r0) atomicAdd(&sh.dia[r0 - i0 + lane], out);
    }
    __syncthreads();
    if (j0 + tid < T) atomicAdd(col + j0 + tid, sh.col[tid]);
#pragma unroll
    for (int x = tid; x < TRI_ROWS + TRI_COLS - 1; x += 256) {
        const int delta = i0 - j0 + x - (TRI_COLS - 1);
        if (delta >= 0 && delta < T) atomicAdd(dia + delta, sh.dia[x]);
    }
}

}  // namespace saf
