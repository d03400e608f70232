// Compact fit of fixed patterns (Section "Fixed-pattern construction and
// fitting", Eq. fit-objective; the fitting step of Algorithm "calibration";
// Appendix "Compact fitting and storage").
//
// Targets: the mean attention of a head, its causal entries floored at 1e-9
// and each row renormalised, Pi(i, j) = max(A(i, j), floor) / s(i).  One pass
// gives the row sums s(i) (fit_rowsum_kernel, one wavefront per row); a second
// pass (fit_target_kernel) gives eta_abs (column sums of Pi), eta_rel (its
// diagonal sums) and sum Pi ln Pi in one read of the triangle (saf_tri.h);
// block partials of the marginals are added atomically, the entropy partial
// goes to a slot of its own.  Both are bound by their reads: 152 us together
// for 12 heads at T = 4096 (2 x 403 MB, 5.3 TB/s, part of the second read from
// the last-level cache; 765 us when the second pass
// walked columns and diagonals separately and the first read 4 bytes a lane).
//
// Fitter: alpha = 0, rho(delta) = log max(eta_rel(delta) / (T - delta),
// floor), then Adam steps on Eq. fit-objective.  One step is three launches
// for all heads at once: the row normalisers (fit_norm_kernel), the marginals
// of the fitted pattern P(i, j) = exp(alpha(j) + rho(i - j) - log Z(i))
// (fit_marginals_kernel), and the update (fit_adam_kernel: the gradient
// (marginal - eta) / T, Adam's moments and step; it also clears the sums for
// the next step).  After the last step the forward's fixed_lse_kernel gives
// log Z, and fit_kl_kernel the acceptance KL, L + (1/T) sum Pi ln Pi with
// L = (1/T)(sum_i log Z(i) - eta_abs . alpha - eta_rel . rho), in float64.
#pragma once

#include "saf_common.h"
#include "saf_tri.h"

namespace saf {

constexpr float FIT_ADAM_BETA1 = 0.9f;
constexpr float FIT_ADAM_BETA2 = 0.999f;
constexpr float FIT_ADAM_EPS = 1e-8f;

struct FitArgs {
    const float* mean;   // [H, T, T] (targets only)
    float* rowsum;       // [H, T]: 1 / row sum
    float* eta_abs;      // [H, T]
    float* eta_rel;      // [H, T]
    double* part;        // [H, lower blocks]: per block sum of Pi ln Pi
    double* neg_entropy; // [H]
    float* alpha;        // [H, T]
    float* rho;          // [H, T]
    float* m;            // [2, H, T]: Adam first moments of alpha, rho
    float* v;            // [2, H, T]: second moments
    float* col;          // [H, T]: column sums of the fitted pattern
    float* diag;         // [H, T]: its diagonal sums
    float* logz;         // [H, T]
    float* kl;           // [H]
    float floor_value, lr, bc1, bc2;  // bias corrections 1 - beta^t of this step
    int H, T, n_rchunks;  // n_rchunks: 256-row blocks of the targets
    // Fit loop (the targets leave rowsum and part to it):
    float* zsum;         // [H, T]: Z(i) exp(-A - R) of the step
    float* shifts;       // [H, n_rchunks, 2]: maxima of alpha and rho over each 256 entries
    int n_blocks, n_btiles, per_head;  // 32-entry blocks, tiles of 32 blocks, workgroups of a head
};

__device__ __forceinline__ float fit_wave_sum(float x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
    return x;
}
__device__ __forceinline__ double fit_wave_sum(double x) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) x += __shfl_xor(x, off);
    return x;
}

// 1 / s(i), s(i) = sum_{j <= i} max(A(i, j), floor): one wavefront per row,
// 16 bytes a lane and step.
__global__ __launch_bounds__(256) void fit_rowsum_kernel(FitArgs p) {
    const int rows_per_head = (p.T + 3) / 4;
    const int h = (int)(blockIdx.x / rows_per_head);
    const int i = (rows_per_head - 1 - (int)(blockIdx.x % rows_per_head)) * 4 + (int)(threadIdx.x >> 6);  // longest first
    const int lane = threadIdx.x & 63;
    if (i >= p.T) return;
    const float* row = p.mean + ((size_t)h * p.T + i) * p.T;
    const float fl = p.floor_value;
    float s0 = 0.0f, s1 = 0.0f;
    int j = 4 * lane;
    for (; j + 256 + 3 <= i; j += 512) {
        const TriQuad a = *reinterpret_cast<const TriQuad*>(row + j);
        const TriQuad b = *reinterpret_cast<const TriQuad*>(row + j + 256);
        s0 += (fmaxf(a.x[0], fl) + fmaxf(a.x[1], fl)) + (fmaxf(a.x[2], fl) + fmaxf(a.x[3], fl));
        s1 += (fmaxf(b.x[0], fl) + fmaxf(b.x[1], fl)) + (fmaxf(b.x[2], fl) + fmaxf(b.x[3], fl));
    }
    for (; j <= i; j += 256)
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (j + k <= i) s0 += fmaxf(row[j + k], fl);
    const float s = fit_wave_sum(s0 + s1);
    if (lane == 0) p.rowsum[(size_t)h * p.T + i] = 1.0f / s;
}

// Block (head, 256 rows, 256 columns); see the header comment.
__global__ __launch_bounds__(TRI_COLS) void fit_target_kernel(FitArgs p) {
    __shared__ double red[TRI_COLS / 64];
    __shared__ TriShared sh;
    int h, k, r, c;
    if (!tri_block_of(blockIdx.x, p.H, p.n_rchunks, h, k, r, c)) return;
    const int T = p.T;
    const float* __restrict__ s = p.rowsum + (size_t)h * T;
    const float fl = p.floor_value;
    float ent = 0.0f;  // sum of Pi log2(Pi)
    tri_block(p.mean + (size_t)h * T * T, T, r * TRI_ROWS, c * TRI_COLS, sh, p.eta_abs + (size_t)h * T, p.eta_rel + (size_t)h * T,
              [&](float m, int i) {
                  const float pc = fmaxf(m, fl) * s[i];
                  ent += pc * __builtin_amdgcn_logf(pc);
                  return pc;
              });
    const double e = fit_wave_sum((double)ent) * 0.6931471805599453;  // ln 2
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < TRI_COLS / 64; ++w) t += red[w];
        p.part[k] = t;
    }
}

// neg_entropy[h] = sum of the head's block partials; one workgroup per head.
__global__ __launch_bounds__(256) void fit_entropy_kernel(FitArgs p) {
    __shared__ double red[4];
    const int h = (int)blockIdx.x;
    const int n = tri_lower(p.n_rchunks);
    double t = 0.0;
    for (int k = (int)threadIdx.x; k < n; k += 256) t += p.part[(size_t)h * n + k];
    t = fit_wave_sum(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0) p.neg_entropy[h] = (red[0] + red[1]) + (red[2] + red[3]);
}

// This workgroup's maxima of alpha and rho (256 entries of a head).
__device__ __forceinline__ void fit_put_shifts(const FitArgs& p, float a, float r, float* red) {
    a = wave_max(a);
    r = wave_max(r);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = a;
        red[4 + (threadIdx.x >> 6)] = r;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const float* x = red + 4 * threadIdx.x;
        p.shifts[2 * (size_t)blockIdx.x + threadIdx.x] = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    }
}

// alpha = 0, rho = log max(eta_rel / (T - delta), floor); moments and sums
// cleared.  Workgroup = 256 entries of a head.
__global__ __launch_bounds__(256) void fit_init_kernel(FitArgs p) {
    __shared__ float red[8];
    const size_t n = (size_t)p.H * p.T;
    const int h = (int)(blockIdx.x / p.n_rchunks);
    const int delta = (int)(blockIdx.x % p.n_rchunks) * 256 + (int)threadIdx.x;
    const size_t k = (size_t)h * p.T + delta;
    float a = -INFINITY, r = -INFINITY;
    if (delta < p.T) {
        a = 0.0f;
        r = logf(fmaxf(p.eta_rel[k] / (float)(p.T - delta), p.floor_value));
        p.alpha[k] = a;
        p.rho[k] = r;
        p.m[k] = 0.0f;
        p.m[n + k] = 0.0f;
        p.v[k] = 0.0f;
        p.v[n + k] = 0.0f;
        p.col[k] = 0.0f;
        p.diag[k] = 0.0f;
        p.zsum[k] = 0.0f;
    }
    fit_put_shifts(p, a, r, red);
}

// ---------------------------------------------------------------------------
// One step's normalisers and marginals as products with Toeplitz matrices.
//
// With A and R the maxima of alpha and rho over the head, ea = exp(alpha - A),
// er = exp(rho - R), Z'(i) = Z(i) exp(-A - R) and w = 1 / Z',
//     Z'(i)  = sum_j er(i - j) ea(j)                    (a causal convolution),
//     col(j) = ea(j) sum_i er(i - j) w(i),
//     dia(d) = er(d) sum_i ea(i - d) w(i)               (two correlations).
// Cut every vector into blocks of 32.  For one block distance D, the terms of
// a convolution are a 32 x 32 Toeplitz matrix of er (entry er(32 D + row -
// column), 0 at negative offsets) times the blocks of ea, one column per
// block: 16 float32 MFMAs (32x32x2) for 32 columns, that is for 1024 results
// and 32 of their distances, where a lane reads 16 + 16 staged values.  (One
// multiply-add per entry and lane takes as many vector instructions and LDS
// reads as entries; the float32 matrix cores do 32 a cycle and SIMD.)  The
// products and sums are float32, as before; a common shift per head replaces
// the shift per block, and rows whose Z' lies below 2^-57 (FAST_GUARD) take
// no part in the products and are added entry by entry instead.
//
// Workgroup = (head, 32 columns of blocks, DCH distances), the distances
// shared out to the wavefronts; their tiles are added in LDS and the sums
// added to memory by float32 atomics.  Bound by the matrix cores (7680 MFMA
// cycles a SIMD for the two correlations of 12 heads at T = 4096) and by
// latency: staging, a few dozen MFMAs a wavefront, the atomics.
// 12 heads at T = 4096: 6.2 us (normalisers) and 10.6 us (marginals) a step,
// 19.4 us with the update, against 21 + 24 + 5 us (46.4 us a step) for one
// multiply-add per entry and lane.
// ---------------------------------------------------------------------------
constexpr int FIT_THREADS = 512;
constexpr int FIT_WAVES = FIT_THREADS / 64;
constexpr int FIT_SPAN = 1024;                           // results per workgroup: 32 blocks
// DCH: block distances per workgroup, 16, 8 or 4 (saf_compact_fit's rule).
template <int DCH> constexpr int fit_nx() { return 32 * DCH + 31; }  // staged offsets 32 D0 - 31 .. 32 (D0 + DCH) - 1
template <int DCH> constexpr int fit_nb() { return 32 + DCH - 1; }   // staged blocks of the other factor
constexpr int FIT_BSTRIDE = 36;                          // floats per staged block: conflict-free 16-byte reads by column
constexpr float FIT_MIN_Z = 0x1p-57f;

// A and R of head h: the largest of its chunks' maxima of alpha and rho, as
// the last update (or the initialisation) left them.  Every wavefront reads
// them for itself.
__device__ __forceinline__ void fit_shifts(const FitArgs& p, int h, float& A, float& R) {
    A = -INFINITY;
    R = -INFINITY;
    for (int x = (int)(threadIdx.x & 63); x < p.n_rchunks; x += 64) {
        const f32x2 m = *reinterpret_cast<const f32x2*>(p.shifts + 2 * ((size_t)h * p.n_rchunks + x));
        A = fmaxf(A, m[0]);
        R = fmaxf(R, m[1]);
    }
    A = wave_max(A);
    R = wave_max(R);
}

__device__ __forceinline__ float fit_exp(float x, float shift) { return fast_exp2((x - shift) * LOG2E); }

// Entries first .. first + N - 1 of x, N / FIT_THREADS a thread, -inf outside 0 .. T - 1 (loads
// only: a launch is short, so everything it reads is asked for at once).
template <int N>
struct FitLoad {
    float v[(N + FIT_THREADS - 1) / FIT_THREADS];
    __device__ __forceinline__ void operator()(const float* x, int first, int T) {
#pragma unroll
        for (int u = 0; u < (N + FIT_THREADS - 1) / FIT_THREADS; ++u) {
            const int k = first + (int)threadIdx.x + FIT_THREADS * u;
            v[u] = (unsigned)k < (unsigned)T ? x[k] : -INFINITY;
        }
    }
    // put(position, exp(x - shift)) for each entry (0 outside).
    template <typename Put>
    __device__ __forceinline__ void put(float shift, Put put) const {
#pragma unroll
        for (int u = 0; u < (N + FIT_THREADS - 1) / FIT_THREADS; ++u) {
            const int k = (int)threadIdx.x + FIT_THREADS * u;
            if (k < N) put(k, fit_exp(v[u], shift));
        }
    }
};

// This workgroup's head, tile of 32 blocks and first distance; `count` gives
// a tile's distances.  The tiles with most distances come first.  False for
// a workgroup past the head's last.
template <int DCH, typename Count>
__device__ __forceinline__ bool fit_place(int n_tiles, int per_head, bool ascending, Count count, int& h, int& c,
                                          int& d0) {
    h = (int)(blockIdx.x / per_head);
    int k = (int)(blockIdx.x % per_head);
    for (int u = 0; u < n_tiles; ++u) {
        c = ascending ? u : n_tiles - 1 - u;
        const int n = (count(c) + DCH - 1) / DCH;
        if (k < n) {
            d0 = k * DCH;
            return true;
        }
        k -= n;
    }
    return false;
}

// The wavefronts' 32 x 32 tiles in LDS, and their sum at x = 32 * column + row.
__device__ __forceinline__ void fit_put_tile(float* tiles, const f32x16& acc) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    float* t = tiles + w * (32 * 33) + (lane & 31) * 33;
#pragma unroll
    for (int v = 0; v < 16; ++v) t[8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)] = acc[v];
}
__device__ __forceinline__ float fit_get_tile(const float* tiles, int x) {
    const int at = (x >> 5) * 33 + (x & 31);
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < FIT_WAVES; w += 2) s += tiles[w * (32 * 33) + at] + tiles[(w + 1) * (32 * 33) + at];
    return s;
}

// Sixteen consecutive floats of a staged block column.
__device__ __forceinline__ void fit_block(const float* b, float (&y)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(b + 4 * q);
#pragma unroll
        for (int u = 0; u < 4; ++u) y[4 * q + u] = v[u];
    }
}

// Z'(i), added into p.zsum (cleared by the step before).  Contraction slot
// (t, half k) of a distance stands for column 16 k + t of the block.
template <int DCH>
__global__ __launch_bounds__(FIT_THREADS) void fit_norm_kernel(FitArgs p) {
    constexpr int NX = fit_nx<DCH>(), NB = fit_nb<DCH>();
    __shared__ float er[NX + 1];
    __shared__ __attribute__((aligned(16))) float ea[NB * FIT_BSTRIDE];
    __shared__ float tiles[FIT_WAVES * 32 * 33];
    int h, c, d0;
    const int nb = p.n_blocks;
    auto count = [&](int t) { return min(32 * t + 32, nb); };
    if (!fit_place<DCH>(p.n_btiles, p.per_head, false, count, h, c, d0)) return;
    const int T = p.T, tid = (int)threadIdx.x;
    const float* __restrict__ al = p.alpha + (size_t)h * T;
    const float* __restrict__ rh = p.rho + (size_t)h * T;
    const int b0 = 32 * c - d0 - (DCH - 1);  // first staged block of ea
    FitLoad<NX> lr;
    FitLoad<32 * NB> la;
    lr(rh, 32 * d0 - 31, T);
    la(al, 32 * b0, T);
    float A, R;
    fit_shifts(p, h, A, R);
    lr.put(R, [&](int x, float v) { er[x] = v; });
    la.put(A, [&](int x, float v) { ea[(x >> 5) * FIT_BSTRIDE + (x & 31)] = v; });
    __syncthreads();
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, k = lane >> 5;
    const int d1 = min(d0 + DCH, count(c));
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    for (int d = d0 + w; d < d1; d += FIT_WAVES) {
        float b[16];
        fit_block(ea + (col + 32 * c - d - b0) * FIT_BSTRIDE + 16 * k, b);
        const float* e = er + 32 * (d - d0) + col - 16 * k + 31;  // er(32 d + row - 16 k), row = col here
#pragma unroll
        for (int t = 0; t < 16; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(e[-t], b[t], acc, 0, 0, 0);
    }
    fit_put_tile(tiles, acc);
    __syncthreads();
    for (int x = tid; x < FIT_SPAN; x += FIT_THREADS) {
        const int i = FIT_SPAN * c + x;
        if (i < T) atomicAdd(p.zsum + (size_t)h * T + i, fit_get_tile(tiles, x));
    }
}

// col(j) and dia(d), added into p.col and p.diag (cleared by the step before).
template <int DCH>
__global__ __launch_bounds__(FIT_THREADS) void fit_marginals_kernel(FitArgs p) {
    constexpr int NX = fit_nx<DCH>(), NB = fit_nb<DCH>();
    __shared__ float er[NX + 1], ea[NX + 1];
    __shared__ __attribute__((aligned(16))) float ws[NB * FIT_BSTRIDE];
    __shared__ float tiles[FIT_WAVES * 32 * 33];
    __shared__ float red[2][FIT_WAVES];
    int h, c, d0;
    const int nb = p.n_blocks;
    auto count = [&](int t) { return nb - 32 * t; };
    if (!fit_place<DCH>(p.n_btiles, p.per_head, true, count, h, c, d0)) return;
    const int T = p.T, tid = (int)threadIdx.x;
    const float* __restrict__ al = p.alpha + (size_t)h * T;
    const float* __restrict__ rh = p.rho + (size_t)h * T;
    const float* __restrict__ zs = p.zsum + (size_t)h * T;
    const int i0 = 32 * (32 * c + d0);  // first staged row of w
    FitLoad<NX> lr, la;
    FitLoad<32 * NB> lz;
    FitLoad<FIT_SPAN> oa, orh;  // alpha and rho of the results
    lr(rh, 32 * d0 - 31, T);
    la(al, 32 * d0 - 31, T);
    lz(zs, i0, T);
    oa(al, FIT_SPAN * c, T);
    orh(rh, FIT_SPAN * c, T);
    float A, R;
    fit_shifts(p, h, A, R);
    lr.put(R, [&](int x, float v) { er[x] = v; });
    la.put(A, [&](int x, float v) { ea[x] = v; });
    bool low = false;  // a row of this tile that the products leave out
#pragma unroll
    for (int u = 0; u < (32 * NB + FIT_THREADS - 1) / FIT_THREADS; ++u) {
        const int x = tid + FIT_THREADS * u;
        const bool row = i0 + x < T;
        const bool small = row && lz.v[u] < FIT_MIN_Z;
        if (x < FIT_SPAN) low |= small;
        if (x < 32 * NB) ws[(x >> 5) * FIT_BSTRIDE + (x & 31)] = row && !small ? 1.0f / lz.v[u] : 0.0f;
    }
    const bool any_low = __syncthreads_or(low);
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, k = lane >> 5;
    const int d1 = min(d0 + DCH, count(c));
    f32x16 ac, ad;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        ac[v] = 0.0f;
        ad[v] = 0.0f;
    }
    for (int d = d0 + w; d < d1; d += FIT_WAVES) {
        float b[16];
        fit_block(ws + (col + d - d0) * FIT_BSTRIDE + 16 * k, b);
        const int at = 32 * (d - d0) - col + 16 * k + 31;  // offset 32 d + 16 k - row, row = col here
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            ac = __builtin_amdgcn_mfma_f32_32x32x2f32(er[at + t], b[t], ac, 0, 0, 0);
            ad = __builtin_amdgcn_mfma_f32_32x32x2f32(ea[at + t], b[t], ad, 0, 0, 0);
        }
    }
    const size_t base = (size_t)h * T;
    fit_put_tile(tiles, ac);
    __syncthreads();
    oa.put(A, [&](int x, float e) {
        if (FIT_SPAN * c + x < T) atomicAdd(p.col + base + FIT_SPAN * c + x, e * fit_get_tile(tiles, x));
    });
    __syncthreads();
    fit_put_tile(tiles, ad);
    __syncthreads();
    orh.put(R, [&](int x, float e) {
        if (FIT_SPAN * c + x < T) atomicAdd(p.diag + base + FIT_SPAN * c + x, e * fit_get_tile(tiles, x));
    });
    if (!any_low || d0 != 0) return;
    // Rows of this tile whose Z' is too small for the shifted products, entry
    // by entry: log Z(i) with a running maximum, then exp(alpha + rho - log Z).
    for (int i = FIT_SPAN * c; i < min(FIT_SPAN * (c + 1), T); ++i) {
        if (!(zs[i] < FIT_MIN_Z)) continue;
        float m = -INFINITY;
        for (int j = tid; j <= i; j += FIT_THREADS) m = fmaxf(m, al[j] + rh[i - j]);
        m = wave_max(m);
        if (lane == 0) red[0][w] = m;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < FIT_WAVES; ++u) m = fmaxf(m, red[0][u]);
        float s = 0.0f;
        for (int j = tid; j <= i; j += FIT_THREADS) s += fast_exp2((al[j] + rh[i - j] - m) * LOG2E);
        s = fit_wave_sum(s);
        if (lane == 0) red[1][w] = s;
        __syncthreads();
        s = 0.0f;
#pragma unroll
        for (int u = 0; u < FIT_WAVES; ++u) s += red[1][u];
        const float lz = m + __log2f(s) * LN2;
        for (int j = tid; j <= i; j += FIT_THREADS) {
            const float pv = fast_exp2((al[j] + rh[i - j] - lz) * LOG2E);
            atomicAdd(p.col + base + j, pv);
            atomicAdd(p.diag + base + i - j, pv);
        }
    }
}

// One Adam step on alpha and rho; clears the sums it read.  Workgroup = 256
// entries of a head, one per thread, every load issued at once; it leaves its
// entries' maxima for the next step's shifts.
__global__ __launch_bounds__(256) void fit_adam_kernel(FitArgs p) {
    __shared__ float red[8];
    const size_t n = (size_t)p.H * p.T;
    const int h = (int)(blockIdx.x / p.n_rchunks);
    const int j = (int)(blockIdx.x % p.n_rchunks) * 256 + (int)threadIdx.x;
    const size_t k = (size_t)h * p.T + j;
    const float invT = 1.0f / (float)p.T;
    float th[2] = {-INFINITY, -INFINITY};
    if (j < p.T) {
        const float g[2] = {(p.col[k] - p.eta_abs[k]) * invT, (p.diag[k] - p.eta_rel[k]) * invT};
        float m[2], v[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            m[q] = p.m[(size_t)q * n + k];
            v[q] = p.v[(size_t)q * n + k];
        }
        th[0] = p.alpha[k];
        th[1] = p.rho[k];
        p.col[k] = 0.0f;
        p.diag[k] = 0.0f;
        p.zsum[k] = 0.0f;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float mq = FIT_ADAM_BETA1 * m[q] + (1.0f - FIT_ADAM_BETA1) * g[q];
            const float vq = FIT_ADAM_BETA2 * v[q] + (1.0f - FIT_ADAM_BETA2) * g[q] * g[q];
            p.m[(size_t)q * n + k] = mq;
            p.v[(size_t)q * n + k] = vq;
            const float mhat = mq / p.bc1;
            const float vhat = vq / p.bc2;
            th[q] -= p.lr * mhat / (sqrtf(vhat) + FIT_ADAM_EPS);
        }
        p.alpha[k] = th[0];
        p.rho[k] = th[1];
    }
    fit_put_shifts(p, th[0], th[1], red);
}

// kl[h] = (sum_i log Z(i) - eta_abs . alpha - eta_rel . rho + sum Pi ln Pi) / T.
__global__ __launch_bounds__(256) void fit_kl_kernel(FitArgs p) {
    __shared__ double red[4];
    const int h = (int)blockIdx.x;
    const size_t base = (size_t)h * p.T;
    double t = 0.0;
    for (int k = (int)threadIdx.x; k < p.T; k += 256)
        t += (double)p.logz[base + k] - (double)p.eta_abs[base + k] * p.alpha[base + k] -
             (double)p.eta_rel[base + k] * p.rho[base + k];
    t = fit_wave_sum(t);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
    __syncthreads();
    if (threadIdx.x == 0)
        p.kl[h] = (float)(((red[0] + red[1]) + (red[2] + red[3]) + p.neg_entropy[h]) / (double)p.T);
}

__global__ void fit_fill_kernel(float* q, size_t n) {
    for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (size_t)gridDim.x * blockDim.x)
        q[k] = 0.0f;
}

}  // namespace saf
