// rowops.hip -- the memory-bound kernels around the product: row-min
// normalisation (canonical form), operand folding for products of powers,
// input validation, traces (Corollary 7), the exact compare of the period
// search, and small fills.  All of them stream rows with 16-byte
// loads and are bounded by HBM bandwidth.
#include <algorithm>

#include "common.h"
#include "trace_rows.h"
#include "trace_tile.h"

namespace mpr {

constexpr int RB = 256;  // threads per row block

__device__ __forceinline__ uint32_t block_min_u32(uint32_t v, uint32_t *sh)
{
    v = wave_min_u32(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) sh[w] = v;
    __syncthreads();
    uint32_t r = sh[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); i++) r = sh[i] < r ? sh[i] : r;
    return r;
}
__device__ __forceinline__ int64_t block_min_i64(int64_t v, int64_t *sh)
{
    v = wave_min_i64(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) sh[w] = v;
    __syncthreads();
    int64_t r = sh[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); i++) r = sh[i] < r ? sh[i] : r;
    return r;
}
__device__ __forceinline__ uint64_t block_sum_u64(uint64_t v, uint64_t *sh)
{
    v = wave_sum_u64(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) sh[w] = v;
    __syncthreads();
    uint64_t r = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) r += sh[i];
    return r;
}

// Subtract r from a packed pair, keeping infinity; flags results > FMAX.
__device__ __forceinline__ uint32_t sub_pair(uint32_t w, uint32_t r, bool &over)
{
    uint32_t lo = w & 0xFFFFu, hi = w >> 16;
    lo = lo == 0xFFFFu ? lo : lo - r;
    hi = hi == 0xFFFFu ? hi : hi - r;
    over |= (lo != 0xFFFFu && lo > FMAX16) || (hi != 0xFFFFu && hi > FMAX16);
    return lo | (hi << 16);
}

__device__ __forceinline__ uint32_t min_pair(uint32_t m, uint32_t w) { return min(m, min(w & 0xFFFFu, w >> 16)); }

constexpr int NCH = 12;  // 16-byte chunks a thread keeps in registers

// One block per row: r = least finite entry, row -= r, R_out = R_in + r (+ add).
// Rows of up to RB * 8 * NCH entries (24576) are read from HBM once and kept
// in registers between the minimum and the subtraction; longer rows are read
// twice.
__global__ __launch_bounds__(RB) void normalise_kernel(u16 *C, int64_t ldc, int64_t N, const int64_t *R_in,
                                                       const int64_t *add_scalar, int64_t *R_out, int32_t *st,
                                                       int vec)
{
    __shared__ uint64_t sh[RB / 64];
    const int64_t i = blockIdx.x;
    u16 *row = C + i * ldc;
    uint32_t mn = 0xFFFFu;
    const bool resident = vec && N <= (int64_t)RB * 8 * NCH;
    uint4 keep[NCH];
    if (resident) {
#pragma unroll
        for (int q = 0; q < NCH; q++) {
            const int64_t c = ((int64_t)threadIdx.x + (int64_t)q * RB) * 8;
            keep[q] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
            if (c + 8 <= N) {
                keep[q] = *(const uint4 *)(row + c);
            } else if (c < N) {
                uint32_t w[4];
                for (int e = 0; e < 4; e++) {
                    const uint32_t lo = c + 2 * e < N ? row[c + 2 * e] : 0xFFFFu;
                    const uint32_t hi = c + 2 * e + 1 < N ? row[c + 2 * e + 1] : 0xFFFFu;
                    w[e] = lo | (hi << 16);
                }
                keep[q] = make_uint4(w[0], w[1], w[2], w[3]);
            }
            mn = min_pair(min_pair(mn, keep[q].x), keep[q].y);
            mn = min_pair(min_pair(mn, keep[q].z), keep[q].w);
        }
    } else if (vec) {
        for (int64_t c = (int64_t)threadIdx.x * 8; c < N; c += RB * 8) {
            if (c + 8 <= N) {
                const uint4 v = *(const uint4 *)(row + c);
                mn = min_pair(min_pair(mn, v.x), v.y);
                mn = min_pair(min_pair(mn, v.z), v.w);
            } else {
                for (int64_t j = c; j < N; j++) mn = min(mn, (uint32_t)row[j]);
            }
        }
    } else {
        for (int64_t j = threadIdx.x; j < N; j += RB) mn = min(mn, (uint32_t)row[j]);
    }
    const uint32_t r = block_min_u32(mn, (uint32_t *)sh);
    if (threadIdx.x == 0) {
        const int64_t rin = R_in ? R_in[i] : 0;
        const int64_t add = add_scalar ? *add_scalar : 0;
        const bool none = r == 0xFFFFu || rin == ROW_NONE || add == ROW_NONE;
        R_out[i] = none ? ROW_NONE : rin + (int64_t)r + add;
    }
    bool over = false;
    if (r != 0xFFFFu) {
        if (resident) {
#pragma unroll
            for (int q = 0; q < NCH; q++) {
                const int64_t c = ((int64_t)threadIdx.x + (int64_t)q * RB) * 8;
                if (c >= N) continue;
                uint32_t w[4] = {keep[q].x, keep[q].y, keep[q].z, keep[q].w};
#pragma unroll
                for (int e = 0; e < 4; e++) w[e] = sub_pair(w[e], r, over);
                if (c + 8 <= N) {
                    *(uint4 *)(row + c) = make_uint4(w[0], w[1], w[2], w[3]);
                } else {
                    for (int e = 0; e < 8 && c + e < N; e++) row[c + e] = (u16)(w[e >> 1] >> ((e & 1) * 16));
                }
            }
        } else if (vec) {
            for (int64_t c = (int64_t)threadIdx.x * 8; c < N; c += RB * 8) {
                if (c + 8 <= N) {
                    uint4 v = *(const uint4 *)(row + c);
                    uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int q = 0; q < 4; q++) w[q] = sub_pair(w[q], r, over);
                    *(uint4 *)(row + c) = make_uint4(w[0], w[1], w[2], w[3]);
                } else {
                    for (int64_t j = c; j < N; j++) {
                        uint32_t x = row[j];
                        x = x == 0xFFFFu ? x : x - r;
                        over |= x != 0xFFFFu && x > FMAX16;
                        row[j] = (u16)x;
                    }
                }
            }
        } else {
            for (int64_t j = threadIdx.x; j < N; j += RB) {
                uint32_t x = row[j];
                x = x == 0xFFFFu ? x : x - r;
                over |= x != 0xFFFFu && x > FMAX16;
                row[j] = (u16)x;
            }
        }
    }
    if (over) set_status(st, MPR_EOVERFLOW);
}

mpr_status normalise_launch(int64_t M, int64_t N, u16 *C, int64_t ldc, const int64_t *R_in,
                            const int64_t *add_scalar, int64_t *R_out, int32_t *st, hipStream_t s)
{
    if (M == 0) return MPR_OK;
    if (M > INT32_MAX) return MPR_EUNSUPPORTED;
    const int vec = aligned16(C) && ldc % 8 == 0;
    hipLaunchKernelGGL(normalise_kernel, dim3((unsigned)M), dim3(RB), 0, s, C, ldc, N, R_in, add_scalar, R_out, st, vec);
    return check_launch();
}

// The elementwise passes walk whole rows, one block a row at a time, in
// 16-byte chunks where the rows allow it (one entry per thread and a 64-bit
// division each took 58 us to check, 81 us to copy and 185 us to compare
// matrices of 7411 states; now 19, 36 and 62).
constexpr int64_t kRowBlocks = 8192;
static unsigned row_blocks(int64_t rows) { return (unsigned)std::min<int64_t>(rows, kRowBlocks); }

// 8 values of a row from column c (c < n), infinite past its end.
__device__ __forceinline__ uint4 chunk8(const gu16 *row, int64_t c, int64_t n, bool vec)
{
    if (vec && c + 8 <= n) return gload16(row + c);
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const uint32_t lo = c + 2 * e < n ? row[c + 2 * e] : 0xFFFFu;
        const uint32_t hi = c + 2 * e + 1 < n ? row[c + 2 * e + 1] : 0xFFFFu;
        w[e] = lo | (hi << 16);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}
__device__ __forceinline__ void put8(gu16 *row, int64_t c, int64_t n, bool vec, const uint4 &v)
{
    if (vec && c + 8 <= n) {
        gstore16(row + c, v);
        return;
    }
#pragma unroll
    for (int e = 0; e < 8; e++)
        if (c + e < n) row[c + e] = (u16)(comp(v, e >> 1) >> ((e & 1) * 16));
}

// Rows of any shape, for operands that need not be square: `1 << shift` lanes
// share a row (no more than it has chunks), RB >> shift rows a block, and the
// chunks of a row are split over gridDim.y where there are few rows.  A block
// to a row, whatever its length, took 302 us to check 10^6 x 8 and 8 x 8
// (with the product), now 145, and 255 us to fold and multiply 33 x 200000,
// now 178 (K = 33).
struct RowGrid {
    dim3 grid;
    int shift;
};
static RowGrid row_grid(int64_t rows, int64_t cols)
{
    const int64_t chunks = (cols + 7) / 8;
    int shift = 0;
    while ((1 << shift) < RB && (1 << shift) < chunks) shift++;
    const int64_t blocks = row_blocks((rows + (RB >> shift) - 1) / (RB >> shift));
    const int64_t parts = std::min<int64_t>((chunks + (1 << shift) - 1) >> shift, std::max<int64_t>(2048 / blocks, 1));
    return RowGrid{dim3((unsigned)blocks, (unsigned)parts), shift};
}
// body(row, first column of a chunk) for every chunk of the rows x cols.
template <class F>
__device__ __forceinline__ void row_walk(int64_t rows, int64_t cols, int shift, F body)
{
    const int64_t c0 = ((int64_t)blockIdx.y << shift) + (threadIdx.x & ((1 << shift) - 1));
    for (int64_t i = (int64_t)blockIdx.x * (RB >> shift) + (threadIdx.x >> shift); i < rows;
         i += (int64_t)gridDim.x * (RB >> shift))
        for (int64_t c = c0 * 8; c < cols; c += ((int64_t)gridDim.y << shift) * 8) body(i, c);
}

// Flags a finite entry above MPR_FMAX.
__global__ __launch_bounds__(RB) void validate_kernel(const u16 *X, int64_t rows, int64_t cols, int64_t ld, int shift,
                                                      int vec, int32_t *st)
{
    bool over = false;
    row_walk(rows, cols, shift, [&](int64_t i, int64_t c) {
        const uint4 v = chunk8(glob(X) + i * ld, c, cols, vec != 0);
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const uint32_t lo = comp(v, e) & 0xFFFFu, hi = comp(v, e) >> 16;
            over |= (lo != 0xFFFFu && lo > FMAX16) || (hi != 0xFFFFu && hi > FMAX16);
        }
    });
    if (over) set_status(st, MPR_EOVERFLOW);
}

mpr_status validate_launch(const u16 *X, int64_t rows, int64_t cols, int64_t ld, int32_t *st, hipStream_t s)
{
    if (!st || rows == 0 || cols == 0) return MPR_OK;
    const RowGrid g = row_grid(rows, cols);
    hipLaunchKernelGGL(validate_kernel, g.grid, dim3(RB), 0, s, X, rows, cols, ld, g.shift,
                       aligned16(X) && ld % 8 == 0 ? 1 : 0, st);
    return check_launch();
}

__global__ __launch_bounds__(RB) void copy_kernel(const u16 *src, int64_t lds, u16 *dst, int64_t ldd, int64_t rows,
                                                  int64_t cols, int vec)
{
    for (int64_t i = blockIdx.x; i < rows; i += gridDim.x)
        for (int64_t c = (int64_t)threadIdx.x * 8; c < cols; c += RB * 8)
            put8(glob(dst) + i * ldd, c, cols, vec != 0, chunk8(glob(src) + i * lds, c, cols, vec != 0));
}

mpr_status copy_launch(const u16 *src, int64_t lds, u16 *dst, int64_t ldd, int64_t rows, int64_t cols, hipStream_t s)
{
    if (rows == 0 || cols == 0) return MPR_OK;
    const int vec = aligned16(src) && aligned16(dst) && lds % 8 == 0 && ldd % 8 == 0;
    hipLaunchKernelGGL(copy_kernel, dim3(row_blocks(rows)), dim3(RB), 0, s, src, lds, dst, ldd, rows, cols, vec);
    return check_launch();
}

// s = min over rows with an offset of Rb[l] (ROW_NONE if none).
__global__ __launch_bounds__(1024) void min_offset_kernel(const int64_t *R, int64_t n, int64_t *out)
{
    __shared__ int64_t sh[16];
    int64_t v = ROW_NONE;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) v = R[i] < v ? R[i] : v;
    v = block_min_i64(v, sh);
    if (threadIdx.x == 0) *out = v;
}

// B'[l][j] = B[l][j] + (Rb[l] - s); infinity stays, an empty row stays empty.
__global__ __launch_bounds__(RB) void fold_kernel(const u16 *B, int64_t ldb, const int64_t *Rb, const int64_t *s_ptr,
                                                  int64_t K, int64_t N, u16 *Bp, int64_t ldp, int shift, int vec,
                                                  int32_t *st)
{
    const int64_t s = *s_ptr;
    bool over = false;
    row_walk(K, N, shift, [&](int64_t l, int64_t c) {
        const int64_t rb = Rb[l];
        // more than MPR_FMAX puts every finite entry past it
        const uint32_t add = rb == ROW_NONE ? 0u : (uint32_t)(rb - s < 0x8000 ? rb - s : 0x8000);
        const uint4 v = chunk8(glob(B) + l * ldb, c, N, vec != 0);
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            uint32_t h[2] = {comp(v, e) & 0xFFFFu, comp(v, e) >> 16};
#pragma unroll
            for (int q = 0; q < 2; q++) {
                const bool finite = h[q] != 0xFFFFu && rb != ROW_NONE;
                const bool big = finite && h[q] + add > FMAX16;
                over |= big;
                h[q] = finite && !big ? h[q] + add : 0xFFFFu;
            }
            w[e] = h[0] | (h[1] << 16);
        }
        put8(glob(Bp) + l * ldp, c, N, vec != 0, make_uint4(w[0], w[1], w[2], w[3]));
    });
    if (over) set_status(st, MPR_EOVERFLOW);
}

mpr_status fold_launch(const u16 *B, int64_t ldb, const int64_t *Rb, int64_t K, int64_t N, u16 *Bp, int64_t ldp,
                       int64_t *s_out, int32_t *st, hipStream_t s)
{
    hipLaunchKernelGGL(min_offset_kernel, dim3(1), dim3(1024), 0, s, Rb, K, s_out);
    mpr_status e = check_launch();
    if (e != MPR_OK || K == 0 || N == 0) return e;
    const int vec = aligned16(B) && aligned16(Bp) && ldb % 8 == 0 && ldp % 8 == 0;
    const RowGrid g = row_grid(K, N);
    hipLaunchKernelGGL(fold_kernel, g.grid, dim3(RB), 0, s, B, ldb, Rb, (const int64_t *)s_out, K, N, Bp, ldp, g.shift,
                       vec, st);
    return check_launch();
}

// Corollary 7: min_i (R[i] + N[i][i]).
__global__ __launch_bounds__(1024) void trace_kernel(const u16 *N, int64_t n, int64_t ld, const int64_t *R,
                                                     int64_t *out)
{
    __shared__ int64_t sh[16];
    int64_t v = ROW_NONE;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
        const uint32_t d = N[i * ld + i];
        const int64_t r = R ? R[i] : 0;
        if (d != 0xFFFFu && r != ROW_NONE) {
            const int64_t x = r + (int64_t)d;
            v = x < v ? x : v;
        }
    }
    v = block_min_i64(v, sh);
    if (threadIdx.x == 0) *out = v;
}

mpr_status trace_launch(const u16 *N, int64_t n, int64_t ld, const int64_t *R, int64_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(trace_kernel, dim3(1), dim3(1024), 0, s, N, n, ld, R, out);
    return check_launch();
}

__global__ void fill_i64_kernel(int64_t *p, int64_t count, int64_t v)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x)
        p[t] = v;
}
__global__ void fill_i32_kernel(int32_t *p, int64_t count, int32_t v)
{
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < count; t += (int64_t)gridDim.x * blockDim.x)
        p[t] = v;
}

mpr_status fill_i32_launch(int32_t *p, int64_t count, int32_t v, hipStream_t s)
{
    if (count == 0) return MPR_OK;
    const int64_t blocks = std::min<int64_t>((count + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, count, v);
    return check_launch();
}

// Trace of (RX (+) X) (x) (RY (+) Y): min over (i, l) of
// RX[i] + X[i][l] + RY[l] + Y[l][i], one tile per block (trace_tile.h).
__global__ __launch_bounds__(256) void trace_product_kernel(const u16 *X, const int64_t *RX, const u16 *Y,
                                                            const int64_t *RY, int64_t n, int64_t ld, int64_t *out,
                                                            int vec, int chunk)
{
    // `chunk` consecutive tiles per block, a running minimum, and one fold
    // into the result word per block.
    __shared__ TPShared sh;
    const int64_t tiles = (n + TPI - 1) / TPI, total = tiles * tiles;
    const int64_t t0 = (int64_t)blockIdx.x * chunk, t1 = t0 + chunk < total ? t0 + chunk : total;
    int64_t best = ROW_NONE;
    for (int64_t t = t0; t < t1; t++) {
        int64_t ti, tl;
        tp_tile_of(t, tiles, ti, tl);
        const int64_t v = tp_tile(X, RX, Y, RY, n, ld, ti * TPI, tl * TPL, vec != 0, sh);
        best = v < best ? v : best;
        __syncthreads();  // the next tile reuses sh
    }
    if (threadIdx.x == 0) tp_fold_min(out, best);
}

mpr_status trace_product_launch(const u16 *X, const int64_t *RX, const u16 *Y, const int64_t *RY, int64_t n,
                                int64_t ld, int64_t *out, hipStream_t s)
{
    static_assert(TPI == TPL, "square tiles");
    hipLaunchKernelGGL(fill_i64_kernel, dim3(1), dim3(64), 0, s, out, (int64_t)1, ROW_NONE);
    mpr_status e = check_launch();
    if (e != MPR_OK || n == 0) return e;
    const int64_t tiles = (n + TPI - 1) / TPI;
    const int vec = aligned16(X) && aligned16(Y) && ld % 8 == 0;
    const int64_t grid = tp_blocks(tiles);  // <= 2^18 for n <= 65536
    if (grid > INT32_MAX) return MPR_EUNSUPPORTED;
    hipLaunchKernelGGL(trace_product_kernel, dim3((unsigned)grid), dim3(256), 0, s, X, RX, Y, RY, n, ld, out, vec,
                       tp_chunk(tiles));
    return check_launch();
}

// Trace of (RX (+) X) (x) Y with Y given as the canonical form (YT, CY) of
// its transpose: TR_ROWS rows per block (trace_rows.h).
__global__ __launch_bounds__(256) void trace_product_t_kernel(const u16 *X, const int64_t *RX, const u16 *YT,
                                                              const int64_t *CY, int64_t n, int64_t ld,
                                                              int64_t *out, int vec)
{
    tr_rows(X, RX, YT, CY, n, ld, (int64_t)blockIdx.x * TR_ROWS, vec != 0, out);
}

mpr_status trace_product_t_launch(const u16 *X, const int64_t *RX, const u16 *YT, const int64_t *CY, int64_t n,
                                  int64_t ld, int64_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(fill_i64_kernel, dim3(1), dim3(64), 0, s, out, (int64_t)1, ROW_NONE);
    mpr_status e = check_launch();
    if (e != MPR_OK || n == 0) return e;
    const int64_t grid = tr_blocks(n);
    if (grid > INT32_MAX) return MPR_EUNSUPPORTED;
    const int vec = aligned16(X) && aligned16(YT) && ld % 8 == 0;
    hipLaunchKernelGGL(trace_product_t_kernel, dim3((unsigned)grid), dim3(256), 0, s, X, RX, YT, CY, n, ld, out, vec);
    return check_launch();
}

// dst = src^T for an n x n matrix, 64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void transpose_kernel(const u16 *src, int64_t lds, u16 *dst, int64_t ldd, int64_t n)
{
    __shared__ u16 t[64][66];
    const int64_t tiles = (n + 63) / 64;
    const int64_t i0 = ((int64_t)blockIdx.x / tiles) * 64, j0 = ((int64_t)blockIdx.x % tiles) * 64;
    const int c = (int)(threadIdx.x & 63), r = (int)(threadIdx.x >> 6);
#pragma unroll
    for (int k = 0; k < 16; k++) {  // rows i0 + r + 4k of src, columns j0 + c
        const int64_t i = i0 + r + 4 * k, j = j0 + c;
        t[r + 4 * k][c] = (i < n && j < n) ? src[i * lds + j] : (u16)0xFFFF;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 16; k++) {  // rows j0 + r + 4k of dst, columns i0 + c
        const int64_t j = j0 + r + 4 * k, i = i0 + c;
        if (i < n && j < n) dst[j * ldd + i] = t[c][r + 4 * k];
    }
}

mpr_status transpose_launch(const u16 *src, int64_t lds, u16 *dst, int64_t ldd, int64_t n, hipStream_t s)
{
    if (n == 0) return MPR_OK;
    const int64_t tiles = (n + 63) / 64;
    if (tiles * tiles > INT32_MAX) return MPR_EUNSUPPORTED;
    hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)(tiles * tiles)), dim3(256), 0, s, src, lds, dst, ldd, n);
    return check_launch();
}

// Exact compare of two canonical forms up to a scalar shift.
// out3[0] = number of differing entries of N plus rows whose emptiness
// differs, out3[1] / out3[2] = min / max of RY[i] - RX[i] over non-empty rows.
__global__ __launch_bounds__(RB) void compare_kernel(const u16 *X, const int64_t *RX, const u16 *Y, const int64_t *RY,
                                                     int64_t n, int64_t rows, int64_t cols, int64_t ld, int vec,
                                                     int64_t *out3)
{
    __shared__ int64_t sh[RB / 64];
    int64_t diff = 0, lo = ROW_NONE, hi = -ROW_NONE;
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
        for (int64_t c = (int64_t)threadIdx.x * 8; i < rows && c < cols; c += RB * 8) {
            const uint4 x = chunk8(glob(X) + i * ld, c, cols, vec != 0), y = chunk8(glob(Y) + i * ld, c, cols, vec != 0);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t d = comp(x, e) ^ comp(y, e);
                diff += ((d & 0xFFFFu) != 0) + ((d >> 16) != 0);
            }
        }
        if (threadIdx.x == 0) {
            const bool ex = RX[i] == ROW_NONE, ey = RY[i] == ROW_NONE;
            diff += ex != ey;
            if (!ex && !ey) {
                const int64_t d = RY[i] - RX[i];
                lo = d < lo ? d : lo;
                hi = d > hi ? d : hi;
            }
        }
    }
    diff = (int64_t)block_sum_u64((uint64_t)diff, (uint64_t *)sh);
    if (threadIdx.x != 0) return;
    if (diff) atomicAdd((unsigned long long *)&out3[0], (unsigned long long)diff);
    if (lo != ROW_NONE) atomicMin((long long *)&out3[1], (long long)lo);
    if (hi != -ROW_NONE) atomicMax((long long *)&out3[2], (long long)hi);
}

__global__ void compare_init_kernel(int64_t *out3)
{
    out3[0] = 0;
    out3[1] = ROW_NONE;
    out3[2] = -ROW_NONE;
}

mpr_status compare_rows_launch(const u16 *X, const int64_t *RX, const u16 *Y, const int64_t *RY, int64_t n, int64_t rows,
                               int64_t cols, int64_t ld, int64_t *out3, hipStream_t s)
{
    hipLaunchKernelGGL(compare_init_kernel, dim3(1), dim3(1), 0, s, out3);
    mpr_status e = check_launch();
    if (e != MPR_OK || n == 0) return e;
    const int vec = aligned16(X) && aligned16(Y) && ld % 8 == 0;
    const unsigned blocks = (unsigned)std::min<int64_t>(n, 2048);  // three atomics each
    hipLaunchKernelGGL(compare_kernel, dim3(blocks), dim3(RB), 0, s, X, RX, Y, RY, n, rows, cols, ld, vec, out3);
    return check_launch();
}

}  // namespace mpr
