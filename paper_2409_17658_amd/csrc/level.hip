// level.hip -- single (min,+) products on the matrix cores (level.h), and the
// choice between them and the VALU tiles of gemm.hip.
#include <algorithm>

#include "level.h"

namespace mpr {

// Tile of a block: each XCD (block b runs on XCD b % 8) takes a contiguous
// run of tiles, walked in groups of 8 tile rows, so that the 64 blocks
// resident on one XCD share 8 row and 8 column panels in its L2.
__device__ __forceinline__ bool level_tile(int tiles_m, int tiles_n, int &tm, int &tn)
{
    const int nb = (int)gridDim.x;  // a multiple of 8
    const int t = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    if (t >= tiles_m * tiles_n) return false;
    const int first = t / (8 * tiles_n) * 8, gs = min(tiles_m - first, 8), w = t - first * tiles_n;
    tm = first + w % gs;
    tn = w / gs;
    return true;
}

// A block that the levels can not hold is computed in the f16 form or in
// uint16, by its values (level_view): here, or, ELSEWHERE, by the launch behind
// this one, which its cells are marked for (gemm_past_launch).
template <class C, bool ELSEWHERE>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2))) void level_gemm_kernel(
    const u16 *__restrict__ A, int64_t lda, const u16 *__restrict__ B, int64_t ldb, u16 *__restrict__ Cm, int64_t ldc,
    int64_t M, int64_t N, int64_t K, int tiles_m, int tiles_n, int vec)
{
    using T = typename LevelBack<C>::T;
    __shared__ uint4 lds[ELSEWHERE ? C::LDS_CHUNKS : LevelLds<C>::CHUNKS];
    __shared__ int cnt[LEVEL_COUNTS];
    int tm, tn;
    if (!level_tile(tiles_m, tiles_n, tm, tn)) return;
    const int64_t m0 = (int64_t)tm * C::BM, n0 = (int64_t)tn * C::BN;
    const int rows = (int)min<int64_t>(C::BM, M - m0), cols = (int)min<int64_t>(C::BN, N - n0);
    LevelA<C> aop(glob(A) + m0 * lda, lda, rows, K);
    LevelB<C> bop(glob(B) + n0, ldb, cols, K);
    LevelView view;
    {
        LevelAcc<C> acc;
        view = level_kloop<C, true>(K, aop, bop, lds, acc, cnt);
        if (view <= LEVEL_PAST &&
            (level_sure<C>(acc, rows, cols) || (view == LEVEL_IN && level_clean<C>(K, aop, bop, lds)))) {
            level_store<C>(glob(Cm) + m0 * ldc + n0, ldc, rows, cols, acc);
            return;
        }
    }
    if constexpr (ELSEWHERE) {
        constexpr int ACROSS = C::BN / MARK_CELL;
        const int r = (int)threadIdx.x / ACROSS * MARK_CELL, c = (int)threadIdx.x % ACROSS * MARK_CELL;
        if (r < rows && c < cols) glob(Cm)[(m0 + r) * ldc + n0 + c] = view == LEVEL_U16 ? MARK_U16 : MARK_F16;
    } else {
        TileAcc<T> acc;
        tile_mainloop<T, true>(A, lda, B, ldb, M, N, K, m0, n0, vec != 0, (u16 *)lds, acc, view == LEVEL_U16);
        tile_store<T>(Cm, ldc, M, N, m0, n0, vec != 0, acc);
    }
}

template <class C, bool ELSEWHERE = false>
static mpr_status level_launch(int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B, int64_t ldb,
                               u16 *Cm, int64_t ldc, hipStream_t s, size_t pad_lds)
{
    const int64_t tiles_m = (M + C::BM - 1) / C::BM, tiles_n = (N + C::BN - 1) / C::BN;
    const int64_t tiles = tiles_m * tiles_n;
    if (tiles > (int64_t)INT32_MAX - 8) return MPR_EUNSUPPORTED;
    const bool vec = aligned16(A) && aligned16(B) && aligned16(Cm) && lda % 8 == 0 && ldb % 8 == 0 && ldc % 8 == 0;
    hipLaunchKernelGGL((level_gemm_kernel<C, ELSEWHERE>), dim3((unsigned)round_up(tiles, 8)), dim3(C::NT), pad_lds, s, A,
                       lda, B, ldb, Cm, ldc, M, N, K, (int)tiles_m, (int)tiles_n, vec ? 1 : 0);
    return check_launch();
}

// Block shape of an M x N output (0..4 = LCfg0..4).  Large blocks move and
// convert fewer operand values per output, so the largest shape is taken
// whose blocks (one per CU at 128 x 256, two at 128 x 128) fill most of the
// 256 CUs; while a CU holds only one 128 x 128 block, two groups of waves
// share its slices of K.  Measured (us, shape 0 / 1 / 2 / 3 / 4): N = 848
// 21 / 12 / 19 / 10.5 / 26; N = 1300 27 / 20 / 24 / 19 / 35; 1000 x 3333 x
// 2507 (112 blocks of 128 x 256) 50 / 54 / 45 / 57 / 66; N = 2507 (200) 68 /
// 86 / 79 / 91 / 62; N = 4096 179 / 276 / 228 / 282 / 173; N = 16384 11440 /
// 16204 / 11693 / 18066 / 9787.
int level_shape(int64_t M, int64_t N)
{
    const int64_t rows = (M + 127) / 128, tiles = rows * ((N + 127) / 128), cus = device_cu_count();
    if (rows * ((N + 255) / 256) >= cus * 3 / 4) return 4;
    return tiles >= cus ? 0 : tiles >= cus * 5 / 8 ? 2 : 3;
}

// Whether a product runs in the level form.  K >= 128: with fewer pairs per
// output the minimum of moderate values (0..40, a third infinite) often
// exceeds 30 and most blocks would be computed twice; at 128 none is expected
// to.  The staging uses 32-bit offsets and whole 8-byte pieces of a row of B.
static bool level_product(int64_t M, int64_t N, int64_t K, int64_t lda, int64_t ldb)
{
    return M > 0 && K >= 128 && N >= 4 && level_strides(lda, ldb);
}

// Tiny products: one row and two columns per thread, no LDS, 8 k in flight.
// The smallest VALU tile (64 x 64, staged through LDS) takes 9.2 us at 33 x 33
// x 33, nearly all of it latency of its first instructions, loads and
// barriers; this takes 3.8.
__global__ __launch_bounds__(256) void tiny_product_kernel(const u16 *__restrict__ A, int64_t lda,
                                                           const u16 *__restrict__ B, int64_t ldb, u16 *__restrict__ Cm,
                                                           int64_t ldc, int M, int N, int K)
{
    const int pairs = (N + 1) / 2, t = (int)(blockIdx.x * 256 + threadIdx.x), i = t / pairs, j = t % pairs * 2;
    if (i >= M) return;
    const gu16 *a = glob(A) + i * lda, *b = glob(B) + j;
    const int second = j + 1 < N ? 1 : 0;
    u16x2 m = {0xFFFF, 0xFFFF};
    int k = 0;
    for (; k + 8 <= K; k += 8) {
        u16 x[8];
        u16x2 y[8];
#pragma unroll
        for (int q = 0; q < 8; q++) {
            x[q] = a[k + q];
            const gu16 *p = b + (int64_t)(k + q) * ldb;
            y[q] = (u16x2){p[0], p[second]};
        }
#pragma unroll
        for (int q = 0; q < 8; q++) m = min2(m, add_sat((u16x2){x[q], x[q]}, y[q]));
    }
    for (; k < K; k++) {
        const gu16 *p = b + (int64_t)k * ldb;
        m = min2(m, add_sat((u16x2){a[k], a[k]}, (u16x2){p[0], p[second]}));
    }
    gu16 *c = glob(Cm) + i * ldc + j;
    c[0] = m.x;
    if (second) c[1] = m.y;
}
// Up to so many outputs (K < 128: the level form takes the others).
constexpr int64_t TINY_OUTPUTS = 1 << 14;

// Whether the blocks of a product whose values leave the levels are computed by
// a launch of their own behind the level form's, in the configuration that the
// tile table has for its size, and not where they are, in the level form's
// shape.  Where a CU would get more of the work in blocks of 128 x 256 than in
// 128 x 128, the stand-in loses to quantisation (entries 1000..10000, N = 3000:
// 1586 us, in its own launch 1003, without the level form 996); elsewhere to its
// two waves a SIMD, some 5 % (N = 2700: 770 us, 731 without the level form; N =
// 4096 with its own launch 1967 and 1946).  The launch costs a product in the
// levels 3 to 4 us (N = 3000, entries 0..40: 122 us without, 124.6), so short
// ones that quantisation spares go without.
static bool past_elsewhere(int64_t M, int64_t N, int64_t K)
{
    const int64_t rows = (M + 127) / 128, tiles = rows * ((N + 127) / 128), cus = device_cu_count();
    if (tiles < cus) return false;
    const int64_t wide = (rows * ((N + 255) / 256) + cus - 1) / cus, square = (tiles + cus - 1) / cus;
    return (level_shape(M, N) == 4 && 2 * wide > square) || (double)M * (double)N * (double)K >= 3e10;
}

mpr_status product_launch(int cfg, int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B,
                          int64_t ldb, u16 *Cm, int64_t ldc, hipStream_t s)
{
    if (cfg < 0 && M > 0 && N > 0 && K > 0 && K < 128 && M * N <= TINY_OUTPUTS) {
        const unsigned blocks = (unsigned)((M * ((N + 1) / 2) + 255) / 256);
        hipLaunchKernelGGL(tiny_product_kernel, dim3(blocks), dim3(256), 0, s, A, lda, B, ldb, Cm, ldc, (int)M, (int)N,
                           (int)K);
        return check_launch();
    }
    if (cfg >= 0 || !level_product(M, N, K, lda, ldb)) return gemm_launch(cfg, M, N, K, A, lda, B, ldb, Cm, ldc, s);
    const int shape = level_shape(M, N);
    if (past_elsewhere(M, N, K)) {  // shape 0 or 4
        const mpr_status e = shape == 4 ? level_launch<LCfg4, true>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0)
                                        : level_launch<LCfg0, true>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0);
        return e != MPR_OK ? e : gemm_past_launch(false, M, N, K, A, lda, B, ldb, Cm, ldc, s);
    }
    switch (shape) {
    case 0: return level_launch<LCfg0>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0);
    case 2: return level_launch<LCfg2>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0);
    case 4: return level_launch<LCfg4>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0);
    default: return level_launch<LCfg3>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0);
    }
}

mpr_status product_launch_spare(int cfg, int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B,
                                int64_t ldb, u16 *Cm, int64_t ldc, hipStream_t s)
{
    if (cfg >= 0 || !level_product(M, N, K, lda, ldb))
        return gemm_launch_spare(cfg, M, N, K, A, lda, B, ldb, Cm, ldc, s);
    // 128 x 128 blocks hold half of a CU's registers each: with so much LDS
    // that a second one does not fit, the other half stays free
    const size_t pad = 84 * 1024 - sizeof(uint4) * LCfg0::LDS_CHUNKS;
    if (level_shape(M, N) % 4 == 0) {  // and one wave a SIMD is too few for the VALU forms
        const mpr_status e = level_launch<LCfg0, true>(M, N, K, A, lda, B, ldb, Cm, ldc, s, pad);
        return e != MPR_OK ? e : gemm_past_launch(true, M, N, K, A, lda, B, ldb, Cm, ldc, s);
    }
    return level_launch<LCfg1>(M, N, K, A, lda, B, ldb, Cm, ldc, s, 0);
}

// One step of a chain (LevelStep).
template <class C, bool FIRST>
__global__ __launch_bounds__(C::NT) __attribute__((amdgpu_waves_per_eu(2))) void level_step_kernel(LevelStep p,
                                                                                                  int tiles,
                                                                                                  int32_t *st)
{
    __shared__ uint4 lds[LevelLds<C>::CHUNKS];
    int tm, tn;
    if (!level_tile(tiles, tiles, tm, tn)) return;
    level_step_block<C, typename LevelBack<C>::T, FIRST>(p, (int64_t)tm * C::BM, (int64_t)tn * C::BN, lds, st);
}

template <class C>
static mpr_status step_launch(const LevelStep &p, bool first, int32_t *st, hipStream_t s)
{
    const int64_t side = (p.n + C::BM - 1) / C::BM;
    auto kernel = first ? level_step_kernel<C, true> : level_step_kernel<C, (C::MI > 2)>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)round_up(side * side, 8)), dim3(C::NT), 0, s, p, (int)side, st);
    return check_launch();
}

mpr_status level_step_launch(const LevelStep &p, bool first, int32_t *st, hipStream_t s)
{
    switch (level_shape(p.n, p.n)) {
    case 0: case 4: return step_launch<LCfg0>(p, first, st, s);
    case 2: return step_launch<LCfg2>(p, first, st, s);
    default: return step_launch<LCfg3>(p, first, st, s);
    }
}

__global__ void level_prepare_kernel(uint32_t *low, uint32_t *big, uint32_t *past, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 2 * LEVEL_PASTS) past[i] = 0;
    if (i >= n) return;
    low[i] = big[i] = 0;  // the first power is canonical
    low[n + i] = LOW_NONE;
    big[n + i] = 0;
}

mpr_status level_prepare_launch(uint32_t *low, uint32_t *big, uint32_t *past, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(level_prepare_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, low, big, past, n);
    return check_launch();
}

}  // namespace mpr

namespace mpr {

// Whether a finite value of v is above MPR_FMAX.
__device__ __forceinline__ bool past_fmax(const uint4 &v)
{
    bool over = false;
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const uint32_t x = comp(v, e), lo = x & 0xFFFFu, hi = x >> 16;
        over |= (lo > FMAX16 && lo != 0xFFFFu) || (hi > FMAX16 && hi != 0xFFFFu);
    }
    return over;
}
// Whether a finite entry of A or B is above MPR_FMAX, as far as thread t0 of
// `step` looks.
__device__ __forceinline__ bool check_values(const u16 *A, int64_t rows_a, int64_t cols_a, int64_t lda, const u16 *B,
                                             int64_t rows_b, int64_t cols_b, int64_t ldb, int64_t t0, int64_t step)
{
    bool over = false;
    auto look = [&](const u16 *X, int64_t rows, int64_t cols, int64_t ld) {
        const int64_t per = (cols + 7) / 8, total = rows * per;
        for (int64_t t = t0; t < total; t += step) {
            const uint4 v = load8(X, ld, t / per, t % per * 8, rows, cols, ((uintptr_t)X & 15u) == 0 && ld % 8 == 0);
            over |= past_fmax(v);
        }
    };
    look(A, rows_a, cols_a, lda);
    look(B, rows_b, cols_b, ldb);
    return over;
}
// The verdict in rec[0] (host memory).  One block also ends the record; more
// blocks leave that to check_end_kernel.
__global__ __launch_bounds__(1024) void check_kernel(const u16 *A, int64_t rows_a, int64_t cols_a, int64_t lda,
                                                     const u16 *B, int64_t rows_b, int64_t cols_b, int64_t ldb,
                                                     int64_t *rec, int64_t seq)
{
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool any = __syncthreads_or(
        check_values(A, rows_a, cols_a, lda, B, rows_b, cols_b, ldb, t0, (int64_t)gridDim.x * blockDim.x));
    if (threadIdx.x != 0) return;
    if (any) __hip_atomic_store(&rec[0], (int64_t)MPR_EOVERFLOW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (gridDim.x == 1) __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
// A product of at most TINY_BLOCK pairs of outputs and its check by one block:
// the values are checked on their way into LDS, in one round trip to memory (two
// launches, the check behind the product, take 23.2 us at 33 x 33 x 33, this 19.4).
// Every wave's results have left it before the record tells of them (its
// release writes them back).
constexpr int TINY_BLOCK = 1024, TINY_VALUES = 1 << 14;
static int64_t tiny_values(int64_t M, int64_t N, int64_t K) { return M * round_up(K, 8) + K * round_up(N, 8); }
__global__ __launch_bounds__(TINY_BLOCK) void tiny_checked_kernel(const u16 *__restrict__ A, int64_t lda,
                                                                  const u16 *__restrict__ B, int64_t ldb,
                                                                  u16 *__restrict__ Cm, int64_t ldc, int M, int N, int K,
                                                                  int64_t *rec, int64_t seq)
{
    __shared__ __attribute__((aligned(16))) u16 lds[TINY_VALUES];
    const int t = (int)threadIdx.x, pa = (K + 7) / 8, pb = (N + 7) / 8, ca = M * pa, cb = K * pb;
    const bool va = ((uintptr_t)A & 15u) == 0 && lda % 8 == 0, vb = ((uintptr_t)B & 15u) == 0 && ldb % 8 == 0;
    bool over = false;
    for (int c = t; c < ca + cb; c += TINY_BLOCK) {
        const int d = c - ca;
        const uint4 v = d < 0 ? load8(A, lda, c / pa, c % pa * 8, M, K, va) : load8(B, ldb, d / pb, d % pb * 8, K, N, vb);
        *(uint4 *)(lds + 8 * c) = v;
        over |= past_fmax(v);
    }
    const bool any = __syncthreads_or(over);
    const int pairs = (N + 1) / 2, i = t / pairs, j = t % pairs * 2;
    if (i < M) {
        const u16 *a = lds + i * pa * 8, *b = lds + 8 * ca + j;
        u16x2 m = {0xFFFF, 0xFFFF};
#pragma unroll 8
        for (int k = 0; k < K; k++)
            m = min2(m, add_sat((u16x2){a[k], a[k]}, as_u16x2(*(const uint32_t *)(b + k * pb * 8))));
        gu16 *c = glob(Cm) + i * ldc + j;
        c[0] = m.x;
        if (j + 1 < N) c[1] = m.y;
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    if (t != 0) return;
    if (any) __hip_atomic_store(&rec[0], (int64_t)MPR_EOVERFLOW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__global__ void check_end_kernel(int64_t *rec, int64_t seq)
{
    __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace mpr

using namespace mpr;

// The product with its inputs checked and the verdict on the host, which waits
// for it in a pinned record that tells of the product's end too: the check is
// launched behind the product, or is part of its kernel (a device status word,
// two checks, a copy back and a synchronisation cost 43 us at 33 x 33 x 33
// through the binding, this 19.4).
extern "C" mpr_status mpr_minplus_gemm_checked(int cfg, int spare, int64_t M, int64_t N, int64_t K, const uint16_t *A,
                                               int64_t lda, const uint16_t *B, int64_t ldb, uint16_t *C, int64_t ldc,
                                               int32_t *status_host, mpr_stream stream)
{
    if (!status_host) return MPR_EINVAL;
    *status_host = 0;
    auto product = [&] {
        return spare ? mpr_minplus_gemm_spare(cfg, M, N, K, A, lda, B, ldb, C, ldc, nullptr, stream)
                     : mpr_minplus_gemm_cfg(cfg, M, N, K, A, lda, B, ldb, C, ldc, nullptr, stream);
    };
    mpr_status e = mpr_gemm_args(cfg, M, N, K, A, lda, B, ldb, C, ldc);
    if (e != MPR_OK) return e;
    if ((e = ensure_init()) != MPR_OK) return e;
    const int64_t values = M * K + K * N;
    hipStream_t s = as_stream(stream);
    if (values == 0) {
        e = product();
        return e == MPR_OK && hipStreamSynchronize(s) != hipSuccess ? MPR_EHIP : e;
    }
    HostRecord rec(s);
    if (!rec.p) return MPR_ENOMEM;
    rec.p[0] = 0;
    const bool tiny = cfg < 0 && M > 0 && N > 0 && K > 0 && K < 128 && M <= TINY_BLOCK &&
                      M * ((N + 1) / 2) <= TINY_BLOCK && tiny_values(M, N, K) <= TINY_VALUES;
    if (!tiny && (e = product()) != MPR_OK) return e;
    const int64_t seq = rec.ticket();
    if (tiny) {
        hipLaunchKernelGGL(tiny_checked_kernel, dim3(1), dim3(TINY_BLOCK), 0, s, A, lda, B, ldb, C, ldc, (int)M, (int)N,
                           (int)K, rec.p, seq);
    } else {
        const unsigned blocks = (unsigned)std::min<int64_t>(values / (8 * 8192) + 1, 2048);
        hipLaunchKernelGGL(check_kernel, dim3(blocks), dim3(1024), 0, s, A, M, K, lda, B, K, N, ldb, rec.p, seq);
        if (blocks > 1) hipLaunchKernelGGL(check_end_kernel, dim3(1), dim3(1), 0, s, rec.p, seq);
    }
    if ((e = check_launch()) == MPR_OK) e = rec.wait(rec.p, seq);
    if (e == MPR_OK) *status_host = (int32_t)rec.p[0];
    return e;
}
