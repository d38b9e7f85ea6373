// sparse.hip -- the chain step N_k = N_(k-1) (x) A when A is sparse.
//
// A transfer matrix stays sparse (0.5 - 3 % finite for m = 6..9) while its
// powers are dense, so in the chain A^k = A^(k-1) (x) A only the rows l of A
// with a finite entry in an output column can contribute to that column.
// For a block J of BN output columns let L_J be those rows of A; then
//     C[:, J] = N[:, L_J] (x) A[L_J, J],
// a dense (min,+) product with inner dimension |L_J| instead of n.  A plan
// built once per matrix (on the device, no host round trip) stores, per
// block, the sorted list L_J (padded with row 0 to a multiple of BK) and the
// packed rows A[L_J, J] (padding rows infinite, so they never win).  The
// step runs the shared tile routine with the left operand gathered through
// L_J.  The result is the same product, entry for entry.
#include <algorithm>
#include <atomic>

#include "level.h"

namespace mpr {

using SCfg = TileCfg<64, 64, 32, 4, 8>;  // 128 threads; 64-column blocks
constexpr int SBN = SCfg::BN;
constexpr int SBK = SCfg::BK;

// ------------------------------------------------ the plan
// The lists take whole aligned groups of 8 rows (those below n) once one row
// of the group has a finite entry in the block's columns: a transfer matrix's
// rows hit a block in runs of about 80, so the groups add about a tenth, and
// they make 8 consecutive entries of a list 8 consecutive rows.
//
// One workgroup of 16 waves per column block.  A wave reads a group's 8 rows
// x 64 columns with one 16-byte load per lane (whole 128-byte lines, PU groups
// in flight), so a pass reads A once, coalesced; one thread per row, each
// walking its own line, took 0.57 ms to count and 1.80 ms to fill at m = 9
// (0.10 and 0.50 at m = 8); now 0.45 and 0.47 (0.056 and 0.070).
constexpr int PT = 1024;       // threads
constexpr int PW = PT / 64;    // waves
constexpr int PWIN = 8 * PT;   // groups per window (65536 rows)
constexpr int PU = 4;

// Lane (r, c) = (lane / 8, lane % 8): values 8 c .. 8 c + 7 of row 8 g + r in
// columns [j0, j0 + SBN); infinite outside the matrix.
__device__ __forceinline__ uint4 plan_load(const u16 *A, int64_t lda, int64_t n, int64_t g, int64_t j0, bool vec)
{
    const int lane = (int)(threadIdx.x & 63);
    return load8(A, lda, g * 8 + (lane >> 3), j0 + (lane & 7) * 8, n, n, vec);
}
__device__ __forceinline__ bool plan_hit(const uint4 &v)
{
    return __ballot((v.x & v.y & v.z & v.w) != 0xFFFFFFFFu) != 0;
}

// rows[g] = rows of group g0 + g in the list of column block j0 / SBN (0 when
// none hits it), for the window's `groups` groups; ends with a barrier.
__device__ __forceinline__ void plan_window(const u16 *A, int64_t lda, int64_t n, int64_t g0, int groups, int64_t j0,
                                            bool vec, uint8_t *rows)
{
    const int w = (int)(threadIdx.x >> 6);
    for (int g = w * PU; g < groups; g += PW * PU) {
        uint4 v[PU];
#pragma unroll
        for (int u = 0; u < PU; u++) v[u] = plan_load(A, lda, n, g0 + g + u, j0, vec);  // past the end: infinite
#pragma unroll
        for (int u = 0; u < PU; u++) {
            const bool hit = plan_hit(v[u]);
            if ((threadIdx.x & 63) == 0 && g + u < groups)
                rows[g + u] = hit ? (uint8_t)min<int64_t>(8, n - (g0 + g + u) * 8) : 0;
        }
    }
    __syncthreads();
}

// Exclusive sum of v over the workgroup (and the total); ends with a barrier.
__device__ __forceinline__ int plan_scan(int v, int *wsum, int &total)
{
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    int x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off, 64);
        x += lane >= off ? y : 0;
    }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int before = 0;
    total = 0;
    for (int q = 0; q < PW; q++) {
        before += q < w ? wsum[q] : 0;
        total += wsum[q];
    }
    __syncthreads();
    return before + x - v;
}

// counts[J] = |L_J| rounded up to a multiple of SBK.
__global__ __launch_bounds__(PT) void sp_count_kernel(const u16 *A, int64_t lda, int64_t n, int64_t *counts, int vec)
{
    __shared__ uint8_t rows[PWIN];
    __shared__ int wsum[PW];
    const int64_t j0 = (int64_t)blockIdx.x * SBN, groups = (n + 7) / 8;
    int64_t all = 0;
    for (int64_t g0 = 0; g0 < groups; g0 += PWIN) {
        const int cnt = (int)min<int64_t>(PWIN, groups - g0);
        plan_window(A, lda, n, g0, cnt, j0, vec != 0, rows);
        int c = 0, total;
        for (int g = (int)threadIdx.x; g < cnt; g += PT) c += rows[g];
        plan_scan(c, wsum, total);
        all += total;
    }
    if (threadIdx.x == 0) counts[blockIdx.x] = (all + SBK - 1) / SBK * SBK;
}

// off[J] = sum of counts before J, off[nblk] = total; order[r] = the column
// block with the r-th largest |L_J| (ties by index): the tile and entry forms
// launch the costliest blocks first so the launch does not end on a few long
// blocks (|L_J| varies by 50x within one transfer matrix).  One block, the
// counts in LDS when they fit; the total also goes to rec when given.
constexpr int PCOUNTS = 8 * PT;
__global__ __launch_bounds__(PT) void sp_scan_kernel(const int64_t *counts, int64_t nblk, int64_t *off, int32_t *order,
                                                     int64_t *rec, int64_t seq)
{
    __shared__ int wsum[PW];
    __shared__ int cs[PCOUNTS];
    const bool fits = nblk <= PCOUNTS;
    int64_t run = 0;
    for (int64_t b0 = 0; b0 < nblk; b0 += PT) {
        const int64_t b = b0 + threadIdx.x;
        const int c = b < nblk ? (int)counts[b] : 0;  // at most n + SBK
        if (fits && b < nblk) cs[b] = c;
        int total;
        const int before = plan_scan(c, wsum, total);
        if (b < nblk) off[b] = run + before;
        run += total;
    }
    if (threadIdx.x == 0) {
        off[nblk] = run;
        if (rec) {
            rec[0] = run;
            __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
    __syncthreads();
    for (int64_t J = threadIdx.x; J < nblk; J += PT) {
        const int c = fits ? cs[J] : (int)counts[J];
        int64_t rank = 0;
        for (int64_t K = 0; K < nblk; K++) {
            const int d = fits ? cs[K] : (int)counts[K];
            rank += (d > c) || (d == c && K < J);
        }
        order[rank] = (int32_t)J;
    }
}

// Ordered compaction of block J: idx[off[J] + t] = t-th row of L_J and
// Bp[(off[J] + t) * SBN + c] = A[l][j0 + c]; padding rows are row 0 / infinite.
// A plan whose rows (off[nblk]) exceed the capacity `cap` of its workspace
// is not written: *st = MPR_ENOMEM, and the step kernel then does nothing.
// IMAGES (the step in bytes): Bp holds the images of the values instead, 8 rows
// of a column to a 16-byte chunk, as the matrix instruction reads them, and
// top[J] the largest finite value of the block.
template <bool IMAGES>
__global__ __launch_bounds__(PT) void sp_fill_kernel(const u16 *A, int64_t lda, int64_t n, const int64_t *off,
                                                     int64_t nblk, int64_t cap, int32_t *idx, u16 *Bp, int vec,
                                                     int32_t *top, uint32_t *past, int32_t *st)
{
    if (blockIdx.x == 0 && threadIdx.x < 3 * LEVEL_PASTS) past[threadIdx.x] = 0;  // (SparsePlan)
    __shared__ uint8_t rows[PWIN];
    typedef u32x4 __attribute__((may_alias)) chunk_bits;
    __shared__ __attribute__((aligned(16))) u16 turn[IMAGES ? PW : 1][8 * SBN];  // a wave's 8 rows
    __shared__ int most;
    uint32_t mx = 0;  // largest finite value + 1
    if (threadIdx.x == 0) most = 0;
    __shared__ int pos[PWIN];
    __shared__ int wsum[PW];
    if (off[nblk] > cap) {  // uniform over the grid
        if (blockIdx.x == 0 && threadIdx.x == 0) set_status(st, MPR_ENOMEM);
        return;
    }
    const int64_t J = blockIdx.x, j0 = J * SBN, base = off[J], end = off[J + 1], groups = (n + 7) / 8;
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    int64_t run = 0;
    for (int64_t g0 = 0; g0 < groups; g0 += PWIN) {
        const int cnt = (int)min<int64_t>(PWIN, groups - g0);
        plan_window(A, lda, n, g0, cnt, j0, vec != 0, rows);
        const int per = PWIN / PT, first = (int)threadIdx.x * per;
        int mine = 0, total;
        for (int g = first; g < first + per && g < cnt; g++) mine += rows[g];
        int at = plan_scan(mine, wsum, total);
        for (int g = first; g < first + per && g < cnt; g++) {
            pos[g] = at;
            at += rows[g];
        }
        __syncthreads();
        for (int g = w * PU; g < cnt; g += PW * PU) {
            uint4 v[PU];
#pragma unroll
            for (int u = 0; u < PU; u++)
                if (g + u < cnt && rows[g + u]) v[u] = plan_load(A, lda, n, g0 + g + u, j0, vec != 0);
#pragma unroll
            for (int u = 0; u < PU; u++)
                if (g + u < cnt && (lane >> 3) < rows[g + u]) {
                    const int64_t t = base + run + pos[g + u] + (lane >> 3);
                    if constexpr (!IMAGES) gstore16(glob(Bp) + t * SBN + (lane & 7) * 8, v[u]);
                    if ((lane & 7) == 0) idx[t] = (int32_t)((g0 + g + u) * 8 + (lane >> 3));
                }
            if constexpr (IMAGES) {
#pragma unroll
                for (int u = 0; u < PU; u++)
                    if (g + u < cnt && rows[g + u]) {  // uniform in the wave; rows past n were loaded as infinite
                        ((chunk_bits *)turn[w])[lane] = (u32x4){v[u].x, v[u].y, v[u].z, v[u].w};
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        const u16 *col = turn[w] + lane;
                        uint32_t x[4];
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            const uint32_t lo = col[2 * q * SBN], hi = col[(2 * q + 1) * SBN];
                            mx = max(mx, max((lo + 1) & 0xFFFFu, (hi + 1) & 0xFFFFu));
                            x[q] = level_image(lo | hi << 16);
                        }
                        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        gstore16(glob(Bp) + (base + run + pos[g + u]) * SBN + lane * 8, make_uint4(x[0], x[1], x[2], x[3]));
                    }
            }
        }
        run += total;
        __syncthreads();
    }
    // padding up to the multiple of SBK
    const uint32_t none = IMAGES ? 0u : 0xFFFFFFFFu;
    const int64_t filled = IMAGES ? (run + 7) & ~(int64_t)7 : run;
    for (int64_t e = (base + run) * 8 + threadIdx.x; e < end * 8; e += PT) {
        if (e >= (base + filled) * 8) gstore16(glob(Bp) + e * 8, make_uint4(none, none, none, none));
        if (e % 8 == 0) idx[e / 8] = 0;
    }
    if constexpr (IMAGES) {
        if (mx) atomicMax(&most, (int)mx - 1);
        __syncthreads();
        if (threadIdx.x == 0) top[J] = most;
    }
}

// One value's f16 image (to_h16 for a single uint16): signed, 0xFFFF is -1
// and survives min(., 0x800); unsigned, it then meets 0x7C00.
__device__ __forceinline__ u16 to_h16_1(u16 x)
{
    const short c = __builtin_elementwise_min((short)x, (short)0x800);
    return __builtin_elementwise_min((u16)c, (u16)0x7C00);
}

// Left operand of the compressed-K step: N[m0 + row][L_J[k]] for the BK-deep
// slice.  Thread t handles k = t % BK (fixed: NT is a multiple of BK), so it
// reads its index once per slice, and rows t / BK + e * (NT / BK); a wave thus
// reads 32 consecutive gathered columns (sorted, mostly adjacent) of two rows
// per instruction, and the values go to LDS one 16-bit store each.
template <class T>
struct GatherA {
    static_assert(T::NT % T::BK == 0, "fixed k per thread");
    static constexpr int PER = T::BM * T::BK / T::NT;  // values per thread
    static constexpr int RSTEP = T::NT / T::BK;        // rows between them
    const gu16 *N;
    int64_t ldn, n, m0;
    const __attribute__((address_space(1))) int32_t *idx;
    bool full;  // all BM rows of the block are < n (block-uniform)
    const uint32_t *low;  // offsets to take off the rows from m0 on, or null
    uint32_t v[PER];
    __device__ __forceinline__ void load(int64_t k0)
    {
        const int k = (int)(threadIdx.x % T::BK), r0 = (int)(threadIdx.x / T::BK);
        const int64_t col = idx[k0 + k];
        if (full) {
#pragma unroll
            for (int e = 0; e < PER; e++) v[e] = N[(m0 + r0 + e * RSTEP) * ldn + col];
        } else {
#pragma unroll
            for (int e = 0; e < PER; e++) {
                const int64_t r = m0 + r0 + e * RSTEP;
                v[e] = r < n ? (uint32_t)N[r * ldn + col] : 0xFFFFu;
            }
        }
        if (low) {
#pragma unroll
            for (int e = 0; e < PER; e++)
                if (v[e] != 0xFFFFu) v[e] -= low[r0 + e * RSTEP];
        }
    }
    template <bool H>
    __device__ __forceinline__ void store(u16 *as) const
    {
        const int k = (int)(threadIdx.x % T::BK), r0 = (int)(threadIdx.x / T::BK);
#pragma unroll
        for (int e = 0; e < PER; e++)
            as[(r0 + e * RSTEP) * T::LDA_S + k] = H ? to_h16_1((u16)v[e]) : (u16)v[e];
    }
};

// One SCfg tile of C = N[:, L_J] (x) A[L_J, J], in form H (tile.h).
template <bool H>
__global__ __launch_bounds__(SCfg::NT) __attribute__((amdgpu_waves_per_eu(4))) void sp_step_kernel(const u16 *__restrict__ Np, int64_t ldn, int64_t n,
                                                           const int64_t *__restrict__ off,
                                                           const int32_t *__restrict__ order,
                                                           const int32_t *__restrict__ idx,
                                                           const u16 *__restrict__ Bp, u16 *__restrict__ C,
                                                           int64_t ldc, int tiles_m, int nblk, int64_t cap, int vec)
{
    __shared__ __attribute__((aligned(16))) u16 lds[SCfg::LDS_ELEMS];
    // Column blocks costliest first (order[]), all row tiles of one column
    // block consecutively; consecutive blocks go to different XCDs, so every
    // XCD gets the same mix of costs.
    const int t = (int)blockIdx.x;
    if (t >= tiles_m * nblk) return;
    const int tm = t % tiles_m, J = order[t / tiles_m];
    const int64_t m0 = (int64_t)tm * SCfg::BM, n0 = (int64_t)J * SBN;
    if (off[nblk] > cap) {
        // The plan did not fit its workspace (sp_fill_kernel reported it and
        // wrote nothing): the output is all infinite, so no later pass reads
        // stale values.
        TileAcc<SCfg> none;
#pragma unroll
        for (int r = 0; r < SCfg::TM; r++)
#pragma unroll
            for (int q = 0; q < SCfg::NACC; q++) none.v[r][q] = (u16x2){0xFFFF, 0xFFFF};
        tile_store<SCfg>(C, ldc, n, n, m0, n0, vec != 0, none);
        return;
    }
    const int64_t kbeg = off[J], K = off[J + 1] - kbeg;
    const gu16 *gN = glob(Np);
    const __attribute__((address_space(1))) int32_t *gi = glob(idx) + kbeg;
    const gu16 *gB = glob(Bp) + kbeg * SBN;
    TileAcc<SCfg> acc;
    GatherA<SCfg> aop{gN, ldn, n, m0, gi, m0 + SCfg::BM <= n, nullptr, {}};
    auto bop = chunk_b<SCfg>([&](int64_t k0, int kr, int jc) { return gload16(gB + (k0 + kr) * SBN + jc); });
    tile_product<SCfg, H>(K / SBK, aop, bop, lds, acc);
    tile_store<SCfg>(C, ldc, n, n, m0, n0, vec != 0, acc);
}

// ------------------------------------------- entry-list form of the step
// (by request, MPR_SPARSE_ENTRIES, and for the tiles that the level form leaves.)
// The tile above multiplies whole 64-column rows of A[L_J, J]; for a
// transfer matrix about nine in ten of those entries are infinite (a
// column has 25 to 120 finite entries, its block's L_J ten times as many),
// so nine in ten of its pairs cannot win.  This form visits the finite
// entries only.  A block takes 512 rows and one column block; each of its
// eight waves owns 8 whole columns (all 512 rows, 8 per lane), so the
// entries of a column are the same for every lane of the wave.  Per slice
// of 32 rows of L_J, the gathered N[rows, L_J-slice] is stored in LDS
// transposed (l-major), and per column a wave holds the column's 32 values
// of A (one per lane, loaded a slice ahead straight into registers), turns
// the finite ones into a wave-uniform bit mask, and for each set bit l adds
// the scalar A[l][j] to the lane's eight values N[i][l] (one 16-byte LDS
// read) and keeps the minimum.  Two columns are walked together, two reads
// in flight; a column whose mask has run out adds infinity, which changes
// nothing, and a pair with many entries in the slice walks its rows in
// order (one read for both columns, infinity where one of them has no
// entry, rows where neither has one skipped).  The same
// plan, the same minimum over the same entries: the same bits as the tile
// form.
constexpr int EBM = 512;                 // rows per block
constexpr int ENT = 512;                 // threads: 8 waves
constexpr int ECOLS = SBN / (ENT / 64);  // columns per wave
constexpr int ERL = EBM / 64;            // rows per lane
constexpr int ELDN = EBM + 8;            // transposed slice row (u16), 16-byte aligned
constexpr int E_NT = SBK * ELDN;         // one transposed slice buffer
constexpr int ERP = ENT / SBK;           // row pairs staged per slice by one k
static_assert(ENT == EBM, "one output row per thread in the epilogue");
static_assert(EBM % (2 * ERP) == 0, "staging covers the tile's rows");
static_assert(ECOLS == 8 && ERL == 8, "a lane: 8 columns of A (one 16-byte load), 8 rows (one 16-byte read)");
static_assert(SBN * ELDN <= 2 * E_NT, "the output tile fits the two slice buffers");
constexpr int kEntryDense = 12;          // more entries than this in a column's slice: walk the rows in order
constexpr int ESV = EBM / ERP;           // values a thread stages per slice

// One 512-row tile of the entry-list step; FULL: every row of the tile is
// < n (so the gathers need no row test).  LATE: the rows lose their offsets
// low[row of the tile] on the way in, and leave their minima and maxima (low_out,
// big_out, the tile's first row).  COUNT: returns the largest finite result + 1
// of this thread's row.
template <bool FULL, bool LATE, bool COUNT>
__device__ __forceinline__ uint32_t entry_tile(const u16 *__restrict__ Np, int64_t ldn, int64_t n, int64_t m0,
                                           int64_t j0, const int32_t *__restrict__ idx, const u16 *__restrict__ Bp,
                                           int64_t kbeg, int64_t nk, u16 *__restrict__ C, int64_t ldc, int vec,
                                           u16 *nt, const uint32_t *low, uint32_t *low_out, uint32_t *big_out,
                                           u16 *low_lds)
{
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    u16x2 acc[ECOLS][ERL / 2];
#pragma unroll
    for (int c = 0; c < ECOLS; c++)
#pragma unroll
        for (int h = 0; h < ERL / 2; h++) acc[c][h] = (u16x2){0xFFFF, 0xFFFF};

    // staging: thread (k = t % 32, row pair p = t / 32) gathers
    // N[m0 + 2 ERP e + 2p + h][L_J[k]], h < 2.  The values stay as loaded
    // until they are stored (the wait for them falls after the slice's
    // compute), and the column index is read one slice ahead.
    const int sk = (int)(threadIdx.x % SBK), sp = (int)(threadIdx.x / SBK);  // sk == lane % 32
    const gu16 *gN = glob(Np);
    const gbytes *gNb = (const gbytes *)(gN + m0 * ldn);  // this tile's rows; offsets < 2^32 (host)
    const uint32_t rowb = (uint32_t)ldn * 2u;             // bytes per row
    const int nloc = (int)(n - m0 < EBM ? n - m0 : EBM);  // rows of the tile below n (>= 1)
    const __attribute__((address_space(1))) int32_t *gi = glob(idx) + kbeg;
    const gu16 *gB = glob(Bp) + kbeg * SBN;
    uint32_t sv[ESV];
    uint4 bn, bcur;  // A[L_J[32 sl + lane % 32]][j0 + 8 w .. + 7]: the next slice's, this one's
    auto row_of = [&](int e) { return (e >> 1) * (2 * ERP) + 2 * sp + (e & 1); };
    auto load = [&](int64_t sl, uint32_t col) {
        bn = gload16(gB + (sl * SBK + sk) * SBN + w * ECOLS);
        if (FULL) {
            const uint32_t o = (uint32_t)(2 * sp) * rowb + col * 2u;
#pragma unroll
            for (int e = 0; e < ESV; e++)
                sv[e] = *(const gu16 *)(gNb + (uint32_t)(o + (uint32_t)((e >> 1) * (2 * ERP) + (e & 1)) * rowb));
        } else {
            // rows past n read the last row (every load unconditional, so
            // none waits for another); store() puts infinity in their place
#pragma unroll
            for (int e = 0; e < ESV; e++) {
                const int r = row_of(e);
                const uint32_t rr = (uint32_t)(r < nloc ? r : nloc - 1);
                sv[e] = *(const gu16 *)(gNb + (uint32_t)(rr * rowb + col * 2u));
            }
        }
    };
    auto store = [&](int buf) {
        u16 *q = nt + buf * E_NT + sk * ELDN + 2 * sp;
#pragma unroll
        for (int e = 0; e < ESV / 2; e++) {
            uint32_t lo = sv[2 * e], hi = sv[2 * e + 1];
            if (!FULL) {
                lo = row_of(2 * e) < nloc ? lo : 0xFFFFu;
                hi = row_of(2 * e + 1) < nloc ? hi : 0xFFFFu;
            }
            if constexpr (LATE) {
                const uint32_t l = *(const uint32_t *)(low_lds + row_of(2 * e));  // of the pair of rows
                lo = lo == 0xFFFFu ? lo : lo - (l & 0xFFFFu);
                hi = hi == 0xFFFFu ? hi : hi - (l >> 16);
            }
            *(uint32_t *)(q + 2 * ERP * e) = lo | (hi << 16);
        }
    };
    auto upd = [&](int c, const uint4 &v, uint32_t wgt) {
        const u16x2 a = (u16x2){(u16)wgt, (u16)wgt};
        const u16x2 s0 = add_sat(as_u16x2(v.x), a), s1 = add_sat(as_u16x2(v.y), a);
        const u16x2 s2 = add_sat(as_u16x2(v.z), a), s3 = add_sat(as_u16x2(v.w), a);
        acc[c][0] = min2(acc[c][0], s0);
        acc[c][1] = min2(acc[c][1], s1);
        acc[c][2] = min2(acc[c][2], s2);
        acc[c][3] = min2(acc[c][3], s3);
    };
    auto compute = [&](int buf) {
        const u16 *nl = nt + buf * E_NT + lane * ERL;
        // lanes 0-31: column c, lanes 32-63: column c + 1, k = lane % 32
        const int hsh = (lane >> 5) * 16;
#pragma unroll
        for (int c = 0; c < ECOLS; c += 2) {
            const uint32_t bv = (comp(bcur, c / 2) >> hsh) & 0xFFFFu;
            const uint64_t mask = __ballot(bv != 0xFFFFu);
            uint32_t lo = (uint32_t)mask, hi = (uint32_t)(mask >> 32);
            if (__builtin_popcount(lo) > kEntryDense || __builtin_popcount(hi) > kEntryDense) {
                const uint32_t any = lo | hi;  // rows where neither column has an entry are skipped
#pragma unroll
                for (int k = 0; k < SBK; k++) {
                    if (!((any >> k) & 1u)) continue;
                    const uint32_t wl = (uint32_t)__builtin_amdgcn_readlane((int)bv, k);
                    const uint32_t wh = (uint32_t)__builtin_amdgcn_readlane((int)bv, k + 32);
                    const uint4 v = *(const uint4 *)(nl + k * ELDN);
                    upd(c, v, wl);
                    upd(c + 1, v, wh);
                }
                continue;
            }
            while (lo | hi) {
                // an exhausted mask reads row 31 and adds infinity (no branch;
                // the test is on the scanned bit, so it stays scalar)
                const int kl = __builtin_ctz(lo | 0x80000000u), kh = __builtin_ctz(hi | 0x80000000u);
                const uint32_t rl = (uint32_t)__builtin_amdgcn_readlane((int)bv, kl);
                const uint32_t rh = (uint32_t)__builtin_amdgcn_readlane((int)bv, kh + 32);
                const uint32_t wl = (lo >> kl) & 1u ? rl : 0xFFFFu, wh = (hi >> kh) & 1u ? rh : 0xFFFFu;
                lo &= ~(1u << kl);
                hi &= ~(1u << kh);
                const uint4 vl = *(const uint4 *)(nl + kl * ELDN);
                const uint4 vh = *(const uint4 *)(nl + kh * ELDN);
                upd(c, vl, wl);
                upd(c + 1, vh, wh);
            }
        }
    };
    if constexpr (LATE) {  // 0xFFFF (no finite value) takes nothing off infinity
        const int r = (int)threadIdx.x;
        low_lds[r] = (u16)(r < nloc ? low[r] : 0u);
        __syncthreads();
    }
    if (nk > 0) {
        uint32_t col = (uint32_t)gi[sk];
        load(0, col);
        col = nk > 1 ? (uint32_t)gi[SBK + sk] : 0u;
        store(0);
        bcur = bn;
        __syncthreads();
        for (int64_t sl = 0; sl < nk; sl++) {
            const int buf = (int)(sl & 1);
            if (sl + 1 < nk) {
                load(sl + 1, col);
                col = sl + 2 < nk ? (uint32_t)gi[(sl + 2) * SBK + sk] : 0u;
            }
            compute(buf);
            if (sl + 1 < nk) {
                store(buf ^ 1);
                bcur = bn;
            }
            __syncthreads();
        }
    }
    // epilogue: the tile through LDS as [column][row], then each thread
    // writes one row's 64 columns in 16-byte pieces
    u16 *ct = nt;
#pragma unroll
    for (int c = 0; c < ECOLS; c++)
        *(uint4 *)(ct + (w * ECOLS + c) * ELDN + lane * ERL) =
            make_uint4(as_u32(acc[c][0]), as_u32(acc[c][1]), as_u32(acc[c][2]), as_u32(acc[c][3]));
    __syncthreads();
    const int r = (int)threadIdx.x;
    const int64_t i = m0 + r;
    if (i >= n) return 0;
    gu16 *crow = glob(C) + i * ldc + j0;
    uint32_t least = 0xFFFFu, most = 0;
#pragma unroll
    for (int c8 = 0; c8 < SBN; c8 += 8) {
        uint32_t v[8];
#pragma unroll
        for (int q = 0; q < 8; q++) v[q] = ct[(c8 + q) * ELDN + r];
        if constexpr (LATE || COUNT) {  // columns past n are infinite
#pragma unroll
            for (int q = 0; q < 8; q++) {
                least = min(least, v[q]);
                most = max(most, (v[q] + 1) & 0xFFFFu);
            }
        }
        if (vec && j0 + c8 + 8 <= n) {
            gstore16(crow + c8, make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16),
                                           v[6] | (v[7] << 16)));
        } else {
            for (int q = 0; q < 8; q++)
                if (j0 + c8 + q < n) crow[c8 + q] = (u16)v[q];
        }
    }
    if (LATE && most) {
        atomicMin(&low_out[r], least);
        atomicMax(&big_out[r], most - 1);
    }
    return most;
}

__global__ __launch_bounds__(ENT) __attribute__((amdgpu_waves_per_eu(4))) void sp_entry_kernel(
    const u16 *__restrict__ Np, int64_t ldn, int64_t n, const int64_t *__restrict__ off,
    const int32_t *__restrict__ order, const int32_t *__restrict__ idx, const u16 *__restrict__ Bp,
    u16 *__restrict__ C, int64_t ldc, int tiles_m, int nblk, int64_t cap, int vec)
{
    __shared__ __attribute__((aligned(16))) u16 nt[2 * E_NT];
    const int t = (int)blockIdx.x;
    if (t >= tiles_m * nblk) return;
    // Column blocks costliest first, all row tiles of one column block
    // consecutively (one strip of rows at a time, blocks costliest first
    // within it, measured slower: the last strip's costly blocks start late).
    const int tm = t % tiles_m, J = order[t / tiles_m];
    const int64_t m0 = (int64_t)tm * EBM, j0 = (int64_t)J * SBN;
    // A plan that did not fit its workspace (sp_fill_kernel reported it and
    // wrote nothing) leaves the tile infinite, as the tile form does.
    const int64_t kbeg = off[J];
    const int64_t nk = off[nblk] > cap ? 0 : (off[J + 1] - kbeg) / SBK;
    if (m0 + EBM <= n)
        entry_tile<true, false, false>(Np, ldn, n, m0, j0, idx, Bp, kbeg, nk, C, ldc, vec, nt, nullptr, nullptr, nullptr, nullptr);
    else
        entry_tile<false, false, false>(Np, ldn, n, m0, j0, idx, Bp, kbeg, nk, C, ldc, vec, nt, nullptr, nullptr, nullptr, nullptr);
}

// ------------------------------------------- level form of the step
// The tile product on the matrix cores (level.h).  The lists L_J hold whole
// aligned groups of 8 rows, so 8 consecutive k are 8 consecutive columns of
// N: one 16-byte load, as in a plain product.  Each XCD takes a contiguous
// run of the tiles, two row panels at a time, both panels of a column block in
// turn: neighbouring column blocks read overlapping columns of the panels
// from that XCD's L2 and each block's entries serve both (us a step with 1 /
// 2 / 4 / 8 panels together, normalisation included: m = 8 295 / 265 / 267 /
// 278, m = 9 3594 / 3532 / 3857 / 4323).  At m = 9 the panels (5.6 MB each) do
// not fit: 20 GB a step miss L2, 5.7 TB/s, which is the bound there.
using PCfg = LevelCfg<4, 2, 2, 2>;  // 256 threads, 128 x 64
using PBack = TileCfg<128, 64, 32, 4, 8>;
static_assert(PCfg::BM == PBack::BM && PCfg::BN == SBN && PBack::BN == SBN && PCfg::NT == PBack::NT, "stand-in tile");

// Staging of N[m0 .., L_J]: LevelA with the k groups of the list (SUB as there).
template <class C, bool SUB = false>
struct LevelGather {
    gbytes *base;
    const __attribute__((address_space(1))) int32_t *idx, *at;
    int64_t n, K;
    uint32_t off[C::A_CPT];
    int col;   // first column of the thread's k group in the slice that load() takes
    int back;  // columns to step back from there to stay in the row (slice 0 only)
    uint32_t low2[SUB ? C::A_CPT : 1];
    uint4 r[C::A_CPT];
    __device__ __forceinline__ LevelGather(const gu16 *p, int64_t ld, int rows, int64_t n_, const int32_t *list,
                                           int64_t K_, const uint32_t *low = nullptr)
        : base((gbytes *)p), idx(glob(list) + C::tid() % C::KC * 8), n(n_), K(K_)
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) {
            const int row = min(C::tid() / C::KC + q * (C::GT / C::KC), rows - 1);
            off[q] = (uint32_t)row * (uint32_t)ld * 2u;
            if constexpr (SUB) {
                const uint32_t v = low[row] & 0x7FFFu;  // 0xFFFF (no finite value): any offset will do
                low2[q] = v | (v << 16);
            }
        }
    }
    __device__ __forceinline__ uint32_t value2(uint32_t x, int q) const
    {
        if constexpr (SUB) return as_u32((u16x2)(as_u16x2(x) - as_u16x2(low2[q])));
        return x;
    }
    __device__ __forceinline__ void seek(int64_t k0) { point(k0, k0 >= 0); }
    // to the slice at k0; a thread with no group there reads column 0
    __device__ __forceinline__ void point(int64_t k0, bool in)
    {
        at = idx + k0;
        col = in ? *at : 0;
        back = max(0, (int)(col + 8 - n));
    }
    __device__ __forceinline__ void load_chunk(int q) { r[q] = uload16(base, off[q] + (uint32_t)(col - back) * 2u); }
    __device__ __forceinline__ void advance()
    {
        at -= C::BK * C::KS;
        col = at >= idx ? *at : 0;
        back = 0;  // lists ascend and slices descend: only slice 0 has the matrix's last group
    }
    // The last group of the matrix may end before its 8th column: it was read
    // from the end of the row back (its rows of A past the end are infinite,
    // so any value will do there).
    __device__ __forceinline__ void settle()
    {
        if (back) {
#pragma unroll
            for (int q = 0; q < C::A_CPT; q++) r[q] = shift_in_inf(r[q], back);
        }
    }
    __device__ __forceinline__ void load()
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) load_chunk(q);
        settle();
        advance();
    }
    __device__ __forceinline__ void load_tail(int64_t k0)  // K is a multiple of SBK = 32
    {
        // the list ends at K: past it is another block's list or no list
        const bool in = k0 + C::tid() % C::KC * 8 < K;
        point(k0, in);
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) load_chunk(q);
        settle();
        if (!in) {
#pragma unroll
            for (int q = 0; q < C::A_CPT; q++)
                r[q] = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
        }
    }
    __device__ __forceinline__ void store_chunk(uint4 *as, int q) const
    {
        as[(C::tid() % C::KC) * C::PA + (C::tid() / C::KC ^ C::tid() % C::KC) + q * (C::GT / C::KC)] =
            make_uint4(level_image(value2(r[q].x, q)), level_image(value2(r[q].y, q)),
                       level_image(value2(r[q].z, q)), level_image(value2(r[q].w, q)));
    }
    __device__ __forceinline__ uint32_t first() const  // as LevelA's
    {
        const int row = C::tid() / C::KC;
        const uint64_t lo = (uint64_t)r[0].y << 32 | r[0].x, hi = (uint64_t)r[0].w << 32 | r[0].z;
        const uint32_t v = value2((uint32_t)(((row & 2) ? hi : lo) >> (row & 1) * 32), 0);
        return v >> (row & 4) * 4 & 0xFFFFu;
    }
    __device__ __forceinline__ i16x2 largest(i16x2 m) const
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                m = __builtin_elementwise_max(m, __builtin_bit_cast(i16x2, value2(comp(r[q], e), q)));
        return m;
    }
};

// One 128 x 64 tile of a step.  LATE: the rows of p.L are normalised on the
// way in and their minima left behind (LevelStep); otherwise p.L is canonical
// and only L, O, their strides, n and the past words of p are used.  FIRST: the first
// step of a chain, which looks at its values; the others go by the step before
// (LevelStep).  ELSEWHERE: a tile past the levels is marked by its first value and
// left to sp_entry_past_kernel.
template <bool LATE, bool FIRST, bool ELSEWHERE>
__global__ __launch_bounds__(PCfg::NT) __attribute__((amdgpu_waves_per_eu(3))) void sp_level_kernel(
    LevelStep p, const int64_t *__restrict__ off, const int32_t *__restrict__ idx, const u16 *__restrict__ Bp,
    int tiles_m, int nblk, int64_t cap, int vec, int32_t *st)
{
    using C = PCfg;
    constexpr int BACK = (PBack::LDS_ELEMS + 7) / 8;
    __shared__ uint4 lds[C::LDS_CHUNKS > BACK ? C::LDS_CHUNKS : BACK];
    const int nb = (int)gridDim.x;  // a multiple of 8
    const int t = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    if (t >= tiles_m * nblk) return;
    const int first = t / (2 * nblk) * 2, gs = min(tiles_m - first, 2), w = t - first * nblk, J = w / gs;
    const int64_t n = p.n, m0 = (int64_t)(first + w % gs) * C::BM, j0 = (int64_t)J * SBN;
    const int rows = (int)min<int64_t>(C::BM, n - m0), cols = (int)min<int64_t>(SBN, n - j0);
    const int64_t kbeg = off[J], K = off[nblk] > cap ? 0 : off[J + 1] - kbeg;
    gu16 *out = glob(p.O) + m0 * p.ldo + j0;
    __shared__ int cnt[LEVEL_COUNTS];
    const uint32_t past = p.past_in[0], deep = p.past_in[1];
    if (t == 0 && threadIdx.x < LEVEL_PASTS) p.past_next[threadIdx.x] = 0;
    bool far = false;
    if constexpr (LATE) far = level_step_rows<C>(p, m0, rows, J == 0, st);
    if (K == 0) {  // no finite entry in these columns, or a plan that did not fit: infinite
        for (int e = (int)threadIdx.x; e < rows * SBN; e += C::NT)
            if (e % SBN < cols) out[(int64_t)(e / SBN) * p.ldo + e % SBN] = 0xFFFF;
        return;
    }
    LevelView view = 2 * deep > past ? LEVEL_U16 : LEVEL_F16;
    if (!far && (int64_t)past <= (int64_t)tiles_m * nblk) {  // 2 tiles of 64 x 64 each
        LevelGather<C, LATE> aop(glob(p.L) + m0 * p.ldl, p.ldl, rows, n, idx + kbeg, K, LATE ? p.low_in + m0 : nullptr);
        LevelB<C> bop(glob(Bp) + kbeg * SBN, SBN, SBN, K);
        LevelAcc<C> acc;
        view = level_kloop<C, FIRST>(K, aop, bop, lds, acc, cnt);
        if (view <= LEVEL_PAST &&
            (level_sure<C>(acc, rows, cols) || (view == LEVEL_IN && level_clean<C>(K, aop, bop, lds)))) {
            if constexpr (LATE) level_row_low<C>(acc, rows, cols, p.low_out + m0);
            level_store<C>(out, p.ldo, rows, cols, acc);
            return;
        }
    }
    if constexpr (ELSEWHERE) {
        if (threadIdx.x == 0) out[0] = MARK_F16;
        return;
    }
    const gu16 *gB = glob(Bp) + kbeg * SBN;
    TileAcc<PBack> acc;
    GatherA<PBack> aop{glob(p.L), p.ldl, n, m0, glob(idx) + kbeg, rows == C::BM, LATE ? p.low_in + m0 : nullptr, {}};
    auto bop = chunk_b<PBack>([&](int64_t k0, int kr, int jc) { return gload16(gB + (k0 + kr) * SBN + jc); });
    tile_product<PBack, true>(K / PBack::BK, aop, bop, (u16 *)lds, acc, view == LEVEL_U16);
    level_step_back<PBack, LATE>(p, m0, j0, rows, vec != 0, acc);
}

// The marked tiles of a step (sp_level_kernel) in the entry-list form, which
// takes a fraction of the tile form's pairs.  Where none is marked, as in the
// steps of a transfer matrix, a block ends after 4 reads (m = 8: 5 us of a step of 285).
constexpr int EPARTS = EBM / PCfg::BM;
template <bool LATE>
__global__ __launch_bounds__(ENT) __attribute__((amdgpu_waves_per_eu(4))) void sp_entry_past_kernel(
    LevelStep p, const int64_t *__restrict__ off, const int32_t *__restrict__ order, const int32_t *__restrict__ idx,
    const u16 *__restrict__ Bp, int tiles_m, int nblk, int vec)
{
    __shared__ __attribute__((aligned(16))) u16 nt[2 * E_NT];
    __shared__ __attribute__((aligned(4))) u16 low[LATE ? EBM : 2];
    const int t = (int)blockIdx.x, J = order[t / tiles_m];
    const int64_t n = p.n, m0 = (int64_t)(t % tiles_m) * EBM, j0 = (int64_t)J * SBN;
    const int64_t row = m0 + (int64_t)(threadIdx.x % EPARTS) * PCfg::BM;
    if (!__syncthreads_or(threadIdx.x < EPARTS && row < n && glob(p.O)[row * p.ldo + j0] == MARK_F16)) return;
    const int64_t kbeg = off[J], nk = (off[J + 1] - kbeg) / SBK;
    const uint32_t *li = LATE ? p.low_in + m0 : nullptr;
    uint32_t *lo = LATE ? p.low_out + m0 : nullptr, *bo = LATE ? p.big_out + m0 : nullptr;
    uint32_t most;
    if (m0 + EBM <= n)
        most = entry_tile<true, LATE, true>(p.L, p.ldl, n, m0, j0, idx, Bp, kbeg, nk, p.O, p.ldo, vec, nt, li, lo, bo, low);
    else
        most = entry_tile<false, LATE, true>(p.L, p.ldl, n, m0, j0, idx, Bp, kbeg, nk, p.O, p.ldo, vec, nt, li, lo, bo, low);
    if (__syncthreads_or(most > LV_MAX + 1) && threadIdx.x == 0)  // (the form has no use for the other word)
        atomicAdd(&p.past_out[0], 2u * (uint32_t)min<int64_t>(EPARTS, (n - m0 + PCfg::BM - 1) / PCfg::BM));
}

// ------------------------------------------- the step in bytes
// For the period search, which owns its powers: a canonical value v <= 30 is
// kept as the byte 93 - 3 v (0 for infinity), half the exponent field of its
// image and so the image's upper byte (the lower is 0), and a raw result as
// the byte t (255 for infinity).  A step reads and writes half the bytes, and
// the image of two values is one byte permutation.  At m = 9 the 128 rows of N that a panel reads are
// 2.8 MB and fit an XCD's L2.  A result that the levels do not prove raises a
// flag, and the search starts again in u16.
// A power lies in column groups: [column / 8][row][column % 8].  The gathered
// columns are whole groups, so the 64 rows of a wave's load are 512 bytes one
// after the other, and the group is the same for the whole wave.  With rows
// one after the other a load touched up to 64 lines: whole searches of m = 9
// 79.0 ms, now 73.1, m = 8 6.63 and 6.55, m = 6 0.68 and 0.71.
template <class C>
struct LevelGather8 {
    gbytes *base;
    const int32_t *idx, *at;
    int64_t K, group8;  // bytes of a column group
    uint32_t off;
    int32_t col[C::A_CPT];
    uint2 r[C::A_CPT];
    static_assert(C::GT % C::BM == 0 && C::BM % 64 == 0 && C::KC % C::A_CPT == 0, "a wave's chunk in one group");
    static __device__ __forceinline__ int row() { return C::tid() % C::BM; }
    static __device__ __forceinline__ int first() { return __builtin_amdgcn_readfirstlane(C::tid() / C::BM) * C::A_CPT; }
    __device__ __forceinline__ LevelGather8(const uint8_t *p, int64_t group8_, int rows, const int32_t *list, int64_t K_)
        : base((gbytes *)p), idx(list + first() * 8), K(K_), group8(group8_), off((uint32_t)min(row(), rows - 1) * 8u)
    {
    }
    __device__ __forceinline__ void fetch()
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) col[q] = at >= idx ? at[8 * q] : 0;
    }
    __device__ __forceinline__ void seek(int64_t k0)
    {
        at = idx + k0;
        fetch();
    }
    __device__ __forceinline__ void load_chunk(int q)
    {
        const u32x2 v = *(const __attribute__((address_space(1))) u32x2 *)(base + (col[q] >> 3) * group8 + off);
        r[q] = make_uint2(v.x, v.y);
    }
    __device__ __forceinline__ void advance()
    {
        at -= C::BK * C::KS;
        fetch();
    }
    __device__ __forceinline__ void load()
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) load_chunk(q);
        advance();
    }
    __device__ __forceinline__ void load_tail(int64_t k0)  // the list ends at K, a multiple of SBK = 32
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) {
            const bool in = k0 + (first() + q) * 8 < K;
            col[q] = in ? idx[k0 + 8 * q] : 0;
            load_chunk(q);
            if (!in) r[q] = make_uint2(0, 0);
        }
    }
    __device__ __forceinline__ void store_chunk(uint4 *as, int q) const
    {
        auto image = [](uint32_t w, uint32_t sel) { return __builtin_amdgcn_perm(w, w, sel); };
        as[(first() + q) * C::PA + row()] =
            make_uint4(image(r[q].x, 0x010C000Cu), image(r[q].x, 0x030C020Cu), image(r[q].y, 0x010C000Cu),
                       image(r[q].y, 0x030C020Cu));
    }
};

// Staging of the right operand from its images: two 16-byte loads a thread and
// slice and no conversion, where values took eight loads of 4 bytes and 24
// instructions of the 113 (whole searches of m = 8 6.55 ms, now 5.98; m = 9
// 72.2, now 65.3).
template <class C>
struct LevelImages {
    gbytes *base, *at;
    int64_t K;
    uint4 r[C::B_COLS];
    static __device__ __forceinline__ int chunk(int j) { return C::tid() + j * C::GT; }  // (k / 8) * BN + column
    __device__ __forceinline__ LevelImages(const u16 *p, int64_t K_) : base((gbytes *)glob(p)), K(K_) {}
    __device__ __forceinline__ void seek(int64_t k0) { at = base + k0 * (C::BN * 2); }
    __device__ __forceinline__ void load()
    {
#pragma unroll
        for (int j = 0; j < C::B_COLS; j++) r[j] = gload16((const gu16 *)(at + chunk(j) * 16));
        at -= C::BK * C::KS * C::BN * 2;
    }
    __device__ __forceinline__ void load_tail(int64_t k0)
    {
#pragma unroll
        for (int j = 0; j < C::B_COLS; j++) {
            const bool in = k0 + chunk(j) / C::BN * 8 < K;
            r[j] = in ? gload16((const gu16 *)(base + k0 * (C::BN * 2) + chunk(j) * 16)) : make_uint4(0, 0, 0, 0);
        }
    }
    __device__ __forceinline__ void settle() {}
    __device__ __forceinline__ void store_chunk(uint4 *bs, int j) const
    {
        const int n = chunk(j) % C::BN;
        bs[chunk(j) / C::BN * C::PB + (n ^ ((n >> 3) & 3))] = r[j];
    }
};

// Row panels that run side by side over the column blocks (whole searches with
// 1, 2, 3, 4: m = 8 7.45, 6.79, 6.87, 6.62 ms, m = 9 85.4, 79.8, 82.1, 80.3).  A
// block that took 2 neighbouring column blocks, the second's first loads ahead
// of the first's stores, left too few blocks: 8.40 and 91.8 ms.
constexpr int PANELS8 = 2;
struct P8Cfg : PCfg {
    static constexpr bool SWZ = false;  // rows are staged in order
};
__global__ __launch_bounds__(PCfg::NT) __attribute__((amdgpu_waves_per_eu(3))) void sp_level8_kernel(
    const uint8_t *__restrict__ N, int64_t group8, int64_t n, const int64_t *__restrict__ off,
    const int32_t *__restrict__ idx, const u16 *__restrict__ Bp, uint8_t *__restrict__ O, int tiles_m, int nblk,
    int64_t cap, const int32_t *top, int32_t *wide, const int32_t *big)
{
    using C = P8Cfg;
    __shared__ uint4 lds[C::LDS_CHUNKS];
    const int nb = (int)gridDim.x;  // a multiple of 8
    const int t = ((int)blockIdx.x & 7) * (nb >> 3) + ((int)blockIdx.x >> 3);
    if (t >= tiles_m * nblk) return;
    const int first = t / (PANELS8 * nblk) * PANELS8, gs = min(tiles_m - first, PANELS8), w = t - first * nblk, J = w / gs;
    const int64_t m0 = (int64_t)(first + w % gs) * C::BM, j0 = (int64_t)J * SBN;
    const int rows = (int)min<int64_t>(C::BM, n - m0), cols = (int)min<int64_t>(SBN, n - j0);
    const int64_t kbeg = off[J], K = off[nblk] > cap ? 0 : off[J + 1] - kbeg;
    LevelAcc<C> acc;
    if (K > 0) {
        LevelGather8<C> aop(N + m0 * 8, group8, rows, idx + kbeg, K);
        LevelImages<C> bop(Bp + kbeg * SBN, K);
        level_kloop<C>(K, aop, bop, lds, acc);
        if (!level_sure<C>(acc, rows, cols)) {
            // exact when the largest values of N and of these columns sum to
            // what the float range holds
            const int b = top[J];
            if (threadIdx.x == 0 && (b > (int)LV_MAX || *big + b > (int)LV_SUM)) set_status(wide, 1);
        }
    } else {  // no finite entry in these columns, or a plan that did not fit
#pragma unroll
        for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
            for (int ni = 0; ni < C::NI; ni++)
#pragma unroll
                for (int r = 0; r < 4; r++) acc.v[mi][ni][r] = 0;
    }
    __attribute__((address_space(1))) uint8_t *out = glob(O) + (j0 >> 3) * group8 + m0 * 8;
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++) {
        const int row = level_row<C>(mi);
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++) {
            const int col = level_col<C>(ni);
            uint32_t x = 0;
#pragma unroll
            for (int r = 0; r < 4; r++) x |= (level_value(acc.v[mi][ni][r]) & 0xFFu) << (8 * r);
            if (row < rows && j0 + col < (n + 7 & ~(int64_t)7))  // columns past n, up to the group's end, are infinite
                *(__attribute__((address_space(1))) uint32_t *)(out + (col >> 3) * group8 + row * 8 + (col & 7)) = x;
        }
    }
}

// ------------------------------------------------------------ host side
// Plan layout: counts[nblk + 1] | off[nblk + 1] | order[nblk] | idx[cap] |
// Bp[cap * SBN], every piece 256-byte aligned; cap (rows) follows from the
// bytes the caller gives the plan.  Its rows are sum_J |L_J| rounded up to
// SBK per block, at most nblk * round_up(n, SBK) (the worst case, a dense
// A); a transfer matrix needs a few per cent of that.
static int64_t plan_fixed_bytes(int64_t nblk)
{
    return round_up((nblk + 1) * 8, 256) * 2 + round_up(nblk * 4, 256);
}

size_t sparse_plan_bytes_rows(int64_t n, int64_t rows)
{
    const int64_t nblk = (n + SBN - 1) / SBN;
    return (size_t)(plan_fixed_bytes(nblk) + round_up(rows * 4, 256) + round_up(rows * SBN * 2, 256) + 256);
}

size_t sparse_plan_bytes(int64_t n)
{
    const int64_t nblk = (n + SBN - 1) / SBN;
    return sparse_plan_bytes_rows(n, nblk * round_up(n, SBK));
}

// Rows a plan workspace of `bytes` holds: the largest cap with
// sparse_plan_bytes_rows(n, cap) <= bytes (so a workspace sized for `rows`
// rows holds at least `rows`).  The first guess is at least that cap and
// the roundings to 256 bytes take it at most a few rows past it.
static int64_t plan_capacity(int64_t n, size_t bytes)
{
    const int64_t nblk = (n + SBN - 1) / SBN;
    const int64_t avail = (int64_t)bytes - plan_fixed_bytes(nblk) - 256;
    if (avail <= 0) return 0;
    int64_t cap = avail / (4 + SBN * 2);
    while (cap > 0 && sparse_plan_bytes_rows(n, cap) > bytes) cap--;
    return cap;
}

struct SparsePlan {
    int64_t nblk, cap;
    int64_t *counts;  // of rows; of a finished plan, the 3 x LEVEL_PASTS words of its steps (level_step)
    int64_t *off;
    int32_t *order, *idx;
    u16 *Bp;
};

static SparsePlan carve_plan(void *ws, int64_t n, size_t bytes)
{
    SparsePlan p;
    p.nblk = (n + SBN - 1) / SBN;
    p.cap = plan_capacity(n, bytes);
    char *c = (char *)ws;
    p.counts = (int64_t *)c;
    c += round_up((p.nblk + 1) * 8, 256);
    p.off = (int64_t *)c;
    c += round_up((p.nblk + 1) * 8, 256);
    p.order = (int32_t *)c;
    c += round_up(p.nblk * 4, 256);
    p.idx = (int32_t *)c;
    c += round_up(p.cap * 4, 256);
    p.Bp = (u16 *)c;
    return p;
}

// The counts, their prefix sums (off[nblk] = the plan's rows) and the order
// of the blocks: the part of a plan that needs no room for rows.
static void plan_count(const u16 *A, int64_t n, int64_t lda, const SparsePlan &p, int64_t *rec, int64_t seq,
                       hipStream_t s)
{
    const int vec = aligned16(A) && lda % 8 == 0;
    hipLaunchKernelGGL(sp_count_kernel, dim3((unsigned)p.nblk), dim3(PT), 0, s, A, lda, n, p.counts, vec);
    hipLaunchKernelGGL(sp_scan_kernel, dim3(1), dim3(PT), 0, s, (const int64_t *)p.counts, p.nblk, p.off,
                       p.order, rec, seq);
}

mpr_status sparse_plan_rows(const u16 *A, int64_t n, int64_t lda, void *ws, hipStream_t s, int64_t *rows)
{
    SparsePlan p = carve_plan(ws, n, 0);
    HostRecord rec(s);
    if (!rec.p) return MPR_ENOMEM;
    const int64_t seq = rec.ticket();
    plan_count(A, n, lda, p, rec.p, seq, s);
    const mpr_status e = check_launch();
    if (e != MPR_OK) return e;
    const mpr_status w = rec.wait(rec.p, seq);
    if (w == MPR_OK) *rows = rec.p[0];
    return w;
}

mpr_status sparse_plan_fill(const u16 *A, int64_t n, int64_t lda, void *ws, size_t bytes, bool images, int32_t *st,
                            hipStream_t s)
{
    SparsePlan p = carve_plan(ws, n, bytes);
    const int vec = aligned16(A) && lda % 8 == 0;
    // with images, the blocks' largest values take the place of their order,
    // which only the VALU forms read
    hipLaunchKernelGGL(images ? sp_fill_kernel<true> : sp_fill_kernel<false>, dim3((unsigned)p.nblk), dim3(PT), 0, s, A,
                       lda, n, (const int64_t *)p.off, p.nblk, p.cap, p.idx, p.Bp, vec, p.order, (uint32_t *)p.counts, st);
    return check_launch();
}

mpr_status sparse_plan_launch(const u16 *A, int64_t n, int64_t lda, void *ws, size_t bytes, int32_t *st,
                              hipStream_t s)
{
    const SparsePlan p = carve_plan(ws, n, bytes);
    plan_count(A, n, lda, p, nullptr, 0, s);
    return sparse_plan_fill(A, n, lda, ws, bytes, false, st, s);
}

static std::atomic<int> g_sparse_arith{MPR_ARITH_U16};  // process-wide, set from any thread
static std::atomic<int> g_sparse_form{MPR_SPARSE_AUTO};

bool sparse_step_late(int64_t n, int64_t ldl, int64_t ldo)
{
    return g_sparse_form == MPR_SPARSE_AUTO && n >= 8 && level_strides(ldl, ldo);
}

// From so many states on, tiles past the levels are left to the entry-list form
// (a launch more a step): below, the tile form is as fast or faster on them.
constexpr int64_t ENTRY_MIN_N = 7000;

// Step `step` (from 0) over a plan's lists; the past words lie where the plan's
// counts were, which its other parts replace.
template <bool LATE>
static mpr_status level_step(LevelStep q, const SparsePlan &p, int64_t step, int vec, int32_t *st, hipStream_t s)
{
    uint32_t *past = (uint32_t *)p.counts;
    q.past_in = past + step % 3 * LEVEL_PASTS;
    q.past_out = past + (step + 1) % 3 * LEVEL_PASTS;
    q.past_next = past + (step + 2) % 3 * LEVEL_PASTS;
    const bool elsewhere = q.n >= ENTRY_MIN_N && g_sparse_arith == MPR_ARITH_U16 && (int64_t)EBM * q.ldl * 2 < ((int64_t)1 << 32);
    const int64_t tiles_m = (q.n + PCfg::BM - 1) / PCfg::BM, tiles = tiles_m * p.nblk;
    if (tiles > (int64_t)INT32_MAX - 8) return MPR_EUNSUPPORTED;
    auto kernel = elsewhere ? (step == 0 ? sp_level_kernel<LATE, true, true> : sp_level_kernel<LATE, false, true>)
                            : (step == 0 ? sp_level_kernel<LATE, true, false> : sp_level_kernel<LATE, false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)round_up(tiles, 8)), dim3(PCfg::NT), 0, s, q, (const int64_t *)p.off,
                       (const int32_t *)p.idx, (const u16 *)p.Bp, (int)tiles_m, (int)p.nblk, p.cap, vec, st);
    if (elsewhere) {
        const int64_t rows = (q.n + EBM - 1) / EBM;  // fewer tiles than above
        hipLaunchKernelGGL(sp_entry_past_kernel<LATE>, dim3((unsigned)(rows * p.nblk)), dim3(ENT), 0, s, q,
                           (const int64_t *)p.off, (const int32_t *)p.order, (const int32_t *)p.idx, (const u16 *)p.Bp, (int)rows, (int)p.nblk, vec);
    }
    return check_launch();
}

mpr_status sparse_step8_launch(const uint8_t *N, int64_t n, void *ws, size_t bytes, uint8_t *O,
                               int32_t *wide, const int32_t *big, hipStream_t s)
{
    const SparsePlan p = carve_plan(ws, n, bytes);
    const int64_t tiles_m = (n + PCfg::BM - 1) / PCfg::BM, tiles = tiles_m * p.nblk;
    if (tiles > (int64_t)INT32_MAX - 8) return MPR_EUNSUPPORTED;
    hipLaunchKernelGGL(sp_level8_kernel, dim3((unsigned)round_up(tiles, 8)), dim3(PCfg::NT), 0, s, N, level_group8(n), n,
                       (const int64_t *)p.off, (const int32_t *)p.idx, (const u16 *)p.Bp, O, (int)tiles_m, (int)p.nblk,
                       p.cap, (const int32_t *)p.order, wide, big);
    return check_launch();
}

mpr_status sparse_step_late_launch(const LevelStep &q, void *ws, size_t bytes, int64_t step, int32_t *st, hipStream_t s)
{
    return level_step<true>(q, carve_plan(ws, q.n, bytes), step, aligned16(q.O) && q.ldo % 8 == 0, st, s);
}

mpr_status sparse_step_launch(const u16 *Np, int64_t ldn, int64_t n, void *ws, size_t bytes, u16 *C, int64_t ldc,
                              int64_t step, hipStream_t s)
{
    SparsePlan p = carve_plan(ws, n, bytes);
    const int vec = aligned16(C) && ldc % 8 == 0;
    const int form = g_sparse_form;
    if (sparse_step_late(n, ldn, ldc)) {
        LevelStep q{};
        q.L = Np;
        q.O = C;
        q.ldl = ldn;
        q.ldo = ldc;
        q.n = n;
        return level_step<false>(q, p, step, vec, nullptr, s);
    }
    if (form == MPR_SPARSE_ENTRIES && g_sparse_arith == MPR_ARITH_U16 && (int64_t)EBM * ldn * 2 < ((int64_t)1 << 32)) {
        const int64_t tiles_m = (n + EBM - 1) / EBM;
        const int64_t tiles = tiles_m * p.nblk;
        if (tiles > (int64_t)INT32_MAX - 8) return MPR_EUNSUPPORTED;
        hipLaunchKernelGGL(sp_entry_kernel, dim3((unsigned)tiles), dim3(ENT), 0, s, Np, ldn, n,
                           (const int64_t *)p.off, (const int32_t *)p.order, (const int32_t *)p.idx,
                           (const u16 *)p.Bp, C, ldc, (int)tiles_m, (int)p.nblk, p.cap, vec);
        return check_launch();
    }
    const int64_t tiles_m = (n + SCfg::BM - 1) / SCfg::BM;
    const int64_t tiles = tiles_m * p.nblk;
    if (tiles > (int64_t)INT32_MAX - 8) return MPR_EUNSUPPORTED;
    auto kernel = g_sparse_arith == MPR_ARITH_F16 ? sp_step_kernel<true> : sp_step_kernel<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(SCfg::NT), 0, s, Np, ldn, n, (const int64_t *)p.off,
                       (const int32_t *)p.order, (const int32_t *)p.idx, (const u16 *)p.Bp, C, ldc, (int)tiles_m,
                       (int)p.nblk, p.cap, vec);
    return check_launch();
}

}  // namespace mpr

extern "C" mpr_status mpr_set_sparse_form(int form)
{
    if (form != MPR_SPARSE_AUTO && form != MPR_SPARSE_TILES && form != MPR_SPARSE_ENTRIES) return MPR_EINVAL;
    mpr::g_sparse_form = form;
    return MPR_OK;
}

extern "C" mpr_status mpr_set_sparse_arith(int arith)
{
    if (arith != MPR_ARITH_U16 && arith != MPR_ARITH_F16) return MPR_EINVAL;
    mpr::g_sparse_arith = arith;
    return MPR_OK;
}
