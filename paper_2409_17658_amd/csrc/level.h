// level.h -- the (min,+) block product on the matrix cores ("level form").
//
// A value v <= 30 is written as the power of two 2^(59 - 6 v) in bf16,
// infinity (and every larger value) as 0.  The product of two such numbers
// is 2^(118 - 6 (a + b)), and a sum of 32 of them lies in
// [2^(118 - 6 t), 2^(118 - 6 t + 5)] with t the least a + b among them: the
// exponent of the sum names t, because 32 equal terms raise it by 5 and one
// level is worth 6.  So one f32 accumulator over 32 values of k (one
// v_mfma_f32_16x16x32_bf16) holds the minimum of 32 pairs exactly, and the
// minimum over all k is the maximum of those positive floats (an unsigned
// integer maximum of their bits, two accumulators per v_max3_u32).  Every
// term is a power of two and no sum loses its largest term, so rounding
// inside the matrix core can not change the exponent's level.
//
// Exactness.  A result t <= 30 is exact: every pair that sums to 30 or less
// has both values <= 30.  Any other result (t > 30, or no term at all) is
// exact only when no finite operand of the block exceeds 30 and their
// largest sum stays within the f32 range (LV_SUM, the smallest subnormals);
// a block with such a result looks at its operands' largest finite values
// once (level_clean) and, when they do not allow the conclusion, is computed
// by the VALU forms of tile.h instead.  The product is the same bit for bit
// on every input.
//
// Conversion: min(v, 31) and one multiply-add give the bf16 bit pattern
// (the exponent field is linear in v and is 0 at v = 31), two packed
// instructions per two values, done once per block while a slice is staged
// into LDS.  LDS holds 16-byte chunks of 8 consecutive k: [k / 8][row] for
// A, [k / 8][column] for B (transposed on the way by v_perm_b32), the order
// the matrix instruction reads its operands in.
//
// What bounds it: the issue slots of the VALU (level_slice) and the power of
// the chip.  N = 16384, entries 0..15: 117.0 ms (37.6 T pairs/s) in the uint16
// form, 9.75 ms (451 T pairs/s) in this one; a bf16 library product of 8192 x 8192 x 8192
// reaches 604 T multiply-adds/s on the same card.
#pragma once

#include "tile.h"

namespace mpr {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int LV_STEP = 6;                       // exponent bits per level
constexpr uint32_t LV_MAX = 30;                  // largest value with a nonzero image
constexpr int LV_BIAS = LV_STEP * (LV_MAX + 1);  // exponent field of level 0: 186 = 127 + 59
constexpr int LV_TOP = 2 * (LV_BIAS - 127);      // exponent of a product of two level-0 images
constexpr uint32_t LV_SUM = 44;                  // 2^(118 - 6 * 44) = 2^-146, a subnormal f32
// Bits of the least sum that proves a result <= LV_MAX: 2^(118 - 180).
constexpr uint32_t LV_SURE = (uint32_t)(127 + LV_TOP - LV_STEP * (int)LV_MAX) << 23;

// MI x NI tiles of 16 x 16 outputs per wave, WM x WN waves per block, KS such
// groups of waves that share the block's slices of K between them (for
// products of few tiles, which are a chain of memory round trips: KS times
// the loads in flight, a KS-th of the trips).
template <int MI_, int NI_, int WM_, int WN_, int KS_ = 1>
struct LevelCfg {
    static constexpr int MI = MI_, NI = NI_, WM = WM_, WN = WN_, KS = KS_;
    static constexpr int BM = 16 * MI * WM, BN = 16 * NI * WN;
    static constexpr int GT = 64 * WM * WN, NT = GT * KS;  // threads of a group, of the block
    // Thread in its group, wave in its group, group.
    static __device__ __forceinline__ int tid() { return (int)threadIdx.x % GT; }
    static __device__ __forceinline__ int wave() { return (int)(threadIdx.x >> 6) % (WM * WN); }
    static __device__ __forceinline__ int group()
    {
        return KS == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / GT);
    }
    static constexpr int BK = 64, KC = BK / 8;
    // Chunks per k group.  Row r of A lies at r ^ (k group) when SWZ, so the 8
    // lanes that stage the 8 k groups of one row write to 8 different 16-byte
    // bank groups, and the rows of a read stay in whole groups of 4 (an odd
    // pitch instead left reads of two k groups in conflict: 12 chains 33.8 ms,
    // now 33.4; N = 16384 10.3 and 10.2).
    static constexpr int PA = BM, PB = BN;
    static constexpr bool SWZ = true;
    static constexpr int STAGE = KC * (PA + PB);
    static constexpr int LDS_CHUNKS = 2 * STAGE * KS;
    static constexpr int A_CPT = BM * KC / GT;   // A chunks a thread stages
    static constexpr int B_COLS = BN * KC / GT;  // columns of 8 k a thread stages
    static_assert(NI % 2 == 0, "level_store pairs neighbouring tiles");
    static_assert(GT / KC % 8 == 0, "a thread's rows differ above the swizzle");
    static_assert(BM * KC % GT == 0 && (B_COLS == 2 || B_COLS == 4), "staging split");
};

// 2^(59 - 6 v) in bf16 for both halves; 0 for v > 30.
__device__ __forceinline__ uint32_t level_image(uint32_t x)
{
    const u16x2 y = min2(as_u16x2(x), (u16x2){LV_MAX + 1, LV_MAX + 1});
    constexpr u16 mul = (u16)(0u - (LV_STEP << 7)), add = (u16)(LV_BIAS << 7);
    return as_u32((u16x2)(y * (u16x2){mul, mul} + (u16x2){add, add}));
}

// 16 / 8 / 4 bytes of a row that need not be aligned (global loads take any
// 2-byte aligned address).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
typedef u32x2 __attribute__((aligned(2))) u32x2_any;
typedef uint32_t __attribute__((aligned(2))) u32_any;
typedef const __attribute__((address_space(1))) unsigned char gbytes;
__device__ __forceinline__ uint4 uload16(gbytes *base, uint32_t off)
{
    const u32x4 r = *(const __attribute__((address_space(1))) u32x4_any *)(base + off);
    return make_uint4(r.x, r.y, r.z, r.w);
}
__device__ __forceinline__ void ustore16(gu16 *p, const uint4 &v)
{
    const u32x4 r = {v.x, v.y, v.z, v.w};
    *(__attribute__((address_space(1))) u32x4_any *)p = r;
}

// 8 consecutive values shifted down by s >= 0 of them, infinity moving in.
__device__ __forceinline__ uint4 shift_in_inf(const uint4 &v, int s)
{
    uint64_t lo = ~((uint64_t)v.y << 32 | v.x), hi = ~((uint64_t)v.w << 32 | v.z);
    if (s >= 4) {
        lo = hi;
        hi = 0;
        s -= 4;
    }
    if (s >= 4) lo = s = 0;
    if (s > 0) lo = lo >> (16 * s) | hi << (64 - 16 * s);
    hi >>= 16 * s;
    return make_uint4(~(uint32_t)lo, ~(uint32_t)(lo >> 32), ~(uint32_t)hi, ~(uint32_t)(hi >> 32));
}

// Staging of the left operand, `rows` (>= 1) rows of K >= 8 values from
// `base`: chunk q of a thread is row tid / 8 + q NT / 8, k group tid % 8 of
// the slice.  Rows past the end read the last row (their results are not
// used); k past the end reads as infinity.  SUB: the rows still carry the
// offsets low[row] <= 0x7FFF (each row's least value, or no finite value at
// all), taken off while staging; infinity stays above every level.
template <class C, bool SUB = false>
struct LevelA {
    gbytes *base, *at;  // the operand; the slice the next load() takes
    int64_t K;
    uint32_t off[C::A_CPT];  // bytes from a slice's start to each chunk
    uint32_t low2[SUB ? C::A_CPT : 1];
    uint4 r[C::A_CPT];
    __device__ __forceinline__ LevelA(const gu16 *p, int64_t ld, int rows, int64_t K_,
                                      const uint32_t *low = nullptr)
        : base((gbytes *)p), K(K_)
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) {
            const int row = min(C::tid() / C::KC + q * (C::GT / C::KC), rows - 1);
            off[q] = (uint32_t)row * (uint32_t)ld * 2u + (uint32_t)(C::tid() % C::KC) * 16u;
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
    __device__ __forceinline__ void seek(int64_t k0) { at = base + k0 * 2; }
    // a full slice, chunk by chunk; the group's next one is KS slices before it
    __device__ __forceinline__ void load_chunk(int q) { r[q] = uload16(at, off[q]); }
    __device__ __forceinline__ void advance() { at -= C::BK * C::KS * 2; }
    __device__ __forceinline__ void load()
    {
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) load_chunk(q);
        advance();
    }
    // the last K % BK values, in a slice of their own from k0
    __device__ __forceinline__ void load_tail(int64_t k0)
    {
        gbytes *b = base + k0 * 2;
        const int over = (int)(k0 - K) + C::tid() % C::KC * 8 + 8;  // values past the end
        const int back = over > 0 ? over : 0;
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) {
            r[q] = uload16(b - 2 * back, off[q]);
            r[q] = shift_in_inf(r[q], back);
        }
    }
    __device__ __forceinline__ void store_chunk(uint4 *as, int q) const
    {
        as[(C::tid() % C::KC) * C::PA + (C::tid() / C::KC ^ C::tid() % C::KC) + q * (C::GT / C::KC)] =
            make_uint4(level_image(value2(r[q].x, q)), level_image(value2(r[q].y, q)),
                       level_image(value2(r[q].z, q)), level_image(value2(r[q].w, q)));
    }
    // one value, of another k by row (rows past the end are all the last one)
    __device__ __forceinline__ uint32_t first() const
    {
        const int row = C::tid() / C::KC;
        const uint64_t lo = (uint64_t)r[0].y << 32 | r[0].x, hi = (uint64_t)r[0].w << 32 | r[0].z;
        const uint32_t v = value2((uint32_t)(((row & 2) ? hi : lo) >> (row & 1) * 32), 0);
        return v >> (row & 4) * 4 & 0xFFFFu;
    }
    // largest finite value (signed: infinity is negative)
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

// Staging of the right operand, K rows from `base` (the block's first
// column; `cols` >= 1 of the block's columns exist, and the row has at least
// B_COLS up to its end): a thread takes 8 consecutive k (its k group) of
// B_COLS consecutive columns and writes one chunk per column.  Rows past K
// read the last row (the left operand is infinite there) and columns past
// the end hold any values of the row (their results are not used).
// Column n of a k group lies at chunk n ^ (n / 8 % 4): 8 consecutive lanes
// write to 8 different bank groups, and so do 8 lanes that read consecutive
// columns.
template <class C>
struct LevelB {
    static constexpr int TPG = C::BN / C::B_COLS;  // threads per k group
    gbytes *base, *at;
    int64_t K;
    uint32_t ldb2, coff;  // row bytes; byte offset of the thread's columns
    int back;             // columns that offset was moved back by to stay in the row
    uint32_t r[8][C::B_COLS / 2];
    __device__ __forceinline__ LevelB(const gu16 *p, int64_t ld, int cols, int64_t K_)
        : base((gbytes *)p), K(K_), ldb2((uint32_t)ld * 2u)
    {
        const int col = (C::tid() % TPG) * C::B_COLS;
        const int c = min(col, cols - C::B_COLS);  // may be negative: columns before the block
        back = col - c;
        base += min(0, cols - C::B_COLS) * 2;
        coff = (uint32_t)(c - min(0, cols - C::B_COLS)) * 2u;
    }
    __device__ __forceinline__ void take(int k, gbytes *b, uint32_t o)
    {
        if constexpr (C::B_COLS == 4) {
            const u32x2 v = *(const __attribute__((address_space(1))) u32x2_any *)(b + o);
            r[k][0] = v.x;
            r[k][1] = v.y;
        } else {
            r[k][0] = *(const __attribute__((address_space(1))) u32_any *)(b + o);
        }
    }
    __device__ __forceinline__ void seek(int64_t k0) { at = base + k0 * ldb2; }
    __device__ __forceinline__ void load()
    {
        const uint32_t o = (uint32_t)(C::tid() / TPG) * 8u * ldb2 + coff;
#pragma unroll
        for (int k = 0; k < 8; k++) take(k, at + (uint64_t)k * ldb2, o);
        at -= (uint64_t)(C::BK * C::KS) * ldb2;
    }
    __device__ __forceinline__ void load_tail(int64_t k0)
    {
        gbytes *b = base + k0 * ldb2;
        const int kg = C::tid() / TPG;
        const int last = (int)(K - k0) - 1;
#pragma unroll
        for (int k = 0; k < 8; k++) take(k, b, (uint32_t)min(kg * 8 + k, last) * ldb2 + coff);
    }
    // before the first store_chunk of a slice: columns moved back into place
    __device__ __forceinline__ void settle()
    {
        if (back) {
#pragma unroll
            for (int k = 0; k < 8; k++) {
                if constexpr (C::B_COLS == 4) {
                    const uint64_t v = ((uint64_t)r[k][1] << 32 | r[k][0]) >> (16 * (back & 3));
                    r[k][0] = (uint32_t)v;
                    r[k][1] = (uint32_t)(v >> 32);
                } else {
                    r[k][0] >>= 16 * (back & 1);
                }
            }
        }
    }
    __device__ __forceinline__ void store_chunk(uint4 *bs, int j) const
    {
        const int kg = C::tid() / TPG, n = C::tid() % TPG * C::B_COLS + j;
        uint32_t w[4];
#pragma unroll
        for (int p = 0; p < 4; p++)
            w[p] = level_image(__builtin_amdgcn_perm(r[2 * p + 1][j / 2], r[2 * p][j / 2],
                                                     (j & 1) ? 0x07060302u : 0x05040100u));
        bs[kg * C::PB + (n ^ ((n >> 3) & 3))] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    __device__ __forceinline__ uint32_t first() const { return r[0][0] & 0xFFFFu; }
    __device__ __forceinline__ i16x2 largest(i16x2 m) const
    {
#pragma unroll
        for (int k = 0; k < 8; k++)
#pragma unroll
            for (int e = 0; e < C::B_COLS / 2; e++)
                m = __builtin_elementwise_max(m, __builtin_bit_cast(i16x2, r[k][e]));
        return m;
    }
};

template <class C>
struct LevelAcc {
    uint32_t v[C::MI][C::NI][4];
};

// What a look at a block's values says: all that it saw are in the levels; a
// finite one is past LV_MAX, so its results can not all be proved by
// level_clean; so few are in range that the block gives up, for the f16 form or
// (minima of 2048 and more to be expected) the uint16 form of tile.h.
enum LevelView { LEVEL_IN, LEVEL_PAST, LEVEL_F16, LEVEL_U16 };
// Counts among n values of an operand: up to LV_MAX, up to LV_HALF, and finite
// ones past that.
struct LevelCount {
    int64_t in, half, over, n;
};
// The view that the counts of A and B give.  About half of the a.in b.in K /
// (a.n b.n) pairs of an output with both values in range sum to at most
// LV_MAX, and some ten of them are needed for all outputs of a block to have
// one.  A pass over K in vain costs a tenth of the VALU form that follows, and
// the VALU form in vain ten times the pass: so a block, which counts few
// values, gives up below LEVEL_NEED = 8 such pairs.  Likewise the f16 form, which is
// exact but for results of 2048 and more: uint16 where few pairs are of values
// up to LV_HALF and it is not infinity that takes their place.
constexpr int LEVEL_NEED = 8;
__device__ __forceinline__ LevelView level_view(const LevelCount &a, const LevelCount &b, int64_t K)
{
    const int64_t need = LEVEL_NEED * a.n * b.n;
    if (a.in * b.in * K >= need) return LEVEL_PAST;
    return a.half * b.half * K < need && (4 * a.over > a.half || 4 * b.over > b.half) ? LEVEL_U16 : LEVEL_F16;
}
constexpr int LEVEL_COUNTS = 6;  // words of LDS for a block's counts
constexpr uint32_t LV_HALF = 1023;
__device__ __forceinline__ int lanes_up_to(uint32_t v, uint32_t most) { return (int)__popcll(__ballot(v <= most)); }

// First values of the 64 x 64 cells of a block that leaves its outputs to
// another launch, for the f16 form or for uint16 at once: no block in the levels
// has such values (up to LV_SUM, or infinity).
constexpr u16 MARK_F16 = 0xFFFE, MARK_U16 = 0xFFFD;
constexpr int MARK_CELL = 64;

// The slices of K: slice 0 is the partial one at the end of K when there is
// one, so that no loop has an edge, and the others follow from the end to the
// start; group g of a block takes slices g, g + KS, ...
template <class C, class AOp, class BOp>
__device__ __forceinline__ void level_first(int64_t K, AOp &aop, BOp &bop)
{
    const int64_t full = K / C::BK;
    const int g = C::group();
    if (g == 0 && K % C::BK) {
        aop.load_tail(full * C::BK);
        bop.load_tail(full * C::BK);
        aop.seek((full - C::KS) * C::BK);
        bop.seek((full - C::KS) * C::BK);
    } else {
        const int64_t at = full - 1 - g + (K % C::BK ? 1 : 0);
        aop.seek(at * C::BK);
        bop.seek(at * C::BK);
        if (at < 0) return;  // fewer slices than groups
        aop.load();
        bop.load();
    }
}

// One slice: the products of LDS stage (as, bs), and beside them, when STORE,
// the next slice's registers into LDS and, when LOAD, the loads of the slice
// after that into the registers just freed.  All three kinds of work are
// interleaved by hand: a matrix instruction runs for 16 cycles, in which the
// wave's VALU takes two of the four maxima of the tile two before (its sums
// wait in registers meanwhile) and, on some tiles, converts a staged chunk.
// In the order the compiler chose, the matrix core idled during the maxima
// and the staging (N = 8192: matrix core 32 %, VALU 49 % busy).  A matrix
// instruction also takes two VALU issue slots (measured: 16 x 16 x 32 with
// four v_max_u32 26 cycles, 16.4 and 18 alone), so per slice of 64 x 64
// outputs a SIMD needs 162 VALU instructions and 32 x 2 slots: that, not the
// matrix core, is the bound, and the clock falls to 1.95 GHz under this load.
template <class C, bool STORE, bool LOAD, class AOp, class BOp>
__device__ __forceinline__ void level_slice(const uint4 *as0, const uint4 *as1, const uint4 *bs0, const uint4 *bs1,
                                            uint4 *next, AOp &aop, BOp &bop, LevelAcc<C> &acc)
{
    constexpr int T = C::MI * C::NI, PIECES = C::A_CPT + C::B_COLS, LAG = 2;
    bf16x8 bf[C::NI][2], af[2][2];
    auto readb = [&](int ni) {
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
            bf[ni][ks] = __builtin_bit_cast(bf16x8, ((ni & 1) ? bs1 : bs0)[4 * ks * C::PB + 16 * ni]);
    };
    readb(0);
#pragma unroll
    for (int ks = 0; ks < 2; ks++) af[0][ks] = __builtin_bit_cast(bf16x8, (ks ? as1 : as0)[0]);
    f32x4 t[LAG + 1][2];
    if (STORE) bop.settle();
    int piece = 0;
#pragma unroll
    for (int i = 0; i < T + LAG; i++) {
        const int mi = i / C::NI, ni = i % C::NI, o = i - LAG;
        if (i == 0) {
            readb(1);
            if (C::NI > 2) readb(2);
        } else if (i + 2 < C::NI) {
            readb(i + 2);
        }
        if (i < T && ni == 0 && mi + 1 < C::MI) {  // the next row of tiles' operand, a row ahead
#pragma unroll
            for (int ks = 0; ks < 2; ks++)
                af[(mi + 1) & 1][ks] = __builtin_bit_cast(bf16x8, (ks ? as1 : as0)[16 * (mi + 1)]);
        }
#pragma unroll
        for (int ks = 0; ks < 2; ks++) {
            if (i < T) {
                const f32x4 zero = {};
                t[i % (LAG + 1)][ks] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[ni][ks], af[mi & 1][ks], zero, 0, 0, 0);
            }
            if (o >= 0) {
#pragma unroll
                for (int r = 2 * ks; r < 2 * ks + 2; r++) {
                    const float f0 = t[o % (LAG + 1)][0][r], f1 = t[o % (LAG + 1)][1][r];
                    uint32_t &d = acc.v[o / C::NI][o % C::NI][r];
                    d = max(max(d, __builtin_bit_cast(uint32_t, f0)), __builtin_bit_cast(uint32_t, f1));
                }
            }
            if (ks == 1 && STORE) {
                const int upto = ((i + 1) * PIECES + T - 1) / T;
#pragma unroll
                for (; piece < upto && piece < PIECES; piece++) {
                    if (piece < C::A_CPT) {
                        aop.store_chunk(next, piece);
                        if (LOAD) aop.load_chunk(piece);
                    } else {
                        bop.store_chunk(next + C::KC * C::PA, piece - C::A_CPT);
                        if (LOAD && piece == PIECES - 1) bop.load();
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (LOAD) aop.advance();
}

// The k loop: acc = the largest 32-term sum of each output (its f32 bits),
// complete in group 0.  The product is taken transposed (D = B^T A^T): a lane
// then holds one row of C and runs of 4 consecutive columns.  With CHECK, a
// block whose first slice holds values past LV_MAX takes one value per thread
// of each operand there (cnt: LEVEL_COUNTS words of LDS) and returns what
// level_view makes of them: given up, the rest of the pass over K is saved
// (values 0..3000, 2200 x 2500 x 9000: 2.34 ms without, 2.10 with; values
// 0..15 at N = 16384: no difference).
template <class C, bool CHECK = false, class AOp, class BOp>
__device__ __forceinline__ LevelView level_kloop(int64_t K, AOp &aop, BOp &bop, uint4 *lds, LevelAcc<C> &acc,
                                                 int *cnt = nullptr)
{
    const int lane = (int)(threadIdx.x & 63);
    const int wm = C::wave() / C::WN, wn = C::wave() % C::WN;
    // k groups 0..3 and 4..7 of A
    const int aoff0 = (lane >> 4) * C::PA + wm * 16 * C::MI + ((lane & 15) ^ (C::SWZ ? lane >> 4 : 0));
    const int aoff1 = (aoff0 ^ (C::SWZ ? 4 : 0)) + 4 * C::PA;
    // even and odd tiles of 16 columns (LevelB's order of the chunks)
    const int boff0 = C::KC * C::PA + (lane >> 4) * C::PB + wn * 16 * C::NI + ((lane & 15) ^ ((lane >> 3) & 1));
    const int boff1 = boff0 ^ 2;
    uint4 *const all = lds;
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++)
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++)
#pragma unroll
            for (int r = 0; r < 4; r++) acc.v[mi][ni][r] = 0;
    // slices of this group, and the trips of the block (those of group 0)
    const int64_t slices = (K + C::BK - 1) / C::BK;
    int64_t left = (slices - C::group() + C::KS - 1) / C::KS, trips = (slices + C::KS - 1) / C::KS;
    lds += C::group() * 2 * C::STAGE;
    level_first<C>(K, aop, bop);
    bool past = false;
    uint32_t va = 0xFFFFu, vb = 0xFFFFu;
    if (left > 0) {
        if constexpr (CHECK) {
            const i16x2 m = bop.largest(aop.largest((i16x2){-1, -1}));
            past = max(m.x, m.y) > (int)LV_MAX;
            va = aop.first();
            vb = bop.first();
        }
#pragma unroll
        for (int q = 0; q < C::A_CPT; q++) aop.store_chunk(lds, q);
        bop.settle();
#pragma unroll
        for (int j = 0; j < C::B_COLS; j++) bop.store_chunk(lds + C::KC * C::PA, j);
    }
    if (left > 1) {
        aop.load();
        bop.load();
    }
    LevelView view = LEVEL_IN;
    if constexpr (CHECK) {
        if (threadIdx.x < LEVEL_COUNTS) cnt[threadIdx.x] = 0;
        if (__syncthreads_or(past)) {
            const auto finite = [](uint32_t v) { return v < 0x8000u ? v : 0u; };
            const int c[6] = {lanes_up_to(va, LV_MAX),       lanes_up_to(va, LV_HALF), 64 - lanes_up_to(finite(va), LV_HALF),
                              lanes_up_to(vb, LV_MAX),       lanes_up_to(vb, LV_HALF), 64 - lanes_up_to(finite(vb), LV_HALF)};
            if (lane == 0)
#pragma unroll
                for (int q = 0; q < 6; q++) atomicAdd(&cnt[q], c[q]);
            __syncthreads();
            // the partial slice of group 0 has infinity past K
            const int64_t groups = slices < C::KS ? slices : C::KS, part = K % C::BK ? K % C::BK : C::BK;
            const LevelCount ca{cnt[0], cnt[1], cnt[2], C::GT * (groups - 1) + C::GT * part / C::BK};
            const LevelCount cb{cnt[3], cnt[4], cnt[5], C::GT * groups};
            view = level_view(ca, cb, K);
            if (view > LEVEL_PAST) return view;
        }
    } else {
        __syncthreads();
    }
    for (int cur = 0;; cur ^= 1) {
        left--;  // slices of the group after this one
        uint4 *next = lds + (cur ^ 1) * C::STAGE;
        const uint4 *st = lds + cur * C::STAGE, *a0 = st + aoff0, *a1 = st + aoff1, *b0 = st + boff0, *b1 = st + boff1;
        if (left > 1)
            level_slice<C, true, true>(a0, a1, b0, b1, next, aop, bop, acc);
        else if (left == 1)
            level_slice<C, true, false>(a0, a1, b0, b1, next, aop, bop, acc);
        else if (left == 0)
            level_slice<C, false, false>(a0, a1, b0, b1, next, aop, bop, acc);
        __syncthreads();
        if (--trips == 0) break;
    }
    if constexpr (C::KS > 1) {  // the groups' maxima into group 0
        constexpr int REGS = C::MI * C::NI * 4;
        uint32_t *sh = (uint32_t *)all + C::tid();
        for (int g = 1; g < C::KS; g++) {
            if (C::group() == g) {
#pragma unroll
                for (int r = 0; r < REGS; r++) sh[r * C::GT] = acc.v[r / (C::NI * 4)][r / 4 % C::NI][r % 4];
            }
            __syncthreads();
            if (C::group() == 0) {
#pragma unroll
                for (int r = 0; r < REGS; r++) {
                    uint32_t &d = acc.v[r / (C::NI * 4)][r / 4 % C::NI][r % 4];
                    d = max(d, sh[r * C::GT]);
                }
            }
            __syncthreads();
        }
    }
    return view;
}

// Block row, and first of the 4 block columns, that the accumulators of wave
// tile (mi, ni) hold.
template <class C>
__device__ __forceinline__ int level_row(int mi)
{
    return (C::wave() / C::WN * C::MI + mi) * 16 + (int)(threadIdx.x & 15);
}
template <class C>
__device__ __forceinline__ int level_col(int ni)
{
    return (C::wave() % C::WN * C::NI + ni) * 16 + 4 * (int)((threadIdx.x >> 4) & 3);
}

// The value an accumulator stands for (infinity when no term was found).
__device__ __forceinline__ uint32_t level_value(uint32_t u)
{
    // u = m 2^e with m in [1/2, 1): e = 119 - 6 t .. 124 - 6 t
    const int e = __builtin_amdgcn_frexp_expf(__builtin_bit_cast(float, u));
    const uint32_t t = ((uint32_t)(LV_TOP + 6 - e) * 171u) >> 10;  // floor of a sixth, exact below 512
    return u == 0 ? 0xFFFFu : t;
}

// True (block-uniform) when every result of the block inside rows x cols is
// certainly exact: no accumulator below LV_SURE.
template <class C>
__device__ __forceinline__ bool level_sure(const LevelAcc<C> &acc, int rows, int cols)
{
    bool bad = false;
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++) {
        const bool rin = C::group() == 0 && level_row<C>(mi) < rows;
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++)
#pragma unroll
            for (int j = 0; j < 4; j++) bad |= rin && level_col<C>(ni) + j < cols && acc.v[mi][ni][j] < LV_SURE;
    }
    return !__syncthreads_or(bad);
}

// Largest finite value over the block of what `fold` makes of m (a pair of
// signed halves, infinity negative); lds is free before and after.
template <class C, class Fold>
__device__ __forceinline__ int level_largest(uint4 *lds, Fold fold)
{
    const i16x2 m = fold((i16x2){-1, -1});
    int *sh = (int *)lds;
    if (threadIdx.x == 0) sh[0] = 0;
    __syncthreads();
    atomicMax(&sh[0], max((int)m.x, (int)m.y));
    __syncthreads();
    const int a = sh[0];
    __syncthreads();
    return a;
}

// True (block-uniform) when no finite operand of the block exceeds LV_MAX
// and no finite sum exceeds LV_SUM, so every accumulator is exact.  One more
// pass over the operands; lds is free.
template <class C, class AOp, class BOp>
__device__ __forceinline__ bool level_clean(int64_t K, AOp &aop, BOp &bop, uint4 *lds)
{
    const int64_t slices = (K + C::BK - 1) / C::BK, left = (slices - C::group() + C::KS - 1) / C::KS;
    i16x2 mb = {-1, -1};
    const int a = level_largest<C>(lds, [&](i16x2 ma) {
        if (left > 0) level_first<C>(K, aop, bop);
        for (int64_t j = 0; j < left; j++) {
            if (j > 0) {
                aop.load();
                bop.load();
            }
            ma = aop.largest(ma);
            mb = bop.largest(mb);
        }
        return ma;
    });
    const int b = level_largest<C>(lds, [&](i16x2 m) { return __builtin_elementwise_max(m, mb); });
    return a <= (int)LV_MAX && b <= (int)LV_MAX && a + b <= (int)LV_SUM;
}

// Writes the block's results inside rows x cols to C (row 0, column 0 of the
// block at `out`).  The 16-lane rows 0..3 of a wave hold columns 0-3, 4-7,
// 8-11 and 12-15 of a tile; the odd ones trade with their neighbours between
// two tiles, so that each lane writes 8 consecutive columns (16 bytes).
template <class C>
__device__ __forceinline__ void level_store(gu16 *out, int64_t ldc, int rows, int cols, const LevelAcc<C> &acc)
{
    const int quarter = (int)((threadIdx.x >> 4) & 3);
    if (C::group() != 0) return;
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++) {
        const int row = level_row<C>(mi);
#pragma unroll
        for (int ni = 0; ni < C::NI; ni += 2) {
            uint32_t w[2][2];
#pragma unroll
            for (int e = 0; e < 2; e++)
#pragma unroll
                for (int h = 0; h < 2; h++)
                    w[e][h] = level_value(acc.v[mi][ni + e][2 * h]) | (level_value(acc.v[mi][ni + e][2 * h + 1]) << 16);
            const auto s0 = __builtin_amdgcn_permlane16_swap(w[0][0], w[1][0], false, false);
            const auto s1 = __builtin_amdgcn_permlane16_swap(w[0][1], w[1][1], false, false);
            const int col = (C::wave() % C::WN * C::NI + ni + (quarter & 1)) * 16 + (quarter >> 1) * 8;
            if (row >= rows) continue;
            gu16 *g = out + (int64_t)row * ldc + col;
            const uint4 v = make_uint4(s0[0], s1[0], s0[1], s1[1]);
            if (col + 8 <= cols) {
                ustore16(g, v);
            } else {
#pragma unroll
                for (int e = 0; e < 8; e++)
                    if (col + e < cols) g[e] = (u16)(comp(v, e >> 1) >> ((e & 1) * 16));
            }
        }
    }
}

// ------------------------------------------------ a chain step, normalised late
// One step O = L (x) A of a chain whose rows keep their offsets until the
// next step reads them: L holds the raw previous product, low_in[i] its row
// minima and big_in[i] its rows' largest finite values where they can exceed
// MPR_FMAX, so the step multiplies the canonical form L - low_in (the scalar
// rule of Section 3) and R gains low_in.  That saves the pass over the matrix,
// and the launch, that a normalisation after every product costs.  The step
// leaves the row minima and maxima of O in low_out / big_out (set to LOW_NONE
// and 0 before) and prepares low_next / big_next for the step after.
struct LevelStep {
    const u16 *L, *A;
    u16 *O;
    int64_t ldl, lda, ldo, n;
    int64_t *R;
    const uint32_t *low_in, *big_in;
    uint32_t *low_out, *big_out, *low_next, *big_next;
    // Outputs, in tiles of 64 x 64, of blocks that had a finite result past
    // LV_MAX in the step before, and of those with one past 2047; the same of
    // this step; the words to clear (rotated in the same way).  Where most of
    // the step before was past the levels, a block goes to the VALU tile at
    // once (n = 848, entries 0..3000: 57 us a step with the pass over K in
    // vain, 42 without).  The first step has 0 and 0, and looks at its values.
    const uint32_t *past_in;
    uint32_t *past_out, *past_next;
};
constexpr int LEVEL_PASTS = 2;
constexpr uint32_t LOW_NONE = 0xFFFFu;  // no finite value in the row

// Row minima of the block into low (the block's first row), from the largest
// accumulator of each row.
template <class C>
__device__ __forceinline__ void level_row_low(const LevelAcc<C> &acc, int rows, int cols, uint32_t *low)
{
    if (C::group() != 0) return;
#pragma unroll
    for (int mi = 0; mi < C::MI; mi++) {
        uint32_t u = 0;
#pragma unroll
        for (int ni = 0; ni < C::NI; ni++)
#pragma unroll
            for (int r = 0; r < 4; r++) u = max(u, level_col<C>(ni) + r < cols ? acc.v[mi][ni][r] : 0u);
        u = max(u, (uint32_t)__shfl_xor((int)u, 16, 64));
        u = max(u, (uint32_t)__shfl_xor((int)u, 32, 64));
        const int row = level_row<C>(mi);
        if ((threadIdx.x & 63) < 16 && row < rows && u) atomicMin(&low[row], level_value(u));
    }
}

// The rows' bookkeeping, by the block of column 0: the offsets they lost to
// the previous step move into R, and the buffers of the step after are
// cleared.  Returns (to every thread) whether an offset of the block's rows
// passes 0x7FFF: no room above the levels for infinity then.
template <class C>
__device__ __forceinline__ bool level_step_rows(const LevelStep &p, int64_t m0, int rows, bool first, int32_t *st)
{
    bool far = false;
    for (int r = threadIdx.x; r < rows; r += C::NT) {
        const int64_t i = m0 + r;
        const uint32_t l = p.low_in[i];
        far |= l > FMAX16 && l != LOW_NONE;
        if (first) {
            p.low_next[i] = LOW_NONE;
            p.big_next[i] = 0;
            p.R[i] = (l == LOW_NONE || p.R[i] == ROW_NONE) ? ROW_NONE : p.R[i] + (int64_t)l;
            if (l != LOW_NONE && p.big_in[i] > l + FMAX16) set_status(st, MPR_EOVERFLOW);
        }
    }
    return __syncthreads_or(far);
}

// Takes the offset l off the halves of x; infinity stays.
__device__ __forceinline__ uint32_t take_low(uint32_t x, uint32_t l)
{
    const uint32_t lo = x & 0xFFFFu, hi = x >> 16;
    return (lo == 0xFFFFu ? lo : lo - l) | (hi == 0xFFFFu ? hi : hi - l) << 16;
}

// A block that the VALU tile computed: its results, row minima and maxima, and
// what they tell the next step (called by every thread).  LOW: the minima and
// maxima are wanted.
template <class T, bool LOW = true>
__device__ __forceinline__ void level_step_back(const LevelStep &p, int64_t m0, int64_t n0, int rows, bool vec,
                                                const TileAcc<T> &acc)
{
    uint32_t most = 0;  // largest finite value + 1
    if (T::group() == 0) {
        tile_store<T>(p.O, p.ldo, p.n, p.n, m0, n0, vec, acc);
#pragma unroll
        for (int r = 0; r < T::TM; r++) {
            // columns and rows past the end are infinite
            u16x2 mn = {0xFFFF, 0xFFFF}, mx = {0, 0};  // mx: largest finite value + 1
#pragma unroll
            for (int q = 0; q < T::NACC; q++) {
                mn = min2(mn, acc.v[r][q]);
                mx = __builtin_elementwise_max(mx, (u16x2)(acc.v[r][q] + (u16x2){1, 1}));
            }
            uint32_t m = min((uint32_t)mn.x, (uint32_t)mn.y), x = max((uint32_t)mx.x, (uint32_t)mx.y);
#pragma unroll
            for (int off = 1; off < T::TX; off <<= 1) {
                m = min(m, (uint32_t)__shfl_xor((int)m, off, 64));
                x = max(x, (uint32_t)__shfl_xor((int)x, off, 64));
            }
            most = max(most, x);
            const int row = tile_row<T>(r);
            if (LOW && T::tid() % T::TX == 0 && row < rows && x) {
                atomicMin(&p.low_out[m0 + row], m);
                atomicMax(&p.big_out[m0 + row], x - 1);
            }
        }
    }
    constexpr uint32_t AREA = T::BM * T::BN / (64 * 64);
    const bool past = __syncthreads_or(most > LV_MAX + 1), deep = __syncthreads_or(most > 0x800);
    if (threadIdx.x != 0) return;
    if (past) atomicAdd(&p.past_out[0], AREA);
    if (deep) atomicAdd(&p.past_out[1], AREA);
}

// The block of rows m0.. and columns n0.. of a step; T is the VALU tile of
// the same shape and threads for blocks whose values leave the level range.
// FIRST: the first step of a chain.
template <class C, class T, bool FIRST>
__device__ __forceinline__ void level_step_block(const LevelStep &p, int64_t m0, int64_t n0, uint4 *lds, int32_t *st)
{
    __shared__ int cnt[LEVEL_COUNTS];
    const int rows = (int)min<int64_t>(C::BM, p.n - m0), cols = (int)min<int64_t>(C::BN, p.n - n0);
    const uint32_t past = p.past_in[0], deep = p.past_in[1];
    if (m0 == 0 && n0 == 0 && threadIdx.x < LEVEL_PASTS) p.past_next[threadIdx.x] = 0;
    const bool far = level_step_rows<C>(p, m0, rows, n0 == 0, st);
    LevelView view = 2 * deep > past ? LEVEL_U16 : LEVEL_F16;
    if (!far && 2 * 64 * 64 * (int64_t)past <= p.n * p.n) {
        LevelA<C, true> aop(glob(p.L) + m0 * p.ldl, p.ldl, rows, p.n, p.low_in + m0);
        LevelB<C> bop(glob(p.A) + n0, p.lda, cols, p.n);
        LevelAcc<C> acc;
        // (a look in every step costs one of n = 848 3 %; large blocks nothing)
        view = level_kloop<C, FIRST || (C::MI > 2)>(p.n, aop, bop, lds, acc, cnt);
        if (view <= LEVEL_PAST &&
            (level_sure<C>(acc, rows, cols) || (view == LEVEL_IN && level_clean<C>(p.n, aop, bop, lds)))) {
            level_row_low<C>(acc, rows, cols, p.low_out + m0);
            level_store<C>(glob(p.O) + m0 * p.ldo + n0, p.ldo, rows, cols, acc);
            return;
        }
    }
    const bool vec = (uintptr_t)p.L % 16 == 0 && (uintptr_t)p.A % 16 == 0 && (uintptr_t)p.O % 16 == 0 &&
                     p.ldl % 8 == 0 && p.lda % 8 == 0 && p.ldo % 8 == 0;
    TileAcc<T> acc;
    tile_split<T>(
        (p.n + T::BK - 1) / T::BK,
        [&](int64_t k0, int row, int kc) {
            const uint4 v = load8(p.L, p.ldl, m0 + row, k0 + kc, p.n, p.n, vec);
            const uint32_t l = row < rows ? p.low_in[m0 + row] : 0;
            return make_uint4(take_low(v.x, l), take_low(v.y, l), take_low(v.z, l), take_low(v.w, l));
        },
        [&](int64_t k0, int kr, int jc) { return load8(p.A, p.lda, k0 + kr, n0 + jc, p.n, p.n, vec); }, (u16 *)lds,
        acc, view == LEVEL_U16);
    level_step_back<T>(p, m0, n0, rows, vec, acc);
}

// Block shapes of the products and steps, each with the VALU tile that
// stands in for it.
using LCfg0 = LevelCfg<4, 4, 2, 2>;  // 256 threads, 128 x 128
using LCfg1 = LevelCfg<2, 2, 2, 2>;  // 256 threads, 64 x 64
using LCfg2 = LevelCfg<4, 4, 2, 2, 2>;  // 512 threads, 128 x 128
using LCfg3 = LevelCfg<2, 2, 2, 2, 2>;  // 512 threads, 64 x 64
using LCfg4 = LevelCfg<4, 4, 2, 4>;     // 512 threads, 128 x 256
template <class C> struct LevelBack;
template <> struct LevelBack<LCfg0> { using T = TileCfg<128, 128, 32, 8, 8>; };
template <> struct LevelBack<LCfg1> { using T = TileCfg<64, 64, 16, 4, 8, 2>; };
template <> struct LevelBack<LCfg2> { using T = TileCfg<128, 128, 32, 8, 8, 2>; };
template <> struct LevelBack<LCfg4> { using T = TileCfg<128, 256, 32, 8, 8>; };
template <> struct LevelBack<LCfg3> { using T = TileCfg<64, 64, 32, 4, 8, 4>; };
// LDS of a block (16-byte chunks): its own, or the VALU tile's if larger.
template <class C>
struct LevelLds {
    using T = typename LevelBack<C>::T;
    static_assert(T::NT * T::G == C::NT && C::BM == T::BM && C::BN == T::BN, "stand-in tile");
    static constexpr int BACK = (T::G * T::LDS_ELEMS + 7) / 8;
    static constexpr int CHUNKS = C::LDS_CHUNKS > BACK ? C::LDS_CHUNKS : BACK;
};

// sparse.hip: the rows of a plan whose counts sparse_plan_rows left in ws, as
// values or (for sparse_step8_launch) as level images.
mpr_status sparse_plan_fill(const u16 *A, int64_t n, int64_t lda, void *ws, size_t bytes, bool images, int32_t *st,
                            hipStream_t s);

// period.hip: one pass over a power of a period search (canonical form to dst,
// offsets, and into rec the class hash, trace, status and seq), and the
// accumulator of 8 n bytes, rounded up to 256, that it folds into (cleared
// once; every pass leaves it clear).
mpr_status period_clear_launch(void *acc, int64_t n, hipStream_t s);
// The same over a power in bytes, in groups of 8 columns: [column / 8][row]
// [column % 8], the rows padded to whole lines, at most as large as its n rows
// of u16.  Raw sums with 255 = infinity (or, first not null, the u16 matrix
// `first`, row stride lda) become level bytes, 93 - 3 v for v <= 30 and 0 for
// infinity, padding included.  A larger value raises *wide; *big receives the
// largest v.  rec[3] = *wide.
inline int64_t level_group8(int64_t n) { return 8 * round_up(n, 16); }  // bytes of a group
mpr_status period_rows8_launch(const u16 *first, int64_t lda, uint8_t *N, int64_t n, const int64_t *R_in,
                               int64_t *R_out, void *acc, int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                               int64_t seq, hipStream_t s);
// The step and that pass at once, for n <= PERIOD_SMALL_N: N the power before
// (null: the power is A itself), O the next, level bytes in rows of ld8 >= n.
constexpr int64_t PERIOD_SMALL_N = 64;
mpr_status period_small_launch(const u16 *A, int64_t lda, const uint8_t *N, uint8_t *O, int64_t ld8, int64_t n,
                               const int64_t *R_in, int64_t *R_out, int64_t *rec, int64_t seq, hipStream_t s);
// rowops.hip: exact compare of two canonical forms up to a scalar shift, `rows`
// <= n rows of `cols` values and n offsets.
mpr_status compare_rows_launch(const u16 *X, const int64_t *RX, const u16 *Y, const int64_t *RY, int64_t n, int64_t rows,
                               int64_t cols, int64_t ld, int64_t *out3, hipStream_t s);
// sparse.hip: the compressed-K step from level bytes to raw bytes; raises
// *wide when a block can not be decided from values up to *big.
mpr_status sparse_step8_launch(const uint8_t *N, int64_t n, void *ws, size_t bytes, uint8_t *O,
                               int32_t *wide, const int32_t *big, hipStream_t s);
mpr_status period_rows_launch(const u16 *src, int64_t lds_, u16 *dst, int64_t ldd, int64_t n, const int64_t *R_in,
                              int64_t *R_out, bool raw, void *acc, int32_t *st, int64_t *rec, int64_t seq, hipStream_t s);

// abi.hip: 16 words of pinned host memory, two records of 8 words that kernels
// on stream s write (word 7 last, when the others are in place), and the wait
// for one.  A few stay allocated between calls (a pinned allocation and its
// release take 50 us); taken and given back from any thread.  Every writer has
// a ticket of its own, taken before its launch: no other call's late write can
// be taken for it, and a record whose newest ticket has not been seen is given
// back only once the stream is idle.
struct HostRecord {
    int64_t *p;
    explicit HostRecord(hipStream_t stream);
    ~HostRecord();
    HostRecord(const HostRecord &) = delete;
    HostRecord &operator=(const HostRecord &) = delete;
    int64_t ticket();
    mpr_status wait(const int64_t *rec, int64_t seq);
    mpr_status drain();  // waits for the stream

private:
    hipStream_t s;
    int64_t newest = 0, seen = 0;
};

// The compressed-K step (sparse.hip) in the same way; p.A is not read.
bool sparse_step_late(int64_t n, int64_t ldl, int64_t ldo);  // whether it applies
mpr_status sparse_step_late_launch(const LevelStep &p, void *ws, size_t bytes, int64_t step, int32_t *st,
                                   hipStream_t s);

// abi.hip: the argument checks of a product.
mpr_status mpr_gemm_args(int cfg, int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B, int64_t ldb,
                         const u16 *C, int64_t ldc);

inline bool level_strides(int64_t lda, int64_t ldb) { return lda < (1 << 22) && ldb < (1 << 22); }
int level_shape(int64_t M, int64_t N);

// A chain step in the shape for its size, and the row minima and maxima of
// the first power and for its first step (3 n words each in rotation: a step
// reads one third, writes the next and clears the last), and likewise the 3
// LEVEL_PASTS words.  first: the first step of a chain.
mpr_status level_step_launch(const LevelStep &p, bool first, int32_t *st, hipStream_t s);
mpr_status level_prepare_launch(uint32_t *low, uint32_t *big, uint32_t *past, int64_t n, hipStream_t s);

// gemm.hip: the tiles of C with a marked cell, in the tile table's configuration.
mpr_status gemm_past_launch(bool spare, int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B,
                            int64_t ldb, u16 *C, int64_t ldc, hipStream_t s);

// The product C = A (x) B: configuration cfg of gemm.hip, or (cfg = -1) the
// level form where it applies and the tile table's configuration elsewhere.
mpr_status product_launch(int cfg, int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B,
                          int64_t ldb, u16 *C, int64_t ldc, hipStream_t s);
// The same, leaving room on every CU for other launches.
mpr_status product_launch_spare(int cfg, int64_t M, int64_t N, int64_t K, const u16 *A, int64_t lda, const u16 *B,
                                int64_t ldb, u16 *C, int64_t ldc, hipStream_t s);

}  // namespace mpr
