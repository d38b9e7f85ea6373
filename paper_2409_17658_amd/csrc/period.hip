// period.hip -- what the period search does with each power it computes, in
// one pass: row minima taken off (canonical form), offsets, the hash of the
// power's class up to a scalar shift, its trace and its overflow check, with
// the results written where the host reads them.
//
// Bound by memory: a power is read and written once (m = 9: 1.92 GB).  The
// class hash only sorts powers before an exact comparison, so it is chosen
// for its cost: per row the sum of (w0 + k0) (w1 + k1) over pairs of 32-bit
// words with keys by position (the NH hash of UMAC, Black et al. 1999), one
// multiply-add per 4 entries instead of two 64-bit multiplications per entry,
// and for the offsets a linear sum, whose shift by the least offset can be
// taken off at the end.  Each block folds its row into one of PSLOTS slots
// and the last block combines them, where two more kernels of one block used
// to read n words each (m = 8: 68 + 13 + 9 us, in bytes 30; m = 9: 410 + 51 +
// 24 us, in bytes 246; m = 3: 6.0 + 3.4 + 3.3 us and a copy to the host, now
// within the 6.7 us of a whole power).
#include <algorithm>

#include "level.h"

namespace mpr {

constexpr int PSLOTS = 32;
constexpr int RT = 256;  // threads per row

struct PeriodSlot {
    uint64_t hash, offsets, keys;  // sums over the rows
    int64_t least, trace;          // minima over the rows
    uint32_t done, pad[5];         // blocks folded in
};
static_assert(sizeof(PeriodSlot) == 64, "a slot to a half line");
struct PeriodAcc {
    uint32_t full, pad[15];  // slots complete
    PeriodSlot slot[PSLOTS];
};
// Slots in use: as many as fit the 8 n bytes, rounded up to 256, that a
// workspace has for the accumulator.
static int period_slots(int64_t n)
{
    return (int)std::min<int64_t>(PSLOTS, round_up(8 * n, 256) / (int64_t)sizeof(PeriodSlot) - 1);
}

__device__ __forceinline__ void period_clear(PeriodAcc *a, int t, int slots)
{
    if (t < slots) {
        PeriodSlot z{};
        z.least = z.trace = ROW_NONE;
        a->slot[t] = z;
    }
    if (t == 0) a->full = 0;
}
__global__ void period_clear_kernel(PeriodAcc *a, int slots) { period_clear(a, (int)threadIdx.x, slots); }

template <class X>
__device__ __forceinline__ X agent_add(X *p, X v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t agent_min(int64_t *p, int64_t v)
{
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keys by position: multiples of 2^32 / phi, told apart by multipliers of
// MurmurHash3's finaliser and of xxHash (any odd constants would do).
__device__ __forceinline__ uint64_t nh4(const uint32_t w[4], uint32_t pos)
{
    const uint32_t k = (pos + 1u) * 0x9E3779B1u;
    return (uint64_t)(w[0] + k) * (w[1] + (k ^ 0x85EBCA6Bu)) +
           (uint64_t)(w[2] + (k ^ 0xC2B2AE35u)) * (w[3] + (k ^ 0x27D4EB2Fu));
}

// 8 values of a row from column c, infinite past its end n.
__device__ __forceinline__ uint4 row8(const gu16 *row, int64_t c, int64_t n)
{
    if (c + 8 <= n) {
        const u32x4 v = *(const __attribute__((address_space(1))) u32x4_any *)(row + c);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const uint32_t lo = c + 2 * e < n ? row[c + 2 * e] : 0xFFFFu;
        const uint32_t hi = c + 2 * e + 1 < n ? row[c + 2 * e + 1] : 0xFFFFu;
        w[e] = lo | (hi << 16);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// One row's part in its power (m: least value, diag: diagonal value, h: hash
// of its entries); its offset goes to R_out.
struct RowPart {
    uint64_t hash, offsets, keys;
    int64_t least, trace;
};
__device__ __forceinline__ RowPart period_row(int64_t i, uint32_t m, uint32_t diag, uint64_t h, const int64_t *R_in,
                                              int64_t *R_out)
{
    const int64_t rin = R_in ? R_in[i] : 0;
    const bool none = m == 0xFFFFu || rin == ROW_NONE;
    const int64_t R = none ? ROW_NONE : rin + (int64_t)m;
    R_out[i] = R;
    const uint64_t rh = mix64(h ^ mix64((uint64_t)i ^ 0x6A09E667F3BCC909ull));
    const uint64_t key = mix64((uint64_t)i ^ 0xBB67AE8584CAA73Bull);
    if (none) return RowPart{rh + 1, 0, 0, ROW_NONE, ROW_NONE};
    return RowPart{rh, key * (uint64_t)R, key, R, diag != 0xFFFFu ? R + (int64_t)(diag - m) : ROW_NONE};
}

// Folds a block's rows into the power, called by every thread (x and refuse
// of thread 0; refuse: 1 out of range, 2 wide).  wide: a second status word
// for the record, or null.
__device__ __forceinline__ void period_fold(const RowPart &x, int refuse, PeriodAcc *acc, int nslots, int32_t *st,
                                            int32_t *wide, int64_t *rec, int64_t seq, int *last)
{
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    if (threadIdx.x == 0) {
        PeriodSlot *s = &acc->slot[blockIdx.x % (uint32_t)nslots];
        // every fold completes (its old value arrives) before the block counts
        uint64_t seen = agent_add(&s->hash, x.hash);
        if (x.least != ROW_NONE) {
            seen |= agent_add(&s->offsets, x.offsets) | agent_add(&s->keys, x.keys);
            seen |= (uint64_t)agent_min(&s->least, x.least);
            if (x.trace != ROW_NONE) seen |= (uint64_t)agent_min(&s->trace, x.trace);
        }
        if (refuse & 1)
            seen |= (uint64_t)__hip_atomic_exchange(st, MPR_EOVERFLOW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (refuse & 2) seen |= (uint64_t)__hip_atomic_exchange(wide, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" : : "v"(seen) : "memory");
        const uint32_t blocks = ((uint32_t)gridDim.x + nslots - 1 - blockIdx.x % (uint32_t)nslots) / nslots;  // of this slot
        const uint32_t slots = min((uint32_t)gridDim.x, (uint32_t)nslots);
        *last = 0;
        if (agent_add(&s->done, 1u) + 1 == blocks) *last = agent_add(&acc->full, 1u) + 1 == slots;
    }
    __syncthreads();
    if (!*last || w != 0) return;
    // The last block of the power: one lane per slot (reads at the place where
    // the folds happened), then the record and a clear accumulator.
    PeriodSlot *s = &acc->slot[lane < nslots ? lane : 0];
    uint64_t hs = lane < nslots ? agent_add(&s->hash, (uint64_t)0) : 0;
    uint64_t os = lane < nslots ? agent_add(&s->offsets, (uint64_t)0) : 0;
    uint64_t ks = lane < nslots ? agent_add(&s->keys, (uint64_t)0) : 0;
    const int64_t lo = wave_min_i64(agent_min(&s->least, ROW_NONE));
    const int64_t tr = wave_min_i64(agent_min(&s->trace, ROW_NONE));
    hs = wave_sum_u64(hs);
    os = wave_sum_u64(os);
    ks = wave_sum_u64(ks);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    period_clear(acc, lane, nslots);
    if (lane != 0) return;
    const int32_t code = __hip_atomic_load(st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    rec[0] = (int64_t)mix64(hs + mix64(os - (lo == ROW_NONE ? 0 : (uint64_t)lo * ks)));
    rec[1] = tr;
    rec[2] = code;
    rec[3] = wide ? __hip_atomic_load(wide, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Row i = blockIdx.x of src (raw) to dst (canonical; may be src).  RAW: src is
// an input matrix, whose finite entries must not exceed MPR_FMAX either.  NCH
// chunks of 8 columns per thread stay in registers between the minimum and
// the subtraction; 0 reads the row twice.  rec (host or device): [0] hash,
// [1] trace, [2] status, then [7] = seq once the others are written.
template <int NCH>
__global__ __launch_bounds__(RT) void period_rows_kernel(const u16 *src, int64_t lds_, u16 *dst, int64_t ldd, int64_t n,
                                                         const int64_t *R_in, int64_t *R_out, int raw, PeriodAcc *acc,
                                                         int nslots, int32_t *st, int64_t *rec, int64_t seq)
{
    __shared__ uint32_t least[RT / 64];
    __shared__ uint64_t hsum[RT / 64];
    __shared__ uint32_t diag;
    __shared__ int last, refuse;
    const int64_t i = blockIdx.x;
    const gu16 *row = glob(src) + i * lds_;
    gu16 *out = glob(dst) + i * ldd;
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    uint4 keep[NCH > 0 ? NCH : 1];
    u16x2 mn = {0xFFFF, 0xFFFF};
    bool over = false;
    auto fold = [&](const uint4 &v) {
#pragma unroll
        for (int e = 0; e < 4; e++) mn = min2(mn, as_u16x2(comp(v, e)));
        if (raw)  // a finite value past MPR_FMAX: bit 15 set and not infinity
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t x = comp(v, e), lo = x & 0xFFFFu, hi = x >> 16;
                over |= (lo > FMAX16 && lo != 0xFFFFu) || (hi > FMAX16 && hi != 0xFFFFu);
            }
    };
    const int64_t c0 = (int64_t)threadIdx.x * 8;
    if constexpr (NCH > 0) {
#pragma unroll
        for (int q = 0; q < NCH; q++) {
            const int64_t c = c0 + (int64_t)q * RT * 8;
            keep[q] = c < n ? row8(row, c, n) : make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
            fold(keep[q]);
        }
    } else {
        for (int64_t c = c0; c < n; c += RT * 8) fold(row8(row, c, n));
    }
    uint32_t m = wave_min_u32(min((uint32_t)mn.x, (uint32_t)mn.y));
    if (lane == 0) least[w] = m;
    if (threadIdx.x == 0) {
        diag = row[i];  // before the row is rewritten
        refuse = 0;
    }
    __syncthreads();
    m = min(min(least[0], least[1]), min(least[2], least[3]));
    const bool empty = m == 0xFFFFu;
    const u16x2 m2 = {(u16)m, (u16)m};
    uint64_t h = 0;
    auto finish = [&](const uint4 &v, int64_t c) {
        uint32_t x[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const u16x2 a = as_u16x2(comp(v, e));
            const u16x2 inf = {(u16)(a.x == 0xFFFF ? 0xFFFF : 0), (u16)(a.y == 0xFFFF ? 0xFFFF : 0)};
            const u16x2 s = empty ? a : (u16x2)((a - m2) | inf);
            over |= (s.x > FMAX16 && s.x != 0xFFFF) || (s.y > FMAX16 && s.y != 0xFFFF);
            x[e] = as_u32(s);
        }
        h += nh4(x, (uint32_t)(c >> 3));
        if (c + 8 <= n) {
            ustore16(out + c, make_uint4(x[0], x[1], x[2], x[3]));
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++)
                if (c + e < n) out[c + e] = (u16)(x[e >> 1] >> ((e & 1) * 16));
        }
    };
    if constexpr (NCH > 0) {
#pragma unroll
        for (int q = 0; q < NCH; q++) {
            const int64_t c = c0 + (int64_t)q * RT * 8;
            if (c < n) finish(keep[q], c);
        }
    } else {
        for (int64_t c = c0; c < n; c += RT * 8) finish(row8(row, c, n), c);
    }
    if (over) refuse = 1;
    h = wave_sum_u64(h);
    if (lane == 0) hsum[w] = h;
    __syncthreads();
    RowPart x{};
    if (threadIdx.x == 0) x = period_row(i, m, diag, hsum[0] + hsum[1] + hsum[2] + hsum[3], R_in, R_out);
    period_fold(x, refuse, acc, nslots, st, nullptr, rec, seq, &last);
}

// The same in bytes (level bytes in column groups, sparse.hip), 16 rows to a
// block, whose bytes of a group are one 128-byte line: a lane takes 2 rows of
// 8 columns, 8 lanes a line, NCH groups a thread in registers (0: read
// twice).  FIRST: the source is the u16 matrix X.  *big receives the largest
// canonical value, for the step that reads it.  A row to a fold left the pass
// to its atomics (m = 8 47 us, m = 9 300; now 30 and 246, 0.96 GB at 3.9 TB/s).
constexpr int GROWS = 16;
template <int T, int NCH, bool FIRST>
__global__ __launch_bounds__(T) void period_rows8_kernel(const u16 *X, int64_t ldx, uint8_t *N, int64_t group8, int64_t n,
                                                         const int64_t *R_in, int64_t *R_out, PeriodAcc *acc,
                                                         int nslots, int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                                                         int64_t seq)
{
    constexpr int W = T / 64, GSTEP = T / 8;  // groups of a sweep
    __shared__ uint32_t least[W][GROWS], most[W][GROWS], diag[GROWS];
    __shared__ uint64_t hash[W][GROWS];
    __shared__ int last;
    const int t = (int)threadIdx.x, lane = t & 63, w = t >> 6, pr = t & 7;
    const int64_t i0 = (int64_t)blockIdx.x * GROWS, i = i0 + 2 * pr, groups = (n + 7) / 8;
    // a sweep's first byte is the same for all threads; 127 groups span 32 bits
    const uint32_t at = (uint32_t)(i * 8 + (t >> 3) * group8);
    if (t < GROWS) {
        const int64_t d = i0 + t;
        uint32_t v = 0xFFFF;
        if (d < n) {
            v = FIRST ? (uint32_t)glob(X)[d * ldx + d] : (uint32_t)glob(N)[(d >> 3) * group8 + d * 8 + (d & 7)];
            if (!FIRST && v == 0xFF) v = 0xFFFF;
        }
        diag[t] = v;
    }
    // even and odd columns 2 q, 2 q + 1 of 4: u[2 row + half] = columns 4 half ..
    struct Piece {
        u16x2 ev[4], od[4];
    };
    typedef __attribute__((address_space(1))) u32x4 piece_bytes;
    auto split = [&](u32x4 d) {
        Piece x;
        const uint32_t u[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int q = 0; q < 4; q++) {
            x.ev[q] = as_u16x2(u[q] & 0x00FF00FFu);
            x.od[q] = as_u16x2(u[q] >> 8 & 0x00FF00FFu);
        }
        return x;
    };
    auto first = [&](int64_t g) {
        Piece x;
#pragma unroll
        for (int r = 0; r < 2; r++) {
            uint4 v = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
            if (i + r < n) v = row8(glob(X) + (i + r) * ldx, g * 8, n);
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const uint32_t lo = h ? v.z : v.x, hi = h ? v.w : v.y;
                x.ev[2 * r + h] = as_u16x2(__builtin_amdgcn_perm(hi, lo, 0x05040100u));
                x.od[2 * r + h] = as_u16x2(__builtin_amdgcn_perm(hi, lo, 0x07060302u));
            }
        }
        return x;
    };
    constexpr u16 INFV = FIRST ? 0xFFFF : 0xFF;
    u16x2 mn[2], mx[2];  // mx: largest finite value + 1 (infinity + 1 is 0)
    mn[0] = mn[1] = (u16x2){0xFFFF, 0xFFFF};
    mx[0] = mx[1] = (u16x2){0, 0};
    auto fold = [&](const Piece &x) {
        const u16x2 one = {1, 1}, mask = {INFV, INFV};
#pragma unroll
        for (int q = 0; q < 4; q++) {
            mn[q / 2] = min2(mn[q / 2], min2(x.ev[q], x.od[q]));
            mx[q / 2] = __builtin_elementwise_max(mx[q / 2], __builtin_elementwise_max((u16x2)((x.ev[q] + one) & mask),
                                                                                      (u16x2)((x.od[q] + one) & mask)));
        }
    };
    const int64_t g0 = t >> 3;
    auto piece = [&](int64_t sweep) { return (piece_bytes *)(glob(N) + sweep * group8 + at); };
    u32x4 keep[NCH > 0 ? NCH : 1];
    if constexpr (NCH > 0) {
#pragma unroll
        for (int k = 0; k < NCH; k++) {
            const int64_t g = g0 + (int64_t)k * GSTEP;
            keep[k] = (u32x4){0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
            if (g < groups) keep[k] = *piece((int64_t)k * GSTEP);
        }
#pragma unroll
        for (int k = 0; k < NCH; k++) {
            fold(split(keep[k]));
            __builtin_amdgcn_sched_barrier(0);  // else many are split at once and their registers spill
        }
    } else {
        for (int64_t g = g0; g < groups; g += GSTEP) {
            if constexpr (FIRST)
                fold(first(g));
            else
                fold(split(*piece(g - g0)));
        }
    }
#pragma unroll
    for (int r = 0; r < 2; r++) {
        uint32_t m = min((uint32_t)mn[r].x, (uint32_t)mn[r].y), top1 = max((uint32_t)mx[r].x, (uint32_t)mx[r].y);
        for (int off = 8; off < 64; off <<= 1) {
            m = min(m, (uint32_t)__shfl_xor((int)m, off, 64));
            top1 = max(top1, (uint32_t)__shfl_xor((int)top1, off, 64));
        }
        if (lane < 8) {
            least[w][2 * pr + r] = m;
            most[w][2 * pr + r] = top1;
        }
    }
    __syncthreads();
    uint32_t m[2];
    u16 base_of[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        m[r] = least[0][2 * pr + r];
        for (int k = 1; k < W; k++) m[r] = min(m[r], least[k][2 * pr + r]);
        // v = x - m (infinity apart) as the level byte 93 - 3 v
        base_of[r] = (u16)(LV_BIAS / 2 + LV_STEP / 2 * m[r]);
    }
    uint64_t h[2] = {0, 0};
    auto finish = [&](const Piece &x, int64_t g) {
        constexpr u16 mul = (u16)(0u - LV_STEP / 2);
        uint32_t o[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const u16 b = base_of[q / 2];
            auto image = [&](u16x2 v) {
                const u16x2 e = v * (u16x2){mul, mul} + (u16x2){b, b};
                if constexpr (FIRST) {
                    return (u16x2){(u16)(v.x == INFV ? 0 : e.x & 0xFF), (u16)(v.y == INFV ? 0 : e.y & 0xFF)};
                } else {
                    // all ones where v is 255: only there v + 1 carries into bit 8
                    const u16x2 inf = (u16x2){0, 0} - (u16x2)((v + (u16x2){1, 1}) >> (u16x2){8, 8});
                    return (u16x2)(e & ~inf & (u16x2){0xFF, 0xFF});
                }
            };
            o[q] = as_u32(image(x.ev[q])) | as_u32(image(x.od[q])) << 8;
            if (i + q / 2 >= n) o[q] = 0;  // rows past n: infinite, as two powers are compared with them
        }
        const uint32_t k = ((uint32_t)g + 1u) * 0x9E3779B1u;
        h[0] += (uint64_t)(o[0] + k) * (o[1] + (k ^ 0x85EBCA6Bu));
        h[1] += (uint64_t)(o[2] + k) * (o[3] + (k ^ 0x85EBCA6Bu));
        *piece(g - g0) = (u32x4){o[0], o[1], o[2], o[3]};
    };
    if constexpr (NCH > 0) {
#pragma unroll
        for (int k = 0; k < NCH; k++) {
            const int64_t g = g0 + (int64_t)k * GSTEP;
            asm volatile("" : "+v"(keep[k]));  // split again rather than kept split, in twice the registers
            if (g < groups) finish(split(keep[k]), g);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        for (int64_t g = g0; g < groups; g += GSTEP) {
            if constexpr (FIRST)
                finish(first(g), g);
            else
                finish(split(*piece(g - g0)), g);
        }
    }
#pragma unroll
    for (int r = 0; r < 2; r++) {
        for (int off = 8; off < 64; off <<= 1) h[r] += __shfl_xor(h[r], off, 64);
        if (lane < 8) hash[w][2 * pr + r] = h[r];
    }
    __syncthreads();
    RowPart x{0, 0, 0, ROW_NONE, ROW_NONE};
    int refuse = 0;
    if (w == 0) {  // lane t: row i0 + t
        const int64_t row = i0 + lane;
        uint32_t v = 0;
        if (lane < GROWS && row < n) {
            uint32_t mr = least[0][lane], top1 = most[0][lane];
            uint64_t hr = hash[0][lane];
            for (int k = 1; k < W; k++) {
                mr = min(mr, least[k][lane]);
                top1 = max(top1, most[k][lane]);
                hr += hash[k][lane];
            }
            if (mr == INFV) mr = 0xFFFFu;
            x = period_row(row, mr, diag[lane], hr, R_in, R_out);
            v = top1 ? top1 - 1 - mr : 0;  // the row's largest canonical value
            refuse = (FIRST && top1 > FMAX16 + 1u ? 1 : 0) | (v > LV_MAX ? 2 : 0);
        }
        for (int off = GROWS / 2; off > 0; off >>= 1) {
            x.hash += __shfl_xor(x.hash, off, 64);
            x.offsets += __shfl_xor(x.offsets, off, 64);
            x.keys += __shfl_xor(x.keys, off, 64);
            x.least = min(x.least, (int64_t)__shfl_xor((long long)x.least, off, 64));
            x.trace = min(x.trace, (int64_t)__shfl_xor((long long)x.trace, off, 64));
            v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
        }
        refuse = (__any(refuse & 1) ? 1 : 0) | (__any(refuse & 2) ? 2 : 0);
        v = min(v, LV_MAX);
        // read by the next step, a later kernel; few blocks raise it
        if (lane == 0 && (int)v > __hip_atomic_load(big, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(big, (int)v);
    }
    period_fold(x, refuse, acc, nslots, st, wide, rec, seq, &last);
}

mpr_status period_rows8_launch(const u16 *first, int64_t lda, uint8_t *N, int64_t n, const int64_t *R_in,
                               int64_t *R_out, void *acc, int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                               int64_t seq, hipStream_t s)
{
    if (n > INT32_MAX) return MPR_EUNSUPPORTED;
    const dim3 grid((unsigned)((n + GROWS - 1) / GROWS));
    const int64_t group8 = level_group8(n), groups = (n + 7) / 8;
#define ROWS8(T, NCH, FIRST)                                                                                           \
    hipLaunchKernelGGL((period_rows8_kernel<T, NCH, FIRST>), grid, dim3(T), 0, s, first, lda, N, group8, n, R_in, R_out, \
                       (PeriodAcc *)acc, period_slots(n), st, wide, big, rec, seq)
    // the forms keep a row's groups in registers (m = 9: 1024 threads spilled,
    // 301 us; 512 with twice the groups each do not, 246)
    if (first)
        ROWS8(512, 0, true);
    else if (groups <= 2 * 64)
        ROWS8(512, 2, false);
    else if (groups <= 4 * 128)
        ROWS8(1024, 4, false);
    else if (groups <= 16 * 64)
        ROWS8(512, 16, false);
    else if (groups <= 44 * 64)
        ROWS8(512, 44, false);
    else
        ROWS8(1024, 0, false);
#undef ROWS8
    return check_launch();
}

// A whole power of up to SMALL_N states, step and pass, by one workgroup: the
// power before (bytes) and A in LDS, a half wave to a row and a lane to two
// columns, sums in 16 bits (no value passes 30 + FMAX), nothing left to
// atomics.  Two kernels whose blocks meet in an accumulator are latency alone
// at this size (n = 33: 4.5 + 8.8 us a power, now 6.7).
constexpr int SMALL_N = PERIOD_SMALL_N, SMALL_T = 1024;
__global__ __launch_bounds__(SMALL_T) void period_small_kernel(const u16 *A, int64_t lda, const uint8_t *N, uint8_t *O,
                                                               int ld8, int n, const int64_t *R_in, int64_t *R_out,
                                                               int64_t *rec, int64_t seq)
{
    constexpr int HP = SMALL_N / 2;  // lanes of a row: column pairs
    static_assert(HP == 32, "a half wave to a row");
    __shared__ uint32_t a[SMALL_N][HP + 1];
    __shared__ u16 l[SMALL_N][SMALL_N + 2];
    __shared__ RowPart part[SMALL_N];
    __shared__ int refused;
    const int t = (int)threadIdx.x, lane = t & 63, half = t / HP, p = t % HP;
    if (t == 0) refused = 0;
    if (t < SMALL_N) part[t] = RowPart{0, 0, 0, ROW_NONE, ROW_NONE};
    for (int e = t; e < SMALL_N * HP; e += SMALL_T) {
        const int i = e / HP, c = e % HP * 2;
        const gu16 *row = glob(A) + (int64_t)i * lda;
        const uint32_t lo = i < n && c < n ? row[c] : 0xFFFFu, hi = i < n && c + 1 < n ? row[c + 1] : 0xFFFFu;
        a[i][c / 2] = lo | hi << 16;
    }
    if (N) {
        for (int e = t; e < n * n; e += SMALL_T) {
            const int i = e / n, c = e - i * n;
            const uint32_t b = glob(N)[i * ld8 + c];
            l[i][c] = b ? (u16)((LV_BIAS / 2 - b) * 86 >> 8) : INF16;  // v <= 30: 86 / 256 is 1 / 3 there
        }
    }
    __syncthreads();
    for (int i = half; i < n; i += SMALL_T / HP) {  // uniform in a half wave
        u16x2 v = as_u16x2(a[i][p]);
        if (N) {
            v = (u16x2){0xFFFF, 0xFFFF};
#pragma unroll 8
            for (int k = 0; k < n; k++) v = min2(v, add_sat((u16x2){l[i][k], l[i][k]}, as_u16x2(a[k][p])));
        }
        const int c = 2 * p;
        uint32_t m = min((uint32_t)v.x, (uint32_t)v.y);
        // largest finite value + 1, or 0
        uint32_t top1 = max(v.x == 0xFFFF ? 0u : v.x + 1u, v.y == 0xFFFF ? 0u : v.y + 1u);
        for (int off = HP / 2; off > 0; off >>= 1) {
            m = min(m, (uint32_t)__shfl_xor((int)m, off, 64));
            top1 = max(top1, (uint32_t)__shfl_xor((int)top1, off, 64));
        }
        auto image = [&](uint32_t x) { return x == 0xFFFFu ? 0u : (LV_BIAS / 2 - LV_STEP / 2 * (x - m)) & 0xFFu; };
        const uint32_t x = image(v.x) | image(v.y) << 8;
        uint64_t h = mix64((uint64_t)(p + 1) << 32 | x);
        for (int off = HP / 2; off > 0; off >>= 1) h += __shfl_xor(h, off, 64);
        const uint32_t pair = (uint32_t)__shfl((int)as_u32(v), (lane & HP) + i / 2, 64);
        if (c < ld8) *(__attribute__((address_space(1))) u16 *)(glob(O) + i * ld8 + c) = (u16)x;  // ld8 is even
        if (p == 0) {
            part[i] = period_row(i, m, i & 1 ? pair >> 16 : pair & 0xFFFFu, h, R_in, R_out);
            const int r = (!N && top1 > FMAX16 + 1u ? 1 : 0) | (top1 && top1 - 1 - m > LV_MAX ? 2 : 0);
            if (r) atomicOr(&refused, r);
        }
    }
    __syncthreads();
    if (t >= 64) return;
    const RowPart x = part[lane];
    const uint64_t hs = wave_sum_u64(x.hash), os = wave_sum_u64(x.offsets), ks = wave_sum_u64(x.keys);
    const int64_t lo = wave_min_i64(x.least), tr = wave_min_i64(x.trace);
    if (lane != 0) return;
    rec[0] = (int64_t)mix64(hs + mix64(os - (lo == ROW_NONE ? 0 : (uint64_t)lo * ks)));
    rec[1] = tr;
    rec[2] = refused & 1 ? MPR_EOVERFLOW : MPR_OK;
    rec[3] = refused >> 1;
    __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

mpr_status period_small_launch(const u16 *A, int64_t lda, const uint8_t *N, uint8_t *O, int64_t ld8, int64_t n,
                               const int64_t *R_in, int64_t *R_out, int64_t *rec, int64_t seq, hipStream_t s)
{
    if (n > SMALL_N || ld8 > SMALL_N) return MPR_EUNSUPPORTED;
    hipLaunchKernelGGL(period_small_kernel, dim3(1), dim3(SMALL_T), 0, s, A, lda, N, O, (int)ld8, (int)n, R_in, R_out, rec,
                       seq);
    return check_launch();
}

mpr_status period_clear_launch(void *acc, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(period_clear_kernel, dim3(1), dim3(64), 0, s, (PeriodAcc *)acc, period_slots(n));
    return check_launch();
}

mpr_status period_rows_launch(const u16 *src, int64_t lds_, u16 *dst, int64_t ldd, int64_t n, const int64_t *R_in,
                              int64_t *R_out, bool raw, void *acc, int32_t *st, int64_t *rec, int64_t seq, hipStream_t s)
{
    if (n > INT32_MAX) return MPR_EUNSUPPORTED;
    auto kernel = n <= RT * 8       ? period_rows_kernel<1>
                  : n <= 4 * RT * 8 ? period_rows_kernel<4>
                  : n <= 12 * RT * 8 ? period_rows_kernel<12>
                                     : period_rows_kernel<0>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(RT), 0, s, src, lds_, dst, ldd, n, R_in, R_out, raw ? 1 : 0,
                       (PeriodAcc *)acc, period_slots(n), st, rec, seq);
    return check_launch();
}

}  // namespace mpr
