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
// taken off at the end.  Each block folds its row into one of PSLOTS records
// and the last block combines them, where two more kernels of one block used
// to read n words each (m = 8: 68 + 13 + 9 us, in bytes 31; m = 9: 410 + 51 +
// 24 us, in bytes 280; m = 3: 6.0 + 3.4 + 3.3 us and a copy to the host, now
// within the 6.7 us of a whole power).
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
    PeriodSlot slot[PSLOTS];
    uint32_t full, pad[15];  // slots complete
};
size_t period_acc_bytes() { return sizeof(PeriodAcc); }

__device__ __forceinline__ void period_clear(PeriodAcc *a, int t)
{
    if (t < PSLOTS) {
        PeriodSlot z{};
        z.least = z.trace = ROW_NONE;
        a->slot[t] = z;
    }
    if (t == 0) a->full = 0;
}
__global__ void period_clear_kernel(PeriodAcc *a) { period_clear(a, (int)threadIdx.x); }

template <class X>
__device__ __forceinline__ X agent_add(X *p, X v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int64_t agent_min(int64_t *p, int64_t v)
{
    return __hip_atomic_fetch_min(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

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
__device__ __forceinline__ void period_fold(const RowPart &x, int refuse, PeriodAcc *acc, int32_t *st, int32_t *wide,
                                            int64_t *rec, int64_t seq, int *last)
{
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    if (threadIdx.x == 0) {
        PeriodSlot *s = &acc->slot[blockIdx.x % PSLOTS];
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
        const uint32_t blocks = ((uint32_t)gridDim.x + PSLOTS - 1 - blockIdx.x % PSLOTS) / PSLOTS;  // of this slot
        const uint32_t slots = min((uint32_t)gridDim.x, (uint32_t)PSLOTS);
        *last = 0;
        if (agent_add(&s->done, 1u) + 1 == blocks) *last = agent_add(&acc->full, 1u) + 1 == slots;
    }
    __syncthreads();
    if (!*last || w != 0) return;
    // The last block of the power: one lane per slot (reads at the place where
    // the folds happened), then the record and a clear accumulator.
    PeriodSlot *s = &acc->slot[lane % PSLOTS];
    uint64_t hs = lane < PSLOTS ? agent_add(&s->hash, (uint64_t)0) : 0;
    uint64_t os = lane < PSLOTS ? agent_add(&s->offsets, (uint64_t)0) : 0;
    uint64_t ks = lane < PSLOTS ? agent_add(&s->keys, (uint64_t)0) : 0;
    const int64_t lo = wave_min_i64(agent_min(&s->least, ROW_NONE));
    const int64_t tr = wave_min_i64(agent_min(&s->trace, ROW_NONE));
    hs = wave_sum_u64(hs);
    os = wave_sum_u64(os);
    ks = wave_sum_u64(ks);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    period_clear(acc, lane);
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
                                                         int32_t *st, int64_t *rec, int64_t seq)
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
    period_fold(x, refuse, acc, st, nullptr, rec, seq, &last);
}

// The same in bytes (level bytes, sparse.hip), a wave per row: lane t takes
// the 16 columns at 16 t, 16 t + 1024, ..., NCH of them in registers (0: the
// row is read twice).  FIRST: the source is the u16 matrix X.  *big receives
// the largest canonical value, for the step that reads it.  Four rows share
// one fold: with one each, the atomics bound the pass (m = 9: 300 us).
template <int NCH, bool FIRST>
__global__ __launch_bounds__(RT) void period_rows8_kernel(const u16 *X, int64_t ldx, uint8_t *N, int64_t ld8, int64_t n,
                                                          const int64_t *R_in, int64_t *R_out, PeriodAcc *acc,
                                                          int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                                                          int64_t seq)
{
    __shared__ RowPart part[RT / 64];
    __shared__ int refused[RT / 64], most[RT / 64];
    __shared__ int last;
    constexpr u16 INFV = FIRST ? 0xFFFF : 0xFF;
    constexpr int W = FIRST ? 8 : 4;  // dwords of 16 columns
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    const int64_t i = (int64_t)blockIdx.x * (RT / 64) + w;
    if (lane == 0) {
        part[w] = RowPart{0, 0, 0, ROW_NONE, ROW_NONE};
        refused[w] = most[w] = 0;
    }
    if (i < n) {  // wave-uniform
        const gu16 *xrow = glob(X) + (FIRST ? i * ldx : 0);
        __attribute__((address_space(1))) uint8_t *row = glob(N) + i * ld8;
        auto load = [&](int64_t c, uint32_t d[W]) {
            if constexpr (FIRST) {
                const uint4 inf = make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
                const uint4 a = row8(xrow, c, n), b = c + 8 < n ? row8(xrow, c + 8, n) : inf;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    d[q] = comp(a, q);
                    d[4 + q] = comp(b, q);
                }
            } else {
                const u32x4 v = *(const __attribute__((address_space(1))) u32x4 *)(row + c);
                d[0] = v.x;
                d[1] = v.y;
                d[2] = v.z;
                d[3] = v.w;
            }
        };
        // values 4q, 4q + 2 and 4q + 1, 4q + 3 of 16 columns
        auto split = [&](const uint32_t d[W], int q, u16x2 &ev, u16x2 &od) {
            if constexpr (FIRST) {
                ev = as_u16x2(__builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x05040100u));
                od = as_u16x2(__builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x07060302u));
            } else {
                ev = as_u16x2(d[q] & 0x00FF00FFu);
                od = as_u16x2(d[q] >> 8 & 0x00FF00FFu);
            }
        };
        uint32_t keep[NCH > 0 ? NCH : 1][W];
        u16x2 mn = {0xFFFF, 0xFFFF}, mx = {0, 0};  // mx: largest finite value + 1 (infinity + 1 is 0)
        auto fold = [&](const uint32_t d[W]) {
            const u16x2 one = {1, 1}, mask = {INFV, INFV};
#pragma unroll
            for (int q = 0; q < 4; q++) {
                u16x2 ev, od;
                split(d, q, ev, od);
                mn = min2(mn, min2(ev, od));
                mx = __builtin_elementwise_max(mx, __builtin_elementwise_max((u16x2)((ev + one) & mask),
                                                                             (u16x2)((od + one) & mask)));
            }
        };
        const int64_t c0 = (int64_t)lane * 16;
        if constexpr (NCH > 0) {
#pragma unroll
            for (int k = 0; k < NCH; k++) {
                const int64_t c = c0 + (int64_t)k * 1024;
#pragma unroll
                for (int q = 0; q < W; q++) keep[k][q] = 0xFFFFFFFFu;
                if (c < n) load(c, keep[k]);
            }
#pragma unroll
            for (int k = 0; k < NCH; k++) fold(keep[k]);
        } else {
            for (int64_t c = c0; c < n; c += 1024) {
                load(c, keep[0]);
                fold(keep[0]);
            }
        }
        uint32_t diag = FIRST ? (uint32_t)xrow[i] : (uint32_t)row[i];
        if (diag == INFV) diag = 0xFFFFu;
        uint32_t m = wave_min_u32(min((uint32_t)mn.x, (uint32_t)mn.y));
        const uint32_t top1 = ~wave_min_u32(~max((uint32_t)mx.x, (uint32_t)mx.y));  // largest finite value + 1, or 0
        if (m == INFV) m = 0xFFFFu;
        // v = x - m (infinity apart) as the level byte 186 - 6 v
        const u16 base = (u16)(LV_BIAS + LV_STEP * m), mul = (u16)(0u - LV_STEP);
        uint64_t h = 0;
        auto image = [&](u16x2 x) {
            const u16x2 e = x * (u16x2){mul, mul} + (u16x2){base, base};
            if constexpr (FIRST) {
                return (u16x2){(u16)(x.x == INFV ? 0 : e.x & 0xFF), (u16)(x.y == INFV ? 0 : e.y & 0xFF)};
            } else {
                // all ones where x is 255: only there x + 1 carries into bit 8
                const u16x2 inf = (u16x2){0, 0} - (u16x2)((x + (u16x2){1, 1}) >> (u16x2){8, 8});
                return (u16x2)(e & ~inf & (u16x2){0xFF, 0xFF});
            }
        };
        auto finish = [&](const uint32_t d[W], int64_t c) {
            uint32_t x[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                u16x2 ev, od;
                split(d, q, ev, od);
                x[q] = as_u32(image(ev)) | as_u32(image(od)) << 8;
            }
            h += nh4(x, (uint32_t)(c >> 4));
            *(__attribute__((address_space(1))) u32x4 *)(row + c) = (u32x4){x[0], x[1], x[2], x[3]};
        };
        if constexpr (NCH > 0) {
#pragma unroll
            for (int k = 0; k < NCH; k++) {
                const int64_t c = c0 + (int64_t)k * 1024;
                if (c < n) finish(keep[k], c);
            }
        } else {
            for (int64_t c = c0; c < n; c += 1024) {
                load(c, keep[0]);
                finish(keep[0], c);
            }
        }
        h = wave_sum_u64(h);
        if (lane == 0) {
            part[w] = period_row(i, m, diag, h, R_in, R_out);
            const uint32_t v = top1 ? top1 - 1 - m : 0;  // the row's largest canonical value
            refused[w] = (FIRST && top1 > FMAX16 + 1u ? 1 : 0) | (v > LV_MAX ? 2 : 0);
            most[w] = (int)min(v, (uint32_t)LV_MAX);
        }
    }
    __syncthreads();
    RowPart x{0, 0, 0, ROW_NONE, ROW_NONE};
    int refuse = 0;
    if (threadIdx.x == 0) {
        int v = 0;
        for (int k = 0; k < RT / 64; k++) {
            x.hash += part[k].hash;
            x.offsets += part[k].offsets;
            x.keys += part[k].keys;
            x.least = min(x.least, part[k].least);
            x.trace = min(x.trace, part[k].trace);
            refuse |= refused[k];
            v = max(v, most[k]);
        }
        // read by the next step, a later kernel; few blocks raise it
        if (v > __hip_atomic_load(big, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(big, v);
    }
    period_fold(x, refuse, acc, st, wide, rec, seq, &last);
}

mpr_status period_rows8_launch(const u16 *first, int64_t lda, uint8_t *N, int64_t ld8, int64_t n, const int64_t *R_in,
                               int64_t *R_out, void *acc, int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                               int64_t seq, hipStream_t s)
{
    if (n > INT32_MAX) return MPR_EUNSUPPORTED;
    auto kernel = first          ? period_rows8_kernel<0, true>
                  : n <= 1024     ? period_rows8_kernel<1, false>
                  : n <= 8 * 1024 ? period_rows8_kernel<8, false>
                  : n <= 24 * 1024 ? period_rows8_kernel<24, false>
                                   : period_rows8_kernel<0, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((n + 3) / 4)), dim3(RT), 0, s, first, lda, N, ld8, n, R_in, R_out, (PeriodAcc *)acc,
                       st, wide, big, rec, seq);
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
            l[i][c] = b ? (u16)((LV_BIAS - b) * 43 >> 8) : INF16;  // v <= 30: 43 / 256 is 1 / 6 there
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
        auto image = [&](uint32_t x) { return x == 0xFFFFu ? 0u : (LV_BIAS - LV_STEP * (x - m)) & 0xFFu; };
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

mpr_status period_clear_launch(void *acc, hipStream_t s)
{
    hipLaunchKernelGGL(period_clear_kernel, dim3(1), dim3(64), 0, s, (PeriodAcc *)acc);
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
                       (PeriodAcc *)acc, st, rec, seq);
    return check_launch();
}

}  // namespace mpr
