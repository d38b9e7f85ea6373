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
// to read n words each (m = 8: 68 + 13 + 9 us, now ROWS8; m = 9: 410 + 51 +
// 24 us, now ROWS9; m = 3: 6.0 + 3.4 + 3.3 us and a copy to the host, now
// ROWS3).
#include "level.h"

namespace mpr {

constexpr int PSLOTS = 32;
constexpr int RT = 256;  // threads per row

struct PeriodSlot {
    uint64_t hash, offsets, keys;  // sums over the rows
    int64_t least, trace;          // minima over the rows
    uint32_t done, pad[5];         // rows folded in
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

// The row's part in its power, by every thread of its block (m: least value,
// diag: diagonal value, h: hash of its entries, refuse: out of range; of
// thread 0).  wide: a second status word for the record, or null.
__device__ __forceinline__ void period_fold(int64_t i, uint32_t m, uint32_t diag, uint64_t h, int refuse,
                                            const int64_t *R_in, int64_t *R_out, PeriodAcc *acc, int32_t *st,
                                            int32_t *wide, int64_t *rec, int64_t seq, int *last)
{
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    if (threadIdx.x == 0) {
        const int64_t rin = R_in ? R_in[i] : 0;
        const bool none = m == 0xFFFFu || rin == ROW_NONE;
        const int64_t R = none ? ROW_NONE : rin + (int64_t)m;
        R_out[i] = R;
        const uint64_t rh = mix64(h ^ mix64((uint64_t)i ^ 0x6A09E667F3BCC909ull));
        const uint64_t key = mix64((uint64_t)i ^ 0xBB67AE8584CAA73Bull);
        PeriodSlot *s = &acc->slot[blockIdx.x % PSLOTS];
        // every fold completes (its old value arrives) before the row counts
        uint64_t seen = agent_add(&s->hash, none ? rh + 1 : rh);
        if (!none) {
            seen |= agent_add(&s->offsets, key * (uint64_t)R) | agent_add(&s->keys, key);
            seen |= (uint64_t)agent_min(&s->least, R);
            if (diag != 0xFFFFu) seen |= (uint64_t)agent_min(&s->trace, R + (int64_t)(diag - m));
        }
        if (refuse & 1)
            seen |= (uint64_t)__hip_atomic_exchange(st, MPR_EOVERFLOW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (refuse & 2) seen |= (uint64_t)__hip_atomic_exchange(wide, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" : : "v"(seen) : "memory");
        const uint32_t rows = ((uint32_t)gridDim.x + PSLOTS - 1 - blockIdx.x % PSLOTS) / PSLOTS;  // of this slot
        const uint32_t slots = min((uint32_t)gridDim.x, (uint32_t)PSLOTS);
        *last = 0;
        if (agent_add(&s->done, 1u) + 1 == rows) *last = agent_add(&acc->full, 1u) + 1 == slots;
    }
    __syncthreads();
    if (!*last || w != 0) return;
    // The last row of the power: one lane per slot (reads at the place where
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
    period_fold(i, m, diag, hsum[0] + hsum[1] + hsum[2] + hsum[3], refuse, R_in, R_out, acc, st, nullptr, rec, seq, &last);
}

// The same in bytes (level bytes, sparse.hip): 16 columns per thread and
// chunk.  FIRST: the source is the u16 matrix X.  *big receives the largest
// canonical value of the power, for the step that reads it.
template <int NCH, bool FIRST>
__global__ __launch_bounds__(RT) void period_rows8_kernel(const u16 *X, int64_t ldx, uint8_t *N, int64_t ld8, int64_t n,
                                                          const int64_t *R_in, int64_t *R_out, PeriodAcc *acc,
                                                          int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                                                          int64_t seq)
{
    __shared__ uint32_t least[RT / 64], most[RT / 64];
    __shared__ uint64_t hsum[RT / 64];
    __shared__ uint32_t diag;
    __shared__ int last, refuse;
    constexpr u16 INFV = FIRST ? 0xFFFF : 0xFF;
    constexpr int Q = NCH > 0 ? NCH : 1;
    const int64_t i = blockIdx.x;
    const gu16 *xrow = glob(X) + (FIRST ? i * ldx : 0);
    __attribute__((address_space(1))) uint8_t *row = glob(N) + i * ld8;
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    // values 0, 2 / 4, 6 / .. and 1, 3 / 5, 7 / .. of 16 columns from c
    auto load = [&](int64_t c, u16x2 ev[4], u16x2 od[4]) {
        if constexpr (FIRST) {
            const uint4 a = row8(xrow, c, n), b = c + 8 < n ? row8(xrow, c + 8, n)
                                                            : make_uint4(0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu);
            const uint32_t d[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int q = 0; q < 4; q++) {
                ev[q] = as_u16x2(__builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x05040100u));
                od[q] = as_u16x2(__builtin_amdgcn_perm(d[2 * q + 1], d[2 * q], 0x07060302u));
            }
        } else {
            const u32x4 v = *(const __attribute__((address_space(1))) u32x4 *)(row + c);
            const uint32_t d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; q++) {
                ev[q] = as_u16x2(d[q] & 0x00FF00FFu);
                od[q] = as_u16x2(d[q] >> 8 & 0x00FF00FFu);
            }
        }
    };
    u16x2 ke[Q][4], ko[Q][4];
    u16x2 mn = {0xFFFF, 0xFFFF};
    bool over = false;
    const int64_t c0 = (int64_t)threadIdx.x * 16;
    auto fold = [&](const u16x2 ev[4], const u16x2 od[4]) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            mn = min2(mn, min2(ev[q], od[q]));
            if (FIRST) {
                const uint32_t x[4] = {ev[q].x, ev[q].y, od[q].x, od[q].y};
#pragma unroll
                for (int e = 0; e < 4; e++) over |= x[e] > FMAX16 && x[e] != 0xFFFFu;
            }
        }
    };
    if constexpr (NCH > 0) {
#pragma unroll
        for (int k = 0; k < NCH; k++) {
            const int64_t c = c0 + (int64_t)k * RT * 16;
            if (c < n) {
                load(c, ke[k], ko[k]);
                fold(ke[k], ko[k]);
            }
        }
    } else {
        for (int64_t c = c0; c < n; c += RT * 16) {
            load(c, ke[0], ko[0]);
            fold(ke[0], ko[0]);
        }
    }
    uint32_t m = wave_min_u32(min((uint32_t)mn.x, (uint32_t)mn.y));
    if (lane == 0) least[w] = m;
    if (threadIdx.x == 0) {
        diag = FIRST ? (uint32_t)xrow[i] : (uint32_t)row[i];  // before the row is rewritten
        if (diag == INFV) diag = 0xFFFFu;
        refuse = 0;
    }
    __syncthreads();
    m = min(min(least[0], least[1]), min(least[2], least[3]));
    if (m == INFV) m = 0xFFFFu;
    // 186 - 6 (x - m), a level byte when x - m <= 30
    const u16 top = (u16)(LV_BIAS + LV_STEP * m);
    uint64_t h = 0;
    u16x2 small = {0xFFFF, 0xFFFF};  // least nonzero image: the largest value
    bool far = false;
    auto image = [&](u16x2 x) {
        const u16x2 e = x * (u16x2){(u16)(0u - LV_STEP), (u16)(0u - LV_STEP)} + (u16x2){top, top};
        const bool fx = x.x != INFV, fy = x.y != INFV;
        far |= (fx && (uint32_t)x.x - m > LV_MAX) || (fy && (uint32_t)x.y - m > LV_MAX);
        small = min2(small, (u16x2){fx ? e.x : (u16)0xFFFF, fy ? e.y : (u16)0xFFFF});
        return (u16x2){(u16)(fx ? e.x & 0xFF : 0), (u16)(fy ? e.y & 0xFF : 0)};
    };
    auto finish = [&](const u16x2 ev[4], const u16x2 od[4], int64_t c) {
        uint32_t x[4];
#pragma unroll
        for (int q = 0; q < 4; q++) x[q] = as_u32(image(ev[q])) | as_u32(image(od[q])) << 8;
        h += nh4(x, (uint32_t)(c >> 4));
        *(__attribute__((address_space(1))) u32x4 *)(row + c) = (u32x4){x[0], x[1], x[2], x[3]};
    };
    if constexpr (NCH > 0) {
#pragma unroll
        for (int k = 0; k < NCH; k++) {
            const int64_t c = c0 + (int64_t)k * RT * 16;
            if (c < n) finish(ke[k], ko[k], c);
        }
    } else {
        for (int64_t c = c0; c < n; c += RT * 16) {
            load(c, ke[0], ko[0]);
            finish(ke[0], ko[0], c);
        }
    }
    if (over) atomicOr(&refuse, 1);
    if (far) atomicOr(&refuse, 2);
    h = wave_sum_u64(h);
    const uint32_t lo = wave_min_u32(min((uint32_t)small.x, (uint32_t)small.y));
    if (lane == 0) {
        hsum[w] = h;
        most[w] = lo;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t e = min(min(most[0], most[1]), min(most[2], most[3]));
        // read by the next step, a later kernel; few rows raise it
        const int32_t v = e <= LV_BIAS ? (int32_t)((LV_BIAS - e) / LV_STEP) : 0;
        if (v > __hip_atomic_load(big, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(big, v);
    }
    period_fold(i, m, diag, hsum[0] + hsum[1] + hsum[2] + hsum[3], refuse, R_in, R_out, acc, st, wide, rec, seq, &last);
}

mpr_status period_rows8_launch(const u16 *first, int64_t lda, uint8_t *N, int64_t ld8, int64_t n, const int64_t *R_in,
                               int64_t *R_out, void *acc, int32_t *st, int32_t *wide, int32_t *big, int64_t *rec,
                               int64_t seq, hipStream_t s)
{
    if (n > INT32_MAX) return MPR_EUNSUPPORTED;
    auto kernel = first             ? period_rows8_kernel<0, true>
                  : n <= RT * 16     ? period_rows8_kernel<1, false>
                  : n <= 2 * RT * 16 ? period_rows8_kernel<2, false>
                  : n <= 6 * RT * 16 ? period_rows8_kernel<6, false>
                                     : period_rows8_kernel<0, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)n), dim3(RT), 0, s, first, lda, N, ld8, n, R_in, R_out, (PeriodAcc *)acc,
                       st, wide, big, rec, seq);
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
