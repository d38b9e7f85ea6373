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
    if (threadIdx.x == 0) {
        const int64_t rin = R_in ? R_in[i] : 0;
        const bool none = empty || rin == ROW_NONE;
        const int64_t R = none ? ROW_NONE : rin + (int64_t)m;
        R_out[i] = R;
        const uint64_t rh = mix64((hsum[0] + hsum[1] + hsum[2] + hsum[3]) ^ mix64((uint64_t)i ^ 0x6A09E667F3BCC909ull));
        const uint64_t key = mix64((uint64_t)i ^ 0xBB67AE8584CAA73Bull);
        PeriodSlot *s = &acc->slot[blockIdx.x % PSLOTS];
        // every fold completes (its old value arrives) before the row counts
        uint64_t seen = agent_add(&s->hash, none ? rh + 1 : rh);
        if (!none) {
            seen |= agent_add(&s->offsets, key * (uint64_t)R) | agent_add(&s->keys, key);
            seen |= (uint64_t)agent_min(&s->least, R);
            if (diag != 0xFFFFu) seen |= (uint64_t)agent_min(&s->trace, R + (int64_t)(diag - m));
        }
        if (refuse)
            seen |= (uint64_t)__hip_atomic_exchange(st, MPR_EOVERFLOW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" : : "v"(seen) : "memory");
        const uint32_t rows = ((uint32_t)gridDim.x + PSLOTS - 1 - blockIdx.x % PSLOTS) / PSLOTS;  // of this slot
        const uint32_t slots = min((uint32_t)gridDim.x, (uint32_t)PSLOTS);
        last = 0;
        if (agent_add(&s->done, 1u) + 1 == rows) last = agent_add(&acc->full, 1u) + 1 == slots;
    }
    __syncthreads();
    if (!last || w != 0) return;
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
    __hip_atomic_store(&rec[7], seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
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
