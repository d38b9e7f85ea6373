// transfer.hip -- the transfer matrix A(G) of Corollary 7 built on the GPU.
//
// States are the correct words of Definition 4 (no ad, da, ab, ba, bb as
// vertical neighbours) in increasing base-4 order, row 1 the most
// significant letter, a=0 b=1 c=2 d=3.  Instead of enumerating all 4^m
// words, each lane unranks its own words with a table of suffix counts:
// S[len][x] = number of correct words of length len that start with x.
// Entry (q, p) is 2 p(a) + p(b) when p can follow q (the rule lists of
// Section 4.1, with the intermediate-row "p_1 = d" read as p_i = d), else
// infinity.
#include <string.h>

#include "common.h"

namespace mpr {

constexpr int MAXM = 12;

struct WordTable {
    int m;
    int64_t S[MAXM + 1][4];  // S[len][first letter]
};

// May letter y sit directly below letter x in a column?
__host__ __device__ __forceinline__ bool adjacent_ok(int x, int y)
{
    // forbidden vertical pairs: ad, da, ab, ba, bb  (bit 4*x + y)
    constexpr uint32_t bad = (1u << (0 * 4 + 3)) | (1u << (3 * 4 + 0)) | (1u << (0 * 4 + 1)) | (1u << (1 * 4 + 0)) |
                             (1u << (1 * 4 + 1));
    return !((bad >> (4 * x + y)) & 1u);
}

static void make_table(int m, WordTable &t)
{
    memset(&t, 0, sizeof(t));
    t.m = m;
    for (int x = 0; x < 4; x++) t.S[1][x] = 1;
    for (int len = 2; len <= m; len++)
        for (int x = 0; x < 4; x++)
            for (int y = 0; y < 4; y++)
                if (adjacent_ok(x, y)) t.S[len][x] += t.S[len - 1][y];
}

static int64_t word_count(const WordTable &t)
{
    int64_t c = 0;
    for (int x = 0; x < 4; x++) c += t.S[t.m][x];
    return c;
}

// Letters of the word of rank r, packed two bits per row, row 0 in bits 0-1.
__host__ __device__ __forceinline__ uint32_t unrank(const WordTable &t, int64_t r)
{
    uint32_t w = 0;
    int prev = -1;
    for (int i = 0; i < t.m; i++) {
        const int len = t.m - i;
        for (int x = 0; x < 4; x++) {
            if (prev >= 0 && !adjacent_ok(prev, x)) continue;
            if (r < t.S[len][x]) {
                w |= (uint32_t)x << (2 * i);
                prev = x;
                break;
            }
            r -= t.S[len][x];
        }
    }
    return w;
}

// Letters allowed for p_i after q_i: always (first mask) or only when a
// vertical neighbour of p_i in the new column is an a (second mask).
//   q_i = a: p_i in {a, c}
//   q_i = b: p_i = d, or p_i = c next to an a
//   q_i = c: p_i in {a, b, d}, or p_i = c next to an a
//   q_i = d: p_i = a
__device__ __constant__ uint8_t kAlways[4] = {(1 << 0) | (1 << 2), (1 << 3), (1 << 0) | (1 << 1) | (1 << 3), (1 << 0)};
__device__ __constant__ uint8_t kWithA[4] = {0, (1 << 2), (1 << 2), 0};

// The rule lists for all rows of a column at once.  blocked(p) has, for each
// letter x of the previous column, the rows i where p_i may not follow
// q_i = x (16 bits a letter); letters(q) has the rows where q_i = x.  p can
// follow q when the two have no bit in common.
__device__ __forceinline__ uint64_t letters(uint32_t w, int m)
{
    uint64_t r = 0;
    for (int i = 0; i < m; i++) r |= (uint64_t)(1u << i) << (16 * ((w >> (2 * i)) & 3u));
    return r;
}
__device__ __forceinline__ uint64_t blocked(uint32_t w, int m)
{
    uint32_t is[4] = {0, 0, 0, 0};
    for (int i = 0; i < m; i++) {
        const uint32_t x = (w >> (2 * i)) & 3u;
#pragma unroll
        for (uint32_t y = 0; y < 4; y++) is[y] |= (x == y ? 1u : 0u) << i;
    }
    const uint32_t near_a = is[0] << 1 | is[0] >> 1, rows = (1u << m) - 1u;
    uint64_t r = 0;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        uint32_t ok = 0;
#pragma unroll
        for (int y = 0; y < 4; y++) {
            if (kAlways[q] >> y & 1u) ok |= is[y];
            if (kWithA[q] >> y & 1u) ok |= is[y] & near_a;
        }
        r |= (uint64_t)(rows & ~ok) << (16 * q);
    }
    return r;
}

// A block writes TROWS rows of TCOLS columns, 8 columns per thread: each word
// of its rows and columns is unranked once, into LDS; an entry is then two
// ANDs and a compare, and the kernel is bound by its writes (one thread per
// entry, unranking both words each time, took 10.2 ms at m = 9 and 1.10 ms at
// m = 8; now 0.24 and 0.06).
constexpr int TROWS = 64, TCOLS = 256 * 8;
__global__ __launch_bounds__(256) void transfer_kernel(WordTable t, int64_t n, u16 *A, int64_t lda, int vec)
{
    __shared__ uint64_t q_letters[TROWS], p_blocked[TCOLS];
    __shared__ uint8_t p_weight[TCOLS];
    const int64_t q0 = (int64_t)blockIdx.y * TROWS, c0 = (int64_t)blockIdx.x * TCOLS;
    const int rows = (int)min<int64_t>(TROWS, n - q0), cols = (int)min<int64_t>(TCOLS, n - c0);
    for (int r = (int)threadIdx.x; r < rows; r += 256) q_letters[r] = letters(unrank(t, q0 + r), t.m);
    for (int c = (int)threadIdx.x; c < cols; c += 256) {
        const uint32_t w = unrank(t, c0 + c);
        uint32_t weight = 0;
        for (int i = 0; i < t.m; i++) {
            const uint32_t x = (w >> (2 * i)) & 3u;
            weight += x == 0 ? 2u : x == 1 ? 1u : 0u;
        }
        p_blocked[c] = blocked(w, t.m);
        p_weight[c] = (uint8_t)weight;
    }
    __syncthreads();
    const int p0 = (int)threadIdx.x * 8;
    if (p0 >= cols) return;
    uint64_t block[8];
    uint32_t weight[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        const int c = p0 + e < cols ? p0 + e : p0;
        block[e] = p_blocked[c];
        weight[e] = p_weight[c];
    }
    gu16 *out = glob(A) + q0 * lda + c0 + p0;
    for (int r = 0; r < rows; r++, out += lda) {
        const uint64_t q = q_letters[r];
        uint32_t v[8];
#pragma unroll
        for (int e = 0; e < 8; e++) v[e] = (q & block[e]) == 0 ? weight[e] : 0xFFFFu;
        if (vec && p0 + 8 <= cols) {
            gstore16(out, make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16));
        } else {
#pragma unroll
            for (int e = 0; e < 8; e++)
                if (p0 + e < cols) out[e] = (u16)v[e];
        }
    }
}

// Border ("loss") matrix of the appendix for a strip of m rows.  Rows
// 1..m-1 follow the rule lists above; the m-th row need not be dominated,
// so after q_m = d everything allowed after q_m = c is allowed.  The arc
// label is 10 p(a) + 5 p(b) - 2 nd(q, p), nd(q, p) = newly dominated
// vertices by Algorithm 3 (per row: (a,a) 1, (b,c) 1, (c,a) 2, (c|d, b|c) 1,
// (d,a) 3; plus 1 when p_m = a, for the vertex below the strip).  Labels
// can be negative down to -2 (3m + 1); entries are stored shifted by
// shift = 2 (3m + 1) so that they fit uint16, and every closed walk of n
// arcs then weighs n * shift more.
__global__ __launch_bounds__(256) void border_transfer_kernel(WordTable t, int64_t n, u16 *A, int64_t lda, int shift)
{
    const int64_t q = blockIdx.x;
    const uint32_t wq = unrank(t, q);
    const int m = t.m;
    for (int64_t p = threadIdx.x; p < n; p += blockDim.x) {
        const uint32_t wp = unrank(t, p);
        bool ok = true;
        int label = 0, nd = 0;
        for (int i = 0; i < m; i++) {
            const int qi = (wq >> (2 * i)) & 3, pi = (wp >> (2 * i)) & 3;
            const bool a_up = i > 0 && ((wp >> (2 * (i - 1))) & 3) == 0;
            const bool a_down = i + 1 < m && ((wp >> (2 * (i + 1))) & 3) == 0;
            const int qr = (i == m - 1 && qi == 3) ? 2 : qi;  // last row: d behaves like c
            const uint32_t allowed = kAlways[qr] | ((a_up || a_down) ? kWithA[qr] : 0);
            ok = ok && ((allowed >> pi) & 1u);
            label += pi == 0 ? 10 : (pi == 1 ? 5 : 0);
            if (qi == 0 && pi == 0) nd += 1;
            else if (qi == 1 && pi == 2) nd += 1;
            else if (qi == 2 && pi == 0) nd += 2;
            else if (qi >= 2 && (pi == 1 || pi == 2)) nd += 1;
            else if (qi == 3 && pi == 0) nd += 3;
        }
        if (((wp >> (2 * (m - 1))) & 3) == 0) nd += 1;
        A[q * lda + p] = ok ? (u16)(label - 2 * nd + shift) : (u16)0xFFFF;
    }
}

int border_shift(int m) { return 2 * (3 * m + 1); }

mpr_status border_transfer_launch(int m, u16 *A, int64_t lda, hipStream_t s)
{
    WordTable t;
    make_table(m, t);
    const int64_t n = word_count(t);
    if (lda < n) return MPR_EINVAL;
    hipLaunchKernelGGL(border_transfer_kernel, dim3((unsigned)n), dim3(256), 0, s, t, n, A, lda, border_shift(m));
    return check_launch();
}

mpr_status transfer_launch(int m, u16 *A, int64_t lda, hipStream_t s)
{
    WordTable t;
    make_table(m, t);
    const int64_t n = word_count(t);
    if (lda < n) return MPR_EINVAL;
    hipLaunchKernelGGL(transfer_kernel, dim3((unsigned)((n + TCOLS - 1) / TCOLS), (unsigned)((n + TROWS - 1) / TROWS)),
                       dim3(256), 0, s, t, n, A, lda, aligned16(A) && lda % 8 == 0 ? 1 : 0);
    return check_launch();
}

int64_t transfer_size(int m)
{
    WordTable t;
    make_table(m, t);
    return word_count(t);
}

void transfer_words(int m, uint8_t *out, int64_t count)
{
    WordTable t;
    make_table(m, t);
    for (int64_t r = 0; r < count; r++) {
        const uint32_t w = unrank(t, r);
        for (int i = 0; i < m; i++) out[r * m + i] = (uint8_t)((w >> (2 * i)) & 3);
    }
}

}  // namespace mpr
