// The bitmap route (Sec. I-A, "bitmaps ... AND ... count the number of 1s"; the
// PBI-GPU layout of Sec. I-B): every tidlist becomes a row of a bit matrix, one
// bit per transaction, and all supports are the Gram matrix A A^T, taken on
// the matrix cores.
//
// The bits become 4-bit floats (E2M1) in registers: bit 0, 1 or 2 of a nibble
// alone is 0.5, 1 or 2, so one AND with 0x11111111, 0x22222222 or 0x44444444
// turns a word of 32 bits into eight operands, and the instruction's block
// scale (an exact power of two) brings every product of two set bits to 1.
// v_mfma_scale_f32_32x32x64_f8f6f4 adds them in fp32: counts are whole numbers,
// exact up to 2^24, and no segment sums more than 2^24 transactions before its
// counts become u32 (kGramMaxStages).
#include <algorithm>

#include "bm_internal.h"

namespace bm {

namespace {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------- bit rows

// First position in [lo, hi) of the sorted `a` with a[pos] >= x, by a whole
// wavefront: 64 probes a round narrow the range 64-fold (three dependent loads
// for a set of 10^5 where a binary search takes seventeen).
__device__ inline uint64_t wave_lower_bound(const uint32_t *a, uint64_t lo, uint64_t hi, uint64_t x)
{
    const uint32_t lane = threadIdx.x & 63;
    while (hi - lo > 64) {
        const uint64_t step = (hi - lo + 63) / 64;
        const uint64_t at = lo + lane * step;
        const uint64_t below = __ballot(at < hi && a[at] < x);  // a prefix of the lanes
        const uint32_t c = (uint32_t)__popcll(below);
        if (c == 0)
            return lo;
        hi = std::min(hi, lo + c * step);
        lo = lo + (uint64_t)(c - 1) * step + 1;
    }
    const uint64_t at = lo + lane;
    return lo + (uint64_t)__popcll(__ballot(at < hi && a[at] < x));
}

// One workgroup per (row, segment of kBitSeg transactions): the segment is
// put together in LDS (zeros, then the bits of the row's tids that fall in it)
// and leaves in 16-byte stores, so every word of the matrix is written once.
// Four consecutive tids a thread: the bits of one word are merged before the
// LDS atomic (in a dense row all four share a word).  Row n_rows is all zero:
// the rows that pad a tile read it.
// A segment of 2^17 transactions takes 16 KB of LDS: eight workgroups a CU.
__global__ void __launch_bounds__(kBitRowThreads) bit_rows_kernel(const uint64_t *__restrict__ off,
                                                       const uint32_t *__restrict__ tids,
                                                       const uint32_t *__restrict__ items, uint32_t n_rows,
                                                       uint64_t ld, uint32_t n_seg, uint32_t *__restrict__ bits)
{
    __shared__ __attribute__((aligned(16))) uint32_t seg[kBitSeg / 32];
    __shared__ uint64_t range[2];
    const uint32_t row = blockIdx.x / n_seg, c = blockIdx.x % n_seg;
    const uint64_t w0 = (uint64_t)c * (kBitSeg / 32);
    const uint32_t len = (uint32_t)std::min<uint64_t>(ld - w0, kBitSeg / 32);  // words, a multiple of 16
    uint64_t e0 = 0, e1 = 0;
    if (row < n_rows) {
        const uint32_t item = items ? items[row] : row;
        e0 = off[item];
        e1 = off[item + 1];
    }
    for (uint32_t b = threadIdx.x * 4; b < len; b += blockDim.x * 4)
        *reinterpret_cast<uint4 *>(seg + b) = make_uint4(0, 0, 0, 0);
    if (threadIdx.x < 128) {  // wavefront 0 finds the segment's first tid, wavefront 1 its end
        const uint32_t w = threadIdx.x >> 6;
        uint64_t at = w ? e1 : e0;
        if (n_seg > 1 && e1 > e0 && (w ? c + 1 < n_seg : c > 0))
            at = wave_lower_bound(tids, e0, e1, (uint64_t)(c + w) * kBitSeg);
        if ((threadIdx.x & 63) == 0)
            range[w] = at;
    }
    __syncthreads();
    const uint64_t k1 = range[1];
    const uint32_t base = c * kBitSeg;
    for (uint64_t k = range[0] + 4 * threadIdx.x; k < k1; k += 4 * blockDim.x) {
        uint32_t t[4];
        const uint32_t cnt = (uint32_t)std::min<uint64_t>(4, k1 - k);
#pragma unroll
        for (uint32_t q = 0; q < 4; q++)
            t[q] = tids[k + (q < cnt ? q : 0)] - base;  // a short tail repeats its first tid
        uint32_t w = t[0] >> 5, acc = 1u << (t[0] & 31);
#pragma unroll
        for (uint32_t q = 1; q < 4; q++) {
            const uint32_t bit = 1u << (t[q] & 31);
            if ((t[q] >> 5) != w) {
                atomicOr(&seg[w], acc);
                w = t[q] >> 5;
                acc = 0;
            }
            acc |= bit;
        }
        atomicOr(&seg[w], acc);
    }
    __syncthreads();
    uint32_t *dst = bits + (uint64_t)row * ld + w0;
    for (uint32_t b = threadIdx.x * 4; b < len; b += blockDim.x * 4)
        *reinterpret_cast<uint4 *>(dst + b) = *reinterpret_cast<const uint4 *>(seg + b);
}

// ---------------------------------------------------------------- Gram matrix

constexpr uint32_t kStageBytes = kGramStage / 8;       // of a row, per stage: 64
constexpr uint32_t kLdsRow = kStageBytes + 16;         // LDS row stride: 16-byte reads of 32 rows spread over all banks

// Tile t of the grid: row-major over the rectangle, or over the tiles on and
// above the diagonal.
__device__ inline void tile_at(const GramArgs &g, uint32_t t, uint32_t &ti, uint32_t &tj)
{
    if (!g.tri) {
        ti = t / g.TC;
        tj = t % g.TC;
        return;
    }
    ti = 0;
    while (t >= g.TR - ti) {
        t -= g.TR - ti;
        ti++;
    }
    tj = ti + t;
}

__device__ inline void put_count(const GramArgs &g, uint32_t i, uint32_t j, uint32_t v)
{
    if (g.tri) {
        if (i < j && j < g.b.n)
            g.out[(uint64_t)i * g.n_out - (uint64_t)i * (i + 1) / 2 + (j - i - 1)] = v;
    } else if (i < g.a.n && j < g.b.n) {
        g.out[(uint64_t)i * g.n_out + j] = v;
    }
}

__device__ inline void add_count(const GramArgs &g, uint32_t i, uint32_t j, uint32_t v)
{
    if (v == 0)
        return;
    if (g.tri) {
        if (i < j && j < g.b.n)
            atomicAdd(&g.out[(uint64_t)i * g.n_out - (uint64_t)i * (i + 1) / 2 + (j - i - 1)], v);
    } else if (i < g.a.n && j < g.b.n) {
        atomicAdd(&g.out[(uint64_t)i * g.n_out + j], v);
    }
}

// A workgroup is WR x WC wavefronts, each owning BR x BC blocks of 32 x 32
// counts.  Lane l holds row (or column) l mod 32 of a block and the 16 bytes
// l / 32 of the current 32: rows and columns read their bits in the same order,
// so which bit meets which operand slot does not matter.  Result register e of
// lane l is row 8 (e / 4) + 4 (l / 32) + e mod 4, column l mod 32.
//
// The work is the list of all (tile, stage) in tile order, cut into W equal
// runs, one per workgroup: whatever the tile count, no workgroup idles.  A run
// that covers a whole tile writes its counts; a part of a tile goes to the
// workgroup's own place in ws (its first run part in place 2 w, its last in
// 2 w + 1), and gram_reduce_kernel adds the parts.  (Device atomics run at about
// 27 * 10^9 a second here: 0.6 ms for 256 parts of 256 x 256, against 0.03 ms
// for writing them out and reading them back.)  kAdd: those atomics all the same,
// where there is no scratch (plan_gram_add).
//
// Bound by the matrix cores: 32 MFMAs of 32 cycles a wavefront against 6 LDS
// reads and 120 VALU operations per 256 transactions (128 x 64 counts).  Bits
// rather than bytes or nibbles in memory and LDS make the panels 8 and 4 times
// smaller: a workgroup reads 32 KB per 512 transactions of 256 x 256 counts,
// about 3 TB/s over the chip at full rate, so that no tile order for the L2s is
// needed.  m = 2^20, n = 4096: 2.5 ms, 7.0 * 10^15 operations (2 m per pair) a
// second; the int8 kernel before it (0/1 bytes, v_mfma_i32_16x16x64_i8, bound by
// its LDS reads) took 9.8 ms.
template <int BR, int BC, int WR, int WC, bool kAdd = false>
__device__ __forceinline__ void gram_run(const GramArgs &g, uint32_t wg, uint8_t (*lds)[32 * (BR * WR + BC * WC)][kLdsRow])
{
    constexpr int R = 32 * BR * WR, C = 32 * BC * WC, NT = 64 * WR * WC;
    constexpr int Q = (R + C) * 4 / NT;  // 16-byte pieces a thread stages
    const uint32_t tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, wr = wv / WC, wc = wv % WC;
    const uint64_t u0 = g.U * wg / g.W, u1 = g.U * (wg + 1) / g.W;
    for (uint64_t u = u0; u < u1;) {
        const uint32_t t = (uint32_t)(u / g.S), s0 = (uint32_t)(u % g.S);
        const uint32_t steps = (uint32_t)std::min<uint64_t>(g.S - s0, u1 - u);
        uint32_t ti, tj;
        tile_at(g, t, ti, tj);
        const v4u *src[Q];
#pragma unroll
        for (int q = 0; q < Q; q++) {
            const uint32_t id = tid + NT * q, r = id / 4;
            const BitMat &m = r < (uint32_t)R ? g.a : g.b;
            const uint32_t p = r < (uint32_t)R ? ti * R + r : tj * C + (r - R);
            const uint32_t row = p < m.n ? (m.rows ? m.rows[p] : p) : m.zero;
            src[q] = reinterpret_cast<const v4u *>(m.bits + (uint64_t)row * m.ld) + (uint64_t)s0 * 4 + id % 4;
        }
        v16f acc[BR][BC];
#pragma unroll
        for (int a = 0; a < BR; a++)
#pragma unroll
            for (int b = 0; b < BC; b++)
#pragma unroll
                for (int e = 0; e < 16; e++)
                    acc[a][b][e] = 0.f;
        v4u held[Q];
#define BM_GRAM_FETCH(ST)                                      \
    _Pragma("unroll") for (int q = 0; q < Q; q++) held[q] = src[q][(uint64_t)(ST) * 4]
#define BM_GRAM_STORE(TO)                                      \
    _Pragma("unroll") for (int q = 0; q < Q; q++)              \
        *reinterpret_cast<v4u *>(&lds[TO][(tid + NT * q) / 4][(tid + NT * q) % 4 * 16]) = held[q]
        BM_GRAM_FETCH(0);
        BM_GRAM_STORE(0);
        if (steps > 1)
            BM_GRAM_FETCH(1);
        __syncthreads();
        for (uint32_t st = 0; st < steps; st++) {
            const int cur = (int)(st & 1);
#pragma unroll
            for (int sub = 0; sub < (int)kStageBytes / 32; sub++) {
                v4u wa[BR], wb[BC];
#pragma unroll
                for (int a = 0; a < BR; a++)
                    wa[a] = *reinterpret_cast<const v4u *>(
                        &lds[cur][(wr * BR + a) * 32 + (lane & 31)][sub * 32 + (lane >> 5) * 16]);
#pragma unroll
                for (int b = 0; b < BC; b++)
                    wb[b] = *reinterpret_cast<const v4u *>(
                        &lds[cur][R + (wc * BC + b) * 32 + (lane & 31)][sub * 32 + (lane >> 5) * 16]);
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    // bit j of every nibble: values 0.5, 1, 2 and (moved down one) 2; the scale of the
                    // row operand, 2^(s - 127), makes each product 1
                    constexpr uint32_t kMask[4] = {0x11111111u, 0x22222222u, 0x44444444u, 0x44444444u};
                    constexpr int kScale[4] = {129, 127, 125, 125};
                    auto nib = [&](v4u w) {
                        const int s = j == 3 ? 1 : 0;
                        return v8i{(int)((w.x >> s) & kMask[j]), (int)((w.y >> s) & kMask[j]),
                                   (int)((w.z >> s) & kMask[j]), (int)((w.w >> s) & kMask[j]), 0, 0, 0, 0};
                    };
                    v8i fa[BR], fb[BC];
#pragma unroll
                    for (int a = 0; a < BR; a++)
                        fa[a] = nib(wa[a]);
#pragma unroll
                    for (int b = 0; b < BC; b++)
                        fb[b] = nib(wb[b]);
#pragma unroll
                    for (int a = 0; a < BR; a++)
#pragma unroll
                        for (int b = 0; b < BC; b++)
                            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(
                                fa[a], fb[b], acc[a][b], 4, 4, 0, kScale[j], 0, 127);
                }
            }
            // the other stage was last read during step st - 1, which every wavefront ended
            // before the barrier that closed it
            if (st + 1 < steps)
                BM_GRAM_STORE(cur ^ 1);
            if (st + 2 < steps)
                BM_GRAM_FETCH(st + 2);
            __syncthreads();
        }
#undef BM_GRAM_STORE
#undef BM_GRAM_FETCH
        if (steps == g.S) {
#pragma unroll
            for (int a = 0; a < BR; a++)
#pragma unroll
                for (int b = 0; b < BC; b++)
#pragma unroll
                    for (int e = 0; e < 16; e++)
                        put_count(g, ti * R + (wr * BR + a) * 32 + 8 * (e / 4) + 4 * (lane >> 5) + e % 4,
                                  tj * C + (wc * BC + b) * 32 + (lane & 31), (uint32_t)acc[a][b][e]);
        } else if constexpr (kAdd) {
#pragma unroll
            for (int a = 0; a < BR; a++)
#pragma unroll
                for (int b = 0; b < BC; b++)
#pragma unroll
                    for (int e = 0; e < 16; e++)
                        add_count(g, ti * R + (wr * BR + a) * 32 + 8 * (e / 4) + 4 * (lane >> 5) + e % 4,
                                  tj * C + (wc * BC + b) * 32 + (lane & 31), (uint32_t)acc[a][b][e]);
        } else {
            float *part = g.ws + (uint64_t)(2 * wg + (u != u0)) * ((uint64_t)R * C) + wv * (BR * BC * 1024) + lane;
#pragma unroll
            for (int a = 0; a < BR; a++)
#pragma unroll
                for (int b = 0; b < BC; b++)
#pragma unroll
                    for (int e = 0; e < 16; e++)
                        part[((a * BC + b) * 16 + e) * 64] = acc[a][b][e];
        }
        u += steps;
    }
}

template <int BR, int BC, int WR, int WC, bool kAdd>
__global__ void __launch_bounds__(64 * WR * WC, BR * BC >= 8 ? 2 : BR * BC >= 4 ? 3 : 4) bit_gram_kernel(const GramArgs g)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][32 * (BR * WR + BC * WC)][kLdsRow];
    gram_run<BR, BC, WR, WC, kAdd>(g, blockIdx.x, lds);
}

// The job that owns workgroup w.
template <uint32_t GramJob::*First>
__device__ __forceinline__ const GramJob &job_at(const GramJob *jobs, uint32_t n, uint32_t w)
{
    uint32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) / 2;
        if (jobs[mid].*First <= w)
            lo = mid;
        else
            hi = mid;
    }
    return jobs[lo];
}

// The runs of several families, each with its own tile size (see plan_gram_set).
// Eight families of 100 to 3,000 items over 10^4 to 4 10^5 transactions: 0.45 ms,
// against 0.55 with two launches a family on four streams.
__global__ void __launch_bounds__(256, 3) bit_gram_jobs_kernel(const GramJob *jobs, uint32_t n)
{
    __shared__ __attribute__((aligned(16))) uint8_t lds[2][256][kLdsRow];
    const GramJob &j = job_at<&GramJob::w0>(jobs, n, blockIdx.x);
    const GramArgs g = j.g;
    const uint32_t wg = blockIdx.x - j.w0;
    if (j.tile == 128)
        gram_run<2, 2, 2, 2>(g, wg, lds);
    else
        gram_run<1, 1, 2, 2>(g, wg, reinterpret_cast<uint8_t (*)[128][kLdsRow]>(&lds[0][0][0]));
}

// Adds the parts of the tiles that several workgroups shared, in the order in
// which bit_gram_kernel left them, and writes the counts.  Four counts a
// thread; Y threads share the parts of the same counts (a tile of a small query
// has hundreds of parts).
template <int BR, int BC, int WR, int WC, int Y>
__device__ __forceinline__ void gram_reduce(const GramArgs &g, uint32_t block, uint4 *lds)
{
    constexpr uint32_t R = 32 * BR * WR, C = 32 * BC * WC, X = 256 / Y, kParts = R * C / (4 * X);
    const uint32_t t = block / kParts, p = block % kParts;
    const uint64_t t0 = (uint64_t)t * g.S, t1 = t0 + g.S;  // the tile's stages
    // the workgroup that ran stage u: U w / W <= u < U (w + 1) / W, both rounded down
    auto at = [&](uint64_t u) {
        uint64_t w = u * g.W / g.U;
        while (g.U * (w + 1) < (u + 1) * g.W)
            w++;
        while (g.U * w >= (u + 1) * g.W)
            w--;
        return (uint32_t)w;
    };
    const uint32_t wa = at(t0), wb = at(t1 - 1);
    if (wa == wb)
        return;  // one workgroup covered the tile and wrote its counts
    const uint32_t x = threadIdx.x % X, y = threadIdx.x / X;
    const uint32_t e4 = (p * X + x) * 4;
    // whether the first group came to the tile from another one (its U wa / W is not t0)
    const uint32_t late = g.U * wa < t0 * g.W || g.U * wa >= (t0 + 1) * g.W;
    uint4 sum = make_uint4(0, 0, 0, 0);
#pragma unroll 4
    for (uint32_t w = wa + y; w <= wb; w += Y) {
        const uint32_t place = 2 * w + (w == wa ? late : 0);
        const float4 v = *reinterpret_cast<const float4 *>(g.ws + (uint64_t)place * (R * C) + e4);
        sum.x += (uint32_t)v.x;
        sum.y += (uint32_t)v.y;
        sum.z += (uint32_t)v.z;
        sum.w += (uint32_t)v.w;
    }
    if constexpr (Y > 1) {
        uint4 *mine = lds + threadIdx.x;
        *mine = sum;
        __syncthreads();
#pragma unroll
        for (uint32_t half = Y / 2; half > 0; half /= 2) {
            if (y < half) {
                const uint4 v = mine[half * X];
                sum.x += v.x;
                sum.y += v.y;
                sum.z += v.z;
                sum.w += v.w;
                *mine = sum;
            }
            __syncthreads();
        }
        if (y != 0)
            return;
    }
    uint32_t ti, tj;
    tile_at(g, t, ti, tj);
    const uint32_t lane = e4 & 63, e = (e4 >> 6) & 15, blk = e4 >> 10;
    const uint32_t b = blk % BC, a = blk / BC % BR, wv = blk / (BC * BR), wr = wv / WC, wc = wv % WC;
    const uint32_t i = ti * R + (wr * BR + a) * 32 + 8 * (e / 4) + 4 * (lane >> 5) + e % 4;
    const uint32_t j = tj * C + (wc * BC + b) * 32 + (lane & 31);
    put_count(g, i, j, sum.x);
    put_count(g, i, j + 1, sum.y);
    put_count(g, i, j + 2, sum.z);
    put_count(g, i, j + 3, sum.w);
}

template <int BR, int BC, int WR, int WC, int Y>
__global__ void __launch_bounds__(kReduceThreads) gram_reduce_kernel(const GramArgs g, uint32_t first)
{
    __shared__ uint4 lds[kReduceThreads];
    gram_reduce<BR, BC, WR, WC, Y>(g, first + blockIdx.x, lds);
}

__global__ void __launch_bounds__(256) gram_reduce_jobs_kernel(const GramJob *jobs, uint32_t n)
{
    __shared__ uint4 lds[256];
    const GramJob &j = job_at<&GramJob::r0>(jobs, n, blockIdx.x);
    const GramArgs g = j.g;
    const uint32_t block = blockIdx.x - j.r0, fold = j.fold;
    if (j.tile == 128) {
        if (fold == 1)
            gram_reduce<2, 2, 2, 2, 1>(g, block, lds);
        else if (fold == 4)
            gram_reduce<2, 2, 2, 2, 4>(g, block, lds);
        else
            gram_reduce<2, 2, 2, 2, 16>(g, block, lds);
    } else {
        if (fold == 1)
            gram_reduce<1, 1, 2, 2, 1>(g, block, lds);
        else if (fold == 4)
            gram_reduce<1, 1, 2, 2, 4>(g, block, lds);
        else
            gram_reduce<1, 1, 2, 2, 16>(g, block, lds);
    }
}

template <int BR, int BC, int WR, int WC>
hipError_t run_gram(const GramArgs &g, const GramPlan &p, hipStream_t s)
{
    auto *product = p.add ? bit_gram_kernel<BR, BC, WR, WC, true> : bit_gram_kernel<BR, BC, WR, WC, false>;
    product<<<g.W, 64 * WR * WC, 0, s>>>(g);
    hipError_t e = hipGetLastError();
    if (p.ws_floats == 0)
        return e;
    const uint32_t fold = gram_reduce_fold(p, 64);
    auto *kernel = fold == 64   ? gram_reduce_kernel<BR, BC, WR, WC, 64>
                   : fold == 16 ? gram_reduce_kernel<BR, BC, WR, WC, 16>
                   : fold == 4  ? gram_reduce_kernel<BR, BC, WR, WC, 4>
                                : gram_reduce_kernel<BR, BC, WR, WC, 1>;
    const uint64_t blocks = gram_reduce_blocks(p, fold);
    for (uint64_t first = 0; first < blocks && e == hipSuccess; first += kReduceGrid) {
        kernel<<<gram_reduce_launch(blocks, first), kReduceThreads, 0, s>>>(g, (uint32_t)first);
        e = hipGetLastError();
    }
    return e;
}

GramArgs gram_args(const GramPlan &p, const BitMat &a, const BitMat &b, uint32_t *out, uint64_t n_out, float *ws)
{
    GramArgs g;
    g.a = a;
    g.b = b;
    g.TR = p.tile_rows;
    g.TC = p.tile_cols;
    g.S = p.stages;
    g.W = p.groups;
    g.U = (uint64_t)p.tiles * p.stages;
    g.tri = p.tri;
    g.out = out;
    g.n_out = n_out;
    g.ws = ws;
    return g;
}

}  // namespace

hipError_t launch_bit_rows(const uint64_t *off, const uint32_t *tids, const uint32_t *items, uint32_t n_rows,
                           uint32_t m, uint32_t *bits, hipStream_t s)
{
    const uint64_t ld = bit_row_words(m);
    const uint64_t n_seg = (ld + kBitSeg / 32 - 1) / (kBitSeg / 32);
    const uint64_t blocks = bit_row_blocks(n_rows, ld);
    if (!grid_fits(blocks, kBitRowThreads))
        return hipErrorInvalidValue;
    bit_rows_kernel<<<(uint32_t)blocks, kBitRowThreads, 0, s>>>(off, tids, items, n_rows, ld, (uint32_t)n_seg, bits);
    return hipGetLastError();
}

hipError_t launch_gram(const GramPlan &p, const BitMat &a, const BitMat &b, uint32_t *out, uint64_t n_out, float *ws,
                       hipStream_t s)
{
    if (p.tiles == 0)
        return hipSuccess;
    if (a.ld != b.ld || a.ld != (uint64_t)p.stages * (kGramStage / 32) || (p.ws_floats && !ws))
        return hipErrorInvalidValue;
    const GramArgs g = gram_args(p, a, b, out, n_out, ws);
    switch (p.tile) {
    case 256: return run_gram<4, 2, 2, 4>(g, p, s);
    case 128: return run_gram<2, 2, 2, 2>(g, p, s);
    default: return run_gram<1, 1, 2, 2>(g, p, s);
    }
}

GramJobs gram_jobs(const GramSetPlan &set, const BitMat *a, uint32_t *const *out, float *ws, GramJob *jobs)
{
    GramJobs j;
    for (size_t q = 0; q < set.plan.size(); q++) {
        const GramPlan &p = set.plan[q];
        if (!set.joint[q])
            continue;
        GramJob &o = jobs[j.n++];
        o.g = gram_args(p, a[q], a[q], out[q], a[q].n, ws);
        o.tile = (uint32_t)p.tile;
        o.fold = gram_reduce_fold(p, 16);
        o.w0 = j.groups;
        o.r0 = j.reduce_blocks;
        j.groups += p.groups;
        if (p.ws_floats)
            j.reduce_blocks += (uint32_t)gram_reduce_blocks(p, o.fold);
        ws += p.ws_floats;
    }
    return j;
}

hipError_t launch_gram_jobs(const GramJob *jobs, const GramJobs &j, hipStream_t s)
{
    if (j.groups == 0)
        return hipSuccess;
    bit_gram_jobs_kernel<<<j.groups, 256, 0, s>>>(jobs, j.n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || j.reduce_blocks == 0)
        return e;
    gram_reduce_jobs_kernel<<<j.reduce_blocks, 256, 0, s>>>(jobs, j.n);
    return hipGetLastError();
}

}  // namespace bm
