// Ingest (Sec. I, "Set representations"): validation of the vertical format
// (sorted tidlists) and conversion of the horizontal format (transactions) to
// it.  The conversion is a stable sort of (item, tid) pairs by item: pairs
// arrive in tid order, so every tidlist comes out sorted.  Where the incidences
// are not too sparse it goes through bit rows instead (txn_bits_kernel).
#include <algorithm>

#include "bm_internal.h"

namespace bm {

namespace {

constexpr int kBlock = 256;

uint32_t blocks_for(uint64_t n, uint32_t cap = 1u << 20)
{
    uint64_t g = (n + kBlock - 1) / kBlock;
    if (g < 1)
        g = 1;
    return (uint32_t)(g > cap ? cap : g);
}

// row_of[k] = b for every k in transaction b.  A wavefront takes 64
// consecutive transactions, keeps their offsets in LDS and writes their
// incidences in order, 256 at a time: a lane takes four consecutive ones,
// finds the first one's transaction by binary search (the last offset <= k,
// which skips empty transactions), steps forward for the other three and
// stores the four at once.
__global__ void expand_rows_kernel(const uint64_t *row_off, uint32_t m, uint32_t *row_of)
{
    __shared__ uint32_t offs_all[kBlock / 64][65];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
    uint32_t *offs = offs_all[wave];
    const uint64_t n_blocks = ((uint64_t)m + 63) / 64;
    const uint64_t stride = (uint64_t)gridDim.x * (blockDim.x / 64u);
    for (uint64_t rb = (uint64_t)blockIdx.x * (blockDim.x / 64u) + wave; rb < n_blocks; rb += stride) {
        const uint64_t b0 = rb * 64;
        const uint32_t rows = (uint32_t)(m - b0 < 64 ? m - b0 : 64);
        // the block's row starts relative to its first element (an index
        // holds fewer than 2^32 incidences)
        const uint64_t first = row_off[b0];
        offs[lane] = (uint32_t)(row_off[b0 + (lane < rows ? lane : rows)] - first);
        if (lane == 0)
            offs[64] = (uint32_t)(row_off[b0 + rows] - first);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t len = offs[64];
        // four consecutive outputs a lane, in quads aligned to four elements;
        // the partial quads at either end hold other blocks' elements too
        const uint64_t q0 = first & ~3ull;
        for (uint64_t a = q0 + 4ull * lane; a < first + len; a += 256) {
            const int64_t rel = (int64_t)(a - first);  // -3 .. -1 in the first quad
            const uint32_t k0 = rel < 0 ? 0u : (uint32_t)rel;
            uint32_t lo = 0, hi = rows;  // offs[lo] <= k0 < offs[hi]
            while (hi - lo > 1) {
                const uint32_t mid = (lo + hi) >> 1;
                if (offs[mid] <= k0)
                    lo = mid;
                else
                    hi = mid;
            }
            uint32_t v[4];
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int64_t k = rel + j;
                if (k >= 0 && k < (int64_t)len) {
                    while (offs[lo + 1] <= (uint32_t)k)
                        lo++;
                }
                v[j] = (uint32_t)(b0 + lo);
            }
            if (rel >= 0 && rel + 4 <= (int64_t)len) {
                *reinterpret_cast<uint4 *>(row_of + a) = make_uint4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++)
                    if (rel + j >= 0 && rel + j < (int64_t)len)
                        row_of[a + j] = v[j];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

__global__ void check_items_kernel(const uint32_t *items, uint64_t nnz, uint32_t n, uint32_t *flag)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += stride)
        bad |= items[k] >= n;
    if (bad)
        atomicOr(flag, 1u);
}

// Row offsets of a transactions CSR: bit 1 when offsets[0] != 0, bit 2 when
// they decrease somewhere.  The first form is one workgroup's and clears the
// second word too, which saves a small build the launch that would.
__global__ void __launch_bounds__(1024) check_offsets_small_kernel(const uint64_t *off, uint32_t m, uint32_t *flags)
{
    bool down = false;
    for (uint32_t b = threadIdx.x; b < m; b += blockDim.x)
        down |= off[b + 1] < off[b];
    const int any = __syncthreads_or(down);
    if (threadIdx.x == 0) {
        flags[0] = (any ? 4u : 0u) | (off[0] != 0 ? 2u : 0u);
        flags[1] = 0;
    }
}

__global__ void check_offsets_kernel(const uint64_t *off, uint32_t m, uint32_t *flag)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    bool down = false;
    for (uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; b < m; b += stride)
        down |= off[b + 1] < off[b];
    if (down)
        atomicOr(flag, 4u);
    if (blockIdx.x == 0 && threadIdx.x == 0 && off[0] != 0)
        atomicOr(flag, 2u);
}

__global__ void mark_dups_kernel(const uint32_t *keys, const uint32_t *vals, uint64_t nnz, uint32_t *keep,
                                 uint32_t *n_dup)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    uint32_t dups = 0;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += stride) {
        bool dup = k > 0 && keys[k] == keys[k - 1] && vals[k] == vals[k - 1];
        keep[k] = dup ? 0u : 1u;
        dups += dup;
    }
    if (dups)
        atomicAdd(n_dup, dups);
}

__global__ void compact_pairs_kernel(const uint32_t *keys, const uint32_t *vals, const uint32_t *keep,
                                     const uint64_t *pos, uint64_t nnz, uint32_t *ko, uint32_t *vo)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += stride) {
        if (keep[k]) {
            ko[pos[k]] = keys[k];
            vo[pos[k]] = vals[k];
        }
    }
}

// off[a] = first position whose key is >= a, for a in [0, n]; keys sorted.
__global__ void offsets_from_sorted_kernel(const uint32_t *keys, uint64_t nnz, uint32_t n, uint64_t *off)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k <= nnz; k += stride) {
        uint32_t lo = k == 0 ? 0u : keys[k - 1] + 1u;     // first key not yet started
        uint32_t hi = k == nnz ? n : keys[k];              // keys that start here
        for (uint32_t a = lo; a <= hi && a <= n; a++)
            off[a] = k;
    }
}

// offsets_from_sorted and, in the same pass, the number of adjacent equal
// (key, value) pairs (an item repeated within one transaction).  A thread
// takes four consecutive pairs with 16-byte loads (the pair before them is a
// neighbour's: it comes from the lane below, or from memory for lane 0);
// position nnz, the end, is handled by thread 0.
__device__ inline void offsets_at(uint64_t k, uint32_t prev, uint32_t cur, uint32_t n, uint64_t *off)
{
    // keys prev + 1 .. cur start at k (all of 0 .. cur when k = 0)
    for (uint32_t a = k == 0 ? 0u : prev + 1u; a <= cur && a <= n; a++)
        off[a] = k;
}

__global__ void offsets_and_dups_kernel(const uint32_t *keys, const uint32_t *vals, uint64_t nnz, uint32_t n,
                                        uint64_t *off, uint32_t *n_dup)
{
    const uint64_t quads = nnz / 4;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t dups = 0;
    // full quads, in rounds that keep every lane of a wavefront active
    const uint64_t rounds = (quads + stride - 1) / stride;
    for (uint64_t r = 0; r < rounds; r++) {
        const uint64_t q = r * stride + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
        const bool live = q < quads;
        uint4 kv = make_uint4(0, 0, 0, 0), vv = make_uint4(0, 0, 0, 0);
        if (live) {
            kv = reinterpret_cast<const uint4 *>(keys)[q];
            vv = reinterpret_cast<const uint4 *>(vals)[q];
        }
        // the pair before this quad: the lane below's last, or loaded
        uint32_t pk = __shfl_up(kv.w, 1, 64), pv = __shfl_up(vv.w, 1, 64);
        if (live && lane == 0 && q > 0) {
            pk = keys[4 * q - 1];
            pv = vals[4 * q - 1];
        }
        if (live) {
            const uint64_t k = 4 * q;
            const uint32_t ks[4] = {kv.x, kv.y, kv.z, kv.w}, vs[4] = {vv.x, vv.y, vv.z, vv.w};
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const uint32_t prev = e == 0 ? pk : ks[e - 1], prevv = e == 0 ? pv : vs[e - 1];
                const bool first = k + e == 0;
                if (first || ks[e] != prev)
                    offsets_at(k + e, prev, ks[e], n, off);
                else if (vs[e] == prevv)
                    dups++;
            }
        }
    }
    // the tail (fewer than four pairs) and the end position
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g < nnz - 4 * quads) {
        const uint64_t k = 4 * quads + g;
        const uint32_t cur = keys[k], prev = k == 0 ? 0u : keys[k - 1];
        if (k == 0 || cur != prev)
            offsets_at(k, prev, cur, n, off);
        else if (vals[k] == vals[k - 1])
            dups++;
    }
    if (g == 0)
        offsets_at(nnz, nnz == 0 ? 0u : keys[nnz - 1], n, n, off);
    if (dups)
        atomicAdd(n_dup, dups);
}

// ------------------------------------------------- transactions -> bit rows
// A workgroup takes 32 TW consecutive transactions, sets one bit per incidence
// in an LDS block of (n + 1) x TW words (the row of no item stays zero) and
// writes the block into the bit rows, 4 TW bytes of every row.  The rows are
// what the tidlists are then read from, in order and without repeats, so that
// no sort is needed: the incidences are read once and the rows move three
// times (written, counted, expanded) where each pass of the radix sort moves 16
// bytes an incidence.  LDS rows are TW + 1 words apart: the incidences of a
// transaction (same word, other items) spread over the banks.  Consecutive
// chunks run on one XCD, whose L2 puts the pieces of a line together.  Bound by
// memory: m = 10^6, n = 2000, 4 * 10^7 incidences (160 MB in, 250 MB out) 125 us,
// and 39 us to count them.
template <int TW>
__global__ void __launch_bounds__(kTxnBitsThreads)
    txn_bits_kernel(const uint64_t *__restrict__ row_off, const uint32_t *__restrict__ items, uint32_t m, uint32_t n,
                    uint64_t ld, uint32_t n_chunks, uint32_t per_xcd, uint32_t *__restrict__ bits, uint32_t *flag)
{
    extern __shared__ uint32_t blk[];  // (n + 1) (TW + 1) words
    __shared__ uint32_t offs[32 * TW + 1];
    const uint32_t c = blockIdx.x % kXcds * per_xcd + blockIdx.x / kXcds;
    if (blockIdx.x / kXcds >= per_xcd || c >= n_chunks)
        return;
    const uint32_t t0 = c * (32 * TW), rows = min(32u * TW, m > t0 ? m - t0 : 0u);
    for (uint32_t i = threadIdx.x; i < (n + 1) * (TW + 1); i += kTxnBitsThreads)
        blk[i] = 0;
    const uint64_t base = row_off[min(t0, m)];
    for (uint32_t i = threadIdx.x; i <= rows; i += kTxnBitsThreads)
        offs[i] = (uint32_t)(row_off[min(t0, m) + i] - base);
    __syncthreads();
    const uint32_t total = offs[rows];
    bool bad = false;
    // four consecutive incidences a thread: one search for the first one's
    // transaction (the last offset <= e, which skips empty ones), then steps forward
    for (uint64_t e4 = threadIdx.x * 4; e4 < total; e4 += kTxnBitsThreads * 4) {
        const uint32_t e = (uint32_t)e4;
        uint32_t it[4];
        const uint32_t cnt = min(4u, total - e);
        if (cnt == 4) {
            __builtin_memcpy(it, items + base + e, 16);
        } else {
            for (uint32_t q = 0; q < 4; q++)
                it[q] = items[base + e + (q < cnt ? q : 0)];
        }
        uint32_t lo = 0, hi = rows;  // offs[lo] <= e < offs[hi]
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) / 2;
            if (offs[mid] <= e)
                lo = mid;
            else
                hi = mid;
        }
#pragma unroll
        for (uint32_t q = 0; q < 4; q++) {
            if (q < cnt) {
                while (offs[lo + 1] <= e + q)
                    lo++;
                if (it[q] < n)
                    atomicOr(&blk[it[q] * (TW + 1) + (lo >> 5)], 1u << (lo & 31));
                else
                    bad = true;
            }
        }
    }
    if (bad)
        atomicOr(flag, 1u);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < (n + 1) * (TW / 4); i += kTxnBitsThreads) {
        const uint32_t item = i / (TW / 4), w = i % (TW / 4) * 4;
        const uint64_t at = (uint64_t)c * TW + w;
        if (at < ld) {  // a multiple of 16 words
            const uint32_t *src = &blk[item * (TW + 1) + w];
            *reinterpret_cast<uint4 *>(bits + item * ld + at) = make_uint4(src[0], src[1], src[2], src[3]);
        }
    }
}

// Ones of every (row, segment of kSegWords words), and a 0 behind them.
__global__ void __launch_bounds__(256) bit_count_kernel(const uint32_t *__restrict__ bits, uint64_t ld,
                                                        uint32_t n_seg, uint32_t *count)
{
    __shared__ uint32_t part[4];
    const uint32_t item = blockIdx.x / n_seg, seg = blockIdx.x % n_seg;
    const uint32_t len = (uint32_t)min((uint64_t)kSegWords, ld - (uint64_t)seg * kSegWords);
    const uint32_t *row = bits + item * ld + (uint64_t)seg * kSegWords;
    uint32_t sum = 0;
    for (uint32_t w = threadIdx.x * 4; w < len; w += 1024) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row + w);
        sum += __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
        sum += __shfl_xor(sum, o, 64);
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x / 64] = sum;
    __syncthreads();
    if (threadIdx.x == 0)
        count[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
    if (blockIdx.x == 0 && threadIdx.x == 0)
        count[gridDim.x] = 0;  // where the scan leaves the sum
}

// The tids of one (row, segment), in order, at tids[start[row n_seg + seg] ..).
// W consecutive words a thread and round: their ones are counted, ranked over
// the workgroup and set down in LDS, then written out coalesced.  W is chosen
// so that a round's tids mostly fit the LDS buffer (the rest go out directly),
// as 16-bit offsets in the round (W <= 4); the buffer skips a word after every 32
// of them, since in a dense row the lanes write 32 apart.  Large Zipf (410 MB
// moved): 123 us; with segments of 4096 words, whose dense ones end the launch,
// 183, and with 32-bit offsets, which halve the workgroups a CU, 209.
constexpr uint32_t kExpandBuf = 8192;

template <int W>  // 256 W 32 tids a round: 16 bits
__device__ void expand_segment(const uint32_t *row, uint32_t len, uint32_t t0, uint32_t *out, uint16_t *buf,
                               uint32_t *part)
{
    uint32_t done = 0;
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    for (uint32_t r0 = 0; r0 < len; r0 += 256 * W) {
        const uint32_t w0 = r0 + threadIdx.x * W;
        uint32_t v[W];
        uint32_t ones = 0;
#pragma unroll
        for (int k = 0; k < W; k++) {
            v[k] = w0 < len ? row[w0 + k] : 0u;  // len is a multiple of 16
            ones += __popc(v[k]);
        }
        uint32_t incl = ones;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = __shfl_up(incl, o, 64);
            incl += lane >= (uint32_t)o ? up : 0u;
        }
        if (lane == 63)
            part[wave] = incl;
        __syncthreads();
        uint32_t pos = incl - ones, total = 0;
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) {
            pos += k < wave ? part[k] : 0u;
            total += part[k];
        }
#pragma unroll
        for (int k = 0; k < W; k++) {
            const uint32_t t = (threadIdx.x * W + k) * 32;  // within the round
            for (uint32_t b = v[k]; b; b &= b - 1, pos++) {
                const uint32_t x = t + __builtin_ctz(b);
                if (pos < kExpandBuf)
                    buf[pos + pos / 32 * 2] = (uint16_t)x;
                else
                    out[done + pos] = t0 + r0 * 32 + x;
            }
        }
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < min(total, kExpandBuf); i += 256)
            out[done + i] = t0 + r0 * 32 + buf[i + i / 32 * 2];
        done += total;
        __syncthreads();  // buf and part are written again
    }
}

__global__ void __launch_bounds__(256) bit_expand_kernel(const uint32_t *__restrict__ bits, uint64_t ld, uint32_t n,
                                                         uint32_t n_seg, const uint64_t *__restrict__ start,
                                                         uint64_t *__restrict__ off, uint32_t *__restrict__ tids)
{
    __shared__ uint16_t buf[kExpandBuf + kExpandBuf / 16];
    __shared__ uint32_t part[4];
    const uint32_t item = blockIdx.x / n_seg, seg = blockIdx.x % n_seg;
    const uint64_t s0 = start[blockIdx.x], s1 = start[blockIdx.x + 1];
    if (threadIdx.x == 0 && seg == 0)
        off[item] = s0;
    if (threadIdx.x == 0 && blockIdx.x + 1 == gridDim.x)
        off[n] = s1;
    if (s1 == s0)
        return;
    const uint32_t len = (uint32_t)min((uint64_t)kSegWords, ld - (uint64_t)seg * kSegWords);
    const uint32_t *row = bits + item * ld + (uint64_t)seg * kSegWords;
    const uint32_t t0 = seg * (kSegWords * 32);
    uint32_t *out = tids + s0;
    // about kExpandBuf / 2 tids a round, and every thread at work on short rows
    const uint32_t ones = (uint32_t)(s1 - s0);
    const uint32_t rounds = max(ones / (kExpandBuf / 2), 1u);
    const uint32_t w = min((len + 255) / 256, max(len / (256 * rounds), 1u));
    if (w > 1)
        expand_segment<4>(row, len, t0, out, buf, part);
    else
        expand_segment<1>(row, len, t0, out, buf, part);
}

// One block per set: every tid < m and strictly increasing.
// flags[0] |= 1 on a range error, flags[1] |= 1 on an order error.
__global__ void validate_sets_kernel(const uint64_t *off, const uint32_t *tids, uint32_t n, uint32_t m,
                                     uint32_t *flags)
{
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
        uint64_t b = off[i], e = off[i + 1];
        bool range = false, order = false;
        for (uint64_t k = b + threadIdx.x; k < e; k += blockDim.x) {
            uint32_t t = tids[k];
            range |= t >= m;
            order |= (k > b) && (t <= tids[k - 1]);
        }
        if (range)
            atomicOr(&flags[0], 1u);
        if (order)
            atomicOr(&flags[1], 1u);
    }
}

}  // namespace

hipError_t launch_expand_rows(const uint64_t *row_off, uint32_t m, uint32_t *row_of, hipStream_t s)
{
    // the kernel stores four row ids at a time at 16-byte aligned positions
    if (reinterpret_cast<uintptr_t>(row_of) & 15u)
        return hipErrorInvalidValue;
    expand_rows_kernel<<<blocks_for(((uint64_t)m + 63) / 64 * 64, 8192), kBlock, 0, s>>>(row_off, m, row_of);
    return hipGetLastError();
}

hipError_t launch_offsets_and_dups(const uint32_t *keys, const uint32_t *vals, uint64_t nnz, uint32_t n, uint64_t *off,
                                  uint32_t *n_dup, hipStream_t s)
{
    // the kernel reads keys and vals 16 bytes at a time
    if (((uintptr_t)keys | (uintptr_t)vals) & 15u)
        return hipErrorInvalidValue;
    offsets_and_dups_kernel<<<blocks_for(nnz / 4 + 4, 4096), kBlock, 0, s>>>(keys, vals, nnz, n, off, n_dup);
    return hipGetLastError();
}

hipError_t launch_check_offsets(const uint64_t *off, uint32_t m, uint32_t *flags, hipStream_t s)
{
    if (m <= 16384) {
        check_offsets_small_kernel<<<1, 1024, 0, s>>>(off, m, flags);
        return hipGetLastError();
    }
    hipError_t e = fill_u32(flags, 2, 0, s);
    if (e != hipSuccess)
        return e;
    check_offsets_kernel<<<blocks_for(m, 4096), kBlock, 0, s>>>(off, m, flags);
    return hipGetLastError();
}

hipError_t launch_check_items(const uint32_t *items, uint64_t nnz, uint32_t n, uint32_t *flag, hipStream_t s)
{
    if (nnz == 0)
        return hipSuccess;
    check_items_kernel<<<blocks_for(nnz, 4096), kBlock, 0, s>>>(items, nnz, n, flag);
    return hipGetLastError();
}

hipError_t launch_mark_dups(const uint32_t *keys, const uint32_t *vals, uint64_t nnz, uint32_t *keep,
                            uint32_t *n_dup, hipStream_t s)
{
    if (nnz == 0)
        return hipSuccess;
    mark_dups_kernel<<<blocks_for(nnz, 4096), kBlock, 0, s>>>(keys, vals, nnz, keep, n_dup);
    return hipGetLastError();
}

hipError_t launch_compact_pairs(const uint32_t *keys, const uint32_t *vals, const uint32_t *keep,
                                const uint64_t *pos, uint64_t nnz, uint32_t *ko, uint32_t *vo, hipStream_t s)
{
    if (nnz == 0)
        return hipSuccess;
    compact_pairs_kernel<<<blocks_for(nnz, 4096), kBlock, 0, s>>>(keys, vals, keep, pos, nnz, ko, vo);
    return hipGetLastError();
}

hipError_t launch_offsets_from_sorted(const uint32_t *keys, uint64_t nnz, uint32_t n, uint64_t *off, hipStream_t s)
{
    offsets_from_sorted_kernel<<<blocks_for(nnz + 1, 4096), kBlock, 0, s>>>(keys, nnz, n, off);
    return hipGetLastError();
}

hipError_t launch_validate_sets(const uint64_t *off, const uint32_t *tids, uint32_t n, uint64_t nnz, uint32_t m,
                                uint32_t *flags, hipStream_t s)
{
    (void)nnz;
    uint32_t g = n < 65536 ? n : 65536;
    validate_sets_kernel<<<g, kBlock, 0, s>>>(off, tids, n, m, flags);
    return hipGetLastError();
}

hipError_t launch_txn_bits(const uint64_t *row_off, const uint32_t *items, uint32_t m, uint32_t n, uint32_t lds,
                           uint32_t n_cu, uint32_t *bits, uint32_t *flag, hipStream_t s)
{
    const uint64_t ld = bit_row_words(m);
    const uint32_t tw = txn_bits_words(m, n, lds, n_cu);
    if (!bit_ingest_fits(m, n, lds, n_cu))
        return hipErrorInvalidValue;
    const uint32_t n_chunks = (uint32_t)((ld + tw - 1) / tw), per_xcd = (n_chunks + kXcds - 1) / kXcds;
    const uint32_t bytes = (n + 1) * (tw + 1) * 4;
    const void *f = tw == 8    ? reinterpret_cast<const void *>(txn_bits_kernel<8>)
                    : tw == 16 ? reinterpret_cast<const void *>(txn_bits_kernel<16>)
                               : reinterpret_cast<const void *>(txn_bits_kernel<32>);
    if (bytes > 32768) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess)
            return e;
    }
    const uint32_t grid = (uint32_t)txn_bits_blocks(m, tw);
    if (tw == 8)
        txn_bits_kernel<8><<<grid, kTxnBitsThreads, bytes, s>>>(row_off, items, m, n, ld, n_chunks, per_xcd, bits, flag);
    else if (tw == 16)
        txn_bits_kernel<16><<<grid, kTxnBitsThreads, bytes, s>>>(row_off, items, m, n, ld, n_chunks, per_xcd, bits,
                                                                 flag);
    else
        txn_bits_kernel<32><<<grid, kTxnBitsThreads, bytes, s>>>(row_off, items, m, n, ld, n_chunks, per_xcd, bits,
                                                                 flag);
    return hipGetLastError();
}

hipError_t launch_bit_count(const uint32_t *bits, uint32_t m, uint32_t n, uint32_t *count, hipStream_t s)
{
    const uint64_t ld = bit_row_words(m);
    const uint32_t n_seg = (uint32_t)((ld + kSegWords - 1) / kSegWords);
    bit_count_kernel<<<n * n_seg, 256, 0, s>>>(bits, ld, n_seg, count);
    return hipGetLastError();
}

hipError_t launch_bit_expand(const uint32_t *bits, uint32_t m, uint32_t n, const uint64_t *start, uint64_t *off,
                             uint32_t *tids, hipStream_t s)
{
    const uint64_t ld = bit_row_words(m);
    const uint32_t n_seg = (uint32_t)((ld + kSegWords - 1) / kSegWords);
    bit_expand_kernel<<<n * n_seg, 256, 0, s>>>(bits, ld, n, n_seg, start, off, tids);
    return hipGetLastError();
}

}  // namespace bm
