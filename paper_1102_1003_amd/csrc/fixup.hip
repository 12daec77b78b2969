// Failed-insertion correction (Sec. III-C) and support >= sigma filtering.
//
// Correction: for every failed insertion (a, b) -- tid b of item a that is in
// no table of B_a -- and every other item c whose tidlist holds b (c is in
// A_b, the transaction's items), the pair {a, c} lost exactly the shared
// element b in the slot compare and gains one back.  When c failed at b too,
// the pair is added once, from the smaller of a and c.  The pairs are built
// once per index as a list of (lo, hi) entries, one per lost shared element,
// and added into any later result.
#include "bm_internal.h"

namespace bm {

namespace {

constexpr int kBlock = 256;

__device__ inline uint64_t packed_index(uint64_t n, uint64_t i, uint64_t j)
{
    return i * n - i * (i + 1) / 2 + (j - i - 1);
}

__device__ inline int64_t find_tid(const uint32_t *a, uint64_t n, uint32_t x)
{
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        uint64_t mid = (lo + hi) >> 1;
        if (a[mid] < x)
            lo = mid + 1;
        else
            hi = mid;
    }
    return (lo < n && a[lo] == x) ? (int64_t)lo : -1;
}

// Thread per (failure f, item c).  cap == 0 only counts.  A workgroup's finds take
// their places by one atomic: one a wavefront, all on the same counter, was most of
// the pass (30,011 x 613: 23 us, now 11).
__global__ void __launch_bounds__(kBlock)
    corrections_kernel(const uint32_t *failed, uint32_t n_failed, const uint32_t *n_failed_dev, const uint64_t *off,
                       const uint32_t *tids, const uint32_t *failed_bits, const uint8_t *has_map, uint32_t n,
                       uint32_t *pairs, uint64_t cap, unsigned long long *count)
{
    __shared__ uint32_t found;
    __shared__ unsigned long long place;
    if (n_failed_dev)
        n_failed = min(n_failed, *n_failed_dev);
    const uint64_t total = (uint64_t)n_failed * n, stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t e0 = (uint64_t)blockIdx.x * kBlock; e0 < total; e0 += stride) {
        if (threadIdx.x == 0)
            found = 0;
        __syncthreads();
        const uint64_t e = e0 + threadIdx.x;
        uint32_t a = 0, c = 0, at = 0;
        bool hit = false;
        if (e < total) {
            const uint32_t f = (uint32_t)(e / n);
            c = (uint32_t)(e - (uint64_t)f * n);
            a = failed[2 * (uint64_t)f];
            const uint32_t b = failed[2 * (uint64_t)f + 1];
            const uint64_t o = off[c];
            const int64_t k = c != a && has_map[c] ? find_tid(tids + o, off[c + 1] - o, b) : -1;
            if (k >= 0) {
                const uint64_t kk = o + (uint64_t)k;
                // both failed at b: the failure of min(a, c) adds it
                hit = c > a || !((failed_bits[kk / 32] >> (kk % 32)) & 1u);
            }
        }
        if (hit)
            at = atomicAdd(&found, 1u);
        __syncthreads();
        if (threadIdx.x == 0 && found)
            place = atomicAdd(count, (unsigned long long)found);
        __syncthreads();
        if (hit && place + at < cap) {
            pairs[2 * (place + at)] = min(a, c);
            pairs[2 * (place + at) + 1] = max(a, c);
        }
    }
}

// Two families A (output rows) and B (output columns), out[i * n_b + j]:
// the pair (i, j) lost every shared element that failed in A_i or in B_j.
// Thread per (failure f of family X, item c of the other family Y): when
// the failed tid is in Y_c the pair gains one, unless the tid failed in Y_c
// too and X is B (then A's pass adds it).  x_is_a: X is A (the failure's
// item is the row).  failed_bits_y: Y's failed incidences (bit per tid of
// its tidlists), consulted only when X is B.
__global__ void cross_corrections_kernel(const uint32_t *failed, uint32_t n_failed, const uint64_t *off_y,
                                         const uint32_t *tids_y, uint32_t n_y, const uint32_t *failed_bits_y,
                                         uint32_t *out, uint64_t n_b, int x_is_a)
{
    const uint64_t total = (uint64_t)n_failed * n_y;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
        const uint32_t f = (uint32_t)(e / n_y), c = (uint32_t)(e % n_y);
        const uint32_t item = failed[2 * (uint64_t)f], t = failed[2 * (uint64_t)f + 1];
        const int64_t k = find_tid(tids_y + off_y[c], off_y[c + 1] - off_y[c], t);
        if (k < 0)
            continue;
        if (!x_is_a) {
            const uint64_t kk = off_y[c] + (uint64_t)k;
            if ((failed_bits_y[kk / 32] >> (kk % 32)) & 1u)
                continue;  // failed on both sides: counted from A's failure
        }
        const uint64_t cell = x_is_a ? (uint64_t)item * n_b + c : (uint64_t)c * n_b + item;
        atomicAdd(&out[cell], 1u);
    }
}

__global__ void apply_corrections_kernel(const uint32_t *pairs, uint64_t n_corr, uint32_t *out, uint64_t n)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_corr; e += stride)
        atomicAdd(&out[packed_index(n, pairs[2 * e], pairs[2 * e + 1])], 1u);
}

__global__ void apply_corrections_subset_kernel(const uint32_t *pairs, uint64_t n_corr, const uint32_t *pos_of_item,
                                                uint32_t *out, uint64_t k)
{
    uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n_corr; e += stride) {
        uint32_t pa = pos_of_item[pairs[2 * e]], pb = pos_of_item[pairs[2 * e + 1]];
        if (pa == kEmpty || pb == kEmpty)
            continue;
        uint32_t lo = pa < pb ? pa : pb, hi = pa < pb ? pb : pa;
        atomicAdd(&out[packed_index(k, lo, hi)], 1u);
    }
}

// --------------------------------------------------------------- threshold
constexpr int kThrItems = 16;
constexpr uint64_t kThrTile = (uint64_t)kBlock * kThrItems;

// A thread's words of the block's tile, kBlock apart (neighbouring lanes read and
// write neighbouring places), and which of them count: bit i, word i >= sigma.
__device__ inline uint32_t load_tile(const uint32_t *sup, uint64_t n, uint32_t sigma, uint32_t (&v)[kThrItems])
{
    const uint64_t base = (uint64_t)blockIdx.x * kThrTile + threadIdx.x;
    uint32_t hits = 0;
    if (base - threadIdx.x + kThrTile <= n) {
#pragma unroll
        for (int i = 0; i < kThrItems; i++)
            v[i] = sup[base + i * kBlock];
#pragma unroll
        for (int i = 0; i < kThrItems; i++)
            hits |= v[i] >= sigma ? 1u << i : 0u;
    } else {
#pragma unroll
        for (int i = 0; i < kThrItems; i++) {
            const bool in = base + i * kBlock < n;
            v[i] = in ? sup[base + i * kBlock] : 0u;
            hits |= in && v[i] >= sigma ? 1u << i : 0u;
        }
    }
    return hits;
}

// The tile's hits in order: each one's place in the tile and its count.
struct TileHits {
    uint32_t value[kThrTile];
    uint16_t at[kThrTile];
};

// Fills h and returns how many there are: gathered in LDS first, they are worked on
// and written by neighbouring lanes, whether few or all of the tile's words are hits
// (8 * 10^6 pairs, all kept: 37 us against 127 with sixteen consecutive words a
// thread; 2 * 10^6 of which 10^5 are kept: 9.1 against 11).
__device__ inline uint32_t tile_hits(const uint32_t *sup, uint64_t n, uint32_t sigma, TileHits &h)
{
    constexpr uint32_t kWaves = kBlock / 64;
    __shared__ uint32_t ahead[kThrItems * kWaves + 1];
    static_assert(kThrItems * kWaves == 64, "one wavefront scans them");
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x / 64;
    uint32_t v[kThrItems];
    const uint32_t hits = load_tile(sup, n, sigma, v);
#pragma unroll
    for (int i = 0; i < kThrItems; i++) {
        const unsigned long long b = __ballot(hits >> i & 1u);
        if (lane == 0)
            ahead[i * kWaves + wave] = __popcll(b);
    }
    __syncthreads();
    if (wave == 0) {
        const uint32_t mine = ahead[lane];
        uint32_t incl = mine;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = __shfl_up(incl, d, 64);
            incl += lane >= (uint32_t)d ? u : 0u;
        }
        ahead[lane] = incl - mine;
        if (lane == 63)
            ahead[64] = incl;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kThrItems; i++) {
        const unsigned long long b = __ballot(hits >> i & 1u);
        if (hits >> i & 1u) {
            const uint32_t to = ahead[i * kWaves + wave] + __popcll(b & ((1ull << lane) - 1));
            h.value[to] = v[i];
            h.at[to] = (uint16_t)(i * kBlock + threadIdx.x);
        }
    }
    __syncthreads();
    return ahead[64];
}

__global__ void __launch_bounds__(kBlock)
    threshold_count_kernel(const uint32_t *sup, uint64_t n_pairs, uint32_t sigma, uint32_t *block_counts)
{
    __shared__ uint32_t sum;
    if (threadIdx.x == 0)
        sum = 0;
    __syncthreads();
    uint32_t v[kThrItems];
    uint32_t c = __popc(load_tile(sup, n_pairs, sigma, v));
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
        c += __shfl_xor(c, d, 64);
    if ((threadIdx.x & 63) == 0)
        atomicAdd(&sum, c);
    __syncthreads();
    if (threadIdx.x == 0)
        block_counts[blockIdx.x] = sum;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        block_counts[gridDim.x] = 0;  // where the scan leaves the sum
}

// Row of packed index k in an n-item upper triangle: the root in fp32 (within one row
// for n < 2^23), then steps to the row itself.
__device__ inline uint32_t row_of_packed(uint64_t k, uint32_t n)
{
    const uint64_t a = 2ull * n - 1;
    const uint32_t root = (uint32_t)__builtin_amdgcn_sqrtf((float)(a * a - 8 * k));
    uint32_t i = min((uint32_t)(a - min((uint64_t)root, a)) / 2, n - 2);
    auto start = [n](uint32_t r) { return (uint64_t)r * n - (uint64_t)r * (r + 1) / 2; };
    while (i > 0 && start(i) > k)
        i--;
    while (i + 1 <= n - 2 && start(i + 1) <= k)
        i++;
    return i;
}

// Writes nothing when the total (block_off[n_blocks]) exceeds capacity, so the
// write can be queued before the host has read the total.
// ids: the item of each of the n positions (null: position p is item p).
// kSum: `block_off` holds the blocks' counts, not yet scanned: every block adds
// those before it and all of them (the first one leaves the sum after them for the
// caller), which for few blocks takes less than a scan's launch.
template <bool kSum>
__global__ void threshold_write_kernel(const uint32_t *sup, uint64_t n_pairs, uint64_t n, const uint32_t *ids,
                                       uint32_t sigma, const uint32_t *block_counts, uint64_t *block_off,
                                       uint32_t n_blocks, uint64_t capacity, bm_pair *out)
{
    uint64_t first;
    if constexpr (kSum) {
        __shared__ uint32_t sums[2];
        if (threadIdx.x < 2)
            sums[threadIdx.x] = 0;
        __syncthreads();
        uint32_t all = 0, ahead = 0;
        for (uint32_t b = threadIdx.x; b < n_blocks; b += kBlock) {
            const uint32_t c = block_counts[b];
            all += c;
            ahead += b < blockIdx.x ? c : 0u;
        }
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            all += __shfl_xor(all, d, 64);
            ahead += __shfl_xor(ahead, d, 64);
        }
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&sums[0], all);
            atomicAdd(&sums[1], ahead);
        }
        __syncthreads();
        if (blockIdx.x == 0 && threadIdx.x == 0)
            block_off[n_blocks] = sums[0];
        if (sums[0] > capacity)
            return;
        first = sums[1];
    } else {
        if (block_off[n_blocks] > capacity)
            return;  // the same value for every thread of the grid
        first = block_off[blockIdx.x];
    }
    __shared__ TileHits h;
    const uint32_t count = tile_hits(sup, n_pairs, sigma, h);
    for (uint32_t q = threadIdx.x; q < count; q += kBlock) {
        const uint64_t k = (uint64_t)blockIdx.x * kThrTile + h.at[q];
        const uint32_t row = row_of_packed(k, (uint32_t)n);
        bm_pair pr;
        pr.i = row;
        pr.j = (uint32_t)(row + 1 + (k - ((uint64_t)row * n - (uint64_t)row * (row + 1) / 2)));
        if (ids) {
            pr.i = ids[pr.i];
            pr.j = ids[pr.j];
        }
        pr.support = h.value[q];
        out[first + q] = pr;
    }
}

// The same compaction over a row-major rectangle of n_cols columns: entry k
// is the pair (k / n_cols, k % n_cols).
__global__ void threshold_write_rect_kernel(const uint32_t *sup, uint64_t n_cells, uint64_t n_cols, uint32_t sigma,
                                            const uint64_t *block_off, uint32_t n_blocks, uint64_t capacity,
                                            bm_pair *out)
{
    if (block_off[n_blocks] > capacity)
        return;  // the same value for every thread of the grid
    __shared__ TileHits h;
    const uint32_t count = tile_hits(sup, n_cells, sigma, h);
    for (uint32_t q = threadIdx.x; q < count; q += kBlock) {
        const uint64_t k = (uint64_t)blockIdx.x * kThrTile + h.at[q];
        bm_pair pr;
        pr.i = (uint32_t)(k / n_cols);
        pr.j = (uint32_t)(k % n_cols);
        pr.support = h.value[q];
        out[block_off[blockIdx.x] + q] = pr;
    }
}

// Subset query preparation: pos_of_item[item] = query position; flags repeats,
// out-of-range ids and items without a BatMap.
__global__ void subset_prepare_kernel(const uint32_t *items, uint32_t k, uint32_t n, const int32_t *sorted_pos,
                                      uint32_t *pos_of_item, uint32_t *flag)
{
    for (uint32_t p = blockIdx.x * blockDim.x + threadIdx.x; p < k; p += gridDim.x * blockDim.x) {
        uint32_t it = items[p];
        if (it >= n) {
            atomicOr(flag, 1u);
            continue;
        }
        if (sorted_pos[it] < 0)
            atomicOr(flag, 4u);
        uint32_t old = atomicExch(&pos_of_item[it], p);
        if (old != kEmpty)
            atomicOr(flag, 2u);
    }
}

}  // namespace

hipError_t launch_corrections(const uint32_t *failed, uint32_t n_failed, const uint32_t *n_failed_dev,
                              const uint64_t *off, const uint32_t *tids, const uint32_t *failed_bits,
                              const uint8_t *has_map, uint32_t n, uint32_t *pairs, uint64_t cap,
                              unsigned long long *count, hipStream_t s)
{
    uint64_t total = (uint64_t)n_failed * n;
    if (total == 0)
        return hipSuccess;
    // a count read on the device is usually far below the bound n_failed:
    // one full-occupancy grid strides over whatever it is
    const uint64_t max_blocks = n_failed_dev ? 2048 : (1u << 20);
    const uint64_t blocks = std::min<uint64_t>((total + kBlock - 1) / kBlock, max_blocks);
    corrections_kernel<<<(uint32_t)blocks, kBlock, 0, s>>>(failed, n_failed, n_failed_dev, off, tids, failed_bits,
                                                            has_map, n, pairs, cap, count);
    return hipGetLastError();
}

hipError_t launch_cross_corrections(const uint32_t *failed, uint32_t n_failed, const uint64_t *off_y,
                                    const uint32_t *tids_y, uint32_t n_y, const uint32_t *failed_bits_y, uint32_t *out,
                                    uint64_t n_b, bool x_is_a, hipStream_t s)
{
    const uint64_t total = (uint64_t)n_failed * n_y;
    if (total == 0)
        return hipSuccess;
    uint64_t blocks = (total + kBlock - 1) / kBlock;
    if (blocks > (1u << 20))
        blocks = 1u << 20;
    cross_corrections_kernel<<<(uint32_t)blocks, kBlock, 0, s>>>(failed, n_failed, off_y, tids_y, n_y, failed_bits_y,
                                                                  out, n_b, x_is_a ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_threshold_write_rect(const uint32_t *sup, uint64_t n_cells, uint64_t n_cols, uint32_t sigma,
                                       const uint64_t *block_off, uint32_t n_blocks, uint64_t capacity, bm_pair *out,
                                       hipStream_t s)
{
    if (n_blocks == 0)
        return hipSuccess;
    threshold_write_rect_kernel<<<n_blocks, kBlock, 0, s>>>(sup, n_cells, n_cols, sigma, block_off, n_blocks,
                                                             capacity, out);
    return hipGetLastError();
}

hipError_t launch_apply_corrections(const uint32_t *pairs, uint64_t n_corr, uint32_t *out, uint64_t n, hipStream_t s)
{
    if (n_corr == 0)
        return hipSuccess;
    uint64_t blocks = (n_corr + kBlock - 1) / kBlock;
    if (blocks > 65536)
        blocks = 65536;
    apply_corrections_kernel<<<(uint32_t)blocks, kBlock, 0, s>>>(pairs, n_corr, out, n);
    return hipGetLastError();
}

hipError_t launch_apply_corrections_subset(const uint32_t *pairs, uint64_t n_corr, const uint32_t *pos_of_item,
                                           uint32_t *out, uint64_t k, hipStream_t s)
{
    if (n_corr == 0)
        return hipSuccess;
    uint64_t blocks = (n_corr + kBlock - 1) / kBlock;
    if (blocks > 65536)
        blocks = 65536;
    apply_corrections_subset_kernel<<<(uint32_t)blocks, kBlock, 0, s>>>(pairs, n_corr, pos_of_item, out, k);
    return hipGetLastError();
}

uint32_t threshold_blocks(uint64_t n_pairs) { return (uint32_t)((n_pairs + kThrTile - 1) / kThrTile); }

hipError_t launch_threshold_count(const uint32_t *sup, uint64_t n_pairs, uint32_t sigma, uint32_t *block_counts,
                                  uint32_t n_blocks, hipStream_t s)
{
    if (n_blocks == 0)
        return hipSuccess;
    threshold_count_kernel<<<n_blocks, kBlock, 0, s>>>(sup, n_pairs, sigma, block_counts);
    return hipGetLastError();
}

hipError_t launch_threshold_write(const uint32_t *sup, uint64_t n_pairs, uint64_t n, const uint32_t *ids,
                                  uint32_t sigma, const uint32_t *block_counts, uint64_t *block_off, uint32_t n_blocks,
                                  uint64_t capacity, bm_pair *out, hipStream_t s)
{
    if (n_blocks == 0)
        return hipSuccess;
    auto *kernel = block_counts ? threshold_write_kernel<true> : threshold_write_kernel<false>;
    kernel<<<n_blocks, kBlock, 0, s>>>(sup, n_pairs, n, ids, sigma, block_counts, block_off, n_blocks, capacity, out);
    return hipGetLastError();
}

hipError_t launch_subset_prepare(const uint32_t *items, uint32_t k, uint32_t n, const int32_t *sorted_pos,
                                 uint32_t *pos_of_item, uint32_t *flag, hipStream_t s)
{
    uint32_t blocks = (k + kBlock - 1) / kBlock;
    if (blocks == 0)
        return hipSuccess;
    subset_prepare_kernel<<<blocks, kBlock, 0, s>>>(items, k, n, sorted_pos, pos_of_item, flag);
    return hipGetLastError();
}

}  // namespace bm
