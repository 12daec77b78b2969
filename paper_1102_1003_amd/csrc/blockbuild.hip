// Construction with the block family of permutations (8-bit maps of order
// two).  With pi_t(x) = H r_0 + beta_{t,H}(a) for y = sigma(x) = H r_0 + a,
// every hash value of an element in a map of width r_i = R r_0 falls in the
// same block j = H mod R of the Fig. 4 layout in all three tables, and that
// block is 3 r_0 consecutive slots of the map.  So the map is built block by
// block: the elements are first bucketed by (map, block), then one workgroup
// per block runs the whole of Sec. II-A and Fig. 3 for it in LDS (insertion
// by exchanges, MaxLoop, the failure policy, the indicators) and writes the
// block's bit-sliced bytes straight to the arena.  No device-wide atomics
// take part in the insertion.
#include <algorithm>
#include <cstring>

#include "bm_internal.h"

namespace bm {

namespace {

constexpr uint32_t kEmptyCode = 0x7Fu;
constexpr uint32_t kMaxBlocksH = kBlockKeysH;
constexpr uint32_t kBlockFailCap = 1024;  // nestless elements one block may leave
constexpr int kBucketThreads = 256;
constexpr int kBucketPer = kBucketChunk / kBucketThreads;

struct BlockHead {
    uint32_t count;  // nestless elements
    uint32_t pad[3];  // keeps the code bytes after it 16-byte aligned
    uint32_t elem[kBlockFailCap];
};

size_t block_lds_bytes(uint32_t r0)
{
    return sizeof(BlockHead) + 3ull * r0 + 3ull * r0 / 8;
}

// beta_{t,H}'s keys of every block (H < 128: m <= 127 r_0) and table, made on
// the host and kept in LDS by each workgroup of the build: x = m1 | m2 << 16,
// y = c1 | c2 << 16, z = i1 | i2 << 16 (all below 2^15).
inline uint4 pack_key(const BetaKey &k)
{
    return make_uint4(k.m1 | (k.m2 << 16), k.c1 | (k.c2 << 16), k.i1 | (k.i2 << 16), 0u);
}

__device__ inline BetaKey unpack_key(uint4 w)
{
    BetaKey k;
    k.m1 = w.x & 0xFFFFu;
    k.m2 = w.x >> 16;
    k.c1 = w.y & 0xFFFFu;
    k.c2 = w.y >> 16;
    k.i1 = w.z & 0xFFFFu;
    k.i2 = w.z >> 16;
    return k;
}

// Byte i of the LDS tables set to v; returns the byte it held.  One masked
// exchange (clear the mask's bits, set v's, return the word): a compare-and-swap
// loop needs a read before it and a round for every neighbour that changed (large
// Zipf build 663 us; with this, keys from the host, the next copy loaded ahead and
// byte reads 530).
__device__ inline uint32_t lds_swap_byte(uint32_t *W, uint32_t i, uint32_t v)
{
    typedef __attribute__((address_space(3))) uint32_t LdsWord;
    const uint32_t at = (uint32_t)(uintptr_t)(LdsWord *)W + (i & ~3u), sh = (i & 3u) * 8u;
    uint32_t old;
    asm volatile("ds_mskor_rtn_b32 %0, %1, %2, %3\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(old)
                 : "v"(at), "v"(0xFFu << sh), "v"(v << sh)
                 : "memory");
    return (old >> sh) & 0xFFu;
}

// Byte i emptied if it holds v.
__device__ inline void lds_clear_byte(uint32_t *W, uint32_t i, uint32_t v)
{
    uint32_t *w = W + (i >> 2);
    const uint32_t sh = (i & 3u) * 8u;
    uint32_t old = *w;
    while (((old >> sh) & 0xFFu) == v) {
        const uint32_t prev = atomicCAS(w, old, (old & ~(0xFFu << sh)) | (kEmptyCode << sh));
        if (prev == old)
            break;
        old = prev;
    }
}

__device__ inline uint32_t lds_get_byte(const uint32_t *W, uint32_t i)
{
    return reinterpret_cast<const uint8_t *>(W)[i];
}

__device__ inline int64_t find_sorted(const uint32_t *a, uint64_t n, uint32_t x)
{
    uint64_t lo = 0, hi = n;
    while (lo < hi) {
        const uint64_t mid = (lo + hi) >> 1;
        if (a[mid] < x)
            lo = mid + 1;
        else
            hi = mid;
    }
    return (lo < n && a[lo] == x) ? (int64_t)lo : -1;
}

// What the build's other kernels start from, in one launch (five took 10 us of
// a build's 90 at m = 10^4, n = 200, each over in 2 us): see BlockPrep.  The last
// threads of the grid take the maps, the first ones the first hops.
__global__ void block_prep_kernel(BlockPrep a, BlockPerm B)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, nt = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t w = i0; w < a.failed_words; w += nt)
        a.failed_bits[w] = 0;
    for (uint64_t w = i0; w < a.zeroed_words; w += nt)
        a.zeroed[w] = 0;
    for (uint64_t p = nt - 1 - i0; p < a.n; p += nt) {
        const uint32_t item = a.sorted_items[p];
        const bool built = p >= a.first;
        a.sorted_pos[item] = built ? (int32_t)p : -1;
        a.has_map[item] = built;
        if (built && a.bucket_map) {
            const uint64_t b1 = a.goff[p + 1] / a.gb;
            for (uint64_t b = a.goff[p] / a.gb; b < b1; b++)
                a.bucket_map[b] = (uint32_t)p;
        }
    }
    // hops[(t n_blocks + H) r_0 + beta_{t,H}(a)] = beta_{t+1,H}(a)
    for (uint64_t x = a.hops ? i0 : B.m; x < B.m; x += nt) {  // H r_0 + a
        const uint32_t H = (uint32_t)x >> B.l0, len = block_len(B, H);
        uint32_t pos[3];
#pragma unroll
        for (uint32_t t = 0; t < 3; t++)
            pos[t] = beta_fwd(B, unpack_key(a.keys[t * kMaxBlocksH + H]), (uint32_t)x & B.mask, len);
#pragma unroll
        for (uint32_t t = 0; t < 3; t++)
            a.hops[((t * B.n_blocks + H) << B.l0) + pos[t]] = (uint16_t)pos[t == 2 ? 0 : t + 1];
    }
}

// The chunk's elements, relabelled, and their blocks within the map.
struct ChunkView {
    const uint32_t *T;  // the map's tidlist
    uint32_t e0, e1;    // this chunk's part of it
    uint32_t R;         // blocks of the map (a power of two)
    uint64_t b0;        // the map's first block
};

__device__ inline ChunkView chunk_view(const BucketChunk &c, const uint32_t *tids, const uint64_t *off,
                                       const uint32_t *sorted_items, const uint32_t *r_sorted, const uint64_t *goff,
                                       uint32_t gb, uint32_t l0)
{
    const uint32_t item = sorted_items[c.p];
    const uint64_t base = off[item];
    const uint32_t size = (uint32_t)(off[item + 1] - base);
    ChunkView v;
    v.T = tids + base;
    v.e0 = c.e0;
    v.e1 = min(c.e0 + kBucketChunk, size);
    v.R = r_sorted[c.p] >> l0;
    v.b0 = goff[c.p] / gb;
    return v;
}

// This thread's elements of the chunk (0 past its end), all on their way at once: a
// whole chunk's without a test each, which would make one wait for the other.
__device__ inline void load_chunk(const ChunkView &v, uint32_t (&x)[kBucketPer])
{
    const uint32_t *t = v.T + v.e0 + threadIdx.x;
    if (v.e1 - v.e0 == kBucketChunk) {
#pragma unroll
        for (int k = 0; k < kBucketPer; k++)
            x[k] = t[k * kBucketThreads];
    } else {
#pragma unroll
        for (int k = 0; k < kBucketPer; k++)
            x[k] = v.e0 + k * kBucketThreads + threadIdx.x < v.e1 ? t[k * kBucketThreads] : 0u;
    }
}

// Counts per block: a histogram of the chunk in LDS (a map has at most 256
// blocks, since r_i <= 2 * 2^ceil(log2 m) and m <= 127 r_0; one of R blocks counts
// each in 256 / R words, a lane to each, since 64 lanes that add to a few words
// wait for one another), then an atomic per nonempty block.  4 * 10^7 elements,
// Zipf: 51 us, 3.1 TB/s (76 with one word a block and a load a step).
template <bool K24>
__global__ void __launch_bounds__(kBucketThreads)
    bucket_count_kernel(const BucketChunk *chunks, const uint32_t *__restrict__ tids, const uint64_t *off,
                        const uint32_t *sorted_items, const uint32_t *r_sorted, const uint64_t *goff, uint32_t gb,
                        BlockPerm B, uint32_t *count)
{
    __shared__ uint32_t hist[256];
    const ChunkView v = chunk_view(chunks[blockIdx.x], tids, off, sorted_items, r_sorted, goff, gb, B.l0);
    hist[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t rep = 256u / v.R, own = threadIdx.x & (rep - 1u);
    uint32_t xs[kBucketPer];
    load_chunk(v, xs);
#pragma unroll
    for (int k = 0; k < kBucketPer; k++)
        if (v.e0 + k * kBucketThreads + threadIdx.x < v.e1)
            atomicAdd(&hist[((perm_eval_k<K24>(B.sig, 0, xs[k]) >> B.l0) & (v.R - 1u)) * rep + own], 1u);
    __syncthreads();
    const uint32_t fold = min(rep, 64u);
    uint32_t sum = hist[threadIdx.x];
    for (uint32_t o = 1; o < fold; o <<= 1)
        sum += __shfl_xor(sum, o, 64);
    if (threadIdx.x % fold == 0 && sum)
        atomicAdd(&count[v.b0 + threadIdx.x / rep], sum);
}

// The chunk's y values into their blocks' runs: ranked per block and put in
// block order in LDS, the chunk reserves its part of each run with one atomic,
// and the values leave in that order, neighbouring lanes to neighbouring words
// (4 * 10^7 elements, Zipf: 70 us, 4.5 TB/s, as fast as a copy; 100 with one counter
// a block; written straight from the tidlist's order, a wavefront's 64 stores went
// to as many lines: 160).
//
// kWhole: every map is one chunk (its elements from ebase[p] on), so the chunk's own
// counts are the runs: nothing is counted or scanned before, and the blocks' starts
// and maps are written here (30,011 x 613: 8 us, against 23 for count, scan and scatter).
template <bool K24, bool kWhole>
__global__ void __launch_bounds__(kBucketThreads)
    bucket_scatter_kernel(const BucketChunk *chunks, const uint32_t *ebase, uint32_t p_first,
                          const uint32_t *__restrict__ tids, const uint64_t *off, const uint32_t *sorted_items,
                          const uint32_t *r_sorted, const uint64_t *goff, uint32_t gb, BlockPerm B, uint32_t *bstart,
                          uint32_t *cursor, uint32_t *bucket_map, uint32_t *__restrict__ bk)
{
    __shared__ uint32_t hist[256], shift[256];  // shift: run position minus position in `vals`
    __shared__ uint32_t wsum[kBucketThreads / 64];
    __shared__ uint32_t vals[kBucketChunk];
    static_assert(kBucketThreads == 256, "one thread per block of a map");
    const BucketChunk c = kWhole ? BucketChunk{p_first + blockIdx.x, 0} : chunks[blockIdx.x];
    const ChunkView v = chunk_view(c, tids, off, sorted_items, r_sorted, goff, gb, B.l0);
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x / 64u;
    const uint32_t rep = 256u / v.R, own = threadIdx.x & (rep - 1u);
    hist[threadIdx.x] = 0;
    __syncthreads();
    uint32_t ys[kBucketPer], rank[kBucketPer];
    load_chunk(v, ys);
#pragma unroll
    for (int k = 0; k < kBucketPer; k++) {
        const uint32_t e = v.e0 + k * kBucketThreads + threadIdx.x;
        if (e < v.e1) {
            ys[k] = perm_eval_k<K24>(B.sig, 0, ys[k]);
            rank[k] = atomicAdd(&hist[((ys[k] >> B.l0) & (v.R - 1u)) * rep + own], 1u);
        }
    }
    __syncthreads();
    const uint32_t part = hist[threadIdx.x];
    uint32_t incl = part;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o, 64);
        incl += lane >= (uint32_t)o ? up : 0u;
    }
    if (lane == 63)
        wsum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - part;
#pragma unroll
    for (uint32_t w = 0; w < kBucketThreads / 64; w++)
        before += w < wave ? wsum[w] : 0u;
    hist[threadIdx.x] = before;
    __syncthreads();
    const uint32_t j = threadIdx.x, first = j < v.R ? hist[j * rep] : 0u;  // block j's place in `vals`
    if constexpr (kWhole) {
        const uint32_t e0 = ebase[c.p];
        if (j < v.R) {
            bstart[v.b0 + j] = e0 + first;
            bucket_map[v.b0 + j] = c.p;
        }
        if (blockIdx.x == gridDim.x - 1 && j == 0)
            bstart[v.b0 + v.R] = e0 + v.e1;
        shift[j] = e0;
    } else if (j < v.R) {
        const uint32_t mine = (j + 1 < v.R ? hist[(j + 1) * rep] : v.e1 - v.e0) - first;
        shift[j] = (mine ? bstart[v.b0 + j] + atomicAdd(&cursor[v.b0 + j], mine) : 0u) - first;
    }
#pragma unroll
    for (int k = 0; k < kBucketPer; k++) {
        const uint32_t e = v.e0 + k * kBucketThreads + threadIdx.x;
        if (e < v.e1)
            vals[hist[((ys[k] >> B.l0) & (v.R - 1u)) * rep + own] + rank[k]] = ys[k];
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < v.e1 - v.e0; i += kBucketThreads) {
        const uint32_t y = vals[i];
        bk[shift[(y >> B.l0) & (v.R - 1u)] + i] = y;
    }
}

// One workgroup per block of 3 r_0 slots (tables 0, 1, 2 of r_0 positions
// each, in the order of the Fig. 4 layout).  LDS holds the block's code bytes
// (0x7F when empty): the code pi >> s and the position fix pi, so an evicted
// element is recovered by inverting beta, with no staging of tids.
//
// kHops: `hops` holds, for a copy at position pos of table t in a block of H's,
// its position in the next table (block_prep_kernel); one load then takes the
// place of two keys, beta's inverse and beta.  A chain's moves wait for one
// another, so in small builds, where the longest chains (failures: 3 MaxLoop moves)
// are what the launch takes, a move's latency is all that counts.
template <bool kHops>
__global__ void __launch_bounds__(1024)
    block_build_kernel(const uint32_t *__restrict__ bk, const uint32_t *__restrict__ bstart,
                       const uint32_t *__restrict__ bucket_map, const uint64_t *__restrict__ goff,
                       const uint32_t *__restrict__ sorted_items, const uint32_t *__restrict__ r_sorted,
                       const uint32_t *__restrict__ tids, const uint64_t *__restrict__ off, BlockPerm B,
                       const uint4 *__restrict__ keys, const uint16_t *__restrict__ hops, uint32_t shift,
                       uint32_t max_loop, uint32_t *__restrict__ arena, uint32_t *failed_bits, uint32_t *failed, uint32_t *n_failed,
                       uint32_t fail_cap, uint32_t *overflow)
{
    extern __shared__ uint32_t lds_dyn[];
    __shared__ uint4 KT[3 * kMaxBlocksH];  // beta_{t,H}'s keys at t * kMaxBlocksH + H
    BlockHead &Hd = *reinterpret_cast<BlockHead *>(lds_dyn);
    const uint32_t b = blockIdx.x;
    const uint32_t p = bucket_map[b];
    const uint32_t r0 = 1u << B.l0;
    const uint32_t gb = 3u * r0 / kSlotsPerGroup;
    uint32_t *W = lds_dyn + sizeof(BlockHead) / 4;  // 3 r0 code bytes
    uint32_t *IND = W + 3u * r0 / 4u;               // their indicator bits
    const uint32_t *Y = bk + bstart[b];
    const uint32_t n_el = bstart[b + 1] - bstart[b];
    const uint32_t csh = B.l0 - shift;  // code = H << csh | pos >> shift

    // the lanes' first copies and the keys are on their way while the tables are cleared
    const uint32_t nt = blockDim.x, copies = 2u * n_el;
    uint32_t c = threadIdx.x, y_next = c < copies ? Y[c >> 1] : 0u;
    for (uint32_t i = threadIdx.x; i < 3u * kMaxBlocksH; i += nt)
        KT[i] = keys[i];
    for (uint32_t i = threadIdx.x * 4; i < 3u * r0 / 4u; i += nt * 4)
        *reinterpret_cast<uint4 *>(W + i) = make_uint4(0x7F7F7F7Fu, 0x7F7F7F7Fu, 0x7F7F7F7Fu, 0x7F7F7F7Fu);
    for (uint32_t i = threadIdx.x; i < 3u * r0 / 32u; i += nt)
        IND[i] = 0;
    if (threadIdx.x == 0)
        Hd.count = 0;
    __syncthreads();

    // Insertion (Sec. II-A).  Copy c of the block is chain c mod 2 of element
    // c / 2, entering at A_1 or A_2 and then cycling through the tables; a
    // lane takes its next copy (loaded while it worked on the one before) as
    // soon as its chain ends.  An exchange with the element's own other copy
    // just passes the chain on.
    {
        const uint32_t steps = 3u * max_loop;
        uint32_t H = 0, pos = 0, tb = 0, left = 0;  // the copy in hand: its block and position in table tb
        bool busy = false;
        for (;;) {
            if (!busy) {
                if (c >= copies)
                    break;
                H = y_next >> B.l0;
                tb = c & 1u;
                pos = beta_fwd(B, unpack_key(KT[tb * kMaxBlocksH + H]), y_next & B.mask, block_len(B, H));
                left = steps;
                busy = true;
                c += nt;
                y_next = c < copies ? Y[c >> 1] : 0u;
            }
            if (left == 0) {
                const uint32_t slot = atomicAdd(&Hd.count, 1u);
                if (slot < kBlockFailCap)
                    Hd.elem[slot] = (H << B.l0) | beta_inv(B, unpack_key(KT[tb * kMaxBlocksH + H]), pos,
                                                           block_len(B, H));
                busy = false;
                continue;
            }
            const uint32_t old = lds_swap_byte(W, tb * r0 + pos, (H << csh) | (pos >> shift));
            if (old == kEmptyCode) {
                busy = false;
            } else {
                const uint32_t tn = tb == 2u ? 0u : tb + 1u;
                H = old >> csh;
                if constexpr (kHops) {
                    pos = hops[((tb * B.n_blocks + H) << B.l0) + pos];
                } else {
                    const uint32_t len = block_len(B, H);
                    const uint32_t a = beta_inv(B, unpack_key(KT[tb * kMaxBlocksH + H]), pos, len);
                    pos = beta_fwd(B, unpack_key(KT[tn * kMaxBlocksH + H]), a, len);
                }
                tb = tn;
                left--;
            }
        }
    }
    __syncthreads();
    const uint32_t nf = Hd.count;
    if (nf > kBlockFailCap) {
        // too many nestless elements to resolve here: the host builds the
        // index again with the chain family
        if (threadIdx.x == 0)
            atomicOr(overflow, 1u);
        return;
    }

    // failures: delete the remaining copy, record the element once
    const uint32_t item = sorted_items[p];
    const uint64_t e_first = off[item];
    const uint32_t size = (uint32_t)(off[item + 1] - e_first);
    for (uint32_t f = threadIdx.x; f < nf; f += blockDim.x) {
        const uint32_t y = Hd.elem[f];
        const uint32_t H = y >> B.l0;
        for (uint32_t t = 0; t < 3; t++) {
            const uint32_t pos = beta_fwd(B, unpack_key(KT[t * kMaxBlocksH + H]), y & B.mask, block_len(B, H));
            lds_clear_byte(W, t * r0 + pos, (H << csh) | (pos >> shift));
        }
        const uint32_t x = perm_inverse_lane(B.sig, 0, y);  // failures are few: 32-bit multiplies
        const int64_t k = find_sorted(tids + e_first, size, x);
        if (k < 0)
            continue;  // cannot happen: x came from this set
        const uint64_t kk = e_first + (uint64_t)k;
        const uint32_t bit = 1u << (kk % 32);
        const uint32_t prev = atomicOr(&failed_bits[kk / 32], bit);
        if (!(prev & bit)) {
            const uint32_t slot = atomicAdd(n_failed, 1u);
            if (slot < fail_cap) {
                failed[2 * (uint64_t)slot] = item;
                failed[2 * (uint64_t)slot + 1] = x;
            }
        }
    }
    __syncthreads();

    // Indicators (Fig. 3), by element: the copy in table t is flagged when the
    // other copy sits in table t - 1 (mod 3).  A placed element has exactly
    // two copies, so exactly one of them is flagged; a failed one has none.
    for (uint32_t e = threadIdx.x; e < n_el; e += blockDim.x) {
        const uint32_t y = Y[e];
        const uint32_t H = y >> B.l0;
        uint32_t pos[3];
        bool in[3];
        const uint32_t len = block_len(B, H);
#pragma unroll
        for (int t = 0; t < 3; t++) {
            const uint32_t q = beta_fwd(B, unpack_key(KT[t * kMaxBlocksH + H]), y & B.mask, len);
            pos[t] = (uint32_t)t * r0 + q;
            in[t] = lds_get_byte(W, pos[t]) == ((H << csh) | (q >> shift));
        }
#pragma unroll
        for (int t = 0; t < 3; t++)
            if (in[t] && in[t == 0 ? 2 : t - 1])
                atomicOr(&IND[pos[t] >> 5], 1u << (pos[t] & 31u));
    }
    __syncthreads();

    // Encoding: a wavefront per 8 groups (256 slots), lane = (group, plane).
    // Plane b < 7 gathers bit b of the group's 32 code bytes, eight at a time by
    // two dot products with 1, 2, 4, 8 and 16 .. 128 (2^b times the eight bits);
    // plane 7 is the group's indicator word.
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64u);
    const uint32_t n_waves = blockDim.x / 64u;
    const uint32_t plane = lane & 7u;
    const uint64_t g_first = goff[p] + (uint64_t)(b - goff[p] / gb) * gb;
    uint32_t *out = arena + g_first * kWordsPerGroup;
    for (uint32_t v0 = wave * 256u; v0 < 3u * r0; v0 += n_waves * 256u) {
        const uint32_t v = v0 + (lane >> 3) * kSlotsPerGroup;
        if (v < 3u * r0) {
            const uint8_t *src = reinterpret_cast<const uint8_t *>(W) + v;
            const uint4 lo = *reinterpret_cast<const uint4 *>(src);
            const uint4 hi = *reinterpret_cast<const uint4 *>(src + 16);
            const uint32_t d[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
            const uint32_t bit = 0x01010101u << plane;
            uint32_t word = 0;
#pragma unroll
            for (int k = 0; k < 8; k += 2) {
                const uint32_t low = __builtin_amdgcn_udot4(d[k] & bit, 0x08040201u, 0u, false);
                word |= __builtin_amdgcn_udot4(d[k + 1] & bit, 0x80402010u, low, false) >> plane << (4 * k);
            }
            if (plane == 7u)
                word = IND[v >> 5];
            out[(uint64_t)(v / kSlotsPerGroup) * kWordsPerGroup + plane] = word;
        }
    }
}

__global__ void gen_block_perms_kernel(BlockPerm B, uint32_t *out)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t x = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; x < B.m; x += stride) {
        const uint32_t y = perm_eval(B.sig, 0, (uint32_t)x);
#pragma unroll
        for (int t = 0; t < 3; t++)
            out[(uint64_t)t * B.m + x] = block_pi(B, t, y);
    }
}

int block_lds_limit()
{
    static int limit = -1;
    if (limit < 0) {
        // the kernels' static LDS (their key table) comes out of the same budget
        int dev = 0, bytes = 0;
        limit = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) == hipSuccess) {
            int dyn = bytes;
            bool good = true;
            for (const void *f : {reinterpret_cast<const void *>(block_build_kernel<false>),
                                  reinterpret_cast<const void *>(block_build_kernel<true>)}) {
                hipFuncAttributes attr;
                good = good && hipFuncGetAttributes(&attr, f) == hipSuccess && bytes > (int)attr.sharedSizeBytes;
                if (good)
                    dyn = std::min(dyn, bytes - (int)attr.sharedSizeBytes);
            }
            for (const void *f : {reinterpret_cast<const void *>(block_build_kernel<false>),
                                  reinterpret_cast<const void *>(block_build_kernel<true>)})
                good = good && hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn) == hipSuccess;
            if (good)
                limit = dyn;
        }
        (void)hipGetLastError();
    }
    return limit;
}

}  // namespace

uint32_t block_build_max_r0()
{
    uint32_t r = 0;
    for (uint32_t c = kMinR0; c <= kBlockMaxR0; c <<= 1)
        if (block_lds_bytes(c) <= (uint64_t)block_lds_limit())
            r = c;
    return r;
}

BlockPerm make_block_perm(uint32_t m, uint32_t l0, uint64_t seed)
{
    BlockPerm B;
    memset(&B, 0, sizeof(B));
    B.sig = make_perm_spec(m, seed ^ 0x5161A7E1B10Cull);
    B.m = m;
    B.l0 = l0;
    B.mask = (1u << l0) - 1u;
    B.h = (l0 + 1) / 2;
    B.n_blocks = (uint32_t)(((uint64_t)m + B.mask) >> l0);
    B.last_len = m - ((B.n_blocks - 1u) << l0);
    uint64_t x = seed ^ 0xB10CB10Cull;
    auto next = [&x]() {  // splitmix64
        uint64_t z = (x += 0x9E3779B97F4A7C15ull);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    };
    for (int t = 0; t < 3; t++) {
        B.key1[t] = (uint32_t)next();
        B.key2[t] = (uint32_t)next();
    }
    return B;
}

void make_block_keys(const BlockPerm &B, uint4 *keys)
{
    for (uint32_t t = 0; t < 3; t++)
        for (uint32_t H = 0; H < kMaxBlocksH; H++)
            keys[t * kMaxBlocksH + H] =
                H < B.n_blocks ? pack_key(beta_key(B, H, B.key1[t], B.key2[t])) : make_uint4(0, 0, 0, 0);
}

uint64_t block_hops_entries(const BlockPerm &B) { return 3ull * B.n_blocks << B.l0; }

hipError_t launch_block_prep(const BlockPrep &a, const BlockPerm &B, hipStream_t s)
{
    const uint64_t most = std::max({(uint64_t)a.n, a.failed_words / 4, a.zeroed_words / 4, a.hops ? (uint64_t)B.m : 0});
    block_prep_kernel<<<(uint32_t)std::min<uint64_t>((most + 255) / 256, 2048), 256, 0, s>>>(a, B);
    return hipGetLastError();
}

hipError_t launch_bucket_count(const BucketChunk *chunks, uint32_t n_chunks, const uint32_t *tids,
                               const uint64_t *off, const uint32_t *sorted_items, const uint32_t *r_sorted,
                               const uint64_t *goff, uint32_t gb, const BlockPerm &B, uint32_t *count, hipStream_t s)
{
    if (n_chunks == 0)
        return hipSuccess;
    if (B.sig.mask <= 0xFFFFFFu)
        bucket_count_kernel<true><<<n_chunks, kBucketThreads, 0, s>>>(chunks, tids, off, sorted_items, r_sorted, goff,
                                                                      gb, B, count);
    else
        bucket_count_kernel<false><<<n_chunks, kBucketThreads, 0, s>>>(chunks, tids, off, sorted_items, r_sorted,
                                                                       goff, gb, B, count);
    return hipGetLastError();
}

hipError_t launch_bucket_scatter(const BucketChunk *chunks, uint32_t n_chunks, const uint32_t *tids,
                                 const uint64_t *off, const uint32_t *sorted_items, const uint32_t *r_sorted,
                                 const uint64_t *goff, uint32_t gb, const BlockPerm &B, uint32_t *bstart,
                                 uint32_t *cursor, uint32_t *bk, hipStream_t s)
{
    if (n_chunks == 0)
        return hipSuccess;
    auto *kernel =
        B.sig.mask <= 0xFFFFFFu ? bucket_scatter_kernel<true, false> : bucket_scatter_kernel<false, false>;
    kernel<<<n_chunks, kBucketThreads, 0, s>>>(chunks, nullptr, 0, tids, off, sorted_items, r_sorted, goff, gb, B,
                                               bstart, cursor, nullptr, bk);
    return hipGetLastError();
}

hipError_t launch_bucket_whole(const uint32_t *ebase, uint32_t p_first, uint32_t n, const uint32_t *tids,
                               const uint64_t *off, const uint32_t *sorted_items, const uint32_t *r_sorted,
                               const uint64_t *goff, uint32_t gb, const BlockPerm &B, uint32_t *bstart,
                               uint32_t *bucket_map, uint32_t *bk, hipStream_t s)
{
    if (p_first >= n)
        return hipSuccess;
    auto *kernel = B.sig.mask <= 0xFFFFFFu ? bucket_scatter_kernel<true, true> : bucket_scatter_kernel<false, true>;
    kernel<<<n - p_first, kBucketThreads, 0, s>>>(nullptr, ebase, p_first, tids, off, sorted_items, r_sorted, goff,
                                                  gb, B, bstart, nullptr, bucket_map, bk);
    return hipGetLastError();
}

hipError_t launch_block_build(const uint32_t *bk, const uint32_t *bstart, const uint32_t *bucket_map,
                              uint32_t n_blocks, const uint64_t *goff, const uint32_t *sorted_items,
                              const uint32_t *r_sorted, const uint32_t *tids, const uint64_t *off, const BlockPerm &B,
                              const uint4 *keys, const uint16_t *hops, uint32_t shift, uint32_t max_loop,
                              uint32_t *arena, uint32_t *failed_bits,
                              uint32_t *failed, uint32_t *n_failed, uint32_t fail_cap, uint32_t *overflow,
                              hipStream_t s)
{
    if (n_blocks == 0)
        return hipSuccess;
    const uint32_t r0 = 1u << B.l0;
    if (r0 > block_build_max_r0() || r0 < kMinR0 || shift > B.l0)
        return hipErrorInvalidValue;
    const size_t lds = block_lds_bytes(r0);
    // 3 r_0 / 256 wavefront steps of the encoding; about r_0 / 2 elements
    const int threads = r0 >= 32768 ? 1024 : (r0 >= 8192 ? 512 : 256);
    auto *kernel = hops ? block_build_kernel<true> : block_build_kernel<false>;
    kernel<<<n_blocks, threads, lds, s>>>(bk, bstart, bucket_map, goff, sorted_items, r_sorted, tids, off, B, keys,
                                          hops, shift, max_loop, arena, failed_bits, failed, n_failed, fail_cap,
                                          overflow);
    return hipGetLastError();
}

hipError_t launch_gen_block_perms(const BlockPerm &B, uint32_t *out, hipStream_t s)
{
    if (B.m == 0)
        return hipSuccess;
    const uint32_t blocks = (uint32_t)std::min<uint64_t>(((uint64_t)B.m + 255) / 256, 65536);
    gen_block_perms_kernel<<<blocks, 256, 0, s>>>(B, out);
    return hipGetLastError();
}

}  // namespace bm
