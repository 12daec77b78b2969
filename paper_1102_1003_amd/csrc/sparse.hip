// Counting by transactions, for sparse sets (Sec. I: horizontal format): the
// support of (i, j) is the number of transactions of S_i that hold j, so a row of
// the result is one walk over the transactions of S_i.  The walk reads every
// transaction once per item in it, sum |T_b|^2 items in all, whatever n and m;
// at 0.05 % density that is 4 items an incidence where the slot compare visits
// 3 max(r_i, r_j) slots a pair.
#include "bm_internal.h"

namespace bm {

namespace {

// Transaction sizes: one device atomic an incidence.
__global__ void txn_count_kernel(const uint32_t *__restrict__ tids, uint64_t nnz, uint32_t *count)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nnz; k += stride)
        atomicAdd(&count[tids[k]], 1u);
}

// The m transaction sizes d: their pairs, the longest, and the sums over those of more
// than kTxnLong items.
__global__ void __launch_bounds__(256) txn_walk_kernel(const uint32_t *__restrict__ count, uint32_t m, TxnWalk *walk)
{
    unsigned long long pairs = 0, items = 0, squares = 0, longest = 0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < m; t += stride) {
        const unsigned long long d = count[t];
        pairs += d ? d * (d - 1) / 2 : 0;
        items += d > kTxnLong ? d : 0;
        squares += d > kTxnLong ? d * d : 0;
        longest = max(longest, d);
    }
    for (int o = 32; o > 0; o >>= 1) {
        pairs += __shfl_xor(pairs, o, 64);
        items += __shfl_xor(items, o, 64);
        squares += __shfl_xor(squares, o, 64);
        longest = max(longest, __shfl_xor(longest, o, 64));
    }
    // one workgroup's atomics: they all meet on one line
    __shared__ unsigned long long part[4][4];
    if ((threadIdx.x & 63) == 0) {
        const uint32_t w = threadIdx.x / 64;
        part[w][0] = pairs;
        part[w][1] = items;
        part[w][2] = squares;
        part[w][3] = longest;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; w++) {
            pairs += part[w][0];
            items += part[w][1];
            squares += part[w][2];
            longest = max(longest, part[w][3]);
        }
        if (longest == 0)
            return;
        atomicAdd(reinterpret_cast<unsigned long long *>(&walk->pairs), pairs);
        atomicMax(reinterpret_cast<unsigned long long *>(&walk->longest), longest);
        if (items) {
            atomicAdd(reinterpret_cast<unsigned long long *>(&walk->long_items), items);
            atomicAdd(reinterpret_cast<unsigned long long *>(&walk->long_squares), squares);
        }
    }
}

// items[cursor[t]++] = item of every incidence, a workgroup per item (the order
// inside a transaction does not matter).
__global__ void __launch_bounds__(256) txn_scatter_kernel(const uint64_t *__restrict__ off,
                                                          const uint32_t *__restrict__ tids, uint32_t n,
                                                          uint32_t *cursor, uint32_t *items)
{
    for (uint32_t i = blockIdx.x; i < n; i += gridDim.x)
        for (uint64_t k = off[i] + threadIdx.x; k < off[i + 1]; k += blockDim.x)
            items[atomicAdd(&cursor[tids[k]], 1u)] = i;
}

// One workgroup per row i of the packed triangle: the counters of the items
// after i live in LDS, the lanes walk the transactions of S_i, and the row leaves
// once, in order (no zero fill, no device atomics: added into device memory
// the counts would run at 27 * 10^9 a second, and slower where pairs are hot).
// Bound by the random loads tid -> transaction -> items: at 2^20 x 8192 and 0.05 % (4.3
// * 10^6 incidences, 4 items a transaction, 134 MB of counts) they read 870 MB past
// the L2s, and the waves wait for them nine tenths of their time: 0.18 ms, the slot
// compare 4.8 ms.
__global__ void txn_rows_kernel(const uint64_t *__restrict__ off, const uint32_t *__restrict__ tids,
                                const uint32_t *__restrict__ start, const uint32_t *__restrict__ items, uint32_t n,
                                uint32_t *__restrict__ out)
{
    extern __shared__ uint32_t cnt[];
    const uint32_t i = blockIdx.x, len = n - 1 - i;
    for (uint32_t q = threadIdx.x; q < len; q += blockDim.x)
        cnt[q] = 0;
    __syncthreads();
    const uint64_t k1 = off[i + 1];
    for (uint64_t k = off[i] + threadIdx.x; k < k1; k += blockDim.x) {
        const uint32_t t = tids[k];
        const uint32_t e = start[t + 1];
        for (uint32_t p = start[t]; p < e; p++) {
            const uint32_t j = items[p];
            if (j > i)
                atomicAdd(&cnt[j - i - 1], 1u);
        }
    }
    __syncthreads();
    uint32_t *row = out + ((uint64_t)i * n - (uint64_t)i * (i + 1) / 2);
    for (uint32_t q = threadIdx.x; q < len; q += blockDim.x)
        row[q] = cnt[q];
}

}  // namespace

hipError_t launch_txn_count(const uint32_t *tids, uint64_t nnz, uint32_t m, uint32_t *count, TxnWalk *walk,
                            hipStream_t s)
{
    if (nnz) {
        const uint64_t blocks = (nnz + 255) / 256;
        txn_count_kernel<<<(uint32_t)(blocks < 8192 ? blocks : 8192), 256, 0, s>>>(tids, nnz, count);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    const uint32_t blocks = (m + 255) / 256;
    txn_walk_kernel<<<blocks < 256 ? blocks : 256, 256, 0, s>>>(count, m, walk);
    return hipGetLastError();
}

hipError_t launch_txn_scatter(const uint64_t *off, const uint32_t *tids, uint32_t n, uint32_t *cursor,
                              uint32_t *items, hipStream_t s)
{
    txn_scatter_kernel<<<n < 65536 ? n : 65536, 256, 0, s>>>(off, tids, n, cursor, items);
    return hipGetLastError();
}

hipError_t launch_txn_rows(const uint64_t *off, const uint32_t *tids, const uint32_t *start, const uint32_t *items,
                           uint32_t n, uint32_t *out, hipStream_t s)
{
    if (n < 2)
        return hipSuccess;
    if (n > kTxnMaxItems)
        return hipErrorInvalidValue;
    // the counters of the longest row; wide rows leave few workgroups a CU, so those are larger
    const uint32_t lds = (n - 1) * 4;
    txn_rows_kernel<<<n - 1, lds > 32768 ? 1024 : 256, lds, s>>>(off, tids, start, items, n, out);
    return hipGetLastError();
}

}  // namespace bm
