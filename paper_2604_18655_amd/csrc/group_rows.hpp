// Stable grouping of rows by adapter inside one workgroup, results in LDS.
#pragma once
#include "common.hpp"

namespace mlora {

struct GroupLds {
    int count[MLORA_MAX_ADAPTERS + 1];            // histogram, then running write offsets
    unsigned short perm[MLORA_MAX_ROWS];
    unsigned short seg_adapter[MLORA_MAX_ADAPTERS];
    unsigned short seg_start[MLORA_MAX_ADAPTERS + 1];
    int n_seg;
    int bad;                                      // an index was outside [-1, n_adapters)
};

// Rows without adapter (-1, or an out-of-range index) go to bucket n_adapters, which sorts last.
__device__ inline int bucket_of(int a, int n_adapters, bool &bad)
{
    bad = (a < -1) || (a >= n_adapters);
    return (a < 0 || a >= n_adapters) ? n_adapters : a;
}

// At most 64 rows: one wave, one row per lane.  The position of a row in the sorted order is (#rows in a
// smaller bucket) + (#earlier rows in the same bucket); both sets are built as lane masks from one
// ballot per bit of the bucket id.
struct RowPlace {
    int bucket;
    unsigned long long smaller, before;            // lanes of smaller buckets; earlier lanes of the own one
    bool valid, has_adapter, bad;
    __device__ int rank() const { return __popcll(before); }
    __device__ int position() const { return __popcll(smaller) + rank(); }
    // how many of the lanes in `mask` come earlier in the sorted order
    __device__ int ahead(unsigned long long mask) const { return __popcll(mask & smaller) + __popcll(mask & before); }
};
__device__ inline RowPlace place_row(const int *row_adapter, int M, int n_adapters)
{
    const int lane = threadIdx.x & 63;
    RowPlace r;
    r.valid = lane < M;
    r.bad = false;
    r.bucket = 0;
    if (r.valid) r.bucket = bucket_of(row_adapter[lane], n_adapters, r.bad);
    unsigned long long eq = __ballot(r.valid), lt = 0;
    const int nbits = 32 - __clz(n_adapters);      // buckets 0..n_adapters
    for (int bit = nbits - 1; bit >= 0; --bit) {
        const bool set = (r.bucket >> bit) & 1;
        const unsigned long long bal = __ballot(r.valid && set);
        if (set) { lt |= eq & ~bal; eq &= bal; }
        else     { eq &= ~bal; }
    }
    r.smaller = lt;
    r.before = eq & ((1ull << lane) - 1ull);
    r.has_adapter = r.valid && r.bucket < n_adapters;
    return r;
}

template <class G>
__device__ inline void group_rows_wave(const int *row_adapter, int M, int n_adapters, G &g)
{
    const int lane = threadIdx.x & 63;
    const RowPlace r = place_row(row_adapter, M, n_adapters);
    const bool first = r.has_adapter && r.rank() == 0;
    const unsigned long long first_mask = __ballot(first);
    if (r.valid) g.perm[r.position()] = (unsigned short)lane;
    if (first) {
        const int idx = r.ahead(first_mask);
        g.seg_adapter[idx] = (unsigned short)r.bucket;
        g.seg_start[idx] = (unsigned short)r.position();
    }
    const int n_seg = __popcll(first_mask);
    const int with_adapter = __popcll(__ballot(r.has_adapter));
    const unsigned long long any_bad = __ballot(r.bad);
    if (lane == 0) {
        g.seg_start[n_seg] = (unsigned short)with_adapter;
        g.n_seg = n_seg;
        g.bad = any_bad != 0;
    }
}

// The rows of every adapter cut into tiles of 16, in the order of the adapters.
struct RowTiles {
    unsigned short perm[64];                       // rows in sorted order
    unsigned short first[65], adapter[64];         // of tile t: position of its first row (the next tile's ends it), adapter
    int n_tiles;
};
// Called by one wave, at most 64 rows.
__device__ inline void cut_row_tiles(const int *row_adapter, int M, int n_adapters, RowTiles &g)
{
    const int lane = threadIdx.x & 63;
    const RowPlace r = place_row(row_adapter, M, n_adapters);
    const bool first = r.has_adapter && r.rank() % 16 == 0;
    const unsigned long long first_mask = __ballot(first);
    if (r.valid) g.perm[r.position()] = (unsigned short)lane;
    if (first) {
        const int t = r.ahead(first_mask);
        g.first[t] = (unsigned short)r.position();
        g.adapter[t] = (unsigned short)r.bucket;
    }
    const int with_adapter = __popcll(__ballot(r.has_adapter));
    if (lane == 0) {
        g.n_tiles = __popcll(first_mask);
        g.first[g.n_tiles] = (unsigned short)with_adapter;
    }
}

// Any M: counting sort with the histogram in LDS; wave 0 scans it and scatters the rows in
// ascending order, 64 at a time.
__device__ inline void group_rows_counting(const int *row_adapter, int M, int n_adapters, GroupLds &g)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nthreads = blockDim.x;
    for (int b = tid; b <= n_adapters; b += nthreads) g.count[b] = 0;
    if (tid == 0) g.bad = 0;
    __syncthreads();
    for (int m = tid; m < M; m += nthreads) {
        bool bad;
        const int b = bucket_of(row_adapter[m], n_adapters, bad);
        if (bad) g.bad = 1;
        atomicAdd(&g.count[b], 1);
    }
    __syncthreads();
    if (wave == 0) {
        volatile int *cnt = g.count;
        const unsigned long long below = (1ull << lane) - 1ull;
        // exclusive scan of the histogram, 64 buckets at a time; non-empty adapters become segments
        int carry = 0, nseg = 0;
        for (int base = 0; base <= n_adapters; base += 64) {
            const int b = base + lane;
            const int c = (b <= n_adapters) ? cnt[b] : 0;
            int incl = c;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int v = __shfl_up(incl, d);
                if (lane >= d) incl += v;
            }
            const int excl = incl - c + carry;
            const bool is_seg = (b < n_adapters) && (c > 0);
            const unsigned long long mask = __ballot(is_seg);
            if (b <= n_adapters) cnt[b] = excl;
            if (is_seg) {
                const int idx = nseg + __popcll(mask & below);
                g.seg_adapter[idx] = (unsigned short)b;
                g.seg_start[idx] = (unsigned short)excl;
            }
            carry += __shfl(incl, 63);
            nseg += __popcll(mask);
        }
        if (lane == 0) {
            g.seg_start[nseg] = (unsigned short)cnt[n_adapters];   // rows that carry an adapter
            g.n_seg = nseg;
        }
        // stable scatter: within a chunk each distinct bucket is served in turn and its rows
        // keep their lane order
        for (int base = 0; base < M; base += 64) {
            const int m = base + lane;
            const bool valid = m < M;
            int bucket = 0;
            if (valid) {
                bool bad;
                bucket = bucket_of(row_adapter[m], n_adapters, bad);
            }
            unsigned long long remaining = __ballot(valid);
            while (remaining) {
                const int leader = __ffsll((long long)remaining) - 1;
                const int bl = __builtin_amdgcn_readlane(bucket, leader);
                const bool mine = valid && bucket == bl;
                const unsigned long long same = __ballot(mine);
                const int off = cnt[bl];
                if (mine) g.perm[off + __popcll(same & below)] = (unsigned short)m;
                if (lane == leader) cnt[bl] = off + __popcll(same);
                remaining &= ~same;
            }
        }
    }
}

// Called by all threads of a block.  On return g holds the permutation and the segments.
__device__ inline void group_rows_lds(const int *row_adapter, int M, int n_adapters, GroupLds &g)
{
    if (M <= 64) {
        if ((threadIdx.x >> 6) == 0) group_rows_wave(row_adapter, M, n_adapters, g);
    } else {
        group_rows_counting(row_adapter, M, n_adapters, g);
    }
    __syncthreads();
}

}  // namespace mlora
