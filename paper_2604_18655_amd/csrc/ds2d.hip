// DS2D step on the device (Section 3.5 and Appendix A.2 of the paper): from the logits of all
// rows of a step, verify the draft tree greedily and draft the next one.  Two kernels (large steps read the forecast rows
// after the walk, see ds2d_walk_draft):
//
//   ds2d_best_partial  a wavefront per (slice of 4096 logits, row): the k best logits of the row inside
//                      the slice, k = 1 for token rows (only the arg-max is needed), b'_j for
//                      forecast embedding j, as sortable 64-bit keys.  Reads every logit once:
//                      this is the kernel that is bound by HBM.
//   ds2d_verify_draft  one block per stream: arg-max of every token row from the partial keys,
//                      the walk down the tree, then the b'_i best of the forecast rows of the node
//                      where the walk ended, and the token rows of the next step.
//
// A candidate is a 64-bit key: the logit mapped to an unsigned number that orders like the
// stated rule (larger logit first, +0 = -0, NaN last) in the high half, the complement of the
// token id in the low half (lower id first among equals).  Keys of different tokens differ; 0 marks
// an empty slot.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/mlora_ds2d.h"

namespace mlora {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int DS_THREADS = 256;
constexpr int DS_SLICE = 4096;                         // logits per wavefront
constexpr int DS_KMAX = MLORA_DS2D_MAX_BRANCH;

struct Ds2dArgs {
    const void *logits;
    const int32_t *tokens;
    int32_t *n_accepted, *accepted_rows, *emitted, *next_tokens;
    unsigned long long *partial;      // [S * R][slices][DS_KMAX]; late drafts: see ds2d_walk_draft
    long long total;                  // S * R * V
    int V, S, R, T, T_next, m, depth, next_depth, slices, fp32;
    int rows;                         // rows of a stream that ds2d_best_partial looks at: R, or T (late drafts)
    int next_branch[MLORA_DS2D_MAX_FORECAST];
    signed char parent[MLORA_DS2D_MAX_ROWS];   // of the token rows
};

__device__ inline unsigned long long key_of(float v, unsigned token)
{
    unsigned b = __float_as_uint(v);
    unsigned hi;
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) hi = 0u;                     // NaN: after everything
    else {
        if (b == 0x80000000u) b = 0u;                                 // -0 counts as +0
        hi = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    }
    return ((unsigned long long)hi << 32) | (unsigned long long)(~token);
}
// Keys may be read by another block of the launch that writes them: accesses that go through to memory.
__device__ __forceinline__ void put_key(unsigned long long *p, unsigned long long key) { __hip_atomic_store(p, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <bool SAME_LAUNCH>
__device__ __forceinline__ unsigned long long get_key(const unsigned long long *p)
{
    if constexpr (SAME_LAUNCH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return *p;
}
__device__ inline float bf16_value(unsigned short h) { return __uint_as_float((unsigned)h << 16); }

// how many candidates a row needs: 1 for a token row, b'_j for forecast embedding j
__device__ inline int wanted(const Ds2dArgs &a, int r)
{
    if (r < a.T) return 1;
    const int j = (r - a.T) % a.m;                     // 0-based number of the embedding
    return j < a.next_depth ? a.next_branch[j] : 0;
}

// the largest value over a wavefront (rows of 16 lanes by DPP rotations, then the four rows)
template <int N>
__device__ __forceinline__ int ror_i32(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x120 + N, 0xF, 0xF, false); }
__device__ __forceinline__ int wave_max_i32(int v)
{
    v = max(v, ror_i32<8>(v));
    v = max(v, ror_i32<4>(v));
    v = max(v, ror_i32<2>(v));
    v = max(v, ror_i32<1>(v));
    return max(max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}
__device__ inline unsigned long long wave_max(unsigned long long v)
{
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const unsigned long long o = __shfl_xor(v, s, 64);
        v = o > v ? o : v;
    }
    return v;
}

// element j of a 16-byte vector of logits: the bit pattern as a signed number (among positive numbers it
// orders like the logit, and it is negative where the logit is), or what ordered() made of it.
template <bool FP32>
__device__ __forceinline__ int element(const u32x4 &q, int j)
{
    if constexpr (FP32) return (int)q[j];
    else return (j & 1) ? (int)q[j >> 1] >> 16 : (int)(short)(q[j >> 1] & 0xFFFFu);
}
template <bool FP32>
__device__ __forceinline__ int vector_max(const u32x4 &q)
{
    if constexpr (FP32) {
        return max(max((int)q[0], (int)q[1]), max((int)q[2], (int)q[3]));
    } else {
        // two 16-bit maxima per instruction
        // (the words as plain numbers first: a bit cast of a vector's element takes the vector's start)
        typedef short s16x2 __attribute__((ext_vector_type(2)));
        const unsigned w0 = q[0], w1 = q[1], w2 = q[2], w3 = q[3];
        const s16x2 a = __builtin_elementwise_max(__builtin_bit_cast(s16x2, w0), __builtin_bit_cast(s16x2, w1));
        const s16x2 b = __builtin_elementwise_max(__builtin_bit_cast(s16x2, w2), __builtin_bit_cast(s16x2, w3));
        const s16x2 c = __builtin_elementwise_max(a, b);
        return max((int)c[0], (int)c[1]);
    }
}

// Bit patterns -> signed numbers that order like all logits: sign and magnitude become a two's
// complement, which makes one of +0 and -0, and a shift that wraps around puts NaN below -inf.
template <bool FP32>
struct Order {
    static constexpr int SHIFT = FP32 ? 0x7FFFFF : 0x7F;                // +inf + SHIFT is the largest number
    static constexpr int LEAST = FP32 ? -0x7F000001 : -0x7F01;          // -inf + SHIFT; what lies below is NaN
    static __device__ __forceinline__ unsigned bits(int ordered)        // back again (of a number)
    {
        const int v = ordered - SHIFT;
        return v < 0 ? (FP32 ? 0x80000000u : 0x8000u) | (unsigned)-v : (unsigned)v;
    }
};
template <bool FP32>
__device__ __forceinline__ u32x4 ordered(u32x4 q)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const unsigned w = q[i];
        if constexpr (FP32) {
            const unsigned s = (unsigned)((int)w >> 31);
            q[i] = ((w & 0x7FFFFFFFu) ^ s) - s + (unsigned)Order<true>::SHIFT;
        } else {
            typedef short s16x2 __attribute__((ext_vector_type(2)));
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            const u16x2 s = __builtin_bit_cast(u16x2, __builtin_bit_cast(s16x2, w) >> (short)15);
            const u16x2 a = __builtin_bit_cast(u16x2, w & 0x7FFF7FFFu);
            q[i] = __builtin_bit_cast(unsigned, (u16x2)((a ^ s) - s + (unsigned short)Order<false>::SHIFT));
        }
    }
    return q;
}

// Slices with fewer numbers than winners wanted (short ones, NaN): all elements by their keys, the best
// one below the last winner's per round.
// (Reads the slice again every round: what matters here is that the common path keeps its registers.)
template <bool FP32>
__device__ __forceinline__ void slice_by_keys(const Ds2dArgs &a, long long slice_first, int pos_lo, int pos_hi, unsigned token_lo, int k,
                                              unsigned long long *out, int lane)
{
    unsigned long long below = ~0ull;
    for (int round = 0; round < k; ++round) {
        unsigned long long best = 0ull;
#pragma unroll 4
        for (int pos = pos_lo + lane; pos < pos_hi; pos += 64) {
            const long long e = slice_first + pos;
            const float v = FP32 ? reinterpret_cast<const float *>(a.logits)[e] : bf16_value(reinterpret_cast<const unsigned short *>(a.logits)[e]);
            unsigned long long key = key_of(v, (unsigned)(pos - pos_lo) + token_lo);
            key = key < below ? key : 0ull;
            best = key > best ? key : best;
        }
        best = wave_max(best);
        if (lane == 0) put_key(out + round, best);
        below = best;                            // (0: the slice holds fewer than k logits, the rest are empty slots)
    }
}

// What bounds it: reading the logits once.  A wavefront owns a slice and needs no barrier: 16-byte
// loads, eight (bf16) in flight per lane, a packed maximum per vector, and only one vector per lane and
// round is looked at element by element.  That works on bit patterns as signed numbers, as long as the
// winners lie above zero; a slice whose next best logit does not is put in order in its registers
// (four packed operations per two logits) and starts again.  240 rows of 128256 bf16 logits (61.6 MB): a
// block per slice with keys for all elements 25.3 us, this 15.3 us (4.0 TB/s); the whole step 20.7
// us, on the same logits less 50, all negative, 25.4 (31.2 with keys for all, 63 with rounds over memory).  Four wavefronts per SIMD: the registers for
// eight spill (35 us).
template <bool FP32>
__device__ __forceinline__ void slice_best(const Ds2dArgs &a, int row, int slice, int k, unsigned long long *out, int lane)
{
    // The row's logits are elements [row * V, row * V + V) of the whole array.  They are read
    // with aligned 16-byte loads counted from the start of the array (rows need no alignment of
    // their own); elements of a vector that belong to a neighbouring row are ignored.
    constexpr int EPV = FP32 ? 4 : 8;                                   // elements per vector
    constexpr int VPT = DS_SLICE / EPV / 64;                            // vectors per lane
    const long long first = (long long)row * a.V, last = first + a.V;
    const long long vec0 = first / EPV + (long long)slice * (64 * VPT);
    const long long full_vectors = a.total / EPV;
    const long long slice_first = vec0 * EPV;                           // element at position 0
    // the row's part of this slice, as positions pos_lo .. pos_hi, and the token id at pos_lo
    const int pos_lo = first > slice_first ? (int)(first - slice_first) : 0;
    const int pos_hi = last - slice_first < DS_SLICE ? (last > slice_first ? (int)(last - slice_first) : 0) : DS_SLICE;
    const unsigned token_lo = (unsigned)(slice_first + pos_lo - first);
    if (pos_hi <= pos_lo) {
        if (lane < k) put_key(out + lane, 0ull);
        return;
    }
    if (__builtin_expect(pos_hi - pos_lo <= 64, 0)) {                   // (the last few logits of a row: one per lane)
        slice_by_keys<FP32>(a, slice_first, pos_lo, pos_hi, token_lo, k, out, lane);
        return;
    }
    u32x4 q[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        // (vectors past the array: re-reads of its last whole one, outside the row; there is one)
        const long long vi = min(vec0 + u * 64 + lane, full_vectors - 1);
        q[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(a.logits) + vi);
    }
    if (__builtin_expect(pos_hi > (full_vectors - vec0) * EPV, 0)) {
        // the slice with the last, partial vector of the array: that one element by element, zeros past its end
        u32x4 last_vector = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int j = 0; j < EPV; ++j) {
            const long long e = full_vectors * EPV + j;
            if (e >= a.total) continue;
            if constexpr (FP32) last_vector[j] = reinterpret_cast<const unsigned *>(a.logits)[e];
            else last_vector[j >> 1] |= (unsigned)reinterpret_cast<const unsigned short *>(a.logits)[e] << (16 * (j & 1));
        }
#pragma unroll
        for (int u = 0; u < VPT; ++u)
            if (vec0 + u * 64 + lane == full_vectors) q[u] = last_vector;
    }
    constexpr int LOWEST = FP32 ? (int)0x80000000 : -32768;             // below every positive number; never a winner
    // the largest element of a vector (its first position: base) that lies in the row and comes after (top,
    // winner) in the order of candidates
    auto rest_max = [&](const u32x4 &v, int base, int top, int winner) {
        int m = LOWEST;
#pragma unroll
        for (int j = 0; j < EPV; ++j) {
            const int e = element<FP32>(v, j), pos = base + j;
            if (pos >= pos_lo && pos < pos_hi && (e < top || (e == top && pos > winner))) m = max(m, e);
        }
        return m;
    };
    const bool whole = pos_lo == 0 && pos_hi == DS_SLICE;
    // the k winners in turn; false if they run out (two copies of the code: the first one, which nearly all
    // slices take, has no choices to make)
    auto take = [&](auto order) {
        constexpr bool in_order = decltype(order)::value;
        int vm[VPT], best = LOWEST;
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            vm[u] = whole ? vector_max<FP32>(q[u]) : rest_max(q[u], (u * 64 + lane) * EPV, 0x7FFFFFFF, -1);
            best = max(best, vm[u]);
        }
        int last_top = 0x7FFFFFFF, last_winner = -1;
        for (int round = 0; round < k; ++round) {
            const int top = wave_max_i32(best);
            if (in_order ? top < Order<FP32>::LEAST : top <= 0 || top > (FP32 ? 0x7F800000 : 0x7F80)) return false;   // (uniform)
            // lowest position that holds it: the first vector of a lane that does (a lane's vectors are in the
            // order of positions), then the first element that has not been a winner before
            // (every lane does it, with its own first vector that reaches its maximum: branches would cost more)
            int pos = DS_SLICE, at = 0;
            u32x4 v = q[0];
#pragma unroll
            for (int u = VPT - 1; u >= 1; --u) at = vm[u] == best ? u : at;
            at = vm[0] == best ? 0 : at;
#pragma unroll
            for (int u = 1; u < VPT; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = at == u ? q[u][e] : v[e];
            const int base = (at * 64 + lane) * EPV, from = top == last_top ? max(pos_lo, last_winner + 1) : pos_lo;
#pragma unroll
            for (int j = EPV - 1; j >= 0; --j)
                if (element<FP32>(v, j) == top && base + j >= from && base + j < pos_hi) pos = base + j;
            const int winner = -wave_max_i32(-pos);
            if (lane == 0) {
                const unsigned bits = in_order ? Order<FP32>::bits(top) : (unsigned)top;
                put_key(out + round, key_of(__uint_as_float(FP32 ? bits : bits << 16), (unsigned)(winner - pos_lo) + token_lo));
            }
            if (round + 1 < k) {                                        // the winner's lane: its next best
                const int rest = rest_max(v, base, top, winner);
                const bool mine = pos == winner;
                best = LOWEST;
#pragma unroll
                for (int u = 0; u < VPT; ++u) {
                    vm[u] = mine && at == u ? rest : vm[u];
                    best = max(best, vm[u]);
                }
            }
            last_top = top;
            last_winner = winner;
        }
        return true;
    };
    if (__builtin_expect(take(std::false_type{}), 1)) return;
#pragma unroll
    for (int u = 0; u < VPT; ++u) q[u] = ordered<FP32>(q[u]);
    if (take(std::true_type{})) return;
    slice_by_keys<FP32>(a, slice_first, pos_lo, pos_hi, token_lo, k, out, lane);
}

template <bool FP32>
__global__ __launch_bounds__(DS_THREADS, 4) void ds2d_best_partial(const Ds2dArgs a)
{
    const int stream = (int)blockIdx.y / a.rows, r = (int)blockIdx.y - stream * a.rows, row = stream * a.R + r;
    const int k = wanted(a, r);
    const int lane = threadIdx.x & 63;
    const int slice = (int)blockIdx.x * (DS_THREADS / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (k == 0 || slice >= a.slices) return;
    unsigned long long *out = a.partial + ((size_t)row * a.slices + slice) * DS_KMAX;
    // (late drafts: the count of the stream's blocks in the next launch starts from zero)
    if (a.rows != a.R && r == 0 && slice == 0 && lane == 0) put_key(out + 1, 0ull);
    slice_best<FP32>(a, row, slice, k, out, lane);
}

// One block per stream: a chain of latencies, kept short.  Sixteen lanes reduce a token row's slices
// without atomics; the walk is a ballot per level; the best candidates of a level are ranked by
// counting, without rounds; many of them in two steps: the best of every slice, then the lists of the slices
// that have the b' best of those (the others hold no winner), at most 16 x 16 keys.
// 8 streams of 30 rows over 128256 logits: 7.6 -> 6.8 us, of which about half are the launch and two
// dependent trips to memory.
constexpr int DS_POOL = 2048;                          // candidate keys held in LDS
// Up to this many candidates of a level all are ranked among all: one barrier less and no lists to look up.
// 4 streams, in us, all against the best of the slices first: 9 slices x 16 20.4 against 23.5, 33 x 4 11.4
// and 11.5, 33 x 8 16.3 and 16.0, 65 x 4 18.6 and 13.2, 33 x 16 32.9 and 27.0, 129 x 16 217 and 39.7.
constexpr int DS_COUNT_ALL = 160;
__device__ __forceinline__ unsigned long long row16_max(unsigned long long v)
{
    auto step = [&](auto n) {
        constexpr int N = decltype(n)::value;
        const unsigned long long o = ((unsigned long long)(unsigned)ror_i32<N>((int)(v >> 32)) << 32) | (unsigned)ror_i32<N>((int)v);
        v = o > v ? o : v;
    };
    step(std::integral_constant<int, 8>{});
    step(std::integral_constant<int, 4>{});
    step(std::integral_constant<int, 2>{});
    step(std::integral_constant<int, 1>{});
    return v;
}
struct VerifyLds {
    unsigned long long best_key[MLORA_DS2D_MAX_ROWS];
    unsigned long long pool[DS_POOL];
    int walk_end, walk_token;
    int cand[MLORA_DS2D_MAX_FORECAST][DS_KMAX];
    int lists[MLORA_DS2D_MAX_FORECAST][DS_KMAX];           // slices whose best is among the b' best of all
};
// The walk down stream s's tree: lds.walk_end and walk_token, and (`write`) the accepted rows and tokens.
__device__ __forceinline__ void walk_tree(const Ds2dArgs &a, int s, VerifyLds &lds, bool write)
{
    const int tid = threadIdx.x;
    const unsigned long long *base = a.partial + (size_t)s * a.R * a.slices * DS_KMAX;
    const int my_tok = tid < a.T ? a.tokens[(size_t)s * a.T + tid] : 0;
    const int my_parent = tid < a.T ? a.parent[tid] : -1;
    // arg-max of every token row: the best of the first keys of its slices, four loads in flight per lane
    for (int r = tid >> 4; r < a.T; r += DS_THREADS / 16) {
        const unsigned long long *p = base + (size_t)r * a.slices * DS_KMAX;
        unsigned long long best = 0ull;
        for (int c0 = tid & 15; c0 < a.slices; c0 += 64) {
            unsigned long long v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = p[(size_t)min(c0 + 16 * u, a.slices - 1) * DS_KMAX];
#pragma unroll
            for (int u = 0; u < 4; ++u) best = v[u] > best ? v[u] : best;
        }
        best = row16_max(best);
        if ((tid & 15) == 0) lds.best_key[r] = best;
    }
    __syncthreads();

    // the walk, by the first wavefront: lane c looks after token row c (at most 32 of them)
    if (tid < 64) {
        int32_t *rows = a.accepted_rows + (size_t)s * (a.m + 1);
        int32_t *out = a.emitted + (size_t)s * (a.m + 1);
        const int target = tid < a.T ? (int)(~(unsigned)(lds.best_key[tid] & 0xFFFFFFFFull)) : 0;
        int cur = 0, n = 0, my_row = tid == 0 ? 0 : -1, my_out = -1;          // lane i holds entry i of both lists
        while (true) {
            const int want = __builtin_amdgcn_readlane(target, cur);
            if (tid == n) my_out = want;
            const unsigned long long kids = n < a.depth ? __ballot(my_parent == cur && tid < a.T && my_tok == want) : 0ull;
            if (!kids) {
                if (tid == 0) lds.walk_token = want;
                break;
            }
            cur = (int)__builtin_ctzll(kids);
            ++n;
            if (tid == n) my_row = cur;
        }
        if (write && tid <= a.m) {
            rows[tid] = my_row;
            out[tid] = my_out;
        }
        if (tid == 0) {
            if (write) a.n_accepted[s] = n;
            lds.walk_end = cur;
        }
    }
    __syncthreads();
}

// The next tree of stream s from the lists of level i's candidates in row first_row + i of the stream.
template <bool SAME_LAUNCH>
__device__ __forceinline__ void draft_tree(const Ds2dArgs &a, int s, VerifyLds &lds, int first_row)
{
    const int tid = threadIdx.x, cur = lds.walk_end;
    unsigned long long *const pool = lds.pool;
    auto &cand = lds.cand;
    auto &lists = lds.lists;
    int32_t *nt = a.next_tokens + (size_t)s * a.T_next;
    if (tid == 0) nt[0] = lds.walk_token;

    // Level i of the next tree: the b'_i best of forecast embedding i of the node `cur`, by rank: a
    // candidate with r better ones is number r (keys differ).  Common case: the candidates of all levels
    // fit the pool and are requested at once, candidate t % 16 of slices t / 16, t / 16 + 16, ... by thread t.
    const unsigned long long *rows_of_cur = a.partial + (size_t)(s * a.R + first_row) * a.slices * DS_KMAX;
    const int r16 = tid & 15, s16 = tid >> 4;
    int total = 0, most = 0;
    for (int i = 0; i < a.next_depth; ++i) {
        total += a.slices * a.next_branch[i];
        most = max(most, a.slices * a.next_branch[i]);
    }
    if (most > DS_COUNT_ALL && tid < MLORA_DS2D_MAX_FORECAST * DS_KMAX) lists[tid / DS_KMAX][tid % DS_KMAX] = -1;
    if (total <= DS_POOL) {
        int at = 0;
        for (int i = 0; i < a.next_depth; ++i) {
            const int b = a.next_branch[i];
            const unsigned long long *p = rows_of_cur + (size_t)i * a.slices * DS_KMAX;
            if (r16 < b)
                for (int c = s16; c < a.slices; c += 16) pool[at + c * b + r16] = get_key<SAME_LAUNCH>(p + (size_t)c * DS_KMAX + r16);
            at += a.slices * b;
        }
        __syncthreads();
        at = 0;
        if (most <= DS_COUNT_ALL) {
            for (int i = 0; i < a.next_depth; ++i) {
                const int b = a.next_branch[i], n_cand = a.slices * b;
                const unsigned long long *list = pool + at;
                if (tid < n_cand) {
                    const unsigned long long key = list[tid];
                    int better = 0;
#pragma unroll 8
                    for (int o = 0; o < n_cand; ++o) better += list[o] > key ? 1 : 0;
                    if (key && better < b) cand[i][better] = (int)(~(unsigned)(key & 0xFFFFFFFFull));
                }
                at += n_cand;
            }
        } else {
            for (int i = 0; i < a.next_depth; ++i) {
                const int b = a.next_branch[i];
                const unsigned long long *heads = pool + at;
                for (int c = tid; c < a.slices; c += DS_THREADS) {
                    const unsigned long long key = heads[c * b];
                    int better = 0;
#pragma unroll 8
                    for (int o = 0; o < a.slices; ++o) better += heads[o * b] > key ? 1 : 0;
                    if (key && better < b) lists[i][better] = c;
                }
                at += a.slices * b;
            }
            __syncthreads();
            at = 0;
            for (int i = 0; i < a.next_depth; ++i) {
                const int b = a.next_branch[i];
                const unsigned long long *all = pool + at;
                if (tid < b * b && lists[i][tid / b] >= 0) {
                    int better = 0;
                    const unsigned long long key = all[lists[i][tid / b] * b + tid % b];
                    for (int l = 0; l < b && lists[i][l] >= 0; ++l) {
                        const unsigned long long *list = all + lists[i][l] * b;
#pragma unroll 4
                        for (int o = 0; o < b; ++o) better += list[o] > key ? 1 : 0;
                    }
                    if (key && better < b) cand[i][better] = (int)(~(unsigned)(key & 0xFFFFFFFFull));
                }
                at += a.slices * b;
            }
        }
    } else {
        // the best of a level's slices in pieces, the b' best so far at the front of the pool
        const int epv = a.fp32 ? 4 : 8;
        for (int i = 0; i < a.next_depth; ++i) {
            const int b = a.next_branch[i];
            const unsigned long long *p = rows_of_cur + (size_t)i * a.slices * DS_KMAX;
            int kept = 0;
            for (int c0 = 0; c0 < a.slices;) {
                const int n_new = min(a.slices - c0, DS_POOL - kept), n = kept + n_new;
                __syncthreads();
                for (int c = tid; c < n_new; c += DS_THREADS) pool[kept + c] = get_key<SAME_LAUNCH>(p + (size_t)(c0 + c) * DS_KMAX);
                __syncthreads();
                constexpr int OWN = DS_POOL / DS_THREADS;
                unsigned long long own[OWN];
                int rank[OWN];
#pragma unroll
                for (int u = 0; u < OWN; ++u) {
                    const int c = u * DS_THREADS + tid;
                    own[u] = c < n ? pool[c] : 0ull;
                    rank[u] = 0;
                }
                for (int o = 0; o < n; ++o) {
                    const unsigned long long other = pool[o];
#pragma unroll
                    for (int u = 0; u < OWN; ++u) rank[u] += other > own[u] ? 1 : 0;
                }
                __syncthreads();
                if (tid < b) pool[tid] = 0ull;
                __syncthreads();
#pragma unroll
                for (int u = 0; u < OWN; ++u)
                    if (own[u] && rank[u] < b) pool[rank[u]] = own[u];
                kept = b;
                c0 += n_new;
            }
            __syncthreads();
            // their lists (a token's slice follows from its id: slices are counted from the vector of 16
            // bytes that the row starts in), then the candidates' ranks
            const long long first = ((long long)s * a.R + a.T + cur * a.m + i) * a.V;
            unsigned long long key = 0ull;
            if (tid < b * b) {
                const unsigned long long head = pool[tid / b];
                const int slice = (int)(((unsigned)(first % epv) + ~(unsigned)(head & 0xFFFFFFFFull)) / DS_SLICE);
                if (head) key = get_key<SAME_LAUNCH>(p + (size_t)slice * DS_KMAX + tid % b);
            }
            __syncthreads();
            if (tid < b * b) pool[tid] = key;
            __syncthreads();
            int better = 0;
            for (int o = 0; o < b * b; ++o) better += pool[o] > key ? 1 : 0;
            if (key && better < b) cand[i][better] = (int)(~(unsigned)(key & 0xFFFFFFFFull));
        }
    }
    __syncthreads();
    int offset = 1, width = 1;
    for (int i = 0; i < a.next_depth; ++i) {
        const int b = a.next_branch[i];
        width *= b;
        for (int q = tid; q < width; q += DS_THREADS) nt[offset + q] = cand[i][q % b];
        offset += width;
    }
}

__global__ __launch_bounds__(DS_THREADS) void ds2d_verify_draft(const Ds2dArgs a)
{
    __shared__ VerifyLds lds;
    walk_tree(a, blockIdx.x, lds, true);
    draft_tree<false>(a, blockIdx.x, lds, a.T + lds.walk_end * a.m);
}

// Late drafts: of a stream's forecast rows the step needs those of the node where the walk ends, so where reading the
// others takes longer than walking first, ds2d_best_partial looks at the token rows only and this kernel follows.
// Every block makes the walk for itself (T * slices keys, a trip to memory that runs beside nothing else), takes four
// slices of one forecast row, and the last block of a stream, by a count that the launch before has set to zero, drafts.
// The lists of level i lie where those of node 0's row would.  8 streams of 30 rows over 128256 bf16 logits, of which 24.6
// of 61.5 MB are read: 21.8 -> 17.0 us a step.
template <bool FP32>
__global__ __launch_bounds__(DS_THREADS, 4) void ds2d_walk_draft(const Ds2dArgs a)
{
    __shared__ VerifyLds lds;
    __shared__ bool last;
    const int s = (int)blockIdx.y / a.next_depth, level = (int)blockIdx.y - s * a.next_depth, lane = threadIdx.x & 63;
    walk_tree(a, s, lds, blockIdx.x == 0 && level == 0);
    const int slice = (int)blockIdx.x * (DS_THREADS / 64) + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    unsigned long long *const lists = a.partial + (size_t)(s * a.R + a.T + level) * a.slices * DS_KMAX;
    if (slice < a.slices) slice_best<FP32>(a, s * a.R + a.T + lds.walk_end * a.m + level, slice, a.next_branch[level], lists + (size_t)slice * DS_KMAX, lane);
    // (the keys, then the count: see put_key; all of a wave's stores are acknowledged before the block meets)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned *const count = reinterpret_cast<unsigned *>(a.partial + (size_t)s * a.R * a.slices * DS_KMAX + 1);
        last = atomicAdd(count, 1u) + 1u == gridDim.x * (unsigned)a.next_depth;
    }
    __syncthreads();
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (last) draft_tree<true>(a, s, lds, a.T);
}

}  // namespace mlora

using namespace mlora;

namespace {

bool tree_sizes(const int32_t *branch, int depth, int m, int &tokens, int &rows)
{
    if (m < 1 || m > MLORA_DS2D_MAX_FORECAST || depth < 0 || depth > m) return false;
    long long t = 1, w = 1;
    for (int i = 0; i < depth; ++i) {
        if (branch[i] < 1 || branch[i] > MLORA_DS2D_MAX_BRANCH) return false;
        w *= branch[i];
        t += w;
        if (t * (1 + m) > MLORA_DS2D_MAX_ROWS) return false;
    }
    if (t * (1 + m) > MLORA_DS2D_MAX_ROWS) return false;
    tokens = (int)t;
    rows = (int)(t * (1 + m));
    return true;
}

// parent of every token row: level by level, the children of one node next to each other
void token_parents(const int32_t *branch, int depth, int *parent)
{
    parent[0] = -1;
    int level_first = 0, level_count = 1, next = 1;
    for (int i = 0; i < depth; ++i) {
        for (int node = level_first; node < level_first + level_count; ++node)
            for (int c = 0; c < branch[i]; ++c) parent[next++] = node;
        level_first += level_count;
        level_count *= branch[i];
    }
}

int slices_of(const mlora_ds2d &d)
{
    const int epv = d.logits_dtype == MLORA_Y_FP32 ? 4 : 8;
    const long long vectors = (long long)d.vocab / epv + 2;             // a row may straddle two more
    const long long per_block = DS_SLICE / epv;
    return (int)((vectors + per_block - 1) / per_block);
}

// Whether the forecast rows wait for the walk (see ds2d_walk_draft): where that spares more than LATE_BYTES of logits
// (42 drawn steps both ways, us by MB spared: 8 13.3 -> 14.8, 15 14.1 -> 15.1, 21 15.2 -> 15.5 and 26.0 -> 22.0, 28 16.3 ->
// 15.4, 37 21.8 -> 17.0, 47 21.7 -> 16.0; a few kB 8.9 -> 11.9) and the walk that every block makes for itself is not too
// long: its keys lie in lines of their own, so the blocks' walks grow with the square of the vocabulary while what is spared
// grows with the vocabulary.  At most LATE_WALK times the bytes spared (1 to 8 streams, trees of 2 to 10 tokens, up to 20
// million logits a row, time of the late form against the other by that ratio: up to 3.3 0.55 to 1.04, 3.8 to 4.8 0.88 to
// 1.03, 5.7 to 6.4 0.96 to 1.09, 6.9 to 9.6 1.01 to 1.21, above that 1.01 to 2.6; with rows of 128256 bf16 logits it is 0.14).
constexpr long long LATE_BYTES = 22000000;
constexpr double LATE_WALK = 3.5;
bool late_drafts(const mlora_ds2d &d, int T)
{
    const long long row = (long long)d.vocab * (d.logits_dtype == MLORA_Y_FP32 ? 4 : 2), slices = slices_of(d);
    const long long spared = (T - 1) * row;                             // of a stream and level
    const double walk = (double)((slices + 3) / 4) * (double)(T * slices * DS_KMAX * (long long)sizeof(unsigned long long));
    return (long long)d.n_streams * d.next_depth * spared > LATE_BYTES && walk <= LATE_WALK * (double)spared;
}

mlora_status check(const mlora_ds2d *d, int &T, int &R, int &T_next)
{
    if (!d) return MLORA_EINVAL;
    if (d->logits_dtype != MLORA_Y_BF16 && d->logits_dtype != MLORA_Y_FP32) return MLORA_EINVAL;
    int r_next;
    if (d->n_streams < 1 || d->n_streams > 65535) return MLORA_ESHAPE;
    if (!tree_sizes(d->branch, d->depth, d->n_forecast, T, R)) return MLORA_ESHAPE;
    if (!tree_sizes(d->next_branch, d->next_depth, d->n_forecast, T_next, r_next)) return MLORA_ESHAPE;
    if (d->vocab < 1 || d->vocab >= 0x7FFFFFFF) return MLORA_ESHAPE;
    for (int i = 0; i < d->next_depth; ++i)
        if (d->next_branch[i] > d->vocab) return MLORA_ESHAPE;
    if ((long long)d->n_streams * R > 65535) return MLORA_ESHAPE;       // grid y
    return MLORA_OK;
}

}  // namespace

extern "C" {

mlora_status mlora_ds2d_rows(const int32_t *branch, int32_t depth, int32_t n_forecast,
                             int32_t *n_tokens, int32_t *n_rows)
{
    if (!n_tokens || !n_rows || (depth > 0 && !branch)) return MLORA_EINVAL;
    int t, r;
    if (!tree_sizes(branch, depth, n_forecast, t, r)) return MLORA_ESHAPE;
    *n_tokens = t;
    *n_rows = r;
    return MLORA_OK;
}

mlora_status mlora_ds2d_layout(const int32_t *branch, int32_t depth, int32_t n_forecast,
                               int32_t *parent, uint8_t *is_forecast, int32_t *level)
{
    if (!parent || !is_forecast || (depth > 0 && !branch)) return MLORA_EINVAL;
    int T, R;
    if (!tree_sizes(branch, depth, n_forecast, T, R)) return MLORA_ESHAPE;
    int par[MLORA_DS2D_MAX_ROWS];
    token_parents(branch, depth, par);
    for (int r = 0; r < T; ++r) {
        parent[r] = par[r];
        is_forecast[r] = 0;
        if (level) level[r] = r == 0 ? 0 : level[par[r]] + 1;
    }
    for (int t = 0; t < T; ++t)
        for (int j = 0; j < n_forecast; ++j) {
            const int r = T + t * n_forecast + j;
            parent[r] = j == 0 ? t : r - 1;
            is_forecast[r] = 1;
            if (level) level[r] = j + 1;
        }
    return MLORA_OK;
}

size_t mlora_ds2d_workspace_bytes(const mlora_ds2d *d)
{
    int T, R, T_next;
    if (check(d, T, R, T_next) != MLORA_OK) return 0;
    return (size_t)d->n_streams * R * slices_of(*d) * DS_KMAX * sizeof(unsigned long long);
}

int32_t mlora_ds2d_late_drafts(const mlora_ds2d *d)
{
    int T, R, T_next;
    return check(d, T, R, T_next) == MLORA_OK && late_drafts(*d, T) ? 1 : 0;
}

mlora_status mlora_ds2d_step(const mlora_ds2d *d, const void *logits, const int32_t *tokens,
                             int32_t *n_accepted, int32_t *accepted_rows, int32_t *emitted,
                             int32_t *next_tokens, void *workspace, size_t workspace_bytes,
                             void *stream)
{
    int T, R, T_next;
    const mlora_status st = check(d, T, R, T_next);
    if (st != MLORA_OK) return st;
    if (!logits || !tokens || !n_accepted || !accepted_rows || !emitted || !next_tokens) return MLORA_EINVAL;
    if ((reinterpret_cast<uintptr_t>(logits) & 15u) || (reinterpret_cast<uintptr_t>(workspace) & 15u)) return MLORA_EALIGN;
    if (!workspace || workspace_bytes < mlora_ds2d_workspace_bytes(d)) return MLORA_EWORKSPACE;

    Ds2dArgs a;
    a.logits = logits;
    a.tokens = tokens;
    a.n_accepted = n_accepted;
    a.accepted_rows = accepted_rows;
    a.emitted = emitted;
    a.next_tokens = next_tokens;
    a.partial = reinterpret_cast<unsigned long long *>(workspace);
    a.V = d->vocab;
    a.S = d->n_streams;
    a.R = R;
    a.T = T;
    a.T_next = T_next;
    a.m = d->n_forecast;
    a.depth = d->depth;
    a.next_depth = d->next_depth;
    a.slices = slices_of(*d);
    a.fp32 = d->logits_dtype == MLORA_Y_FP32;
    a.total = (long long)d->n_streams * R * d->vocab;
    for (int i = 0; i < MLORA_DS2D_MAX_FORECAST; ++i) a.next_branch[i] = i < d->next_depth ? d->next_branch[i] : 0;
    int par[MLORA_DS2D_MAX_ROWS];
    token_parents(d->branch, d->depth, par);
    for (int r = 0; r < MLORA_DS2D_MAX_ROWS; ++r) a.parent[r] = r < T ? (signed char)par[r] : (signed char)-1;

    hipStream_t s = (hipStream_t)stream;
    const bool late = late_drafts(*d, T);
    a.rows = late ? T : R;
    const dim3 grid((a.slices + 3) / 4, d->n_streams * a.rows), late_grid((a.slices + 3) / 4, d->n_streams * (late ? a.next_depth : 1));
    auto by_type = [&](auto fp32) {
        constexpr bool FP32 = decltype(fp32)::value;
        ds2d_best_partial<FP32><<<grid, dim3(DS_THREADS), 0, s>>>(a);
        if (late) ds2d_walk_draft<FP32><<<late_grid, dim3(DS_THREADS), 0, s>>>(a);
        else      ds2d_verify_draft<<<dim3(d->n_streams), dim3(DS_THREADS), 0, s>>>(a);
    };
    if (a.fp32) by_type(std::true_type{});
    else        by_type(std::false_type{});
    return hipGetLastError() == hipSuccess ? MLORA_OK : MLORA_EHIP;
}

}  // extern "C"
