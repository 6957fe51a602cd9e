#pragma once
// The layer step: one launch.
//
// Base product.  A block of four waves owns one K unit of one tile of 64 output columns for one
// chunk of rows (16, 32 or 64 of them: three kernels, below).  Packed codes come straight from
// HBM with one 128-bit load per lane and k-step, the rows of x and the fp16 scales from L2;
// every code dword becomes four bf16 pairs with 7 instructions and feeds 16x16x32 bf16 MFMAs
// whose A operand is a block of rows of x.  Scales multiply fp32 results, so the codes enter
// the matrix unit exactly.  What several waves add up is added in a fixed order.
//
// Long projections are cut into several K units per tile: units 1.. leave fp32 partial tiles in
// the workspace; unit 0 (the finishing block) adds them in order, adds the LoRA term
// alpha * B[a(m)][n] . t[m] and stores y.
//
// Order inside the launch.  The grid holds the shrink blocks first, then the split-K blocks,
// then the finishing blocks.  A finishing block streams its weights without waiting for
// anything; only before its epilogue does it wait (bounded spin on counters in the workspace)
// until the shrink blocks of its projection and the split-K blocks of its tile have signalled
// completion.  Blocks are dispatched in index order, producers never wait, so every wait
// ends; if one nevertheless runs out, the block sets the workspace status word and goes on.
//
// LoRA shrink, t[m] = A[a(m)] . x[m] in K chunks, MFMA (A operand: rows of x, B operand: 16 rank
// rows of A[adapter]); the partial sums go to t_part[chunk][row][rank].  Up to 16 rows: a block
// per (row, 16 ranks, K chunk).  More rows: the rows of a chunk of 64 are grouped by adapter
// and cut into tiles of 16, and a block's four waves share the inputs of every tile.
#include <type_traits>

#include "group_rows.hpp"

namespace mlora {

// ------------------------------------------------------------------------------------------
// completion counters
// ------------------------------------------------------------------------------------------
// Data one block hands to another inside a launch (split-K partial tiles, the shrink step's t)
// is written and read with agent-scope accesses: they go through to memory and are re-fetched
// from it, so no cache of a compute unit or of a die ever holds a stale copy of it, and no
// cache-wide write-back or invalidate (which every fence at that scope costs) is needed.
__device__ __forceinline__ void store_shared(float *p, float v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_shared(const float *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The same for 16 bytes at a time (the wide kernel's partial tiles).  There is no 128-bit atomic type,
// so this is the plain 128-bit instruction with the cache policy of the 32-bit one above (sc1),
// written out.
typedef float f32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void store_shared16(float *p, f32x4_t v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1" : : "v"(p), "v"(v) : "memory");
}
// 16-byte loads of such data that the compiler can see (and so schedule, and wait for, by
// itself): buffer loads with the same cache policy (sc1, bit 4 of the policy argument) through a
// descriptor over `bytes` bytes at `base` (raw buffer, no stride; accesses past the end return 0).
// `base` and `bytes` must be the same for every lane of a wave.
typedef unsigned int u32x4_v __attribute__((vector_size(16)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t shared_buffer(const float *base, int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ f32x4_t load_shared16(__amdgpu_buffer_rsrc_t rsrc, int byte_offset, int uniform_offset = 0)
{
    return __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rsrc, byte_offset, uniform_offset, 16));
}

// descriptor over `bytes` bytes at `base`, both the same for every lane of a wave (raw buffer, no
// stride; reads past the end return 0)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t wave_buffer(const void *base, unsigned bytes)
{
    const uint64_t at = reinterpret_cast<uint64_t>(base);
    const uint64_t lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)at);
    const uint64_t hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(at >> 32));
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(lo | (hi << 32)), 0, __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000);
}

// The hardware keeps the order "data, then counter" on the producer's side (the wait for the
// stores' acknowledgements below) and "counter, then data" on the consumer's (a wave's loads are
// issued in program order, and these go through to memory).  The compiler must keep it too:
// relaxed accesses to different addresses may be reordered, so a compiler-only fence (no
// instruction, no cache action) stands between the data accesses and the counter access.
__device__ __forceinline__ void compiler_fence() { __atomic_signal_fence(__ATOMIC_SEQ_CST); }

// all threads of the block, after their store_shared calls: wait until the own stores have been
// acknowledged, meet, then count the block as done in `copies` counter lines
__device__ __forceinline__ void signal_done(unsigned *counter, int copies)
{
    compiler_fence();
    __builtin_amdgcn_s_waitcnt(0x0F70);        // vmcnt(0): every store of this wave has completed
    __syncthreads();
    if ((int)threadIdx.x < copies) atomicAdd(counter + threadIdx.x * CTR_STRIDE, 1u);
}

// Wait until *counter has reached expected, polling at most `limit` times; false if the wait ran
// out (limit 0: at once).  Reads of what the counter guards must come after this call: the
// fence keeps the compiler from moving them up.
__device__ __forceinline__ bool wait_count(unsigned *counter, unsigned expected, int limit)
{
    bool ok = false;
    for (int i = 0; i < limit; ++i) {
        if (__hip_atomic_load(counter, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= expected) { ok = true; break; }
        __builtin_amdgcn_s_sleep(1);
    }
    compiler_fence();
    return ok;
}

// ------------------------------------------------------------------------------------------
// base product
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ float half_bits_lo(uint32_t v) { return half_bits_to_float((uint16_t)(v & 0xFFFFu)); }
__device__ __forceinline__ float half_bits_hi(uint32_t v) { return half_bits_to_float((uint16_t)(v >> 16)); }

// (a native vector type: copies of HIP's uint4 struct from global to LDS would be lowered to
// memcpy through a private array instead of going through registers)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// The two halves of a code word as bytes of sign and magnitude (see common.hpp), and eight such bytes -> 8 bf16
// numbers (4 dwords).  Exact, without an offset: with codes + 24 (7 operations as well) every group needed
// one more product per block of rows to take the offset out, and its sums were up to seven times the result.
__device__ __forceinline__ uint32_t low_codes(uint32_t w) { return w & FIELD_MASK; }
__device__ __forceinline__ uint32_t high_codes(uint32_t w) { return __builtin_amdgcn_alignbit(w, w, 4) & FIELD_MASK; }
// (blobs with codes -8 hold m - 1 for negative codes)
__device__ __forceinline__ uint32_t full_codes(uint32_t bytes) { return bytes + ((bytes >> 7) & 0x01010101u); }
__device__ __forceinline__ uint4 codes_to_bf16(uint32_t lo, uint32_t hi)
{
    uint4 o;
    o.x = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.0f, false));
    o.y = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 512.0f, true));
    o.z = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.0f, false));
    o.w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 512.0f, true));
    return o;
}
// The halves of the four code words of a k-step.  `full` is the same for the whole block: every family of blocks
// branches here, once per k-step, in the one loop that it has.  (A second copy of the loop for blobs with codes -8
// costs registers and code: blocks of up to 8 rows spilled 24 registers and of up to 16 rows took 221 instead of 187;
// with requests of its own, which had to wait for the flag, that copy took 17.3 us for the seven projections of a
// layer at 8 rows, 166 for 16 layers, against 15.9 and 144 as it is and 15.0 and 141 for codes + 24.  Two
// operations instead of three, a packed multiply-add on fields with the sign lowest, give nothing in the wide
// blocks and 0.2 us in the layer.)  `RARE` keeps the loop without codes -8 free of jumps: 16.7 -> 16.4 us in a
// graph for the layer at 8 rows; in the wide blocks it costs blobs with codes -8 3 % and the others nothing.
template <int WORDS>
struct CodeBytes {
    uint32_t lo[WORDS], hi[WORDS];
};
template <bool RARE, class Words>
__device__ __forceinline__ auto split_codes(Words w, bool full)
{
    constexpr int WORDS = sizeof(Words) / 4;
    CodeBytes<WORDS> c;
#pragma unroll
    for (int j = 0; j < WORDS; ++j) {
        c.lo[j] = low_codes(w[j]);
        c.hi[j] = high_codes(w[j]);
    }
    if (RARE ? __builtin_expect(full, 0) : full) {
#pragma unroll
        for (int j = 0; j < WORDS; ++j) {
            c.lo[j] = full_codes(c.lo[j]);
            c.hi[j] = full_codes(c.hi[j]);
        }
    }
    return c;
}

__device__ __forceinline__ void pin(f32x16 (&acc)[2]) { asm volatile("" : "+v"(acc[0]), "+v"(acc[1])); }
__device__ __forceinline__ void pin(f32x16 (&acc)[1]) { asm volatile("" : "+v"(acc[0])); }
template <int MB>
__device__ __forceinline__ void pin(f32x4 (&acc)[MB][4])
{
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(acc[mb][0]), "+v"(acc[mb][1]), "+v"(acc[mb][2]), "+v"(acc[mb][3]));
}

// The blob's flag, requested like the codes and ahead of them, so that it is there when they are.  (Through the
// scalar cache it would come from memory as well, and every wait for a kernel argument behind it would
// wait for it: 8 rows, the seven projections of a layer, 14.7 -> 15.6 us.)
__device__ __forceinline__ uint32_t request_flag(const ProjArgs &P)
{
    unsigned at = 0;
    asm volatile("" : "+v"(at));                               // an address in a vector register
    using G = const __attribute__((address_space(1))) uint32_t;
    return ((G *)P.flag)[at];
}
__device__ __forceinline__ bool flag_set(uint32_t flag) { return __builtin_amdgcn_readfirstlane((int)flag) != 0; }

// eight int8 (two words) -> eight bf16, exactly (seven bits and a sign)
__device__ __forceinline__ u32x4 widen_int8(uint32_t lo, uint32_t hi)
{
    u32x4 o;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const uint32_t word = h < 2 ? lo : hi;
        const float e0 = (float)(int)(signed char)(word >> (16 * (h & 1)));
        const float e1 = (float)(int)(signed char)(word >> (16 * (h & 1) + 8));
        o[h] = __builtin_amdgcn_perm(__float_as_uint(e1), __float_as_uint(e0), 0x07060302u);   // the upper halves
    }
    return o;
}

// ------------------------------------------------------------------------------------------
// A wave works through its inputs in rounds of R k-steps.  All operands of a round (R KiB of
// packed codes, the rows of x, the scales) are staged in a wave-private LDS buffer, and the
// math of a round is a ROLLED loop over its scale groups that reads everything back from
// LDS.  The loop is the point of the design: code that runs once is fetched at about 10
// cycles per instruction (instruction-cache misses), a loop body only on its first pass.
//
// The loads run ahead of the math as a register pipeline: two register sets hold the codes
// and scales of the next two rounds (they come from HBM: far), one set the rows of x of the
// next round (from L2: near).  A set goes to LDS as soon as its turn comes and is requested
// again at once, so a wave has 2*R KiB of codes in flight while it computes.
// ------------------------------------------------------------------------------------------
template <int XR, int R>
struct RoundLds {
    static constexpr int W_BYTES = R * 1024;
    static constexpr int SEG = R * 64;                         // bytes of one row of x in a round
    static constexpr int XROW = SEG + 16;                      // +16: rows 4 banks apart
    static constexpr int X_BYTES = XR * XROW;
    static constexpr int SC_BYTES = 1024;                      // up to 8 groups x 128 bytes
    static constexpr int NXL = XR * SEG / 1024;                // wave-wide loads for the rows of x
    static constexpr int BYTES = W_BYTES + X_BYTES + SC_BYTES; // per wave
};

template <int R>
struct RoundW {
    u32x4 w[R];                                  // packed codes
    u32x4 sc;                                    // the round's scale groups (up to 8 x 128 bytes)
};

template <int XR, int R>
struct RoundX {
    u32x4 x[RoundLds<XR, R>::NXL];
};

// Request the codes and scales of one round: k-steps [ks, ks + R) of the tile.  A request past
// the wave's range (!in) becomes a read of the tile's first 16 bytes by every lane: all loads
// stay unconditional, so the waits the compiler derives stay exact.
template <int R>
__device__ __forceinline__ void round_issue_w(RoundW<R> &rw, const uint4 *codes_tile, const uint2 *scales_tile,
                                              int spg, int ks, bool in, int lane)
{
    const u32x4 *wp = reinterpret_cast<const u32x4 *>(codes_tile) + (in ? (size_t)ks * 64 + lane : 0);
#pragma unroll
    for (int i = 0; i < R; ++i) rw.w[i] = __builtin_nontemporal_load(wp + (in ? i * 64 : 0));   // (read once)
    // the round's groups are contiguous: 128 bytes each, lane l takes bytes 16*l.. (past the
    // round's last group the blob's slack keeps the read in bounds)
    // (R / spg groups of 128 bytes: the lanes beyond them re-read the first 16 bytes)
    const bool mine = lane < (R / spg) * 8;
    rw.sc = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(scales_tile) +
                                       (in ? (size_t)(ks / spg) * 8 + (mine ? lane : 0) : 0));
}

// Request the rows of x (clamped to the chunk's rows and to K) of one round.
template <int XR, int R>
__device__ __forceinline__ void round_issue_x(RoundX<XR, R> &rx, const uint16_t *x, int K, int m0, int rows_here,
                                              int ks, bool in, int lane)
{
    using L = RoundLds<XR, R>;
    // (one uniform base and a 32-bit offset per load: eight 64-bit addresses would cost registers)
    const unsigned char *xb = reinterpret_cast<const unsigned char *>(x + (size_t)m0 * K);
#pragma unroll
    for (int i = 0; i < L::NXL; ++i) {
        const int byte = i * 1024 + lane * 16;
        const int row = min(byte / L::SEG, rows_here - 1);
        const int k = min(ks * KSTEP + (byte % L::SEG) / 2, K - 8);
        const unsigned off = in ? ((unsigned)row * (unsigned)K + (unsigned)k) * 2u : 0u;
        rx.x[i] = *reinterpret_cast<const u32x4 *>(xb + off);
    }
}

template <int XR, int R>
__device__ __forceinline__ void round_to_lds(const RoundW<R> &rw, const RoundX<XR, R> &rx, unsigned char *buf, int lane)
{
    using L = RoundLds<XR, R>;
#pragma unroll
    for (int i = 0; i < R; ++i) *reinterpret_cast<u32x4 *>(buf + i * 1024 + lane * 16) = rw.w[i];
#pragma unroll
    for (int i = 0; i < L::NXL; ++i) {
        const int byte = i * 1024 + lane * 16;
        *reinterpret_cast<u32x4 *>(buf + L::W_BYTES + (byte / L::SEG) * L::XROW + byte % L::SEG) = rx.x[i];
    }
    *reinterpret_cast<u32x4 *>(buf + L::W_BYTES + L::X_BYTES + lane * 16) = rw.sc;
}

// Math of one round: n_steps (a multiple of 4) k-steps starting at the front of the buffer.
// One loop pass = one scale group = SPG k-steps.
template <int MB, int XR, int R, int SPG>
__device__ __forceinline__ void round_compute(f32x4 (&acc)[MB][4], const unsigned char *buf,
                                              int n_steps, int rows_here, bool full, int lane)
{
    using L = RoundLds<XR, R>;
    const int l16 = lane & 15, lq = lane >> 4;
    const unsigned char *wl = buf + lane * 16;
    const unsigned char *xl[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
        xl[mb] = buf + L::W_BYTES + min(mb * 16 + l16, rows_here - 1) * L::XROW + 16 * lq;
    const unsigned char *sl = buf + L::W_BYTES + L::X_BYTES + l16 * 8;
#pragma nounroll
    for (int g = 0; g < n_steps / SPG; ++g) {
        uint4 xf[MB][SPG];
        u32x4 wf[SPG];
#pragma unroll
        for (int s = 0; s < SPG; ++s) {
            wf[s] = *reinterpret_cast<const u32x4 *>(wl + (g * SPG + s) * 1024);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
                xf[mb][s] = *reinterpret_cast<const uint4 *>(xl[mb] + (g * SPG + s) * 64);
        }
        const uint2 sv = *reinterpret_cast<const uint2 *>(sl + g * 128);
        f32x4 d[MB][4];
#pragma unroll
        for (int s = 0; s < SPG; ++s) {
            const auto cb = split_codes<false>(wf[s], full);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint4 wb = codes_to_bf16(cb.lo[j], cb.hi[j]);
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) d[mb][j] = mfma16(xf[mb][s], wb, s == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : d[mb][j]);
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float sj = j == 0 ? half_bits_lo(sv.x) : j == 1 ? half_bits_hi(sv.x)
                           : j == 2 ? half_bits_lo(sv.y) : half_bits_hi(sv.y);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[mb][j][e] = fmaf(d[mb][j][e], sj, acc[mb][j][e]);
        }
    }
}

// ------------------------------------------------------------------------------------------
// Decode shapes (at most 16 rows per chunk): a wave has at most 16 k-steps, so there is no
// steady state to speak of and the K loop is a register pipeline instead of rounds.  The rows
// of x for the wave's whole range go to a wave-private LDS buffer once; the packed codes stay
// in registers, four k-steps deep, and each k-step's register is refilled as soon as it has
// been consumed.  Little state per wave (4 KiB of codes in flight, under 128 registers) lets
// four blocks share a compute unit, so every block of a decoder layer is resident at once and
// the bytes in flight come from the number of waves rather than from the depth of each.
// ------------------------------------------------------------------------------------------
template <int XR>
struct StreamLds {
    static constexpr int XSTEPS = UNIT_SUPER_STEPS;            // k-steps per wave: (16 super-steps x 4) / 4 waves
    static constexpr int XROW = XSTEPS * 64 + 16;              // bytes of a row of x; +16: rows 4 banks apart
    static constexpr int BYTES = XR * XROW;                    // per wave
};

// Codes and scales of one super-step (four k-steps); a wave keeps two of them in flight.
struct StreamRegs {
    u32x4 w[4];
    uint2 sc[4];                                               // one per scale group of the super-step
};

// Request super-step `ss` of the wave (wp0/sp0 = the wave's first chunk / first group WITHOUT the
// lane's offset).  A request past the wave's range (ss >= n_ss) becomes one 16-byte read of the
// first chunk by all lanes: every load stays unconditional, so the waits the compiler derives
// stay exact, and the useless ones cost next to nothing.
// gs = scale groups of a super-step, at most MAX_GS; what is left of the registers takes the last one.
template <int MAX_GS>
__device__ __forceinline__ void stream_request(StreamRegs &r, const u32x4 *wp0, const uint2 *sp0, int ss, int n_ss, int lane, int gs)
{
    const bool in = ss < n_ss;
    const u32x4 *wn = wp0 + (in ? (size_t)ss * 256 + lane : 0);
    const uint2 *sn = sp0 + (in ? (size_t)ss * gs * 16 + (lane & 15) : 0);
#pragma unroll
    for (int u = 0; u < 4; ++u) r.w[u] = __builtin_nontemporal_load(wn + (in ? u * 64 : 0));
#pragma unroll
    for (int g = 0; g < MAX_GS; ++g) {
        // (the scales' type is HIP's struct, which the builtin does not take: read as two words)
        const unsigned long long v = __builtin_nontemporal_load(
            reinterpret_cast<const unsigned long long *>(sn + (in ? min(g, gs - 1) * 16 : 0)));
        r.sc[g] = make_uint2((unsigned)v, (unsigned)(v >> 32));
    }
}

// The math of one super-step; xs = this lane's row of x in LDS at the super-step's first k-step.
template <int SPG>
__device__ __forceinline__ void stream_math(f32x4 (&acc)[4], const StreamRegs &r, const unsigned char *xs, bool full)
{
    constexpr int GS = 4 / SPG;                                // scale groups per super-step
#pragma unroll
    for (int g = 0; g < GS; ++g) {
        f32x4 d[4];
#pragma unroll
        for (int t = 0; t < SPG; ++t) {
            const uint4 xa = *reinterpret_cast<const uint4 *>(xs + (g * SPG + t) * 64);
            const auto cb = split_codes<true>(r.w[g * SPG + t], full);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                d[j] = mfma16(xa, codes_to_bf16(cb.lo[j], cb.hi[j]), t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : d[j]);
        }
        const uint2 sv = r.sc[g];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float sj = j == 0 ? half_bits_lo(sv.x) : j == 1 ? half_bits_hi(sv.x)
                           : j == 2 ? half_bits_lo(sv.y) : half_bits_hi(sv.y);
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(d[j][e], sj, acc[j][e]);
        }
    }
}

// n_ss super-steps (at most 4), two per pass: set A holds the even ones, set B the odd ones, and
// each set is requested again (two super-steps ahead) as soon as it has been consumed.  xl = this
// lane's row of x in LDS (+ 16 * (lane/16)).  During the last pass the wave also reads the two
// completion counters its epilogue depends on (poll_s, poll_p; before that, and for a wave that
// depends on nothing, a dummy address): if they are complete by then, the epilogue need not wait
// for a poll of its own.
template <int SPG>
__device__ __forceinline__ void stream_loop(f32x4 (&acc)[4], bool full, StreamRegs &ra, StreamRegs &rb, const u32x4 *wp0,
                                            const uint2 *sp0, int n_ss, const unsigned char *xl, int lane,
                                            const unsigned *poll_s, const unsigned *poll_p,
                                            unsigned &seen_s, unsigned &seen_p)
{
    constexpr int GS = 4 / SPG;                                // scale groups per super-step
    const unsigned *dummy = reinterpret_cast<const unsigned *>(wp0);
#pragma nounroll
    for (int ss = 0; ss < n_ss; ss += 2) {
        const bool last = ss + 2 >= n_ss;
        seen_s = __hip_atomic_load(last ? poll_s : dummy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        seen_p = __hip_atomic_load(last ? poll_p : dummy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        stream_math<SPG>(acc, ra, xl + ss * 256, full);
        stream_request<GS>(ra, wp0, sp0, ss + 2, n_ss, lane, GS);
        if (ss + 1 < n_ss) stream_math<SPG>(acc, rb, xl + (ss + 1) * 256, full);
        stream_request<GS>(rb, wp0, sp0, ss + 3, n_ss, lane, GS);
    }
}

// Loads the epilogue needs that do not depend on other blocks, requested ahead of their use (all
// unconditional; a thread with nothing to fetch re-reads a valid address).  The N outputs of a
// thread lie in one row, 16 columns apart, so their rows of B differ by a fixed stride.
template <int N, int MBR, int FR>
struct EpiPrefetch {
    static constexpr int H = FR / 16;        // entries of t per thread and row block
    const uint16_t *bad[MBR];                // B of each row's adapter (or a safe address)
    int brank[MBR];                          // rank (0 with the safe address: every offset is 0)
    int n0, nlast;                           // column of output 0; last valid column
    // entries of t this thread sums: row t_ml + 16 * i, rank indices t_jj + 16 * h
    const float *tp[MBR][H];                 // the entry in t_part[0] (or a safe address)
    size_t tstride[MBR][H];                  // distance between K chunks of t_part (0 with the safe address)
    int kch, t_ml, t_jj;
    bool t_mine[MBR][H];
    uint4 b[N > 0 ? N : 1][FR / 8];
    __device__ __forceinline__ void issue()
    {
        // (global, not generic, loads: a generic load also counts as an LDS access, and every
        // later wait for LDS would wait for these as well)
        using G = const __attribute__((address_space(1))) u32x4;
#pragma unroll
        for (int q = 0; q < N; ++q) {
            const int mb = q >> 2;
            // the address passes through an empty asm: without it the compiler hoists these loads
            // to the top of the kernel and then spills their results across the whole K loop
            if ((q & 3) == 0) asm volatile("" : "+v"(bad[mb]));
            const uint16_t *row = bad[mb] + (unsigned)(min(n0 + 16 * (q & 3), nlast) * brank[mb]);
#pragma unroll
            for (int c = 0; c < FR / 8; ++c)     // (pieces past the rank re-read the first one)
                b[q][c] = __builtin_bit_cast(uint4, *(G *)(row + (brank[mb] > 8 * c ? 8 * c : 0)));
        }
    }
};

// sum over the 16 lanes of a row of lanes (DPP rotations, fixed order); every lane gets the result
__device__ __forceinline__ float row_sum16(float v)
{
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x122, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x121, 0xF, 0xF, false));
    return v;
}

// Outputs of a fused call: the four values a lane holds of one row, columns 16 * j + l16 of a
// tile (so (v[0], v[2]) and (v[1], v[3]) are the pairs 32 columns apart), go through the
// projection's EpiArgs and are stored one by one.  The 16 lanes that differ in l16 only hold the
// same row and reach these calls together (m does not depend on l16): they share the sums over a
// row.  What the output stage reads from memory is fetched by fused_fetch, which a caller may
// issue well before the values are there (the loads then overlap what else it waits for).
struct FusedOperands {
    float scale_or_sum;            // row_scale[m], or this lane's share of the sums of squares
    float cs[2], sn[2];            // rotary cosines and sines of the lane's two pairs
    float res[4];                  // residual of the lane's four (SwiGLU: two) outputs
};

__device__ __forceinline__ FusedOperands fused_fetch(const LaunchArgs &a, const ProjArgs &P, int pi, int m, int tile, int l16)
{
    FusedOperands f;
    const EpiArgs &E = a.epi[pi];
    const int mm = min(m, a.M - 1);                        // (rows past the end fetch a valid row and store nothing)
    f.scale_or_sum = 1.0f;
    if (E.row_scale) f.scale_or_sum = E.row_scale[mm];
    if (E.sq_in) {
        float sum = 0.f;
        for (int p = l16; p < E.sq_parts; p += 16) sum += E.sq_in[(size_t)mm * E.sq_parts + p];
        f.scale_or_sum = sum;
    }
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
        f.cs[jj] = 1.0f;
        f.sn[jj] = 0.0f;
        if (E.pair_op == PAIR_ROPE) {
            f.cs[jj] = E.rope_cos[(size_t)mm * 32 + 16 * jj + l16];
            f.sn[jj] = E.rope_sin[(size_t)mm * 32 + 16 * jj + l16];
        }
    }
    const int n_out = E.pair_op == PAIR_SWIGLU ? P.N >> 1 : P.N;
    const int n0 = tile * (E.pair_op == PAIR_SWIGLU ? TILE_N / 2 : TILE_N) + l16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f.res[j] = 0.0f;
        if (E.residual && (E.pair_op != PAIR_SWIGLU || j < 2))
            f.res[j] = bf16_bits_to_float(E.residual[(size_t)mm * n_out + min(n0 + 16 * j, n_out - 1)]);
    }
    return f;
}

__device__ __forceinline__ void fused_store(const LaunchArgs &a, const ProjArgs &P, int pi, int m, int tile, int l16,
                                            const FusedOperands &f, float (&v)[4])
{
    if (m >= a.M) return;
    const EpiArgs &E = a.epi[pi];
    float rs = f.scale_or_sum;
    if (E.sq_in) rs = 1.0f / sqrtf(row_sum16(f.scale_or_sum) / (float)P.K + E.sq_eps);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] *= rs;
    const int N = P.N;
    float sq = 0.f;                                        // squares of what this lane stores
    auto put = [&](size_t at, float o) {
        if (a.y_fp32) {
            reinterpret_cast<float *>(P.y)[at] = o;
        } else {
            const uint16_t h = float_to_bf16_bits(o);
            reinterpret_cast<uint16_t *>(P.y)[at] = h;
            o = bf16_bits_to_float(h);
        }
        sq = fmaf(o, o, sq);
    };
    if (E.pair_op == PAIR_SWIGLU) {
        const int n_out = N >> 1;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
            const int n = tile * (TILE_N / 2) + 16 * jj + l16;
            const float g = v[jj];
            if (n < n_out) put((size_t)m * n_out + n, g / (1.0f + expf(-g)) * v[jj + 2] + f.res[jj]);
        }
    } else {
        if (E.pair_op == PAIR_ROPE) {
#pragma unroll
            for (int jj = 0; jj < 2; ++jj) {
                const float x0 = v[jj], x1 = v[jj + 2];
                v[jj] = x0 * f.cs[jj] - x1 * f.sn[jj];
                v[jj + 2] = x1 * f.cs[jj] + x0 * f.sn[jj];
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = tile * TILE_N + 16 * j + l16;
            if (n < N) put((size_t)m * N + n, v[j] + f.res[j]);
        }
    }
    if (E.sq_out) {
        sq = row_sum16(sq);
        if (l16 == 0) E.sq_out[(size_t)m * tiles_n(N) + tile] = sq;
    }
}

__device__ __forceinline__ void store_fused(const LaunchArgs &a, const ProjArgs &P, int pi, int m, int tile, int l16,
                                            float (&v)[4])
{
    const FusedOperands f = fused_fetch(a, P, pi, m, tile, l16);
    fused_store(a, P, pi, m, tile, l16, f, v);
}

// the epilogue prefetch covers ranks up to this: 16 in the kernels for up to 16 rows (their register
// budget), 32 where a chunk has 32 rows (the prefetch there starts once the K loop's registers are free)
template <int MB> constexpr int fast_rank() { return MB == 1 ? 16 : 32; }

// LDS of a base block: the per-wave staging buffers, the per-wave partial tiles (red) and
// alpha * t of the chunk's rows.  Decode shapes: a wave's partial tile lies over its OWN staging
// buffer and t has room of its own, so a wave that is done with its K loop need not wait for the
// others before it writes either.  Above 16 rows red and t lie over the staging buffers of all
// waves and the block meets first.
template <int MB, int XR, int WAVES, int R>
struct BaseLds {
    static constexpr bool PRIVATE = MB == 1;
    static constexpr int WAVE_STAGE = PRIVATE ? StreamLds<XR>::BYTES : RoundLds<XR, R>::BYTES;
    static constexpr int STAGE_BYTES = WAVES * WAVE_STAGE;
    static constexpr int RED_WAVE = MB * 1024 * 4;             // bytes of one wave's partial tile
    static constexpr int TS_STRIDE = MLORA_MAX_RANK + 4;
    static constexpr int TS_BYTES = (PRIVATE ? XR : 16 * MB) * TS_STRIDE * 4;
    static constexpr int T_AT = PRIVATE ? STAGE_BYTES : WAVES * RED_WAVE;
    static constexpr int BYTES = T_AT + TS_BYTES > STAGE_BYTES ? T_AT + TS_BYTES : STAGE_BYTES;
    static_assert(!PRIVATE || WAVE_STAGE >= RED_WAVE, "a wave's partial tile must fit its own staging buffer");
    unsigned char *base;
    __device__ unsigned char *stage(int wave) const { return base + wave * WAVE_STAGE; }
    __device__ float *red(int wave) const
    {
        return reinterpret_cast<float *>(base + wave * (PRIVATE ? WAVE_STAGE : RED_WAVE));
    }
    __device__ float *t_row(int ml) const { return reinterpret_cast<float *>(base + T_AT) + ml * TS_STRIDE; }
};

__device__ __forceinline__ float dot8(uint4 b8, const float *t, float l)
{
    l = fmaf(bf16_bits_to_float(b8.x & 0xFFFFu), t[0], l);
    l = fmaf(bf16_bits_to_float(b8.x >> 16), t[1], l);
    l = fmaf(bf16_bits_to_float(b8.y & 0xFFFFu), t[2], l);
    l = fmaf(bf16_bits_to_float(b8.y >> 16), t[3], l);
    l = fmaf(bf16_bits_to_float(b8.z & 0xFFFFu), t[4], l);
    l = fmaf(bf16_bits_to_float(b8.z >> 16), t[5], l);
    l = fmaf(bf16_bits_to_float(b8.w & 0xFFFFu), t[6], l);
    l = fmaf(bf16_bits_to_float(b8.w >> 16), t[7], l);
    return l;
}

// ku == 0: finish the tile (add split-K partials, LoRA term, store y); ku > 0: leave a partial.
// WAVES (= 4) waves split the unit's super-steps.  In the MFMA result layout lane l holds, for
// row block mb and column block j, the rows 16*mb + 4*(l/16) + e (e = 0..3) of column 16*j + l%16;
// thread (wave w, lane l) finishes e = w of every (mb, j): EPT = 4*MB outputs that lie in MB rows
// (one adapter each), 16 columns apart.
template <int MB, int XR, int WAVES, int R, int FR>
__device__ __forceinline__ void base_unit(const LaunchArgs &a, const ProjArgs &P, int pi, int tile, int ku,
                                 int m0, const BaseLds<MB, XR, WAVES, R> &lds)
{
    constexpr int ROWS = 16 * MB;
    constexpr int NT = 64 * WAVES;
    constexpr int EPT = MB * 16 / WAVES;
    const int K = P.K, N = P.N, M = a.M;
    int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int l16 = lane & 15, lq = lane >> 4;
    // the units of a split projection form the longest chain of the launch: they go first
    // wherever they share a SIMD with other waves
    if (P.ksplit > 1) __builtin_amdgcn_s_setprio(2);

    // super-steps of this K unit, then of this wave (balanced splits)
    const int nss = K / SUPER_K;
    const int uq = P.unit_q, ur = P.unit_r;
    const int unit_beg = ku * uq + min(ku, ur), unit_cnt = uq + (ku < ur ? 1 : 0);
    const int q = unit_cnt / WAVES, r = unit_cnt % WAVES;
    const int my_cnt = q + (wave < r ? 1 : 0);
    // a wave without work still issues (valid) loads: point it at the unit's first super-step
    const int my_beg = my_cnt > 0 ? unit_beg + wave * q + min(wave, r) : unit_beg;

    const int ksteps = K / KSTEP;
    const int ngroups = ksteps >> P.spg_shift;
    const uint4 *codes_tile = P.codes + (size_t)tile * ksteps * 64;
    const uint2 *scales_tile = P.scales + (size_t)tile * ngroups * 16;

    // what this thread will finish, and the adapter of each of its rows
    const bool lora = (ku == 0) && (a.row_adapter != nullptr) && (P.n_adapters > 0);
    const int rows_here = min(ROWS, M - m0);
    constexpr bool PREFETCH = EPT <= 8;                    // more outputs per thread: too many registers
    // (ranks up to FR: the entries of t of a chunk number at most MB * FR / 16 per thread)
    const bool fast = PREFETCH && lora && P.rank <= FR;
    // element qq of this thread: tile row and column (cheap to recompute, so not kept live)
    static_assert(WAVES == 4, "one wave per element of an MFMA result register");
    auto elem_ml = [&](int qq) { return (qq >> 2) * 16 + 4 * lq + wave; };
    auto elem_col = [&](int qq) { return 16 * (qq & 3) + l16; };
    const int *ra_safe = lora ? a.row_adapter : reinterpret_cast<const int *>(P.codes);
    const int ra_last = lora ? M - 1 : 0;
    int ad_raw[MB];                                        // as loaded, one per row of this thread
    auto elem_ad = [&](int qq) {
        const int v = ad_raw[qq >> 2];
        return (lora && m0 + elem_ml(qq) < M && v >= 0 && v < P.n_adapters) ? v : -1;
    };

    f32x4 acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[mb][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // epilogue operands fetched while the last round is being computed: the rows of B of this
    // thread's outputs (ranks up to FR) and its entries of t
    EpiPrefetch<PREFETCH ? EPT : 0, MB, FR> pf;
    constexpr int TH = FR / 16;
    auto prefetch_setup = [&]() {
        pf.t_ml = tid >> 4;
        pf.t_jj = tid & 15;
        pf.n0 = tile * TILE_N + l16;
        pf.nlast = N - 1;
        pf.kch = P.kch;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int ad = elem_ad(4 * i);
            const bool ok = fast && ad >= 0;
            pf.bad[i] = ok ? P.lora_b + (size_t)ad * N * P.rank : reinterpret_cast<const uint16_t *>(P.codes);
            pf.brank[i] = ok ? P.rank : 0;
#pragma unroll
            for (int h = 0; h < TH; ++h) {
                pf.t_mine[i][h] = fast && pf.t_ml + 16 * i < rows_here && pf.t_jj + 16 * h < P.r16;
                pf.tp[i][h] = pf.t_mine[i][h] ? P.t_part + (size_t)(m0 + pf.t_ml + 16 * i) * P.r16 + pf.t_jj + 16 * h
                                              : reinterpret_cast<const float *>(P.codes);
                pf.tstride[i][h] = pf.t_mine[i][h] ? (size_t)M * P.r16 : 0;
            }
        }
    };
    // alpha * t of this thread's entries -> LDS: the K-chunk partials of the shrink step, all
    // requested at once and summed in fixed order
    auto t_entries_to_lds = [&]() {
        constexpr int E = MB * TH;                         // entries of this thread: (row block i, half h) = e / TH, e % TH
        float ts[E];
        if (pf.kch <= 4) {
            float tv[E][4];
#pragma unroll
            for (int e = 0; e < E; ++e)
#pragma unroll
                for (int kc = 0; kc < 4; ++kc)
                    tv[e][kc] = load_shared(pf.tp[e / TH][e % TH] + (size_t)min(kc, pf.kch - 1) * pf.tstride[e / TH][e % TH]);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                ts[e] = 0.f;
#pragma unroll
                for (int kc = 0; kc < 4; ++kc) ts[e] += kc < pf.kch ? tv[e][kc] : 0.f;
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                float tv[MAX_KCHUNKS];
#pragma unroll
                for (int kc = 0; kc < MAX_KCHUNKS; ++kc)
                    tv[kc] = load_shared(pf.tp[e / TH][e % TH] + (size_t)min(kc, pf.kch - 1) * pf.tstride[e / TH][e % TH]);
                ts[e] = 0.f;
#pragma unroll
                for (int kc = 0; kc < MAX_KCHUNKS; ++kc) ts[e] += kc < pf.kch ? tv[kc] : 0.f;
            }
        }
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (pf.t_mine[e / TH][e % TH]) lds.t_row(pf.t_ml + 16 * (e / TH))[pf.t_jj + 16 * (e % TH)] = ts[e] * P.alpha;
    };

    // counters this block depends on (or signals): see common.hpp
    const int tiles = tiles_n(N);
    const int chunk = m0 / ROWS, chunks = a.m_pad / ROWS;
    const int fin = tile * chunks + chunk;                 // this finishing block among its projection's
    const int copies = P.ctr_copies;                       // copies of the shrink counter in use (a power of two)
    unsigned *const sctr = a.ctrl + shrink_ctr(pi, fin & (copies - 1));
    unsigned *const pctr = a.ctrl + P.part_ctr + fin * CTR_STRIDE;
    const bool need_s = lora, need_p = ku == 0 && P.ksplit > 1;
    unsigned seen_s = 0, seen_p = 0;                       // what an early look at them showed

    unsigned char *buf = lds.stage(wave);
    const int ks_first = my_beg * 4, ks_total = my_cnt * 4;
    const int rows_x = min(rows_here, XR);
    if constexpr (MB == 1) {
        // decode shapes: rows of x of the wave's whole range -> LDS, then the register pipeline
        using L = StreamLds<XR>;
        u32x4 xr[XR];
        const int kx = min(ks_first * KSTEP + lane * 8, K - 8);
#pragma unroll
        for (int i = 0; i < XR; ++i)
            xr[i] = *reinterpret_cast<const u32x4 *>(P.x + (size_t)(m0 + min(i, rows_x - 1)) * K + kx);
        // adapters of this thread's rows: requested here (unconditionally), decoded below
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) ad_raw[mb] = ra_safe[min(m0 + elem_ml(4 * mb), ra_last)];
        const u32x4 *wp = reinterpret_cast<const u32x4 *>(codes_tile) + (size_t)ks_first * 64;
        const uint2 *sp = scales_tile + (size_t)(ks_first >> P.spg_shift) * 16;
        const unsigned char *xl = buf + min(l16, rows_x - 1) * L::XROW + 16 * lq;
        const unsigned *dummy = reinterpret_cast<const unsigned *>(wp);
        const unsigned *poll_s = need_s ? sctr : dummy, *poll_p = need_p ? pctr : dummy;
        StreamRegs sa, sb;
        auto request = [&](auto max_gs, int gs) {
            const uint32_t flag = request_flag(P);
            // an idle wave requests (and ignores) the unit's first super-step
            stream_request<decltype(max_gs)::value>(sa, wp, sp, 0, max(my_cnt, 1), lane, gs);
            stream_request<decltype(max_gs)::value>(sb, wp, sp, 1, my_cnt, lane, gs);
            __builtin_amdgcn_sched_barrier(0);                 // (the requests stay ahead of the wait for x)
#pragma unroll
            for (int i = 0; i < XR; ++i) *reinterpret_cast<u32x4 *>(buf + lane * 16 + i * L::XROW) = xr[i];
            return flag;
        };
        auto by_group = [&](auto go) {
            if (P.spg == 1)      go(std::integral_constant<int, 1>{});
            else if (P.spg == 2) go(std::integral_constant<int, 2>{});
            else                 go(std::integral_constant<int, 4>{});
        };
        auto loop = [&](auto spg, uint32_t flag) {
            stream_loop<decltype(spg)::value>(acc[0], flag_set(flag), sa, sb, wp, sp, my_cnt, xl, lane, poll_s, poll_p, seen_s, seen_p);
        };
        // The first requests belong to the loop of their group size: made ahead of the branch, each register set would
        // be moved to where the loop wants it, and a move waits for its data (16 layers at 16 rows 195 us against
        // 190).  But the branch is a jump to code that is not in the cache yet, and units of at most two super-steps per
        // wave have nothing else to hide it: with 9 to 16 rows per block they make their requests first, in the code
        // that follows (640 x 3673 at 27 rows 9.1 -> 8.5 us, 768 x 3847 at 28 9.2 -> 8.7, 1024 x 1078 at 28 9.2 -> 8.9).
        if (XR == 16 && __builtin_expect(unit_cnt <= 2 * WAVES, 1)) {
            const uint32_t flag = request(std::integral_constant<int, 4>{}, 4 >> P.spg_shift);
            by_group([&](auto spg) { loop(spg, flag); });
        } else {
            by_group([&](auto spg) {
                constexpr int GS = 4 / decltype(spg)::value;
                loop(spg, request(std::integral_constant<int, GS>{}, GS));
            });
        }
        // Everything below derives its indices afresh from the thread id: values shared with the
        // code above the loop would have to live across it, in registers the loop needs.
        asm volatile("" : "+v"(tid));
        lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
        // rows of B: in flight during what follows.  (The empty asm keeps the decoding of the
        // adapter index, and with it state that would live across the loop, behind the loop.)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) asm volatile("" : "+v"(ad_raw[mb]));
        prefetch_setup();
        pf.issue();
    } else {
        // K loop, two rounds per pass.  An idle wave (my_cnt == 0) still requests one round at a
        // valid place and computes nothing.
        const int nr = ks_total / R;                           // rounds of this wave
        RoundW<R> wa, wb;
        RoundX<XR, R> xr;
        const uint32_t flag = request_flag(P);
        round_issue_w<R>(wa, codes_tile, scales_tile, P.spg, ks_first, true, lane);
        round_issue_w<R>(wb, codes_tile, scales_tile, P.spg, ks_first + R, 1 < nr, lane);
        round_issue_x<XR, R>(xr, P.x, K, m0, rows_x, ks_first, true, lane);
        // (keeps all of these requests ahead of the first wait)
        __builtin_amdgcn_sched_barrier(0);
        const bool full = flag_set(flag);
        auto compute = [&](int n) {
            if (P.spg == 1)      round_compute<MB, XR, R, 1>(acc, buf, n, rows_x, full, lane);
            else if (P.spg == 2) round_compute<MB, XR, R, 2>(acc, buf, n, rows_x, full, lane);
            else                 round_compute<MB, XR, R, 4>(acc, buf, n, rows_x, full, lane);
        };
#pragma nounroll
        for (int r0 = 0; r0 < max(nr, 1); r0 += 2) {
            round_to_lds<XR, R>(wa, xr, buf, lane);
            round_issue_w<R>(wa, codes_tile, scales_tile, P.spg, ks_first + (r0 + 2) * R, r0 + 2 < nr, lane);
            round_issue_x<XR, R>(xr, P.x, K, m0, rows_x, ks_first + (r0 + 1) * R, r0 + 1 < nr, lane);
            // (the scheduler would otherwise sink the requests below the math to save registers)
            __builtin_amdgcn_sched_barrier(0);
            compute(r0 < nr ? R : 0);
            round_to_lds<XR, R>(wb, xr, buf, lane);
            round_issue_w<R>(wb, codes_tile, scales_tile, P.spg, ks_first + (r0 + 3) * R, r0 + 3 < nr, lane);
            round_issue_x<XR, R>(xr, P.x, K, m0, rows_x, ks_first + (r0 + 2) * R, r0 + 2 < nr, lane);
            __builtin_amdgcn_sched_barrier(0);
            compute(r0 + 1 < nr ? R : 0);
        }
        // Everything below derives its indices afresh from the thread id: values shared with the
        // code above the loop would have to live across it, in registers the loop needs.
        asm volatile("" : "+v"(tid));
        lane = tid & 63, wave = tid >> 6, l16 = lane & 15, lq = lane >> 4;
        // adapters of this thread's rows, then their rows of B: requested once the rounds'
        // registers are free
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) ad_raw[mb] = ra_safe[min(m0 + elem_ml(4 * mb), ra_last)];
        prefetch_setup();
        pf.issue();
    }

    // Above 16 rows the partial tiles and t lie over the staging buffers of all waves: meet first.
    if constexpr (!BaseLds<MB, XR, WAVES, R>::PRIVATE) __syncthreads();
    // What the epilogue reads from other blocks.  Every wave makes sure of it for itself (all
    // lanes poll the same word), unless the look during its last super-step already showed it.
    // A wave whose wait runs out sets the workspace's status word and stores NaN in place of its
    // outputs: a call that went wrong must not look like one that went right.
    bool poisoned = false;
    {
        const int limit = a.spin_limit;
        bool ok = true;
        if (need_s && (limit == 0 || seen_s < (unsigned)P.n_shrink_blocks)) ok = wait_count(sctr, (unsigned)P.n_shrink_blocks, limit);
        if (need_p && (limit == 0 || seen_p < (unsigned)(P.ksplit - 1))) ok = wait_count(pctr, (unsigned)(P.ksplit - 1), limit) && ok;
        compiler_fence();
        if (!ok && lane == 0) atomicOr(a.status, 1u);
        poisoned = !ok;
    }
    const float nan_f = __uint_as_float(0x7FC00000u);

    // partial tiles -> LDS: element (mb, j, e) of lane l at red_at(mb, e, l) + j, so that the thread
    // that finishes e of every j reads four of them at once
    auto red_at = [](int mb, int e, int l) { return ((mb * 4 + e) * 64 + l) * 4; };
    {
        float *red = lds.red(wave);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                *reinterpret_cast<f32x4 *>(red + red_at(mb, e, lane)) =
                    f32x4{acc[mb][0][e], acc[mb][1][e], acc[mb][2][e], acc[mb][3][e]};
    }

    constexpr int PU = 7;                                  // split-K units (beside the block's own) the short way out adds
    // The common decode case gets a short, nearly branch-free way out (code that runs once per
    // launch is paid for by the instruction fetch, so its length is its cost): a finishing block
    // whose LoRA term, if any, was prefetched above and whose K has at most PU + 1 units.
    const bool lean = PREFETCH && ku == 0 && (!lora || fast) && P.ksplit <= PU + 1;
    if (lean) {
        if constexpr (PREFETCH) {
            // a fused call's operands of the output stage: on their way while t and the partial
            // tiles are fetched
            FusedOperands fo[MB];
            if (a.fused) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb) fo[mb] = fused_fetch(a, P, pi, m0 + elem_ml(4 * mb), tile, l16);
            }
            if (lora) t_entries_to_lds();
            float pv[EPT][PU];
            if (P.ksplit > 1) {
                const size_t ustride = (size_t)tiles * a.m_pad * TILE_N;
#pragma unroll
                for (int qq = 0; qq < EPT; ++qq) {
                    const int m = min(m0 + elem_ml(qq), M - 1);
                    const float *src = P.partial + ((size_t)tile * a.m_pad + m) * TILE_N + elem_col(qq);
#pragma unroll
                    for (int u = 0; u < 3; ++u) pv[qq][u] = load_shared(src + (size_t)min(u, P.ksplit - 2) * ustride);
                }
                // (more than four units: K above 8192; the common case does not pay for these loads)
                if (PU > 3 && P.ksplit > 4) {
#pragma unroll
                    for (int qq = 0; qq < EPT; ++qq) {
                        const int m = min(m0 + elem_ml(qq), M - 1);
                        const float *src = P.partial + ((size_t)tile * a.m_pad + m) * TILE_N + elem_col(qq);
#pragma unroll
                        for (int u = 3; u < PU; ++u) pv[qq][u] = load_shared(src + (size_t)min(u, P.ksplit - 2) * ustride);
                    }
                } else {
#pragma unroll
                    for (int qq = 0; qq < EPT; ++qq)
#pragma unroll
                        for (int u = 3; u < PU; ++u) pv[qq][u] = 0.f;
                }
            }
            __syncthreads();
            const int n0 = tile * TILE_N + l16;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                f32x4 v = *reinterpret_cast<const f32x4 *>(lds.red(0) + red_at(mb, wave, lane));
#pragma unroll
                for (int w = 1; w < WAVES; ++w)
                    v += *reinterpret_cast<const f32x4 *>(lds.red(w) + red_at(mb, wave, lane));
                if (P.ksplit > 1) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int u = 0; u < PU; ++u) v[j] += u + 1 < P.ksplit ? pv[4 * mb + j][u] : 0.f;
                }
                if (lora) {
                    // (entries of a row of t past the rank are not written and not used)
                    float t[FR];
                    const f32x4 *tr = reinterpret_cast<const f32x4 *>(lds.t_row(elem_ml(4 * mb)));
#pragma unroll
                    for (int i = 0; i < FR / 4; ++i) {
                        const f32x4 tq = tr[i];
                        t[4 * i] = tq[0]; t[4 * i + 1] = tq[1]; t[4 * i + 2] = tq[2]; t[4 * i + 3] = tq[3];
                    }
                    const bool mine = elem_ad(4 * mb) >= 0;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        float l = dot8(pf.b[4 * mb + j][0], t, 0.f);
#pragma unroll
                        for (int c = 1; c < FR / 8; ++c)
                            if (P.rank > 8 * c) l = dot8(pf.b[4 * mb + j][c], t + 8 * c, l);
                        v[j] += mine ? l : 0.f;
                    }
                }
                const int m = m0 + elem_ml(4 * mb);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = poisoned ? nan_f : v[j];
                if (a.fused) {
                    float vv[4] = {v[0], v[1], v[2], v[3]};
                    fused_store(a, P, pi, m, tile, l16, fo[mb], vv);
                } else if (m < M) {
                    if (a.y_fp32) {
                        float *yp = reinterpret_cast<float *>(P.y) + (size_t)m * N + n0;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (n0 + 16 * j < N) yp[16 * j] = v[j];
                    } else {
                        uint16_t *yp = reinterpret_cast<uint16_t *>(P.y) + (size_t)m * N + n0;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            if (n0 + 16 * j < N) yp[16 * j] = float_to_bf16_bits(v[j]);
                    }
                }
            }
        }
    } else {
        // split-K partials of this thread's outputs: all requested at once (a thread with nothing to
        // add re-reads a valid address), consumed after the reduction below
        constexpr int PU = 3;
        float pv[EPT][PU];
#pragma unroll
        for (int qq = 0; qq < EPT; ++qq)
#pragma unroll
            for (int u = 0; u < PU; ++u) {
                const int m = m0 + elem_ml(qq);
                const bool ok = ku == 0 && u + 1 < P.ksplit && m < M;
                const float *src = ok ? P.partial + (((size_t)u * tiles + tile) * a.m_pad + m) * TILE_N + elem_col(qq)
                                      : reinterpret_cast<const float *>(P.codes);
                pv[qq][u] = load_shared(src);
            }
        // t[m] = alpha * sum of the shrink step's K-chunk partials (fixed order)
        if (fast) {
            t_entries_to_lds();
        } else if (lora && MB == 1) {
            // (the kernels for up to 16 rows keep this path short: it is rare there, and its size
            // costs the common path instruction fetches)
            for (int idx = tid; idx < rows_here * P.r16; idx += NT) {
                const int ml = idx / P.r16, jj = idx % P.r16;
                const int ad = a.row_adapter[m0 + ml];
                float v = 0.f;
                if (ad >= 0 && ad < P.n_adapters)
                    for (int kc = 0; kc < P.kch; ++kc)
                        v += load_shared(P.t_part + ((size_t)kc * M + (m0 + ml)) * P.r16 + jj);
                lds.t_row(ml)[jj] = v * P.alpha;
            }
        } else if (lora) {
            // four entries of t per thread and four K chunks at a time: 16 loads in flight instead of
            // one after another (a rank of 32 at 32 rows is four entries per thread, each the sum
            // of up to 16 partials)
            for (int i0 = 0; i0 < rows_here * P.r16; i0 += 4 * NT) {
                float v[4] = {0.f, 0.f, 0.f, 0.f};
                bool live[4];
                const float *src[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int idx = i0 + q * NT + tid;
                    const int ml = min(idx / P.r16, rows_here - 1), jj = idx % P.r16;
                    const int ad = a.row_adapter[m0 + ml];
                    live[q] = idx < rows_here * P.r16 && ad >= 0 && ad < P.n_adapters;
                    src[q] = live[q] ? P.t_part + (size_t)(m0 + ml) * P.r16 + jj : P.t_part;
                }
                for (int kc0 = 0; kc0 < P.kch; kc0 += 4) {
                    float pv[4][4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            pv[q][c] = load_shared(src[q] + (live[q] ? (size_t)min(kc0 + c, P.kch - 1) * M * P.r16 : 0));
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (kc0 + c < P.kch) v[q] += pv[q][c];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int idx = i0 + q * NT + tid;
                    if (idx < rows_here * P.r16) lds.t_row(idx / P.r16)[idx % P.r16] = live[q] ? v[q] * P.alpha : 0.f;
                }
            }
        }
        __syncthreads();

        float fv[EPT];                                     // a fused call's outputs, stored after the loop
#pragma unroll
        for (int qq = 0; qq < EPT; ++qq) fv[qq] = 0.f;
        // ranks above 16: B[a(m)][n] . t[m] of this thread's outputs, the rows of B fetched 32 ranks
        // of four outputs at a time (16 loads in flight), summed in rank order
        float ll[EPT];
#pragma unroll
        for (int qq = 0; qq < EPT; ++qq) ll[qq] = 0.f;
        if (MB == 2 && lora && !fast && ku == 0) {
            for (int jj0 = 0; jj0 < P.rank; jj0 += 32) {
#pragma unroll
                for (int h = 0; h < EPT; h += 4) {
                    uint4 bq[4][4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int ad = elem_ad(h + q);
                        const int n = min(tile * TILE_N + elem_col(h + q), N - 1);
                        const uint16_t *brow = P.lora_b + ((size_t)max(ad, 0) * N + n) * P.rank;
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            bq[q][c] = *reinterpret_cast<const uint4 *>(brow + min(jj0 + 8 * c, P.rank - 8));
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const bool mine = elem_ad(h + q) >= 0;
                        const float *tr = lds.t_row(elem_ml(h + q));
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (mine && jj0 + 8 * c < P.rank) ll[h + q] = dot8(bq[q][c], tr + jj0 + 8 * c, ll[h + q]);
                    }
                }
            }
        }
#pragma unroll
        for (int qq = 0; qq < EPT; ++qq) {
            const int off = red_at(qq >> 2, wave, lane) + (qq & 3);
            float v = lds.red(0)[off];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) v += lds.red(w)[off];
            const int ml = elem_ml(qq), col = elem_col(qq);
            const int m = m0 + ml;
            const int n = tile * TILE_N + col;
            if (ku > 0) {
                store_shared(P.partial + (((size_t)(ku - 1) * tiles + tile) * a.m_pad + m) * TILE_N + col, v);
                continue;
            }
            if (m < M && n < N) {
#pragma unroll
                for (int u = 0; u < PU; ++u)
                    if (u + 1 < P.ksplit) v += pv[qq][u];
                for (int u = PU + 1; u < P.ksplit; ++u)
                    v += load_shared(P.partial + (((size_t)(u - 1) * tiles + tile) * a.m_pad + m) * TILE_N + col);
                const int ad = elem_ad(qq);
                if (ad >= 0) {
                    float l = 0.f;
                    if (fast) {
                        if constexpr (PREFETCH) {
                            l = dot8(pf.b[qq][0], lds.t_row(ml), l);
#pragma unroll
                            for (int c = 1; c < FR / 8; ++c)
                                if (P.rank > 8 * c) l = dot8(pf.b[qq][c], lds.t_row(ml) + 8 * c, l);
                        }
                    } else if (MB == 2) {
                        l = ll[qq];
                    } else {
                        const uint16_t *brow = P.lora_b + ((size_t)ad * N + n) * P.rank;
                        for (int jj = 0; jj < P.rank; jj += 8)
                            l = dot8(*reinterpret_cast<const uint4 *>(brow + jj), lds.t_row(ml) + jj, l);
                    }
                    v += l;
                }
                v = poisoned ? nan_f : v;
                if (a.fused) fv[qq] = v;
                else if (a.y_fp32) reinterpret_cast<float *>(P.y)[(size_t)m * N + n] = v;
                else reinterpret_cast<uint16_t *>(P.y)[(size_t)m * N + n] = float_to_bf16_bits(v);
            }
        }
        if (a.fused && ku == 0) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                float vv[4] = {fv[4 * mb], fv[4 * mb + 1], fv[4 * mb + 2], fv[4 * mb + 3]};
                store_fused(a, P, pi, m0 + elem_ml(4 * mb), tile, l16, vv);
            }
        }
    }
    if (ku > 0) signal_done(pctr, 1);
    // Counters go back to zero for the next call: a tile's split-K counter once every wave has
    // passed it (the barrier above), a copy of the shrink counter by the last block that used it.
    if (tid == 0 && need_p) __hip_atomic_store(pctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0 && need_s) {
        const int users = (P.n_finish_blocks >> (31 - __clz(copies))) + ((fin & (copies - 1)) < (P.n_finish_blocks & (copies - 1)) ? 1 : 0);
        if (atomicAdd(sctr + 1, 1u) + 1u == (unsigned)users) {
            __hip_atomic_store(sctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(sctr + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ------------------------------------------------------------------------------------------
// LoRA shrink
// ------------------------------------------------------------------------------------------
// Rows of x and rank rows of A are both K elements apart, a power of two as a rule: a request
// that takes 16 bytes from each of 16 such rows (an MFMA fragment read directly) lands in one
// memory channel and holds up every other wave of its compute unit.  So both are read in
// contiguous runs (4 rows x 256 bytes per instruction) and turned into fragments through a
// wave-private LDS buffer, four k-steps at a time.
//
// Grouped shrink (more than 16 rows per call).  A block = (chunk of 64 rows, share of the chunk's row
// tiles, 16 ranks, chunk of K).  Wave 0 cuts the rows of every adapter into tiles of 16 (a few ballots).
// Each wave takes a quarter of the K chunk of every tile of the block; the quarters are added through LDS,
// up to four tiles at a time.  What bounds a block is the trips to memory behind one another: a quarter of
// 256 inputs is one trip (two batches in registers), where a wave that worked through a K chunk of a tile by
// itself needed four (t of 14336 inputs, 64 rows, 32 adapters of rank 64: 34 -> 21 us after the start of
// the launch, the whole call 46 -> 33 us).  In a K chunk of one or two batches a quarter would be a batch with one or two
// k-steps in it, and every wave would stage every tile: there one or two waves share a tile (128 x 4991 at 276 rows,
// rank 128, 19.6 -> 16.9 us; 41 drawn calls of 128 inputs 0.94 of the time, 64 of 256 inputs 0.99).  DEPTH = batches
// in registers: four where 256 are there (whose kernels have no registers for that second form).  Blocks of eight waves
// cut a K chunk in eight and stage two k-steps at a time: with four waves at work, or batches of four k-steps (11
// registers spilled), calls with many shrink blocks lost 20 % (14336 x 4096 as above 31.4 -> 39.3 us, now 31.3).
template <int WAVES>
struct ShrinkLds {
    static constexpr int SB = WAVES == 4 ? 4 : 2;           // k-steps per batch
    static constexpr int ROW = SB * 64 + 16;                // bytes of a staged row; +16: rows 4 banks apart
    RowTiles g;
    alignas(16) unsigned char a[WAVES][16 * ROW];           // (16-byte LDS accesses)
    alignas(16) unsigned char x[WAVES][16 * ROW];
    alignas(16) f32x4 red[WAVES][4][64];                    // a wave's share of four tiles
};

// The tiles of one block: share, share + shares, ... of its chunk of rows, four at a time.  PARTS waves share the
// inputs of a tile (a balanced split of the block's k-steps), the others have tiles of their own.
template <bool A8, int DEPTH, int PARTS, int WAVES>
__device__ __forceinline__ void shrink_tiles(const LaunchArgs &a, const ProjArgs &P, ShrinkLds<WAVES> &lds, int m_base, int share, int shares,
                                             int jb, int kc, int blk_beg, int blk_cnt)
{
    using L = ShrinkLds<WAVES>;
    constexpr int SB = L::SB;
    constexpr int LPR = SB * 4, RPI = 64 / LPR;             // lanes per staged row; rows per instruction
    constexpr int STEP = WAVES / PARTS;                     // a wave's tiles of the four: my_slot, my_slot + STEP, ...
    static_assert(STEP <= 4, "every wave has a share of the four tiles");
    RowTiles &g = lds.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lq = lane >> 4, st_row = lane / LPR, st_piece = lane % LPR;
    const int part = wave % PARTS, my_slot = wave / PARTS;
    const int wq = blk_cnt / PARTS, wr = blk_cnt % PARTS;
    const int my_beg = blk_beg + part * wq + min(part, wr), my_cnt = wq + (part < wr ? 1 : 0);
    const int batches = (my_cnt + SB - 1) / SB;
    unsigned char *la = lds.a[wave], *lx = lds.x[wave];
    const u32x4 zero = {0u, 0u, 0u, 0u};
    const int n_tiles = g.n_tiles;
    // the sums of tile t, lane (rank column l16, quarter lq) with tile rows 4*lq + e
    auto store_tile = [&](int t, const f32x4 &v) {
        const int first = g.first[t], rows_here = (int)g.first[t + 1] - first;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 4 * lq + e;
            if (i < rows_here) {
                const int m = m_base + g.perm[first + i];
                store_shared(P.t_part + ((size_t)kc * a.M + m) * P.r16 + jb * 16 + l16, v[e]);
            }
        }
    };

    for (int t0 = share; t0 < n_tiles; t0 += 4 * shares) {
        const int n_here = min(4, (n_tiles - t0 + shares - 1) / shares);
        // what is requested next: tile and first k-step.  Instruction i covers staged rows RPI*i + lane/LPR
        // (rows of x; rank rows of A), 16 bytes per lane (lane%LPR of LPR).
        int rq_tile = my_slot, rq_s0 = 0;
        const uint16_t *xsrc[SB], *asrc[SB];
        bool x_ok[SB], a_ok[SB];
        u32x4 xv[DEPTH][SB], av[DEPTH][SB];
        auto request = [&](int set) {
            if (rq_tile >= n_here) return;
            if (rq_s0 == 0) {
                const int t = t0 + rq_tile * shares;
                const int first = g.first[t], rows_here = (int)g.first[t + 1] - first, adapter = g.adapter[t];
#pragma unroll
                for (int i = 0; i < SB; ++i) {
                    const int rr = RPI * i + st_row;
                    x_ok[i] = rr < rows_here;
                    const int row = m_base + (x_ok[i] ? (int)g.perm[first + rr] : 0);
                    // (int8 rows: the same element offsets, one byte each; kept as a uint16 pointer and
                    // turned into a byte address where it is used)
                    const size_t at = (size_t)row * P.K + (size_t)my_beg * KSTEP + st_piece * 8;
                    xsrc[i] = A8 ? reinterpret_cast<const uint16_t *>(reinterpret_cast<const unsigned char *>(P.x) + at) : P.x + at;
                    const int j = jb * 16 + rr;
                    a_ok[i] = j < P.rank;
                    asrc[i] = P.lora_a + ((size_t)adapter * P.rank + (a_ok[i] ? j : 0)) * P.K + (size_t)my_beg * KSTEP + st_piece * 8;
                }
            }
            const bool k_ok = (st_piece >> 2) < my_cnt - rq_s0;    // this lane's 8 inputs lie in k-step rq_s0 + st_piece/4
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                if constexpr (A8) {
                    uint2 v = make_uint2(0u, 0u);
                    if (x_ok[i] && k_ok) v = *reinterpret_cast<const uint2 *>(reinterpret_cast<const unsigned char *>(xsrc[i]) + (size_t)rq_s0 * KSTEP);
                    xv[set][i] = u32x4{v.x, v.y, 0u, 0u};   // (widened where it is used: here it would be waited for)
                } else {
                    xv[set][i] = (x_ok[i] && k_ok) ? *reinterpret_cast<const u32x4 *>(xsrc[i] + (size_t)rq_s0 * KSTEP) : zero;
                }
                av[set][i] = (a_ok[i] && k_ok) ? *reinterpret_cast<const u32x4 *>(asrc[i] + (size_t)rq_s0 * KSTEP) : zero;
            }
            rq_s0 += SB;
            if (rq_s0 >= my_cnt) {
                rq_s0 = 0;
                rq_tile += STEP;
            }
        };
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        int tile = my_slot, batch = 0;
        auto consume = [&](int set) {
            // (wave-private buffers: the wave's own LDS accesses are ordered, no barrier)
#pragma unroll
            for (int i = 0; i < SB; ++i) {
                *reinterpret_cast<u32x4 *>(lx + (RPI * i + st_row) * L::ROW + st_piece * 16) = A8 ? widen_int8(xv[set][i][0], xv[set][i][1]) : xv[set][i];
                *reinterpret_cast<u32x4 *>(la + (RPI * i + st_row) * L::ROW + st_piece * 16) = av[set][i];
            }
#pragma unroll
            for (int s = 0; s < SB; ++s) {
                const uint4 xa = *reinterpret_cast<const uint4 *>(lx + l16 * L::ROW + s * 64 + 16 * lq);
                const uint4 ab = *reinterpret_cast<const uint4 *>(la + l16 * L::ROW + s * 64 + 16 * lq);
                acc = mfma16(xa, ab, acc);
            }
            if (++batch == batches) {
                if constexpr (PARTS == 1) store_tile(t0 + tile * shares, acc);
                else                      lds.red[part][tile][lane] = acc;
                acc = f32x4{0.f, 0.f, 0.f, 0.f};
                batch = 0;
                tile += STEP;
            }
        };
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) request(d);
        const int items = (n_here - my_slot + STEP - 1) / STEP * batches;
        for (int i = 0; i < items; i += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                if (i + d < items) {
                    consume(d);
                    request(d);
                }
            }
        }
        if constexpr (PARTS == 1) continue;
        __syncthreads();
        if (wave < n_here) {
            f32x4 v = lds.red[0][wave][lane];
#pragma unroll
            for (int w = 1; w < PARTS; ++w) v += lds.red[w][wave][lane];
            store_tile(t0 + wave * shares, v);
        }
        if (t0 + 4 * shares < n_tiles) __syncthreads();     // (the next tiles' sums go to the same place)
    }
}

template <bool A8, int DEPTH, int WAVES>
__device__ __forceinline__ void shrink_block(const LaunchArgs &a, const ProjArgs &P, int pi, int local, ShrinkLds<WAVES> &lds)
{
    constexpr int SB = ShrinkLds<WAVES>::SB;
    RowTiles &g = lds.g;
    const int jblocks = P.r16 / 16;
    const int shares = shrink_tile_shares(a.M_plan, P.n_adapters, a.shrink_tiles);
    const int kc = local % P.kch;
    const int jb = (local / P.kch) % jblocks;
    const int share = (local / (P.kch * jblocks)) % shares;
    const int chunk = local / (P.kch * jblocks * shares);
    const int m_base = chunk * SHRINK_CHUNK_ROWS;

    if (threadIdx.x < 64) cut_row_tiles(a.row_adapter + m_base, min(SHRINK_CHUNK_ROWS, a.M - m_base), P.n_adapters, g);
    __syncthreads();

    // k-steps of this block's K chunk (balanced split; a K chunk has at least four)
    const int nks = P.K / KSTEP;
    const int q = nks / P.kch, r = nks % P.kch;
    const int blk_beg = kc * q + min(kc, r), blk_cnt = q + (kc < r ? 1 : 0);
    // (The long form first, without a jump to it: its code is not in the cache yet, and every wave that finishes outputs
    // waits for it.  14336 x 4096 at 64 rows, 32 adapters of rank 64, 52.5 -> 50.1 us, 4096 x 14336 53.0 -> 50.0, with one form
    // alone 50.2 and 49.6; 3072 x 8192 at 128 rows 18.5 either way, alone 18.3.  One copy of the code with the split known at
    // run time: 52.3, 48.7 and 18.2, but 256 x 9000 at 300 rows 15.3 -> 17.7 and 128 x 4991 at 276 32.1 -> 35.7.)
    if (DEPTH != 2 || __builtin_expect(blk_cnt > WAVES / 2 * SB, 1))
        shrink_tiles<A8, DEPTH, WAVES>(a, P, lds, m_base, share, shares, jb, kc, blk_beg, blk_cnt);
    else if (blk_cnt > WAVES / 4 * SB) shrink_tiles<A8, DEPTH, WAVES / 2>(a, P, lds, m_base, share, shares, jb, kc, blk_beg, blk_cnt);
    else                               shrink_tiles<A8, DEPTH, WAVES / 4>(a, P, lds, m_base, share, shares, jb, kc, blk_beg, blk_cnt);
    signal_done(a.ctrl + shrink_ctr(pi, 0), P.ctr_copies);
}


// Decode shapes (at most 16 rows): one block per (row, block of 16 ranks, K chunk) and no
// grouping.  The row's adapter index is one scalar load away, so the block's requests go out
// before the base blocks have filled the memory queues; rows that share an adapter read its A
// once each, from the cache.  Row 0 of the MFMA's A operand carries x[m]; the other rows are 0.
//
// A[adapter] is read in runs of 512 contiguous bytes per rank row and turned into MFMA fragments
// through a wave-private LDS buffer.  Reading the fragments directly (16 bytes from each of 16
// rows per lane group) would address rows a power of two apart, which all lie in the same
// memory channel: measured, those requests held up every other wave of their compute unit for
// about 5 us.
struct ShrinkRowLds {
    static constexpr int SB = 8;                            // k-steps per batch
    static constexpr int AROW = SB * 64 + 16;               // bytes of a rank row in a batch; +16: rows 4 banks apart
    unsigned char a[4][16 * AROW];
    unsigned char x[4][SB * 64];
    float red[4][16];
};

__device__ __forceinline__ void shrink_row_block(const LaunchArgs &a, const ProjArgs &P, int pi, int local,
                                                 ShrinkRowLds &lds)
{
    using L = ShrinkRowLds;
    constexpr int SB = L::SB;
    const int jblocks = P.r16 / 16;
    const int kc = local % P.kch;
    const int jb = (local / P.kch) % jblocks;
    const int m = local / (P.kch * jblocks);               // < M: the grid has M such rows of blocks
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l16 = lane & 15, lq = lane >> 4;
    const int half = lane >> 5, l32 = lane & 31;            // loads: two rank rows per instruction

    // k-steps of this block, then of this wave (balanced splits)
    const int nks = P.K / KSTEP;
    const int q = nks / P.kch, r = nks % P.kch;
    const int blk_beg = kc * q + min(kc, r), blk_cnt = q + (kc < r ? 1 : 0);
    const int wq_ = blk_cnt / 4, wr = blk_cnt % 4;
    const int my_beg = blk_beg + wave * wq_ + min(wave, wr);
    const int my_cnt = wq_ + (wave < wr ? 1 : 0);

    const u32x4 zero = {0u, 0u, 0u, 0u};
    const int adapter = a.row_adapter[m];
    const bool valid = adapter >= 0 && adapter < P.n_adapters;      // uniform
    const uint16_t *xrow = P.x + (size_t)m * P.K + (size_t)my_beg * KSTEP + l32 * 8;
    const uint16_t *arow = P.lora_a + (size_t)(valid ? adapter : 0) * P.rank * P.K + (size_t)my_beg * KSTEP + l32 * 8;
    unsigned char *la = lds.a[wave], *lx = lds.x[wave];

    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < my_cnt && valid; s0 += SB) {
        const int cnt = min(SB, my_cnt - s0);               // k-steps of this batch
        const bool k_ok = (l32 >> 2) < cnt;                 // this lane's 8 inputs lie in k-step l32/4
        const u32x4 xv = (half == 0 && k_ok) ? *reinterpret_cast<const u32x4 *>(xrow + (size_t)s0 * KSTEP) : zero;
        u32x4 av[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = jb * 16 + 2 * i + half;
            av[i] = (k_ok && j < P.rank) ? *reinterpret_cast<const u32x4 *>(arow + (size_t)j * P.K + (size_t)s0 * KSTEP)
                                         : zero;
        }
        if (half == 0) *reinterpret_cast<u32x4 *>(lx + l32 * 16) = xv;
#pragma unroll
        for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4 *>(la + (2 * i + half) * L::AROW + l32 * 16) = av[i];
        // (wave-private buffer: the wave's own LDS accesses are ordered, no barrier)
#pragma unroll
        for (int s = 0; s < SB; ++s) {
            const uint4 ab = *reinterpret_cast<const uint4 *>(la + l16 * L::AROW + s * 64 + 16 * lq);
            uint4 xa = *reinterpret_cast<const uint4 *>(lx + s * 64 + 16 * lq);
            if (l16 != 0) xa = make_uint4(0, 0, 0, 0);
            acc = mfma16(xa, ab, acc);
        }
    }
    if (valid) {
        // row 0 of the result: element 0 of lanes 0..15
        if (lq == 0) lds.red[wave][l16] = acc[0];
        __syncthreads();
        if (tid < 16) {
            const float v = ((lds.red[0][tid] + lds.red[1][tid]) + lds.red[2][tid]) + lds.red[3][tid];
            store_shared(P.t_part + ((size_t)kc * a.M + m) * P.r16 + jb * 16 + tid, v);
        }
    }
    // (a base-only row has nothing to write, but the finishing blocks count its blocks all the same)
    signal_done(a.ctrl + shrink_ctr(pi, 0), P.ctr_copies);
}

// ------------------------------------------------------------------------------------------
// kernels
// ------------------------------------------------------------------------------------------
// MB blocks of 16 rows per chunk, XR rows staged in LDS (the smallest multiple of 8 that holds
// the rows of a chunk decides which instance runs): 4 waves per block, rounds of R k-steps
// (two rounds = 2*R KiB of codes in flight per wave).
template <int MB> struct Shape;
template <> struct Shape<1> { static constexpr int WAVES = 4, R = 8; };
template <> struct Shape<2> { static constexpr int WAVES = 4, R = 4; };

template <int MB, int XR>
using BaseLdsOf = BaseLds<MB, XR, Shape<MB>::WAVES, Shape<MB>::R>;
template <int MB, int XR>
constexpr int pre_lds_bytes()
{
    constexpr int shrink = MB == 1 ? (int)sizeof(ShrinkRowLds) : (int)sizeof(ShrinkLds<4>);   // (MB == 1: M <= 16)
    return BaseLdsOf<MB, XR>::BYTES > shrink ? BaseLdsOf<MB, XR>::BYTES : shrink;
}

// Fetch every field of a projection's argument block at once.  Kernel arguments sit behind a
// scalar cache that is cold at every launch (about 0.4 us per dependent access); left alone,
// the compiler loads each field where it is first used, one round trip after another.  Pinning
// all fields to registers at one point makes it issue the loads together.
template <int G>
__device__ __forceinline__ ProjArgs fetch_proj(const GroupArgs<G> &a, int pi)
{
    ProjArgs P = a.p[pi];
    asm volatile("" :: "s"(P.codes), "s"(P.scales), "s"(P.flag), "s"(P.x), "s"(P.y), "s"(P.lora_a), "s"(P.lora_b),
                 "s"(P.t_part), "s"(P.partial));
    asm volatile("" :: "s"(P.K), "s"(P.N), "s"(P.spg), "s"(P.n_adapters), "s"(P.rank), "s"(P.r16),
                 "s"(P.kch), "s"(P.alpha), "s"(P.ksplit));
    asm volatile("" :: "s"(P.unit_q), "s"(P.unit_r), "s"(P.spg_shift), "s"(P.ctr_copies), "s"(P.lora_units), "s"(P.tiles_inv));
    return P;
}

// The three block-table rows of the block's group and the scalar fields at the end of the launch
// arguments, all requested together at the kernel's start: one scalar round trip (the cache
// behind the kernel arguments is cold at every launch) instead of one for the scalars, a
// dependent one for the table of the block's kind and then the projection's record.  Left alone,
// the compiler loads each value where it is first used; and a pointer to the table of the
// block's kind would turn the search below into 16 dependent loads.
typedef int i32x16 __attribute__((ext_vector_type(16)));
static_assert(GROUP_PROJ == 16, "the block tables of a group are read as vectors of 16");
struct LaunchTables {
    i32x16 shrink, pre, main;
    int shrink_blocks, pre_base_blocks, group_blocks;
};
template <int G>
__device__ __forceinline__ LaunchTables pin_launch_args(const GroupArgs<G> &a, int z)
{
    LaunchTables t;
    t.shrink = *reinterpret_cast<const i32x16 *>(a.shrink_begin[z]);
    t.pre = *reinterpret_cast<const i32x16 *>(a.pre_begin[z]);
    t.main = *reinterpret_cast<const i32x16 *>(a.main_begin[z]);
    t.shrink_blocks = a.shrink_blocks[z];
    t.pre_base_blocks = a.pre_base_blocks[z];
    t.group_blocks = a.group_blocks[z];
    asm volatile("" :: "s"(t.shrink), "s"(t.pre), "s"(t.main), "s"(a.row_adapter), "s"(a.M), "s"(a.y_fp32),
                       "s"(a.m_pad), "s"(a.row_blocks), "s"(a.half_shift), "s"(t.shrink_blocks), "s"(t.pre_base_blocks), "s"(t.group_blocks),
                       "s"(a.ctrl), "s"(a.status), "s"(a.spin_limit));
    return t;
}

// Entries past the last projection hold INT_MAX, so all 16 comparisons can be made without a
// loop.  first = begin[pi], picked from the same registers (begins are non-decreasing).
__device__ __forceinline__ int find_proj(const i32x16 &begin, int b, int &first)
{
    int pi = 0;
    first = begin[0];
#pragma unroll
    for (int i = 1; i < GROUP_PROJ; ++i) {
        pi += (b >= begin[i]) ? 1 : 0;
        first = (b >= begin[i]) ? begin[i] : first;
    }
    return pi;
}

// Block index -> (block of the group, row chunk).  The row chunks of one block of columns stream
// the same weights.  Workgroups go to the chip's 8 XCDs in turn (index mod 8), and every XCD has
// an L2 of its own, so behind the shrink blocks (filled up to a multiple of 8; they exist once, for all
// chunks: a grid of shrink blocks x chunks started 15232 blocks that had nothing to do among the 32256 of
// 16 layers at 512 rows) the grid is laid out in runs of 8 blocks x all chunks with the chunk
// varying in steps of 8: index = (b / 8) * 8 * chunks + chunk * 8 + b % 8.  All chunks of a block
// then run on one XCD at about the same time, and its weights come from HBM once and from that
// L2 for the other chunks.  (Chunk-major order, a whole pass over the weights between two chunks,
// read 5.9 x the algorithmic bytes from HBM at 512 rows.)  A producer still has a smaller index
// than its consumer: a split-K block and the block that finishes its tile have the same chunk.
// b past the group's last block: nothing to do.
__device__ __forceinline__ void split_block_index(const LaunchArgs &a, const LaunchTables &t, int &b, int &chunk)
{
    const unsigned id = blockIdx.x, chunks = (unsigned)a.row_blocks, shrink = (unsigned)t.shrink_blocks;
    const unsigned first = filled_up(shrink);
    chunk = 0;
    if (chunks == 1 || id < shrink) {
        b = (int)id;
    } else if (id < first) {
        b = 0x7FFFFFFF;
    } else {
        const unsigned run = (id - first) / (8u * chunks), r = (id - first) - run * 8u * chunks;
        chunk = (int)(r >> 3);
        b = (int)(shrink + run * 8u + (r & 7u));
    }
}

// blocks per compute unit the registers are budgeted for (LDS allows as many for these shapes)
template <int MB, int XR> constexpr int occupancy_of() { return MB == 1 && XR == 8 ? 3 : 2; }

// ------------------------------------------------------------------------------------------
// Wide shapes: the product is a dense contraction.  A block covers 32 or 64 rows x 256 columns: its
// four waves share the rows of x (staged in LDS, double-buffered) and each wave owns one
// 64-column tile, whose packed codes it streams into registers eight k-steps ahead and unpacks
// once for all its rows.  No K split inside the block; long K is cut into units as for the decode
// shapes, and a launch with few blocks is cut further by the host.
// ------------------------------------------------------------------------------------------
constexpr int WIDE_TILES = 4;

// MB blocks of 16 rows per base block: 4 (64 rows) in long launches, else 2 (32 rows).  A stage of
// x holds XSTEPS k-steps of every row: 16 KiB.
template <int MB>
struct WideLds {
    static constexpr int ROWS = 16 * MB;
    static constexpr int XSTEPS = MB == 2 ? 8 : 4;
    static constexpr int XROW = XSTEPS * 64 + 16;          // bytes of a row of x per stage; +16: rows 4 banks apart
    static constexpr int X_STAGE = ROWS * XROW;
    // t as two bf16 halves, with one row more than the block has: zeros.  It has a place of its own
    // beside the stages of x, so that a block that starts after its shrink blocks have finished
    // can fetch it ahead of the K loop.
    static constexpr int T_ROW = MLORA_MAX_RANK * 2 + 16;  // bytes; +16: rows 4 banks apart
    static constexpr int T_HALF = (ROWS + 1) * T_ROW;
    // after the K loop, over the stages, per wave: 16 rows of outputs on their way out
    template <int CB>
    struct Out {
        static constexpr int ROW = 32 * CB + 8;            // floats; rows 4 apart lie 32 banks apart
        static constexpr int BYTES = 16 * ROW * 4;
        static_assert(2 / CB * WIDE_TILES * BYTES <= 2 * X_STAGE, "the outputs fit the stages");
    };
    // the same of a fused call where two waves share a tile: the rows of the block, a tile after the other
    static constexpr int TILE_ROW = TILE_N + 2;
    static_assert(MB != 2 || WIDE_TILES * 32 * TILE_ROW * 4 <= 2 * X_STAGE, "the tiles fit the stages");
    alignas(16) unsigned char buf[2 * X_STAGE];
    alignas(16) unsigned char t[2 * T_HALF];
    int waited_out;                                        // a wave gave up waiting for t: the block's share of it is not known
    template <int CB>
    __device__ float *out(int wave) { return reinterpret_cast<float *>(buf + wave * Out<CB>::BYTES); }
};

// ------------------------------------------------------------------------------------------
// The K loop of the wide blocks.  Per wave: the packed codes of the next 8 k-steps and their
// scales are in registers (8 KiB in flight), each register set requested again as soon as its
// k-step is consumed; the rows of x come through LDS in stages of 16 KiB, double-buffered, one
// barrier per stage, shared by the block's four waves.  Codes, scales and x come with buffer loads:
// the lane's place in a vector register, the k-step in a scalar one, no vector arithmetic for
// addresses.  The codes enter the matrix units exactly; the scale multiplies the fp32 sum of a
// group with fp32 FMAs.
//
// 32 rows: products of 32 x 32 x 16 (a permlane swap of two code words turns the blob's order, made for
// 16 columns, into theirs).  Per k-step of a group of 32 inputs 70 vector instructions (28 to unpack, 32
// FMAs) and 4 products of 32 cycles, which run beside them: what bounds a compute unit's work is
// then the vector instructions, and what bounds a launch is how many blocks wait at once for memory.
// The loop and all that follows it fit 168 registers without spills for every group size, so that three
// blocks share a compute unit: 16 layers of a 1B-like model at 32 rows 191 -> 170 us (products of 16 x 16
// x 32, two blocks).  A group of 128 inputs is two runs of two k-steps: in one run its fragments of x do
// not fit (10 registers spilled inside the loop, the same launch in groups of 128 163 us against 146).
// 64 rows: products of 16 x 16 x 32, whose 64 sums per lane leave the registers for it; with products of 32 x 32
// x 16, whatever their order, 4 to 6 % fewer cycles of a clock that is 3 to 4 % slower (16 layers at 512 rows
// 1391 us against 1394 and 1395).  No spills in the loop; the sum of partial tiles keeps 9 registers (int8
// rows: 16) in scratch memory.
// Codes that one block of rows reads (AGAIN false) are marked as used once; where several blocks of rows
// read them, they stay in the cache for the next one (14336 x 4096 in groups of 128 at 64 rows, 32
// adapters of rank 64: 46.1 -> 43.7 us; unmarked where one block reads them, 16 layers at 32 rows: 159 -> 168).
// int8 rows are widened to bf16 (exact: seven bits and a sign) on their way into LDS: sums of a group
// stay integers below 2^24, exact in fp32, and the loop has fewer vector instructions than one
// over int8 products, whose int32 sums need a conversion each (16 layers at 32 rows 188 -> 171 us).
// ------------------------------------------------------------------------------------------
// A wave looks after 32 * CB columns, from column 32 * half of its tile on: a lane's code words of a k-step, and its
// scales of a group.
template <int CB> struct WaveWords;
template <> struct WaveWords<2> { typedef u32x4 codes; typedef uint2 scales; };
template <> struct WaveWords<1> { typedef unsigned int codes __attribute__((ext_vector_type(2))); typedef uint32_t scales; };
__device__ __forceinline__ uint32_t scale_pair(uint2 sc, int cb) { return cb == 0 ? sc.x : sc.y; }
__device__ __forceinline__ uint32_t scale_pair(uint32_t sc, int) { return sc; }

template <int SPG, int MB, bool A8, bool AGAIN, int CB, int XP, class Acc, class Early>
__device__ __forceinline__ void stream_loop(Acc &acc, __amdgpu_buffer_rsrc_t codes, __amdgpu_buffer_rsrc_t scales,
                                            __amdgpu_buffer_rsrc_t xsrc, const int (&xoff)[XP], int piece16, int xdst0,
                                            unsigned char *lds_x, const unsigned char *xfrag, int n_ksteps,
                                            int lane, int half, const ProjArgs &P, const Early &early)
{
    using L = WideLds<MB>;
    constexpr int S = L::XSTEPS;                           // k-steps per stage of x
    constexpr int W = 8;                                   // k-steps of codes in registers
    constexpr int HALVES = W / S;                          // stages per pass over the register sets
    static_assert(S % SPG == 0 && W % S == 0, "a stage holds whole scale groups; the sets hold whole stages");
    const int last = n_ksteps - 1;
    const int lane16 = lane * 16 + half * 8, col8 = (lane & 15) * 8 + half * 4, half16 = lane & 16;
    typename WaveWords<CB>::codes w[W];
    typename WaveWords<CB>::scales sc[W / SPG];
    constexpr int RPI = 16 * MB / XP;                      // rows a block moves per instruction (XP pieces of 16 bytes per thread and stage)
    u32x4 xr[XP];
    // (requests past the unit's end re-read its last k-step: all loads stay unconditional)
    auto load_codes = [&](int k) {
        const int at = min(k, last) * 1024;
        if constexpr (CB == 2) return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(codes, lane16, at, AGAIN ? 0 : 2));
        else                   return __builtin_bit_cast(WaveWords<1>::codes, __builtin_amdgcn_raw_buffer_load_b64(codes, lane16, at, AGAIN ? 0 : 2));
    };
    auto load_scales = [&](int k) {
        const int at = min(k, last) / SPG * 128;
        if constexpr (CB == 2) return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(scales, col8, at, 0));
        else                   return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(scales, col8, at, 0);
    };
    // (a last stage of half its length re-reads the unit's last inputs in place of those past it)
    constexpr int XB = A8 ? 32 : 64;                       // bytes of a row of x per k-step
    const int x_last = n_ksteps * XB - 16;
    auto load_x = [&](int st) {
        const int at = min(st * S * XB + piece16, x_last);
#pragma unroll
        for (int i = 0; i < XP; ++i) xr[i] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xsrc, xoff[i] + at, 0, 0));
    };
    auto store_x = [&](int buf) {
#pragma unroll
        for (int i = 0; i < XP; ++i) {
            unsigned char *dst = lds_x + buf + xdst0 + i * RPI * L::XROW;
            if constexpr (A8) {
                *reinterpret_cast<u32x4 *>(dst) = widen_int8(xr[i][0], xr[i][1]);
                *reinterpret_cast<u32x4 *>(dst + 16) = widen_int8(xr[i][2], xr[i][3]);
            } else {
                *reinterpret_cast<u32x4 *>(dst) = xr[i];
            }
        }
    };
    const int n_stages = (n_ksteps + S - 1) / S;
    load_x(0);
    const uint32_t flag = request_flag(P);
#pragma unroll
    for (int k = 0; k < W; ++k) {
        w[k] = load_codes(k);
        if (k % SPG == 0) sc[k / SPG] = load_scales(k);
    }
    __builtin_amdgcn_sched_barrier(0);                     // (all of these ahead of the first wait)
    early();
    store_x(0);
    const bool full_blob = flag_set(flag);

    // one stage: register sets [h * S, h * S + S), x buffer st & 1
    auto stage = [&](auto half, int st, auto full) {
        constexpr int H = decltype(half)::value;
        __syncthreads();                                   // this stage's rows of x are in place; the other buffer is free
        const int buf = (st & 1) * L::X_STAGE;
        load_x(min(st + 1, n_stages - 1));
        // the math of NK k-steps of this stage (NK = S, or 4 in the last stage of a unit that ends
        // on an odd super-step): straight code but for split_codes' branch per run
        auto stage_math = [&](auto nk) {
            constexpr int NK = decltype(nk)::value;
            // A scale group is worked through in runs of SG k-steps (at most 2, whose fragments of x
            // fit the registers): products, FMAs with the scale.
            constexpr int SG = SPG < 2 ? SPG : 2;
            constexpr int G0 = (H * S) / SPG;              // first scale group of this stage's register sets
#pragma unroll
            for (int r = 0; r < NK / SG; ++r) {
                const int g = r * SG / SPG;                // scale group of the run within the stage
                const unsigned char *xs = xfrag + buf + r * SG * 64;
                const auto sv = sc[G0 + g];
                if constexpr (MB == 2) {
                    uint4 xk[SG][2];
#pragma unroll
                    for (int t = 0; t < SG; ++t)
#pragma unroll
                        for (int o = 0; o < 2; ++o) xk[t][o] = *reinterpret_cast<const uint4 *>(xs + t * 64 + o * 16);
                    if ((r + 1) * SG % SPG == 0) sc[G0 + g] = load_scales(st * S + g * SPG + W);   // (last run of its group)
                    CodeBytes<2 * CB> cw[SG];
#pragma unroll
                    for (int t = 0; t < SG; ++t) cw[t] = split_codes<false>(w[H * S + r * SG + t], full_blob);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        f32x16 d = f32x16{0.f};
#pragma unroll
                        for (int t = 0; t < SG; ++t) {
                            const auto lo = __builtin_amdgcn_permlane16_swap(cw[t].lo[2 * cb], cw[t].lo[2 * cb + 1], false, false);
                            const auto hi = __builtin_amdgcn_permlane16_swap(cw[t].hi[2 * cb], cw[t].hi[2 * cb + 1], false, false);
#pragma unroll
                            for (int o = 0; o < 2; ++o) d = mfma32(xk[t][o], codes_to_bf16(lo[o], hi[o]), d);
                        }
                        float sj = half_bits_to_float((uint16_t)(scale_pair(sv, cb) >> half16));
                        asm volatile("" : "+v"(sj));       // a float in a register: plain fp32 FMAs below
#pragma unroll
                        for (int e = 0; e < 16; ++e) acc[cb][e] = fmaf(d[e], sj, acc[cb][e]);
                    }
                } else {
                    uint4 xk[SG][MB];
#pragma unroll
                    for (int t = 0; t < SG; ++t)
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
                            xk[t][mb] = *reinterpret_cast<const uint4 *>(xs + mb * 16 * L::XROW + t * 64);
                    if ((r + 1) * SG % SPG == 0) sc[G0 + g] = load_scales(st * S + g * SPG + W);   // (last run of its group)
                    CodeBytes<4> cw[SG];
#pragma unroll
                    for (int t = 0; t < SG; ++t) cw[t] = split_codes<false>(w[H * S + r * SG + t], full_blob);
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        f32x4 d[MB];
#pragma unroll
                        for (int t = 0; t < SG; ++t) {
                            const uint4 wb = codes_to_bf16(cw[t].lo[j], cw[t].hi[j]);
#pragma unroll
                            for (int mb = 0; mb < MB; ++mb) d[mb] = mfma16(xk[t][mb], wb, t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : d[mb]);
                        }
                        float sj = j == 0 ? half_bits_lo(sv.x) : j == 1 ? half_bits_hi(sv.x)
                                 : j == 2 ? half_bits_lo(sv.y) : half_bits_hi(sv.y);
                        asm volatile("" : "+v"(sj));
#pragma unroll
                        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                            for (int e = 0; e < 4; ++e) acc[mb][j][e] = fmaf(d[mb][e], sj, acc[mb][j][e]);
                    }
                }
                // the run's register sets are used up: request their next k-steps (after the last
                // use, so that no copy of the old contents has to be kept)
#pragma unroll
                for (int t = 0; t < SG; ++t) w[H * S + r * SG + t] = load_codes(st * S + r * SG + t + W);
                pin(acc);
            }
        };
        // (a unit is a whole number of 4-k-step super-steps: a stage of 8 k-steps is full, or the
        // unit's last one with 4)
        if constexpr (decltype(full)::value) stage_math(std::integral_constant<int, S>{});
        else                                 stage_math(std::integral_constant<int, 4>{});
        store_x(L::X_STAGE - buf);
    };
    // The loop holds full stages only; a last stage of 4 k-steps (S = 8) follows it.  One variant of
    // the stage inside the loop: the two would meet at the loop's end with their values in
    // different registers, and the moves that reconcile them were 5 % of the loop's instructions.
    constexpr std::true_type full_stage{};
    if constexpr (HALVES == 2) {
#pragma nounroll
        for (int st = 0; st < n_stages; st += 2) {
            stage(std::integral_constant<int, 0>{}, st, full_stage);
            if (st + 1 < n_stages) stage(std::integral_constant<int, 1>{}, st + 1, full_stage);
        }
    } else {
        const int n_full = n_ksteps / S;
#pragma nounroll
        for (int st = 0; st < n_full; ++st) stage(std::integral_constant<int, 0>{}, st, full_stage);
        if constexpr (S > 4) {
            if (n_full < n_stages) stage(std::integral_constant<int, 0>{}, n_full, std::false_type{});
        }
    }
}

// group = index of the block's four tiles among the projection's; ku as in base_unit.  SPG =
// k-steps per scale group, the same for every projection of the launch; MB = blocks of 16 rows
// per base block (4 where wide64_pays, else 2); AGAIN = other blocks of rows read the same codes.
// CB = blocks of 32 columns per wave: 2, a wave per tile, or 1, two waves per tile (see wide_short_kernel).
template <int SPG, int MB, bool A8, bool AGAIN, int CB>
__device__ __forceinline__ void wide_unit(const LaunchArgs &a, const ProjArgs &P, int pi, int group, int ku,
                                          int m0, WideLds<MB> &lds)
{
    using L = WideLds<MB>;
    constexpr int ROWS = L::ROWS;
    constexpr int RB = MB / 2;                             // blocks of 32 rows
    constexpr int WPT = 2 / CB, THREADS = 64 * WIDE_TILES * WPT;   // waves per tile; threads of the block
    static_assert(CB == 2 || MB == 2, "two waves per tile: blocks of 32 rows");
    const int K = P.K, N = P.N, M = a.M;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int tiles = tiles_n(N);
    const int half = CB == 2 ? 0 : wave & 1, col0 = 32 * half;     // first column of the tile that this wave looks after
    const int tile_raw = group * WIDE_TILES + wave / WPT;
    // (uniform per wave.  A spare wave computes and drops the block's first tile, whose counter it may
    // wait on: that tile's own wave puts it back to zero only after the barrier both pass.)
    const bool tile_ok = tile_raw < tiles;
    const int tile = tile_ok ? tile_raw : group * WIDE_TILES;

    const int uq = P.unit_q, ur = P.unit_r;
    const int unit_beg = ku * uq + min(ku, ur), unit_cnt = uq + (ku < ur ? 1 : 0);
    const int ksteps = K / KSTEP;
    constexpr int gs = 4 / SPG;
    const u32x4 *wp = reinterpret_cast<const u32x4 *>(P.codes + (size_t)tile * ksteps * 64) + (size_t)unit_beg * 256;
    const uint2 *sp = P.scales + ((size_t)tile * (ksteps / SPG) + (size_t)unit_beg * gs) * 16;

    // The first P.lora_units K units of a tile take a share of the LoRA term each (the adapters of the chunk are dealt
    // out to them in turn): all of them where the rows of B of many adapters are more than the finishing
    // blocks alone can fetch in good time.  Such a unit waits for the shrink blocks, and
    // P.n_finish_blocks counts (tile, chunk, such a unit, wave of the tile) here.
    const bool lora = a.row_adapter != nullptr && P.n_adapters > 0 && ku < P.lora_units;
    const int rows_here = min(ROWS, M - m0);
    const int chunk = m0 / ROWS, chunks = a.row_blocks;
    const int fin = tile * chunks + chunk;
    const int user = (fin * P.lora_units + ku) * WPT + half;
    const int copies = P.ctr_copies;
    unsigned *const sctr = a.ctrl + shrink_ctr(pi, user & (copies - 1));
    const int lines = (chunks + a.half_shift) >> a.half_shift;     // counter lines per tile
    unsigned *const pctr = a.ctrl + P.part_ctr + (tile * lines + (chunk >> a.half_shift)) * CTR_STRIDE +
                           (chunk & a.half_shift) * (CTR_STRIDE / 2) + half * (CTR_STRIDE / 4);
    const bool need_s = lora, need_p = ku == 0 && P.ksplit > 1;

    if (tid == 0) lds.waited_out = 0;                      // (ahead of the K loop's barriers)

    // t = alpha * sum over the K chunks of the shrink partials, in fixed order, as two bf16 halves
    // that make up its first 17 bits.  A thread takes four neighbouring ranks of one row (16
    // bytes of a partial sum); the requests of several quads and K chunks overlap.  A wave's share:
    // ROWS / 4 rows.
    auto gather_t = [&]() {
        constexpr int TPR = THREADS / ROWS;                // threads per row
        const int ml = tid / TPR, q0 = tid % TPR;
        const int quads = P.r16 / 4;
        const float t_factor = A8 ? P.alpha * P.x_scale : P.alpha;   // (the shrink blocks saw x as integers)
        const int t_chunk = M * P.r16 * 4;                 // bytes of a K chunk's partial sums
        const __amdgpu_buffer_rsrc_t rt = wave_buffer(P.t_part, (unsigned)P.kch * (unsigned)t_chunk);
        const int at = (m0 + min(ml, rows_here - 1)) * P.r16 * 4;
        unsigned char *const dst = lds.t + ml * L::T_ROW;
        auto quads_of = [&](auto nq, auto nc, int qb) {        // nq quads of ranks, nc K chunks at a time
            constexpr int Q = decltype(nq)::value, C = decltype(nc)::value;
            f32x4_t v[Q];
#pragma unroll
            for (int u = 0; u < Q; ++u) v[u] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            for (int kc0 = 0; kc0 < P.kch; kc0 += C) {
                f32x4_t pv[Q][C];
#pragma unroll
                for (int u = 0; u < Q; ++u)
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        pv[u][c] = load_shared16(rt, at + min(qb + u * TPR, quads - 1) * 16 + min(kc0 + c, P.kch - 1) * t_chunk);
#pragma unroll
                for (int u = 0; u < Q; ++u)
#pragma unroll
                    for (int c = 0; c < C; ++c)
                        if (kc0 + c < P.kch) v[u] += pv[u][c];
            }
#pragma unroll
            for (int u = 0; u < Q; ++u) {
                const int quad = qb + u * TPR;
                if (quad >= quads) continue;
                v[u] *= t_factor;
                // (a t above the largest bf16 must not round to infinity: the rest stays in the low half)
                constexpr float top = 0x1.FEp127f;
                f32x4_t w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = __builtin_amdgcn_fmed3f(v[u][e], -top, top);
                const uint2 h = make_uint2(pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3]));
                const f32x4_t l = {v[u][0] - bf16_bits_to_float(h.x & 0xFFFFu), v[u][1] - __uint_as_float(h.x & 0xFFFF0000u),
                                   v[u][2] - bf16_bits_to_float(h.y & 0xFFFFu), v[u][3] - __uint_as_float(h.y & 0xFFFF0000u)};
                *reinterpret_cast<uint2 *>(dst + quad * 8) = h;
                *reinterpret_cast<uint2 *>(dst + L::T_HALF + quad * 8) = make_uint2(pack_bf16(l[0], l[1]), pack_bf16(l[2], l[3]));
            }
        };
        if (quads <= TPR) {
            if (q0 < quads) quads_of(std::integral_constant<int, 1>{}, std::integral_constant<int, 4>{}, q0);
        } else {
            for (int qb = q0; qb < quads; qb += 2 * TPR) quads_of(std::integral_constant<int, 2>{}, std::integral_constant<int, 4>{}, qb);
        }
        // the row of zeros that stands for rows of other adapters
        if (tid < L::T_ROW / 16) {
            *reinterpret_cast<u32x4 *>(lds.t + ROWS * L::T_ROW + tid * 16) = u32x4{0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4 *>(lds.t + L::T_HALF + ROWS * L::T_ROW + tid * 16) = u32x4{0u, 0u, 0u, 0u};
        }
    };
    // A wave that finds its shrink blocks done when it starts (all but the first blocks of a long
    // launch) fetches its share of t ahead of the K loop, behind the requests for x and codes.
    const bool try_early = lora && a.spin_limit > 0;
    unsigned seen = 0;
    if (try_early) seen = __hip_atomic_load(sctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool have_t = false;
    auto early = [&]() {
        if (try_early && seen >= (unsigned)P.n_shrink_blocks) {
            compiler_fence();
            gather_t();
            have_t = true;
        }
    };

    // element i of acc[rb][cb]: row 32*rb + 8*(i/4) + 4*hi + i%4 of the chunk, column col0 + 32*cb + l32 of the tile
    f32x16 acc[RB][CB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x16{0.f};
    {
        constexpr int EB = A8 ? 1 : 2;                     // bytes per input
        // Descriptors of what the wave reads, so that a load needs no vector arithmetic for its
        // address: the lane's place in a vector register, the k-step in a scalar one.  Rows of x: the
        // chunk's, from the unit's first input to the end of the chunk's last row.
        const unsigned char *x0 = reinterpret_cast<const unsigned char *>(P.x) + ((size_t)m0 * K + (size_t)unit_beg * SUPER_K) * EB;
        const __amdgpu_buffer_rsrc_t rx = wave_buffer(x0, ((unsigned)rows_here * (unsigned)K - (unsigned)unit_beg * SUPER_K) * EB);
        const __amdgpu_buffer_rsrc_t rw = wave_buffer(wp, (unsigned)unit_cnt * 4096u);
        const __amdgpu_buffer_rsrc_t rs = wave_buffer(sp, (unsigned)unit_cnt * (unsigned)(gs * 128));
        // rows of x: thread t moves, per stage, 16-byte piece t % PPR of rows t / PPR + RPI * i (PPR
        // pieces per row and stage, RPI rows per instruction of the block); int8 rows are half as long
        constexpr int PPR = L::XSTEPS * 2 * EB, RPI = THREADS / PPR, XP = ROWS / RPI;
        static_assert(XP >= 1 && XP * RPI == ROWS, "every row of a stage is moved once");
        int xoff[XP];
        const int piece16 = (tid % PPR) * 16;
#pragma unroll
        for (int i = 0; i < XP; ++i) xoff[i] = min(tid / PPR + RPI * i, rows_here - 1) * K * EB;
        const int xdst0 = (tid / PPR) * L::XROW + piece16 * (2 / EB);
        if constexpr (MB == 2) {
            stream_loop<SPG, MB, A8, AGAIN, CB, XP>(acc[0], rw, rs, rx, xoff, piece16, xdst0, lds.buf, lds.buf + l32 * L::XROW + hi * 32,
                                     unit_cnt * 4, lane, half, P, early);
        } else {
            // Products of 16 x 16: lane (l16, lq) gets rows 4 * lq + e of a block of 16 and columns 16 * j +
            // l16.  With the rows of their A operand in the order that trades the two bits of row / 4,
            // one swap of lanes 16 apart per register turns them into the order of acc.
            const int l16 = lane & 15, arow = (l16 & 3) | ((l16 & 4) << 1) | ((l16 & 8) >> 1);
            f32x4 acc16[MB][4];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc16[mb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            stream_loop<SPG, MB, A8, AGAIN, CB, XP>(acc16, rw, rs, rx, xoff, piece16, xdst0, lds.buf, lds.buf + arow * L::XROW + (lane >> 4) * 16,
                                     unit_cnt * 4, lane, half, P, early);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc16[mb][2 * cb][e]),
                                                                         __float_as_uint(acc16[mb][2 * cb + 1][e]), false, false);
                        acc[mb >> 1][cb][8 * (mb & 1) + e] = __uint_as_float(sw[0]);
                        acc[mb >> 1][cb][8 * (mb & 1) + 4 + e] = __uint_as_float(sw[1]);
                    }
        }
        if constexpr (A8) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[rb][cb] *= P.x_scale;
        }
    }

    // LoRA term: one pass per adapter that occurs in the chunk and run of 16 ranks (one 32x32x16
    // product per block of 32 rows, 32 columns and half of t).  A pass needs the run's part of B for
    // the tile's 64 columns: 16 bytes per lane and 32 columns.  Passes go in the order adapter,
    // run (a row of B is fetched in one piece), in rounds of NB that form a two-deep pipeline: the
    // rows of B of the next round are on their way while the current round is computed.
    constexpr int NB = MB == 2 ? 4 : 8;
    const int runs = P.r16 / 16;
    const int n_lane = tile * TILE_N + col0 + l32;
    // lane l looks after row l of the chunk (a spare wave and a call without LoRA: no row)
    int ad_row = -1;
    if (lora && tile_ok && lane < rows_here) {
        const int v = a.row_adapter[m0 + lane];
        ad_row = (v >= 0 && v < P.n_adapters) ? v : -1;
    }
    struct Round {
        int cur[NB], run[NB];                          // adapter (-1: no more passes) and run of ranks of each pass
    };
    // where the enumeration stands: adapter, its next run, rows not yet looked at, adapters seen
    int st_cur = -1, st_run = 0, st_ordinal = 0;
    unsigned long long st_remaining = __ballot(ad_row >= 0);
    auto next_round = [&](Round &r) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (st_cur >= 0 && ++st_run == runs) st_cur = -1;
            while (st_cur < 0 && st_remaining) {       // next adapter that this K unit looks after
                const int next = __builtin_amdgcn_readlane(ad_row, (int)__builtin_ctzll(st_remaining));
                st_remaining &= ~__ballot(ad_row == next);
                if (st_ordinal++ % P.lora_units == ku) {
                    st_cur = next;
                    st_run = 0;
                }
            }
            r.cur[b] = st_cur;
            r.run[b] = st_run;
        }
    };
    auto request = [&](u32x4 (&bf)[NB][CB], const Round &r) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (r.cur[b] < 0) break;
            // (ranks past the adapter's meet zeros of t: their part of B is a re-read of the first ranks)
            const int k = 16 * r.run[b] + 8 * hi;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const int n = min(n_lane + 32 * cb, N - 1);
                bf[b][cb] = *reinterpret_cast<const u32x4 *>(P.lora_b + ((size_t)r.cur[b] * N + n) * P.rank + (k < P.rank ? k : 0));
            }
        }
    };
    // The first round's rows of B do not depend on t: they are requested before the wait for
    // the shrink blocks and arrive while t is gathered.
    Round ra_, rb_;
    u32x4 bfa[NB][CB], bfb[NB][CB];
    ra_.cur[0] = -1;
    if (lora && tile_ok) {
        next_round(ra_);
        request(bfa, ra_);
    }

    // (a wave whose wait runs out sets the status word, and the whole block, all of whose waves use the
    // rows of t it gathers, stores NaN in place of its outputs or partial tiles; a spare wave waits
    // too: it gathers its share of t)
    if (need_s && !have_t) {
        if (!wait_count(sctr, (unsigned)P.n_shrink_blocks, a.spin_limit) && lane == 0) {
            lds.waited_out = 1;
            atomicOr(a.status, 1u);
        }
        gather_t();
    }
    __syncthreads();                                       // t is in place; every wave is done with the x buffers
    bool poisoned = lds.waited_out != 0;
    auto poison = [&]() {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[rb][cb] = f32x16{0.f} + __uint_as_float(0x7FC00000u);
    };
    if (lora) {                                            // (uniform over the block)
        if (tile_ok) {
            auto compute = [&](const u32x4 (&bf)[NB][CB], const Round &r) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (r.cur[b] < 0) break;
                    const unsigned long long same = __ballot(ad_row == r.cur[b]);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        const unsigned rows = (unsigned)(same >> (32 * rb));
                        if (!rows) continue;
                        const int row = (rows >> l32) & 1u ? 32 * rb + l32 : ROWS;
                        const int k = r.run[b] * 32 + hi * 16;
                        const uint4 th = *reinterpret_cast<const uint4 *>(lds.t + row * L::T_ROW + k);
                        const uint4 tl = *reinterpret_cast<const uint4 *>(lds.t + L::T_HALF + row * L::T_ROW + k);
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            const uint4 b4 = __builtin_bit_cast(uint4, bf[b][cb]);
                            acc[rb][cb] = mfma32(th, b4, acc[rb][cb]);
                            acc[rb][cb] = mfma32(tl, b4, acc[rb][cb]);
                        }
                    }
                }
            };
            while (ra_.cur[0] >= 0) {
                next_round(rb_);
                request(bfb, rb_);
                compute(bfa, ra_);
                if (rb_.cur[0] < 0) break;
                next_round(ra_);
                request(bfa, ra_);
                compute(bfb, rb_);
            }
        }
    }
    if (ku > 0) {
        if (poisoned) poison();
        // A partial tile (the chunk's rows x 64 columns) lies in the workspace in the order of the
        // MFMA results, quarter q of block (rb, cb) of lane l at (((rb * 2 + cb) * 4 + q) * 64 + l) * 4:
        // producer and consumer use the same mapping, and a lane moves 16 bytes per instruction.
        if (tile_ok) {
            float *dst = P.partial + (((size_t)(ku - 1) * tiles + tile) * a.m_pad + m0) * TILE_N + half * 1024 + lane * 4;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        store_shared16(dst + ((rb * 2 + cb) * 4 + q) * 256, f32x4_t{acc[rb][cb][4 * q], acc[rb][cb][4 * q + 1],
                                                                                    acc[rb][cb][4 * q + 2], acc[rb][cb][4 * q + 3]});
            compiler_fence();
            __builtin_amdgcn_s_waitcnt(0x0F70);            // vmcnt(0): this wave's stores have completed
            if (lane == 0) atomicAdd(pctr, 1u);
        }
    } else if (tile_ok && need_p) {
        if (!wait_count(pctr, (unsigned)(P.ksplit - 1), a.spin_limit)) {
            poisoned = true;
            if (lane == 0) atomicOr(a.status, 1u);
        }
        // The other units' partial tiles, added in the order of the units.  Two sets of registers:
        // a unit's tile is added while the next one is on its way (a projection with a long K has
        // a dozen of them, and one round trip after another was most of its finishing block's time).
        // These are loads the compiler sees (it places the waits): values it does not know to be
        // in flight must not stay in registers across other code, which it may spill or reuse.
        constexpr int NP = 2 * MB * CB;
        const int np = P.ksplit - 1;
        auto request = [&](f32x4_t (&pv)[NP], int u) {
            // (the tile of unit u for this wave's chunk and columns: NP KiB, the same place for all lanes)
            const float *base = P.partial + (((size_t)u * tiles + tile) * a.m_pad + m0) * TILE_N + half * 1024;
            const __amdgpu_buffer_rsrc_t rsrc = shared_buffer(base, NP * 1024);
#pragma unroll
            for (int i = 0; i < NP; ++i) pv[i] = load_shared16(rsrc, lane * 16, i * 1024);
        };
        auto fold = [&](const f32x4_t (&pv)[NP]) {
#pragma unroll
            for (int i = 0; i < NP; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i / (4 * CB)][(i / 4) % CB][(i % 4) * 4 + e] += pv[i][e];
        };
        // (inside the loop every request is unconditional: the waits can then count the requests behind
        // the data they need, where a branch would make them wait for everything in flight)
        f32x4_t pa[NP], pb[NP];
        request(pa, 0);
        int u = 0;
        for (; u + 2 < np; u += 2) {
            request(pb, u + 1);
            fold(pa);
            request(pa, u + 2);
            fold(pb);
        }
        if (u + 1 < np) {
            request(pb, u + 1);
            fold(pa);
            fold(pb);
        } else {
            fold(pa);
        }
    }
    if (poisoned && ku == 0) poison();
    if (CB == 1 && ku == 0 && a.fused) {
        // the fused output stage takes four columns 16 apart of one row from a lane: the two waves of a tile put
        // their halves together in LDS and take 16 rows each
        float *const whole = reinterpret_cast<float *>(lds.buf) + wave / WPT * 32 * L::TILE_ROW;
#pragma unroll
        for (int i = 0; i < 16; ++i) whole[(8 * (i >> 2) + 4 * hi + (i & 3)) * L::TILE_ROW + col0 + l32] = acc[0][0][i];
        __syncthreads();
        if (tile_ok) {
            const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = 16 * half + 4 * lq + e;
                float vv[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) vv[j] = whole[row * L::TILE_ROW + 16 * j + l16];
                store_fused(a, P, pi, m0 + row, tile, l16, vv);
            }
        }
    } else if (CB == 2 && tile_ok && ku == 0 && a.fused) {
        // the fused output stage takes four columns 16 apart of one row from a lane: rows (i, i + 4)
        // of the two halves of 32 columns trade places, after which lane (l16, lq) holds columns
        // 16 * j + l16 of row 8 * (lq % 2) + 4 * (lq / 2) + e of every 16
        const int l16 = lane & 15, lq = lane >> 4;
#pragma unroll
        for (int h = 0; h < MB; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float vv[4];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[h >> 1][cb][8 * (h & 1) + e]),
                                                                     __float_as_uint(acc[h >> 1][cb][8 * (h & 1) + 4 + e]), false, false);
                    vv[2 * cb] = __uint_as_float(sw[0]);
                    vv[2 * cb + 1] = __uint_as_float(sw[1]);
                }
                store_fused(a, P, pi, m0 + 16 * h + 8 * (lq & 1) + 4 * (lq >> 1) + e, tile, l16, vv);
            }
    } else if (tile_ok && ku == 0) {
        const bool full = tile * TILE_N + TILE_N <= N;
        if (full) {
            // rows of outputs through a wave-private LDS buffer, so that a lane stores 8 * CB neighbouring columns
            // at once instead of single values
            using Out = typename L::template Out<CB>;
            float *st = lds.template out<CB>(wave);
            const int row = lane >> 2, c0 = (lane & 3) * 8 * CB;
            const f32x4 *src = reinterpret_cast<const f32x4 *>(st + row * Out::ROW + c0);
#pragma unroll
            for (int h = 0; h < MB; ++h) {                 // 16 rows at a time
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
                        st[(8 * (e >> 2) + 4 * hi + (e & 3)) * Out::ROW + 32 * cb + l32] = acc[h >> 1][cb][8 * (h & 1) + e];
                const int m = m0 + 16 * h + row;
                f32x4 o[2 * CB];
#pragma unroll
                for (int q = 0; q < 2 * CB; ++q) o[q] = src[q];
                if (m < M) {
                    const size_t at = (size_t)m * N + tile * TILE_N + col0 + c0;
                    if (a.y_fp32) {
                        f32x4 *dst = reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(P.y) + at);
#pragma unroll
                        for (int q = 0; q < 2 * CB; ++q) dst[q] = o[q];
                    } else {
                        u32x4 *dst = reinterpret_cast<u32x4 *>(reinterpret_cast<uint16_t *>(P.y) + at);
#pragma unroll
                        for (int q = 0; q < CB; ++q)
                            dst[q] = u32x4{pack_bf16(o[2 * q][0], o[2 * q][1]), pack_bf16(o[2 * q][2], o[2 * q][3]),
                                           pack_bf16(o[2 * q + 1][0], o[2 * q + 1][1]), pack_bf16(o[2 * q + 1][2], o[2 * q + 1][3])};
                    }
                }
            }
        } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int m = m0 + 32 * rb + 8 * (i >> 2) + 4 * hi + (i & 3);
                    if (m >= M) continue;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        const int n = tile * TILE_N + col0 + 32 * cb + l32;
                        if (n >= N) continue;
                        if (a.y_fp32) reinterpret_cast<float *>(P.y)[(size_t)m * N + n] = acc[rb][cb][i];
                        else reinterpret_cast<uint16_t *>(P.y)[(size_t)m * N + n] = float_to_bf16_bits(acc[rb][cb][i]);
                    }
                }
        }
    }

    // counters back to zero for the next call (every wave owns its counters of its tile)
    if (tile_ok && lane == 0) {
        if (need_p) __hip_atomic_store(pctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (need_s) {
            const int users = (P.n_finish_blocks >> (31 - __clz(copies))) + ((user & (copies - 1)) < (P.n_finish_blocks & (copies - 1)) ? 1 : 0);
            if (atomicAdd(sctr + 1, 1u) + 1u == (unsigned)users) {
                __hip_atomic_store(sctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(sctr + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <int MB, int CB>
constexpr int wide_lds_bytes()
{
    constexpr int wide = (int)sizeof(WideLds<MB>), shrink = (int)sizeof(ShrinkLds<8 / CB>);
    return wide > shrink ? wide : shrink;
}

// What a block of a launch of wide blocks does.
template <int SPG, int MB, bool A8, bool AGAIN, int CB, int G>
__device__ __forceinline__ void wide_block(const GroupArgs<G> &a, unsigned char *smem)
{
    const int z = (int)blockIdx.z;
    const LaunchTables tables = pin_launch_args(a, z);
    int b, chunk;
    split_block_index(a, tables, b, chunk);
    if (b >= tables.group_blocks) return;
    int first;
    if (b < tables.shrink_blocks) {
        const int pi = z * GROUP_PROJ + find_proj(tables.shrink, b, first);
        shrink_block<A8, MB == 2 ? 2 : 4>(a, fetch_proj(a, pi), pi, b - first, *reinterpret_cast<ShrinkLds<8 / CB> *>(smem));
        return;
    }
    WideLds<MB> &lds = *reinterpret_cast<WideLds<MB> *>(smem);
    // (one call site for both kinds of base block: the code is large, and a second copy is fetched cold)
    const bool pre = b < tables.shrink_blocks + tables.pre_base_blocks;
    const int bb = b - tables.shrink_blocks - (pre ? 0 : tables.pre_base_blocks);
    const int pi = z * GROUP_PROJ + find_proj(pre ? tables.pre : tables.main, bb, first);
    const ProjArgs P = fetch_proj(a, pi);
    const int local = bb - first;
    const int groups = (tiles_n(P.N) + WIDE_TILES - 1) / WIDE_TILES;
    const int unit = pre ? local / groups : 0;
    wide_unit<SPG, MB, A8, AGAIN, CB>(a, P, pi, local - unit * groups, pre ? 1 + unit : 0, chunk * 16 * MB, lds);
}

}  // namespace mlora
