// Shared device-side definitions of the mlora_w4 library: blob layout, kernel
// argument blocks, small bit helpers.  gfx950 only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include "../../include/mlora_w4.h"

namespace mlora {

// ---------------------------------------------------------------------------------------------
// Prepacked weight blob.
//
// The weight is cut into tiles of 64 output columns (4 blocks of 16) and k-steps of 32 inputs:
// one 16x16x32 bf16 MFMA consumes a block of 16 columns x 32 inputs as its B operand, lane l
// holding column l%16 and the 8 consecutive inputs 8*(l/16) .. +7.  The blob stores, for
// every (tile, k-step), one 1 KiB chunk laid out exactly as a wavefront reads it with one
// 128-bit load per lane: lane l's uint4 holds, in component j, the 8 codes of column
// 64*tile + 16*j + l%16 at inputs 32*step + 8*(l/16) + 0..7.
//
// Inside a dword the 8 codes are stored as sign and magnitude in fields placed so that each of
//   w & 0x87878787   and   (w rotr 4) & 0x87878787
// is four bytes s0000mmm, the codes of inputs 0..3 and 4..7.  Read as 8-bit floats (1-4-3) such bytes are
// the numbers +-m * 2^-9, exactly: one conversion instruction (v_cvt_scalef32_pk_bf16_fp8, as fast as a
// logical operation) turns two of them into a pair of bf16 codes.
// Four bits of sign and magnitude do not hold all of -8 .. 7.  A blob with a code -8 anywhere (a
// quantiser that scales by max / 7 makes none) has its flag set, the first word of the blob's last 16
// bytes, and stores m - 1 for its negative codes; the kernels' unpacking adds the 1 back, six operations per
// word (see split_codes for what that costs).
//
// Scales follow the codes: fp16, index ((tile * K/group + g) * 16 + c) * 4 + j for column
// 64*tile + 16*j + c, so the lane that holds column c of all four blocks reads its four
// scales of a group with one 64-bit load.  Columns beyond N are stored as code 0, scale 0.
// ---------------------------------------------------------------------------------------------
constexpr int TILE_N = 64;
constexpr int KSTEP = 32;
constexpr int SUPER_K = 128;       // k-steps are consumed four at a time

__host__ __device__ inline int tiles_n(int N) { return (N + TILE_N - 1) / TILE_N; }
__host__ __device__ inline size_t blob_code_bytes(int K, int N) {
    return (size_t)tiles_n(N) * (size_t)(K / KSTEP) * 1024u;
}
__host__ __device__ inline size_t blob_scale_bytes(int K, int N, int group) {
    return (size_t)tiles_n(N) * (size_t)(K / group) * 128u;
}
// The kernels request whole batches of super-steps without clamping the last ones, so a wave
// may read (and ignore) up to 3 super-steps of codes and as many groups of scales past the end
// of its tile: the blob ends with slack that keeps those reads inside the allocation.
constexpr size_t BLOB_SLACK_BYTES = 16384;
constexpr uint32_t FIELD_MASK = 0x87878787u;
__host__ __device__ inline size_t blob_flag_at(int K, int N, int group)
{
    return blob_code_bytes(K, N) + blob_scale_bytes(K, N, group) + BLOB_SLACK_BYTES - 16;
}
__host__ __device__ inline uint32_t rotl32(uint32_t v, int s) {
    s &= 31;
    return s ? (v << s) | (v >> (32 - s)) : v;
}
// code (-8 .. 7) of input i <-> its fields in the dword
__host__ __device__ inline uint32_t code_field(int code, int i, bool full)
{
    const uint32_t m = code < 0 ? (uint32_t)(-code) - (full ? 1u : 0u) : (uint32_t)code;
    return rotl32((code < 0 ? 0x80u : 0u) | m, 8 * (i & 3) + (i < 4 ? 0 : 4));
}
__host__ __device__ inline int field_code(uint32_t w, int i, bool full)
{
    const uint32_t b = rotl32(w, 32 - (8 * (i & 3) + (i < 4 ? 0 : 4)));
    const int m = (int)(b & 7u);
    return b & 0x80u ? -(m + (full ? 1 : 0)) : m;
}

// ---------------------------------------------------------------------------------------------
// Kernel argument block of one grouped call (passed by value; a block reads only
// the launch scalars, the three table rows of its group and the record of its projection).
// The projections of a launch are cut into groups of up to 16; group z owns slice z of the grid
// (blockIdx.z) and the block tables of a group are one vector of 16 each.
// ---------------------------------------------------------------------------------------------
constexpr int GROUP_PROJ = 16;
constexpr int MAX_GROUPS = 8;
constexpr int MAX_PROJ_PER_LAUNCH = GROUP_PROJ * MAX_GROUPS;
constexpr int ROWS_PER_BLOCK16 = 16;
constexpr int MAX_KCHUNKS = 16;    // partial sums of the shrink step the epilogue adds up

struct ProjArgs {
    const uint4 *codes;        // blob, code region
    const uint2 *scales;       // blob, scale region (4 fp16 per entry)
    const uint32_t *flag;      // blob: not zero if it holds a code -8 (see above)
    const uint16_t *x;         // bf16 [M][K]
    void *y;                   // [M][N]
    const uint16_t *lora_a;    // bf16 [n_adapters][rank][K]
    const uint16_t *lora_b;    // bf16 [n_adapters][N][rank]
    float *t_part;             // fp32 [kch][M][r16], written by the shrink blocks
    float *partial;            // fp32 [ksplit-1][tiles][m_pad][64], written by the split-K units
    int K, N;
    int spg;                   // k-steps per scale group (group / 32)
    int n_adapters, rank;
    int r16;                   // rank rounded up to a multiple of 16
    int kch;                   // number of K chunks of the shrink step
    float alpha;
    float x_scale;             // int8 activations: the per-tensor scale of x (1 otherwise)
    int ksplit;                // K units per tile; unit 0 finishes the tile, the others run ahead
    int n_shrink_blocks;       // shrink blocks of this projection (each bumps its counter once)
    int n_finish_blocks;       // who waits for this projection's shrink blocks: tile blocks, the finishing blocks (tiles x
                               // blocks of rows); wide blocks, the waves that make a LoRA term (tiles x blocks of rows x
                               // lora_units x waves per tile)
    int part_ctr;              // index of this projection's first split-K counter line in ctrl
    // Derived on the host so that no block starts with integer divisions (each one costs some 30
    // cold instructions, and they sat in front of the first memory request of every block):
    int unit_q, unit_r;        // (K / 128) / ksplit and (K / 128) % ksplit: super-steps per K unit
    int spg_shift;             // log2(spg)
    int ctr_copies;            // copies of the shrink counter in use: a power of two, at most
                               // min(CTR_REPL, n_finish_blocks)
    int lora_units;            // wide blocks: K units of a tile that share its LoRA term (the first ones; see LORA_FEW_PASSES)
    unsigned tiles_inv;        // ceil(2^32 / tiles) for tiles > 1: block index / tiles = umulhi(index,
                               // tiles_inv), exact while index * tiles < 2^32
};

// Counters in the workspace that order the blocks of one launch (all zero between calls).
// Every counter has a 128-byte line of its own, and what many blocks wait for exists in
// CTR_REPL copies, each polled by a share of the waiting blocks: hundreds of blocks polling one
// line queue up behind each other in one memory channel, and since a wave's loads return in
// order that stalls their weight streams too.
//   shrink_ctr(p, r)      + 0: shrink blocks of projection p that have finished (copy r)
//                         + 1: those of n_finish_blocks that have used copy r (the last one resets both)
//   part_ctr + (tile * chunks + chunk) * CTR_STRIDE: split-K units of that tile that have finished; two blocks of 32 rows in a
//                           chunk of 64 have a word each, CTR_STRIDE / 2 apart, two waves of a tile CTR_STRIDE / 4 apart
constexpr int CTR_REPL = 16;
constexpr int CTR_STRIDE = 32;                 // uint32 per counter line
__host__ __device__ inline int shrink_ctr(int p, int r) { return (p * CTR_REPL + r) * CTR_STRIDE; }
constexpr size_t WS_HEADER_BYTES = 256;        // status word at the front of every workspace
constexpr int SPIN_LIMIT_DEFAULT = 200000;     // x ~0.5 us: far beyond any launch, still finite

// What a fused call does to the outputs of a projection before they are stored (all optional):
//   v = row_scale[m] * (base + LoRA term); a pair operation on columns (c, c + 32) of every
//   64-column tile; + residual[m][n].  The row scale is either handed in or made from sq_in,
//   the per-tile sums of squares that the projection which produced x left in its sq_out: the
//   RMSNorm between two projections then needs no kernel of its own.
// Pair operations: PAIR_ROPE rotates (v[c], v[c+32]) by the angle whose cosine and sine are
// rope_cos/sin[m][c % 32] (heads of 64 features: a tile is a head); PAIR_SWIGLU stores
// silu(v[c]) * v[c+32] at column 32 * tile + c % 32 of an output of N / 2 columns (the weight
// holds 32 gate columns and the 32 up columns of the same features in every tile).
enum { PAIR_NONE = 0, PAIR_ROPE = 1, PAIR_SWIGLU = 2 };
struct EpiArgs {
    const float *row_scale;        // fp32 [M]
    const float *rope_cos;         // fp32 [M][32]
    const float *rope_sin;
    const uint16_t *residual;      // bf16 [M][N_out]
    const float *sq_in;            // fp32 [M][sq_parts]: partial sums of squares of the rows of x (another
                                   // projection's sq_out); row scale = 1 / sqrt(sum / K + sq_eps)
    float *sq_out;                 // fp32 [M][tiles]: sum of squares of the outputs a tile stores, as stored
    int pair_op;
    int sq_parts;
    float sq_eps;
    int pad_;
};

// What every block of a launch needs, whatever the number of its projections.
struct LaunchArgs {
    const int *row_adapter;    // may be null
    unsigned *ctrl;            // completion counters of this launch
    unsigned *status;          // workspace status word: set non-zero if a wait ran out
    int n_proj;
    int M;
    int M_plan;                // the row count the launch was laid out for (shrink blocks): M, except
                               // that calls with int8 activations always run wide blocks and are
                               // laid out as for at least 17 rows
    int y_fp32;
    int m_pad;                 // M rounded up to whole row chunks
    int block_rows;            // rows of a base block: 16, 32 or 64
    int row_blocks;            // base blocks along the rows
    int half_shift;            // 1: two blocks of 32 rows per row chunk of 64 (they share its counter lines)
    int shrink_tiles;          // grouped shrink blocks: most row tiles of a block (see shrink_tile_shares)
    int spin_limit;            // polls a block makes before it gives up waiting (0: gives up at once)
    int a8;                    // x is int8 with one scale per tensor (ProjArgs::x_scale)
    int wide;                  // the launch runs wide blocks (see below)
    int waves_per_tile;        // wide blocks: 1, or 2 in short launches (see wide_short_kernel)
    int fused;                 // outputs go through epi[] (one group of at most 16 projections)
    EpiArgs epi[GROUP_PROJ];
};

// The argument block of a kernel for up to G groups.  A launch copies all of it: of the 5.2 us that a call of one
// projection took, 1.7 went into the 20 KiB of records that it had no use for, so the kernels of short launches exist
// for one group as well (3.7 KiB).
template <int G>
struct GroupArgs : LaunchArgs {
    // Slice z of the grid holds, in this order, the shrink blocks, the split-K blocks (units 1..)
    // and the finishing blocks (unit 0) of the projections of group z; first block of each
    // projection within its kind (entries past the group's last projection: INT_MAX):
    alignas(64) int shrink_begin[G][GROUP_PROJ];           // (a block reads a row of each at once)
    int pre_begin[G][GROUP_PROJ];
    int main_begin[G][GROUP_PROJ];
    int shrink_blocks[G];      // shrink blocks of the group (first in its slice)
    int pre_base_blocks[G];    // split-K blocks of the group (after its shrink blocks)
    int group_blocks[G];       // all blocks of the group; the slice's other blocks exit at once
    ProjArgs p[G * GROUP_PROJ];
};
using LayerArgs = GroupArgs<MAX_GROUPS>;
inline GroupArgs<1> first_group(const LayerArgs &a)
{
    GroupArgs<1> one;
    static_cast<LaunchArgs &>(one) = a;
    memcpy(one.shrink_begin, a.shrink_begin, sizeof one.shrink_begin);
    memcpy(one.pre_begin, a.pre_begin, sizeof one.pre_begin);
    memcpy(one.main_begin, a.main_begin, sizeof one.main_begin);
    one.shrink_blocks[0] = a.shrink_blocks[0];
    one.pre_base_blocks[0] = a.pre_base_blocks[0];
    one.group_blocks[0] = a.group_blocks[0];
    memcpy(one.p, a.p, sizeof one.p);
    return one;
}

// ---------------------------------------------------------------------------------------------
// 16-bit float helpers (bit patterns)
// ---------------------------------------------------------------------------------------------
__device__ inline float bf16_bits_to_float(uint32_t b) { return __uint_as_float(b << 16); }
__device__ inline uint16_t float_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x0040u);  // quiet NaN
    u += 0x7FFFu + ((u >> 16) & 1u);                                              // nearest even
    return (uint16_t)(u >> 16);
}

// two floats -> a pair of bf16 bit patterns (a in the low half), round to nearest even: one instruction
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t pack_bf16(float a, float b) { return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b}); }

__device__ inline float half_bits_to_float(uint16_t b) { return (float)__builtin_bit_cast(_Float16, b); }

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// D[16 rows][16 cols] += A[16][32] * B[32][16]; lane l supplies row l%16 of A and column l%16
// of B at inputs 8*(l/16)..+7, and receives D[4*(l/16) + r][l%16] in element r.
__device__ inline f32x4 mfma16(uint4 a, uint4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

// D[32 rows][32 cols] += A[32][16] * B[16][32]; lane l supplies row l%32 of A and column l%32 of B
// at inputs 8*(l/32)..+7, and receives D[8*(i/4) + 4*(l/32) + i%4][l%32] in element i.
typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ inline f32x16 mfma32(uint4 a, uint4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}

// The grouped shrink step (more than 16 rows) works on chunks of 64 rows: the rows of a chunk are grouped by adapter
// (one wave, no sort) and every segment is cut into tiles of 16 rows.  Upper bound of the tiles of a chunk of `rows`
// rows (at most 64): a tile per 16 rows plus one per segment, at most a tile per row.  The chunk's tiles are shared
// out over blocks.  Fewer tiles per block are a shorter chain ahead of every block that finishes outputs; more are fewer
// blocks, idle ones included, whose signals queue up at the same counters.  The most tiles of a block, the first
// line that holds (S(t) = shrink blocks of the launch with t tiles each, B = its base blocks; us of calls both ways):
//
//   blocks of four waves
//    1  B + S(1) <= 500, all find a place at once, in wide blocks of 32 rows for inputs above 128 (with 128 a tile is one wave's:
//       100 drawn calls at 17 to 700 rows 0.98 of the time with 4): 8192 x 2048 at 64 rows, 8 adapters of rank 16, 16 tiles 40, 4 22.7, 1 19.4
//    2  wide blocks of 32 rows, inputs from 1024 (a tile is several trips to memory), S(2) <= 192, B + S(2) <= 640: 68 drawn
//       calls 0.987 of the time with 4, 5632 x 1700 at 466 rows, 11 adapters of rank 16, 33.3 -> 29.1, the worst 1.06.
//       S(2) above 192: 19 calls 1.04, 12928 x 4198 at 56 rows, 23 of rank 64, 27.6 -> 31.2; blocks of 64 rows: 22 calls 1.02,
//       4480 x 5658 at 302 rows, 19 of rank 24, 42.0 -> 46.4
//    4  B + S(4) <= 500: 4096 x 14336 at 64 rows, 32 adapters of rank 64, 16 tiles 41.5, 4 35.4; 14336 x 4096 49.5 and 32.5
//    4  wide blocks, S(4) <= 300: 4352 x 5466 at 441 rows, 10 adapters of rank 32, 8 tiles 80, 4 49; 280 drawn calls of 3000
//       to 14336 outputs at 150 to 1024 rows 0.97 of the time, 8 of them more than 3 % longer, by 17 % at most; S(4) from 320
//       to 480: as many calls lose as gain, 3328 x 3563 at 593 rows 52 -> 61
//    8  wide blocks of 32 rows
//   16  the others, which have two places per compute unit (16 layers at 512 rows 1313, 1342 with 8; a layer at 32 rows
//       in tile blocks 25, 29 with 8)
//
//   blocks of eight waves (short launches: fewer of them share a compute unit's pipes, and they stand in each other's way sooner)
//    1  B + S(1) <= 300, S(1) <= 160, inputs above 128: at 24 to 150 shrink blocks 1.03 to 1.2 times as fast as 4, from
//       176 on 4 are 1.0 to 1.3 times as fast: 1152 x 4261 at 65 rows, 7 adapters of rank 128, 18.6 and 14.6
//    2  inputs from 2048, S(2) <= 260, B + S(2) <= 500: 2688 x 1103 at 251 rows, 4 of rank 128, 21.1, 4 tiles
//       28.1; shorter inputs, 1152 x 2453 at 450 rows 32.8, 4 tiles 23.2; lost: 10112 x 537 at 84 rows, all on one of 30
//       adapters of rank 24 (most blocks idle), 22.1, 4 tiles 17.5
//    2  the same in calls of several projections from 1024 inputs (their blocks signal to counters of their own): 12
//       drawn calls 0.95 of the time with 4, the worst 1.03, a layer of 512 wide at 177 rows, 11 of rank 16, 16.6 -> 14.5
//    4  128 inputs (a tile is two waves'), B + S(4) <= 280; above, 8: 6 calls 0.88 of the time with 4, 128 x 4442 at 341 rows, 2
//       of rank 128, 18.9 -> 16.6 (between 150 and 280 as many gain as lose, below 150 4 are 1.03 times as fast)
//    4  B + S(4) <= 500, or S(4) <= 300
//    8  the others
// Host (grid size) and device (block index -> chunk, share) use the same figures.
constexpr int SHRINK_CHUNK_ROWS = 64;
__host__ __device__ inline int max_row_tiles(int rows, int n_adapters)
{
    const int segs = n_adapters < rows ? n_adapters : rows;
    const int bound = rows / 16 + segs;
    return bound < rows ? bound : rows;
}
constexpr int SHRINK_ALL_LIVE_BLOCKS = 500, SHRINK_TWO_LIVE_BLOCKS = 640, SHRINK_TWO_BLOCKS = 192;
constexpr int SHRINK_ALL_SHORT_BLOCKS = 300, SHRINK_ONE_SHORT_BLOCKS = 160, SHRINK_TWO_SHORT_BLOCKS = 260;
constexpr int SHRINK_WHOLE_SHORT_BLOCKS = 280;
constexpr int SHRINK_FEW_BLOCKS = 300, SHRINK_LONG_INPUTS = 1024;
__host__ __device__ inline int shrink_tile_shares(int M, int n_adapters, int tiles_per_block)
{
    const int tiles = max_row_tiles(M < SHRINK_CHUNK_ROWS ? M : SHRINK_CHUNK_ROWS, n_adapters);
    return (tiles + tiles_per_block - 1) / tiles_per_block;
}

// Blocks along x of a group of projections in the grid (see split_block_index): shrink blocks once, base blocks for
// every block of rows.
__host__ __device__ inline unsigned filled_up(unsigned blocks) { return (blocks + 7u) & ~7u; }
inline long long group_grid_x(int shrink_blocks, int base_blocks, int row_blocks)
{
    return row_blocks == 1 ? (long long)shrink_blocks + base_blocks
                           : filled_up((unsigned)shrink_blocks) + (long long)filled_up((unsigned)base_blocks) * row_blocks;
}

// host launchers (each file defines its own)
hipError_t launch_prepack(int K, int N, int group, const uint8_t *wq, const uint16_t *scales,
                          void *blob, hipStream_t s);
hipError_t launch_unpack(int K, int N, int group, const void *blob, int8_t *codes, float *w_f32,
                         hipStream_t s);
hipError_t launch_group_rows(const int *row_adapter, int M, int n_adapters, int *perm,
                             int *seg_adapter, int *seg_start, int *n_seg, hipStream_t s);
hipError_t launch_layer(const LayerArgs &a, long long grid_x, int groups, hipStream_t s);
hipError_t launch_wide_short(const LayerArgs &a, const dim3 &grid, hipStream_t s);
hipError_t launch_zero(void *p, size_t bytes, hipStream_t s);
hipError_t launch_rms_scale(const uint16_t *x, int M, int K, float eps, float *scale, hipStream_t s);
hipError_t launch_lora_int16_expand(const int16_t *aq, const int16_t *bq, int n_adapters, int rank, int K, int N,
                                    uint16_t *a4, uint16_t *b4, hipStream_t s);

constexpr int UNIT_SUPER_STEPS = 16;   // a block streams at most 16 super-steps (2048 inputs)
// Two families of base blocks.  "Tile" blocks cover one column tile and their four waves split
// K (many short-lived blocks: what a small launch needs to fill the chip); "wide" blocks cover
// four column tiles, one per wave, and share the rows of x through LDS (a quarter of the x
// traffic and no reduction across waves: what a long weight stream needs).  Up to 16 rows: tile
// blocks.  33 rows and more: wide blocks.  17 to 32 rows (chunks of 32 rows): wide blocks if the
// launch has at least WIDE32_MIN_BLOCKS of them, else tile blocks.
constexpr int WIDE_ALWAYS_ROWS = 33;
constexpr int WIDE32_MIN_ROWS = 17;
constexpr int WIDE32_MIN_BLOCKS = 300;
// From 33 rows on a chunk of 64 rows is the unit of the workspace's layout.  Blocks of 64 rows unpack a
// weight once for twice the rows, but two of them fill a compute unit's registers where three of 32
// rows fit, and their latencies are longer; they pay where the launch has more than about one of them
// per compute unit, and where the rows fill them: with rows a little above a multiple of 64, blocks of 32
// rows waste half as many (lines drawn from 2592 calls of 33 to 1024 rows, ranks 8 to 128, 1 to 32 adapters).
// Measured in us, blocks of 64 rows against 32, groups of 32 / of 128 inputs: 16 layers of a 1B-like
// model at 512 rows (14848 blocks of 64 rows) 1335 against 1529 / 1179 against 1321; one such layer at 512
// rows (928) 98 against 110 / 85 against 94; with the lines drawn, at 128 rows (232) 41 against 38 / 34 against
// 33, 3072 x 9216 twice at 72 rows (288 of 64, 432 of 32) 36 against 25.
constexpr int WIDE64_MIN_BLOCKS = 320;
__host__ inline bool wide64_pays(int blocks64, int blocks32) { return blocks64 >= WIDE64_MIN_BLOCKS && 5ll * blocks32 >= 9ll * blocks64; }
constexpr int WIDE_TILES_PER_BLOCK = 4;
// Blocks of 32 rows have two waves per tile in launches of one group of projections with at most this many base blocks
// (see wide_short_kernel, which also says what both sides measured).
constexpr int WIDE_SHORT_MAX_BLOCKS = 230;
// Passes (adapters of a block's rows x runs of 16 ranks) up to which the finishing block of a tile makes the whole LoRA
// term in launches of at most LORA_FEW_BLOCKS base blocks, one per compute unit: the other K units then leave their partial
// tiles without waiting for t (with more blocks they wait beside others' work, and the share they take is worth more:
// two layers of 1536 with int8 rows at 56 rows, 280 blocks, 24.0 -> 24.3 us; 2432 x 382 at 396 rows, one adapter of rank
// 64 21.5 -> 15.7 us; 3072 x 8192 at 128 rows, 8 adapters of rank 16 19.0 -> 18.6; two layers of 2176 at 130 rows 82 -> 78;
// 85 calls 0.99 of the time, with two adapters of rank 64 as many gain as lose).
constexpr int LORA_FEW_PASSES = 8, LORA_FEW_BLOCKS = 256;
constexpr int CHUNK16_MAX_BLOCKS = 300;    // tile launches of 17 to 32 rows below this run chunks of 16 rows
__host__ inline int rows_per_chunk(int M) { return M <= 16 ? 16 : M <= 32 ? 32 : 64; }
// column tiles a base block covers
__host__ __device__ inline int tiles_per_block(bool wide) { return wide ? WIDE_TILES_PER_BLOCK : 1; }

}  // namespace mlora
