// Wide blocks for launches with few of them.
#include "layer_blocks.hpp"

namespace mlora {

// The block of wide_kernel for 32 rows with eight waves instead of four: two waves share a tile, 32 columns each.  A
// launch of at most about a block per compute unit is a chain: K loop, t, LoRA term, partial tiles, outputs.  The loop
// takes as long as with four waves (440 cycles per k-step either way, more than its vector and matrix instructions would
// take one after the other: 48 of them 21 k cycles, the instructions of the whole launch 19 k); what follows it has half as
// much to do per wave, a shrink block's K chunk is cut over eight waves, and two blocks find room on a compute unit (128
// registers, 70 KB of LDS).
// us in a graph, four waves against eight: 4096 x 14336 at 64 rows, 32 adapters of rank 64 34.5 -> 31.3; 1664 x 977 at 85
// rows, 8 adapters of rank 128 23.5 -> 19.9; 1280 x 6631 at 44 rows 15.6 -> 12.7; a decoder layer of 78 rows (1024
// wide, outputs of gate and up through the fused stage) 92 -> 74.  64 calls of up to 230 blocks: 0.90 of the time; of 231 to
// 256: 3072 x 8192 at 128 rows 19.0 -> 18.9, 8192 x 808 at 231 19.0 -> 21.3.  Requests three or four stages of four
// k-steps ahead instead of one of eight, with a barrier per stage: 19.2 -> 20.2 and 19.9 (3072 x 8192 at 128 rows).
// Codes are never marked as used once here: the two waves of a tile read the same lines.  Marked where one block of rows reads
// them (int8 calls of up to 32 rows; 16 layers one after the other, 1 to 32 rows): 2048 wide 0.99 to 1.01 of the time, 1024
// wide 1.03 to 1.05, 2560 wide 0.99 to 1.01, 1536 wide 0.91 to 1.02.
template <int SPG, bool A8>
__global__ __launch_bounds__(512, 4) void wide_short_kernel(const GroupArgs<1> a)
{
    __shared__ __align__(16) unsigned char smem[wide_lds_bytes<2, 1>()];
    wide_block<SPG, 2, A8, true, 1>(a, smem);
}

hipError_t launch_wide_short(const LayerArgs &a, const dim3 &grid, hipStream_t s)
{
    if (grid.z != 1) return hipErrorInvalidValue;
    const int spg = a.p[0].spg;
    auto go = [&](auto kernel) { kernel<<<grid, dim3(512), 0, s>>>(first_group(a)); };
    auto by_group = [&](auto a8_c) {
        constexpr bool A8 = decltype(a8_c)::value;
        if (spg == 1)      go(wide_short_kernel<1, A8>);
        else if (spg == 2) go(wide_short_kernel<2, A8>);
        else               go(wide_short_kernel<4, A8>);
    };
    if (a.a8) by_group(std::true_type{});
    else      by_group(std::false_type{});
    return hipGetLastError();
}

}  // namespace mlora
