// The kernels of the layer step (see layer_blocks.hpp for what their blocks do) and their launch.
#include "layer_blocks.hpp"

namespace mlora {

template <int MB, int XR, int G>
__global__ __launch_bounds__(64 * Shape<MB>::WAVES, (occupancy_of<MB, XR>())) void layer_kernel(const GroupArgs<G> a)
{
    __shared__ __align__(16) unsigned char smem[pre_lds_bytes<MB, XR>()];
    const int z = (int)blockIdx.z;
    const LaunchTables tables = pin_launch_args(a, z);
    int b, chunk;
    split_block_index(a, tables, b, chunk);
    if (b >= tables.group_blocks) return;                  // (the slices are as long as the longest group)
    int first;
    if (b < tables.shrink_blocks) {
        const int pi = z * GROUP_PROJ + find_proj(tables.shrink, b, first);
        // (the instances with one block of 16 rows are the ones launched for M <= 16)
        if constexpr (MB == 1) shrink_row_block(a, fetch_proj(a, pi), pi, b - first, *reinterpret_cast<ShrinkRowLds *>(smem));
        else                   shrink_block<false, 4>(a, fetch_proj(a, pi), pi, b - first, *reinterpret_cast<ShrinkLds<4> *>(smem));
        return;
    }
    const BaseLdsOf<MB, XR> lds{smem};
    const int m0 = chunk * 16 * MB;
    // (one call site for both kinds of base block: the kernel's code is large, and what runs
    // once per launch is paid for by instruction fetch)
    const bool pre = b < tables.shrink_blocks + tables.pre_base_blocks;
    const int bb = b - tables.shrink_blocks - (pre ? 0 : tables.pre_base_blocks);
    const int pi = z * GROUP_PROJ + find_proj(pre ? tables.pre : tables.main, bb, first);
    const ProjArgs P = fetch_proj(a, pi);
    const int local = bb - first;
    const int tiles = tiles_n(P.N);
    // local / tiles (tiles_inv = ceil(2^32 / tiles) does not fit 32 bits for a single tile)
    const int unit = !pre ? 0 : tiles == 1 ? local : (int)__umulhi((unsigned)local, P.tiles_inv);
    // (the kernel for 9 to 16 rows also runs the 16-row chunks of short launches of up to 32 rows,
    // among them a fused gate/up projection with its LoRA pair of twice the rank: a second copy of
    // the block with the prefetch for ranks up to 32; a call of rank 16 runs the code it always ran)
    if constexpr (MB == 1 && XR == 16) {
        if (P.rank > fast_rank<MB>()) {
            base_unit<MB, XR, Shape<MB>::WAVES, Shape<MB>::R, 32>(a, P, pi, local - unit * tiles, pre ? 1 + unit : 0, m0, lds);
            return;
        }
    }
    base_unit<MB, XR, Shape<MB>::WAVES, Shape<MB>::R, fast_rank<MB>()>(a, P, pi, local - unit * tiles, pre ? 1 + unit : 0, m0, lds);
}

template <int SPG, int MB, bool A8, bool AGAIN>
__global__ __launch_bounds__(256, (MB == 2 ? 3 : 2)) void wide_kernel(const LayerArgs a)
{
    __shared__ __align__(16) unsigned char smem[wide_lds_bytes<MB, 2>()];
    wide_block<SPG, MB, A8, AGAIN, 2>(a, smem);
}

// (blocks of 32 rows run in launches of at least CHUNK16_MAX_BLOCKS blocks only: no short form of theirs)
template <int MB, int XR>
static hipError_t launch_instance(const LayerArgs &a, const dim3 &grid, hipStream_t s)
{
    constexpr int THREADS = 64 * Shape<MB>::WAVES;
    if constexpr (MB == 1) {
        if (grid.z == 1) {
            layer_kernel<MB, XR, 1><<<grid, dim3(THREADS), 0, s>>>(first_group(a));
            return hipGetLastError();
        }
    }
    layer_kernel<MB, XR, MAX_GROUPS><<<grid, dim3(THREADS), 0, s>>>(a);
    return hipGetLastError();
}

// grid: x = the longest of the groups (see group_grid_x), z = groups of up
// to 16 projections; blocks past a group's last one exit at once
hipError_t launch_layer(const LayerArgs &a, long long grid_x, int groups, hipStream_t s)
{
    if (grid_x > 0x7FFFFFFFll) return hipErrorInvalidValue;
    const dim3 grid((unsigned)grid_x, 1u, (unsigned)groups);
    if (a.wide && a.waves_per_tile == 2) return launch_wide_short(a, grid, s);
    if (a.wide) {
        // (the host puts only projections with the same group size into one such launch)
        const int spg = a.p[0].spg;
        auto go = [&](auto kernel) { kernel<<<grid, dim3(256), 0, s>>>(a); };
        auto by_rows = [&](auto spg_c, auto a8_c) {
            constexpr int SPG = decltype(spg_c)::value;
            constexpr bool A8 = decltype(a8_c)::value;
            if (a.block_rows == 64)    go(wide_kernel<SPG, 4, A8, true>);
            else if (a.row_blocks > 1) go(wide_kernel<SPG, 2, A8, true>);
            else                       go(wide_kernel<SPG, 2, A8, false>);
        };
        auto by_group = [&](auto a8_c) {
            if (spg == 1)      by_rows(std::integral_constant<int, 1>{}, a8_c);
            else if (spg == 2) by_rows(std::integral_constant<int, 2>{}, a8_c);
            else               by_rows(std::integral_constant<int, 4>{}, a8_c);
        };
        if (a.a8) by_group(std::true_type{});
        else      by_group(std::false_type{});
        return hipGetLastError();
    }
    // (the rows per block the host laid the launch out for: a short launch of 17 to 32 rows has
    // blocks of 16 rows)
    if (a.row_blocks * a.block_rows < a.M) return hipErrorInvalidValue;
    if (a.block_rows == 16) return a.M <= 8 ? launch_instance<1, 8>(a, grid, s) : launch_instance<1, 16>(a, grid, s);
    if (a.M <= 24) return launch_instance<2, 24>(a, grid, s);
    return launch_instance<2, 32>(a, grid, s);
}

__global__ void zero_kernel(uint4 *p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

hipError_t launch_zero(void *p, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    if (n == 0) return hipSuccess;
    const unsigned blocks = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    zero_kernel<<<dim3(blocks), dim3(256), 0, s>>>(reinterpret_cast<uint4 *>(p), n);
    return hipGetLastError();
}

}  // namespace mlora
