// Instantiates the group kernels of one mode for slice widths HB_PART_LO..HB_PART_HI and registers
// their launchers.  Compiled several times with different -D values so the parts build in parallel.
#include "hb_kernels.hpp"
#include "hb_launch.hpp"

#if !defined(HB_PART_MODE) || !defined(HB_PART_LO) || !defined(HB_PART_HI)
#error "compile with -DHB_PART_MODE=<0..4> -DHB_PART_LO=<w> -DHB_PART_HI=<w>"
#endif

namespace {

template <int W, int MODE>
hipError_t launch_group(const uint64_t *x0, const uint64_t *x1, uint64_t n, int k, uint64_t seedB, uint64_t seedA,
                        uint64_t *o0, uint64_t *o1, hipStream_t stream)
{
    constexpr uint64_t L = hb::Shape<W>::L;
    const uint64_t groups = (n + L - 1) / L;
    const uint64_t blocks = (groups + hb::kBlock - 1) / hb::kBlock;
    if (blocks == 0 || blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    if constexpr (hb::TileTraits<W>::kSupported) {
        if (!hb::force_group_kernel()) {
            const hb::TileGrid grid = hb::tile_grid((n + hb::TileTraits<W>::kTile - 1) / hb::TileTraits<W>::kTile, W, 2, hb::op_of(MODE));
            if (grid.blocks == 0) return hipErrorInvalidConfiguration;
            auto go = [&](auto form) {
                constexpr int kForm = decltype(form)::value;
                hipLaunchKernelGGL((hb::tile_kernel<W, MODE, kForm>), dim3(grid.blocks), dim3(hb::kBlock), (hb::tile_lds_bytes<W, MODE>(hb::has_quarters(kForm))),
                                   stream, x0, x1, n, k, seedB, seedA, o0, o1, grid.whole_blocks);
                return hipGetLastError();
            };
            return hb::with_form<W, hb::runs_supported(W, 2, hb::op_of(MODE))>(grid, go);
        }
    }
    auto go = [&](auto runs) {
        hipLaunchKernelGGL((hb::group_kernel<W, MODE, decltype(runs)::value>), dim3((unsigned)blocks), dim3(hb::kBlock), 0, stream, x0,
                           x1, n, groups, k, seedB, seedA, o0, o1);
        return hipGetLastError();
    };
    if constexpr (!hb::TileTraits<W>::kSupported) {
        if (hb::group_runs(blocks)) return go(std::true_type{});
    }
    return go(std::false_type{});
}

template <int W, int MODE>
hipError_t launch_batch(const hb::BatchArgs &args, hipStream_t stream)
{
    if constexpr (hb::TileTraits<W>::kSupported) {
        const hb::TileGrid grid = hb::tile_grid(args.tiles, W, 2, hb::op_of(MODE));
        if (grid.blocks == 0) return hipErrorInvalidConfiguration;
        auto go = [&](auto form) {
            constexpr int kForm = decltype(form)::value;
            hipLaunchKernelGGL((hb::tile_batch_kernel<W, MODE, kForm>), dim3(grid.blocks), dim3(hb::kBlock), (hb::tile_lds_bytes<W, MODE>(hb::has_quarters(kForm))),
                               stream, args);
            return hipGetLastError();
        };
        // (no entry point takes a set for its sign shares: that launcher is there for the table's sake, in the fewest forms)
        return hb::with_form<W, hb::op_of(MODE) != hb::kSign && hb::runs_supported(W, 2, hb::op_of(MODE))>(grid, go);
    } else {
        return hipErrorInvalidDeviceFunction;
    }
}

template <int W>
hipError_t launch_sim(const float *x, uint64_t n, int k, uint64_t seedB, uint64_t seedA, uint64_t seedS, float *y,
                      hipStream_t stream)
{
    if constexpr (HB_PART_MODE != hb::kRelu) {
        return hipErrorInvalidDeviceFunction;
    } else if constexpr (hb::TileTraits<W>::kSupported) {
        const hb::TileGrid grid = hb::tile_grid((n + hb::TileTraits<W>::kTile - 1) / hb::TileTraits<W>::kTile, W, 2, hb::kSimulator);
        if (grid.blocks == 0) return hipErrorInvalidConfiguration;
        auto go = [&](auto form) {
            constexpr int kForm = decltype(form)::value;
            hipLaunchKernelGGL((hb::tile_sim_kernel<W, kForm>), dim3(grid.blocks), dim3(hb::kBlock), (hb::tile_lds_bytes<W, hb::kRelu>(hb::has_quarters(kForm))),
                               stream, x, n, k, seedB, seedA, seedS, y, grid.whole_blocks);
            return hipGetLastError();
        };
        return hb::with_form<W, true>(grid, go);
    } else {
        const uint64_t blocks = (n + hb::kBlock - 1) / hb::kBlock;
        if (blocks == 0 || blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
        auto go = [&](auto runs) {
            hipLaunchKernelGGL((hb::wide_sim_kernel<W, decltype(runs)::value>), dim3((unsigned)blocks), dim3(hb::kBlock), 0, stream, x, n, k,
                               seedB, seedA, seedS, y);
            return hipGetLastError();
        };
        return hb::group_runs(blocks) ? go(std::true_type{}) : go(std::false_type{});
    }
}

template <int W>
void fill(hb::LauncherTable &t)
{
    if (HB_PART_MODE == hb::kRelu) t.sim[W - 1] = &launch_sim<W>;
    t.f[HB_PART_MODE][W - 1] = &launch_group<W, HB_PART_MODE>;
    t.batch[HB_PART_MODE][W - 1] = hb::TileTraits<W>::kSupported ? &launch_batch<W, HB_PART_MODE> : nullptr;
    if constexpr (W < HB_PART_HI) fill<W + 1>(t);
}

struct Registrar {
    Registrar() { fill<HB_PART_LO>(hb::launcher_table()); }
};
const Registrar g_registrar;

}  // namespace
