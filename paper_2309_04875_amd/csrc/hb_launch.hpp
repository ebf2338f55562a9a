// Table of kernel launchers indexed by (mode, slice width).  The kernels are instantiated in several
// translation units (hb_launch_part.hip compiled once per mode and width range) that register
// themselves here when the library is loaded.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hb_kernels.hpp"
#include "hb_multiparty.hpp"

namespace hb {

using GroupLauncher = hipError_t (*)(const uint64_t *x0, const uint64_t *x1, uint64_t n, int k, uint64_t seedB,
                                     uint64_t seedA, uint64_t *o0, uint64_t *o1, bool vec16, hipStream_t stream);

// Launches the tensors described by `args` (all of one slice width, tile-kernel eligible) in one grid.
using BatchLauncher = hipError_t (*)(const BatchArgs &args, hipStream_t stream);

// The float-in / float-out simulator kernel of one slice width.
using SimLauncher = hipError_t (*)(const float *x, uint64_t n, int k, uint64_t seedB, uint64_t seedA, uint64_t seedS,
                                   float *y, hipStream_t stream);

// DReLU / ReLU among 3 or 4 parties.
using MpLauncher = hipError_t (*)(const MpPointers &ptr, uint64_t n, int k, uint64_t seedB, uint64_t seedA,
                                  hipStream_t stream);

// The party-faithful ReLU.
struct PartyCtx;
using PartyLauncher = hipError_t (*)(const PartyCtx &c, hipStream_t stream);

struct LauncherTable {
    GroupLauncher f[kModes][64];       // [mode][w - 1]
    BatchLauncher batch[kModes][64];   // null where the width has no tile kernel
    SimLauncher sim[64];               // null where the width has no tile kernel
    MpLauncher mp[kMaxParties - 2][2][64];   // [parties - 3][kDrelu | kRelu][w - 1]
    PartyLauncher party[2][64];        // [shared-mask layout][w - 1]
};

LauncherTable &launcher_table();

// Grid of a launch of wave-tiles: `whole_blocks` workgroups of four tiles, then a workgroup for each of the tiles that
// are shared out by quarters.
struct TileGrid {
    uint32_t whole_blocks, blocks;       // blocks 0: more than a grid holds
    bool quarters;                       // blocks > whole_blocks
};
// op: kDrelu, kRelu, kSign or kSimulator.
constexpr int kSimulator = 3;
TileGrid tile_grid(uint64_t tiles, int w, int parties, int op);

// go(std::true_type) where tiles of the grid are shared out, go(std::false_type) otherwise.
template <int W, class Go>
hipError_t with_quarters(const TileGrid &grid, const Go &go)
{
    if constexpr (quarters_supported(W)) {
        if (grid.quarters) return go(std::true_type{});
    }
    return go(std::false_type{});
}

// Debug knob: HB_KERNEL=group in the environment (read once) sends every width to the thread-per-group kernel.
bool force_group_kernel();

}  // namespace hb
