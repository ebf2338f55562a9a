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
                                     uint64_t seedA, uint64_t *o0, uint64_t *o1, hipStream_t stream);

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
    bool runs;                           // which form of the dealer-word generator (mix_words)
};
// op: kDrelu, kRelu, kSign or kSimulator.
constexpr int kSimulator = 3;
TileGrid tile_grid(uint64_t tiles, int w, int parties, int op);

// Whether tile kernels have the form with RUNS (mix_words), which long launches then take (tile_runs).  Not where memory bounds long
// launches, which wavefronts of unequal priority disturb: 2^25 elements, us, without / with: DReLU at w = 6 177 / 183, w = 8 175 /
// 181, w = 9 203 / 199 (16 M elements on the shared-mask layout 96.5 / 98.4), w = 10 217 / 200; sign shares at w = 6 172 / 180, w = 12 211 / 204 (8 M elements 57 / 58), w = 16 241 / 221.
// Among three and four parties DReLU at w = 4 (2^24 elements, three 142 / 146; w = 5 154 / 148).
// Where the form's registers cost a wavefront per SIMD it gains all the same: the simulator at w = 1 (104 registers instead of 81,
// 2.2, 9.2 and 20.5 M elements 21.1 / 18.9, 55.8 / 51.1, 116 / 106) and w = 4 (102 instead of 93; 16.7 / 15.8, 60.3 / 54.0, 126 / 113),
// ReLU of three parties at w = 2 (130 instead of 121; 1.4, 6.0 and 13.4 M 26.8 / 23.9, 70.2 / 66.8, 154 / 139).
constexpr bool runs_supported(int w, int parties, int op)
{
    if (op == kSign) return w >= 13;
    if (op == kDrelu) return parties == 2 ? w >= 10 : w >= 5;
    return true;
}

// The form of the generator (mix_words) for kernels of one thread per group in `blocks` workgroups: RUNS from where a SIMD has a
// second wavefront.  ReLU at w = 64, us, without / with: 256 blocks 4.5 / 4.8, 272 7.0 / 6.3, 4096 44 / 38, 131072 1320 / 1144.
bool group_runs(uint64_t blocks);

// go(std::integral_constant<int, form>) with the form of kernel that the grid asks for.  RUNS: whether there is one with RUNS.
template <int W, bool RUNS, class Go>
hipError_t with_form(const TileGrid &grid, const Go &go)
{
    auto runs_or_not = [&](auto quarters) {
        constexpr int kQuarters = decltype(quarters)::value;
        if constexpr (RUNS) {
            if (grid.runs) return go(std::integral_constant<int, kQuarters | kRunsForm>{});
        }
        return go(std::integral_constant<int, kQuarters>{});
    };
    if constexpr (quarters_supported(W)) {
        if (grid.quarters) return runs_or_not(std::integral_constant<int, kQuartersForm>{});
    }
    return runs_or_not(std::integral_constant<int, kWholeTiles>{});
}

// Debug knob: HB_KERNEL=group in the environment (read once) sends every width to the thread-per-group kernel.
bool force_group_kernel();

}  // namespace hb
