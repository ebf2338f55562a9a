// Instantiates the party-faithful kernels of both dealer layouts for slice widths HB_PART_LO..HB_PART_HI and
// registers their launchers.  Compiled several times with different -D values so the parts build in parallel.
#include "hb_launch.hpp"
#include "hb_party.hpp"

#if !defined(HB_PART_LO) || !defined(HB_PART_HI)
#error "compile with -DHB_PART_LO=<w> -DHB_PART_HI=<w>"
#endif

namespace {

template <int W, bool SHARED>
hipError_t launch_party(const hb::PartyCtx &c, hipStream_t stream)
{
    const uint64_t tiles = (c.groups + hb::kHalfWave - 1) / hb::kHalfWave;
    const uint64_t blocks = (tiles + hb::kWavesPerBlock - 1) / hb::kWavesPerBlock;
    if (blocks == 0 || blocks > 0x7fffffffull) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((hb::party_tile_kernel<W, SHARED>), dim3((unsigned)blocks), dim3(hb::kBlock), 0, stream, c);
    return hipGetLastError();
}

template <int W>
void fill(hb::LauncherTable &t)
{
    t.party[0][W - 1] = &launch_party<W, false>;
    t.party[1][W - 1] = &launch_party<W, true>;
    if constexpr (W < HB_PART_HI) fill<W + 1>(t);
}

struct Registrar {
    Registrar() { fill<HB_PART_LO>(hb::launcher_table()); }
};
const Registrar g_registrar;

}  // namespace
