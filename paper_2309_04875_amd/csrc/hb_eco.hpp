// Zero-error high-cut scan (paper Sec. 4.1.2, the "eco" strategy: keep bits [0, m) with the smallest m
// that changes no DReLU result).  With no low cut the two slices are exact shares of x mod 2^m
// (Theorem 1's proof), so DReLU on [0, m) is 1 - bit_{m-1}(x) and it differs from the full-ring result
// exactly when bit m-1 of x differs from its sign bit.  Per element that is one 64-bit word
// d = x ^ (x >>arith 63), and counts[m-1] is the number of elements with bit m-1 of d set.
//
// The 64 population counts are taken without ever touching a counter per element: every lane keeps a
// bit-sliced counter (plane j holds bit j of all 64 per-position counts) and feeds it through a
// carry-save adder tree, two v_bitop3_b32 per 64-bit carry-save step.
//
// What bounds it: HBM, 16 bytes per element.  A workgroup is 16 wavefronts and a launch one workgroup per compute unit,
// all of it resident at once, and the rows (128 elements, one pair per lane) are dealt out in turn: four wavefronts per
// SIMD keep enough loads in flight, every unit has the same work, and the 64 counters see only 256 workgroups' atomics
// (shorter workgroups lose to those).  12,845,056 elements: 39.6 us with the clearing launch (5.2 TB/s;
// 67,108,864: 164 us, 6.6 TB/s) against 49.4 and 174 when a wavefront took a whole number of 64-element chunks per lane and a
// workgroup four wavefronts, which at the smaller size left a quarter of the units idle.  The butterfly on half words is half
// as long as on whole ones.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hb_kernels.hpp"

namespace hb {

constexpr int kEcoPlanes = 16;          // a lane may count up to 2^16 - 1 elements
constexpr int kEcoBlock = 1024;
constexpr int kEcoWaves = kEcoBlock / kWave;
constexpr int kEcoRow = 2 * kWave;      // elements per row
constexpr int kEcoRows = 4;             // rows consumed by one carry-save tree (8 rows a tree: 40.0 us, 16: 47.0, where 4 take 38.8)
constexpr uint64_t kEcoMaxRows = 16384; // rows per wavefront

// a ^ b ^ c, or the majority of the three
__device__ __forceinline__ uint32_t bit3_32(uint32_t a, uint32_t b, uint32_t c, bool majority)
{
    // xor3: 0xF0 ^ 0xCC ^ 0xAA = 0x96; majority: (a&b)|(a&c)|(b&c) = 0xE8
    return majority ? __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8) : __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint64_t bit3(uint64_t a, uint64_t b, uint64_t c, bool majority)
{
    return ((uint64_t)bit3_32((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), majority) << 32) |
           bit3_32((uint32_t)a, (uint32_t)b, (uint32_t)c, majority);
}

// Sign-disagreement words of the lane's pair in every row of a tree.
template <int ROWS>
struct EcoRows {
    U64x2 a[ROWS], b[ROWS];
    __device__ __forceinline__ void load(const uint64_t *x0, const uint64_t *x1, uint64_t row, uint64_t stride, unsigned lane_offset)
    {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint64_t first = (row + (uint64_t)r * stride) * kEcoRow;      // scalar base, 32-bit lane offset
            a[r] = load_stream2(x0 + first + lane_offset);
            b[r] = load_stream2(x1 + first + lane_offset);
        }
    }
    // the same where rows or the lane's pair may lie beyond the tensor: zero shares, which no counter sees
    __device__ __forceinline__ void load_checked(const uint64_t *x0, const uint64_t *x1, uint64_t n, uint64_t row, uint64_t stride, unsigned lane_offset)
    {
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const uint64_t i = (row + (uint64_t)r * stride) * kEcoRow + lane_offset;
            a[r] = b[r] = U64x2{0, 0};
            if (i + 1 < n) {
                a[r] = load_stream2(x0 + i);
                b[r] = load_stream2(x1 + i);
            } else if (i < n) {
                a[r].a = load_stream(x0 + i);
                b[r].a = load_stream(x1 + i);
            }
        }
    }
    __device__ __forceinline__ void pair(int r, uint64_t &d0, uint64_t &d1) const
    {
        const uint64_t xa = a[r].a + b[r].a, xb = a[r].b + b[r].b;
        d0 = xa ^ (uint64_t)((int64_t)xa >> 63);
        d1 = xb ^ (uint64_t)((int64_t)xb >> 63);
    }
};

// Word of weight 2^J summarising 2^J consecutive inputs starting at input idx * 2^J; planes 0..J-1 absorb the rest.
template <int J, int ROWS>
__device__ __forceinline__ uint64_t eco_level(uint64_t (&plane)[kEcoPlanes], const EcoRows<ROWS> &rows, int idx)
{
    if constexpr (J == 1) {
        uint64_t d0, d1;
        rows.pair(idx, d0, d1);
        const uint64_t carry = bit3(plane[0], d0, d1, true);
        plane[0] = bit3(plane[0], d0, d1, false);
        return carry;
    } else {
        const uint64_t a = eco_level<J - 1, ROWS>(plane, rows, 2 * idx);
        const uint64_t b = eco_level<J - 1, ROWS>(plane, rows, 2 * idx + 1);
        const uint64_t carry = bit3(plane[J - 1], a, b, true);
        plane[J - 1] = bit3(plane[J - 1], a, b, false);
        return carry;
    }
}

__global__ void __launch_bounds__(64) eco_zero_kernel(unsigned long long *counts) { counts[threadIdx.x] = 0; }

// Adds a word of weight 2^J to the counter; planes from `live` on stay zero (uniform).
template <int J>
__device__ __forceinline__ void eco_add(uint64_t (&plane)[kEcoPlanes], uint64_t carry, int live)
{
#pragma unroll
    for (int j = J; j < kEcoPlanes; ++j) {
        if (j < live) {
            const uint64_t t = plane[j] & carry;
            plane[j] ^= carry;
            carry = t;
        }
    }
}

// Wavefront v of all `gridDim.x` * 16 takes the rows v, v + waves, v + 2 waves, ...  live: planes that a lane's
// count can reach.  With one workgroup the counts are stored, otherwise added to what eco_zero_kernel cleared.
__global__ void __launch_bounds__(kEcoBlock)
eco_scan_kernel(const uint64_t *x0, const uint64_t *x1, uint64_t n, uint64_t rows, int live, unsigned long long *counts)
{
    __shared__ unsigned int partial[kEcoWaves][64];
    const int lane = threadIdx.x % kWave, wv = wave_index();
    const uint64_t waves = (uint64_t)gridDim.x * kEcoWaves, wave = (uint64_t)blockIdx.x * kEcoWaves + wv;
    uint64_t row = wave;

    uint64_t plane[kEcoPlanes];
#pragma unroll
    for (int j = 0; j < kEcoPlanes; ++j) plane[j] = 0;

    for (; row + (kEcoRows - 1) * waves < n / kEcoRow; row += kEcoRows * waves) {
        EcoRows<kEcoRows> in;
        in.load(x0, x1, row, waves, 2 * lane);
        const uint64_t carry = eco_level<3, kEcoRows>(plane, in, 0);      // 8 elements -> planes 0..2 and a word of weight 8
        eco_add<3>(plane, carry, live);
    }
    for (; row < rows; row += kEcoRows * waves) {
        EcoRows<kEcoRows> in;
        in.load_checked(x0, x1, n, row, waves, 2 * lane);
        const uint64_t carry = eco_level<3, kEcoRows>(plane, in, 0);
        eco_add<3>(plane, carry, live);
    }

    // Per-position totals of the wavefront: the 64 lanes' bit-sliced counters are summed by six bit-sliced additions.
    // The first also splits the positions: v_permlane32_swap leaves positions 0-31 of both lanes of a pair on the lower
    // one and 32-63 on the upper one, so that everything after it works on half words.  The other five are a butterfly
    // inside each half (an all-reduce); lane b then reads position b out of the planes.
    uint32_t tot[kEcoPlanes + 6];
    {
        uint32_t carry = 0;
#pragma unroll
        for (int j = 0; j < kEcoPlanes + 6; ++j) {
            tot[j] = 0;
            if (j < kEcoPlanes && j < live) {
                typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
                const u32x2_t v = __builtin_amdgcn_permlane32_swap((uint32_t)plane[j], (uint32_t)(plane[j] >> 32), false, false);
                tot[j] = bit3_32(v.x, v.y, carry, false);
                carry = bit3_32(v.x, v.y, carry, true);
            } else if (j == live) {
                tot[j] = carry;                                       // the sum is one plane longer
            }
        }
    }
#pragma unroll
    for (int level = 1; level < 6; ++level) {
        const int stride = 32 >> level;
        uint32_t carry = 0;
#pragma unroll
        for (int j = 0; j < kEcoPlanes + 6; ++j) {
            if (j < live + level) {                                   // planes above are still zero (uniform)
                const uint32_t other = __shfl_xor(tot[j], stride, kWave);
                const uint32_t sum = bit3_32(tot[j], other, carry, false);
                carry = bit3_32(tot[j], other, carry, true);
                tot[j] = sum;
            } else if (j == live + level) {
                tot[j] = carry;
            }
        }
    }
    unsigned int mine = 0;                                            // lane b: the total for position b
#pragma unroll
    for (int j = 0; j < kEcoPlanes + 6; ++j) {
        if (j < live + 6) mine |= ((tot[j] >> (lane & 31)) & 1u) << j;
    }
    partial[wv][lane] = mine;
    __syncthreads();
    if (wv == 0) {
        unsigned long long sum = 0;
#pragma unroll
        for (int v = 0; v < kEcoWaves; ++v) sum += partial[v][lane];
        if (gridDim.x == 1) counts[lane] = sum;
        else if (sum != 0) atomicAdd(&counts[lane], sum);
    }
}

}  // namespace hb
