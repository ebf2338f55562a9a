// Float boundary of the simulator (paper Sec. 4.1.1: convert floating point values to ring elements, generate
// secret shares, ... ): stand-alone encode-and-share and open-and-decode kernels.  Included by one translation unit.
#pragma once

#include "hb_kernels.hpp"

namespace hb {

// What bounds both: HBM (20 bytes per element), and below a few million elements the latency of a launch.  A lane takes one
// pair: 16-byte accesses on the shares, 8-byte ones on the floats, which the interface aligns to 4 bytes only.  With the
// non-temporal hint on the shares 16,777,216 elements are shared in 47 us and revealed in 53 (7.1 and 6.4 TB/s; 59 and 57
// without it; 69 and 62 with one element a lane), 802,816 in 5.7 and 5.6 (6.2 and 6.1).  Sharing, a draw per element between load
// and store, starts sooner in smaller workgroups: 128 threads instead of 256, launch after launch, 65,536 elements 2.09 us instead of
// 2.20, 262,144 2.44 / 2.88, 802,816 3.72 / 4.13, 16,777,216 47.4 / 47.4; revealing takes as long either way.
constexpr int kShareBlock = 128;
typedef float f32x2_t __attribute__((ext_vector_type(2), aligned(4)));

// Encode and share: share0[i] = output i of the stream started at seedS, share1[i] = round(2^16 x[i]) - share0[i].
__global__ void __launch_bounds__(kShareBlock)
share_f32_kernel(const float *x, uint64_t n, uint64_t seedS, uint64_t *s0, uint64_t *s1)
{
    const uint64_t i = 2 * ((uint64_t)blockIdx.x * kShareBlock + threadIdx.x);
    if (i >= n) return;
    const uint64_t z = seedS + (i + 1) * kGamma;
    const uint64_t ra = mix64(z);
    if (i + 1 < n) {
        const f32x2_t v = *reinterpret_cast<const f32x2_t *>(x + i);
        const uint64_t rb = mix64(z + kGamma);
        store_stream2(s0 + i, U64x2{ra, rb});
        store_stream2(s1 + i, U64x2{encode_fixed16(v.x) - ra, encode_fixed16(v.y) - rb});
    } else {
        s0[i] = ra;
        s1[i] = encode_fixed16(x[i]) - ra;
    }
}

// Open and decode: y[i] = (share0[i] + share1[i]) / 2^16 as a float.
__global__ void __launch_bounds__(kBlock)
reveal_f32_kernel(const uint64_t *s0, const uint64_t *s1, uint64_t n, float *y)
{
    const uint64_t i = 2 * ((uint64_t)blockIdx.x * kBlock + threadIdx.x);
    if (i >= n) return;
    if (i + 1 < n) {
        const U64x2 a = load_stream2(s0 + i), b = load_stream2(s1 + i);
        *reinterpret_cast<f32x2_t *>(y + i) = f32x2_t{decode_fixed16(a.a + b.a), decode_fixed16(a.b + b.b)};
    } else {
        y[i] = decode_fixed16(s0[i] + s1[i]);
    }
}

}  // namespace hb
