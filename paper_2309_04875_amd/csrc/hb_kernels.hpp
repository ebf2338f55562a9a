// Kernels of the fused path: both parties of an element live in one thread and every opening stays in registers.
//
//   group_kernel       one thread per group of L = min(64/W, 32) consecutive elements: packs the slices of its
//                      elements into two SWAR words, runs the circuit (gate 0, all prefix rounds, sign), then
//                      finishes its elements one by one (B2A, Beaver multiply).  No LDS.  Used for w > 32.
//   tile_kernel        one wavefront per 64 groups (32 for w <= 3), coalesced 16-byte memory traffic per lane, slices and sign
//   tile_batch_kernel  words exchanged through wave-private LDS (described above the kernel).  The batch form
//                      serves several tensors of one width; tile_sim_kernel is the float-in / float-out form.
//   open_kernel        share0 + share1 or share0 ^ share1.
//
// Nothing but the input shares is read from memory and nothing but the output shares is written: the algorithmic
// traffic is 32 bytes per element (24 for open_kernel, 8 for tile_sim_kernel).
#pragma once

#include <type_traits>

#include "hb_protocol.hpp"

namespace hb {

constexpr int kBlock = 256;

struct alignas(16) U64x2 {
    uint64_t a, b;
};

// Memory accesses with the non-temporal hint: every share is read once and every result written once, so
// nothing is worth keeping in the caches (streaming 2-in / 2-out traffic runs about a tenth faster with it).
// A pair of elements travels as one 16-byte access; the type only promises the 8-byte alignment the interface
// requires (the hardware takes 16-byte global accesses at any 4-byte alignment).
typedef uint64_t u64x2_t __attribute__((ext_vector_type(2), aligned(8)));
__device__ __forceinline__ U64x2 load_stream2(const uint64_t *p)
{
    const u64x2_t v = __builtin_nontemporal_load(reinterpret_cast<const u64x2_t *>(p));
    return U64x2{v.x, v.y};
}
__device__ __forceinline__ void store_stream2(uint64_t *p, U64x2 v)
{
    __builtin_nontemporal_store(u64x2_t{v.a, v.b}, reinterpret_cast<u64x2_t *>(p));
}
__device__ __forceinline__ uint64_t load_stream(const uint64_t *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void store_stream(uint64_t *p, uint64_t v) { __builtin_nontemporal_store(v, p); }

template <int W, int MODE, bool RUNS>
__global__ void __launch_bounds__(kBlock)
group_kernel(const uint64_t *x0, const uint64_t *x1, uint64_t n, uint64_t groups, int k, uint64_t seedB,
             uint64_t seedA, uint64_t *o0, uint64_t *o1)
{
    using S = Shape<W>;
    constexpr int L = S::L;
    // keep the loaded shares in registers across the circuit when that is cheap, else read them again
    constexpr bool kHold = (op_of(MODE) == kRelu) && (L <= 8);

    const uint64_t g = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g >= groups) return;
    const uint64_t i0 = g * (uint64_t)L;
    const bool full = (n - i0) >= (uint64_t)L;
    const int cnt = full ? L : (int)(n - i0);

    uint64_t xa[kHold ? L : 1], xb[kHold ? L : 1];
    uint64_t u0 = 0, u1 = 0;

    if (full && (L % 2 == 0)) {
#pragma unroll
        for (int j = 0; j < L / 2; ++j) {
            const U64x2 a = load_stream2(x0 + i0 + 2 * j), b = load_stream2(x1 + i0 + 2 * j);
            u0 |= ((a.a >> k) & S::kField) << ((2 * j) * W % 64);
            u0 |= ((a.b >> k) & S::kField) << ((2 * j + 1) * W % 64);
            u1 |= ((b.a >> k) & S::kField) << ((2 * j) * W % 64);
            u1 |= ((b.b >> k) & S::kField) << ((2 * j + 1) * W % 64);
            if (kHold) {
                xa[2 * j] = a.a;
                xa[2 * j + 1] = a.b;
                xb[2 * j] = b.a;
                xb[2 * j + 1] = b.b;
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < L; ++j) {
            uint64_t a = 0, b = 0;
            if (j < cnt) {
                a = load_stream(x0 + i0 + j);
                b = load_stream(x1 + i0 + j);
            }
            u0 |= ((a >> k) & S::kField) << (j * W % 64);
            u1 |= ((b >> k) & S::kField) << (j * W % 64);
            if (kHold) {
                xa[j] = a;
                xb[j] = b;
            }
        }
    }

    const uint64_t zg = seedB + (g * (uint64_t)S::words_per_group(shared_of(MODE)) + 1) * kGamma;
    uint64_t wb = 0;
    const Pair sum = a2b_sum<W, shared_of(MODE), op_of(MODE) != kSign, RUNS>(u0, u1, zg, wb);

    const uint64_t zA0 = seedA + (6 * i0 + 1) * kGamma;
    if (full && (L % 2 == 0)) {
#pragma unroll
        for (int j = 0; j < L / 2; ++j) {
            Pair xe{0, 0}, xo{0, 0};
            if (op_of(MODE) == kRelu) {
                if (kHold) {
                    xe = Pair{xa[2 * j], xb[2 * j]};
                    xo = Pair{xa[2 * j + 1], xb[2 * j + 1]};
                } else {
                    const U64x2 a = load_stream2(x0 + i0 + 2 * j);
                    const U64x2 b = load_stream2(x1 + i0 + 2 * j);
                    xe = Pair{a.a, b.a};
                    xo = Pair{a.b, b.b};
                }
            }
            const Pair re = finish_element<W, MODE, RUNS>(sum, wb, 2 * j, xe, zA0 + (uint64_t)(6 * (2 * j)) * kGamma);
            const Pair ro = finish_element<W, MODE, RUNS>(sum, wb, 2 * j + 1, xo, zA0 + (uint64_t)(6 * (2 * j + 1)) * kGamma);
            store_stream2(o0 + i0 + 2 * j, U64x2{re.p0, ro.p0});
            store_stream2(o1 + i0 + 2 * j, U64x2{re.p1, ro.p1});
        }
    } else {
#pragma unroll
        for (int j = 0; j < L; ++j) {
            if (j < cnt) {
                Pair x{0, 0};
                if (op_of(MODE) == kRelu) x = kHold ? Pair{xa[j], xb[j]} : Pair{load_stream(x0 + i0 + j), load_stream(x1 + i0 + j)};
                const Pair r = finish_element<W, MODE, RUNS>(sum, wb, j, x, zA0 + (uint64_t)(6 * j) * kGamma);
                store_stream(o0 + i0 + j, r.p0);
                store_stream(o1 + i0 + j, r.p1);
            }
        }
    }
}

// out = share0 + share1 (mod 2^64) or share0 ^ share1; two elements per thread when VEC.
template <bool VEC>
__global__ void __launch_bounds__(kBlock)
open_kernel(const uint64_t *x0, const uint64_t *x1, uint64_t n, int binary, uint64_t *out)
{
    const uint64_t t = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (VEC) {
        const uint64_t i = 2 * t;
        if (i + 1 < n) {
            const U64x2 a = load_stream2(x0 + i);
            const U64x2 b = load_stream2(x1 + i);
            store_stream2(out + i, binary ? U64x2{a.a ^ b.a, a.b ^ b.b} : U64x2{a.a + b.a, a.b + b.b});
        } else if (i < n) {
            const uint64_t a = load_stream(x0 + i), b = load_stream(x1 + i);
            store_stream(out + i, binary ? (a ^ b) : (a + b));
        }
    } else {
        if (t < n) {
            const uint64_t a = load_stream(x0 + t), b = load_stream(x1 + t);
            store_stream(out + t, binary ? (a ^ b) : (a + b));
        }
    }
}


// ------------------------------------------------------------------------------------------------
// Tile kernel (slice widths up to 32).
//
// A wavefront owns a tile of 64*L consecutive elements = 64 groups (32 groups when L > 16).  Memory traffic and the
// per-element arithmetic are laid out for coalescing: lane l loads / finishes / stores the element
// pairs (2(c*64 + l), +1), so every load and store instruction of the wave covers 1 KiB of
// consecutive addresses.  The circuit is laid out for dealer-word sharing: lane l evaluates group l
// of the tile.  The two layouts meet in the wave's private piece of LDS: owners deposit the sliced
// shares of their elements, group lanes collect the L fields of their group, and after the circuit
// each group lane leaves two bits per element for the owners (Verdict): the opened bit and the dealer's bit, or the two
// parties' sign shares.
// All exchange stays inside one wavefront, whose LDS operations execute in program order, so no
// workgroup barrier is needed; wave_sync() only keeps the compiler from moving LDS accesses across.
// ------------------------------------------------------------------------------------------------

constexpr int kWave = 64;
constexpr int kWavesPerBlock = kBlock / kWave;

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Geometry of a wave-tile for slice width w, shared by the kernels and the host code that counts tiles.
// A wavefront takes 64 groups, or 32 when a group has more than 16 elements (w <= 3): a lane then still owns
// at most 8 element pairs, which is what fits in registers, and only the lower half of the lanes runs the
// (short) circuit.
constexpr int tile_lanes_per_word(int w) { return 64 / w > 32 ? 32 : 64 / w; }
constexpr int tile_groups(int w) { return tile_lanes_per_word(w) > 16 ? 32 : 64; }
constexpr int tile_elements(int w) { return tile_groups(w) * tile_lanes_per_word(w); }
constexpr bool quarters_supported(int w) { return w >= 4 && w <= 32; }      // a tile of 64 groups splits into quarters of 16

// The forms that a tile kernel is built in: with or without the code for quarters of a tile, and with or without RUNS
// (mix_words).
constexpr int kWholeTiles = 0, kQuartersForm = 1, kRunsForm = 2;
constexpr bool has_quarters(int form) { return (form & kQuartersForm) != 0; }
constexpr bool has_runs(int form) { return (form & kRunsForm) != 0; }

template <int W>
struct TileTraits {
    using S = Shape<W>;
    static constexpr int L = S::L;
    static constexpr bool kSupported = (L >= 2);                // every width below 33
    static constexpr int kGroups = tile_groups(W);              // groups per wavefront
    static constexpr int kTile = tile_elements(W);              // elements per wavefront
    static constexpr int kPairs = (kTile / 2 + kWave - 1) / kWave;   // element pairs per lane (the last may be idle)
    // W in {4, 8, 16, 32}: a pair of fields is an addressable LDS item (1, 2, 4, 8 bytes), so owners can
    // write their pair straight into the group's packed word.  Other widths go through one entry per element.
    static constexpr bool kPacked = (W == 4 || W == 8 || W == 16 || W == 32);
    using Item = typename std::conditional<(W == 4), uint8_t,
                 typename std::conditional<(W == 8), uint16_t,
                 typename std::conditional<(W == 16), uint32_t, uint64_t>::type>::type>::type;
};

// Where the owners of GROUPS groups leave the slices of their elements for the group lanes, one of three ways:
//   packed widths        the pair's two fields of a party as an item of that group's word of that party
//   L even, 2W <= 32     one 64-bit entry per pair, party 0's two fields in the lower half and party 1's in the upper,
//                        which a group lane puts in place with one shift (an entry per element took twice the reads and
//                        three times the instructions)
//   other widths         one entry per element, both parties' fields in it
template <int W, int GROUPS>
struct Slices {
    using T = TileTraits<W>;
    using S = Shape<W>;
    static constexpr int L = T::L;
    static constexpr bool kPairEntries = !T::kPacked && L % 2 == 0 && 2 * W <= 32;
    static constexpr int kHalf = (W <= 16) ? 16 : 32;           // bits per party inside an element's entry
    using Entry = typename std::conditional<(W <= 16), uint32_t, uint64_t>::type;
    static constexpr int kBytes = T::kPacked ? 2 * GROUPS * 8 : (GROUPS * L * (int)sizeof(Entry) + 15) / 16 * 16;

    static __device__ __forceinline__ uint64_t field(uint64_t x, int k) { return (x >> k) & S::kField; }
    static __device__ __forceinline__ void deposit(unsigned char *lds, int pr, U64x2 xa, U64x2 xb, int k)
    {
        if constexpr (T::kPacked) {
            using Item = typename T::Item;
            reinterpret_cast<Item *>(lds)[pr] = (Item)(field(xa.a, k) | (field(xa.b, k) << (W % 64)));
            reinterpret_cast<Item *>(lds + GROUPS * 8)[pr] = (Item)(field(xb.a, k) | (field(xb.b, k) << (W % 64)));
        } else if constexpr (kPairEntries) {
            const uint32_t a = (uint32_t)field(xa.a, k) | ((uint32_t)field(xa.b, k) << (W % 32));
            const uint32_t b = (uint32_t)field(xb.a, k) | ((uint32_t)field(xb.b, k) << (W % 32));
            reinterpret_cast<uint64_t *>(lds)[pr] = ((uint64_t)b << 32) | a;
        } else {
            Entry *slices = reinterpret_cast<Entry *>(lds);
            slices[2 * pr] = (Entry)field(xa.a, k) | ((Entry)field(xb.a, k) << kHalf);
            slices[2 * pr + 1] = (Entry)field(xa.b, k) | ((Entry)field(xb.b, k) << kHalf);
        }
    }
    static __device__ __forceinline__ Pair collect(const unsigned char *lds, int grp)
    {
        Pair u{0, 0};
        if constexpr (T::kPacked) {
            u.p0 = reinterpret_cast<const uint64_t *>(lds)[grp];
            u.p1 = reinterpret_cast<const uint64_t *>(lds + GROUPS * 8)[grp];
        } else if constexpr (kPairEntries) {
            const uint64_t *pairs = reinterpret_cast<const uint64_t *>(lds) + grp * (L / 2);
#pragma unroll
            for (int i = 0; i < L / 2; ++i) {
                u.p0 |= lo_word(pairs[i]) << (2 * W * i);
                u.p1 |= (pairs[i] >> 32) << (2 * W * i);
            }
        } else {
            const Entry *slices = reinterpret_cast<const Entry *>(lds) + grp * L;
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const Entry en = slices[j];
                u.p0 |= (uint64_t)(en & (Entry)S::kField) << (j * W);
                u.p1 |= (uint64_t)(en >> kHalf) << (j * W);
            }
        }
        return u;
    }
    static __device__ __forceinline__ uint64_t lo_word(uint64_t v) { return (uint32_t)v; }
};

// ---- what a group lane publishes for the owners of its elements -------------------------------------------------
// Two bits per element: the opened bit z and the dealer's bit r (B2aBits), or the two parties' sign shares.  Where a pair
// of fields is an LDS item (kPacked) they sit at bits jW and jW + 1 of one word per group, where a group has 32 elements
// (kDense, W <= 2) at bits 2j and 2j + 1 of one word, other widths publish a byte per element.  Either way an owner reads its
// pair's item at its pair's index and takes four bits at constant places.
// (Publishing two words per group, for every owner to find its group and shift by its field's place, took 14 more vector
// instructions per pair in the widths that are not packed.)
template <int W, int MODE>
struct Verdict {
    using T = TileTraits<W>;
    using S = Shape<W>;
    static constexpr bool kSigns = op_of(MODE) == kSign;
    static constexpr bool kDense = T::L == 32;
    static constexpr int bytes(int groups) { return T::kPacked || kDense ? 8 * groups : (groups * T::L + 15) / 16 * 16; }

    // bit 2j -> bit jW, for the packed widths
    static __device__ __forceinline__ uint32_t spread_half(uint32_t v)
    {
        if constexpr (W == 32) {
            return v & 1u;
        } else if constexpr (W == 4) {
            v = (v & 0x55u) | ((v & 0x5500u) << 8);
            v = (v | (v << 4)) & 0x05050505u;
            return (v | (v << 2)) & 0x11111111u;
        } else {
            // every bit moves by a multiple of W - 2: one multiply makes all the moves, and what else it produces
            // stays off the places that are kept (sums of two bits carry into the next place only)
            constexpr uint32_t kMoves = (W == 16) ? 0x4001u : 0x41041u, kIn = (W == 16) ? 0x5u : 0x55u;
            constexpr uint32_t kOut = (W == 16) ? 0x10001u : 0x1010101u;
            return ((v & kIn) * kMoves) & kOut;
        }
    }
    template <class Word>
    static __device__ __forceinline__ Word spread(uint64_t v)
    {
        if constexpr (sizeof(Word) == 4) return spread_half((uint32_t)v);
        else return ((uint64_t)spread_half((uint32_t)(v >> (2 * (32 / W)))) << 32) | spread_half((uint32_t)v);
    }
    static __device__ __forceinline__ uint32_t bit_at(uint64_t v, int at)
    {
        return at < 32 ? __builtin_amdgcn_ubfe((uint32_t)v, at, 1) : __builtin_amdgcn_ubfe((uint32_t)(v >> 32), at - 32, 1);
    }
    // bit jW -> bit 2j, for the dense widths
    static __device__ __forceinline__ uint32_t to_even_half(uint32_t v)
    {
        v = (v | (v << 8)) & 0x00ff00ffu;
        v = (v | (v << 4)) & 0x0f0f0f0fu;
        v = (v | (v << 2)) & 0x33333333u;
        return (v | (v << 1)) & 0x55555555u;
    }
    static __device__ __forceinline__ uint64_t to_even(uint64_t v)
    {
        if constexpr (W == 2) return v & 0x5555555555555555ull;
        else return ((uint64_t)to_even_half((uint32_t)v >> 16) << 32) | to_even_half((uint32_t)v & 0xffffu);
    }
    // Bits at .. at + COUNT - 1 (COUNT <= 4) of v; `at` is known at compile time once the loop around is unrolled.
    template <int COUNT>
    static __device__ __forceinline__ uint32_t bits_at(uint64_t v, int at)
    {
        if (at % 32 + COUNT > 32) return (uint32_t)(v >> at) & ((1u << COUNT) - 1);
        return __builtin_amdgcn_ubfe(at < 32 ? (uint32_t)v : (uint32_t)(v >> 32), at % 32, COUNT);
    }
    // Writes the bytes of FIELDS elements, byte(j) or two(j) (those of j and j + 1), four, two or one at a time as their
    // number allows.  Three parties, w = 5, DReLU, 1000 tiles: 10.5 us, with a store per element 11.0; sign shares at w = 6 4.9
    // and 5.1.
    template <int FIELDS, class Byte, class Two>
    static __device__ __forceinline__ void store_bytes(unsigned char *to, const Byte &byte, const Two &two)
    {
        if constexpr (FIELDS % 4 == 0) {
#pragma unroll
            for (int j = 0; j < FIELDS; j += 4) reinterpret_cast<uint32_t *>(to)[j / 4] = two(j) | (two(j + 2) << 16);
        } else if constexpr (FIELDS % 2 == 0) {
#pragma unroll
            for (int j = 0; j < FIELDS; j += 2) reinterpret_cast<uint16_t *>(to)[j / 2] = (uint16_t)two(j);
        } else {
#pragma unroll
            for (int j = 0; j < FIELDS; ++j) to[j] = (unsigned char)byte(j);
        }
    }
    // The FIELDS fields of one word of the circuit's sum; `slot`: number of the word in the tile.  wb: the group's B2A
    // word with the bits of the first of these fields at 0 and 1.
    template <class Word, int FIELDS>
    static __device__ __forceinline__ void publish(unsigned char *lds, int slot, WordPair<Word> sum, uint64_t wb)
    {
        const Word s0 = sum.p0 >> (W - 1), s1 = sum.p1 >> (W - 1), sx = (sum.p0 ^ sum.p1) >> (W - 1);     // field j: bit jW
        const uint64_t rx = wb ^ (wb >> 1);                                                              // bit 2j: r
        constexpr Word ones = (Word)S::ones();
        if constexpr (T::kPacked) {
            Word v;
            if constexpr (kSigns) {
                v = (s0 & ones) | ((s1 & ones) << 1);
            } else {
                const Word r = spread<Word>(rx);
                v = bitop3<kTtAndXor>(ones, sx, r) | (r << 1);
            }
            reinterpret_cast<Word *>(lds)[slot] = v;
        } else if constexpr (kDense) {
            constexpr uint64_t kEven = 0x5555555555555555ull;
            const uint64_t r = rx & kEven;
            reinterpret_cast<uint64_t *>(lds)[slot] = kSigns ? to_even(s0) | (to_even(s1) << 1) : (to_even(sx) ^ r) | (r << 1);
        } else if constexpr (kSigns) {
            const uint64_t both = (uint64_t)(s0 & ones) | ((uint64_t)(s1 & ones) << 1);
            auto byte = [&](int j) { return bits_at<2>(both, j * W); };
            auto two = [&](int j) { return byte(j) | (byte(j + 1) << 8); };
            store_bytes<FIELDS>(lds + slot * FIELDS, byte, two);
        } else {
            // bits above the two of a byte are never looked at
            const uint64_t r = rx & 0x5555555555555555ull, rr = r | (r << 1);
            auto byte = [&](int j) { return bit_at(sx, j * W) ^ bits_at<2>(rr, 2 * j); };
            auto two = [&](int j) {
                const uint32_t r4 = bits_at<4>(rr, 2 * j);
                return (bit_at(sx, j * W) | (bit_at(sx, (j + 1) * W) << 8)) ^ (r4 | (r4 << 6));
            };
            store_bytes<FIELDS>(lds + slot * FIELDS, byte, two);
        }
    }
    // What pair `pr` of the tile reads: its first element's bits at 0 and 1 of `lo`, its second's at kSecond of `hi`.
    static constexpr int kSecond = T::kPacked ? W % 32 : kDense ? 2 : 8;
    static __device__ __forceinline__ void read(const unsigned char *lds, int pr, uint32_t &lo, uint32_t &hi)
    {
        if constexpr (T::kPacked) {
            const typename T::Item it = reinterpret_cast<const typename T::Item *>(lds)[pr];
            lo = (uint32_t)it;
            hi = W == 32 ? (uint32_t)((uint64_t)it >> 32) : lo;
        } else if constexpr (kDense) {
            lo = hi = (uint32_t)lds[pr / 2] >> (4 * (pr & 1));
        } else {
            lo = hi = reinterpret_cast<const uint16_t *>(lds)[pr];
        }
    }
    static __device__ __forceinline__ void pick(const unsigned char *lds, int pr, B2aBits (&t)[2])
    {
        uint32_t lo, hi;
        read(lds, pr, lo, hi);
        t[0] = B2aBits{minus_bit(lo, 0), __builtin_amdgcn_ubfe(lo, 1, 1)};
        t[1] = B2aBits{minus_bit(hi, kSecond), __builtin_amdgcn_ubfe(hi, kSecond + 1, 1)};
    }
    static __device__ __forceinline__ void pick_signs(const unsigned char *lds, int pr, Pair (&sign)[2])
    {
        uint32_t lo, hi;
        read(lds, pr, lo, hi);
        sign[0] = Pair{__builtin_amdgcn_ubfe(lo, 0, 1), __builtin_amdgcn_ubfe(lo, 1, 1)};
        sign[1] = Pair{__builtin_amdgcn_ubfe(hi, kSecond, 1), __builtin_amdgcn_ubfe(hi, kSecond + 1, 1)};
    }
};

// The owner's part for one pair: what `io` stores for elements e, e + 1 of the tile.
template <int W, int MODE, bool RUNS>
__device__ __forceinline__ void finish_pair(const unsigned char *verdict, int pr, U64x2 xa, U64x2 xb, uint64_t zA, Pair (&r)[2])
{
    using V = Verdict<W, MODE>;
    if constexpr (op_of(MODE) == kSign) {
        V::pick_signs(verdict, pr, r);
    } else {
        B2aBits t[2];
        V::pick(verdict, pr, t);
        const Pair x[2] = {Pair{xa.a, xb.a}, Pair{xa.b, xb.b}};
        if constexpr (RUNS && op_of(MODE) == kRelu) {       // twelve words in step would take 16 registers more
            finish_elements<MODE, RUNS, 1>({t[0]}, {x[0]}, zA, &r[0]);
            finish_elements<MODE, RUNS, 1>({t[1]}, {x[1]}, zA + 6 * kGamma, &r[1]);
        } else {
            finish_elements<MODE, RUNS, 2>(t, x, zA, r);
        }
    }
}

// ---- where a tile's element pairs come from and where the results go ----------------------------------------
// Shares in, shares out: the library's normal boundary.
// Element i = tile0 + e: tile0 (the tile's first element) is uniform over the wavefront, e is the lane's
// 32-bit offset inside the tile, so an address is a scalar base plus a 32-bit vector offset.
struct ShareIO {
    static constexpr bool kDraws = false;      // shares are what is loaded
    const uint64_t *x0, *x1;
    uint64_t *o0, *o1;
    template <bool FULL>
    __device__ __forceinline__ void load_pair(uint64_t tile0, unsigned e, uint64_t n, U64x2 &a, U64x2 &b) const
    {
        const uint64_t *t0 = x0 + tile0, *t1 = x1 + tile0;
        if (FULL || tile0 + e + 1 < n) {
            a = load_stream2(t0 + e);
            b = load_stream2(t1 + e);
        } else if (tile0 + e < n) {
            a.a = load_stream(t0 + e);
            b.a = load_stream(t1 + e);
        }
    }
    template <bool FULL>
    __device__ __forceinline__ void store_pair(uint64_t tile0, unsigned e, uint64_t n, Pair r0, Pair r1) const
    {
        uint64_t *t0 = o0 + tile0, *t1 = o1 + tile0;
        if (FULL || tile0 + e + 1 < n) {
            store_stream2(t0 + e, U64x2{r0.p0, r1.p0});
            store_stream2(t1 + e, U64x2{r0.p1, r1.p1});
        } else if (tile0 + e < n) {
            store_stream(t0 + e, r0.p0);
            store_stream(t1 + e, r0.p1);
        }
    }
};

// Fixed point of the paper's setting (Sec. 2.2 "Operation of CrypTen", Sec. 3.1): x = round(2^16 x_f),
// ties to even; NaN encodes as 0 and magnitudes are clamped to 2^62 so the conversion is defined for every float.
__host__ __device__ __forceinline__ uint64_t encode_fixed16(float v)
{
    double d = (double)v * 65536.0;
    if (!(d == d)) d = 0.0;
    d = d > 0x1p62 ? 0x1p62 : (d < -0x1p62 ? -0x1p62 : d);
#if defined(__HIP_DEVICE_COMPILE__)
    return (uint64_t)__double2ll_rn(d);
#else
    return (uint64_t)(long long)__builtin_rint(d);
#endif
}

__host__ __device__ __forceinline__ float decode_fixed16(uint64_t v)
{
    return (float)((double)(int64_t)v * (1.0 / 65536.0));
}

struct alignas(8) F32x2 {
    float a, b;
};

// Plaintext floats in, plaintext floats out (the single-node simulator of Sec. 4.1.1): the load encodes to fixed
// point and shares additively with share0[i] = output i of the SplitMix64 stream started at seedS; the store opens
// the two result shares and decodes.  Nothing but 4 bytes per element travels each way.
struct FloatIO {
    static constexpr bool kDraws = true;       // load_pair leaves encoded numbers in b; share() then draws the shares
    const float *x;
    float *y;
    uint64_t seedS;
    template <bool FULL>
    __device__ __forceinline__ void load_pair(uint64_t tile0, unsigned e, uint64_t n, U64x2 &, U64x2 &b) const
    {
        const uint64_t i = tile0 + e;
        const float *t = x + tile0;
        if (FULL || i + 1 < n) {
            const F32x2 v = *reinterpret_cast<const F32x2 *>(t + e);
            b = U64x2{encode_fixed16(v.a), encode_fixed16(v.b)};
        } else if (i < n) {
            b.a = encode_fixed16(t[e]);
        }
    }
    // Of COUNT pairs, those at elements e, e + 2 kWave, ..  Pairs beyond the tensor get shares that nothing reads.
    template <bool RUNS, int COUNT>
    __device__ __forceinline__ void share(uint64_t tile0, unsigned e, U64x2 *a, U64x2 *b) const
    {
        const uint64_t z = seedS + (tile0 + e + 1) * kGamma;
        uint64_t v[2 * COUNT];
        priority<RUNS, kElsewhere>();
#pragma unroll
        for (int i = 0; i < 2 * COUNT; ++i) v[i] = z + (uint64_t)(i / 2 * 2 * kWave + i % 2) * kGamma;
        mix_words<RUNS>(v);
        if constexpr (RUNS) settle(v);
        priority<RUNS, kElsewhere>();
#pragma unroll
        for (int c = 0; c < COUNT; ++c) {
            a[c] = U64x2{v[2 * c], v[2 * c + 1]};
            b[c] = U64x2{b[c].a - a[c].a, b[c].b - a[c].b};
        }
    }
    template <bool FULL>
    __device__ __forceinline__ void store_pair(uint64_t tile0, unsigned e, uint64_t n, Pair r0, Pair r1) const
    {
        float *t = y + tile0;
        if (FULL || tile0 + e + 1 < n) {
            *reinterpret_cast<F32x2 *>(t + e) = F32x2{decode_fixed16(r0.p0 + r0.p1), decode_fixed16(r1.p0 + r1.p1)};
        } else if (tile0 + e < n) {
            t[e] = decode_fixed16(r0.p0 + r0.p1);
        }
    }
};

// FloatIO::share of all pairs with RUNS, up to four of them in step.  (Without RUNS, and in a quarter, pairs are shared as they
// arrive: in step they took 3 to 5 % longer in launches of 100 to 1100 tiles.)
template <int PAIRS, class IO>
__device__ __forceinline__ void draw_shares(const IO &io, uint64_t tile0, int lane, U64x2 (&xa)[PAIRS], U64x2 (&xb)[PAIRS])
{
    constexpr int kAtOnce = PAIRS < 4 ? PAIRS : 4, kRest = PAIRS % kAtOnce;
#pragma unroll
    for (int c = 0; c + kAtOnce <= PAIRS; c += kAtOnce) io.template share<true, kAtOnce>(tile0, (unsigned)(2 * (c * kWave + lane)), xa + c, xb + c);
    if constexpr (kRest > 0)
        io.template share<true, kRest>(tile0, (unsigned)(2 * ((PAIRS - kRest) * kWave + lane)), xa + PAIRS - kRest, xb + PAIRS - kRest);
}

// Work of one wavefront on wave-tile `tile` of one tensor.  lds: this wave's LDS.  FULL: the whole tile lies inside the
// tensor, so no access needs a bounds check (every tile but a tensor's last).
template <int W, int MODE, bool RUNS, bool FULL, class IO>
__device__ __forceinline__ void tile_body_impl(const IO &io, uint64_t n, int k, uint64_t seedB, uint64_t seedA,
                                               uint64_t tile, int lane, unsigned char *lds)
{
    using T = TileTraits<W>;
    using S = Shape<W>;
    using Sl = Slices<W, T::kGroups>;
    static_assert(T::kSupported, "tile kernel needs W <= 32");
    const uint64_t tile0 = tile * T::kTile;
    unsigned char *verdict = lds + Sl::kBytes;

    priority<RUNS, kElsewhere>();
    // ---- owners: load, slice, deposit -------------------------------------------------------
    U64x2 xa[T::kPairs], xb[T::kPairs];
#pragma unroll
    for (int c = 0; c < T::kPairs; ++c) {
        const int pr = c * kWave + lane;     // pair index inside the tile
        const int e = 2 * pr;
        xa[c] = U64x2{0, 0};
        xb[c] = U64x2{0, 0};
        if (e < T::kTile) {
            io.template load_pair<FULL>(tile0, (unsigned)e, n, xa[c], xb[c]);
            if constexpr (IO::kDraws && !RUNS) io.template share<false, 1>(tile0, (unsigned)e, &xa[c], &xb[c]);
            if constexpr (!IO::kDraws || !RUNS) Sl::deposit(lds, pr, xa[c], xb[c], k);
        }
    }
    if constexpr (IO::kDraws && RUNS) {
        draw_shares(io, tile0, lane, xa, xb);
#pragma unroll
        for (int c = 0; c < T::kPairs; ++c) {
            const int pr = c * kWave + lane;
            if (2 * pr < T::kTile) Sl::deposit(lds, pr, xa[c], xb[c], k);
        }
    }
    wave_sync();

    // ---- group lanes: collect fields, run the circuit, publish the verdict ----------------------
    if (T::kGroups == kWave || lane < T::kGroups) {
        const Pair u = Sl::collect(lds, lane);
        const uint64_t g = tile * T::kGroups + lane;
        const uint64_t zg = seedB + (g * (uint64_t)S::words_per_group(shared_of(MODE)) + 1) * kGamma;
        uint64_t wb = 0;
        const Pair sum = a2b_sum<W, shared_of(MODE), op_of(MODE) != kSign, RUNS>(u.p0, u.p1, zg, wb);
        Verdict<W, MODE>::template publish<uint64_t, T::L>(verdict, lane, sum, wb);
    }
    wave_sync();

    // ---- owners: pick up the verdict of each element's group, finish, store ---------------------
    // In a tensor's last tile every pair has addresses and bounds of its own.  Where keeping them across the circuit costs the
    // kernel a wavefront per SIMD (ReLU at w = 4: 125 registers and four of them, otherwise 136 and three) they are worked out
    // again; elsewhere that would only lengthen the one tile (0.2 us of a small launch).
    constexpr bool kAgain = !FULL && (W == 4 ? op_of(MODE) != kSign : W <= 2 && op_of(MODE) == kRelu);
    int own = lane;
    if constexpr (kAgain) asm("" : "+v"(own));
    const uint64_t zA0 = seedA + (6 * (tile0 + 2 * (uint64_t)own) + 1) * kGamma;   // A[6i] of the lane's first element
#pragma unroll
    for (int c = 0; c < T::kPairs; ++c) {
        const int pr = c * kWave + own, e = 2 * pr;
        if (e < T::kTile) {
            Pair r[2];
            finish_pair<W, MODE, RUNS>(verdict, pr, xa[c], xb[c], zA0 + (uint64_t)(12 * c * kWave) * kGamma, r);
            io.template store_pair<FULL>(tile0, (unsigned)e, n, r[0], r[1]);
        }
    }
}

// ---- a quarter of a tile per wavefront ----------------------------------------------------------------------------
// A launch with few tiles lasts as long as one wavefront's instruction stream (about 2000 vector instructions at w = 8,
// most of it dealer words), and so does the last round of any launch.  Here the four wavefronts of a workgroup share one
// tile, 16 groups each.  The four lanes of a group draw every fourth dealer word of the group each and hand them to one
// another through LDS; where the fields of a word split into two halves (L even) lanes then evaluate the gate logic on
// one half, 32 bits, which halves it.  Owners finish one element pair per lane (at w = 8) instead of four.  Same dealer
// indices, same results; 0.30 of the tile's instructions per wavefront (591 of 1974, ReLU at w = 8), 1.2 times the tile's in
// all, so this form takes only what cannot fill the chip (tile_grid).  4 <= w <= 32.
template <int W, int MODE>
struct QuarterTraits {
    using S = Shape<W>;
    using T = TileTraits<W>;
    static constexpr int L = S::L;
    static constexpr bool kSupported = quarters_supported(W);
    static constexpr bool kShared = shared_of(MODE);
    static constexpr int kSplit = 4;                            // lanes per group
    static constexpr int kGroups = kWave / kSplit;              // groups per wavefront
    static constexpr int kTile = kGroups * L;                   // elements per wavefront
    static constexpr int kPairs = (kTile / 2 + kWave - 1) / kWave;
    static constexpr bool kHalves = (L % 2 == 0);
    using Word = typename std::conditional<kHalves, uint32_t, uint64_t>::type;
    static constexpr int kFields = kHalves ? L / 2 : L;         // fields of a Word
    // evaluated dealer words of a group: those of all gates but the last P-update, then the B2A word
    static constexpr int kGateWords = S::b2a_word(kShared) - (kShared ? 3 : 5);
    static constexpr bool kHasB2a = op_of(MODE) != kSign;
    static constexpr int kWords = kGateWords + (kHasB2a ? 1 : 0);
    static constexpr int kWordsPerLane = (kWords + kSplit - 1) / kSplit;
    // A group's row in LDS, in 32-bit units: the lower halves of its words, then the upper ones (whole words where fields
    // do not split).  An odd multiple of four, so that the 16-byte reads of 16 rows fall into different sets of banks.
    static constexpr int kPad = (kWords + 3) / 4 * 4;
    static constexpr int kRow = 2 * kPad + 4;
    using Sl = Slices<W, kGroups>;
    static constexpr int kWordsAt = Sl::kBytes, kVerdictAt = kWordsAt + kGroups * kRow * 4;
    static constexpr int kLdsBytes = kVerdictAt + Verdict<W, MODE>::bytes(kGroups);
};

template <int W, int MODE, bool RUNS, bool FULL, class IO>
__device__ __forceinline__ void quarter_body_impl(const IO &io, uint64_t n, int k, uint64_t seedB, uint64_t seedA,
                                                  uint64_t quarter, int lane, unsigned char *lds)
{
    using Q = QuarterTraits<W, MODE>;
    using S = Shape<W>;
    using Sl = typename Q::Sl;
    using Word = typename Q::Word;
    const uint64_t tile0 = quarter * Q::kTile;
    unsigned char *verdict = lds + Q::kVerdictAt;

    priority<RUNS, kElsewhere>();
    // ---- owners: load ------------------------------------------------------------------------------------
    U64x2 xa[Q::kPairs], xb[Q::kPairs];
#pragma unroll
    for (int c = 0; c < Q::kPairs; ++c) {
        const int e = 2 * (c * kWave + lane);
        xa[c] = U64x2{0, 0};
        xb[c] = U64x2{0, 0};
        if (e < Q::kTile) {
            io.template load_pair<FULL>(tile0, (unsigned)e, n, xa[c], xb[c]);
            if constexpr (IO::kDraws) io.template share<false, 1>(tile0, (unsigned)e, &xa[c], &xb[c]);
        }
    }

    // ---- every lane, while the loads are under way: its share of the group's dealer words ------------------
    const int grp = lane / Q::kSplit, sub = lane % Q::kSplit, half = sub % 2;
    const uint64_t g = quarter * Q::kGroups + grp;
    const uint64_t zs = seedB + (g * (uint64_t)S::words_per_group(Q::kShared) + 1 + (uint64_t)sub) * kGamma;
    uint32_t *row = reinterpret_cast<uint32_t *>(lds + Q::kWordsAt) + grp * Q::kRow;
    // (one by one: in step they cost 2 to 5 % of a launch of 300 to 700 tiles)
#pragma unroll
    for (int t = 0; t < Q::kWordsPerLane; ++t) {
        const int j = t * Q::kSplit + sub;                      // word j of the group; the last one drawn is the B2A word
        if (Q::kWords % Q::kSplit == 0 || t + 1 < Q::kWordsPerLane || j < Q::kWords) {
            uint64_t z = zs + (uint64_t)(t * Q::kSplit) * kGamma;
            int upper = Q::kFields * W;                         // place of the upper half's first field
            if (Q::kHasB2a && t + 1 == Q::kWordsPerLane && j == Q::kWords - 1) {
                z += (uint64_t)(S::b2a_word(Q::kShared) - Q::kGateWords) * kGamma;
                upper = 2 * Q::kFields;
            }
            const uint64_t v = mix64(z);
            if constexpr (Q::kHalves) {
                row[j] = (uint32_t)v;
                row[Q::kPad + j] = word_at(v, upper);
            } else {
                reinterpret_cast<uint64_t *>(row)[j] = v;
            }
        }
    }

    // ---- owners: slice, deposit ---------------------------------------------------------------------------
#pragma unroll
    for (int c = 0; c < Q::kPairs; ++c) {
        const int pr = c * kWave + lane;
        if (2 * pr < Q::kTile) Sl::deposit(lds, pr, xa[c], xb[c], k);
    }
    wave_sync();

    // ---- every lane: the gate logic of its group, or of its half of the fields ------------------------------
    {
        const Pair u = Sl::collect(lds, grp);
        const Word *words = reinterpret_cast<const Word *>(row + (Q::kHalves ? half * Q::kPad : 0));
        WordPair<Word> v{(Word)u.p0, (Word)u.p1};
        if constexpr (Q::kHalves) {
            const int shift = half * (Q::kFields * W);
            v = WordPair<Word>{word_at(u.p0, shift), word_at(u.p1, shift)};
        }
        const WordPair<Word> sum = a2b_sum_words<W, Q::kShared, Word>(v.p0, v.p1, words);
        const uint64_t wb = Q::kHasB2a ? words[Q::kWords - 1] : 0;
        if (sub < (Q::kHalves ? 2 : 1))
            Verdict<W, MODE>::template publish<Word, Q::kFields>(verdict, Q::kHalves ? 2 * grp + half : grp, sum, wb);
    }
    wave_sync();

    // ---- owners: pick up the verdict of each element's group, finish, store -------------------------------
    const uint64_t zA0 = seedA + (6 * (tile0 + 2 * (uint64_t)lane) + 1) * kGamma;
#pragma unroll
    for (int c = 0; c < Q::kPairs; ++c) {
        const int pr = c * kWave + lane, e = 2 * pr;
        if (e < Q::kTile) {
            Pair r[2];
            finish_pair<W, MODE, RUNS>(verdict, pr, xa[c], xb[c], zA0 + (uint64_t)(12 * c * kWave) * kGamma, r);
            io.template store_pair<FULL>(tile0, (unsigned)e, n, r[0], r[1]);
        }
    }
}

// LDS of a workgroup, allocated at launch.
template <int W, int MODE>
constexpr int whole_lds_bytes()
{
    return Slices<W, tile_groups(W)>::kBytes + Verdict<W, MODE>::bytes(tile_groups(W));      // of a wavefront
}
template <int W, int MODE>
constexpr unsigned tile_lds_bytes(bool quarters)
{
    int most = whole_lds_bytes<W, MODE>();
    if constexpr (quarters_supported(W)) {
        if (quarters && QuarterTraits<W, MODE>::kLdsBytes > most) most = QuarterTraits<W, MODE>::kLdsBytes;
    }
    return (unsigned)(kWavesPerBlock * most);
}

// The wavefront's number inside its workgroup, as a scalar: everything derived from it (tile number, tensor
// descriptor, base addresses) then stays in scalar registers.
__device__ __forceinline__ int wave_index()
{
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
}

// Which part of a launch a wavefront takes: workgroups 0 .. whole_blocks - 1 take four tiles each, the others one tile each.
// Every tile kernel of the widths that have quarters exists with them and without.  The one with QUARTERS holds both forms, and with them the larger one's registers and LDS
// for every workgroup (ReLU at w = 24: 72 registers and 28 KiB; whole tiles alone 60 and 5 KiB, eight wavefronts per SIMD instead
// of five), so launches without shared-out tiles take the one without: w = 24 on the shared-mask layout, 640 tiles 4.43 us instead
// of 4.88, 1536 tiles 6.57 instead of 7.01; three parties at w = 4, DReLU, 4 M elements 37 instead of 41.
struct TileWork {
    uint64_t tile;
    int quarter;        // -1: the whole tile
};
template <bool QUARTERS>
__device__ __forceinline__ TileWork tile_work(uint32_t whole_blocks, int wv)
{
    const uint32_t b = blockIdx.x;
    const bool split = QUARTERS && b >= whole_blocks;
    return TileWork{split ? (uint64_t)whole_blocks * (kWavesPerBlock - 1) + b : (uint64_t)b * kWavesPerBlock + wv, split ? wv : -1};
}

// t.tile must be uniform over the wavefront; the tile lies inside the tensor at least in part.
template <int W, int MODE, int FORM, class IO>
__device__ __forceinline__ void tile_body(const IO &io, uint64_t n, int k, uint64_t seedB, uint64_t seedA, TileWork t, int lane, int wv,
                                          unsigned char *tile_lds)
{
    constexpr bool RUNS = has_runs(FORM);
    if constexpr (has_quarters(FORM)) {
        if (t.quarter >= 0) {
            using Q = QuarterTraits<W, MODE>;
            const uint64_t quarter = t.tile * Q::kSplit + (unsigned)t.quarter;
            unsigned char *lds = tile_lds + wv * Q::kLdsBytes;
            if ((quarter + 1) * Q::kTile <= n)
                quarter_body_impl<W, MODE, RUNS, true>(io, n, k, seedB, seedA, quarter, lane, lds);
            else if (quarter * Q::kTile < n)
                quarter_body_impl<W, MODE, RUNS, false>(io, n, k, seedB, seedA, quarter, lane, lds);
            return;
        }
    }
    unsigned char *lds = tile_lds + wv * whole_lds_bytes<W, MODE>();
    if ((t.tile + 1) * TileTraits<W>::kTile <= n)
        tile_body_impl<W, MODE, RUNS, true>(io, n, k, seedB, seedA, t.tile, lane, lds);
    else
        tile_body_impl<W, MODE, RUNS, false>(io, n, k, seedB, seedA, t.tile, lane, lds);
}

// Wavefronts per SIMD that the registers of a kernel of whole tiles have to leave room for, where the compiler's own choice
// is fewer (ReLU at w = 9 and 10: 128 and 108 registers instead of 91 and 81; w = 13..16 on the shared-mask layout 73 instead
// of 71).
constexpr int whole_tile_waves(int w, int op)
{
    return op != kRelu ? 1 : w == 9 || w == 10 ? 5 : w >= 13 && w <= 16 ? 7 : 1;
}

template <int W, int MODE, int FORM>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(has_quarters(FORM) ? 1 : whole_tile_waves(W, op_of(MODE)))))
tile_kernel(const uint64_t *x0, const uint64_t *x1, uint64_t n, int k, uint64_t seedB, uint64_t seedA, uint64_t *o0,
            uint64_t *o1, uint32_t whole_blocks)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char tile_lds[];
    const int lane = threadIdx.x % kWave, wv = wave_index();
    const TileWork t = tile_work<has_quarters(FORM)>(whole_blocks, wv);
    if (t.tile * TileTraits<W>::kTile >= n) return;        // whole wavefront beyond the tensor (uniform per wave)
    tile_body<W, MODE, FORM>(ShareIO{x0, x1, o0, o1}, n, k, seedB, seedA, t, lane, wv, tile_lds);
}

// Several tensors of one slice width in a single launch.  The descriptors travel in the kernel
// argument block; wave-tiles of all tensors are numbered consecutively and tile_end[t] is the number
// of wave-tiles in tensors 0..t, kNoTile from the last tensor on: a tile's tensor is then the number of entries that do not
// exceed the tile's number, which takes one load of the whole table instead of a chain of loads, one tensor after the other.
constexpr int kBatchMax = 24;
constexpr uint32_t kNoTile = 0x7fffffffu;

struct BatchTensor {
    const uint64_t *x0, *x1;
    uint64_t *o0, *o1;
    uint64_t n, seedB, seedA;
    int k;
    uint32_t first_tile;
};

struct BatchArgs {
    uint32_t whole_blocks;             // tile_grid of all tensors' tiles
    uint32_t tiles;                    // of all tensors
    uint32_t tile_end[kBatchMax];
    BatchTensor t[kBatchMax];
    int count;
};

template <int W, int MODE, int FORM>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(has_quarters(FORM) ? 1 : whole_tile_waves(W, op_of(MODE)))))
tile_batch_kernel(const BatchArgs args)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char tile_lds[];
    const int lane = threadIdx.x % kWave, wv = wave_index();
    TileWork t = tile_work<has_quarters(FORM)>(args.whole_blocks, wv);                          // tile number over the whole batch
    const uint32_t gt = (uint32_t)t.tile;                                      // below 2^31 + 4
    if (gt >= args.tiles) return;
    int ti = 0;
#pragma unroll
    for (int i = 0; i < kBatchMax; ++i) ti += (int)((args.tile_end[i] - 1 - gt) >> 31);   // scalar: the borrow, not a comparison
    const BatchTensor &d = args.t[__builtin_amdgcn_readfirstlane(ti)];
    t.tile = gt - d.first_tile;
    tile_body<W, MODE, FORM>(ShareIO{d.x0, d.x1, d.o0, d.o1}, d.n, d.k, d.seedB, d.seedA, t, lane, wv, tile_lds);
}

// The simulator kernel: ReLU on plaintext floats through the whole protocol, 8 bytes of traffic per element.
// Slice widths up to 32 run the wave-tile body; wider slices (one element per word) take one thread per element.
template <int W, bool RUNS>
__global__ void __launch_bounds__(kBlock)
wide_sim_kernel(const float *x, uint64_t n, int k, uint64_t seedB, uint64_t seedA, uint64_t seedS, float *y)
{
    using S = Shape<W>;
    static_assert(S::L == 1, "one element per word");
    const uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const uint64_t x0 = mix64(seedS + (i + 1) * kGamma);
    const uint64_t x1 = encode_fixed16(x[i]) - x0;
    const uint64_t zg = seedB + (i * (uint64_t)S::words_per_group(false) + 1) * kGamma;
    uint64_t wb = 0;
    const Pair sum = a2b_sum<W, false, true, RUNS>((x0 >> k) & S::kField, (x1 >> k) & S::kField, zg, wb);
    const Pair r = finish_element<W, kRelu, RUNS>(sum, wb, 0, Pair{x0, x1}, seedA + (6 * i + 1) * kGamma);
    y[i] = decode_fixed16(r.p0 + r.p1);
}

template <int W, int FORM>
__global__ void __launch_bounds__(kBlock)
tile_sim_kernel(const float *x, uint64_t n, int k, uint64_t seedB, uint64_t seedA, uint64_t seedS, float *y, uint32_t whole_blocks)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char tile_lds[];
    const int lane = threadIdx.x % kWave, wv = wave_index();
    const TileWork t = tile_work<has_quarters(FORM)>(whole_blocks, wv);
    if (t.tile * TileTraits<W>::kTile >= n) return;
    tile_body<W, kRelu, FORM>(FloatIO{x, y, seedS}, n, k, seedB, seedA, t, lane, wv, tile_lds);
}

}  // namespace hb
