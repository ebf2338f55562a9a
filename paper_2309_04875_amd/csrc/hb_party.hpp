// Party-faithful evaluation of one ReLU: every opening of the protocol is a message of its own.
//
// The fused kernels keep both parties in one thread and open values in registers.  Here each party is evaluated by its
// own threads: lanes 0-31 of a wavefront are party 0 and lanes 32-63 party 1, lane l and lane l + 32 working on the same
// group or elements.  A lane owns its party's share and circuit state, and learns of the other party only what two
// exchange operations inside the wavefront deliver: that party's messages, and what the dealer has to send.  Every word it
// sends it also writes to its party's "wire" (the packed words of paper Sec. 2.2 and Sec. 4.2: every AND, the B2A and the
// multiply open masked values, w-bit fields packed in 64-bit words, depth ceil(log2 w)): a transcript, which nothing
// here reads back.  The message schedule is
//     slice + gate 0  ->  R prefix rounds  ->  B2A bits  ->  multiply openings
// The words on the wires are what a two-GPU run would put on the link, and the result shares are bit-identical to the
// fused kernels'.
//
// Dealer material is generated inline from the same SplitMix64 streams.  A party draws its own triple shares a_p, b_p;
// what the dealer has to send it besides (c_0 to party 0; c_1 to party 1, for which the whole triple is needed; r^A_0 for
// both parties' shares of the B2A bit) is drawn by one half of the wavefront and handed over, two words per generator
// pass: the lower half draws one, the upper half the next.
//
// What bounds it: HBM, with vector-ALU issue close behind (the kernel without its wire stores takes 24 us of the 37 below).
// It moves the 92 bytes per element at w = 8 that it must (shares, results, both wires written once).  2,097,152
// elements at w = 8: 37.2 us, 5.2 TB/s.  One launch per round with all state in memory took 118 us (271 bytes per element:
// every round reloaded the state and both wires, which is how a party got the other's messages, and the masks of a gate were
// drawn twice); the parties in two wavefronts
// that met at workgroup barriers and read each other's wires 64 us (waiting for messages to come back from L2).
//
// Wire of party p (64-bit words): [2G gate 0][4G per round x R][ceil(n/64) B2A][2n multiply]; field j of a
// group word sits at bit j*w and bits that belong to no element are zero.  The last round's P-update gate
// is opened like every other gate (it is part of the opened-bit count) although nothing consumes its result.
// On the shared-mask dealer layout the two gates of a round have one mask for P, so a round sends three words
// per group (P ^ a once, then the two masked second operands): [3G per round x R].
#pragma once

#include "hb_kernels.hpp"

namespace hb {

struct PartyCtx {
    const uint64_t *x[2];
    uint64_t *out[2];
    uint64_t *wire[2];
    uint64_t n, groups;
    uint64_t seedB, seedA;
    uint64_t off_b2a, off_mul;             // word offsets of the B2A and multiply sections of a wire
    int k;
};

constexpr int kHalfWave = kWave / 2;

// Geometry: a wavefront takes 32 groups, 32 lanes of each party.
template <int W>
struct PartyTile {
    static constexpr int L = Shape<W>::L;
    static constexpr int kTile = kHalfWave * L;                          // elements; a multiple of 32
    static constexpr int kPairs = (kTile / 2 + kHalfWave - 1) / kHalfWave;
    static constexpr bool kPacked = TileTraits<W>::kPacked;              // a pair of slices is an LDS item of the group's word
    using Item = typename TileTraits<W>::Item;
    using Entry = typename std::conditional<(W <= 8), uint8_t,
                  typename std::conditional<(W <= 16), uint16_t,
                  typename std::conditional<(W <= 32), uint32_t, uint64_t>::type>::type>::type;
    // LDS per wavefront: the slices, and in the same place, when they are dead, a byte (at W = 4 half a byte) per element
    // and party: the bit that the party sends in the B2A, above it the dealer's bit r
    static constexpr int kSliceBytes = kPacked ? 8 * kWave : 2 * kTile * (int)sizeof(Entry);
    static constexpr int kVerdictBits = W == 4 ? 4 : 8;
    static constexpr int kVerdictBytes = 2 * kTile * kVerdictBits / 8;
    using VerdictPair = typename std::conditional<(W == 4), uint8_t, uint16_t>::type;
    static constexpr int kExchangeBytes = ((kSliceBytes > kVerdictBytes ? kSliceBytes : kVerdictBytes) + 15) / 16 * 16;
};

// What the two halves of the wavefront drew for the dealer, on both lanes of a pair: p0 by lane l, p1 by lane l + 32.
__device__ __forceinline__ Pair dealt(uint64_t v)
{
    typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
    const u32x2_t lo = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    const u32x2_t hi = __builtin_amdgcn_permlane32_swap((uint32_t)(v >> 32), (uint32_t)(v >> 32), false, false);
    return Pair{((uint64_t)hi.x << 32) | lo.x, ((uint64_t)hi.y << 32) | lo.y};
}
// The value of the other party's lane.  The kernel is bound by vector-ALU issue, so openings take the LDS crossbar (one
// instruction per half, no vector instruction); a swap would cost two moves and the swap.
__device__ __forceinline__ uint64_t peer(uint64_t v)
{
    const int at = (int)((threadIdx.x ^ (unsigned)kHalfWave) << 2);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)(uint32_t)v);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(at, (int)(uint32_t)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t opened_xor(uint64_t v) { return v ^ peer(v); }
__device__ __forceinline__ uint64_t opened_sum(uint64_t v) { return v + peer(v); }

// A party's lanes send WORDS 64-bit words each, lane after lane, to `to` (where lane 0's first word goes).  The words pass
// through LDS so that every store instruction covers consecutive addresses (16 or 8 bytes a lane): wire words are written
// once and never read back, and the non-temporal hint, which a lane-strided store pays for with partial lines (69 us
// against 41 for 2,097,152 elements at w = 8), then saves time (39 us).  `words` of the half's 32 x WORDS words are sent (an
// even number of them when WORDS is 4).
template <int WORDS, bool FULL>
__device__ __forceinline__ void send(uint64_t *to, const uint64_t (&m)[WORDS], int words, int p, int l, uint64_t *stage)
{
    uint64_t *s = stage + p * (kHalfWave * 4);
    if constexpr (WORDS == 3) {
#pragma unroll
        for (int t = 0; t < WORDS; ++t) s[WORDS * l + t] = m[t];
        wave_sync();
#pragma unroll
        for (int t = 0; t < WORDS; ++t) {
            const int q = t * kHalfWave + l;
            if (FULL || q < words) store_stream(to + q, s[q]);
        }
    } else {
        static_assert(WORDS == 4, "four words travel as two pairs");
        U64x2 *s2 = reinterpret_cast<U64x2 *>(s);
        s2[2 * l] = U64x2{m[0], m[1]};
        s2[2 * l + 1] = U64x2{m[2], m[3]};
        wave_sync();
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int q = t * kHalfWave + l;
            if (FULL || 2 * q < words) store_stream2(to + 2 * q, s2[q]);
        }
    }
    wave_sync();
}

// One tile.  FULL: the whole tile lies inside the tensor.
template <int W, bool SHARED, bool FULL>
__device__ __forceinline__ void party_tile_body(const PartyCtx &c, uint64_t tile, int lane, unsigned char *lds, uint32_t *opened_bits,
                                                uint64_t *stage)
{
    using S = Shape<W>;
    using T = PartyTile<W>;
    constexpr int L = T::L;
    const int p = lane / kHalfWave, l = lane % kHalfWave;
    const uint64_t tile0 = tile * T::kTile;
    const uint64_t party1 = 0 - (uint64_t)p, party0 = ~party1;  // masks
    const uint64_t own = kGamma & party1;                       // stream distance from a word of party 0 to party p's
    const uint64_t *x = (p ? c.x[1] : c.x[0]) + tile0;
    uint64_t *out = (p ? c.out[1] : c.out[0]) + tile0;
    uint64_t *wire = p ? c.wire[1] : c.wire[0];

    // ---- owners: load own shares, slice, deposit ------------------------------------------------------------
    U64x2 xs[T::kPairs];
#pragma unroll
    for (int i = 0; i < T::kPairs; ++i) {
        const int pr = i * kHalfWave + l;
        const unsigned e = 2 * pr;
        xs[i] = U64x2{0, 0};
        if (e < (unsigned)T::kTile) {
            if (FULL || tile0 + e + 1 < c.n) xs[i] = load_stream2(x + e);
            else if (tile0 + e < c.n) xs[i].a = load_stream(x + e);
            const uint64_t ua = (xs[i].a >> c.k) & S::kField, ub = (xs[i].b >> c.k) & S::kField;
            if constexpr (T::kPacked) {
                reinterpret_cast<typename T::Item *>(lds)[p * (T::kTile / 2) + pr] = (typename T::Item)(ua | (ub << (W % 64)));
            } else {
                reinterpret_cast<typename T::Entry *>(lds)[p * T::kTile + e] = (typename T::Entry)ua;
                reinterpret_cast<typename T::Entry *>(lds)[p * T::kTile + e + 1] = (typename T::Entry)ub;
            }
        }
    }
    wave_sync();

    // ---- group lanes: the circuit ----------------------------------------------------------------------------
    const uint64_t g0 = tile * kHalfWave, g = g0 + l;
    const bool here = FULL || g < c.groups;
    const int groups_here = FULL || c.groups - g0 > kHalfWave ? kHalfWave : (int)(c.groups - g0);
    uint64_t live = S::keep(0);
    if (!FULL) {
        const uint64_t first = g * (uint64_t)L;
        if (here && c.n - first < (uint64_t)L) live = low_bits((int)(c.n - first) * W);               // below 64 bits
    }
    uint64_t u = 0;
    if constexpr (T::kPacked) {
        u = reinterpret_cast<const uint64_t *>(lds)[lane];
    } else {
        const typename T::Entry *sl = reinterpret_cast<const typename T::Entry *>(lds);
#pragma unroll
        for (int j = 0; j < L; ++j) u |= (uint64_t)sl[lane * L + j] << (j * W);
    }
    const uint64_t zg = c.seedB + (g * (uint64_t)S::words_per_group(SHARED) + 1) * kGamma;
    const uint64_t zp = zg + own;                               // a word of the own party: zp + its index for party 0

    // The dealer's share of c for this party: c_0, or c_1 = ((a_0 ^ a_1) & (b_0 ^ b_1)) ^ c_0.
    auto c_share = [&](uint64_t c0, uint64_t a, uint64_t b) {
        return bitop3<kTtXorAnd>(c0, opened_xor(a) & party1, opened_xor(b));
    };
    // Z_p = acc ^ c_p ^ (d & b_p) ^ (e & a_p), party 0 also takes d & e
    auto finish = [&](uint64_t acc, uint64_t cs, uint64_t a, uint64_t b, uint64_t d, uint64_t e) {
        return bitop3<kTtXorAnd>(bitop3<kTtXorAnd>(acc ^ cs, d, bitop3<kTtXorAnd>(b, e, party0)), e, a);
    };

    // gate 0 = X AND Y with X = (u_0, 0), Y = (0, u_1); S_p = P_p = X_p ^ Y_p is party p's own slice
    uint64_t P = u, G, wb;
    {
        const uint64_t a = mix64(zp), b = mix64(zp + 2 * kGamma);
        const U64x2 m{((u & party0) ^ a) & live, ((u & party1) ^ b) & live};
        if (here) store_stream2(wire + 2 * g, m);
        const Pair w = dealt(mix64(zg + (p ? (uint64_t)S::b2a_word(SHARED) : 4) * kGamma));    // c_0, and the B2A word
        wb = w.p1;
        G = finish(0, c_share(w.p0, a, b), a, b, opened_xor(m.a), opened_xor(m.b));
    }
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        constexpr int kWords = SHARED ? 3 : 4;
        const int s = 1 << r;
        const uint64_t keep = S::keep(s);
        const bool last = r + 1 == S::R;
        // words of the round: standard layout a_0 a_1 b_0 b_1 c_0 of the G-update, then of the P-update; shared mask
        // a_0 a_1 | b_0 b_1 c_0 of the G-update | b_0 b_1 c_0 of the P-update
        const uint64_t z0 = not_before((uint64_t)S::round_word(SHARED, r) * kGamma, G);
        const uint64_t zr = zp + z0;
        const uint64_t a = mix64(zr), b = mix64(zr + 2 * kGamma);
        const uint64_t aq = SHARED ? a : mix64(zr + 5 * kGamma), bq = mix64(zr + (SHARED ? 5 : 7) * kGamma);
        const uint64_t m0 = (P ^ a) & live, m1 = (((G << s) & keep) ^ b) & live;
        const uint64_t m2 = SHARED ? m0 : (P ^ aq) & live, m3 = (((P << s) & keep) ^ bq) & live;
        uint64_t *to = wire + 2 * c.groups + (uint64_t)kWords * (c.groups * (uint64_t)r + g0);
        if constexpr (SHARED) send<3, FULL>(to, {m0, m1, m3}, 3 * groups_here, p, l, stage);
        else send<4, FULL>(to, {m0, m1, m2, m3}, 4 * groups_here, p, l, stage);
        // c_0 of the G-update from the lower half, of the P-update from the upper half (the last P-update is opened,
        // but its result is not used: its c_0 is not drawn)
        const Pair c0 = dealt(mix64(zg + z0 + (p && !last ? (uint64_t)(SHARED ? 7 : 9) : 4) * kGamma));
        const uint64_t d = opened_xor(m0);
        G = finish(G, c_share(c0.p0, a, b), a, b, d, opened_xor(m1));
        if (!last) P = finish(0, c_share(c0.p1, aq, bq), aq, bq, SHARED ? d : opened_xor(m2), opened_xor(m3));
    }

    // ---- B2A message: sign share ^ dealer bit share, one bit per element ---------------------------------------
    // The group's lane publishes a byte per element, which an owner finds at its element's index.  (Finding the group and
    // shifting its words by the field's place takes 64-bit shifts by an amount that differs between lanes: word_at.)
    unsigned char *verdict = lds + p * (T::kVerdictBytes / 2);
    wave_sync();
    {
        const uint64_t sign = (u ^ ((G << 1) & S::keep(1))) >> (W - 1);                       // bit jW: sign share
        const uint64_t own_rho = ((wb >> 1) & party1) | (wb & party0), rx = wb ^ (wb >> 1);   // bit 2j: rho_p, r
        if constexpr (T::kVerdictBits == W) {                                                 // the word's fields
            using V = Verdict<W, kRelu>;
            const uint64_t v = ((sign & S::ones()) ^ V::template spread<uint64_t>(own_rho)) | (V::template spread<uint64_t>(rx) << 1);
            reinterpret_cast<uint64_t *>(lds)[lane] = v;
        } else {
            constexpr uint64_t kEven = 0x5555555555555555ull;
            const uint64_t q = (own_rho & kEven) | ((rx & kEven) << 1);
#pragma unroll
            for (int j = 0; j < L; ++j) {
                const uint32_t rho = 2 * j < 32 ? (uint32_t)q >> (2 * j % 32) : (uint32_t)(q >> 32) >> (2 * j % 32);
                verdict[l * L + j] = (unsigned char)(Verdict<5, kRelu>::bit_at(sign, j * W) ^ rho);   // two bits are looked at
            }
        }
    }
    wave_sync();
    uint32_t message = 0, opened = 0;           // lane t < L of a half: bits of elements 32t .. 32t + 31 of the tile
#pragma unroll
    for (int t = 0; t < L; ++t) {
        const int e = t * kHalfWave + l;
        const uint32_t own = W == 4 ? (uint32_t)verdict[e / 2] >> (4 * (l & 1)) : verdict[e];
        const uint64_t sent = __ballot((own & 1) != 0 && (FULL || tile0 + e < c.n));    // party 0's bits, then party 1's
        const uint32_t lo = (uint32_t)sent, hi = (uint32_t)(sent >> 32);
        if (l == t) {
            message = p ? hi : lo;
            opened = lo ^ hi;
        }
    }
    {
        // the wire's words hold 64 bits: a tile writes its L halves, the last one also a half that no element reaches
        uint32_t *bits = reinterpret_cast<uint32_t *>(wire + c.off_b2a) + tile * (uint64_t)L;
        const bool reached = FULL || tile0 + (uint64_t)l * kHalfWave < ((c.n + 63) & ~63ull);
        if (l < (FULL ? L : L + 1) && reached) bits[l] = message;
        if (FULL && L % 2 != 0 && tile0 + T::kTile == c.n && (tile * L + L) % 2 != 0 && l == L) bits[l] = 0;
    }
    if (l < L) opened_bits[l] = opened;         // both halves write the same
    wave_sync();

    // ---- multiply: send x_p - a_p and DReLU_p - b_p, then finish, one element pair per lane at a time ---------
    const uint64_t zA0 = c.seedA + (6 * (tile0 + 2 * (uint64_t)l) + 1) * kGamma;       // A[6i] of the lane's first element
    // In the tensor's last tile every pair has addresses and bounds of its own; worked out again here they are not kept across
    // the circuit.  At W = 4 that is 124 vector registers, four wavefronts per SIMD, instead of 139 and three.
    int own_l = l;
    if constexpr (W == 4 && !FULL) asm("" : "+v"(own_l));
#pragma unroll
    for (int i = 0; i < T::kPairs; ++i) {
        const int pr = i * kHalfWave + own_l;
        const unsigned e = 2 * pr;
        const bool two = e < (unsigned)T::kTile && (FULL || tile0 + e + 1 < c.n);
        const bool one = !FULL && !two && e < (unsigned)T::kTile && tile0 + e < c.n;
        const uint64_t zA = zA0 + (uint64_t)(12 * i * kHalfWave) * kGamma;
        const uint32_t zw = opened_bits[(e / kHalfWave) % L] >> (e % kHalfWave);
        const uint32_t both = reinterpret_cast<const typename T::VerdictPair *>(verdict)[e < (unsigned)T::kTile ? pr : 0];
        // r^A_0 and c_0 of the pair's first element from the lower half, of its second from the upper half
        const uint64_t zh = zA + (6 * kGamma & party1);
        const Pair rA0 = dealt(mix64(zh)), c0 = dealt(mix64(zh + 5 * kGamma));
        uint64_t a[2], b[2], eps[2], del[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int32_t m = minus_bit(zw, h);
            const uint64_t mm = (uint64_t)(int64_t)m;
            const uint32_t r = (both >> (T::kVerdictBits * h + 1)) & (uint32_t)p;            // in party 1's r^A_1 = r - r^A_0 only
            // as in b2a_shares: (~r^A_0 ^ m) + 2 (1 - z) for party 0, ~((~r^A_0 + r) ^ m) + z for party 1
            const uint64_t D = ((~(h ? rA0.p1 : rA0.p0) + r) ^ mm ^ party1) + (uint32_t)(p ? -m : 2 * (m + 1));
            a[h] = mix64(zA + (uint64_t)(6 * h + 1) * kGamma + own);           // A[6i+1] / A[6i+2]
            b[h] = mix64(zA + (uint64_t)(6 * h + 3) * kGamma + own);           // A[6i+3] / A[6i+4]
            eps[h] = (h ? xs[i].b : xs[i].a) - a[h];
            del[h] = D - b[h];
        }
        {
            // a pair's four words; the tensor, or the tile where 32 does not divide its pairs, may end within this chunk
            constexpr int kChunk = 2 * kHalfWave;
            const uint64_t c0e = tile0 + (uint64_t)(i * kChunk);
            constexpr bool kWhole = FULL && T::kTile % kChunk == 0;
            const uint64_t end = tile0 + T::kTile < c.n ? tile0 + T::kTile : c.n;
            const int here_e = c0e >= end ? 0 : end - c0e > (uint64_t)kChunk ? kChunk : (int)(end - c0e);
            uint64_t *to = wire + c.off_mul + 2 * c0e;
            send<4, kWhole>(to, {eps[0], del[0], eps[1], del[1]}, 2 * here_e, p, l, stage);
        }
        U64x2 r;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint64_t E = opened_sum(eps[h]), D = opened_sum(del[h]);
            const uint64_t ab = opened_sum(a[h]) * opened_sum(b[h]), ch = h ? c0.p1 : c0.p0;
            const uint64_t base = p ? ab - ch : ch;                            // c_0; the dealer's c_1 = a b - c_0
            const uint64_t v = sum_of_products(base, E, b[h] + (D & party0), D, a[h]);
            (h ? r.b : r.a) = v;
        }
        if (two) store_stream2(out + e, r);
        else if (one) store_stream(out + e, r.a);
    }
}

// At most four wavefronts per SIMD (two for W <= 2), whatever registers would allow: the writes of more of them get in one
// another's way.  4,000,000 elements, us, with and without the bound: w = 1 63.8 / 67.5, w = 9 108.5 / 112.7, w = 12 107.4 /
// 110.6, w = 48 368 / 392.
template <int W, bool SHARED>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, (W <= 2 ? 2 : 4))))
party_tile_kernel(const PartyCtx c)
{
    using T = PartyTile<W>;
    __shared__ __attribute__((aligned(16))) unsigned char exchange_all[kWavesPerBlock][T::kExchangeBytes];
    __shared__ uint32_t opened_all[kWavesPerBlock][T::L];
    __shared__ __attribute__((aligned(16))) uint64_t stage_all[kWavesPerBlock][kWave * 4];
    const int lane = threadIdx.x % kWave, wv = wave_index();
    const uint64_t tile = (uint64_t)blockIdx.x * kWavesPerBlock + wv;
    if (tile * T::kTile >= c.n) return;        // whole wavefront beyond the tensor (uniform per wave)
    if ((tile + 1) * T::kTile <= c.n)
        party_tile_body<W, SHARED, true>(c, tile, lane, exchange_all[wv], opened_all[wv], stage_all[wv]);
    else
        party_tile_body<W, SHARED, false>(c, tile, lane, exchange_all[wv], opened_all[wv], stage_all[wv]);
}

}  // namespace hb
