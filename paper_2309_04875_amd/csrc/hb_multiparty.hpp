// The protocol among P = 3 or 4 parties, all simulated in one thread (P = 2 is the path of hb_kernels.hpp).
//
// The paper's setting allows any number of parties (Sec. 2.2 "Operation of CrypTen"; Sec. 3.1.2 notes that the
// analysis carries over).  What changes against two parties:
//   - the P sliced shares are summed by a tree of two-operand Kogge-Stone adders on XOR shares:
//     P = 3: (X0 + X1) + X2;  P = 4: (X0 + X1) + (X2 + X3); adders numbered in evaluation order;
//   - an AND gate draws 3P - 1 dealer words a_0..a_{P-1} b_0..b_{P-1} c_0..c_{P-2} (the last c completes a & b);
//   - a group owns (P-1)(1+2R)(3P-1) + 1 words; the last one holds the B2A bits, bit P*j + q = rho_q of lane j;
//   - an element owns 4P - 2 arithmetic words: rA_0..rA_{P-2} | a_0..a_{P-1} | b_0..b_{P-1} | c_0..c_{P-2};
//   - party 0 adds every public term.
//
//   mp_group_kernel   one thread per group, scalar 8-byte accesses: slice widths above 32.
//   mp_tile_kernel    one wavefront per 64 groups (32 below w = 4, where a group has 16 or 21 elements) with
//                     coalesced 16-byte accesses, as tile_kernel: slice widths up to 32.  What cannot fill the chip goes by
//                     quarters of a tile, four lanes per group, as there.
//
// Algorithmic traffic: 16 P bytes per element.
#pragma once

#include "hb_kernels.hpp"

namespace hb {

constexpr int kMaxParties = 4;

template <int P, class Word = uint64_t>
struct Shares {      // one value held as P shares
    Word v[P];
};

struct MpPointers {  // kernel argument: the P input and P output arrays
    const uint64_t *x[kMaxParties];
    uint64_t *o[kMaxParties];
};

template <int W, int P>
struct MpShape {
    static_assert(P >= 3 && P <= kMaxParties, "party count");
    using S = Shape<W>;
    static constexpr int R = S::R;
    static constexpr int L = (64 / W) < (64 / P) ? (64 / W) : (64 / P);   // the B2A word holds P bits per lane
    static constexpr int kGateWords = 3 * P - 1;
    static constexpr int kAdderWords = (1 + 2 * R) * kGateWords;
    static constexpr int kB2aWord = (P - 1) * kAdderWords;
    static constexpr int kWordsPerGroup = kB2aWord + 1;
    static constexpr int kArithWords = 4 * P - 2;
};

// Beaver AND among P parties, returned XORed onto acc share by share; word(i) = the gate's dealer word i.  As in the
// two-party gate the operands enter only through the openings: Ux = XOR over the parties of U_q, Vx = XOR of V_q before the
// field mask `keep` of a shifted operand.
template <int P, class Word, class Words>
__device__ __forceinline__ Shares<P, Word> mp_and(const Words &word, Word Ux, Word Vx, Word keep, const Shares<P, Word> &acc)
{
    Word a[P], b[P], c[P];
    Word as = 0, bs = 0, cs = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        a[q] = word(q);
        b[q] = word(P + q);
        as ^= a[q];
        bs ^= b[q];
    }
#pragma unroll
    for (int q = 0; q < P - 1; ++q) {
        c[q] = word(2 * P + q);
        cs ^= c[q];
    }
    c[P - 1] = bitop3<kTtXorAnd>(cs, as, bs);               // the dealer completes the sharing of c = a & b
    const Word d = Ux ^ as;                                 // opened: XOR over the parties of U_q ^ a_q
    const Word e = bitop3<kTtXorAnd>(bs, Vx, keep);         // opened: XOR over the parties of V_q ^ b_q
    Shares<P, Word> Z;
    // party 0 takes the public d & e term: c_0 ^ (d & b_0) ^ (e & a_0) ^ (d & e)
    Z.v[0] = bitop3<kTtXor3>(acc.v[0], bitop3<kTtXorAnd>(c[0], e, a[0]), bitop3<kTtAndXor>(d, b[0], e));
#pragma unroll
    for (int q = 1; q < P; ++q) Z.v[q] = bitop3<kTtXorAnd>(bitop3<kTtXorAnd>(acc.v[q] ^ c[q], d, b[q]), e, a[q]);
    return Z;
}

// X + Y mod 2^W in every field, on XOR shares.  gate(q, after) gives the accessor of gate q's dealer words, which are not
// drawn before `after` is known (with RUNS not before all shares of the gates before).  The last round's P-update gate is not evaluated (nothing reads it; its words are never
// drawn).  Word = uint32_t: the lower or the upper half of the fields, at bits jW of every word.
template <int W, int P, class Word, bool RUNS, class Gates>
__device__ __forceinline__ Shares<P, Word> mp_add_gates(const Gates &gate, const Shares<P, Word> &X, const Shares<P, Word> &Y)
{
    using S = Shape<W>;
    Shares<P, Word> Pw, Sum, zero;
    Word Xx = 0, Yx = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        Pw.v[q] = Sum.v[q] = X.v[q] ^ Y.v[q];
        zero.v[q] = 0;
        Xx ^= X.v[q];
        Yx ^= Y.v[q];
    }
    Shares<P, Word> G = mp_and<P, Word>(gate(0, Xx), Xx, Yx, (Word)~0ull, zero);
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        const int s = 1 << r;
        const Word keep = (Word)S::keep(s);
        // shifting is linear: the XOR of the parties' shifted shares is the shifted XOR of their shares
        Word Gx = 0, Px = 0;
#pragma unroll
        for (int q = 0; q < P; ++q) {
            Gx ^= G.v[q];
            Px ^= Pw.v[q];
        }
        // one gate's dealer words at a time: 3P - 1 live words instead of the whole adder's
        if constexpr (RUNS) settle(G.v);
        if (RUNS && !(r + 1 == S::R && W >= 34)) settle(Pw.v);      // (a last round on one field reads the upper half only)
        G = mp_and<P, Word>(gate(1 + 2 * r, Gx), Px, (Word)(Gx << s), keep, G);
        if constexpr (RUNS) settle(G.v);
        if (r + 1 < S::R) Pw = mp_and<P, Word>(gate(2 + 2 * r, G.v[0]), Px, (Word)(Px << s), keep, zero);
    }
    const Word keep1 = (Word)S::keep(1);
    Shares<P, Word> out;
#pragma unroll
    for (int q = 0; q < P; ++q) out.v[q] = Sum.v[q] ^ ((G.v[q] << 1) & keep1);
    return out;
}

// N consecutive words; with RUNS and more than ten of them (four parties) in two batches: in step they would take 12 registers
// more, a wavefront per SIMD.
template <bool RUNS, int N>
__device__ __forceinline__ void draw_in_two(uint64_t z, uint64_t (&v)[N])
{
    constexpr int kFirst = RUNS && N > 10 ? (N + 1) / 2 : N, kRest = N - kFirst;
    uint64_t f[kFirst];
    draw_words<RUNS, kFirst>(z, f);
#pragma unroll
    for (int i = 0; i < kFirst; ++i) v[i] = f[i];
    if constexpr (kRest > 0) {
        settle(f);
        uint64_t s[kRest];
        draw_words<RUNS, kRest>(z, s);
#pragma unroll
        for (int i = 0; i < kFirst; ++i) v[i] = f[i];
#pragma unroll
        for (int i = 0; i < kRest; ++i) v[kFirst + i] = s[i];
    }
}

// The adder drawing its words inline; za = generator state of its first dealer word.
template <int W, int P, bool RUNS>
__device__ __forceinline__ Shares<P> mp_add(uint64_t za, const Shares<P> &X, const Shares<P> &Y)
{
    constexpr int kWords = MpShape<W, P>::kGateWords;
    struct Drawn {
        uint64_t v[kWords];
        __device__ __forceinline__ uint64_t operator()(int i) const { return v[i]; }
    };
    auto gate = [za](int q, uint64_t after) {
        const uint64_t zq = za + (uint64_t)(q * kWords) * kGamma;
        uint64_t z = RUNS || q == 0 ? zq : not_before(zq, after);
        Drawn d;
        draw_in_two<RUNS, kWords>(z, d.v);
        return d;
    };
    return mp_add_gates<W, P, uint64_t, RUNS>(gate, X, Y);
}

// XOR shares of (u_0 + ... + u_{P-1}) mod 2^W for one group; add(i, X, Y) is adder i of the tree.
template <int P, class Word, class Add>
__device__ __forceinline__ Shares<P, Word> mp_tree(const Word (&u)[P], const Add &add)
{
    Shares<P, Word> X[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
#pragma unroll
        for (int t = 0; t < P; ++t) X[q].v[t] = (t == q) ? u[q] : 0;    // party q shares its slice trivially
    }
    const Shares<P, Word> s01 = add(0, X[0], X[1]);
    if constexpr (P == 3) {
        return add(1, s01, X[2]);
    } else {
        const Shares<P, Word> s23 = add(1, X[2], X[3]);
        return add(2, s01, s23);
    }
}

// The same drawing its words inline; zg = generator state of the group's first word.
template <int W, int P, bool RUNS>
__device__ __forceinline__ Shares<P> mp_a2b_sum(const uint64_t (&u)[P], uint64_t zg)
{
    auto add = [zg](int i, const Shares<P> &X, const Shares<P> &Y) {
        return mp_add<W, P, RUNS>(zg + (uint64_t)(i * MpShape<W, P>::kAdderWords) * kGamma, X, Y);
    };
    return mp_tree<P, uint64_t>(u, add);
}

// Everything after the circuit for one element.  t: the opened bit and the dealer's bit.  zA = generator state of the element's first arithmetic word.  MODE: kDrelu or kRelu.
// As for two parties (b2a_shares): with c_q = ~r^A_q and q = r^A_{P-1} - 1 = c_0 + ... + c_{P-2} + (P - 2) + r,
//   DReLU_0 = (c_0 ^ m) + 2 (1 - z),  DReLU_q = (c_q ^ m) + (1 - z),  DReLU_{P-1} = ~(q ^ m) + z.
template <int P, int MODE, bool RUNS>
__device__ __forceinline__ Shares<P> mp_finish(B2aBits t, const Shares<P> &x, uint64_t zA)
{
    const uint32_t r = t.r;                                   // known to the dealer only
    const int32_t m = t.m;                                    // -z, the opened bit
    const uint64_t mm = (uint64_t)(int64_t)m;
    uint64_t w[MODE == kRelu ? 4 * P - 2 : P - 1];
    draw_in_two<RUNS>(zA, w);
    uint64_t f[P], csum = 0;
#pragma unroll
    for (int q = 0; q < P - 1; ++q) {
        w[q] = held(~w[q]);
        f[q] = held(w[q] ^ mm);
    }
    if constexpr (RUNS) {
        settle(w);
#pragma unroll
        for (int q = 0; q < P - 1; ++q) settle(f[q]);
        priority<true, kElsewhere>();
    }
#pragma unroll
    for (int q = 0; q < P - 1; ++q) csum += w[q];
    f[P - 1] = held(~((csum + (r + (uint32_t)(P - 2))) ^ mm));
    if (MODE == kDrelu) {
        const uint32_t n = (uint32_t)(m + 1), z = (uint32_t)-m;
        Shares<P> D;
#pragma unroll
        for (int q = 0; q < P; ++q) D.v[q] = f[q] + (q == 0 ? 2 * n : q == P - 1 ? z : n);
        return D;
    }

    uint64_t drelu = f[0];                                    // sum of the DReLU_q
#pragma unroll
    for (int q = 1; q < P; ++q) drelu += f[q];
    drelu = held(drelu + (uint32_t)(P + (P - 1) * m));
    const uint64_t *m_words = w + P - 1;                      // a_0 .. | b_0 .. | c_0 ..
    uint64_t a[P], b[P], c[P];
    uint64_t as = 0, bs = 0, cs = 0, xs = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        a[q] = m_words[q];
        b[q] = m_words[P + q];
        as += a[q];
        bs += b[q];
        xs += x.v[q];
    }
#pragma unroll
    for (int q = 0; q < P - 1; ++q) {
        c[q] = m_words[2 * P + q];
        cs += c[q];
    }
    const uint64_t eps = xs - as;                             // opened: sum over the parties of x_q - a_q
    const uint64_t del = held(drelu - bs);                    // opened: sum of D_q - b_q
    const uint64_t b0_del = del + b[0];
    Shares<P> out;
    // party 0 takes the public term: c_0 + eps * b_0 + del * a_0 + eps * del
    out.v[0] = sum_of_products(c[0], eps, b0_del, del, a[0]);
#pragma unroll
    for (int q = 1; q < P - 1; ++q) out.v[q] = sum_of_products(c[q], eps, b[q], del, a[q]);
    // the last party's c completes the triple: c_{P-1} = a * b - (c_0 + ... + c_{P-2})
    out.v[P - 1] = sum_of_products(0 - cs, as, bs, eps, b[P - 1], del, a[P - 1]);
    return out;
}

template <int W, int P, int MODE, bool RUNS>
__global__ void __launch_bounds__(kBlock)
mp_group_kernel(const MpPointers ptr, uint64_t n, uint64_t groups, int k, uint64_t seedB, uint64_t seedA)
{
    using S = Shape<W>;
    using M = MpShape<W, P>;
    constexpr int L = M::L;
    const uint64_t g = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
    if (g >= groups) return;
    const uint64_t i0 = g * (uint64_t)L;
    const int cnt = (n - i0) >= (uint64_t)L ? L : (int)(n - i0);

    uint64_t u[P];
#pragma unroll
    for (int q = 0; q < P; ++q) u[q] = 0;
#pragma unroll
    for (int j = 0; j < L; ++j) {
        if (j < cnt) {
#pragma unroll
            for (int q = 0; q < P; ++q) u[q] |= ((load_stream(ptr.x[q] + i0 + j) >> k) & S::kField) << (j * W % 64);
        }
    }
    const uint64_t zg = seedB + (g * (uint64_t)M::kWordsPerGroup + 1) * kGamma;
    const Shares<P> sum = mp_a2b_sum<W, P, RUNS>(u, zg);
    const uint64_t wb = mix64(zg + (uint64_t)M::kB2aWord * kGamma);

#pragma unroll
    for (int j = 0; j < L; ++j) {
        if (j < cnt) {
            uint32_t sign = 0;
            Shares<P> x;
#pragma unroll
            for (int q = 0; q < P; ++q) {
                sign |= (uint32_t)((sum.v[q] >> (j * W + W - 1)) & 1) << q;
                x.v[q] = (MODE == kRelu) ? load_stream(ptr.x[q] + i0 + j) : 0;
            }
            const uint32_t rho = (uint32_t)(wb >> (P * j)) & ((1u << P) - 1);
            const uint64_t zA = seedA + ((uint64_t)M::kArithWords * (i0 + j) + 1) * kGamma;
            const B2aBits t{minus_bit((uint32_t)__popc(sign ^ rho), 0), (uint32_t)__popc(rho) & 1u};
            const Shares<P> out = mp_finish<P, MODE, RUNS>(t, x, zA);
#pragma unroll
            for (int q = 0; q < P; ++q) store_stream(ptr.o[q] + i0 + j, out.v[q]);
        }
    }
}

// Tile kernel among P parties: the owner / group-lane scheme of tile_body.  LDS per wavefront: P arrays of one entry (1, 2
// or 4 bytes) per element for the slices, and a byte {z, r} per element for the verdict, as Verdict's in the widths that are
// not packed.  (With sign shares and the B2A word published per group, an owner spent 14 instructions per element on
// finding and decoding them.)
template <int W, int P>
struct MpTileTraits {
    using M = MpShape<W, P>;
    static constexpr int L = M::L;
    static constexpr bool kSupported = (W <= 32);
    static constexpr int kGroups = (W >= 4) ? kWave : kWave / 2;   // half the lanes run the circuit when L > 16:
    static constexpr int kTile = kGroups * L;                      // a lane then owns at most 6 element pairs
    using Entry = typename std::conditional<(W <= 8), uint8_t,
                  typename std::conditional<(W <= 16), uint16_t, uint32_t>::type>::type;
    static constexpr bool kWordIsPacked = (int)sizeof(Entry) * 8 == W;   // the L entries of a group are its SWAR word
    static constexpr int slice_bytes(int groups) { return (groups * L * (int)sizeof(Entry) + 15) / 16 * 16; }   // per party
    static constexpr int verdict_bytes(int groups) { return (groups * L + 15) / 16 * 16; }
    static constexpr int kLdsBytes = P * slice_bytes(kGroups) + verdict_bytes(kGroups);
};

// A quarter of a tile: 16 groups, four lanes per group (QuarterTraits).  The words of one adder are exchanged at a time.
template <int W, int P>
struct MpQuarterTraits {
    using M = MpShape<W, P>;
    using T = MpTileTraits<W, P>;
    static constexpr int L = M::L;
    static constexpr int kSplit = 4, kGroups = kWave / kSplit, kTile = kGroups * L;
    static constexpr bool kHalves = (L % 2 == 0);
    using Word = typename std::conditional<kHalves, uint32_t, uint64_t>::type;
    static constexpr int kFields = kHalves ? L / 2 : L;
    static constexpr int kWords = 2 * M::R * M::kGateWords;        // evaluated words of an adder: all but the last P-update's
    static constexpr int kPad = (kWords + 1 + 3) / 4 * 4;          // and the B2A word, with the last adder's
    static constexpr int kRow = 2 * kPad + 4;                      // 32-bit units, an odd multiple of four
    static constexpr int kWordsAt = P * T::slice_bytes(kGroups), kVerdictAt = kWordsAt + kGroups * kRow * 4;
    static constexpr int kLdsBytes = kVerdictAt + T::verdict_bytes(kGroups);
};

template <int W, int P>
constexpr unsigned mp_lds_bytes(bool quarters)
{
    int most = MpTileTraits<W, P>::kLdsBytes;
    if constexpr (quarters_supported(W)) {
        if (quarters && MpQuarterTraits<W, P>::kLdsBytes > most) most = MpQuarterTraits<W, P>::kLdsBytes;
    }
    return (unsigned)(kWavesPerBlock * most);
}

// Owners' part before the circuit: pair c of a lane (of PAIRS, in a tile of TILE elements) from all parties, and its slices.
template <int P, int PAIRS, int TILE, bool FULL>
__device__ __forceinline__ void mp_load(const MpPointers &ptr, uint64_t tile0, uint64_t n, int lane, int c, U64x2 (&xs)[P][PAIRS])
{
    const unsigned e = 2 * (c * kWave + lane);
#pragma unroll
    for (int q = 0; q < P; ++q) xs[q][c] = U64x2{0, 0};
    if (e < (unsigned)TILE) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            const uint64_t *t = ptr.x[q] + tile0;       // scalar base, 32-bit lane offset
            if (FULL || tile0 + e + 1 < n) {
                xs[q][c] = load_stream2(t + e);
            } else if (tile0 + e < n) {
                xs[q][c].a = load_stream(t + e);
            }
        }
    }
}
template <int W, int P, int PAIRS, int TILE, int BYTES>
__device__ __forceinline__ void mp_deposit(unsigned char *lds, int k, int lane, int c, const U64x2 (&xs)[P][PAIRS])
{
    using S = Shape<W>;
    using Entry = typename MpTileTraits<W, P>::Entry;
    const unsigned e = 2 * (c * kWave + lane);
    if (e < (unsigned)TILE) {
#pragma unroll
        for (int q = 0; q < P; ++q) {
            Entry *sl = reinterpret_cast<Entry *>(lds + q * BYTES);
            sl[e] = (Entry)((xs[q][c].a >> k) & S::kField);
            sl[e + 1] = (Entry)((xs[q][c].b >> k) & S::kField);
        }
    }
}
// The FIELDS fields of word `slot` of one party's slices.
template <int W, int P, class Word, int FIELDS>
__device__ __forceinline__ Word mp_collect(const unsigned char *lds, int slot)
{
    using T = MpTileTraits<W, P>;
    if constexpr (T::kWordIsPacked) {
        return reinterpret_cast<const Word *>(lds)[slot];
    } else {
        const typename T::Entry *sl = reinterpret_cast<const typename T::Entry *>(lds) + slot * FIELDS;
        Word u = 0;
#pragma unroll
        for (int j = 0; j < FIELDS; ++j) u |= (Word)sl[j] << (j * W);
        return u;
    }
}
// {z, r} of the FIELDS fields of word `slot`.  wb: the group's B2A word with the first of these fields' P bits at 0.
template <int W, int P, class Word, int FIELDS>
__device__ __forceinline__ void mp_publish(unsigned char *verdict, int slot, const Shares<P, Word> &sum, uint64_t wb)
{
    Word sx = 0;
    uint64_t rx = 0, ones = 0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        sx ^= sum.v[q];
        rx ^= wb >> q;                                          // bit P j: r
    }
#pragma unroll
    for (int j = 0; j < FIELDS; ++j) ones |= 1ull << (P * j);
    const uint64_t rr = (rx & ones) | ((rx & ones) << 1);
    sx >>= W - 1;                                               // bit jW: XOR of the parties' sign shares
    using V = Verdict<5, kRelu>;
    auto byte = [&](int j) { return V::bit_at(sx, j * W) ^ V::template bits_at<2>(rr, P * j); };
    auto two = [&](int j) { return byte(j) | (byte(j + 1) << 8); };
    V::template store_bytes<FIELDS>(verdict + slot * FIELDS, byte, two);
}
// Owners' part after the circuit.
template <int P, int MODE, bool RUNS, int PAIRS, int TILE, bool FULL>
__device__ __forceinline__ void mp_finish_pairs(const MpPointers &ptr, uint64_t tile0, uint64_t n, int lane, uint64_t seedA,
                                                const U64x2 (&xs)[P][PAIRS], const unsigned char *verdict)
{
    constexpr uint64_t kArithWords = 4 * P - 2;
    // Four parties at w = 4 would hold 128 registers of shares, which the compiler puts into scratch memory and takes out again:
    // read a second time instead (a lane has stored nothing of its pair yet, so also where an output is an input).  1700 tiles
    // 39 us instead of 52, 2^25 elements 611 instead of 673.  With fewer shares to hold, three parties at w = 4 and four at w = 5,
    // the second reading costs more than the registers: 2^25 elements 342 / 443 and 626 / 677.
    constexpr bool kReload = MODE == kRelu && P * PAIRS >= 32;
    uint64_t zA0 = seedA + (kArithWords * (tile0 + 2 * (uint64_t)lane) + 1) * kGamma;
#pragma unroll
    for (int c = 0; c < PAIRS; ++c) {
        const int pr = c * kWave + lane;
        const unsigned e = 2 * pr;
        if (e < (unsigned)TILE) {
            const uint32_t v = reinterpret_cast<const uint16_t *>(verdict)[pr];
            U64x2 own[P];
            if constexpr (kReload) {
                U64x2 again[P][1];
                mp_load<P, 1, TILE, FULL>(ptr, tile0 + 2 * c * kWave, n, lane, 0, again);
#pragma unroll
                for (int q = 0; q < P; ++q) own[q] = again[q][0];
            } else {
#pragma unroll
                for (int q = 0; q < P; ++q) own[q] = xs[q][c];
            }
            Shares<P> r[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const B2aBits t{minus_bit(v, 8 * h), __builtin_amdgcn_ubfe(v, 8 * h + 1, 1)};
                Shares<P> x;
#pragma unroll
                for (int q = 0; q < P; ++q) x.v[q] = h ? own[q].b : own[q].a;
                r[h] = mp_finish<P, MODE, RUNS>(t, x, zA0 + kArithWords * (uint64_t)(2 * c * kWave + h) * kGamma);
                if constexpr (RUNS) settle(r[h].v);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) {
                uint64_t *t = ptr.o[q] + tile0;
                if (FULL || tile0 + e + 1 < n) {
                    store_stream2(t + e, U64x2{r[0].v[q], r[1].v[q]});
                } else if (tile0 + e < n) {
                    store_stream(t + e, r[0].v[q]);
                }
            }
            if constexpr (!RUNS) zA0 = not_before(zA0, r[1].v[P - 1]);               // one pair's dealer words at a time
        }
    }
}

// Work of one wavefront on wave-tile `tile` (uniform over the wavefront).  FULL: the whole tile lies inside the
// tensor, so no access needs a bounds check (every tile but the last).
template <int W, int P, int MODE, bool RUNS, bool FULL>
__device__ __forceinline__ void mp_tile_body(const MpPointers &ptr, uint64_t n, int k, uint64_t seedB, uint64_t seedA,
                                             uint64_t tile, int lane, unsigned char *lds)
{
    using M = MpShape<W, P>;
    using T = MpTileTraits<W, P>;
    constexpr int kPairs = (T::kTile / 2 + kWave - 1) / kWave, kBytes = T::slice_bytes(T::kGroups);
    const uint64_t tile0 = tile * T::kTile;
    unsigned char *verdict = lds + P * kBytes;

    priority<RUNS, kElsewhere>();
    U64x2 xs[P][kPairs];
#pragma unroll
    for (int c = 0; c < kPairs; ++c) {          // pair by pair: DReLU at w = 4 would hold 96 registers of shares at once
        mp_load<P, kPairs, T::kTile, FULL>(ptr, tile0, n, lane, c, xs);
        mp_deposit<W, P, kPairs, T::kTile, kBytes>(lds, k, lane, c, xs);
    }
    wave_sync();

    // ---- group lanes: collect the fields of group `lane`, run the adder tree, publish the verdict
    if (T::kGroups == kWave || lane < T::kGroups) {
        uint64_t u[P];
#pragma unroll
        for (int q = 0; q < P; ++q) u[q] = mp_collect<W, P, uint64_t, T::L>(lds + q * kBytes, lane);
        const uint64_t g = tile * T::kGroups + lane;
        const uint64_t zg = seedB + (g * (uint64_t)M::kWordsPerGroup + 1) * kGamma;
        const Shares<P> sum = mp_a2b_sum<W, P, RUNS>(u, zg);
        mp_publish<W, P, uint64_t, T::L>(verdict, lane, sum, mix64(zg + (uint64_t)M::kB2aWord * kGamma));
    }
    wave_sync();
    mp_finish_pairs<P, MODE, RUNS, kPairs, T::kTile, FULL>(ptr, tile0, n, lane, seedA, xs, verdict);
}

// The same on a quarter of a tile: about 1230 vector instructions per wavefront at w = 8 among three parties where the tile has
// 4250.  4,195,307 elements (8195 tiles: three after the last full round) take 72.6 us, with whole tiles only 76.6; at w = 4
// 53.5 and 63.8.
template <int W, int P, int MODE, bool RUNS, bool FULL>
__device__ __forceinline__ void mp_quarter_body(const MpPointers &ptr, uint64_t n, int k, uint64_t seedB, uint64_t seedA,
                                                uint64_t quarter, int lane, unsigned char *lds)
{
    using M = MpShape<W, P>;
    using T = MpTileTraits<W, P>;
    using Q = MpQuarterTraits<W, P>;
    using Word = typename Q::Word;
    constexpr int kPairs = (Q::kTile / 2 + kWave - 1) / kWave, kBytes = T::slice_bytes(Q::kGroups);
    const uint64_t tile0 = quarter * Q::kTile;
    unsigned char *verdict = lds + Q::kVerdictAt;
    priority<RUNS, kElsewhere>();
    U64x2 xs[P][kPairs];
#pragma unroll
    for (int c = 0; c < kPairs; ++c) mp_load<P, kPairs, Q::kTile, FULL>(ptr, tile0, n, lane, c, xs);

    const int grp = lane / Q::kSplit, sub = lane % Q::kSplit, half = sub % 2;
    const int slot = Q::kHalves ? 2 * grp + half : grp;
    const uint64_t g = quarter * Q::kGroups + grp;
    const uint64_t zs = seedB + (g * (uint64_t)M::kWordsPerGroup + 1 + (uint64_t)sub) * kGamma;
    uint32_t *row = reinterpret_cast<uint32_t *>(lds + Q::kWordsAt) + grp * Q::kRow;
    const int words_at = Q::kWordsAt + 4 * (grp * Q::kRow + (Q::kHalves ? half * Q::kPad : 0));

    auto put = [&](int j, uint64_t v, int upper) {
        if constexpr (Q::kHalves) {
            row[j] = (uint32_t)v;
            row[Q::kPad + j] = word_at(v, upper);
        } else {
            reinterpret_cast<uint64_t *>(row)[j] = v;
        }
    };
    // every lane draws its share of an adder's dealer words, and with the last adder's one of them the B2A word
    auto draw = [&](int adder) {
#pragma unroll
        for (int t = 0; t < (Q::kWords + Q::kSplit - 1) / Q::kSplit; ++t) {
            const int j = t * Q::kSplit + sub;
            if ((t + 1) * Q::kSplit <= Q::kWords || j < Q::kWords)
                put(j, mix64(zs + (uint64_t)(adder * M::kAdderWords + t * Q::kSplit) * kGamma), Q::kFields * W);
        }
        if (adder == P - 2 && sub == 3) put(Q::kWords, mix64(zs + (uint64_t)(M::kB2aWord - 3) * kGamma), P * Q::kFields);
    };
    draw(0);                                                   // while the loads are under way
#pragma unroll
    for (int c = 0; c < kPairs; ++c) mp_deposit<W, P, kPairs, Q::kTile, kBytes>(lds, k, lane, c, xs);
    wave_sync();

    Word u[P];
#pragma unroll
    for (int q = 0; q < P; ++q) u[q] = mp_collect<W, P, Word, Q::kFields>(lds + q * kBytes, slot);
    auto add = [&](int i, const Shares<P, Word> &X, const Shares<P, Word> &Y) {
        if (i > 0) {
            wave_sync();                                       // the adder before has read its words
            draw(i);
            wave_sync();
        }
        // one gate's words in registers at a time: read ahead, those of a whole adder would halve the kernel's occupancy
        auto gate = [&](int q, Word after) {
            int at = words_at;
            asm("" : "+v"(at) : "v"(after));
            const Word *words = reinterpret_cast<const Word *>(__builtin_assume_aligned(lds + at, 16)) + q * M::kGateWords;
            return [words](int w) { return words[w]; };
        };
        return mp_add_gates<W, P, Word, false>(gate, X, Y);
    };
    const Shares<P, Word> sum = mp_tree<P, Word>(u, add);
    if (sub < (Q::kHalves ? 2 : 1))
        mp_publish<W, P, Word, Q::kFields>(verdict, slot, sum, reinterpret_cast<const Word *>(lds + words_at)[Q::kWords]);
    wave_sync();
    mp_finish_pairs<P, MODE, RUNS, kPairs, Q::kTile, FULL>(ptr, tile0, n, lane, seedA, xs, verdict);
}

template <int W, int P, int MODE, int FORM>
__global__ void __launch_bounds__(kBlock)
mp_tile_kernel(const MpPointers ptr, uint64_t n, int k, uint64_t seedB, uint64_t seedA, uint32_t whole_blocks)
{
    using T = MpTileTraits<W, P>;
    static_assert(T::kSupported, "tile kernel needs W <= 32");
    extern __shared__ __attribute__((aligned(16))) unsigned char tile_lds[];
    const int lane = threadIdx.x % kWave, wv = wave_index();
    const TileWork t = tile_work<has_quarters(FORM)>(whole_blocks, wv);
    if (t.tile * T::kTile >= n) return;        // whole wavefront beyond the tensor
    constexpr bool RUNS = has_runs(FORM);
    if constexpr (has_quarters(FORM)) {
        if (t.quarter >= 0) {
            using Q = MpQuarterTraits<W, P>;
            const uint64_t quarter = t.tile * Q::kSplit + (unsigned)t.quarter;
            unsigned char *lds = tile_lds + wv * Q::kLdsBytes;
            if ((quarter + 1) * Q::kTile <= n)
                mp_quarter_body<W, P, MODE, RUNS, true>(ptr, n, k, seedB, seedA, quarter, lane, lds);
            else if (quarter * Q::kTile < n)
                mp_quarter_body<W, P, MODE, RUNS, false>(ptr, n, k, seedB, seedA, quarter, lane, lds);
            return;
        }
    }
    unsigned char *lds = tile_lds + wv * T::kLdsBytes;
    if ((t.tile + 1) * T::kTile <= n)
        mp_tile_body<W, P, MODE, RUNS, true>(ptr, n, k, seedB, seedA, t.tile, lane, lds);
    else
        mp_tile_body<W, P, MODE, RUNS, false>(ptr, n, k, seedB, seedA, t.tile, lane, lds);
}

}  // namespace hb
