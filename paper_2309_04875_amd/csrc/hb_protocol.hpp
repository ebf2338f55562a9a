// Device-side statement of the protocol, in SWAR form: L = min(64/W, 32) elements share one 64-bit word,
// element j of a group occupying bits [jW, jW+W).  Every step below is bitwise, so the L fields never
// interact except through shifts, which are confined to their field by a mask.
//
// Paper: Sec. 2.2 "Evaluating ReLU with GMW" (A2B adder on XOR shares, Beaver AND, sign, B2A),
// Eq. 3 (DReLU on the slice only), Sec. 4.2 (depth ceil(log2 w), packing of w-bit fields in 64-bit words).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hb {

// ---- dealer streams: SplitMix64, output j of a generator started at state s is mix(s + (j+1)*gamma)
constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;

__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__host__ __device__ __forceinline__ uint64_t stream_word(uint64_t s, uint64_t j)
{
    return mix64(s + (j + 1) * kGamma);
}

// ---- compile-time shape of the circuit for slice width W
constexpr int ceil_log2(int w)
{
    int r = 0;
    while ((1 << r) < w) ++r;
    return r;
}

template <int W>
struct Shape {
    static_assert(W >= 1 && W <= 64, "slice width");
    static constexpr int w = W;
    static constexpr int R = ceil_log2(W);                     // prefix rounds (0 when W == 1)
    static constexpr int L = (64 / W) > 32 ? 32 : (64 / W);     // fields per word
    static constexpr int kGates = 1 + 2 * R;                    // gate 0 + two per round

    // Dealer words of one group.  Standard layout: five triple words (a_0 a_1 b_0 b_1 c_0) per gate, then the
    // B2A word.  Shared-mask layout: gate 0 as before; a prefix round owns eight words, a_0 a_1 (the one mask of
    // P that both of its gates use), b_0 b_1 c_0 of the G-update and b_0 b_1 c_0 of the P-update; then the B2A word.
    static constexpr int round_word(bool shared, int r) { return shared ? 5 + 8 * r : 5 * (1 + 2 * r); }
    static constexpr int b2a_word(bool shared) { return round_word(shared, R); }
    static constexpr int words_per_group(bool shared) { return b2a_word(shared) + 1; }
    static constexpr uint64_t kField = (W == 64) ? ~0ull : ((1ull << (W & 63)) - 1);

    // bit 0 of every field
    static constexpr uint64_t ones()
    {
        uint64_t r = 0;
        for (int j = 0; j < L; ++j) r |= 1ull << (j * W);
        return r;
    }
    // positions of a word that still hold data of their own field after a left shift by s
    static constexpr uint64_t keep(int s)
    {
        uint64_t f = (s >= W) ? 0 : ((kField << s) & kField);
        uint64_t r = 0;
        for (int j = 0; j < L; ++j) r |= f << (j * W);
        return r;
    }
};

// The gate logic is bitwise, so it runs on whole words or on a half of one (Word = uint64_t or uint32_t).
template <class Word>
struct WordPair {    // one value held as (party 0 share, party 1 share)
    Word p0, p1;
};

using Pair = WordPair<uint64_t>;

// ---- dealer words, several at a time ---------------------------------------------------------------------------------
// What bounds every kernel here is vector-ALU issue, and three quarters of it are SplitMix64.  A third of its
// instructions, the 32-bit xors, take two cycles of a SIMD instead of four, but only while two of its wavefronts are at such
// instructions at the same time; left to themselves the wavefronts are spread evenly over the generator and pay four for nearly
// every instruction (3.9 on average).  With RUNS the words that a gate or an element needs are drawn in step, the xors of all of
// them in one run, and a wavefront gives way (lowest wave priority) while it is in such a run: the others then use the SIMD for
// their multiplies until they too stand before xors, which are issued two at a time.  Words alone, four wavefronts per
// SIMD, five or ten words in step: 72 cycles a word without priorities whatever the order of the instructions, 61 and 58
// with them, 72 with the priorities the other way round.  One wavefront per SIMD has nobody to share with, and the changes of
// priority cost it 1 to 5 %, so kernels exist with RUNS and without.
// The lowest priority is also the one that kernels without RUNS, and everyone else's, run at: beside a ReLU on another stream they
// get fewer issue slots.  Both on one GPU at a time, us a launch, form before / with RUNS: ReLU at w = 8 (2^24 elements) 211 / 203 and a
// DReLU of as many beside it 133 / 140, a bf16 product of 4096^3 225 / 218, an addition of 2^26 floats 228 / 227; beside ReLU at w = 64 (2^22
// elements) 240 / 129, 257 / 243, 271 / 252.
constexpr int kXorRuns = 0, kElsewhere = 1;        // wave priorities

template <bool RUNS, int PRIORITY>
__device__ __forceinline__ void priority()
{
    if constexpr (RUNS) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(PRIORITY);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The values are computed before, and their uses come after, whatever else has this order (priority() does).  No instruction.
template <class Word>
__device__ __forceinline__ void settle(Word &v) { asm volatile("" : "+v"(v)); }
template <class Word, int N>
__device__ __forceinline__ void settle(Word (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i) settle(v[i]);
}
__device__ __forceinline__ void settle(Pair &v)
{
    settle(v.p0);
    settle(v.p1);
}

// Returns z, which the compiler may not compute before `after` is known.  Dealer words depend only on the group
// or element number, so the scheduler would otherwise generate those of every gate ahead of the circuit and
// hold them all in registers; tying a gate's generator state to the previous gate's result keeps their live
// ranges one gate long.  Emits no instruction.
__device__ __forceinline__ uint64_t not_before(uint64_t z, uint64_t after)
{
    asm("" : "+v"(z) : "v"(after));
    return z;
}

// kGamma in scalar registers, as a value that the compiler does not fold into others: consecutive states are one addition
// each, from one register pair, instead of an addition of a constant that two scalar moves make each time.
__device__ __forceinline__ uint64_t gamma()
{
    uint64_t g = kGamma;
    asm("" : "+s"(g));
    return g;
}

template <int N>
__device__ __forceinline__ void xor_shift(uint64_t (&z)[N], int by)
{
    uint64_t t[N];
#pragma unroll
    for (int i = 0; i < N; ++i) t[i] = z[i] >> by;
    settle(t);
    priority<true, kXorRuns>();
#pragma unroll
    for (int i = 0; i < N; ++i) z[i] ^= t[i];
}
// mix64 of N states.  With RUNS it starts at priority kElsewhere (the states have been computed there) and ends at
// kXorRuns, where the xors that use the words go on; whoever goes on with something else raises it again.
template <bool RUNS, int N>
__device__ __forceinline__ void mix_words(uint64_t (&z)[N])
{
    if constexpr (RUNS) {
        xor_shift(z, 30);
        settle(z);
        priority<true, kElsewhere>();
#pragma unroll
        for (int i = 0; i < N; ++i) z[i] *= 0xBF58476D1CE4E5B9ull;
        xor_shift(z, 27);
        settle(z);
        priority<true, kElsewhere>();
#pragma unroll
        for (int i = 0; i < N; ++i) z[i] *= 0x94D049BB133111EBull;
        xor_shift(z, 31);
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) z[i] = mix64(z[i]);
    }
}

// The next N words of the generator whose next word has state z, which moves on, then (EXTRA = 1) one that lies `skip` words
// further.
template <bool RUNS, int N, int EXTRA = 0>
__device__ __forceinline__ void draw_words(uint64_t &z, uint64_t (&v)[N + EXTRA], int skip = 0)
{
    if constexpr (RUNS) {
        settle(z);
        priority<true, kElsewhere>();
#pragma unroll
        for (int i = 0; i < N; ++i) {
            v[i] = z;
            z += gamma();
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = z + (uint64_t)i * kGamma;
        z += (uint64_t)N * kGamma;
    }
    if constexpr (EXTRA != 0) v[N] = z + (uint64_t)skip * kGamma;
    mix_words<RUNS>(v);
}

// ---- three-input bitwise operations (v_bitop3_b32, one instruction per 32-bit half) ----------------------------
// The 8-bit truth table of a boolean function f(a, b, c), in the instruction's operand order.
constexpr unsigned kTtXor3 = (0xF0 ^ 0xCC ^ 0xAA) & 0xFF;              // a ^ b ^ c
constexpr unsigned kTtXorAnd = (0xF0 ^ (0xCC & 0xAA)) & 0xFF;          // a ^ (b & c)
constexpr unsigned kTtAndXor = (0xF0 & (0xCC ^ 0xAA)) & 0xFF;          // a & (b ^ c)

template <unsigned TT>
__device__ __forceinline__ uint32_t bitop3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, TT);
}
template <unsigned TT>
__device__ __forceinline__ uint64_t bitop3(uint64_t a, uint64_t b, uint64_t c)
{
    const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)a, (uint32_t)b, (uint32_t)c, TT);
    const uint32_t hi = __builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), (uint32_t)(b >> 32), (uint32_t)(c >> 32), TT);
    return ((uint64_t)hi << 32) | lo;
}

// ---- shifts of 64-bit values by an amount that differs between lanes ---------------------------------------------
// No kernel has the 64-bit shift instruction with its amount in a vector register: where that was the last vector register
// of a wavefront's allocation (v63 of 64, the DReLU kernel of w = 10), whole wavefronts got wrong results now and then, and
// the compiler does not keep the amount from there.  That this instruction was the cause is inferred: of the kernels run
// against the oracle only the one with that assignment failed, and without the instruction it no longer did.  The built
// library is searched for the form by a test.

// Bits at .. at + 31 of v, 0 <= at <= 32.
__device__ __forceinline__ uint32_t word_at(uint64_t v, int at)
{
    const uint32_t low = __builtin_amdgcn_alignbit((uint32_t)(v >> 32), (uint32_t)v, (uint32_t)at);
    return at >= 32 ? (uint32_t)(v >> 32) : low;
}
// The lowest `count` bits set, 0 <= count < 64.
__device__ __forceinline__ uint64_t low_bits(int count)
{
    const uint32_t part = (1u << (count & 31)) - 1;
    return count < 32 ? part : ((uint64_t)part << 32) | 0xffffffffu;
}

template <class Word>
struct GateWords {   // the five dealer words of one AND gate, in stream order
    Word a0, a1, b0, b1, c0;
};

// One Beaver AND on XOR-shared words, Z = U & V, returned as acc ^ Z share by share (acc = {0, 0} for the
// plain gate; the G-update of a prefix round passes the old G).  U is masked by a, V by b.
// The gate sees U and V only through the two openings, and an opening is the XOR of what the two parties
// send, (U_0 ^ a_0) ^ (U_1 ^ a_1) = (U_0 ^ U_1) ^ (a_0 ^ a_1); the caller passes Ux = U_0 ^ U_1 and
// Vx = (V_0 ^ V_1) before the field mask `keep` that confines a shifted operand to its field (all ones when
// the operand is not shifted).  Party 0 takes the public d & e term.
template <class Word>
__device__ __forceinline__ WordPair<Word> beaver_and_words(const GateWords<Word> &t, Word Ux, Word Vx, Word keep, WordPair<Word> acc)
{
    const Word a0 = t.a0, a1 = t.a1, b0 = t.b0, b1 = t.b1, c0 = t.c0;
    const Word a = a0 ^ a1, b = b0 ^ b1;                        // the dealer's triple (a, b, a & b)
    const Word d = Ux ^ a;                                      // opened
    const Word e = bitop3<kTtXorAnd>(b, Vx, keep);              // opened: (Vx & keep) ^ b
    WordPair<Word> Z;
    // party 0: acc ^ c_0 ^ (e & a_0) ^ (d & (b_0 ^ e))    [= c_0 ^ (d & b_0) ^ (e & a_0) ^ (d & e)]
    Z.p0 = bitop3<kTtXor3>(acc.p0, bitop3<kTtXorAnd>(c0, e, a0), bitop3<kTtAndXor>(d, b0, e));
    // party 1: acc ^ c_1 ^ (d & b_1) ^ (e & a_1), the dealer having completed c_1 = (a & b) ^ c_0
    const Word c1 = bitop3<kTtXorAnd>(c0, a, b);
    Z.p1 = bitop3<kTtXorAnd>(bitop3<kTtXorAnd>(acc.p1 ^ c1, d, b1), e, a1);
    return Z;
}

// A2B + sign for one group.  u0/u1: the L sliced shares of party 0 / party 1 packed as fields.
// z: generator state of the group's first dealer word.  Returns XOR shares of the sum word
// S ^ (G << 1); the sign of field j is bit jW + W - 1.  The last round's P-update gate is not
// evaluated: nothing reads its result (its dealer words are simply never drawn).  SHARED selects the
// dealer layout in which the two gates of a round share the mask of P: eight words a_0 a_1 | b_0 b_1 c_0 of the G-update |
// b_0 b_1 c_0 of the P-update, of which the last round leaves three undrawn.  B2A: the group's B2A word is drawn with the last gate's and left in `b2a`.
// A gate's words are used up before the next are drawn.  (Ten words in step, those of a round, take 16 registers more, which
// costs a wavefront per SIMD at most widths: w = 8 and 10 as fast, w = 16 6 % slower.)
template <int W, bool SHARED, bool B2A, bool RUNS>
__device__ __forceinline__ Pair a2b_sum(uint64_t u0, uint64_t u1, uint64_t z, uint64_t &b2a)
{
    using S = Shape<W>;
    using GW = GateWords<uint64_t>;
    auto gate = [&] {
        uint64_t v[5];
        draw_words<RUNS, 5>(z, v);
        return GW{v[0], v[1], v[2], v[3], v[4]};
    };
    // the five words of the circuit's last gate, and the B2A word, which lies `skip` words behind them
    auto last_gate = [&](int skip) {
        uint64_t v[B2A ? 6 : 5];
        draw_words<RUNS, 5, B2A ? 1 : 0>(z, v, skip);
        if constexpr (B2A) b2a = v[5];
        return GW{v[0], v[1], v[2], v[3], v[4]};
    };
    // X = (u0, 0), Y = (0, u1): each party XOR-shares its own slice trivially
    const Pair X{u0, 0}, Y{0, u1};
    Pair P{X.p0 ^ Y.p0, X.p1 ^ Y.p1};
    const Pair Sum = P;
    Pair G = beaver_and_words<uint64_t>(S::R == 0 ? last_gate(0) : gate(), X.p0 ^ X.p1, Y.p0 ^ Y.p1, ~0ull, Pair{0, 0});
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        const int s = 1 << r;
        const bool last = r + 1 == S::R;
        const uint64_t keep = S::keep(s);
        // shifting is linear: the XOR of the parties' shifted shares is the shifted XOR of their shares
        const uint64_t Px = P.p0 ^ P.p1;
        const uint64_t Gsx = (G.p0 ^ G.p1) << s, Psx = Px << s;
        if constexpr (RUNS) {
            settle(G);
            if (!(last && W >= 34)) settle(P);             // (a last round on one field reads the upper half only)
        } else {
            z = not_before(z, G.p0);
        }
        if (last) {
            G = beaver_and_words<uint64_t>(last_gate(SHARED ? 3 : 5), Px, Gsx, keep, G);
        } else if constexpr (SHARED) {
            const GW g = gate();
            G = beaver_and_words<uint64_t>(g, Px, Gsx, keep, G);
            if constexpr (RUNS) settle(G);
            uint64_t v[3];
            draw_words<RUNS, 3>(z, v);
            P = beaver_and_words<uint64_t>(GW{g.a0, g.a1, v[0], v[1], v[2]}, Px, Psx, keep, Pair{0, 0});
        } else {
            G = beaver_and_words<uint64_t>(gate(), Px, Gsx, keep, G);
            if constexpr (RUNS) settle(G);
            P = beaver_and_words<uint64_t>(gate(), Px, Psx, keep, Pair{0, 0});
        }
    }
    const uint64_t keep1 = S::keep(1);
    return Pair{Sum.p0 ^ ((G.p0 << 1) & keep1), Sum.p1 ^ ((G.p1 << 1) & keep1)};
}

// The same circuit on dealer words that were generated elsewhere: words[i] is word i of the group (those of the last
// round's P-update gate, which is not evaluated, are not there).  Word = uint32_t: the lower or the upper half of the
// fields, at bits jW of u0, u1 and of every word; S::keep is the same for both.
template <int W, bool SHARED, class Word>
__device__ __forceinline__ WordPair<Word> a2b_sum_words(Word u0, Word u1, const Word *words)
{
    using S = Shape<W>;
    using WP = WordPair<Word>;
    auto gate = [&](int a, int b) { return GateWords<Word>{words[a], words[a + 1], words[b], words[b + 1], words[b + 2]}; };
    const WP X{u0, 0}, Y{0, u1};
    WP P{X.p0 ^ Y.p0, X.p1 ^ Y.p1};
    const WP Sum = P;
    WP G = beaver_and_words<Word>(gate(0, 2), X.p0 ^ X.p1, Y.p0 ^ Y.p1, (Word)~0ull, WP{0, 0});
#pragma unroll
    for (int r = 0; r < S::R; ++r) {
        const int s = 1 << r, w = S::round_word(SHARED, r);
        const Word keep = (Word)S::keep(s);
        const Word Px = P.p0 ^ P.p1;
        const Word Gsx = (G.p0 ^ G.p1) << s, Psx = Px << s;
        G = beaver_and_words<Word>(gate(w, w + 2), Px, Gsx, keep, G);
        if (r + 1 < S::R) P = beaver_and_words<Word>(SHARED ? gate(w, w + 5) : gate(w + 5, w + 7), Px, Psx, keep, WP{0, 0});
    }
    const Word keep1 = (Word)S::keep(1);
    return WP{Sum.p0 ^ ((G.p0 << 1) & keep1), Sum.p1 ^ ((G.p1 << 1) & keep1)};
}

// What an element keeps of its group's verdict: the opened bit z = sign_0 ^ rho_0 ^ sign_1 ^ rho_1 of the B2A, as
// m = -z (0 or all ones), and the dealer's bit r = rho_0 ^ rho_1 (0 or 1).
struct B2aBits {
    int32_t m;
    uint32_t r;
};

// Keeps the compiler from reasoning about a value (a carry chain it would narrow, a sum it would cancel); no instruction.
__device__ __forceinline__ uint64_t held(uint64_t v)
{
    asm("" : "+v"(v));
    return v;
}

// bit `at` of v as B2aBits::m
__device__ __forceinline__ int32_t minus_bit(uint32_t v, int at) { return (int32_t)__builtin_amdgcn_sbfe((int)v, at, 1); }

// B2A of the sign bit and 1 - sign, for one element.  zA: generator state of the element's first arithmetic word
// A[6i] = r^A_0; r^A_1 = r - r^A_0.  sign = z ^ r = z + r - 2zr and party 0 adds the public z, so
//   DReLU_0 = 1 - beta_0 = z ? r^A_0 : 1 - r^A_0,   DReLU_1 = -beta_1 = z ? r^A_1 : -r^A_1.
// A vector instruction costs four SIMD cycles whatever it does, a 64-bit add is one, a subtract, a select or an xor
// two.  -v = ~v + 1 turns the conditional negations into xors with m; with c = ~r^A_0 (the complement is free: the
// generator's last xor becomes an xnor) and q = r^A_1 - 1 = c + r,
//   DReLU_0 = (c ^ m) + 2 (1 - z),   DReLU_1 = ~(q ^ m) + z.
// With the verdict published as (z, r) pairs the w = 8 ReLU tile was 1986 vector instructions per wavefront where selects
// and subtracts on separately shifted sign shares and dealer bits took 2060: 285,212,672 elements in 2.175 ms against
// 2.227, the simulator's 4,194,304 in 34.7 us against 35.6.
struct B2aShares {
    uint64_t f0, f1;    // DReLU_0 less 2 (1 - z), DReLU_1 less z
};
// c: the complement of the element's word r^A_0, held (the compiler would make a subtraction of ~r^A_0 + r); f0: c ^ m.
__device__ __forceinline__ uint64_t b2a_first(B2aBits t, uint64_t c) { return held(c ^ (uint64_t)(int64_t)t.m); }
__device__ __forceinline__ B2aShares b2a_shares(B2aBits t, uint64_t c, uint64_t f0)
{
    const uint64_t q = c + t.r;
    return B2aShares{f0, held(~(q ^ (uint64_t)(int64_t)t.m))};
}
__device__ __forceinline__ Pair b2a_drelu(B2aBits t, B2aShares f)
{
    return Pair{f.f0 + (uint32_t)(2 * (t.m + 1)), f.f1 + (uint32_t)-t.m};
}

// ---- products on Z_2^64 out of 32-bit halves --------------------------------------------------------------------
// x * y mod 2^64 = lo(x) lo(y) + 2^32 (lo(x) hi(y) + hi(x) lo(y)).  v_mad_u64_u32 (32 x 32 + 64 -> 64) adds while it
// multiplies, so a sum of products costs one instruction per 32 x 32 product plus one final add when the cross
// products are accumulated in a 64-bit register of their own, of which only the low half is used.  held() keeps
// that register whole: without it the compiler narrows the chain to 32-bit multiplies followed by separate adds.
__device__ __forceinline__ uint64_t lo32(uint64_t v) { return (uint32_t)v; }
__device__ __forceinline__ uint64_t hi32(uint64_t v) { return v >> 32; }
// low + 2^32 * cross, touching only the high half of `low`
__device__ __forceinline__ uint64_t add_to_high(uint64_t low, uint64_t cross)
{
    uint32_t h = (uint32_t)(low >> 32) + (uint32_t)cross;
    asm("" : "+v"(h));      // keeps the sum a 32-bit add (otherwise it is widened to a 64-bit add of {0, cross})
    return ((uint64_t)h << 32) | (uint32_t)low;
}

// acc + x * y (+ u * v) (+ s * t)  mod 2^64
__device__ __forceinline__ uint64_t sum_of_products(uint64_t acc, uint64_t x, uint64_t y, uint64_t u, uint64_t v)
{
    uint64_t cross = held(lo32(x) * hi32(y));
    cross = held(hi32(x) * lo32(y) + cross);
    cross = held(lo32(u) * hi32(v) + cross);
    cross = held(hi32(u) * lo32(v) + cross);
    const uint64_t low = lo32(u) * lo32(v) + (lo32(x) * lo32(y) + acc);
    return add_to_high(held(low), cross);
}
__device__ __forceinline__ uint64_t sum_of_products(uint64_t acc, uint64_t x, uint64_t y, uint64_t u, uint64_t v,
                                                    uint64_t s, uint64_t t)
{
    uint64_t cross = held(lo32(x) * hi32(y));
    cross = held(hi32(x) * lo32(y) + cross);
    cross = held(lo32(u) * hi32(v) + cross);
    cross = held(hi32(u) * lo32(v) + cross);
    cross = held(lo32(s) * hi32(t) + cross);
    cross = held(hi32(s) * lo32(t) + cross);
    const uint64_t low = lo32(s) * lo32(t) + (lo32(u) * lo32(v) + (lo32(x) * lo32(y) + acc));
    return add_to_high(held(low), cross);
}

// Beaver multiply x * DReLU on Z_2^64 for one element; v: its triple A[6i+1 .. 6i+5].
__device__ __forceinline__ Pair b2a_mul(B2aBits t, B2aShares f, Pair x, const uint64_t *v)
{
    const uint64_t a0 = v[0], a1 = v[1], b0 = v[2], b1 = v[3], c0 = v[4];
    const uint64_t a = a0 + a1, b = b0 + b1;                      // the dealer's triple (a, b, a * b)
    const uint64_t eps = (x.p0 + x.p1) - a;                       // opened: (x_0 - a_0) + (x_1 - a_1)
    // opened: (DReLU_0 - b_0) + (DReLU_1 - b_1).  Party 0 needs b_0 + del besides: an addition, where that first and del out
    // of it are two subtractions (two instructions each, the second waiting for the first's carry).
    const uint64_t del = held(held((f.f0 + f.f1) + (uint32_t)(t.m + 2)) - b);
    const uint64_t b0_del = del + b0;
    Pair out;
    // party 0: c_0 + eps * b_0 + del * a_0 + eps * del
    out.p0 = sum_of_products(c0, eps, b0_del, del, a0);
    // party 1: c_1 + eps * b_1 + del * a_1, the dealer having completed c_1 = a * b - c_0
    out.p1 = sum_of_products(0 - c0, a, b, eps, b1, del, a1);
    return out;
}

// What a launch computes.  The two last modes run the same operation on the shared-mask dealer layout.
enum Mode { kDrelu = 0, kRelu = 1, kSign = 2, kDreluShared = 3, kReluShared = 4, kModes = 5 };

constexpr int op_of(int mode) { return mode >= kDreluShared ? mode - kDreluShared : mode; }
constexpr bool shared_of(int mode) { return mode >= kDreluShared; }

// Everything after the circuit for COUNT consecutive elements: B2A, multiply.  z: generator state of the first element's
// word A[6i].
template <int MODE, bool RUNS, int COUNT>
__device__ __forceinline__ void finish_elements(const B2aBits (&t)[COUNT], const Pair (&x)[COUNT], uint64_t z, Pair *out)
{
    constexpr bool kMul = op_of(MODE) == kRelu;
    constexpr int kWords = kMul ? 6 : 1;                          // of an element; DReLU reads the first only
    if constexpr (!RUNS) {
        // One element after the other, r^A_0 first: this is the order in which a wavefront that is alone on its SIMD waits least
        // (all words first: the simulator at w = 12 and 1050 tiles 7.5 us instead of 7.2, ReLU at w = 7 and 200 tiles 6.2 / 6.0).
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            const uint64_t zi = z + (uint64_t)(6 * i) * kGamma;
            const uint64_t c = held(~mix64(zi));
            const B2aShares f = b2a_shares(t[i], c, b2a_first(t[i], c));
            if constexpr (kMul) {
                uint64_t v[5];
#pragma unroll
                for (int j = 0; j < 5; ++j) v[j] = mix64(zi + (uint64_t)(j + 1) * kGamma);
                out[i] = b2a_mul(t[i], f, x[i], v);
            } else {
                out[i] = b2a_drelu(t[i], f);
            }
        }
    } else {
        uint64_t v[kWords * COUNT], c[COUNT], f0[COUNT];
        if constexpr (kMul) {
            draw_words<true, kWords * COUNT>(z, v);
        } else {
            priority<true, kElsewhere>();
#pragma unroll
            for (int i = 0; i < COUNT; ++i) v[i] = z + (uint64_t)(6 * i) * kGamma;
            mix_words<true>(v);
        }
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            c[i] = held(~v[kWords * i]);
            f0[i] = b2a_first(t[i], c[i]);
        }
        if constexpr (kMul) settle(v);
        settle(c);
        settle(f0);
        priority<true, kElsewhere>();
#pragma unroll
        for (int i = 0; i < COUNT; ++i) {
            const B2aShares f = b2a_shares(t[i], c[i], f0[i]);
            if constexpr (kMul) out[i] = b2a_mul(t[i], f, x[i], v + kWords * i + 1);
            else out[i] = b2a_drelu(t[i], f);
            settle(out[i]);
        }
    }
}

// Everything after the circuit for element j of a group: pick the element's sign and dealer bits
// out of the group words, B2A, multiply.  z as in finish_elements.
template <int W, int MODE, bool RUNS>
__device__ __forceinline__ Pair finish_element(Pair sum, uint64_t wb, int j, Pair x, uint64_t z)
{
    const int sb = j * W + W - 1;
    if (op_of(MODE) == kSign) return Pair{(sum.p0 >> sb) & 1, (sum.p1 >> sb) & 1};
    const uint32_t r = (uint32_t)((wb ^ (wb >> 1)) >> (2 * j)) & 1u;
    const B2aBits t{minus_bit((uint32_t)((sum.p0 ^ sum.p1) >> sb) ^ r, 0), r};
    Pair out;
    finish_elements<MODE, RUNS, 1>({t}, {x}, z, &out);
    return out;
}

}  // namespace hb
