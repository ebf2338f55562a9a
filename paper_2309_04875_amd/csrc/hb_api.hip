// C ABI of the library (include/hb.h): argument checks on the host, closed-form opened-bit counts,
// kernel selection by slice width, launch on the caller's stream.  No allocation, no synchronisation.
#include "../../include/hb.h"

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <exception>
#include <new>
#include <utility>
#include <vector>

#include "hb_eco.hpp"
#include "hb_float.hpp"
#include "hb_kernels.hpp"
#include "hb_launch.hpp"
#include "hb_multiparty.hpp"
#include "hb_party.hpp"

namespace {

thread_local char g_hip_error[256] = "";

int fail_hip(hipError_t e, const char *what)
{
    std::snprintf(g_hip_error, sizeof(g_hip_error), "%s: %s", what, hipGetErrorString(e));
    (void)hipGetLastError();
    return HB_EHIP;
}

// No C++ exception leaves an entry point: what can throw here is the host memory of a set's launches.
template <class Body>
int no_throw(const Body &body)
{
    try {
        return body();
    } catch (const std::exception &) {
        return fail_hip(hipErrorOutOfMemory, "host memory");
    }
}

bool valid_slice(int k, int m) { return k >= 0 && m > k && m <= 64; }

int rounds_of(int w) { return hb::ceil_log2(w); }

struct Range {
    uintptr_t lo, hi;
};

Range range_of(const void *p, size_t n) { return Range{(uintptr_t)p, (uintptr_t)p + n * sizeof(int64_t)}; }

bool same(Range a, Range b) { return a.lo == b.lo; }
bool disjoint(Range a, Range b) { return a.hi <= b.lo || b.hi <= a.lo; }

// Allocations that the checks of ONE call have found to be this GPU's memory.  The buffers of a call mostly lie in a few
// allocations (a framework's allocator cuts many tensors out of one), and two queries of the HIP runtime for each of them
// were 0.2 us a buffer: 0.8 us of a call on one tensor, 12 us of one on 17.  Nothing is kept after the call.
struct KnownAllocations {
    static constexpr int kMost = 16;
    Range at[kMost];
    unsigned found = 0;                  // the newest kMost are kept
    int device = -1;                     // current device, once asked for
};

// The buffer must be memory the GPU can address, and [p, p + bytes) must lie inside one allocation.
int check_device_bytes(const void *p, size_t bytes, KnownAllocations &known)
{
    const Range r{(uintptr_t)p, (uintptr_t)p + bytes};
    for (unsigned i = 0; i < known.found && i < (unsigned)KnownAllocations::kMost; ++i) {
        const Range &a = known.at[i];
        if (r.lo >= a.lo && r.lo < a.hi) return r.hi <= a.hi ? HB_OK : HB_EINVAL;
    }
    hipPointerAttribute_t attr;
    hipError_t e = hipPointerGetAttributes(&attr, p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return HB_EINVAL;  // not known to the HIP runtime: plain host memory or a wild pointer
    }
    switch (attr.type) {
    case hipMemoryTypeDevice:     // memory of another GPU is not addressable from the kernels launched here
        if ((known.device < 0 && hipGetDevice(&known.device) != hipSuccess) || attr.device != known.device) {
            (void)hipGetLastError();
            return HB_EINVAL;
        }
        break;
    case hipMemoryTypeManaged:
        break;
    case hipMemoryTypeHost:  // pinned host memory is usable only through its device-side address
        if (attr.devicePointer != p) return HB_EINVAL;
        break;
    default:  // unregistered host memory, arrays
        return HB_EINVAL;
    }
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    e = hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return HB_OK;  // allocation kinds without a queryable range: the attribute check has passed
    }
    const Range a{(uintptr_t)base, (uintptr_t)base + size};
    if (attr.type == hipMemoryTypeDevice) known.at[known.found++ % KnownAllocations::kMost] = a;
    return (r.lo >= a.lo && r.hi <= a.hi) ? HB_OK : HB_EINVAL;
}

int check_device_buffer(const void *p, size_t n, KnownAllocations &known) { return check_device_bytes(p, n * sizeof(int64_t), known); }

int check_common(const void *const *ptrs, int count, size_t n, KnownAllocations &known)
{
    if (n > HB_MAX_ELEMENTS) return HB_EINVAL;
    if (n == 0) return HB_OK;
    for (int i = 0; i < count; ++i) {
        if (ptrs[i] == nullptr) return HB_EINVAL;
    }
    for (int i = 0; i < count; ++i) {
        if (((uintptr_t)ptrs[i] & 7u) != 0) return HB_EALIGN;
    }
    for (int i = 0; i < count; ++i) {
        const int st = check_device_buffer(ptrs[i], n, known);
        if (st != HB_OK) return st;
    }
    return HB_OK;
}

// A device buffer of n floats with the given alignment.
int check_float_buffer(const void *p, size_t n, unsigned align, KnownAllocations &known)
{
    if (p == nullptr) return HB_EINVAL;
    if (((uintptr_t)p & (align - 1)) != 0) return HB_EALIGN;
    return check_device_bytes(p, n * sizeof(float), known);
}

bool all_aligned16(const void *const *ptrs, int count)
{
    for (int i = 0; i < count; ++i) {
        if (((uintptr_t)ptrs[i] & 15u) != 0) return false;
    }
    return true;
}

// Argument rules of one tensor of a call (no launch): slice, pointers, alignment, device memory, overlaps.
int validate_tensor(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, const int64_t *out0,
                    const int64_t *out1, KnownAllocations &known)
{
    if (!valid_slice(k, m)) return HB_EINVAL;
    const void *ptrs[4] = {share0, share1, out0, out1};
    const int st = check_common(ptrs, 4, n, known);
    if (st != HB_OK) return st;
    if (n > 0) {
        const Range i0 = range_of(share0, n), i1 = range_of(share1, n), r0 = range_of(out0, n), r1 = range_of(out1, n);
        // an output may coincide with an input; every other overlap is refused
        if (!disjoint(r0, r1)) return HB_EINVAL;
        if (!(same(r0, i0) || disjoint(r0, i0)) || !(same(r0, i1) || disjoint(r0, i1))) return HB_EINVAL;
        if (!(same(r1, i0) || disjoint(r1, i0)) || !(same(r1, i1) || disjoint(r1, i1))) return HB_EINVAL;
    }
    return HB_OK;
}

uint64_t mode_bits(int mode, int k, int m, size_t n)
{
    return hb_opened_bits_ex(hb::op_of(mode) == hb::kRelu, k, m, n,
                             hb::shared_of(mode) ? HB_DEALER_SHARED_MASK : HB_DEALER_PER_GATE);
}

// mode of an operation (kDrelu or kRelu) on a dealer layout; -1 for an unknown layout
int mode_on(int op, int dealer)
{
    if (dealer == HB_DEALER_PER_GATE) return op;
    if (dealer == HB_DEALER_SHARED_MASK) return op + hb::kDreluShared;
    return -1;
}

// One kernel launch, ready to be enqueued: either a set of tensors of one width on wave-tiles (large or small) or one
// tensor on the thread-per-group kernel.
struct LaunchItem {
    hb::BatchLauncher tiles = nullptr;   // wave-tile launch of args.t[0 .. args.count)
    hb::GroupLauncher single = nullptr;  // per-tensor launch of args.t[0]
    hb::BatchArgs args = {};
};

hipError_t enqueue(const LaunchItem &it, hipStream_t stream)
{
    if (it.tiles != nullptr) return it.tiles(it.args, stream);
    const hb::BatchTensor &d = it.args.t[0];
    return it.single(d.x0, d.x1, d.n, d.k, d.seedB, d.seedA, d.o0, d.o1, stream);
}

void fill_tensor(hb::BatchTensor &d, const hb_tensor &t)
{
    d.x0 = (const uint64_t *)t.share0;
    d.x1 = (const uint64_t *)t.share1;
    d.o0 = (uint64_t *)t.out0;
    d.o1 = (uint64_t *)t.out1;
    d.n = t.n;
    d.seedB = hb::stream_word(t.seed, 0);
    d.seedA = hb::stream_word(t.seed, 1);
    d.k = t.k;
}

// Turns validated tensors (all of `mode`) into launches: tensors of one slice width that have a wave-tile kernel
// share launches of up to kBatchMax tensors; the others get one launch each.  Tensors with n == 0 are skipped.
// Returns HB_OK or HB_EHIP (no kernel for a width: a build problem).
int plan_launches(int mode, const hb_tensor *tensors, size_t count, std::vector<LaunchItem> &items)
{
    std::vector<char> taken(count, 0);
    for (size_t i = 0; i < count; ++i) {
        if (taken[i]) continue;
        taken[i] = 1;
        const hb_tensor &first = tensors[i];
        if (first.n == 0) continue;
        const int w = first.m - first.k;
        const hb::BatchLauncher big = hb::force_group_kernel() ? nullptr : hb::launcher_table().batch[mode][w - 1];
        if (big == nullptr) {
            LaunchItem it;
            it.single = hb::launcher_table().f[mode][w - 1];
            if (it.single == nullptr) return fail_hip(hipErrorInvalidDeviceFunction, "no kernel was built for this slice width");
            fill_tensor(it.args.t[0], first);
            it.args.count = 1;
            items.push_back(it);
            continue;
        }
        // every tensor of this width, in order
        std::vector<size_t> same;
        for (size_t j = i; j < count; ++j) {
            if ((j == i || !taken[j]) && tensors[j].m - tensors[j].k == w && tensors[j].n > 0) {
                taken[j] = 1;
                same.push_back(j);
            }
        }
        const uint64_t per_tile = (uint64_t)hb::tile_elements(w);
        LaunchItem it;
        auto start = [&] {
            it.tiles = big;
            it.args = hb::BatchArgs{};
            for (uint32_t &e : it.args.tile_end) e = hb::kNoTile;
        };
        auto finish = [&] {
            it.args.whole_blocks = hb::tile_grid(it.args.tiles, w, 2, hb::op_of(mode)).whole_blocks;
            items.push_back(it);
        };
        start();
        for (size_t j : same) {
            const hb_tensor &t = tensors[j];
            const uint64_t tiles = (t.n + per_tile - 1) / per_tile;
            if (tiles >= hb::kNoTile) return fail_hip(hipErrorInvalidConfiguration, "more wave-tiles than a grid holds");
            if (it.args.count == hb::kBatchMax || it.args.tiles + tiles >= hb::kNoTile) {
                finish();
                start();
            }
            hb::BatchTensor &d = it.args.t[it.args.count];
            fill_tensor(d, t);
            d.first_tile = it.args.tiles;
            if (it.args.count > 0) it.args.tile_end[it.args.count - 1] = it.args.tiles;
            it.args.tiles += (uint32_t)tiles;
            ++it.args.count;
        }
        finish();
    }
    return HB_OK;
}

int run(int mode, const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int64_t *out0,
        int64_t *out1, uint64_t *opened_bits, void *stream)
{
    KnownAllocations known;
    const int st = validate_tensor(share0, share1, n, k, m, out0, out1, known);
    if (st != HB_OK) return st;
    const int w = m - k;
    uint64_t bits = 0;
    if (mode == hb::kSign) {
        bits = (uint64_t)n * (2ull * (uint64_t)w * (1 + 2 * (uint64_t)rounds_of(w)));
    } else {
        bits = mode_bits(mode, k, m, n);
    }
    if (n > 0) {
        const uint64_t seedB = hb::stream_word(seed, 0), seedA = hb::stream_word(seed, 1);
        const hb::GroupLauncher f = hb::launcher_table().f[mode][w - 1];
        if (f == nullptr) return fail_hip(hipErrorInvalidDeviceFunction, "no kernel was built for this slice width");
        const hipError_t e = f((const uint64_t *)share0, (const uint64_t *)share1, (uint64_t)n, k, seedB, seedA,
                               (uint64_t *)out0, (uint64_t *)out1, (hipStream_t)stream);
        if (e != hipSuccess) return fail_hip(e, "kernel launch");
    }
    if (opened_bits) *opened_bits = bits;
    return HB_OK;
}

// DReLU / ReLU among `parties` parties.  shares / outs: host arrays of `parties` device pointers.
int run_mp(int op, const int64_t *const *shares, int parties, size_t n, int k, int m, uint64_t seed,
           int64_t *const *outs, uint64_t *opened_bits, void *stream)
{
    if (parties < 2 || parties > hb::kMaxParties) return HB_EINVAL;
    if (shares == nullptr || outs == nullptr) return HB_EINVAL;
    if (parties == 2) return run(op, shares[0], shares[1], n, k, m, seed, outs[0], outs[1], opened_bits, stream);
    if (!valid_slice(k, m)) return HB_EINVAL;
    const void *ptrs[2 * hb::kMaxParties];
    for (int q = 0; q < parties; ++q) {
        ptrs[q] = shares[q];
        ptrs[parties + q] = outs[q];
    }
    KnownAllocations known;
    const int st = check_common(ptrs, 2 * parties, n, known);
    if (st != HB_OK) return st;
    if (n > 0) {
        // an output may coincide with an input; every other overlap is refused
        for (int q = 0; q < parties; ++q) {
            const Range out = range_of(outs[q], n);
            for (int t = 0; t < parties; ++t) {
                const Range in = range_of(shares[t], n);
                if (!(same(out, in) || disjoint(out, in))) return HB_EINVAL;
                if (t != q && !disjoint(out, range_of(outs[t], n))) return HB_EINVAL;
            }
        }
        hb::MpPointers ptr = {};
        for (int q = 0; q < parties; ++q) {
            ptr.x[q] = (const uint64_t *)shares[q];
            ptr.o[q] = (uint64_t *)outs[q];
        }
        const hb::MpLauncher f = hb::launcher_table().mp[parties - 3][op][m - k - 1];
        if (f == nullptr) return fail_hip(hipErrorInvalidDeviceFunction, "no kernel was built for this slice width");
        const hipError_t e = f(ptr, (uint64_t)n, k, hb::stream_word(seed, 0), hb::stream_word(seed, 1),
                               (hipStream_t)stream);
        if (e != hipSuccess) return fail_hip(e, "kernel launch");
    }
    if (opened_bits) *opened_bits = hb_opened_bits_mp(op == hb::kRelu, parties, k, m, n);
    return HB_OK;
}

// Workspace of the party-faithful path: [wire 0][wire 1][reserve 0][reserve 1], every region 256-byte aligned.  The
// kernel uses the wires; the reserves (four words per group and one per element for each party) keep the size that
// callers and HB_PARTY_STATIC_BYTES were told when circuit state lived in memory.
struct PartyLayout {
    uint64_t groups, wire_words, off_b2a, wire_off[2], total_bytes;
};

PartyLayout party_layout(size_t n, int k, int m, int dealer = HB_DEALER_PER_GATE)
{
    const int w = m - k;
    const uint64_t L = (64 / w) > 32 ? 32 : (uint64_t)(64 / w);
    const uint64_t R = (uint64_t)rounds_of(w);
    const uint64_t per_round = dealer == HB_DEALER_SHARED_MASK ? 3 : 4;
    PartyLayout lay = {};
    lay.groups = ((uint64_t)n + L - 1) / L;
    lay.off_b2a = 2 * lay.groups + per_round * lay.groups * R;
    lay.wire_words = lay.off_b2a + ((uint64_t)n + 63) / 64 + 2 * (uint64_t)n;
    auto up = [](uint64_t b) { return (b + 255) & ~255ull; };
    const uint64_t wire_bytes = up(8 * lay.wire_words), reserve_bytes = up(8 * (4 * lay.groups + (uint64_t)n));
    lay.wire_off[0] = 0;
    lay.wire_off[1] = wire_bytes;
    lay.total_bytes = 2 * wire_bytes + 2 * reserve_bytes;
    return lay;
}

// Argument rules of a set of tensors (no launch): each tensor's own rules, then no output of one tensor over any
// buffer of another.  bits: the opened-bit count of the set.
int validate_set(int mode, const hb_tensor *tensors, size_t count, uint64_t *bits)
{
    if (count > 0 && tensors == nullptr) return HB_EINVAL;
    if (count > 4096) return HB_EINVAL;
    KnownAllocations known;
    for (size_t i = 0; i < count; ++i) {
        const hb_tensor &t = tensors[i];
        const int st = validate_tensor(t.share0, t.share1, t.n, t.k, t.m, t.out0, t.out1, known);
        if (st != HB_OK) return st;
    }
    for (size_t i = 0; i < count; ++i) {
        const hb_tensor &a = tensors[i];
        if (a.n == 0) continue;
        const Range outs[2] = {range_of(a.out0, a.n), range_of(a.out1, a.n)};
        for (size_t j = 0; j < count; ++j) {
            const hb_tensor &b = tensors[j];
            if (j == i || b.n == 0) continue;
            const Range others[4] = {range_of(b.share0, b.n), range_of(b.share1, b.n), range_of(b.out0, b.n),
                                     range_of(b.out1, b.n)};
            for (const Range &o : outs) {
                for (const Range &r : others) {
                    if (!disjoint(o, r)) return HB_EINVAL;
                }
            }
        }
    }
    uint64_t total = 0;
    for (size_t i = 0; i < count; ++i) total += mode_bits(mode, tensors[i].k, tensors[i].m, tensors[i].n);
    *bits = total;
    return HB_OK;
}

int run_batch(int mode, const hb_tensor *tensors, size_t count, uint64_t *opened_bits, void *stream)
{
    // validate everything first: on error nothing is enqueued
    uint64_t bits = 0;
    int st = validate_set(mode, tensors, count, &bits);
    if (st != HB_OK) return st;
    std::vector<LaunchItem> items;
    st = no_throw([&] { return plan_launches(mode, tensors, count, items); });
    if (st != HB_OK) return st;
    for (const LaunchItem &it : items) {
        const hipError_t e = enqueue(it, (hipStream_t)stream);
        if (e != hipSuccess) return fail_hip(e, "kernel launch");
    }
    if (opened_bits) *opened_bits = bits;
    return HB_OK;
}

// ---- the library's own workspace for hb_relu_party_static ---------------------------------------------------
// One array per GPU (each device that loads the code object holds its own copy at its own address, until the
// process ends).  In host code the array's name is only a handle for the symbol lookup below; kernels get the
// device address that the lookup returned, as an ordinary argument.
static __device__ __align__(256) unsigned char scratch[HB_PARTY_STATIC_BYTES];

constexpr int kMaxDevices = 64;
std::atomic<void *> g_scratch_of_device[kMaxDevices];

// Device address of `scratch` on the current device; looked up once per device, with that device current.
int party_scratch_of_current_device(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return HB_EINVAL;
    void *p = g_scratch_of_device[dev].load(std::memory_order_acquire);
    if (p == nullptr) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) return fail_hip(e, "hipGetSymbolAddress(scratch)");
        g_scratch_of_device[dev].store(p, std::memory_order_release);   // racing threads store the same address
    }
    *out = p;
    return HB_OK;
}

// The party-faithful path on a given workspace.  `own_workspace`: the workspace is the library's static array
// (its address and size are known good), otherwise a caller's buffer that is checked like every other argument.
int run_party(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int dealer,
              int64_t *out0, int64_t *out1, void *workspace, size_t workspace_bytes, bool own_workspace,
              uint64_t *wire_bytes, void *stream)
{
    if (dealer != HB_DEALER_PER_GATE && dealer != HB_DEALER_SHARED_MASK) return HB_EINVAL;
    KnownAllocations known;
    int st = validate_tensor(share0, share1, n, k, m, out0, out1, known);
    if (st != HB_OK) return st;
    const PartyLayout lay = party_layout(n, k, m, dealer);
    if (n > 0) {
        if (workspace == nullptr || workspace_bytes < lay.total_bytes) return HB_EINVAL;
        if (((uintptr_t)workspace & 255u) != 0) return HB_EALIGN;
        if (!own_workspace) {
            st = check_device_buffer(workspace, (lay.total_bytes + 7) / 8, known);
            if (st != HB_OK) return st;
        }
        const Range ws{(uintptr_t)workspace, (uintptr_t)workspace + lay.total_bytes};
        const Range bufs[4] = {range_of(share0, n), range_of(share1, n), range_of(out0, n), range_of(out1, n)};
        for (const Range &b : bufs) {
            if (!disjoint(ws, b)) return HB_EINVAL;
        }
        // no in-place operation here: a rule of the interface, which the kernel (it loads a tile before it stores it) would not need
        if (!disjoint(bufs[2], bufs[0]) || !disjoint(bufs[2], bufs[1]) || !disjoint(bufs[3], bufs[0]) ||
            !disjoint(bufs[3], bufs[1]))
            return HB_EINVAL;
    }
    if (wire_bytes) *wire_bytes = 8 * lay.wire_words;
    if (n == 0) return HB_OK;

    hb::PartyCtx c = {};
    char *base = (char *)workspace;
    c.x[0] = (const uint64_t *)share0;
    c.x[1] = (const uint64_t *)share1;
    c.out[0] = (uint64_t *)out0;
    c.out[1] = (uint64_t *)out1;
    c.n = n;
    c.groups = lay.groups;
    c.seedB = hb::stream_word(seed, 0);
    c.seedA = hb::stream_word(seed, 1);
    c.k = k;
    for (int p = 0; p < 2; ++p) c.wire[p] = (uint64_t *)(base + lay.wire_off[p]);
    c.off_b2a = lay.off_b2a;
    c.off_mul = lay.off_b2a + (n + 63) / 64;
    const hb::PartyLauncher f = hb::launcher_table().party[dealer == HB_DEALER_SHARED_MASK][m - k - 1];
    if (f == nullptr) return fail_hip(hipErrorInvalidDeviceFunction, "no kernel was built for this slice width");
    const hipError_t e = f(c, (hipStream_t)stream);
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return HB_OK;
}

}  // namespace

namespace hb {
LauncherTable &launcher_table()
{
    static LauncherTable table = {};
    return table;
}

// A tile that runs alone on a SIMD takes as long as a full round of tiles, one per SIMD.  256 tiles shared out by quarters are
// one round of quarters; quarter_rounds says how many of those still cost less than a round of whole tiles, which
// depends on how much of a quarter is spent on gate logic that its lanes repeat (most where a word has few fields), on idle
// owners, and on what an operation spends beside the dealer's words.  Launches of up to that many rounds of quarters share every
// tile out.  Measured, us, quarters / whole tiles:
//              w    512 tiles     768 tiles     1024 tiles                 w    512           768           1024
//   ReLU       4    5.4 / 11.2    6.4 / 11.7    7.5 / 13.3      sign       4    3.7 /  4.9    4.7 /  8.0    5.4 /  9.1
//              5    5.8 /  9.8    7.0 / 10.0    8.2 / 10.4                 6    3.8 /  6.6    4.4 /  6.2    5.4 /  6.3
//              6    5.6 /  9.2    6.9 /  8.5    8.1 /  9.2                 7    4.2 /  5.9    4.9 /  6.1    5.8 /  6.1
//              7    7.2 /  9.2    8.6 /  9.2   10.1 /  9.3                 8    3.8 /  4.9    4.0 /  4.9    4.5 /  5.2
//              8    4.3 /  7.1    5.2 /  7.6    6.0 /  7.7                 9    4.3 /  5.2    5.2 /  5.4    5.9 /  5.6
//              9    5.2 /  8.0    6.4 /  7.8    7.6 /  8.0                10    3.9 /  4.6    4.4 /  5.0    5.1 /  5.2
//             10    4.7 /  6.3    5.7 /  6.9    6.8 /  7.0                11    4.2 /  4.8    5.0 /  4.9    5.8 /  5.1
//             11    5.0 /  6.6    6.2 /  6.7    7.4 /  7.1                12    4.2 /  4.5    5.0 /  4.7    5.9 /  4.9
//             12    5.1 /  6.2    6.3 /  6.5    7.5 /  6.7                16    3.8 /  3.9    4.5 /  3.9    5.1 /  4.1
//             16    4.6 /  5.0    5.5 /  5.2    6.4 /  5.3                17    4.5 /  4.3    5.5 /  4.4    6.4 /  4.5
//             21    5.3 /  5.4    6.6 /  5.6    7.9 /  5.9                24    4.1 /  4.0    4.9 /  4.0    5.6 /  4.1
//             24    4.9 /  4.5    5.9 /  4.6    7.0 /  4.7      sim.       4    5.6 / 10.8    7.0 / 11.0    8.4 / 11.0
//   DReLU      4    3.9 /  6.4    5.0 /  9.4    5.7 / 10.7                 5    6.1 /  9.2    7.7 /  9.2    9.3 /  9.4
//              6    4.2 /  6.8    5.0 /  6.4    5.9 /  6.6                 6    5.9 /  8.1    7.4 /  8.2    9.1 /  8.3
//              7    4.6 /  6.6    5.7 /  6.4    6.7 /  6.6                 7    7.6 /  8.3    9.4 /  8.4   11.1 /  8.5
//              8    3.8 /  5.1    4.3 /  5.0    4.9 /  5.8                 8    4.3 /  7.0    5.3 /  7.1    6.4 /  7.1
//              9    4.6 /  5.8    5.6 /  5.8    6.6 /  6.2                 9    5.1 /  7.6    6.5 /  7.7    7.9 /  7.6
//             10    4.1 /  4.9    4.8 /  5.3    5.6 /  5.5                10    4.7 /  6.3    5.8 /  6.4    7.1 /  6.5
//             11    4.4 /  5.2    5.3 /  5.3    6.3 /  5.5                11    5.0 /  6.3    6.4 /  6.5    7.7 /  6.4
//             12    4.3 /  4.8    5.3 /  5.1    6.3 /  5.2                12    5.0 /  6.4    6.4 /  6.5    7.7 /  6.5
//             16    4.0 /  4.0    4.7 /  4.1    5.4 /  4.4                16    4.6 /  5.2    5.7 /  5.2    6.7 /  5.3
//             17    4.6 /  4.5    5.7 /  4.5    6.8 /  4.6                21    5.3 /  5.7    6.8 /  5.7    8.2 /  5.8
//             24    4.2 /  4.1    5.0 /  4.1    5.8 /  4.2                24    4.9 /  4.6    6.1 /  4.6    7.3 /  4.6
//   three      4    8.3 / 18.1   10.4 / 18.9   14.4 / 19.5      four       4   11.9 / 28.6   15.7 / 30.7   19.8 / 32.7
//              5    9.2 / 15.8   11.4 / 16.5   14.6 / 16.9                 5   13.8 / 22.3   17.8 / 23.2   22.6 / 23.8
//              6    9.0 / 14.7   11.2 / 14.7   13.6 / 14.8                 6   13.8 / 21.8   17.8 / 22.2   22.7 / 22.1
//              7   12.0 / 14.6   14.7 / 14.8   17.3 / 15.0                 7   18.6 / 21.6   25.5 / 21.7   30.6 / 22.1
//              8    7.0 / 12.1    8.7 / 12.4   10.6 / 12.6                 8   11.5 / 18.5   14.4 / 18.9   18.2 / 19.2
//              9    9.6 / 12.8   12.4 / 14.0   15.1 / 14.2                 9   15.9 / 21.1   20.8 / 22.0   26.5 / 22.5
//             10    8.1 / 11.7   10.3 / 12.0   12.5 / 12.2                10   13.2 / 19.3   17.0 / 19.6   21.5 / 20.0
//             11    9.5 / 12.0   12.2 / 12.1   14.7 / 12.1                11   15.7 / 19.4   20.4 / 19.6   26.2 / 20.3
//             16    7.8 /  9.7   10.1 / 10.1   12.1 / 10.2                16   12.7 / 16.9   16.6 / 17.2   21.1 / 17.2
//             24    8.8 /  9.6   11.5 /  9.8   14.4 /  9.9                24   15.2 / 17.5   21.8 / 17.7   26.9 / 17.7
//   its DReLU  4    6.0 / 12.3    7.4 / 12.4    9.3 / 13.5      its DReLU  4    8.8 / 17.1   11.8 / 17.6   14.1 / 18.7
//              6    6.9 / 11.1    8.3 / 11.1    9.8 / 11.1                 6   10.7 / 16.7   13.8 / 17.0   16.7 / 17.4
//              7    8.1 / 10.9   10.1 / 11.0   11.9 / 11.1                 7   13.2 / 16.4   17.0 / 16.8   21.3 / 17.2
//              8    6.0 /  9.4    7.4 /  9.6    8.6 /  9.9                 8    9.6 / 14.7   12.1 / 15.0   14.8 / 15.4
//              9    8.6 / 10.7   10.9 / 11.2   13.1 / 11.2                 9   14.0 / 17.7   18.7 / 18.0   24.1 / 18.5
//             10    7.0 /  9.9    8.9 /  9.9   10.6 / 10.1                10   11.8 / 16.5   15.4 / 16.9   19.5 / 17.1
// (quarters in the form that tile_runs gives them; the shared-mask layout has its ratios within 3 %.)  Five rounds where quarters are
// faster than 1024 whole tiles and 256 by quarters as well: 1280 tiles of ReLU at w = 4 9.5 / 10.2, w = 8 6.8 / 7.0 (1536 7.7 / 7.8, w = 5
// 10.6 / 9.3).  Two rounds up to w = 21, one above.  (Three where the fourth gains
// at its end and loses at its start, 810 tiles of DReLU at w = 6 6.0 / 5.2, sign shares at w = 7 5.9 / 5.4, DReLU of four parties at w = 6 16.6 /
// 15.6, or gains on one card and loses on the next, 810 and 1024 tiles of DReLU at w = 8 4.9 / 4.4 and 4.9 / 4.8, sign shares at w = 10 5.1 / 4.4 and
// 5.2 / 4.9.  DReLU's third at w = 11 and 12 changes sides twice within it.)  w = 7 has 72 pairs in a quarter: two passes
// of the 64 lanes, the second one nearly empty.
constexpr uint64_t kSimds = 1024, kQuarterRound = kSimds / 4;
constexpr int quarter_rounds(int w, int parties, int op)
{
    if (parties == 3) return w <= 6 || w == 8 ? 4 : w == 9 || w == 10 || (w == 7 && op == kDrelu) ? 3 : 2;
    if (parties == 4) return w == 4 || w == 5 || w == 8 ? 4 : w == 6 || w == 10 || (w == 9 && op == kRelu) ? 3 : 2;
    if (w > 12) return w <= 21 ? 2 : 1;
    if (op == kSimulator) return w == 4 || w == 8 ? 4 : w == 7 || w >= 11 ? 2 : 3;
    if (op == kSign) return w >= 11 ? 2 : w == 7 || w >= 9 ? 3 : 4;
    if (op == kDrelu) return w <= 5 ? 4 : 3;
    return w == 4 || w == 8 ? 5 : w == 7 || w >= 11 ? 3 : 4;
}
// Of what a longer launch leaves after its last full round, two rounds of quarters are shared out: 376 tiles left, ReLU,
// w = 8 7.9 / 10.1, w = 16 7.3 / 8.0.  A third one after up to seven full rounds, of ReLU and the simulator at the widths where it
// gains (600 left after one to seven full rounds, shared out / in whole tiles; the shared-mask layout and 520 to 768 left likewise):
//   ReLU w = 4   12.2 / 17.7   18.0 / 22.4   24.8 / 28.4   30.7 / 36.6   37.5 / 41.4   43.4 / 48.2   48.5 / 54.5
//            5   11.6 / 12.5   16.3 / 16.1   20.8 / 20.7   26.8 / 29.1
//            6   10.7 / 11.1   15.2 / 14.2   18.7 / 17.9
//            8    8.4 /  9.4   11.6 / 12.2   14.6 / 15.1   17.9 / 19.0   23.1 / 24.3   26.1 / 26.6   29.5 / 30.4
//            9    9.8 / 10.4   13.1 / 14.0   16.8 / 17.5   20.2 / 20.8   24.0 / 25.8   27.5 / 28.1   31.6 / 32.0
//           10    8.6 /  8.9   11.6 / 11.6   14.7 / 14.4   17.1 / 17.1   20.3 / 20.1   23.8 / 24.7   26.9 / 27.2
//           11    8.9 /  9.2   11.7 / 11.9   14.5 / 14.9   17.7 / 17.7   21.0 / 20.5   23.6 / 24.5   26.5 / 26.5
//           12    9.0 /  9.1   11.9 / 12.0   14.6 / 15.0   17.7 / 17.9   21.0 / 20.6   23.6 / 24.6   26.5 / 26.5
//   sim.     4   12.9 / 15.0   18.3 / 20.3   23.8 / 25.9   29.9 / 32.2   35.0 / 37.2   40.3 / 42.6   45.6 / 48.4
//            8    8.8 /  9.4   12.3 / 12.9   15.9 / 16.5   19.5 / 20.1   22.6 / 23.7   26.1 / 27.1   29.5 / 30.7
//            6   11.3 / 11.2   15.9 / 15.5                     10    9.0 /  8.9   12.1 / 12.1
// Where the sides are within 3 %, w = 10 to 12 after three rounds and more, the card decides: on another w = 10 took 18.2 / 18.6 after four and
// w = 12 20.6 / 21.4 after five.
// DReLU at w = 5 would lose (after two full rounds 13.4 / 11.5).  One round only
//   - from w = 22, among more parties from w = 13 on, and of the simulator at w = 7 and from w = 17 on (376 left 9.0 / 8.8),
//   - of sign shares at w = 5 and 6 after two full rounds (452 left 11.4 / 11.1 and 9.8 / 8.7; after one 6.2 / 6.8, after three
//     15.9 / 17.2 and 12.9 / 13.9): three rounds of them reside together and wait for memory alone.
// None where the quarter form's registers and LDS, which every workgroup of the launch then has, cost a long launch as much as a
// round saves it: after 16 full rounds from w = 22 on (32 rounds and 8 tiles, shared-mask ReLU at w = 24 76.8 / 76.0), after 32
// from w = 17 on among more parties (85 rounds and 8 tiles, four at w = 17 1289 / 1275).
constexpr uint64_t shared_remainder(uint64_t tiles, int w, int parties, int op)
{
    const uint64_t full = tiles / kSimds;
    if (parties > 2 ? w >= 17 && full >= 32 : w >= 22 && full >= 16) return 0;
    if (parties > 2 ? w >= 13 : w >= 22) return kQuarterRound;
    if (op == kSimulator && (w == 7 || w >= 17)) return kQuarterRound;
    if (op == kSign && (w == 5 || w == 6) && full == 2) return kQuarterRound;
    if (parties == 2 && full < 8) {
        if (op == kRelu && (w == 4 || (w >= 8 && w <= 12) || (w == 5 && full <= 4) || (w == 6 && full == 1))) return 3 * kQuarterRound;
        if (op == kSimulator && (w == 4 || w == 8)) return 3 * kQuarterRound;
    }
    return 2 * kQuarterRound;
}

// HB_SMALL_TILE_LIMIT in the environment (read once): launches of fewer tiles share every tile out; 0 switches the quarters off.
uint64_t small_tile_limit(uint64_t usual)
{
    static const char *const v = std::getenv("HB_SMALL_TILE_LIMIT");
    static const uint64_t given = v != nullptr ? (uint64_t)std::strtoull(v, nullptr, 10) : 0;
    return v != nullptr ? given : usual;
}

// Which launches take the form with RUNS (mix_words): those whose SIMDs hold a second wavefront for most of the time, or, where
// tiles are shared out, more than one round of quarters.  Two parties, ReLU, us, without / with:
//      all by quarters             whole tiles             1024 whole tiles and the rest by quarters         longer
//   w   300 tiles   1000 tiles     1000 tiles              1088           1400                               1700           2^25 elements
//   4   5.3 / 5.1    8.7 / 7.9                                            11.1 / 11.4                         15.7 / 14.6    213 / 204
//   6   5.6 / 5.3                   7.9 /  8.2              8.5 / 8.6     10.3 /  9.6                         12.0 / 11.1    248 / 232
//   8   4.2 / 4.0    6.6 / 6.2                              7.0 / 7.3      7.8 /  7.8                         10.1 /  9.5    258 / 240
//  12   4.8 / 4.8                   6.6 /  6.9              7.0 / 7.3      8.4 /  8.0                          9.9 /  9.3    360 / 333
//  16   4.5 / 4.4                   5.0 /  5.3              6.4 / 5.9      7.5 /  6.7                          7.9 /  7.5    375 / 352
//  32                               4.8 /  5.0              6.6 / 5.8      7.1 /  6.5                          7.2 /  6.6   1280 / 1174
// (At w = 7 and below 4 the form wins from the first tile beyond 1024: 1088 tiles 10.1 / 9.2, w = 2 14.1 / 13.1;
// at w = 4 1025 to 1280 tiles, which go by quarters alone, take 4 to 7 % longer with it.)  Beyond 1024 tiles the
// line lies at one round of quarters, 256 tiles, at w = 4 at two.  256, 320 and 376 tiles beyond:
//   ReLU   w = 5   9.2 /  9.5   11.0 / 10.3   10.9 / 10.4     DReLU w = 10   5.6 / 5.6   6.4 / 6.0   6.3 / 6.0
//              9   7.9 /  8.3    9.2 /  8.8    9.2 /  8.9             11   5.6 / 5.9   6.5 / 6.1   6.6 / 6.2
//             10   7.0 /  7.3    8.3 /  7.9    8.3 /  7.9             12   5.6 / 5.8   6.5 / 6.1   6.6 / 6.1
//             11   7.1 /  7.4    8.5 /  7.9    8.5 /  8.0     (w = 4: 376 and 476 beyond 1.03, 676 0.97 of the time without)
//             12   7.1 /  7.5    8.5 /  8.0    8.5 /  8.1
// The simulator, which draws shares besides, has it from the first tile beyond 1024 on (6, 256 and 320 beyond: w = 5 9.5 / 9.2, 9.7 / 9.3,
// 11.9 / 10.6; w = 6 8.9 / 8.4, 9.1 / 8.5, 11.0 / 9.6; w = 9 7.9 / 7.8, 7.9 / 7.9, 9.7 / 8.9; w = 10 7.2 / 6.9, 7.3 / 7.0, 8.6 / 7.8; w = 12 7.3 /
// 6.8, 7.3 / 6.9, 8.9 / 7.9) except at w = 4 (9.9 / 10.2, 10.3 / 10.4, 12.2 / 11.4) and 8 (6.9 / 7.0, 7.0 / 7.1, 8.3 / 7.8).
// Among more parties a kernel's second round counts from its first tile on (76 tiles beyond 1024: w = 8 12.4 / 12.4 and 20.0 / 19.3,
// w = 32 13.3 / 11.3 and 24.1 / 20.5; 676 tiles 5 to 15 % of any width), but for w = 4 (three parties, 256 and 320 beyond, 16.6 / 16.8 and
// 19.3 / 18.1; four, 320, 476 and 676 beyond, 29.2 / 30.5, 29.6 / 31.4, 46.0 / 38.6) and DReLU of three at w = 5 (11.2 / 11.8, 13.0 / 12.0).
// Their ReLU at w = 1 streams 96 and 128 bytes an element past a circuit of one gate an adder: words in step pay while the launch's
// wavefronts reside all at once, in the third and fourth round (three parties, 2.5 M elements 30.2 / 28.7; four, 1.3 M 21.3 / 20.8), not before
// (0.7 M 14.3 / 15.3) and not after (three, 3.6, 5.3 and 8.1 M 42.2 / 44.7, 54.0 / 55.1, 81.7 / 81.3; four, 2.1, 9.2 and 20.5 M 33.2 / 35.6, 112 / 120,
// 246 / 259).
// DReLU of two parties at w = 10 to 12 gains least between 100 and 270 MB of shares and results, which stay in the cache before
// memory in part: 3.7, 5.0, 6.3, 8.0 and 16 M elements w = 10 25.9 / 24.5, 34.3 / 32.9, 42.4 / 41.1, 53.4 / 50.7, 105 / 94.8, w = 11 29.1 /
// 29.2, 38.0 / 38.7, 47.7 / 48.0, 62.2 / 59.4, 121 / 112, w = 12 29.2 / 28.6, 38.3 / 38.2, 47.3 / 47.4, 61.4 / 59.1, 122 / 113; on the
// shared-mask layout 24.9 / 23.4, 32.1 / 30.8, 38.5 / 39.5, 49.4 / 48.0, 97.4 / 91.7; 27.5 / 26.1, 35.8 / 36.3, 43.9 / 45.3, 57.2 / 56.3,
// 112 / 106; 27.4 / 26.0, 35.7 / 36.1, 44.1 / 44.7, 57.0 / 56.0, 112 / 106.  So on three cards; two others took w = 10 up to
// 7 % longer with the form between 3.5 and 7 M, and the rest as these.  A line there would cost on one card what it gives on the next.
bool tile_runs(uint64_t tiles, uint64_t split, int w, int parties, int op)
{
    if (split == tiles) return tiles > kQuarterRound && (w == 8 || tiles <= kSimds);
    if (tiles <= kSimds) return false;
    if (parties > 2 && w == 1) return tiles > 2 * kSimds && tiles <= 4 * kSimds;
    uint64_t line = w == 4 ? 2 : 1;                  // rounds of quarters beyond the full one that go without
    if (parties > 2) line = w == 4 ? (parties == 4 ? 2 : 1) : parties == 3 && w == 5 && op == kDrelu ? 1 : 0;
    else if (op == kSimulator) line = w == 4 || w == 8 ? 1 : 0;
    else if (w <= 3 || w == 7 || w >= 13) line = 0;
    return tiles - kSimds > line * kQuarterRound;
}

TileGrid tile_grid(uint64_t tiles, int w, int parties, int op)
{
    const uint64_t left = tiles % kSimds;
    const uint64_t limit = small_tile_limit((uint64_t)quarter_rounds(w, parties, op) * kQuarterRound + 1);
    uint64_t split = 0;
    if (quarters_supported(w) && limit != 0) split = tiles < limit ? tiles : left <= shared_remainder(tiles, w, parties, op) ? left : 0;
    if (tiles < kSimds && split < tiles) split = 0;          // no full round before them
    const uint64_t whole = (tiles - split + kWavesPerBlock - 1) / kWavesPerBlock, blocks = whole + split;
    if (blocks > 0x7fffffffull) return TileGrid{0, 0, false, false};
    return TileGrid{(uint32_t)whole, (uint32_t)blocks, split != 0, tile_runs(tiles, split, w, parties, op)};
}

bool group_runs(uint64_t blocks) { return blocks > kSimds / kWavesPerBlock; }

bool force_group_kernel()
{
    static const bool forced = [] {
        const char *v = std::getenv("HB_KERNEL");
        return v != nullptr && std::strcmp(v, "group") == 0;
    }();
    return forced;
}
}  // namespace hb

extern "C" {

int hb_drelu(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int64_t *out0,
             int64_t *out1, uint64_t *opened_bits, void *stream)
{
    return run(hb::kDrelu, share0, share1, n, k, m, seed, out0, out1, opened_bits, stream);
}

int hb_relu(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int64_t *out0,
            int64_t *out1, uint64_t *opened_bits, void *stream)
{
    return run(hb::kRelu, share0, share1, n, k, m, seed, out0, out1, opened_bits, stream);
}

int hb_sign_shares(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int64_t *out0,
                   int64_t *out1, uint64_t *opened_bits, void *stream)
{
    return run(hb::kSign, share0, share1, n, k, m, seed, out0, out1, opened_bits, stream);
}

int hb_relu_batch(const hb_tensor *tensors, size_t count, uint64_t *opened_bits, void *stream)
{
    return run_batch(hb::kRelu, tensors, count, opened_bits, stream);
}

int hb_drelu_batch(const hb_tensor *tensors, size_t count, uint64_t *opened_bits, void *stream)
{
    return run_batch(hb::kDrelu, tensors, count, opened_bits, stream);
}

int hb_drelu_ex(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int dealer,
                int64_t *out0, int64_t *out1, uint64_t *opened_bits, void *stream)
{
    const int mode = mode_on(hb::kDrelu, dealer);
    if (mode < 0) return HB_EINVAL;
    return run(mode, share0, share1, n, k, m, seed, out0, out1, opened_bits, stream);
}

int hb_relu_ex(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int dealer,
               int64_t *out0, int64_t *out1, uint64_t *opened_bits, void *stream)
{
    const int mode = mode_on(hb::kRelu, dealer);
    if (mode < 0) return HB_EINVAL;
    return run(mode, share0, share1, n, k, m, seed, out0, out1, opened_bits, stream);
}

int hb_relu_batch_ex(const hb_tensor *tensors, size_t count, int dealer, uint64_t *opened_bits, void *stream)
{
    const int mode = mode_on(hb::kRelu, dealer);
    if (mode < 0) return HB_EINVAL;
    return run_batch(mode, tensors, count, opened_bits, stream);
}

int hb_drelu_batch_ex(const hb_tensor *tensors, size_t count, int dealer, uint64_t *opened_bits, void *stream)
{
    const int mode = mode_on(hb::kDrelu, dealer);
    if (mode < 0) return HB_EINVAL;
    return run_batch(mode, tensors, count, opened_bits, stream);
}

struct hb_plan {
    std::vector<LaunchItem> items;
    uint64_t opened_bits = 0;
};

int hb_plan_create(const hb_tensor *tensors, size_t count, int relu, int dealer, hb_plan **plan)
{
    if (plan == nullptr) return HB_EINVAL;
    *plan = nullptr;
    const int mode = mode_on(relu ? hb::kRelu : hb::kDrelu, dealer);
    if (mode < 0) return HB_EINVAL;
    uint64_t bits = 0;
    int st = validate_set(mode, tensors, count, &bits);
    if (st != HB_OK) return st;
    hb_plan *p = new (std::nothrow) hb_plan;
    if (p == nullptr) return HB_EINVAL;
    st = no_throw([&] { return plan_launches(mode, tensors, count, p->items); });
    if (st != HB_OK) {
        delete p;
        return st;
    }
    p->opened_bits = bits;
    *plan = p;
    return HB_OK;
}

int hb_plan_run(const hb_plan *plan, uint64_t *opened_bits, void *stream)
{
    if (plan == nullptr) return HB_EINVAL;
    for (const LaunchItem &it : plan->items) {
        const hipError_t e = enqueue(it, (hipStream_t)stream);
        if (e != hipSuccess) return fail_hip(e, "kernel launch");
    }
    if (opened_bits) *opened_bits = plan->opened_bits;
    return HB_OK;
}

void hb_plan_destroy(hb_plan *plan) { delete plan; }

int hb_drelu_mp(const int64_t *const *shares, int parties, size_t n, int k, int m, uint64_t seed,
                int64_t *const *outs, uint64_t *opened_bits, void *stream)
{
    return run_mp(hb::kDrelu, shares, parties, n, k, m, seed, outs, opened_bits, stream);
}

int hb_relu_mp(const int64_t *const *shares, int parties, size_t n, int k, int m, uint64_t seed,
               int64_t *const *outs, uint64_t *opened_bits, void *stream)
{
    return run_mp(hb::kRelu, shares, parties, n, k, m, seed, outs, opened_bits, stream);
}

size_t hb_party_wire_words(size_t n, int k, int m)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS) return 0;
    const PartyLayout lay = party_layout(n, k, m);
    return (size_t)lay.wire_words;
}

size_t hb_party_workspace_bytes(size_t n, int k, int m)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS) return 0;
    return (size_t)party_layout(n, k, m).total_bytes;
}

size_t hb_party_wire_offset(size_t n, int k, int m, int party)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS || party < 0 || party > 1) return 0;
    return (size_t)party_layout(n, k, m).wire_off[party];
}

int hb_relu_party(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int64_t *out0,
                  int64_t *out1, void *workspace, size_t workspace_bytes, uint64_t *wire_bytes, void *stream)
{
    return run_party(share0, share1, n, k, m, seed, HB_DEALER_PER_GATE, out0, out1, workspace, workspace_bytes, false,
                     wire_bytes, stream);
}

int hb_relu_party_ex(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed, int dealer,
                     int64_t *out0, int64_t *out1, void *workspace, size_t workspace_bytes, uint64_t *wire_bytes,
                     void *stream)
{
    return run_party(share0, share1, n, k, m, seed, dealer, out0, out1, workspace, workspace_bytes, false, wire_bytes,
                     stream);
}

size_t hb_party_wire_words_ex(size_t n, int k, int m, int dealer)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS || (dealer != HB_DEALER_PER_GATE && dealer != HB_DEALER_SHARED_MASK)) return 0;
    return (size_t)party_layout(n, k, m, dealer).wire_words;
}

size_t hb_party_workspace_bytes_ex(size_t n, int k, int m, int dealer)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS || (dealer != HB_DEALER_PER_GATE && dealer != HB_DEALER_SHARED_MASK)) return 0;
    return (size_t)party_layout(n, k, m, dealer).total_bytes;
}

size_t hb_party_wire_offset_ex(size_t n, int k, int m, int dealer, int party)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS || party < 0 || party > 1 ||
        (dealer != HB_DEALER_PER_GATE && dealer != HB_DEALER_SHARED_MASK))
        return 0;
    return (size_t)party_layout(n, k, m, dealer).wire_off[party];
}

int hb_relu_party_static(const int64_t *share0, const int64_t *share1, size_t n, int k, int m, uint64_t seed,
                         int64_t *out0, int64_t *out1, uint64_t *wire_bytes, void *stream)
{
    if (!valid_slice(k, m) || n > HB_MAX_ELEMENTS) return HB_EINVAL;
    if (party_layout(n, k, m).total_bytes > HB_PARTY_STATIC_BYTES) return HB_ETOOBIG;
    void *ws = nullptr;
    const int st = party_scratch_of_current_device(&ws);
    if (st != HB_OK) return st;
    return run_party(share0, share1, n, k, m, seed, HB_DEALER_PER_GATE, out0, out1, ws, HB_PARTY_STATIC_BYTES, true,
                     wire_bytes, stream);
}

int hb_share_f32(const float *x, size_t n, uint64_t share_seed, int64_t *share0, int64_t *share1, void *stream)
{
    const void *ptrs[2] = {share0, share1};
    KnownAllocations known;
    int st = check_common(ptrs, 2, n, known);
    if (st != HB_OK) return st;
    if (n == 0) return HB_OK;
    st = check_float_buffer(x, n, 4, known);
    if (st != HB_OK) return st;
    const Range rx{(uintptr_t)x, (uintptr_t)x + 4 * n}, r0 = range_of(share0, n), r1 = range_of(share1, n);
    if (!disjoint(r0, r1) || !disjoint(rx, r0) || !disjoint(rx, r1)) return HB_EINVAL;
    const uint64_t blocks = (((uint64_t)n + 1) / 2 + hb::kShareBlock - 1) / hb::kShareBlock;
    if (blocks > 0x7fffffffull) return HB_EINVAL;
    hipLaunchKernelGGL(hb::share_f32_kernel, dim3((unsigned)blocks), dim3(hb::kShareBlock), 0, (hipStream_t)stream, x,
                       (uint64_t)n, share_seed, (uint64_t *)share0, (uint64_t *)share1);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? HB_OK : fail_hip(e, "kernel launch");
}

int hb_reveal_f32(const int64_t *share0, const int64_t *share1, size_t n, float *y, void *stream)
{
    const void *ptrs[2] = {share0, share1};
    KnownAllocations known;
    int st = check_common(ptrs, 2, n, known);
    if (st != HB_OK) return st;
    if (n == 0) return HB_OK;
    st = check_float_buffer(y, n, 4, known);
    if (st != HB_OK) return st;
    const Range ry{(uintptr_t)y, (uintptr_t)y + 4 * n};
    if (!disjoint(ry, range_of(share0, n)) || !disjoint(ry, range_of(share1, n))) return HB_EINVAL;
    const uint64_t blocks = (((uint64_t)n + 1) / 2 + hb::kBlock - 1) / hb::kBlock;
    if (blocks > 0x7fffffffull) return HB_EINVAL;
    hipLaunchKernelGGL(hb::reveal_f32_kernel, dim3((unsigned)blocks), dim3(hb::kBlock), 0, (hipStream_t)stream,
                       (const uint64_t *)share0, (const uint64_t *)share1, (uint64_t)n, y);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? HB_OK : fail_hip(e, "kernel launch");
}

int hb_sim_relu_f32(const float *x, size_t n, int k, int m, uint64_t seed, uint64_t share_seed, float *y, void *stream)
{
    if (!valid_slice(k, m)) return HB_EINVAL;
    if (n > HB_MAX_ELEMENTS) return HB_EINVAL;
    const hb::SimLauncher f = hb::launcher_table().sim[m - k - 1];
    if (f == nullptr) return HB_ENOTSUP;
    if (n == 0) return HB_OK;
    KnownAllocations known;
    int st = check_float_buffer(x, n, 8, known);
    if (st != HB_OK) return st;
    st = check_float_buffer(y, n, 8, known);
    if (st != HB_OK) return st;
    const Range rx{(uintptr_t)x, (uintptr_t)x + 4 * n}, ry{(uintptr_t)y, (uintptr_t)y + 4 * n};
    if (!(rx.lo == ry.lo || disjoint(rx, ry))) return HB_EINVAL;
    const hipError_t e = f(x, (uint64_t)n, k, hb::stream_word(seed, 0), hb::stream_word(seed, 1), share_seed, y,
                           (hipStream_t)stream);
    return e == hipSuccess ? HB_OK : fail_hip(e, "kernel launch");
}

int hb_eco_scan(const int64_t *share0, const int64_t *share1, size_t n, uint64_t *counts, void *stream)
{
    if (counts == nullptr) return HB_EINVAL;
    if (((uintptr_t)counts & 7u) != 0) return HB_EALIGN;
    const void *ptrs[2] = {share0, share1};
    KnownAllocations known;
    int st = check_common(ptrs, 2, n, known);
    if (st != HB_OK) return st;
    st = check_device_buffer(counts, 64, known);
    if (st != HB_OK) return st;
    if (n > 0) {
        const Range c = range_of(counts, 64);
        if (!disjoint(c, range_of(share0, n)) || !disjoint(c, range_of(share1, n))) return HB_EINVAL;
    }
    // One workgroup per compute unit (kEcoWaves x 256 wavefronts), fewer where a wavefront would get less than one tree of rows,
    // more where a lane's counter would overflow.
    const uint64_t rows = ((uint64_t)n + hb::kEcoRow - 1) / hb::kEcoRow;
    uint64_t blocks = (rows + hb::kEcoRows * hb::kEcoWaves - 1) / (hb::kEcoRows * hb::kEcoWaves);
    if (blocks > 256) blocks = 256;
    const uint64_t least = (rows + hb::kEcoMaxRows * hb::kEcoWaves - 1) / (hb::kEcoMaxRows * hb::kEcoWaves);
    if (blocks < least) blocks = least;
    hipError_t e;
    if (blocks != 1) {                  // a single workgroup stores its counts
        hipLaunchKernelGGL(hb::eco_zero_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, (unsigned long long *)counts);
        e = hipGetLastError();
        if (e != hipSuccess) return fail_hip(e, "kernel launch");
    }
    if (n == 0) return HB_OK;
    const uint64_t per_lane = 2 * ((rows + blocks * hb::kEcoWaves - 1) / (blocks * hb::kEcoWaves));
    int live = 1;
    while ((1ull << live) <= per_lane) ++live;      // planes that can be non-zero
    hipLaunchKernelGGL(hb::eco_scan_kernel, dim3((unsigned)blocks), dim3(hb::kEcoBlock), 0, (hipStream_t)stream,
                       (const uint64_t *)share0, (const uint64_t *)share1, (uint64_t)n, rows, live,
                       (unsigned long long *)counts);
    e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return HB_OK;
}

int hb_eco_choose(const uint64_t *counts)
{
    if (counts == nullptr) return HB_EINVAL;
    int m = 64;
    while (m > 1 && counts[m - 2] == 0) --m;
    return m;
}

int hb_open(const int64_t *share0, const int64_t *share1, size_t n, int binary, int64_t *out, void *stream)
{
    const void *ptrs[3] = {share0, share1, out};
    KnownAllocations known;
    const int st = check_common(ptrs, 3, n, known);
    if (st != HB_OK) return st;
    if (n == 0) return HB_OK;
    const Range i0 = range_of(share0, n), i1 = range_of(share1, n), r = range_of(out, n);
    if (!(same(r, i0) || disjoint(r, i0)) || !(same(r, i1) || disjoint(r, i1))) return HB_EINVAL;
    const bool vec = all_aligned16(ptrs, 3);
    const uint64_t threads = vec ? ((uint64_t)n + 1) / 2 : (uint64_t)n;
    const uint64_t blocks = (threads + hb::kBlock - 1) / hb::kBlock;
    if (blocks > 0x7fffffffull) return HB_EINVAL;
    if (vec) {
        hipLaunchKernelGGL((hb::open_kernel<true>), dim3((unsigned)blocks), dim3(hb::kBlock), 0, (hipStream_t)stream,
                           (const uint64_t *)share0, (const uint64_t *)share1, (uint64_t)n, binary, (uint64_t *)out);
    } else {
        hipLaunchKernelGGL((hb::open_kernel<false>), dim3((unsigned)blocks), dim3(hb::kBlock), 0, (hipStream_t)stream,
                           (const uint64_t *)share0, (const uint64_t *)share1, (uint64_t)n, binary, (uint64_t *)out);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_hip(e, "kernel launch");
    return HB_OK;
}

uint64_t hb_tensor_seed(uint64_t root_seed, uint64_t tensor_id) { return hb::stream_word(root_seed, 2 + tensor_id); }

uint64_t hb_opened_bits(int relu, int k, int m, size_t n)
{
    return hb_opened_bits_ex(relu, k, m, n, HB_DEALER_PER_GATE);
}

uint64_t hb_opened_bits_ex(int relu, int k, int m, size_t n, int dealer)
{
    if (!valid_slice(k, m) || (dealer != HB_DEALER_PER_GATE && dealer != HB_DEALER_SHARED_MASK)) return 0;
    const uint64_t w = (uint64_t)(m - k), R = (uint64_t)rounds_of((int)w);
    // gate 0 opens 2w bits; a prefix round opens 4w, or 3w when its two gates share the mask of P
    const uint64_t per_round = dealer == HB_DEALER_SHARED_MASK ? 3 * w : 4 * w;
    const uint64_t per = 2 * w + per_round * R + 1 + (relu ? 128 : 0);
    return (uint64_t)n * per;
}

uint64_t hb_opened_bits_mp(int relu, int parties, int k, int m, size_t n)
{
    if (!valid_slice(k, m) || parties < 2 || parties > hb::kMaxParties) return 0;
    const uint64_t w = (uint64_t)(m - k), R = (uint64_t)rounds_of((int)w);
    // per link and direction: parties - 1 adders of 1 + 2R gates, each opening 2w bits
    return (uint64_t)n * ((uint64_t)(parties - 1) * 2 * w * (1 + 2 * R) + 1 + (relu ? 128 : 0));
}

const char *hb_strerror(int status)
{
    switch (status) {
    case HB_OK: return "success";
    case HB_EINVAL: return "invalid argument (null pointer, bad (k, m), size, overlap, or not device memory)";
    case HB_EALIGN: return "pointer is not 8-byte aligned";
    case HB_EHIP: return "HIP runtime error (see hb_last_hip_error)";
    case HB_ENOTSUP: return "no kernel for this slice width in this entry point";
    case HB_ETOOBIG: return "the call needs more workspace than the library's static array holds";
    default: return "unknown status";
    }
}

const char *hb_last_hip_error(void) { return g_hip_error; }

}  // extern "C"
