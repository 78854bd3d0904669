// Which kernel a call of attn_fwd() goes to and how its work is cut up: plain host arithmetic on sizes, without a device
// and without HIP, so that it can be compiled and checked on its own.
#ifndef PAPER_2603_24517_ATTN_ROUTE_H
#define PAPER_2603_24517_ATTN_ROUTE_H

#include <stdint.h>

#include "../../include/attn.h"

// ATTN_SMALL_PATH: which launches go to the split-key kernel for small problems: 1 (shipped) those whose 256-row work items would occupy at most a quarter of the compute
// units and those of few query rows; 0 none; 2 all.
#ifndef ATTN_SMALL_PATH
#define ATTN_SMALL_PATH 1
#endif
// ATTN_SHARE: which launches of the 256-row kernel share items among workgroups: 1 (shipped) those that it makes
// shorter; 0 none; 2 all that the device memory for it can serve.
#ifndef ATTN_SHARE
#define ATTN_SHARE 1
#endif
// ATTN_ROWS: which calls of the 256-row kernel go to the kernel with workgroups of four wavefronts instead: 1 (shipped, unless
// one of the switches above asks for a certain kernel) those that it makes shorter; 0 none; 2 all, in items of 128 rows; 3 all, in items of 64.
#ifndef ATTN_ROWS
#define ATTN_ROWS (ATTN_SMALL_PATH == 1 && ATTN_SHARE == 1)
#endif

namespace attn {
namespace {        // (nothing of it is exported by the library)

constexpr int HD = 128;              // head dimension
constexpr int BN = 64;               // keys per K/V block
constexpr int NWAVES = 8;            // wavefronts per workgroup; one workgroup fills a CU (registers and LDS)
constexpr int NTHREADS = NWAVES * 64;
constexpr int WG_ROWS = NWAVES * 32; // query rows per workgroup
constexpr int64_t MAX_WGS = UINT32_MAX / NTHREADS;      // a launch has fewer than 2^32 threads
constexpr int SPLIT_KEYS = 32;                                  // keys per block of the split kernel

// Exact n / d for 0 <= n < 2^31 as a multiply-high, an add and a shift.
struct Div { uint32_t mul, shift; };
inline Div make_div(uint32_t d) {
    Div r;
    r.shift = 0;
    while ((1u << r.shift) < d) ++r.shift;
    r.mul = (uint32_t)((((uint64_t)1 << 32) * (((uint64_t)1 << r.shift) - d)) / d + 1);
    return r;
}

// How the work items are dealt out (read by the per-item code only).
struct Sched {
    int total;      // work items = B * Hkv * chunks * ntile
    int per_xcd;    // entries in the work list of one XCD (non-causal: ceil(total / 8))
    int slots;      // workgroups per XCD in this launch (one per CU); the grid is 8 * slots
    int ntile;      // ceil(Sq / tile_pos)
    // causal only: how the (group, tile) pairs are dealt to the XCDs (a group = one batch entry, K/V head and chunk)
    int split;      // every group is cut into `split` sub-groups (a power of two), sub-group r holding the tiles t = r (mod split)
    int split_log2;
    int nsub;       // tiles per sub-group = ceil(ntile / split); the padding entries are skipped
    int sgx;        // sub-groups per XCD = groups * split / 8
    int window;     // sub-groups that one XCD works through together, longest tiles of all of them first
    int per_win;    // window * nsub
    Div d_ntile, d_per_win, d_window;
};
// How the work items are shared (SHARED kernels only).  The items stand in a line, (group, tile) with tiles
// fastest, each as long as its key blocks plus `extra`, and workgroup w takes what lies between cut(w) and
// cut(w + 1), cut(w) = w * total / wgs, moved to an item's end or start where it would leave a part of fewer than
// SHARE_MIN_PART blocks.
struct Share {
    int total;      // length of the line; total * wgs < 2^31
    int wgs;        // workgroups of the launch (a multiple of 8); total / wgs >= extra + 2 SHARE_MIN_PART - 1, so that each has a part
    int groups;     // B * Hkv * chunks
    int group_len;  // total / groups
    int extra;      // what an item costs beside its blocks, in blocks
    int units;      // POOL_UNIT_BYTES units of device memory
};
constexpr int SHARE_MIN_PART = 2;
// Beside its blocks an item costs about 8400 cycles (a block: 2560), and under the causal mask four masked blocks
// of 1300 cycles more each, not all of which the cut falls on.
constexpr int SHARE_EXTRA = 3, SHARE_EXTRA_CAUSAL = 5;
// Tensor shape and head packing (read by the per-item code only).
struct Shape {
    int Sq, Hq;
    int G;          // Hq / Hkv
    int pack;       // query heads of one K/V group served by one workgroup (1, 2, 4 or 8)
    int pack_log2;
    int tile_pos;   // query positions per workgroup = WG_ROWS / pack
    int chunks;     // G / pack
    Div d_chunks, d_hkv;
};
// How the split-key kernel's work is cut up.
struct Split {
    int tile_pos;           // query positions per work item = 32 / pack
    int ntile;              // ceil(Sq / tile_pos)
    int nrest;              // B * Hkv * chunks; items = ntile * nrest
    int splits;             // workgroups that share an item
    int units;              // POOL_UNIT_BYTES units of device memory, 0 if splits == 1
    bool once;              // K and V are each read by one work item, and are more than the last cache holds
    bool once_region;       // the launch reads them past the caches where it has the region, too
};

// Device memory for partial results (g_pool of the kernels): sizes of its units, and of what a launch keeps there.
constexpr int POOL_UNITS = 64;
constexpr uint32_t POOL_UNIT_BYTES = 4u << 20;
constexpr int SPLIT_MAX_ITEMS = 1023;               // of a launch with splits > 1
constexpr int SPLIT_MAX_WGS = 2048;                 // items * splits of such a launch
constexpr int SPLIT_PART_BYTES = 32 * HD * 4 + 3 * 32 * 4;          // one partial result: accumulator, m, l, lr
constexpr uint32_t SPLIT_HEADER_BYTES = 4096;       // at the start of a run: [0] finished items, [1 + item] workgroups that arrived
constexpr int SPLIT_MAX_UNITS = (SPLIT_HEADER_BYTES + SPLIT_MAX_WGS * SPLIT_PART_BYTES + POOL_UNIT_BYTES - 1) / POOL_UNIT_BYTES;
static_assert((1 + SPLIT_MAX_ITEMS) * 4 <= SPLIT_HEADER_BYTES, "header holds a counter per item");
static_assert(SPLIT_MAX_UNITS <= POOL_UNITS / 4, "several launches fit the pool");
// 256-row kernel: a wavefront's part is its accumulator, then m, l, lr, as 17 16-byte pieces per lane.
constexpr uint32_t SHARE_WAVE_BYTES = 17 * 64 * 16;
constexpr uint32_t SHARE_SLOT_BYTES = NWAVES * SHARE_WAVE_BYTES;    // 136 KiB: one part of an item
constexpr uint32_t SHARE_HEADER_BYTES = 64 * 1024;  // [0] workgroups that left, [1 + 8 item + wave] parts that arrived
constexpr int SHARE_MAX_ITEMS = 2047;
constexpr int SHARE_MAX_WGS = 256;                  // two slots each at most: one that starts with its item, one that does not
constexpr int SHARE_MAX_UNITS = (SHARE_HEADER_BYTES + 2 * SHARE_MAX_WGS * SHARE_SLOT_BYTES + POOL_UNIT_BYTES - 1) / POOL_UNIT_BYTES;
static_assert((1 + SHARE_MAX_ITEMS * NWAVES) * 4 <= SHARE_HEADER_BYTES, "header holds a counter per item and wavefront");
static_assert(SHARE_MAX_UNITS <= POOL_UNITS / 3, "several launches fit the pool");
// Behind the pool: the region of the device's null stream.  Its launches follow one another, whoever makes them, so that each finds the region
// free, and its counters zero, as every launch leaves them.  Each kernel has a part of it to itself, because where one has counters the other has
// results.
constexpr int REGION_UNITS = SHARE_MAX_UNITS + SPLIT_MAX_UNITS;
constexpr uint32_t REGION_SHARE_UNIT = POOL_UNITS, REGION_SPLIT_UNIT = POOL_UNITS + SHARE_MAX_UNITS;       // first units
// Whether a launch's counters are set back to zero by whoever takes them to their last value.  Those of the region are: the end of the launch
// comes between that store and the next launch's first count.  Units of the pool belong to another launch as soon as they are given back, which
// nothing orders behind such a store, so that a late one would erase arrivals of that launch; the launch in front clears theirs.
constexpr bool sets_counters_back(uint32_t unit) { return unit >= (uint32_t)POOL_UNITS; }

// How the work of the kernel with workgroups of four wavefronts is cut up: items of 128 / kgroups rows, whose keys are shared by
// `kgroups` groups of wavefronts.
struct Rows {
    int kgroups;            // 1 or 2; 0 if the call is not this kernel's
    int tile_pos;           // query positions per work item = 128 / kgroups / pack
    int ntile;              // ceil(Sq / tile_pos)
    int nrest;              // B * Hkv * chunks; items = ntile * nrest
    // The workgroups run through windows of `window` of these nrest, tiles slowest, last tile first: enough of them that about as many
    // workgroups as run at a time (64 per XCD) read the same few K/V heads.  (window a multiple of 8: a K/V head's tiles are on one XCD.)
    // The first window is the one that may hold fewer, so that the launch ends with short tiles.
    int window, window0;
};
constexpr int ROWS_WAVES = 4;

enum RouteKind { ROUTE_WHOLE, ROUTE_SHARED, ROUTE_SPLIT };     // whole items of 256 rows (or of Rows), shared ones, split-key kernel
struct Route {
    RouteKind kind;
    int Skv;
    Shape shape;
    Sched sched;
    Share share;
    Split split;
    Rows rows;
};

// Key blocks of 64 of a 256-row item, as the kernel counts them.
inline int item_blocks(const Route &p, bool causal, int tile)
{
    const int n = (p.Skv + BN - 1) / BN;
    if (!causal) return n;
    const int end = tile * p.shape.tile_pos + p.shape.tile_pos;
    const int klast = (end < p.shape.Sq ? end : p.shape.Sq) - 1 + p.Skv - p.shape.Sq;
    return klast < 0 ? 0 : klast / BN + 1 < n ? klast / BN + 1 : n;
}
// What the longest workgroup of a launch of whole items takes, in blocks with `extra` for each item; the XCDs are dealt
// alike, and none more than the first.
inline int whole_items_length(const Route &p, bool causal, int extra)
{
    const Sched &sc = p.sched;
    if (!causal) return (sc.per_xcd + sc.slots - 1) / sc.slots * (item_blocks(p, false, 0) + extra);
    int longest = 0;
    for (int slot = 0; slot < sc.slots; ++slot) {
        int sum = 0;
        for (int r = 0; r * sc.slots < sc.per_xcd; ++r) {
            const int j = r * sc.slots + ((r & 1) ? sc.slots - 1 - slot : slot);
            if (j >= sc.per_xcd) continue;
            const int w = j / sc.per_win, i = j - w * sc.per_win;
            const int kw = sc.window < sc.sgx - w * sc.window ? sc.window : sc.sgx - w * sc.window;
            const int tile_r = i / kw * sc.split + ((w * sc.window + i % kw) & (sc.split - 1));
            if (tile_r < sc.ntile) sum += item_blocks(p, true, sc.ntile - 1 - tile_r) + extra;
        }
        longest = sum > longest ? sum : longest;
    }
    return longest;
}

// Workgroups that share one item of the split-key kernel, whose key sequence is `blocks` blocks of 32 keys.
// One workgroup takes about 5 us + 1.3 us per 8 blocks as long as memory keeps up (measured, 8 items: 7.0 us at 16 blocks,
// 15.0 at 64, 43 at 256, 189 at 1024); sharing an item adds about 4 us for the launch in front (which the null stream does not
// have; the number of parts, and with it a call's bits, is the same on every stream) and
// 0.25 us per part to merge, so the sum is least at parts^2 = 0.65 blocks (measured, 8 items: 64 blocks 12.5 us
// with 4 parts, 12.8 with 8; 256 blocks 17.4 with 8 or 16, 20.1 with 24; 1024 blocks 32.9 with 16, 36.2 with 32).
// More workgroups than compute units start a second round: 160 items in two parts 26.5 us, in one 16.2.
//
// From how many blocks on it pays depends on where K and V come from, which more workgroups read faster from HBM.  One
// part / shared, us, K and V from HBM (from the last cache, where a repeated call finds them): 8 items of 40 blocks
// 16.6 / 13.5 (10.9 / 12.0); 64 of 40 18.6 / 16.7 (12.9 / 15.6); 80 of 41 19.4 / 18.5 (13.4 / 17.2); 128, in two parts, of 40
// 20.7 / 22.5 (16.3 / 20.7), of 54 27.2 / 27.0, of 66 32.0 / 30.9 (24.2 / 27.1).  Many tiles of a sequence read the same keys,
// which then come from a cache either way: 13 tiles, 52 items of 54 blocks 14.5 / 15.2 (13.9 / 14.7), of 66 18.8 / 16.7
// (15.5 / 15.3); 7 tiles, 84 items of 66 21.5 / 17.9 (15.4 / 16.3); 22 tiles, 88 items of 66 18.1 / 18.3 (15.4 / 16.4), of 82
// 22.6 / 20.8.
inline int split_parts(int64_t items, int ntile, int blocks, int ncu)
{
    const bool many = items * 3 > ncu;          // at most two parts
    if (items > ncu || blocks < (ntile > 2 ? (many ? 82 : 66) : (many ? 54 : 40))) return 1;
    int s = 1;
    while ((s + 1) * items <= (ncu < 512 ? ncu : 512) && 5 * (s + 1) * (s + 1) <= 2 * blocks) ++s;
    return s;
}

// The same for more items than half of the compute units, which are too many for one round of parts, where K and V come from memory: several
// rounds of shorter workgroups, where whole items leave part of a round empty.  A full round reads 6.64 TB/s, a compute unit by itself
// at most 1.47 times its share of that, a workgroup costs about six blocks beside its own, and the launch in front or the merge five.  (One row, whole items /
// in parts, us: 16384 keys, 144 items 220.2 / 203.5; 264 487.1 / 358.3; 272 492.7 / 370.0; 384 535.3 / 486.0; but 1000 keys, 320 items
// 36.3 / 39.7, and 1500 keys, 280 items, with a launch in front 52.9 / 55.3.)
inline int split_rounds(int64_t items, int blocks, int ncu)
{
    auto cost = [&](int s) {
        const int64_t wgs = items * s, rest = wgs % ncu;
        const double last = rest == 0 ? 0 : (double)rest / ncu > 0.68 ? (double)rest / ncu : 0.68;
        return ((blocks + s - 1) / s + 6) * ((double)(wgs / ncu) + last) + (s > 1 ? 5 : 0);
    };
    int best = 1;
    if (items * 2 <= ncu || items > SPLIT_MAX_ITEMS) return best;
    for (int s = 2; s <= 16 && items * s <= SPLIT_MAX_WGS && blocks >= 16 * s; ++s)
        if (cost(s) < (best == 1 ? 0.95 : 1.0) * cost(best)) best = s;
    return best;
}

// Estimates, in ns, of the three ways to run a launch; they only choose among them.  Measured (us, whole items or split-key
// kernel / shared): 128 items x 32 blocks 42.5 / 42.5, 192 x 24 45.3 / 55.0, 400 x 19 68.7 / 75.4, 576 x 47 229.6 / 208.1, 128 x 128
// 150 / 124; causal: 128 items, 2048 x 2048 43.5 / 37.0; 256, 16384 x 16384 324 / 248; 384, 3000 x 3000 82.0 / 86.1; 640, 5000 x 5000
// 220 / 203; 512, 32768 x 32768 889 / 899; split-key: 64 items, 512 x 16384 234 / 140; 48, 700 x 20000 224 / 123; 64, 4096 x 4096 (not
// causal) 60.7 / 49.7; 32, 200 x 8000 48.8 / 52.6; 8, 64 x 30000 57.3 / 87.9.
//
// Shared: the chip is full and at the clock that goes with it; 17 us for the parts and the launch in front, 1 us for each
// part of an item beyond the second.  (The null stream has no launch in front and takes 3 to 5 us less; one estimate for all streams, so that a call's bits
// do not depend on its stream.)
inline int64_t shared_ns(const Route &p, int64_t items)
{
    const Share &sr = p.share;
    const int64_t more = sr.wgs / items > 1 ? sr.wgs / items - 2 : 0;
    return 17000 + 1650 * (int64_t)sr.total / sr.wgs + 1000 * more;
}
// Whole items: a block takes 1.15 us where half of the chip idles and leaves its power to the other half, 1.55 where three
// quarters are busy.
inline int64_t whole_items_ns(const Route &p, bool causal)
{
    const Share &sr = p.share;
    const int64_t longest = whole_items_length(p, causal, sr.extra);
    const int64_t busy = 1000 * (int64_t)sr.total / (sr.wgs * longest);     // per mille
    const int64_t over = busy < 500 ? 0 : busy > 750 ? 250 : busy - 500;
    return (1150 + over * 400 / 250) * longest;
}
// Split-key kernel: as at split_parts.
inline int64_t split_ns(int64_t items, int ntile, int64_t blocks, int ncu)
{
    const int parts = split_parts(items, ntile, (int)blocks, ncu);
    const int64_t rounds = (items * parts + ncu - 1) / ncu;
    return (5000 + 163 * blocks / parts) * rounds + (parts > 1 ? 4000 + 250 * parts : 0);
}

constexpr int64_t LAST_CACHE_BYTES = 256ll << 20;       // of an MI355X

// Whole items of 256 rows against items of 128 and 64 rows in workgroups of half the size: estimates, in us, fitted to 680 calls (4 to
// 9500 items of 128 rows, 3 to 22000 keys, masked and not; 9 of 10 estimates are within 15 % of what was measured, K and V in the last cache).  How far
// ahead the smaller workgroups have to be stands where they are compared.  Measured (us, 256 rows /
// 128 / 64): causal: 1 x 1111, 32 heads on 8 29.5 / 21.4 / 17.7; 24 x 200, 16 heads 25.3 / 20.0 / 21.2; 300 x 150, 4 heads 64 / 47 / 50; 1 x
// 2000, 16 heads 37.9 / 31.3 / 27.1; 11 x 3694, 4 heads 168 / 156 / 177; 8 x 4096, 16 heads 497 / 530 / 658; no mask: 5 x 1200, 4 heads 30.6
// / 23.3 / 23.0; 2 x 1500, 16 heads 41.7 / 44.0 / 46.5; 42 x 145, 40 heads 77 / 57 / 65.
struct Lengths {
    int Sq, Skv;
    bool causal;
    // blocks of `unit` keys in all tiles of `pos` positions of one head together
    double blocks(int pos, int ntile, int unit) const
    {
        if (!causal) return (double)ntile * ((Skv + unit - 1) / unit);
        // tile t ends with the key of position (t + 1) pos, the last one with Skv; with more rows than keys the first ones have none
        const double off = (double)Skv - Sq;
        const int first = off < 0 ? (int)(-off / pos) : 0, tiles = ntile - first;
        const double ends = tiles * ((first + 1.0 + ntile) * pos * 0.5 + off) - (ntile * (double)pos - Sq);
        return ends / unit + 0.5 * tiles;
    }
};
inline double clamp01(double x) { return x < 0 ? 0 : x > 1 ? 1 : x; }
// One workgroup of eight wavefronts per compute unit, one item after the other.
inline double rows256_us(const Route &p, const Lengths &ln, int ncu, double bytes)
{
    const Sched &sc = p.sched;
    const int groups = p.share.groups, per = item_blocks(p, false, 0);
    // what an item costs beside its blocks, in blocks; an item of fewer than four does not load the next one's tiles
    const double extra = ln.causal ? SHARE_EXTRA_CAUSAL : per < 4 ? 4.4 : SHARE_EXTRA;
    const double all = groups * ln.blocks(p.shape.tile_pos, sc.ntile, BN) + extra * sc.total;
    double longest = all / (8 * sc.slots) * 1.02;       // (many items: none ends much later than the others)
    if (!ln.causal) longest = (sc.per_xcd + sc.slots - 1) / sc.slots * (per + extra);
    else if (sc.total <= 4 * ncu) longest = whole_items_length(p, true, SHARE_EXTRA_CAUSAL);
    const double busy = all / (ncu * longest);
    const double t = longest * (1.149 + 0.026 * clamp01((busy - 0.5) * 4));
    const double us = t * (1 + 0.27 * clamp01(t / 80) * busy);        // (a full chip lowers its clock)
    return 3.5 + (us > bytes * 0.222e-6 ? us : bytes * 0.222e-6);
}
// Two workgroups of four wavefronts per compute unit.
inline double rows_us(const Route &p, const Lengths &ln, int kgroups, int ncu, double bytes, bool cached)
{
    struct Fit { double start, extra, alone, pair, tail, clock, byte, cold; };
    // us: of a launch; turns that an item costs beside its own; of a turn where one or two workgroups are on a compute unit
    static const Fit fits[2] = {{2.99, 6.85, 0.398, 0.731, 0.276, 0.161, 0.181e-6, 0.15}, {2.51, 3.68, 0.538, 0.874, 0.253, 0.133, 0.204e-6, 0.71}};
    const Fit &f = fits[kgroups - 1];
    const int pos = 128 / kgroups / p.shape.pack, ntile = (ln.Sq + pos - 1) / pos;
    const double items = (double)p.share.groups * ntile;
    const double most = (ln.Skv + SPLIT_KEYS * kgroups - 1) / (SPLIT_KEYS * kgroups) + f.extra;
    const double all = p.share.groups * ln.blocks(pos, ntile, SPLIT_KEYS * kgroups) + f.extra * items;
    // the longest item, beside another one for as long as there are others; without a mask the rounds of equal ones
    const double others = all / (2 * ncu) / most, beside = items / ncu - 1;
    double longest = most * (f.alone + (f.pair - f.alone) * clamp01(others < beside ? others : beside));
    if (!ln.causal) {
        const int rounds = (int)(items / (2 * ncu));
        const double rest = items - 2.0 * ncu * rounds;
        longest = rounds < 3 ? most * (rounds * f.pair + (rest == 0 ? 0 : rest <= ncu ? f.alone : f.pair)) : 0;
    }
    if (!cached) longest *= 1 + f.cold;
    double t = all / (2 * ncu) * f.pair;
    t = t * (1 + f.clock * clamp01(t / 80)) + f.tail * most * f.alone;
    const double us = longest > t ? longest : t;
    return f.start + (us > bytes * f.byte ? us : bytes * f.byte);
}

// Sizes as attn_fwd() takes them, all positive: what the kernels' index arithmetic holds.  Returns a code of include/attn.h
// (and, if that is ATTN_OK, the shape).
inline int make_shape(int B, int Hq, int Hkv, int Sq, int Skv, Shape &sh, Sched &sc)
{
    // Key/query indices and the work-item count are 32-bit in the kernel (and below 2^31 for the divisions).
    if ((int64_t)Sq + Skv + WG_ROWS + 8 * BN >= INT32_MAX) return ATTN_E_UNSUPPORTED;
    // Byte offsets within one tile (rows x row pitch) are 32-bit in the kernel.
    if (Hq > 32768 || Hkv > 32768) return ATTN_E_UNSUPPORTED;
    sh.Sq = Sq; sh.Hq = Hq;
    sh.G = Hq / Hkv;
    sh.pack = (sh.G % 8 == 0) ? 8 : (sh.G % 4 == 0) ? 4 : (sh.G % 2 == 0) ? 2 : 1;
    sh.pack_log2 = sh.pack == 8 ? 3 : sh.pack == 4 ? 2 : sh.pack == 2 ? 1 : 0;
    sh.tile_pos = WG_ROWS / sh.pack;
    sh.chunks = sh.G / sh.pack;
    sh.d_chunks = make_div((uint32_t)sh.chunks);
    sh.d_hkv = make_div((uint32_t)Hkv);
    sc.ntile = (Sq + sh.tile_pos - 1) / sh.tile_pos;
    const int64_t total = (int64_t)B * Hkv * sh.chunks * sc.ntile;
    if (total + 8 >= INT32_MAX / 16) return ATTN_E_UNSUPPORTED;
    sc.total = (int)total;
    return ATTN_OK;
}

// The route of a call whose shape make_shape() has accepted, on a device of ncu compute units.
inline void make_route(int B, int Hkv, int Skv, int causal, int ncu, Route &p)
{
    Shape &sh = p.shape;
    Sched &sc = p.sched;
    const int Sq = sh.Sq;
    const int64_t total = sc.total;
    p.Skv = Skv;

    const int cu_slots = ncu >= 8 ? ncu / 8 : 1;
    // One workgroup per CU (a workgroup takes all of a CU's registers and LDS), each working through a list.
    sc.per_xcd = (int)((total + 7) / 8);
    sc.split = sc.nsub = sc.sgx = sc.window = 1;
    sc.split_log2 = 0;
    if (causal) {
        const int64_t groups = (int64_t)B * Hkv * sh.chunks;
        while ((groups * sc.split) % 8 != 0) { sc.split *= 2; ++sc.split_log2; }    // 1, 2, 4 or 8
        sc.nsub = (sc.ntile + sc.split - 1) / sc.split;
        sc.sgx = (int)(groups * sc.split / 8);
        while (sc.window * 2 <= sc.sgx && sc.window * sc.nsub < cu_slots) sc.window *= 2;
        sc.per_xcd = sc.sgx * sc.nsub;          // <= total + padding, far below 2^31 after the check above
    }
    sc.per_win = sc.window * sc.nsub;
    sc.d_ntile = make_div((uint32_t)sc.ntile);
    sc.d_per_win = make_div((uint32_t)sc.per_win);
    sc.d_window = make_div((uint32_t)sc.window);
    sc.slots = sc.per_xcd < cu_slots ? sc.per_xcd : cu_slots;

    const int split_tile_pos = 32 / sh.pack;
    const int split_ntile = (Sq + split_tile_pos - 1) / split_tile_pos;
    const int64_t split_items = (int64_t)B * Hkv * sh.chunks * split_ntile;
    // The same work as a line cut into equal stretches.  From 4 items per compute unit on, whole items leave at most a fifth of the chip idle at the
    // end, and sharing has not been faster.  (5 %: what the estimates are worth; of 60 calls that they put further ahead, none was
    // slower shared.)
    Share &sr = p.share;
    sr.wgs = 8 * cu_slots;
    sr.groups = (int)((int64_t)B * Hkv * sh.chunks);
    sr.extra = causal ? SHARE_EXTRA_CAUSAL : SHARE_EXTRA;
    bool share = false;
    if (ATTN_SHARE != 0 && total <= (ATTN_SHARE == 2 ? SHARE_MAX_ITEMS : 4 * ncu) && total <= SHARE_MAX_ITEMS && sr.wgs <= SHARE_MAX_WGS) {
        int64_t len = 0;
        for (int t = 0; t < sc.ntile; ++t) len += item_blocks(p, causal, t) + sr.extra;
        const int64_t line = len * sr.groups;
        if (line * sr.wgs < INT32_MAX && line >= 8 * (sr.extra + 2 * SHARE_MIN_PART - 1)) {
            sr.group_len = (int)len;
            sr.total = (int)line;
            const int most = sr.total / (sr.extra + 2 * SHARE_MIN_PART - 1) / 8 * 8;
            if (sr.wgs > most) sr.wgs = most;
            const int64_t slots = sr.wgs + (total < sr.wgs ? total : sr.wgs);
            sr.units = (int)((SHARE_HEADER_BYTES + slots * SHARE_SLOT_BYTES + POOL_UNIT_BYTES - 1) / POOL_UNIT_BYTES);
            const int64_t blocks32 = (Skv + SPLIT_KEYS - 1) / SPLIT_KEYS;
            // (The other way of `few` is the split-key kernel.  Its estimate is low on a full chip, above all where K and V come from memory, and
            // some calls that stay with it would be faster shared: 9 x 26 x 27226, 12 heads on 3 204 us and 112.  They stay because it rounds its
            // weights against eight running maxima per part and a shared item against one: O of these calls was off by 2.25e-3 and 2.34e-3 for N(0,1)
            // scores, 1.68e-3 and 1.93e-3 for four times that.)
            const bool few = total * 4 <= ncu && ATTN_SMALL_PATH == 1;
            const int64_t whole = few ? split_ns(split_items, split_ntile, blocks32, ncu) : whole_items_ns(p, causal != 0);
            // Whole items that run at once walk through the keys of a group together, and one of them brings a block into the
            // XCD's L2 for all.  Stretches of the line do not, which tells when K and V are larger than the last cache: 9 x 571 x
            // 33965, 16 heads (2.5 GB), estimated 10 % faster shared, whole 1669, shared 1821; 20 x 281 x 25757 (4.2 GB), 12 %, 1912 and 2014;
            // 13 x 1975 x 14973, 4 heads (0.4 GB), 14 %, 693 and 705; 12 x 221 x 9026 (0.9 GB), 15 %, 248 and 232.
            const bool cached = (int64_t)B * Hkv * Skv * HD * 4 <= LAST_CACHE_BYTES;
            share = ATTN_SHARE == 2 || shared_ns(p, total) * (few || cached ? 105 : 114) < whole * 100;
        }
    }

    // Small problems: few 256-row items would leave most compute units idle, and items of few rows (the
    // query heads of one group times the positions of the sequence) most of each item's rows; 32-row items whose keys
    // are shared out among the wavefronts of a workgroup, and among workgroups, fill the device instead.
    // Few rows, measured, 256-row / split-key kernel, us: 4 rows x 4000 keys, 128 items 77.9 / 42.4; 4 x 4096, 512 items
    // 248.3 / 191.7 (1.07 GB of K and V); 4 x 500, 512 items 35.6 / 24.1; 1 x 8000, 256 items 232.9 / 175.2.
    // More than 32 of them are two tiles, which read the same keys.  That pays while all tiles run at once, and while the keys
    // are few enough for the second tile to find them in a cache, where 256-row items leave much of a round empty: up to three
    // quarters of the compute units' number of them, and from one to five quarters (six, for very few keys).  64 rows x 5000,
    // 256 tiles 93.2 / 70.1; 288 tiles, x 1500 40.1 / 36.1, x 5000 105.9 / 115.0, x 16000 292 / 386; 384 tiles, x 400 20.3 / 17.1,
    // x 1500 47.0 / 44.9, x 5000 131.6 / 158.5; 512 tiles, x 1500 55.2 / 65.6; 544 .. 640 tiles, x 250 24.8 / 20.3, x 1000 57.0 /
    // 51.2, x 1500 78.5 / 73.0, x 2048 96.4 / 110.4; 672 tiles, x 354 30.2 / 25.3; 704, x 715 46.1 / 42.7; 768, x 1000 58.0 / 59.5;
    // 56 rows, 1024 tiles, x 4096 257 / 381.
    const int64_t rows = (int64_t)Sq * sh.pack;
    const bool few_rows = rows <= 32 || (rows <= 64 && (total * 2 <= ncu || (total * 4 <= 3 * ncu && Skv <= 2048) ||
                                                        (total > ncu && total * 4 <= 5 * ncu && Skv <= 1536) ||
                                                        (total > ncu && total * 2 <= 3 * ncu && Skv <= 768)));
    const bool small = ATTN_SMALL_PATH == 2 || (ATTN_SMALL_PATH == 1 && ((total * 4 <= ncu && !share) || few_rows));
    p.kind = share ? ROUTE_SHARED : ROUTE_WHOLE;
    // Loads past the caches (nt) get 7.0 TB/s from HBM on this card, ordinary ones 6.1 (a kernel that only reads); but then a call that is repeated
    // does not find K and V in the last cache, and several items of a K/V head not in an L2: 2 x 16 x 8192, 64 heads on 8, four items 26.0 us
    // and 34.3.  Where they are read by one item, us, ordinary / past the caches, K and V from memory; repeated: items of one workgroup 18 x 1 x 2000,
    // 32 heads on 8 (147 MB) 32.4 / 31.0; 25.9 / 30.2; 9 x 7 x 3200, 16 heads (236 MB) 50.6 / 47.6; 38.7 / 47.1; 280 MB 58.4 / 55.3; 49.3 / 53.5; 299 MB 63.7 /
    // 59.8; 58.5 / 59.1; 306 MB 64.1 / 60.7; 61.4 / 59.9; 328 MB 64.6 / 60.3; 62.9 / 59.4: from nine eighths of the last cache on, nothing is lost.  Shared items
    // 1 x 1 x 32768 (134 MB) 36.1 / 34.5; 31.0 / 33.4; 14 x 1 x 4000 (229 MB) 44.1 / 40.6; 37.5 / 39.6; 16 x 1 x 4000 (262 MB) 48.8 / 44.8; 43.0 / 43.9; 4 x 1 x
    // 4096 (67 MB) 20.0 / 18.6; 17.3 / 16.9; 1 x 1 x 8192 (34 MB, six calls' K and V in turn fit the cache) 15.3 / 18.4.  On the null stream they go past the
    // caches from a quarter on: with no launch in front a repeated call takes no longer than it does on another stream with ordinary loads (33.8, 40.0, 45.3,
    // 20.1; of 150 calls measured one group was slower, 3600 keys, 236 MB, 4 K/V heads: repeated 44.6 / 40.4, from memory 43.0 / 50.8).  On other streams it would
    // take up to 2.6 us more than that.
    const int64_t kv_bytes = (int64_t)B * Hkv * Skv * HD * 4;
    const bool read_once = split_ntile == 1 && sh.chunks == 1;
    const int split_blocks = (Skv + SPLIT_KEYS - 1) / SPLIT_KEYS;
    int splits = split_parts(split_items, split_ntile, split_blocks, ncu);
    const bool shared_once = splits > 1 && read_once && kv_bytes >= LAST_CACHE_BYTES / 4;
    // Rounds of parts pay from memory only, and on other streams a little later, as they have a launch in front (us, whole items / rounds, from memory;
    // repeated: 317 MB, 18 x 1 x 4300 64.7 / 62.4; 59.7 / 61.8; 410 MB, 40 x 1 x 2500 88.4 / 81.5; 88.3 / 81.1).
    if (splits == 1 && read_once && 3 * kv_bytes >= 4 * LAST_CACHE_BYTES) splits = split_rounds(split_items, split_blocks, ncu);
    if (small && split_items * splits <= MAX_WGS) {
        Split &sp = p.split;
        p.kind = ROUTE_SPLIT;
        sp.tile_pos = split_tile_pos;
        sp.ntile = split_ntile;
        sp.nrest = sr.groups;
        sp.splits = splits;
        sp.once = read_once && 8 * kv_bytes >= 9 * LAST_CACHE_BYTES;
        sp.once_region = shared_once;
        if (sp.splits > 1)
            sp.units = (int)((SPLIT_HEADER_BYTES + split_items * sp.splits * SPLIT_PART_BYTES + POOL_UNIT_BYTES - 1) / POOL_UNIT_BYTES);
    }

    // What is left may be faster in smaller workgroups.  (Not what the split-key kernel gets, for the same reason as above: its results are
    // closer to the exact ones.)
    Rows &rw = p.rows;
    rw.kgroups = 0;
    if (ATTN_ROWS != 0 && (ATTN_ROWS != 1 || p.kind != ROUTE_SPLIT)) {
        int kgroups = ATTN_ROWS == 2 ? 1 : ATTN_ROWS == 3 ? 2 : 0;
        if (ATTN_ROWS == 1) {
            const Lengths ln = {Sq, Skv, causal != 0};
            const double kv = (double)B * Hkv * Skv * HD * 4, bytes = kv + (double)B * Hkv * sh.G * Sq * HD * 4;
            const bool cached = kv <= (double)LAST_CACHE_BYTES;
            const double r1 = rows_us(p, ln, 1, ncu, bytes, cached), r2 = rows_us(p, ln, 2, ncu, bytes, cached);
            // How far ahead the smaller workgroups have to be estimated, so that calls are not slower there than in 256-row items, with K and V in the
            // last cache or from memory.  6 % (shared items: 10 to 15) were not enough: of 1020 measured calls that went there, 44 were more than 2 %
            // slower one way or the other.  Chosen on 5000 calls:
            // - Keys more than twice as long as the rows: each tile reads them again, and the two stages of items of 64 rows do not cover reads from
            //   memory, which the estimates do not know (us, 256 rows / smaller, from memory: 2 x 104 x 5599, 64 heads on 8 58.1 / 90.7; 4 x 35 x
            //   4426 48.6 / 74.7; 4 x 264 x 3506, 32 on 4 73.2 / 81.1; 20 x 269 x 2017, 12 on 3 80.9 / 86.6; 9 x 517 x 4612, 6 on 2 97.3 / 106.9).
            // - More rows than keys, masked: most rows have no key, which neither estimate knows well (4 x 1607 x 63, 16 heads 11.3 / 11.8).
            // - From one and a half rounds of 256-row items on, these leave little idle, and where each K/V head has one query head and at most three tiles
            //   (768 rows) both ways are mostly memory: of 131 calls put 6 to 25 % ahead 33 were slower, up to 19 % (22 x 391, 40 heads, masked 105.7 /
            //   120.1; 162 x 221, 4 heads 40.6 / 48.1), of 269 further ahead none.  Above nine rounds 22 of 118 others put 6 to 18 % ahead were slower, up to 6 %
            //   (208 x 315, 12 on 3, masked 141 / 146; 57 x 694, 32 on 8 323 / 336), of 186 further ahead none.
            // - Others are asked for 11 %: of 353 put 6 to 10 % ahead 6 were slower, up to 7 % (4 x 592 x 814, 32 on 4, masked 30.2 / 32.5), of 2439 further
            //   ahead 5 (64 x 64, 32 on 8, no mask 20.4 / 22.4; the others by 1 to 4 %).
            // - Other calls of shared items against items of 64 rows: 21 % ahead, 2 x 2300, 4 heads 32.9 / 35.0; 1 x 3222, 16 heads 58.1 / 59.5.
            const bool far = Skv > 2 * (int64_t)Sq, is_shared = p.kind == ROUTE_SHARED;
            const int best = r1 < r2 || (far && is_shared) ? 1 : 2;
            const double now = is_shared ? shared_ns(p, total) * 1e-3 : rows256_us(p, ln, ncu, bytes);
            const double ahead = is_shared ? (far ? 0.78 : best == 2 ? 0.80 : now < 80 ? 1 / 1.10 : 1 / 1.15) : far || (causal && Sq > Skv) ? 0.70
                                 : 2 * (int64_t)total > 3 * ncu && sh.pack == 1 && Sq <= 768 ? 0.80 : total > 9 * ncu ? 0.85 : 0.90;
            if ((best == 1 ? r1 : r2) < now * ahead) kgroups = best;
        }
        if (kgroups != 0) {
            const int pos = 128 / kgroups / sh.pack, ntile = (Sq + pos - 1) / pos;
            if ((int64_t)sr.groups * ntile <= MAX_WGS) {
                p.kind = ROUTE_WHOLE;
                rw.kgroups = kgroups;
                rw.tile_pos = pos;
                rw.ntile = ntile;
                rw.nrest = sr.groups;
                rw.window = (2 * cu_slots + ntile - 1) / ntile * 8;
                if (rw.window > rw.nrest) rw.window = rw.nrest;
                rw.window0 = rw.nrest - (rw.nrest - 1) / rw.window * rw.window;
            }
        }
    }
}

// The launches of a call: where items are shared and the stream has no region, one that takes the device memory for the parts stands in
// front of the one that uses it and gives it back, and if that fails, another one gives the memory back (or, if none can be launched any more,
// nothing does).  `go` enqueues a step and says whether the runtime took it.  Returns a code of include/attn.h.
inline bool shares_items(const Route &p) { return p.kind == ROUTE_SHARED || (p.kind == ROUTE_SPLIT && p.split.splits > 1); }
enum Step { STEP_TAKE, STEP_MAIN, STEP_GIVE };
template <class Go>
int enqueue(const Route &p, Go &&go, bool region = false)
{
    const bool takes = shares_items(p) && !region;
    if (takes && !go(STEP_TAKE)) return ATTN_E_LAUNCH;
    if (go(STEP_MAIN)) return ATTN_OK;
    if (takes) (void)go(STEP_GIVE);
    return ATTN_E_LAUNCH;
}

}  // namespace
}  // namespace attn
#endif
