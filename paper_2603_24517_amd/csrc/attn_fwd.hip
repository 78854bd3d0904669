// Fused attention forward for MI355X (gfx950, CDNA4).
//
// Computes O = softmax(Q K^T * scale [+ causal mask]) V and the per-row
// log-sum-exp, tile by tile over key blocks with a running row maximum and
// running row sum (paper section 2.2), for multi-head and grouped-query
// attention (sections 4.1, 4.3).  BF16 operands on MFMA, FP32 accumulation.
//
// Data flow of one wavefront (64 lanes), which owns 32 query rows of one head:
//   * S^T = K Q^T with v_mfma_f32_32x32x16_bf16: A = 32 keys x 16 d read from
//     LDS, B = Q^T held in registers for the whole kernel.  The accumulator
//     layout puts ONE query (lane % 32) in each lane and 16 of the tile's 32
//     keys in its registers, so a row maximum / row sum is 15 in-lane
//     operations plus one exchange between lanes l and l^32.
//   * P is rounded to BF16 in registers and is directly the B operand of
//     O^T = V^T P^T: the contraction slots of each P^T operand are the keys
//     the lane already holds, and V^T is fetched from LDS with the matching
//     key order by the transposing read ds_read_b64_tr_b16.  No LDS round
//     trip and no shuffle for P.
//   * O^T keeps lane = query, so the rescale by alpha and the final 1/l are
//     lane-local multiplies.
//
// A workgroup is 8 wavefronts (256 query rows) sharing one K/V block stream:
// tiles go from global memory straight into three XOR-swizzled LDS stages
// (global_load_lds_dwordx4), requested two iterations before use.  For
// grouped-query attention the 256 rows are PACK heads of one K/V group x
// 256/PACK positions, so one K/V tile in LDS serves several query heads.
//
// The key-block loop is software-pipelined three deep inside every wavefront:
// iteration j issues the MFMAs of O += P(j) V(j) and S(j+2) = K(j+2) Q^T while
// its vector instructions turn S(j+1) into P(j+1).  The two instruction kinds
// are independent within an iteration and are interleaved (one MFMA, its LDS
// reads, a few VALU), so the matrix pipe and the vector ALU run at the same
// time (the paper's section 2.2 describes the same need, met on its hardware
// by specialised warps), with one workgroup barrier per iteration.
//
// The launch has one workgroup per CU, and each works through a list of
// (batch entry, K/V head, query tile) items: while an item is in its last
// blocks it already requests the next item's first K/V tiles into the stages
// that fall free and the next item's Q into the rest of LDS, and O leaves
// through LDS as whole rows, so that the matrix pipe idles for little more
// than one short prologue per item.  The per-iteration overhead of the loop
// (stage rotation, request addresses, LDS address arithmetic) is kept out of
// the instruction stream as far as possible, because with two wavefronts per
// SIMD the issue of vector instructions, not the matrix pipe alone, is what
// an iteration's length follows.
//
// Where whole items would leave compute units without work for long (fewer items than compute units, a last
// round with few of them), the kernel's shared form cuts the line of all items' key blocks into
// stretches of equal length, one for each workgroup; an item that a cut falls into is added up from its parts
// (512 rows against 16384 keys, 32 heads on 8, causal: whole items 215 us, shared 127; one sequence of 16384, 4 heads,
// causal: 309 and 238).
//
// A kernel with workgroups of four wavefronts, two on a compute unit, serves what lies between: calls of too few 256-row items to
// fill the chip evenly, and short sequences (at the end of this file).
//
// Another kernel serves small problems (few query
// rows, however many keys): 32-row work items whose key blocks are shared out
// among the wavefronts of a workgroup and whose partial results are merged
// through LDS.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <math.h>
#include <float.h>
#include <type_traits>
#include <atomic>

#include "../../include/attn.h"
#include "attn_route.h"

// ---- Compile-time variants.  The shipped library defines none of these; each alternative is built
// into a library of its own and goes through the same parity tests, so that the choices below can be
// measured against what they replaced (the paper's sections 5.1 and 5.2 analyse the same two
// decisions on its hardware).
//
// ATTN_SOFTMAX: how the softmax of an unmasked key block treats the running maximum.
//   0  (shipped) probabilities against the running maximum as it stands, no search for the block's
//      maximum; the exact path runs only if a partial row sum leaves the safe range
//   1  block maximum every block, accumulator and row sums multiplied by alpha every block, no branch
//   2  block maximum every block, the multiplication skipped under a wave-uniform vote when no lane's
//      maximum rose
//   3  block maximum every block, the reference raised (and the accumulator rescaled) only where the
//      block maximum exceeds it by more than 8 in log2 units
#ifndef ATTN_SOFTMAX
#define ATTN_SOFTMAX 0
#endif
// ATTN_ITEM_OVERLAP: 1 (shipped) the last blocks of an item request the first tiles and the Q tile of the
// next one; 0 every item loads its own tiles and its Q after the epilogue of the item before.
#ifndef ATTN_ITEM_OVERLAP
#define ATTN_ITEM_OVERLAP 1
#endif
// ATTN_POOL: 1 (shipped); 0 every launch that shares its items among workgroups finds the device memory for their parts in
// use, and takes the path for that case.
#ifndef ATTN_POOL
#define ATTN_POOL 1
#endif
// ATTN_LDS_PREFETCH: how many MFMAs ahead of its consumer an LDS operand fragment is read (shipped: 3).
#ifndef ATTN_LDS_PREFETCH
#define ATTN_LDS_PREFETCH 3
#endif
// ATTN_WAVES_PER_SIMD (shipped: 2): the occupancy the attention kernel is compiled for, i.e. its register
// budget: 512 / n vector registers per wavefront.  3 and 4 are for compile-only builds that show what a
// smaller budget costs in spills (the paper's section 5.3 weighs register budgets on its hardware);
// such builds are not meant to be run (see wait_vmcnt below for what a spill costs in this loop).
#ifndef ATTN_WAVES_PER_SIMD
#define ATTN_WAVES_PER_SIMD 2
#endif
// ATTN_CLOCKS (undefined in the shipped library): the first wavefront of the first workgroup stamps the
// shader cycle counter and the constant 100 MHz counter when it starts and when it ends, and the cycle
// counter where the key-block loop of its second and of its third work item starts and ends; the
// library exports attn_clocks_read(), and the benchmark derives the shader clock of a launch, the
// length of an iteration and the stretch between two items from the stamps.
// ATTN_CLOCKS=2 additionally has the first and the last wavefront of that workgroup add up, over its
// second work item, the cycles each phase of an item takes (set-up, first score blocks, first softmax,
// the key-block iterations by kind, epilogue), read with attn_phases_read().  A stamp per iteration
// costs about 1.5 % of the loop, which is why the clock figures come from the build without them.
static_assert(ATTN_SOFTMAX >= 0 && ATTN_SOFTMAX <= 3, "ATTN_SOFTMAX is 0, 1, 2 or 3");
static_assert(ATTN_LDS_PREFETCH >= 1 && ATTN_LDS_PREFETCH <= 8, "ATTN_LDS_PREFETCH is 1 .. 8");

namespace {

using namespace attn;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define LDS_AS __attribute__((address_space(3)))

constexpr int ROW_BYTES = HD * 2;    // one (token, head) row of BF16
constexpr int TILE_BYTES = BN * ROW_BYTES;
constexpr int NSTAGE = 3;                   // LDS stages per operand
constexpr int REQ_AHEAD = NSTAGE - 1;       // tiles are requested this many iterations before use
constexpr int LPT = 16 / NWAVES;            // 1 KiB load instructions per tile and wavefront
constexpr int V_BASE = NSTAGE * TILE_BYTES; // K stages first, V stages after them
constexpr int Q_BASE = 2 * NSTAGE * TILE_BYTES;      // after the stages: Q of the next item, 8 KiB per wavefront
constexpr int Q_WAVE_BYTES = 32 * ROW_BYTES;
constexpr int LDS_BYTES = Q_BASE + NWAVES * Q_WAVE_BYTES;   // 160 KiB, all of a CU's LDS
// Largest partial row sum (16 probabilities of one lane) the fast softmax path accepts: probabilities
// stay below 2^14 relative to the reference maximum, far inside BF16 / FP32 range.
constexpr float P_SUM_LIMIT = 16384.0f;
constexpr int MAT_PREFETCH = ATTN_LDS_PREFETCH;   // LDS reads run this many MFMAs ahead of their consumer
// s_waitcnt vmcnt(n), n < 16, other counters untouched.  The tile requests are counted by hand: "all but
// the newest n vector-memory operations have completed" stands for "the tiles of the iterations before
// have landed".  That holds whatever else is in the queue, because the loads that must have landed are
// always followed by n newer loads and loads complete in order; but it is only CHEAP while the requests
// are the only memory operations of the loop: a register spill would bring reloads of the compiler's own,
// each behind an s_waitcnt vmcnt(0) that waits for every tile request in flight (a memory latency per
// reload, in a loop whose iteration is shorter than one).  So the kernels must compile without scratch
// (a host-side test of the built code object checks that), and the epilogue's stores are issued only
// after the wait that the next item's first tiles need.
constexpr int wait_vmcnt(int n) { return 0x0F70 | n; }
constexpr int WAIT_VMCNT0 = wait_vmcnt(0);
constexpr int WAIT_LGKMCNT0 = 0xC07F;       // s_waitcnt lgkmcnt(0), other counters untouched
// end of an iteration: everything but the loads of the last REQ_AHEAD-1 iterations has landed
constexpr int WAIT_ITER_END = wait_vmcnt((REQ_AHEAD - 1) * 2 * LPT);

// n / d with the constants that make_div() found on the host.
__host__ __device__ inline uint32_t fast_div(uint32_t n, const Div d) {
#ifdef __HIP_DEVICE_COMPILE__
    return (__umulhi(n, d.mul) + n) >> d.shift;
#else
    return (uint32_t)((((uint64_t)n * d.mul) >> 32) + n) >> d.shift;
#endif
}
struct Params {
    const __bf16 *k, *v;
    int Hkv, Skv;
    float c;        // scale * log2(e)
    int pad_;
    // the rest is read from the argument block where it is needed
    const __bf16 *q;
    __bf16 *o;
    float *lse;
    Shape shape;
    Sched sched;
    Share share;
    uint32_t unit;  // SHARED: REGION_SHARE_UNIT if the launch has the region, or POOL_NONE
};

__device__ __forceinline__ float lane32_max(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float lane32_sum(float x) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    bf16x2 p = __builtin_convertvector((f32x2){a, b}, bf16x2);   // v_cvt_pk_bf16_f32, nearest even
    return __builtin_bit_cast(uint32_t, p);
}
// acc + lo(p) + hi(p) for a pair of BF16 values (v_dot2c_f32_bf16 against (1, 1)).
__device__ __forceinline__ float add_bf16_pair(uint32_t p, float acc) {
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, p), ones, acc, false);
}
// The raw score that maximises score * c: the largest one for c >= 0, the smallest for c < 0 (NEG).
template <bool NEG>
__device__ __forceinline__ float ext3(float a, float b, float c) {
    float r;
    if (NEG) asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    else asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// 16 bytes per lane from global memory straight into LDS: lane L's data lands at lds_base + 16*L.
// Issued as inline assembly so that the compiler's counter bookkeeping does not make every later
// LDS read wait for it; the caller waits with s_waitcnt vmcnt(n) before the barrier that publishes
// the tile.
// A wave-uniform pointer as a scalar-register pair, also when the compiler chose to keep it in vector registers.
__device__ __forceinline__ const unsigned char *uniform_ptr(const unsigned char *ptr) {
    const uint64_t v = (uint64_t)(uintptr_t)ptr;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const unsigned char *)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
// Both forms write M0 and say so in their clobber lists: the compiler reserves M0 (it sets it itself
// right before an instruction of its own that reads it) and warns that it will not preserve it across
// the statement, which is exactly what is meant here.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lds_dma16(const unsigned char *base, uint32_t voffset, uint32_t lds_base) {
    base = uniform_ptr(base);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_base), "v"(voffset), "s"(base)
                 : "memory", "m0");
}
// The same for data that is read once: it passes the caches by (nt).
__device__ __forceinline__ void lds_dma16_once(const unsigned char *base, uint32_t voffset, uint32_t lds_base) {
    base = uniform_ptr(base);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt"
                 :
                 : "s"(lds_base), "v"(voffset), "s"(base)
                 : "memory", "m0");
}
// The same with the LDS address given as a scalar plus a compile-time constant (one scalar instruction).
template <int IMM>
__device__ __forceinline__ void lds_dma16_imm(const unsigned char *base, uint32_t voffset, uint32_t lds_base) {
    asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_base), "v"(voffset), "s"(base), "n"(IMM)
                 : "memory", "scc", "m0");
}
#pragma clang diagnostic pop
// Keeps the instruction that produces x at this point of the program order (no code is emitted).
#define PIN(x) asm volatile("" : "+v"(x))
__device__ __forceinline__ void wg_barrier() {
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
}

#ifdef ATTN_CLOCKS
// cycle counter at start / end, 100 MHz counter at start / end; then, for the second and the third item of
// the first workgroup: cycle counter at the start and at the end of the key-block loop, and the loop's iterations
__device__ unsigned long long g_clocks[10];
#define ATTN_STAMP(k, v) do { __builtin_amdgcn_sched_barrier(0); if (bid == 0 && tid == 0 && (item_no == 1 || item_no == 2)) \
                                  g_clocks[4 + 3 * (item_no - 1) + (k)] = (v); __builtin_amdgcn_sched_barrier(0); } while (0)
#else
#define ATTN_STAMP(k, v) do { } while (0)
#endif
#if defined(ATTN_CLOCKS) && ATTN_CLOCKS >= 2
// [first / last wavefront of the first workgroup][phase]: cycles of its second work item spent in
// 0 set-up (next item's lookup, state reset, Q request; a cold item's first tile requests and wait),
// 1 the first two score blocks, 2 the first softmax, 3 the barrier and requests before the loop,
// 4 iterations in which this wavefront took the fast path, 5 their number, 6 other iterations but the
// last, 7 their number, 8 the last iteration, 9 the wait for outstanding loads, 10 the epilogue,
// 11 the whole item.  Not stamped where items are shared: a part has no registers left for it.
__device__ unsigned long long g_phases[2][12];
__device__ __forceinline__ unsigned long long phase_now() {
    __builtin_amdgcn_sched_barrier(0);
    const unsigned long long t = __builtin_readcyclecounter();
    __builtin_amdgcn_sched_barrier(0);
    return t;
}
#define ATTN_PHASE(k) do { if (!SHARED) { const unsigned long long now_ = phase_now(); ph[k] += now_ - ph_prev; ph_prev = now_; } } while (0)
#define ATTN_PHASE_COUNT(k) do { if (!SHARED) ++ph[k]; } while (0)
#else
#define ATTN_PHASE(k) do { } while (0)
#define ATTN_PHASE_COUNT(k) do { } while (0)
#endif

// Device memory for partial results: a part of the code object, so it exists once per device, needs no
// allocation and no host-side bookkeeping, and goes when the library is unloaded.  A launch takes a run of
// units and gives it back, both on the device: a one-workgroup launch in front finds a free run and
// leaves its number in the first LSE element of every item, which is the launch's own memory and is overwritten by the
// result only after all workgroups of the item have read it.  Launches on any number of streams, from any thread and
// replayed from graphs thus never share units.  If no run is free (the pool serves at least POOL_UNITS / SHARE_MAX_UNITS
// launches at a time), the first workgroup of each item takes all of its parts and the others leave, which is slower but
// needs no memory and gives the same bits.
//
// The launch in front takes 4.8 us, with the gap behind it.  A device's null stream, whose launches never overlap, which cannot be captured
// into a graph and whose handle never stands for another, has memory of its own instead and no such launch: it is told the unit by the
// host and reads no mark.  The region's counters are zero when a launch starts, because whoever takes a counter to its last value sets it
// back.  (us, K and V from HBM: 1 x 1 x 32768, 32 heads on 8 38.7, with the region 35.9; 16 x 1 x 4000, 32 on 8 51.8 and 48.4; 1 x 512 x 16384, 32 on 8
// 131.0 and 128.9.)
constexpr uint32_t POOL_NONE = 0xffu;
constexpr uint32_t POOL_SOLO = 0xfeu;       // split-key kernel: items of one workgroup each in the form for shared ones
// How the number (or POOL_NONE) stands in an LSE element: as a NaN whose low half is no result's.  (A NaN of a
// result has the default payload or one that came in with a BF16 value, whose low 16 bits are zero.)  Where no run was
// free, a late workgroup may find the item's result there instead, already stored by the first one, and has to
// take anything but the mark for "none".
constexpr uint32_t POOL_MARK = 0xffe5a500u;
static_assert(POOL_UNITS + REGION_UNITS <= POOL_SOLO, "no unit has the number for none, which fits the low byte of the mark");
__host__ __device__ inline uint32_t pool_mark(uint32_t unit) { return POOL_MARK | unit; }
__host__ __device__ inline uint32_t pool_unmark(uint32_t word) {
    return (word ^ POOL_MARK) < POOL_UNITS ? (word ^ POOL_MARK) : POOL_NONE;
}
__device__ unsigned long long g_pool_taken;         // bit u: unit u belongs to a launch in flight
__device__ __attribute__((aligned(4096))) unsigned char g_pool[(size_t)(POOL_UNITS + REGION_UNITS) * POOL_UNIT_BYTES];
// The one lane that takes a run of n units: first free run, or POOL_NONE.
__device__ inline uint32_t pool_take(int n)
{
    if (!ATTN_POOL) return POOL_NONE;
    const unsigned long long run = (1ull << n) - 1;     // n < 64
    unsigned long long taken = 0;       // (a guess that is usually right: one round trip to memory)
    int tries = 0;
    for (int u = 0; u + n <= POOL_UNITS;) {
        if (taken & (run << u)) { ++u; continue; }
        if (__hip_atomic_compare_exchange_strong(&g_pool_taken, &taken, taken | (run << u), __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return (uint32_t)u;
        // the mask is another one, `taken` holds it now: look at u again, but not more than POOL_UNITS times in all
        if (++tries == POOL_UNITS) break;
    }
    return POOL_NONE;
}
// Partial results pass between workgroups of one launch that may sit on different XCDs, each with an L2 of its
// own.  They are written and read at agent scope element by element (sc1: through the L2 to memory that all
// XCDs share), and a wait for the stores stands before the counter that announces them.  An agent-scope release
// fence instead writes back an XCD's whole L2 for every workgroup: measured 0.17 us each, one after the other
// (512 workgroups: 80 us).
__device__ inline void pool_store4(unsigned char *at, float a, float b, float c, float d)
{
    typedef unsigned long long u64;
    const u64 lo = (u64)__float_as_uint(a) | (u64)__float_as_uint(b) << 32, hi = (u64)__float_as_uint(c) | (u64)__float_as_uint(d) << 32;
    __hip_atomic_store((u64 *)at, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store((u64 *)at + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void pool_load4(const unsigned char *at, float *x)
{
    typedef unsigned long long u64;
    const u64 lo = __hip_atomic_load((const u64 *)at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const u64 hi = __hip_atomic_load((const u64 *)at + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    x[0] = __uint_as_float((uint32_t)lo); x[1] = __uint_as_float((uint32_t)(lo >> 32));
    x[2] = __uint_as_float((uint32_t)hi); x[3] = __uint_as_float((uint32_t)(hi >> 32));
}
// The same at 16 bytes per lane, as buffer accesses with the sc1 bit (agent scope; bounds-checked by the descriptor).
constexpr int POOL_SC1 = 16;
__device__ inline __amdgpu_buffer_rsrc_t pool_rsrc(uint32_t unit, int units)
{
    return __builtin_amdgcn_make_buffer_rsrc(g_pool + (size_t)unit * POOL_UNIT_BYTES, 0, units * (int)POOL_UNIT_BYTES, 0x00020000);
}
__device__ inline void pool_store16(__amdgpu_buffer_rsrc_t rs, uint32_t lane_at, uint32_t at, float a, float b, float c, float d)
{
    const u32x4 x = {__float_as_uint(a), __float_as_uint(b), __float_as_uint(c), __float_as_uint(d)};
    __builtin_amdgcn_raw_buffer_store_b128(x, rs, lane_at, at, POOL_SC1);
}
__device__ inline u32x4 pool_load16(__amdgpu_buffer_rsrc_t rs, uint32_t lane_at, uint32_t at)
{
    return __builtin_amdgcn_raw_buffer_load_b128(rs, lane_at, at, POOL_SC1);
}
__device__ inline void pool_clear(uint32_t unit, uint32_t *counter)
{
    if (sets_counters_back(unit)) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void pool_store(float *at, float a) { __hip_atomic_store(at, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline float pool_load(const float *at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void pool_give(uint32_t u, int n)
{
    if (sets_counters_back(u)) return;        // the region
    __hip_atomic_fetch_and(&g_pool_taken, ~(((1ull << n) - 1) << u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The forms of the 256-row kernel: with or without the causal mask, whole items or shared ones.  A negative scale is a wave-uniform
// branch in the kernel of whole items, where an extreme score is looked for (once per item and where the reference is raised; us, negative scale, a form
// of its own / the branch: 8 x 4096, 16 heads 869.4 / 864.0, masked 494.1 / 490.1, 4 x 4096, 32 on 8, masked 468.2 / 468.1); with shared
// ones, which have no register for it, Q is negated as it is loaded (in the kernel of whole items that costs 0.2 % of a causal launch).
template <bool CAUSAL, bool SHARED>
__global__ __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(ATTN_WAVES_PER_SIMD, ATTN_WAVES_PER_SIMD)))
void attn_fwd_kernel(const Params p)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    // Launch constants that only the per-item code needs are read from the kernel argument block where
    // they are used, instead of occupying scalar registers through the block loop.
    auto cold = [&]() __attribute__((always_inline)) -> const __attribute__((address_space(4))) Params & {
        auto cp = (const __attribute__((address_space(4))) Params *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(cp));
        return *cp;
    };

    // ---- work distribution.  The launch has one workgroup per CU, 8 * slots of them, dealt round-robin
    // to the 8 XCDs by the hardware: workgroup (x = bid % 8, slot = bid / 8) works through entries
    // slot, slot + slots, ... of XCD x's list, one after the other, so that the loads of the next
    // entry can start while the current one finishes.
    // Non-causal: each XCD's list is a contiguous range of items (neighbours share K/V in that XCD's
    // L2).  Causal: tiles differ in length, so each XCD owns whole sub-groups of equal total work and
    // its list walks `window` of them together from their longest tiles to their shortest; odd rounds
    // run through the slots backwards, so that the workgroup that drew the longest tile of one round
    // draws the shortest of the next.
    const int bid = blockIdx.x;
    const int xcd = bid & 7, slot = bid >> 3;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31;
    const int hh = lane >> 5;
#ifdef ATTN_CLOCKS
    if (bid == 0 && tid == 0) { g_clocks[2] = wall_clock64(); g_clocks[0] = __builtin_readcyclecounter(); }
#endif
    const float c = SHARED ? fabsf(p.c) : p.c;
    const int off = p.Skv - cold().shape.Sq;                    // causal: key j valid iff j <= i + off
    const int nfull = p.Skv / BN;                               // tiles below this index are full
    const bool all_full = (p.Skv % BN) == 0;

    // one wide scalar load each, where the per-item code starts
    auto load_sched = [&]() __attribute__((always_inline)) -> Sched {
        Sched sc;
        __builtin_memcpy(&sc, &cold().sched, sizeof(Sched));
        return sc;
    };
    auto load_shape = [&]() __attribute__((always_inline)) -> Shape {
        Shape sh;
        __builtin_memcpy(&sh, &cold().shape, sizeof(Shape));
        return sh;
    };
    // entry j of this XCD's list -> (group, tile); false for a padding entry
    auto decode = [&](const Sched &sc, int j, int &grp, int &tile) __attribute__((always_inline)) -> bool {
        if (CAUSAL) {
            const int w = fast_div(j, sc.d_per_win);
            const int r = j - w * sc.per_win;
            const int kw = min(sc.window, sc.sgx - w * sc.window);      // the last window may be narrower
            const int st = kw == sc.window ? (int)fast_div(r, sc.d_window) : r / kw;
            const int sg = xcd * sc.sgx + w * sc.window + (r - st * kw);
            grp = sg >> sc.split_log2;
            const int tile_r = st * sc.split + (sg & (sc.split - 1));
            tile = sc.ntile - 1 - tile_r;                               // long (late) query tiles first
            return tile_r < sc.ntile;
        }
        const int item = xcd * sc.per_xcd + j;
        grp = fast_div(item, sc.d_ntile);
        tile = item - grp * sc.ntile;
        return item < sc.total;
    };
    // SHARED: this workgroup's stretch of the line, and whether items are shared at all (false: no pool units were
    // free; then the workgroup whose stretch holds an item's start takes all of its parts, one after the other, the later ones
    // in the place of the workgroups `ahead` of it, so that the result is the same to the last bit)
    int cut_lo = 0, cut_hi = 0, ahead = 0;
    bool pooled = true;
    uint32_t unit = POOL_NONE;
    auto load_share = [&]() __attribute__((always_inline)) -> Share {
        Share sr;
        __builtin_memcpy(&sr, &cold().share, sizeof(Share));
        return sr;
    };
    auto set_cuts = [&]() __attribute__((always_inline)) {
        const Share sr = load_share();
        const uint32_t w = xcd * (sr.wgs >> 3) + slot + ahead;      // neighbours in the line are on one XCD
        cut_lo = __builtin_amdgcn_readfirstlane((int)(w * (uint32_t)sr.total / (uint32_t)sr.wgs));
        cut_hi = __builtin_amdgcn_readfirstlane(w + 1 == (uint32_t)sr.wgs ? INT32_MAX : (int)((w + 1) * (uint32_t)sr.total / (uint32_t)sr.wgs));
    };
    auto blocks_of = [&](const Shape &sh, int tile) __attribute__((always_inline)) -> int {
        int n = (p.Skv + BN - 1) / BN;
        if (CAUSAL) {
            const int klast = min(tile * sh.tile_pos + sh.tile_pos, sh.Sq) - 1 + off;
            n = klast < 0 ? 0 : min(n, klast / BN + 1);
        }
        return n;
    };
    // SHARED: first item from (grp, tile), which stands at `at` in the line, that this workgroup has a part of
    auto find_part = [&](int &grp, int &tile, int &at) __attribute__((always_inline)) -> bool {
        const Share sr = load_share();
        const Shape sh = load_shape();
        const int ntile = cold().sched.ntile;
        while (grp < sr.groups) {
            const int n = blocks_of(sh, tile);
            const int first_cut = at + sr.extra + SHARE_MIN_PART, last_cut = at + sr.extra + n - SHARE_MIN_PART;
            if (cut_hi < first_cut) return false;
            if (cut_lo < first_cut || (pooled && cut_lo <= last_cut)) return true;
            at += n + sr.extra;
            if (++tile == ntile) { tile = 0; ++grp; }
        }
        return false;
    };
    // SHARED: the item that `x` of the line lies in
    auto locate = [&](int x, int &grp, int &tile, int &at) __attribute__((always_inline)) {
        const Share sr = load_share();
        const Shape sh = load_shape();
        const int ntile = cold().sched.ntile;
        grp = __builtin_amdgcn_readfirstlane((unsigned)x / (unsigned)sr.group_len);
        at = grp * sr.group_len;
        for (tile = 0; ; tile += 64) {      // 64 tiles at a time; their lengths add up to group_len
            const int len = tile + lane < ntile ? blocks_of(sh, tile + lane) + sr.extra : 0;
            int sum = len;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int o = __shfl_up(sum, d);
                if (lane >= d) sum += o;
            }
            const unsigned long long beyond = __builtin_amdgcn_ballot_w64(at + sum > x);
            if (beyond != 0 || tile + 64 >= ntile) {
                const int k = beyond != 0 ? __builtin_ctzll(beyond) : ntile - 1 - tile;
                at += __builtin_amdgcn_readlane(sum - len, k);
                tile += k;
                return;
            }
            at += __builtin_amdgcn_readlane(sum, 63);
        }
    };
    // first round >= r in which this workgroup has a real entry; false when its list is exhausted
    auto find_item = [&](int &r, int &grp, int &tile) __attribute__((always_inline)) -> bool {
        const Sched sc = load_sched();
        for (; r * sc.slots < sc.per_xcd; ++r) {
            const int j = r * sc.slots + ((CAUSAL && (r & 1)) ? sc.slots - 1 - slot : slot);
            if (j < sc.per_xcd && decode(sc, j, grp, tile)) return true;
        }
        return false;
    };
    // what a wavefront needs to know of an item
    struct Geo {
        int b, head, q0;                 // batch entry, query head and first query row of this wavefront
        int nblk;                        // key blocks of the workgroup (one barrier each)
        int j0, at, item, blocks;        // SHARED: first of them, the item's place in the line, its number and all its blocks
        const unsigned char *kg, *vg;    // first K / V row of the item's batch entry and K/V head
    };
    const size_t kv_row_bytes = (size_t)p.Hkv * HD * 2;
    const size_t tile_gbytes = (size_t)BN * kv_row_bytes;
    auto geometry = [&](int grp, int tile, int at) __attribute__((always_inline)) -> Geo {
        const Shape sh = load_shape();
        Geo g;
        g.j0 = g.at = g.item = g.blocks = 0;
        const int bh = fast_div(grp, sh.d_chunks);
        const int chunk = grp - bh * sh.chunks;
        g.b = fast_div(bh, sh.d_hkv);
        const int hkv = bh - g.b * p.Hkv;
        g.head = hkv * sh.G + chunk * sh.pack + (wave & (sh.pack - 1));
        g.q0 = tile * sh.tile_pos + (wave >> sh.pack_log2) * 32;
        g.nblk = blocks_of(sh, tile);
        g.kg = (const unsigned char *)(p.k + ((size_t)g.b * p.Skv * p.Hkv + hkv) * HD);
        g.vg = (const unsigned char *)(p.v + ((size_t)g.b * p.Skv * p.Hkv + hkv) * HD);
        if (SHARED) {
            const int first = at + cold().share.extra;      // block 0's place in the line
            int j1 = g.nblk;
            if (cut_hi <= first + j1 - SHARE_MIN_PART) j1 = cut_hi - first;
            if (cut_lo >= first + SHARE_MIN_PART) g.j0 = __builtin_amdgcn_readfirstlane(cut_lo - first);
            g.blocks = __builtin_amdgcn_readfirstlane(g.nblk);
            g.nblk = j1 - g.j0;
            g.at = __builtin_amdgcn_readfirstlane(at);
            g.item = __builtin_amdgcn_readfirstlane(grp * cold().sched.ntile + tile);
            g.kg += g.j0 * tile_gbytes;
            g.vg += g.j0 * tile_gbytes;
        }
        // all of it is wave-uniform: say so, so that it lives in scalar registers
        g.b = __builtin_amdgcn_readfirstlane(g.b);
        g.head = __builtin_amdgcn_readfirstlane(g.head);
        g.q0 = __builtin_amdgcn_readfirstlane(g.q0);
        g.nblk = __builtin_amdgcn_readfirstlane(g.nblk);
        g.kg = uniform_ptr(g.kg);
        g.vg = uniform_ptr(g.vg);
        return g;
    };

    // ---- the item in work and the one after it
    int b = 0, head = 0, q0 = 0;
    int nblk = 0;       // key blocks of the workgroup
    int n_w = 0;        // of those, the blocks that hold a key valid for some row of this wavefront
    int n_unm = 0;      // of those, the leading blocks that need no mask at all
    int part_j0 = 0;    // SHARED: first block of the part in work; block numbers and key indices count from there
    auto keys = [&]() __attribute__((always_inline)) -> int { return SHARED ? p.Skv - part_j0 * BN : p.Skv; };
    auto offset = [&]() __attribute__((always_inline)) -> int { return SHARED ? off - part_j0 * BN : off; };
    const unsigned char *kg = nullptr, *vg = nullptr;
    bool warm_next = false;             // the item after this one exists and its first tiles are requested by this one
    int nx_nblk = 0;
    const unsigned char *nx_kg = nullptr, *nx_vg = nullptr;
    int ring0 = 0;                      // LDS stage of block 0 of the item in work
    auto enter = [&](const Geo &g) __attribute__((always_inline)) {
        b = g.b; head = g.head; q0 = g.q0; nblk = g.nblk; kg = g.kg; vg = g.vg;
        if (SHARED) part_j0 = g.j0;
        n_unm = keys() / BN;
        n_w = nblk;
        if (CAUSAL) {
            const int off = offset();
            const int klast_w = q0 + 31 + off;          // last key valid for the last row of the wave
            n_w = klast_w < 0 ? 0 : min(nblk, klast_w / BN + 1);
            const int kfirst_w = q0 + off + 1;          // number of keys valid for every row of the wave
            n_unm = min(n_unm, kfirst_w <= 0 ? 0 : kfirst_w / BN);
        }
        n_unm = min(n_unm, n_w);
    };

    // ---- everything the wavefront keeps across the key-block loop
    bf16x8 qf[8];          // Q^T operand: query lane%32, d = 16*s + 8*(lane/32) .. +7
    f32x16 sa[2], sb[2];   // S^T of two blocks in flight (two 32-key tiles each): the softmax consumes one
                           // while the MFMAs fill the other
    uint32_t pb[2][8];     // P^T of the block whose PV product comes next, BF16 pairs
    f32x16 acc[4];         // O^T accumulator: four 32-d tiles
    float m;               // running maximum in log2 units (score * scale * log2 e)
    float l;               // this lane's share of the running sum (its 16 of every 32 keys), unrounded FP32
                           // probabilities: the sum LSE is formed from
    float lr;              // the same sum over the BF16-rounded probabilities that multiply V: O is
                           // normalised by this one, so that a rounding error in a dominant weight
                           // cancels between numerator and denominator
    auto negate_q = [&]() __attribute__((always_inline)) {
        if (SHARED && p.c < 0.0f) {
#pragma unroll
            for (int s = 0; s < 8; ++s) qf[s] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[s]) ^ 0x80008000u);
        }
    };
    auto load_q = [&](const Geo &g) __attribute__((always_inline)) {
        const int Sq = cold().shape.Sq, Hq = cold().shape.Hq;
        const int qrow = min(g.q0 + l32, Sq - 1);
        const __bf16 *qp = cold().q + ((size_t)((size_t)g.b * Sq + qrow) * Hq + g.head) * HD + 8 * hh;
#pragma unroll
        for (int s = 0; s < 8; ++s) qf[s] = *(const bf16x8 *)(qp + 16 * s);
        negate_q();
    };
    // The same through LDS: requested (wave-private region, the K swizzle) when the item before
    // starts, fetched into registers when that one's last block is done.
    auto request_q = [&](const Geo &g) __attribute__((always_inline)) {
        const int Sq = cold().shape.Sq, Hq = cold().shape.Hq;
        const size_t q_row_bytes = (size_t)Hq * HD * 2;
        const int q0c = min(g.q0, Sq - 1);          // rows past the end of Q re-read the last row
        const unsigned char *qg = (const unsigned char *)(cold().q + ((size_t)((size_t)g.b * Sq + q0c) * Hq + g.head) * HD);
        const int last = Sq - 1 - q0c;
        const uint32_t lbase = (uint32_t)(uintptr_t)lds + Q_BASE + wave * Q_WAVE_BYTES;
        int ln = lane;
        PIN(ln);            // per-lane offsets are formed here, not kept in registers across the block loop
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = 4 * i + (ln >> 4);
            const uint32_t o = (uint32_t)(min(row, last) * q_row_bytes) + (((ln & 15) ^ (row & 15)) << 4);
            lds_dma16(qg, o, lbase + i * 1024);
        }
    };
    auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[dt][r] = 0.0f;
        m = -INFINITY;
        l = 0.0f;
        lr = 0.0f;
    };
    // ---- global -> LDS tile loads.  One instruction moves 1 KiB: lane L's 16
    // bytes land at (wave-uniform LDS base) + 16*L, i.e. row L/16 and physical
    // 16-byte unit L%16 of a 4-row chunk; the lane fetches the logical unit
    // that the swizzle maps there.  K: unit ^ (row & 15), so that 16 lanes
    // reading one d-range of 16 consecutive rows touch 16 different units.
    // V: unit ^ ((row & 3) << 2), so that the 4 rows x 64 bytes a half-wave
    // fetches with the transposing read cover all banks once.
    const int ld_r = lane >> 4, ld_u = lane & 15;
    uint32_t koff[LPT], voff[LPT];   // byte offset of this lane's 16 bytes from the first row of a tile
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
        const int row = (wave * LPT + i) * 4 + ld_r;
        koff[i] = (uint32_t)(row * kv_row_bytes) + ((ld_u ^ (row & 15)) << 4);
        voff[i] = (uint32_t)(row * kv_row_bytes) + ((ld_u ^ ((row & 3) << 2)) << 4);
    }
    const uint32_t lds_wave = (uint32_t)(uintptr_t)lds + wave * (LPT * 1024);
    // The three stages are a ring that runs on from one item to the next: block j of the item in work
    // lives in stage (ring0 + j) % 3, and blocks nblk, nblk+1, ... are blocks 0, 1, ... of the next item.
    auto stage_off = [&](int blk) __attribute__((always_inline)) { return ((blk + ring0) % NSTAGE) * TILE_BYTES; };
    // Global address of the tile that request `blk_req` stands for: a block of this item, or (past its
    // end) a block of the next item if that one is being warmed up; otherwise, and past the end of
    // the next item too, the last block is read again into the (dead) stage the request would have
    // used, so that the number of loads in flight is the same in every iteration.
    auto tile_ptr = [&](int blk_req, bool is_v, int &blk, int &left) __attribute__((always_inline)) -> const unsigned char * {
        const unsigned char *g = is_v ? vg : kg;
        left = keys();      // keys from the item's first block on
        blk = min(blk_req, nblk - 1);
        if (blk_req >= nblk && warm_next) {
            g = is_v ? nx_vg : nx_kg;
            left = p.Skv;       // (SHARED: only the first part of a stretch begins inside an item)
            blk = min(blk_req - nblk, nx_nblk - 1);
        }
        return g + (size_t)blk * tile_gbytes;
    };
    // General form of a tile request: rows past the end of a partial tile re-read the last row (they
    // are masked later).
    auto issue_tile = [&](int blk_req, bool is_v) __attribute__((always_inline)) {
        int blk, left;
        const unsigned char *g = tile_ptr(blk_req, is_v, blk, left);
        const uint32_t lbase = lds_wave + (is_v ? V_BASE : 0) + stage_off(blk_req);
        const bool partial = (blk + 1) * BN > left;
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            uint32_t o = is_v ? voff[i] : koff[i];
            if (partial) {
                int ln = lane;
                PIN(ln);        // formed here, not kept in a register across the block loop
                const int row = (wave * LPT + i) * 4 + (ln >> 4);
                const int rl = min(row, left - 1 - blk * BN);
                o = o - (uint32_t)(row * kv_row_bytes) + (uint32_t)(rl * kv_row_bytes);
            }
            lds_dma16(g, o, lbase + i * 1024);
        }
    };
    // ---- per-lane LDS read addresses
    int kaddr[8];   // K operand: row l32 (+32 per tile), logical unit 2*st + hh
#pragma unroll
    for (int st = 0; st < 8; ++st) kaddr[st] = l32 * ROW_BYTES + (((2 * st + hh) ^ (l32 & 15)) << 4);
    // V operand via the transposing read: lane (i = lane%16, g = (lane%32)/16, hh) supplies the address
    // of key row 4*hh + i/4 and d = 16*g + 4*(i%4) of a 16-key x 32-d block and receives d = 16*g + i
    // of keys 4*hh .. 4*hh+3.
    int vaddr[4];
    {
        const int i16 = lane & 15, g = (lane >> 4) & 1;
        const int row = 4 * hh + (i16 >> 2);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const int d = 32 * dt + 16 * g + 4 * (i16 & 3);
            vaddr[dt] = V_BASE + row * ROW_BYTES + ((((d >> 3) ^ ((row & 3) << 2))) << 4) + (d & 7) * 2;
        }
    }

    // SHARED: all of these once more, so that no registers hold them while parts are added up
    auto read_addresses = [&]() __attribute__((always_inline)) {
        int lane = tid & 63;
        PIN(lane);
        const int l32 = lane & 31, hh = lane >> 5, i16 = lane & 15, g = (lane >> 4) & 1;
#pragma unroll
        for (int i = 0; i < LPT; ++i) {
            const int row = (wave * LPT + i) * 4 + (lane >> 4);
            koff[i] = (uint32_t)(row * kv_row_bytes) + ((i16 ^ (row & 15)) << 4);
            voff[i] = (uint32_t)(row * kv_row_bytes) + ((i16 ^ ((row & 3) << 2)) << 4);
        }
#pragma unroll
        for (int st = 0; st < 8; ++st) kaddr[st] = l32 * ROW_BYTES + (((2 * st + hh) ^ (l32 & 15)) << 4);
        const int row = 4 * hh + (i16 >> 2);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const int d = 32 * dt + 16 * g + 4 * (i16 & 3);
            vaddr[dt] = V_BASE + row * ROW_BYTES + ((((d >> 3) ^ ((row & 3) << 2))) << 4) + (d & 7) * 2;
        }
    };

    // ---- building blocks
    // S^T = K(stage kb) Q^T alone (prologue).
    auto qk_only = [&](f32x16 (&s)[2], int kb) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[t][r] = 0.0f;
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                bf16x8 a = *(const LDS_AS bf16x8 *)(lds + kb + t * 32 * ROW_BYTES + kaddr[st]);
                s[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[st], s[t], 0, 0, 0);
            }
    };
    // The 32 MFMAs of one iteration as one software-pipelined sequence: even slots O^T += V^T P^T
    // (V stage vb, P from pb), odd slots snxt = K Q^T (K stage kb), so that two MFMAs accumulating into
    // the same registers are four slots apart; the LDS reads of slot i+MAT_PREFETCH are issued before
    // the MFMA of slot i.  `between(slot)` is called after each MFMA and carries the caller's vector
    // work for that slot (it must not touch pb entries the remaining PV MFMAs still read).
    auto mfma_block = [&](f32x16 (&snxt)[2], int vb, int kb, auto between) __attribute__((always_inline)) {
        constexpr int PREFETCH = SHARED && MAT_PREFETCH > 3 ? 3 : MAT_PREFETCH;     // (SHARED: no registers for more)
        bf16x8 frag[32];
        int va[4], ka[8];      // stage offsets folded into the per-lane bases: every read is base + immediate
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) va[dt] = vaddr[dt] + vb;
#pragma unroll
        for (int st = 0; st < 8; ++st) ka[st] = kaddr[st] + kb;
        auto fetch = [&](int slot) __attribute__((always_inline)) -> bf16x8 {
            const int i = slot >> 1;
            if ((slot & 1) == 0) {            // V^T operand of PV MFMA i: key group i/4, d tile i%4
                const int ro = (i >> 2) * 16 * ROW_BYTES;
                s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + va[i & 3] + ro));
                s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (LDS_AS s16x4 *)(lds + va[i & 3] + (ro + 8 * ROW_BYTES)));
                s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                return __builtin_bit_cast(bf16x8, av);
            }
            const int st = i >> 1, t = i & 1;   // K operand of QK MFMA i: d step st, key tile t
            return *(const LDS_AS bf16x8 *)(lds + ka[st] + t * 32 * ROW_BYTES);
        };
#pragma unroll
        for (int i = 0; i < PREFETCH; ++i) frag[i] = fetch(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int slot = 0; slot < 32; ++slot) {
            if (slot + PREFETCH < 32) frag[slot + PREFETCH] = fetch(slot + PREFETCH);
            const int i = slot >> 1;
            if ((slot & 1) == 0) {
                const int g = i >> 2;         // key group: tile g/2, half g%2
                u32x4 pw = {pb[g >> 1][4 * (g & 1)], pb[g >> 1][4 * (g & 1) + 1],
                            pb[g >> 1][4 * (g & 1) + 2], pb[g >> 1][4 * (g & 1) + 3]};
                acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    frag[slot], __builtin_bit_cast(bf16x8, pw), acc[i & 3], 0, 0, 0);
            } else {
                const int st = i >> 1, t = i & 1;
                if (st == 0) {
                    f32x16 z;
#pragma unroll
                    for (int r = 0; r < 16; ++r) z[r] = 0.0f;
                    snxt[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[slot], qf[st], z, 0, 0, 0);
                } else {
                    snxt[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[slot], qf[st], snxt[t], 0, 0, 0);
                }
            }
            between(slot);
            __builtin_amdgcn_sched_barrier(0);     // keep the slot order exactly as written
        }
    };
    // O^T += V^T P^T alone: the last iteration of an item, when no further scores are wanted.
    auto pv_only = [&](int vb) __attribute__((always_inline)) {
        constexpr int PREFETCH = SHARED && MAT_PREFETCH > 3 ? 3 : MAT_PREFETCH;     // (SHARED: no registers for more)
        bf16x8 frag[16];
        int va[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) va[dt] = vaddr[dt] + vb;
        auto fetch = [&](int i) __attribute__((always_inline)) -> bf16x8 {
            const int ro = (i >> 2) * 16 * ROW_BYTES;
            s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + va[i & 3] + ro));
            s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + va[i & 3] + (ro + 8 * ROW_BYTES)));
            s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            return __builtin_bit_cast(bf16x8, av);
        };
#pragma unroll
        for (int i = 0; i < PREFETCH; ++i) frag[i] = fetch(i);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (i + PREFETCH < 16) frag[i + PREFETCH] = fetch(i + PREFETCH);
            const int g = i >> 2;
            u32x4 pw = {pb[g >> 1][4 * (g & 1)], pb[g >> 1][4 * (g & 1) + 1],
                        pb[g >> 1][4 * (g & 1) + 2], pb[g >> 1][4 * (g & 1) + 3]};
            acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[i], __builtin_bit_cast(bf16x8, pw), acc[i & 3], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto rescale = [&](float mn, float alpha) __attribute__((always_inline)) {
        m = mn;
        l *= alpha;
        lr *= alpha;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[dt][r] *= alpha;
    };
    // P^T = exp2(S^T * c - m) of an unmasked block into pb; returns this lane's partial row sums: over
    // the unrounded FP32 probabilities, and (through lrs) over the BF16-rounded ones.
    auto probabilities = [&](f32x16 (&s)[2], float &lrs) __attribute__((always_inline)) -> float {
        float ls0 = 0.0f, ls1 = 0.0f, r0 = 0.0f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], c, -m));
                const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r + 1], c, -m));
                ls0 += e0;
                ls1 += e1;
                pb[t][r >> 1] = pack_bf16(e0, e1);
                r0 = add_bf16_pair(pb[t][r >> 1], r0);
            }
        lrs = r0;
        return ls0 + ls1;
    };
    // Raise the running maximum to cover the unmasked block in s; rescale the accumulator and row sum.
    // Maximum of the scaled scores of an unmasked block, per query (log2 units).
    auto block_maximum = [&](f32x16 (&s)[2]) __attribute__((always_inline)) -> float {
        auto extreme = [&](auto sign) __attribute__((always_inline)) -> float {
            constexpr bool NEG = decltype(sign)::value;
            float mx = ext3<NEG>(s[0][0], s[0][1], s[0][2]);
#pragma unroll
            for (int i = 3; i < 31; i += 2) mx = ext3<NEG>(mx, s[i >> 4][i & 15], s[(i + 1) >> 4][(i + 1) & 15]);
            return ext3<NEG>(mx, s[1][15], s[1][15]) * c;
        };
        return lane32_max(!SHARED && c < 0.0f ? extreme(std::true_type{}) : extreme(std::false_type{}));
    };
    auto raise_reference = [&](f32x16 (&s)[2]) __attribute__((always_inline)) {
        // (the same maximum without a branch on the sign: this code stands in the loop many times and is rarely run)
        float mx = s[0][0] * c;
#pragma unroll
        for (int i = 1; i < 32; ++i) mx = fmaxf(mx, s[i >> 4][i & 15] * c);
        const float mn = fmaxf(m, lane32_max(mx));
        rescale(mn, __builtin_amdgcn_exp2f(m - mn));
    };
    // Softmax of a block that may hold masked keys (diagonal block, tail block, or a block that lies
    // wholly past this wavefront's rows): key index per register, limit per lane.  Masked keys get
    // P = 0 exactly, whatever the score registers hold.
    auto softmax_masked = [&](f32x16 (&s)[2], int blk) __attribute__((always_inline)) {
        int ln = lane;
        PIN(ln);                // lane-derived values are formed here, not kept across the block loop
        int lim = keys() - 1;
        if (CAUSAL) lim = min(lim, q0 + (ln & 31) + offset());
        const int kidx = blk * BN + 4 * (ln >> 5);
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kidx + 32 * t + 8 * (r >> 2) + (r & 3);
                mx = fmaxf(mx, key <= lim ? s[t][r] * c : -INFINITY);
            }
        mx = lane32_max(mx);
        if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
            const float mn = fmaxf(m, mx);
            rescale(mn, (mn == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - mn));
        }
        const float mu = (m == -INFINITY) ? 0.0f : m;
        float ls = 0.0f;
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const int key = kidx + 32 * t + 8 * (r >> 2) + (r & 3);
                float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r], c, -mu));
                float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t][r + 1], c, -mu));
                e0 = (key <= lim) ? e0 : 0.0f;
                e1 = (key + 1 <= lim) ? e1 : 0.0f;
                ls += e0 + e1;
                pb[t][r >> 1] = pack_bf16(e0, e1);
                lr = add_bf16_pair(pb[t][r >> 1], lr);
            }
        l += ls;
    };

    // Fast iteration j: MFMAs of PV(j) and S(j+2) interleaved with the softmax of S(j+1) = scur.
    // Softmax is the same against any reference point, so the probabilities are formed against the
    // running maximum as it stands, WITHOUT looking for the block's maximum first.  Only if some lane's
    // partial row sum comes out above P_SUM_LIMIT (or is not a number) did the scores outgrow the
    // reference; then the whole wavefront raises the reference, rescales, and forms the probabilities
    // again.  That branch is wave-uniform and rare: with scores of bounded spread the reference
    // settles after the first blocks.
    // The iteration's four tile requests (K(j+4) from kp into stage kreq, V(j+2) from vp into stage vreq)
    // are spread over the block, one every eight slots, so that the wavefronts' requests do not queue up
    // behind each other in the address unit.
    // s0, s1, s2: stages of blocks j, j+1, j+2 (V is read from s0, K from s2; the requests go to s1 for K
    // and s2 for V).
    // The masked form (diagonal blocks, the partial last block, blocks past the end) does the same with
    // every probability whose key is not valid for the lane's row set to zero, whatever its score
    // register holds; its second pass is the masked softmax, which also copes with a row that has no
    // valid key so far (reference at minus infinity).  It issues no requests: those go through the
    // general form after the block.
    auto fused_iteration = [&](auto masked, f32x16 (&scur)[2], f32x16 (&snxt)[2], int s0, int s1, int s2,
                               const unsigned char *kp, const unsigned char *vp, int blk)
        __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked)::value;
        float ev[32];
        uint32_t pn[16];
        float ls0 = 0.0f, ls1 = 0.0f, lrn = 0.0f, arg = 0.0f;
        const uint32_t klds = lds_wave + s1, vlds = lds_wave + V_BASE + s2;
        int room = 0;       // masked form: key offset c within block blk is valid for this lane's row iff c <= room
        if (MASKED) {
            int ln = lane;
            PIN(ln);
            int lim = keys() - 1;
            if (CAUSAL) lim = min(lim, q0 + (ln & 31) + offset());
            room = lim - blk * BN - 4 * (ln >> 5);
        }
        // Variants 1..3 look for the block's maximum first (the classic running-maximum form); their
        // masked blocks take the MFMA sequence and the exact masked softmax one after the other.
        if (ATTN_SOFTMAX != 0 && MASKED) {
            mfma_block(snxt, s0, s2, [](int) __attribute__((always_inline)) {});
            softmax_masked(scur, blk);
            return;
        }
        float mref = m;     // reference point of this block's probabilities
        if (ATTN_SOFTMAX != 0) {
            const float mx = block_maximum(scur);
            mref = ATTN_SOFTMAX == 3 ? (mx > m + 8.0f ? mx : m) : fmaxf(m, mx);
        }
        mfma_block(snxt, s0, s2, [&](int slot) __attribute__((always_inline)) {
            // element `slot` of the 32 scores of this lane: its exponent was formed one slot earlier, exp now, row-sum add one
            // slot later, so that no instruction waits for the one in front of it (fma and exp in the same slot, us, in turn: 8 x
            // 4096, 16 heads 874.8 instead of 872.5, masked 494.4 instead of 488.4, 16 x 2048, masked 284.1 instead of 282.1: up to 1 %, little more than two runs differ)
            ev[slot] = __builtin_amdgcn_exp2f(slot == 0 ? __builtin_fmaf(scur[0][0], c, -mref) : arg);
            if (slot < 31) {
                arg = __builtin_fmaf(scur[(slot + 1) >> 4][(slot + 1) & 15], c, -mref);
                PIN(arg);
            }
            if (MASKED) {
                const int r = slot & 15;
                ev[slot] = (32 * (slot >> 4) + 8 * (r >> 2) + (r & 3) <= room) ? ev[slot] : 0.0f;
            }
            if (slot >= 1) {
                if ((slot - 1) & 1) { ls1 += ev[slot - 1]; PIN(ls1); } else { ls0 += ev[slot - 1]; PIN(ls0); }
            }
            // BF16 pair k once the PV MFMAs that read the old pb entry k have been issued
            // (entries 4g..4g+3 are read by the even slots 8g..8g+6): pair k goes at slot 2k+9
            if (slot >= 9 && (slot & 1)) {
                const int k = (slot - 9) >> 1;
                pn[k] = pack_bf16(ev[2 * k], ev[2 * k + 1]);
                PIN(pn[k]);
            }
            if (!MASKED) {
                static_assert(LPT == 2, "request slots below are written out for two loads per tile and wavefront");
                if (slot == 4) lds_dma16_imm<0>(kp, koff[0], klds);
                if (slot == 12) lds_dma16_imm<1024>(kp, koff[1], klds);
                if (slot == 20) lds_dma16_imm<0>(vp, voff[0], vlds);
                if (slot == 28) lds_dma16_imm<1024>(vp, voff[1], vlds);
            }
        });
        ls1 += ev[31];
#pragma unroll
        for (int k = 12; k < 16; ++k) pn[k] = pack_bf16(ev[2 * k], ev[2 * k + 1]);
        // The rounded row sum, all 16 dot instructions together after the block's last MFMA: they run on
        // the matrix pipe, and one between two MFMAs stalls both (measured: spread over the slots the
        // loop is 2.5 % slower, placed before the first MFMA of the block 4.5 % slower than here).
#pragma unroll
        for (int k = 0; k < 16; ++k) lrn = add_bf16_pair(pn[k], lrn);
#pragma unroll
        for (int k = 0; k < 16; ++k) pb[k >> 3][k & 7] = pn[k];
        float ls = ls0 + ls1;
        if (ATTN_SOFTMAX != 0) {
            // the accumulator holds P(j) V(j) against the old reference: bring it to the new one
            const float alpha = __builtin_amdgcn_exp2f(m - mref);
            // Variant 1 multiplies every time.  Its test never fails; it stands there because with the 64
            // multiplications in the same basic block as the MFMA sequence the register allocator spills
            // (32 to 100 bytes per lane), and a spill inside this loop is not acceptable (see wait_vmcnt).
            const bool raise = ATTN_SOFTMAX == 1 ? __builtin_amdgcn_ballot_w64(alpha <= 1.0f) != 0
                                                 : __builtin_amdgcn_ballot_w64(mref > m) != 0;
            if (raise) rescale(mref, alpha);
            l += ls;
            lr += lrn;
            return;
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(ls <= P_SUM_LIMIT)) != 0, 0)) {     // (out of line)
            if (MASKED) {
                softmax_masked(scur, blk);      // adds to l and lr itself
                ls = 0.0f;
                lrn = 0.0f;
            } else {
                raise_reference(scur);
                ls = probabilities(scur, lrn);
            }
        }
        l += ls;
        lr += lrn;
    };
    auto fast_iteration = [&](f32x16 (&scur)[2], f32x16 (&snxt)[2], int s0, int s1, int s2,
                              const unsigned char *kp, const unsigned char *vp) __attribute__((always_inline)) {
        fused_iteration(std::false_type{}, scur, snxt, s0, s1, s2, kp, vp, 0);
    };
    // General iteration j, unless block j (and with it every later block) is wholly masked for this
    // wavefront: the MFMAs of PV(j) and S(j+2) with the masked softmax of S(j+1) between them.
    auto general_iteration = [&](f32x16 (&scur)[2], f32x16 (&snxt)[2], int j) __attribute__((always_inline)) {
        if (j < n_w)
            fused_iteration(std::true_type{}, scur, snxt, stage_off(j), 0, stage_off(j + 2), nullptr, nullptr, j + 1);
    };

    // ---- SHARED: the end of a part.  A wavefront needs nothing but the same wavefront's parts of the item, so there is
    // no barrier here.  It leaves its part and counts itself, and the one that completes the count adds all parts up in
    // the order of the keys, so that the result does not depend on the order of arrival (nor on whether parts pass through the
    // pool at all: add_up below does the same sums).  Of two parts, the common
    // case in a line longer than the launch is wide, the second to arrive keeps its own in registers: the counter's
    // low half counts arrivals, the high half parts that are in memory (1 x 1111, 32 heads on 8, causal: 29.9 us, both parts
    // through memory 32.4; with more parts the extra round trip costs more than it saves: 700 x 20000, 16 heads, 142 us
    // against 123).  False if the item's rows are another's to finish.
    auto share_parts = [&](const Geo &g) __attribute__((always_inline)) -> bool {
        const Share sr = load_share();
        const uint32_t wgs = (uint32_t)sr.wgs, total = (uint32_t)sr.total;
        const uint32_t first = (uint32_t)(g.at + sr.extra);
        // the cuts inside the item: SHARE_MIN_PART <= cut - first <= blocks - SHARE_MIN_PART
        const int lo = (int)(((first + SHARE_MIN_PART) * wgs + total - 1) / total);
        const int hi = (int)(((first + (uint32_t)g.blocks - SHARE_MIN_PART + 1) * wgs + total - 1) / total) - 1;
        const int parts = __builtin_amdgcn_readfirstlane(hi - lo + 2);
        uint32_t *arrived = (uint32_t *)(g_pool + (size_t)unit * POOL_UNIT_BYTES) + 1 + g.item * NWAVES + wave;
        const __amdgpu_buffer_rsrc_t rs = pool_rsrc(unit, sr.units);
        // slot of part i: that of the workgroup, and for part 0 one of a second set, by item or by workgroup, whichever are fewer
        const int items = sr.groups * cold().sched.ntile;
        const int slot0 = __builtin_amdgcn_readfirstlane((int)wgs + (items < (int)wgs ? g.item : lo - 1));
        const int w = xcd * (int)(wgs >> 3) + slot;
        int ln = lane;
        PIN(ln);
        const uint32_t lane_at = ln * 16;
        auto slot_of = [&](int i) __attribute__((always_inline)) -> uint32_t {
            return SHARE_HEADER_BYTES + wave * SHARE_WAVE_BYTES + (uint32_t)(i == 0 ? slot0 : lo - 1 + i) * SHARE_SLOT_BYTES;
        };
        const int mine = w - (lo - 1);
        auto leave = [&]() __attribute__((always_inline)) {
            const uint32_t out = slot_of(mine);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                pool_store16(rs, lane_at, out + i * 1024, acc[i >> 2][4 * (i & 3)], acc[i >> 2][4 * (i & 3) + 1],
                             acc[i >> 2][4 * (i & 3) + 2], acc[i >> 2][4 * (i & 3) + 3]);
            pool_store16(rs, lane_at, out + 16 * 1024, m, l, lr, 0.0f);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // they have arrived
        };
        auto count = [&](uint32_t by) __attribute__((always_inline)) -> uint32_t {
            uint32_t n = 0;
            if (ln == 0) n = __hip_atomic_fetch_add(arrived, by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return __builtin_amdgcn_readfirstlane(n);
        };
        if (parts == 2) {
            uint32_t seen = count(1);
            if ((seen & 0xffff) == 0) {
                leave();
                count(0x10000);
                return false;
            }
            // The other has come here before and needs nothing to go on: the wait is for its stores, if they are under way.
            while ((seen >> 16) == 0) {
                __builtin_amdgcn_s_sleep(1);
                seen = __builtin_amdgcn_readfirstlane(__hip_atomic_load(arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            asm volatile("" ::: "memory");
            if (ln == 0) pool_clear(unit, arrived);
            const uint32_t in = slot_of(1 - mine);
            const u32x4 st = pool_load16(rs, lane_at, in + 16 * 1024);
            u32x4 x[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = pool_load16(rs, lane_at, in + k * 1024);
            const float mo = __uint_as_float(st[0]), M = fmaxf(m, mo);      // (neither is minus infinity)
            const float f = __builtin_amdgcn_exp2f(m - M), fo = __builtin_amdgcn_exp2f(mo - M);
            m = M;
            if (mine == 0) {
                l = __builtin_fmaf(fo, __uint_as_float(st[1]), f * l);
                lr = __builtin_fmaf(fo, __uint_as_float(st[2]), f * lr);
#pragma unroll
                for (int k = 0; k < 64; ++k)
                    acc[k >> 4][k & 15] = __builtin_fmaf(fo, __uint_as_float(x[k >> 2][k & 3]), f * acc[k >> 4][k & 15]);
            } else {
                l = __builtin_fmaf(f, l, fo * __uint_as_float(st[1]));
                lr = __builtin_fmaf(f, lr, fo * __uint_as_float(st[2]));
#pragma unroll
                for (int k = 0; k < 64; ++k)
                    acc[k >> 4][k & 15] = __builtin_fmaf(f, acc[k >> 4][k & 15], fo * __uint_as_float(x[k >> 2][k & 3]));
            }
            return true;
        }
        leave();
        if (count(1) != (uint32_t)parts - 1) return false;
        asm volatile("" ::: "memory");
        if (ln == 0) pool_clear(unit, arrived);
        // Part after part in halves of 32 accumulator elements, the next half always in flight.
        reset_state();
        u32x4 st, xa[8], xb[8];
        uint32_t in = slot_of(0);
        st = pool_load16(rs, lane_at, in + 16 * 1024);
#pragma unroll
        for (int k = 0; k < 8; ++k) xa[k] = pool_load16(rs, lane_at, in + k * 1024);
#pragma nounroll
        for (int i = 0; i < parts; ++i) {
#pragma unroll
            for (int k = 0; k < 8; ++k) xb[k] = pool_load16(rs, lane_at, in + (8 + k) * 1024);
            const float mi = __uint_as_float(st[0]), mn = fmaxf(m, mi);
            const float keep = (m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(m - mn);
            const float f = __builtin_amdgcn_exp2f(mi - mn);
            m = mn;
            l = __builtin_fmaf(f, __uint_as_float(st[1]), keep * l);
            lr = __builtin_fmaf(f, __uint_as_float(st[2]), keep * lr);
#pragma unroll
            for (int k = 0; k < 32; ++k)
                acc[k >> 4][k & 15] = __builtin_fmaf(f, __uint_as_float(xa[k >> 2][k & 3]), keep * acc[k >> 4][k & 15]);
            in = slot_of(min(i + 1, parts - 1));        // (the last part again, unused, at the end)
            st = pool_load16(rs, lane_at, in + 16 * 1024);
#pragma unroll
            for (int k = 0; k < 8; ++k) xa[k] = pool_load16(rs, lane_at, in + k * 1024);
#pragma unroll
            for (int k = 0; k < 32; ++k)
                acc[2 + (k >> 4)][k & 15] = __builtin_fmaf(f, __uint_as_float(xb[k >> 2][k & 3]), keep * acc[2 + (k >> 4)][k & 15]);
        }
        asm volatile("" ::: "memory");
        return true;
    };

    // The same without the pool: the parts of an item follow each other in this workgroup, and what the earlier ones add up to
    // waits meanwhile, half of the accumulator in the item's own rows of O, as many bytes, half in the LDS
    // region that would hold the next item's Q, and three numbers in registers.
    float mp = 0.0f, lp = 0.0f, lrp = 0.0f;
    auto add_up = [&](const Geo &g, bool goes_on) __attribute__((always_inline)) -> bool {
        const int Sq = cold().shape.Sq, o_row_bytes = cold().shape.Hq * HD * 2;
        int ln = lane;
        PIN(ln);
        // (rows past the end have nowhere to wait, and no result: the descriptor ends with the last row)
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            cold().o + ((size_t)((size_t)b * Sq + q0) * cold().shape.Hq + head) * HD, 0, max(min(Sq - q0, 32), 0) * o_row_bytes, 0x00020000);
        const uint32_t og = (uint32_t)(ln & 31) * (uint32_t)o_row_bytes + (ln >> 5) * (HD / 2 * 2);
        LDS_AS u32x4 *ol = (LDS_AS u32x4 *)(lds + Q_BASE + wave * Q_WAVE_BYTES) + ln;
        if (g.j0 > 0) {
            const float M = fmaxf(mp, m);       // (neither is minus infinity)
            const float keep = __builtin_amdgcn_exp2f(mp - M), f = __builtin_amdgcn_exp2f(m - M);
            m = M;
            l = __builtin_fmaf(f, l, keep * lp);
            lr = __builtin_fmaf(f, lr, keep * lrp);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const u32x4 x = i >= 8 ? ol[64 * (i - 8)] : __builtin_amdgcn_raw_buffer_load_b128(rs, og, i * 16, 0);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int e = 4 * (i & 3) + k;
                    acc[i >> 2][e] = __builtin_fmaf(f, acc[i >> 2][e], keep * __uint_as_float(x[k]));
                }
            }
        }
        if (!goes_on) return true;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const u32x4 x = {__float_as_uint(acc[i >> 2][4 * (i & 3)]), __float_as_uint(acc[i >> 2][4 * (i & 3) + 1]),
                             __float_as_uint(acc[i >> 2][4 * (i & 3) + 2]), __float_as_uint(acc[i >> 2][4 * (i & 3) + 3])};
            if (i >= 8) ol[64 * (i - 8)] = x;
            else __builtin_amdgcn_raw_buffer_store_b128(x, rs, og, i * 16, 0);
        }
        mp = m; lp = l; lrp = lr;
        return false;
    };

    // ---- the workgroup's items, one after the other
    int r = 0, grp = 0, tile = 0, at = 0;
    bool have;
    if (SHARED) {
        set_cuts();
        // (an item shorter than SHARE_MIN_PART may begin before cut_lo and still be this workgroup's)
        int grp0, tile0, at0;
        locate(max(cut_lo - SHARE_MIN_PART, 0), grp0, tile0, at0);
        grp = grp0; tile = tile0; at = at0;
        have = find_part(grp, tile, at);
        if (have) {
            // the pool units, from the LSE element of the item's first row (nothing writes a result there until this
            // workgroup has handed in its part)
            const Shape sh = load_shape();
            const int bh = fast_div(grp, sh.d_chunks), b = fast_div(bh, sh.d_hkv);
            const int head = (bh - b * p.Hkv) * sh.G + (grp - bh * sh.chunks) * sh.pack;
            unit = cold().unit;
            if (unit == POOL_NONE) {
                unit = ((const __attribute__((address_space(4))) uint32_t *)(uintptr_t)cold().lse)
                    [((size_t)b * sh.Hq + head) * sh.Sq + tile * sh.tile_pos];
                asm volatile("" : "+s"(unit));      // read once, here
                unit = pool_unmark(unit);
            }
            pooled = unit != POOL_NONE;
            if (!pooled) {
                grp = grp0; tile = tile0; at = at0;
                have = find_part(grp, tile, at);
            }
        }
        wg_barrier();       // every wavefront has read it before one of them stores a result
    } else {
        have = find_item(r, grp, tile);
    }
    Geo cur = {};
    if (have) {
        cur = geometry(grp, tile, at);
        load_q(cur);
    }
    bool warm = false;          // the first tiles of the item about to start were requested by the item before it
#ifdef ATTN_CLOCKS
    int item_no = 0;
#endif
#if defined(ATTN_CLOCKS) && ATTN_CLOCKS >= 2
    unsigned long long ph[11], ph_prev = 0, ph_item = 0;
#endif
    while (have) {
#if defined(ATTN_CLOCKS) && ATTN_CLOCKS >= 2
#pragma unroll
        for (int k = 0; k < 11; ++k) ph[k] = 0;
        if (!SHARED) ph_prev = ph_item = phase_now();
#endif
        enter(cur);
        reset_state();
        // the item after this one
        Geo nxt = cur;
        int r2 = r + 1;
        bool have2, goes_on = false;        // goes_on: the next part of the same item is this workgroup's as well
        if (SHARED) {
            goes_on = !pooled && cut_hi <= cur.at + cold().share.extra + cur.blocks - SHARE_MIN_PART;
            if (goes_on) {
                ++ahead;
                set_cuts();
                have2 = true;
            } else {
                if (ahead != 0) { ahead = 0; set_cuts(); }
                at += cur.blocks + cold().share.extra;
                if (++tile == cold().sched.ntile) { tile = 0; ++grp; }
                have2 = find_part(grp, tile, at);
            }
        } else {
            have2 = find_item(r2, grp, tile);
        }
        if (have2) nxt = geometry(grp, tile, at);
        // Its tiles K'(0..2), V'(0) ride on this item's last iterations (requests K(j+4), V(j+2) of
        // iterations j >= nblk-4), which takes four iterations to host them.
        warm_next = ATTN_ITEM_OVERLAP && have2 && pooled && nblk >= 2 + REQ_AHEAD && nxt.nblk > 0;
        nx_nblk = nxt.nblk; nx_kg = nxt.kg; nx_vg = nxt.vg;
        // Its Q goes into this wavefront's LDS region now (the epilogue of the item before is done with
        // it) and into registers when this item's last block is done; being the oldest request of the
        // item, it never holds up a wait for tiles.
        if (ATTN_ITEM_OVERLAP && have2 && pooled) request_q(nxt);

        if (nblk > 0) {
            // Iteration j reads K(j+2) and V(j) and requests K(j+4) and V(j+2) into the stages of K(j+1)
            // and V(j-1), whose last readers finished before the previous barrier.  It ends by waiting until
            // only those four loads are still in flight, i.e. until K(j+3) and V(j+1) have landed, then the
            // barrier publishes them.
            if (!warm) {
                // Every wavefront is past the last barrier of the item before, so no stage is being read.
                issue_tile(0, false);
                issue_tile(1, false);
                issue_tile(2, false);
                issue_tile(0, true);
                __builtin_amdgcn_s_waitcnt(wait_vmcnt(2 * LPT));   // K(0), K(1) landed
                wg_barrier();
            }
            // warm: K(0), K(1) landed before the last barrier of the item before, and Q is in registers
            ATTN_PHASE(0);
            qk_only(sa, stage_off(0));
            qk_only(sb, stage_off(1));
            ATTN_PHASE(1);
            // P(0).  A first block without masked keys (every one but a causal item's diagonal start or a
            // short tail) takes its maximum as the reference and has nothing to rescale yet; the masked
            // path also handles an empty first block.
            // In a shared item a row's scores may be minus infinity in all of a part's first block, and finite in another
            // part; any finite reference will do until this part sees a finite one.
            if (n_unm > 0) {
                m = block_maximum(sa);
                if (SHARED) m = fmaxf(m, -FLT_MAX);
                l = probabilities(sa, lr);
            } else {
                softmax_masked(sa, 0);
                if (SHARED) m = fmaxf(m, -FLT_MAX);
            }
            ATTN_PHASE(2);
            // K(2), V(0) landed: a warm item waited for them before the epilogue of the item before, and
            // what it still has in flight are that epilogue's stores, which nothing here depends on
            if (!warm) __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
            wg_barrier();                                 // and every wavefront is done with K(0), K(1)
            issue_tile(3, false);                         // the requests of "iteration -1"
            issue_tile(1, true);

            // Blocks >= n_unm go through the masked softmax, which yields P = 0 where a key is not valid:
            // blocks masked out entirely for this wavefront, and the blocks past the end that the last
            // iterations multiply from stages that hold other tiles, then contribute nothing, with no
            // branch around the MFMA sequences.  Iteration j: scur = S(j+1) (sb for even j), snxt
            // receives S(j+2).
            int j = 0;
            ATTN_STAMP(0, __builtin_readcyclecounter());
            ATTN_PHASE(3);
            // Iterations j < fast_end take the fast path: S(j+1) needs no mask, and the tiles requested are
            // full ones (past the last block: of the next item, or the last block again).
            const int fast_end = all_full ? n_unm - 1 : min(n_unm - 1, (SHARED ? keys() / BN : nfull) - (2 + REQ_AHEAD));
            // Request addresses of the fast loop.  K and V have the same shape, so V's address is K's of
            // two iterations earlier plus the distance between the tensors; K's moves on by one tile per
            // iteration, except at the item's last block (on to block 0 of the next item, or stay) and,
            // if there is no next item, after it (stay).
            const ptrdiff_t dv = (const unsigned char *)p.v - (const unsigned char *)p.k;
            int unused, unused2;
            const unsigned char *kp = uniform_ptr(tile_ptr(2 + REQ_AHEAD, false, unused, unused2));
            const unsigned char *vp = uniform_ptr(tile_ptr(REQ_AHEAD, true, unused, unused2));
            const unsigned char *vp1 = uniform_ptr(tile_ptr(1 + REQ_AHEAD, true, unused, unused2));
            int kleft = nblk - 1 - (2 + REQ_AHEAD);      // whole-tile steps left before K's request reaches the last block
            const ptrdiff_t kjump = warm_next ? nx_kg - (kg + (size_t)(nblk - 1) * tile_gbytes) : 0;
            const ptrdiff_t kafter = warm_next ? (ptrdiff_t)tile_gbytes : 0;
            // (written out twice below rather than as a lambda: selecting between captured variables
            // would keep them in memory)
#define ATTN_ADVANCE_REQUESTS()                                                              \
            do {                                                                             \
                ptrdiff_t step = kleft < 0 ? kafter : kjump;                                 \
                step = kleft > 0 ? (ptrdiff_t)tile_gbytes : step;                            \
                vp = vp1;                                                                    \
                vp1 = kp + dv;                                                               \
                kp += step;                                                                  \
                --kleft;                                                                     \
            } while (0)
#define ATTN_FAST(scur, snxt, a0, a1, a2)                                                    \
            do {                                                                             \
                fast_iteration(scur, snxt, a0, a1, a2, kp, vp);                              \
                ATTN_ADVANCE_REQUESTS();                                                     \
                __builtin_amdgcn_s_waitcnt(WAIT_ITER_END);                                   \
                wg_barrier();                                                                \
                ATTN_PHASE(4);                                                               \
                ATTN_PHASE_COUNT(5);                                                         \
            } while (0)
            // The bulk of the fast iterations runs in a loop unrolled six times (two score buffers x three
            // stages), in which every LDS address is a register plus a constant.  That loop wants block j in
            // stage 0; a two-iteration loop with the stages in registers brings j there, and takes what
            // is left afterwards.
            static_assert(NSTAGE == 3, "the unrolled loop below is written for three stages");
            const int j_align = ring0 == 0 ? 0 : 2 * ring0 == 2 ? 2 : 4;     // smallest even j with (ring0 + j) % 3 == 0
#pragma nounroll
            for (int round = 0; round < 2; ++round) {
                const int lim = round == 0 ? min(fast_end, j_align) : fast_end;
                int s0 = stage_off(j), s1 = stage_off(j + 1), s2 = stage_off(j + 2);
#pragma nounroll
                for (; j + 1 < lim; j += 2) {
                    ATTN_FAST(sb, sa, s0, s1, s2);
                    ATTN_FAST(sa, sb, s1, s2, s0);
                    { const int t = s0; s0 = s2; s2 = s1; s1 = t; }
                }
                if (round == 0) {
                    constexpr int T0 = 0, T1 = TILE_BYTES, T2 = 2 * TILE_BYTES;
#pragma nounroll
                    for (; j + 5 < fast_end; j += 6) {
                        ATTN_FAST(sb, sa, T0, T1, T2);
                        ATTN_FAST(sa, sb, T1, T2, T0);
                        ATTN_FAST(sb, sa, T2, T0, T1);
                        ATTN_FAST(sa, sb, T0, T1, T2);
                        ATTN_FAST(sb, sa, T1, T2, T0);
                        ATTN_FAST(sa, sb, T2, T0, T1);
                    }
                }
            }
            // an item without masks whose last fast iteration is left over by the loops of two
            if (j == nblk - 2 && fast_end == nblk - 1) {
                ATTN_FAST(sb, sa, stage_off(j), stage_off(j + 1), stage_off(j + 2));
                ++j;
            }
#undef ATTN_FAST
#undef ATTN_ADVANCE_REQUESTS
            // The last iteration of an item that warms up the next one requests nothing (K'(3) would
            // land in the stage of K'(0), which is read only after this item's last barrier).
            auto iteration_end = [&](int jj) __attribute__((always_inline)) {
                if (!(warm_next && jj == nblk - 1)) {
                    issue_tile(jj + 2 + REQ_AHEAD, false);
                    issue_tile(jj + REQ_AHEAD, true);
                }
                __builtin_amdgcn_s_waitcnt(WAIT_ITER_END);
                wg_barrier();
                if (jj == nblk - 1) {
                    ATTN_PHASE(8);
                } else {
                    ATTN_PHASE(6);
                    ATTN_PHASE_COUNT(7);
                }
            };
#pragma nounroll
            for (; j < nblk - 1; j += 2) {
                general_iteration(sb, sa, j);
                iteration_end(j);
                if (j + 1 < nblk - 1) {
                    general_iteration(sa, sb, j + 1);
                    iteration_end(j + 1);
                }
            }
            // the last iteration has only its PV product left to do
            if (nblk - 1 < n_w) pv_only(stage_off(nblk - 1));
            iteration_end(nblk - 1);
            ATTN_STAMP(1, __builtin_readcyclecounter());
            ATTN_STAMP(2, (unsigned long long)nblk);
        }
        // Nothing may still be writing LDS at exit; the next item's Q has landed; and its K'(2), V'(0) are
        // waited for here, before the epilogue's stores join the queue, so that its first barrier can
        // publish them.
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
        ATTN_PHASE(9);

        bool last_part = true;
        if (SHARED && (cur.j0 != 0 || cur.nblk != cur.blocks)) {        // a part, not a whole item
            if (pooled) {
                last_part = share_parts(cur);
                mp = lp = lrp = 0.0f;       // (unused, and no register for them through the above)
            } else {
                last_part = add_up(cur, goes_on);
            }
            read_addresses();
        }
        // ---- Q of the next item into registers, from this wavefront's LDS region
        // (SHARED: also if there is none, so that the old values are not kept through the above)
        if (ATTN_ITEM_OVERLAP && (SHARED || have2)) {
#pragma unroll
            for (int s = 0; s < 8; ++s)
                qf[s] = *(const LDS_AS bf16x8 *)(lds + Q_BASE + wave * Q_WAVE_BYTES + kaddr[s]);
        }
        if (ATTN_ITEM_OVERLAP && have2) negate_q();
        if (last_part) {
            // ---- epilogue: O = acc / lr (BF16), LSE = ln2 * (m + log2 l).  A lane holds one query's values
            // in pieces of 8 bytes; they go through the same LDS region (32 rows of 256 bytes, 16-byte units
            // swizzled by the row), so that each store instruction writes whole rows.
            const float lt = lane32_sum(l);
            const float lrt = lane32_sum(lr);
            const float inv = lrt > 0.0f ? 1.0f / lrt : 0.0f;
            {
                const int ob = Q_BASE + wave * Q_WAVE_BYTES;
                int ln = lane;
                PIN(ln);        // per-lane offsets are formed here, not kept in registers across the block loop
                const int orow = ln >> 4, ounit = ln & 15, l32 = ln & 31, hh = ln >> 5;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int rg = 0; rg < 4; ++rg) {
                        u32x2 ww = {pack_bf16(acc[dt][4 * rg] * inv, acc[dt][4 * rg + 1] * inv),
                                    pack_bf16(acc[dt][4 * rg + 2] * inv, acc[dt][4 * rg + 3] * inv)};
                        *(LDS_AS u32x2 *)(lds + ob + l32 * ROW_BYTES + (((4 * dt + rg) ^ (l32 & 15)) << 4) + 8 * hh) = ww;
                    }
                const int Sq = cold().shape.Sq, Hq = cold().shape.Hq;
                const size_t o_row_bytes = (size_t)Hq * HD * 2;
                unsigned char *og = (unsigned char *)(cold().o + ((size_t)((size_t)b * Sq + q0) * Hq + head) * HD);
                const int rows = Sq - q0;               // rows of this wavefront that exist
                // (the row pitch is below 2^23 bytes, so the lane's first offset fits 32 bits; the rest are additions)
                unsigned char *gp = og + ((uint32_t)orow * (uint32_t)o_row_bytes + 16u * (uint32_t)ounit);
                const size_t gstep = 4 * o_row_bytes;
                if (rows >= 32) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int row = 4 * i + orow;
                        const u32x4 val = *(const LDS_AS u32x4 *)(lds + ob + row * ROW_BYTES + ((ounit ^ (row & 15)) << 4));
                        *(u32x4 *)gp = val;
                        gp += gstep;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int row = 4 * i + orow;
                        const u32x4 val = *(const LDS_AS u32x4 *)(lds + ob + row * ROW_BYTES + ((ounit ^ (row & 15)) << 4));
                        if (row < rows) *(u32x4 *)gp = val;
                        gp += gstep;
                    }
                }
                if (l32 < rows && hh == 0) {
                    const float lse = lt > 0.0f ? (m + __builtin_amdgcn_logf(lt)) * 0.6931471805599453f : -INFINITY;
                    cold().lse[((size_t)b * Hq + head) * Sq + q0 + l32] = lse;
                }
            }

        }
        if ((!ATTN_ITEM_OVERLAP || !pooled) && (SHARED || have2)) load_q(nxt);
#if defined(ATTN_CLOCKS) && ATTN_CLOCKS >= 2
        ATTN_PHASE(10);
        if (!SHARED && bid == 0 && item_no == 1 && (tid == 0 || tid == NTHREADS - 64)) {
#pragma unroll
            for (int k = 0; k < 11; ++k) g_phases[tid != 0][k] = ph[k];
            g_phases[tid != 0][11] = ph_prev - ph_item;
        }
#endif
#ifdef ATTN_CLOCKS
        ++item_no;
#endif
        ring0 = (ring0 + nblk) % NSTAGE;
        warm = warm_next;
        have = have2;
        r = r2;
        cur = nxt;
    }
    if (SHARED && unit != POOL_NONE) {
        // Every workgroup has a part of some item and so knows the units; the last one to leave gives them back.  (One count
        // per workgroup: 8 per item, all on one address, took 16 us of a launch of 512 items.)
        wg_barrier();
        if (tid == 0) {
            const Share sr = load_share();
            uint32_t *left = (uint32_t *)(g_pool + (size_t)unit * POOL_UNIT_BYTES);
            const uint32_t n = __hip_atomic_fetch_add(left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (n == (uint32_t)sr.wgs - 1) {
                pool_clear(unit, left);
                pool_give(unit, sr.units);
            }
        }
    }
#ifdef ATTN_CLOCKS
    if (bid == 0 && tid == 0) { g_clocks[1] = __builtin_readcyclecounter(); g_clocks[3] = wall_clock64(); }
#endif
}

// ---------------------------------------------------------------------------------------------------
// The kernel for small problems.  With 256 query rows per work item a short query sequence (or few
// heads) leaves most compute units without work, however long the key sequence is.  Here a work item
// is 32 query rows that share a K/V head -- PACK query heads of one group x 32/PACK positions, so that
// grouped-query heads share the K/V blocks here too -- and the eight wavefronts of the workgroup share its
// KEYS instead of its rows: wavefront w takes the 32-key blocks w, w + 8, ... with a running maximum and running
// sums of its own (the same online softmax, paper section 2.2), staging its K and V blocks through a
// private 16 KiB of LDS, and the eight partial results are merged through LDS at the end:
//     M = max_w m_w,  f_w = 2^(m_w - M),  O = sum_w f_w acc_w / sum_w f_w lr_w,  LSE = ln2 (M + log2 sum_w f_w l_w).
// No barrier inside the key loop.
//
// When the items are fewer than the compute units, or would leave part of a round of them without work for long, each item is
// shared by `splits` workgroups, which take contiguous ranges of its key blocks.  They leave (acc, m, l, lr) in device memory and the one that arrives last
// merges them, in the order of the ranges, whatever the order of arrival, so that the result does not depend on it.  Nor does it
// depend on the memory: where none is free, an item's first workgroup takes the same ranges one after the other and adds them up
// the same way.
struct SplitParams {
    const __bf16 *q, *k, *v;
    __bf16 *o;
    float *lse;
    int Hq, Hkv, Sq, Skv, G;
    int pack, pack_log2;    // query heads of one K/V group in a work item (8, 4, 2 or 1); row r is head r % pack, position r / pack
    int chunks;             // G / pack
    int tile_pos;           // query positions per work item = 32 / pack
    int ntile;              // ceil(Sq / tile_pos)
    int nrest;              // B * Hkv * chunks; items = ntile * nrest
    Div d_nrs, d_chunks, d_hkv;     // exact division by nrest * splits, chunks, Hkv
    int off;                // key j valid iff j <= i + off: Skv - Sq, or without a mask a number that makes all of them valid
    float c;                // scale * log2(e)
    // (up to here, within two cache lines, what items of one workgroup need; for the shared form:)
    int splits;             // workgroups that share an item
    int once;               // K and V are read once and past the caches
    Div d_splits;
    int units;              // POOL_UNIT_BYTES units of device memory the launch needs, 0 if splits == 1
    uint32_t unit;          // REGION_SPLIT_UNIT if the launch has the region, POOL_SOLO if splits == 1, or POOL_NONE
    int reserve;            // > 0: this launch is one workgroup that takes the units for the launch behind it, and clears
                            // this many counters per item (the item geometry is that launch's); < 0: one that gives them
                            // back, because there was no launch behind it
};
static_assert(offsetof(SplitParams, splits) <= 128, "two cache lines of kernel arguments");
constexpr int SPLIT_TILE_BYTES = SPLIT_KEYS * ROW_BYTES;        // 8 KiB: one K or V block
constexpr int SPLIT_WAVE_BYTES = 2 * SPLIT_TILE_BYTES;          // per wavefront: its K block, then its V block
constexpr int SPLIT_STATE_BASE = NWAVES * SPLIT_WAVE_BYTES;     // after them: m, l, lr of every wavefront
constexpr int SPLIT_Q_BASE = SPLIT_STATE_BASE + NWAVES * 3 * 32 * 4;   // then the item's 32 Q rows (K's swizzle)
constexpr int SPLIT_LDS_BYTES = SPLIT_Q_BASE + 32 * ROW_BYTES;
static_assert(SPLIT_Q_BASE % 1024 == 0 && NWAVES * 4 == 32, "each wavefront requests four of the 32 Q rows, 1 KiB");
static_assert(SPLIT_WAVE_BYTES == 32 * HD * 4, "a wavefront's partial accumulator takes the place of its two blocks");
static_assert(SPLIT_LDS_BYTES <= LDS_BYTES, "a workgroup fits a CU");

// Two forms: items of one workgroup each, and SHARED ones (with the launch in front of them), which also takes the calls whose K and V are
// read past the caches: 1.3 KB more code, which cost small launches 0.2 us of 12.5 in the other form.  The mask is a number, not a
// form: every block goes through the masked softmax anyway.  (One kernel for both, with the code of the shared items beside
// the rest: 64 items of 512 keys 8.0 us instead of 7.7, 60 of 45 keys 5.7 instead of 5.45.)
template <bool SHARED>
__global__ __launch_bounds__(NTHREADS) void attn_fwd_split_kernel(const SplitParams p)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    // blockIdx.x -> (tile, rest, part), parts fastest and tiles slowest, last tile first: under the causal mask
    // the long items start first, and where nrest * splits is a multiple of 8 the workgroups that read
    // the same keys are on one XCD (204 x 4354, 32 heads, without a mask: 32.5 us, tiles fastest 74.5).
    const int bid = blockIdx.x;
#ifdef ATTN_CLOCKS
    if (bid == 0 && tid == 0) { g_clocks[2] = wall_clock64(); g_clocks[0] = __builtin_readcyclecounter(); }
#endif
    // first element of an item's LSE
    auto item_lse = [&](int rest, int q0) __attribute__((always_inline)) -> size_t {
        const int bh = fast_div(rest, p.d_chunks), chunk = rest - bh * p.chunks;
        const int b = fast_div(bh, p.d_hkv), hkv = bh - b * p.Hkv;
        return ((size_t)b * p.Hq + hkv * p.G + chunk * p.pack) * p.Sq + q0;
    };
    if (SHARED && p.reserve < 0) {
        const uint32_t unit = pool_unmark(((const uint32_t *)p.lse)[item_lse(0, 0)]);
        if (tid == 0 && unit != POOL_NONE) pool_give(unit, p.units);
        return;
    }
    if (SHARED && p.reserve) {
        uint32_t *shared = (uint32_t *)smem;
        if (tid == 0) shared[0] = pool_take(p.units);
        __syncthreads();
        const uint32_t unit = shared[0];
        const int items = p.nrest * p.ntile;
        if (unit != POOL_NONE) {
            uint32_t *header = (uint32_t *)(g_pool + (size_t)unit * POOL_UNIT_BYTES);
            for (int i = tid; i <= items * p.reserve; i += NTHREADS) header[i] = 0;
        }
        for (int i = tid; i < items; i += NTHREADS)
            ((uint32_t *)p.lse)[item_lse(i % p.nrest, i / p.nrest * p.tile_pos)] = pool_mark(unit);
        return;
    }
    const int tile_r = fast_div(bid, p.d_nrs), rest_s = bid - tile_r * (SHARED ? p.nrest * p.splits : p.nrest);
    int rest = rest_s, part = 0;
    if (SHARED) {
        rest = fast_div(rest_s, p.d_splits);
        part = rest_s - rest * p.splits;
    }
    const int tile = p.ntile - 1 - tile_r;
    const int bh = fast_div(rest, p.d_chunks), chunk = rest - bh * p.chunks;
    const int b = fast_div(bh, p.d_hkv), hkv = bh - b * p.Hkv;
    const int q0 = tile * p.tile_pos;
    // this lane's query: head and position (rows past the end of Q compute on the last row and are not stored)
    const int head = hkv * p.G + chunk * p.pack + (l32 & (p.pack - 1));
    const int qpos = q0 + (l32 >> p.pack_log2);
    // keys 0 .. klast are valid for some row of the tile
    const int klast = min(p.Skv - 1, min(q0 + p.tile_pos - 1, p.Sq - 1) + p.off);
    const int item_nb = klast < 0 ? 0 : klast / SPLIT_KEYS + 1;
    int first = 0, nb = item_nb;        // this workgroup's blocks: first .. nb - 1
    // SHARED: part i, of `splits` ranges of equal length (the last ones may be shorter or empty)
    auto take_part = [&](int i) __attribute__((always_inline)) {
        const int len = fast_div(item_nb + p.splits - 1, p.d_splits);
        first = min(item_nb, i * len);
        nb = min(item_nb, first + len);
    };
    uint32_t unit = POOL_NONE;
    if (SHARED) {
        // (read as a constant: where units were taken, nothing writes it until every workgroup of the item has read it)
        unit = p.unit;
        if (unit == POOL_NONE) {
            unit = ((const __attribute__((address_space(4))) uint32_t *)(uintptr_t)p.lse)[item_lse(rest, q0)];
            asm volatile("" : "+s"(unit));      // read once, here
            unit = pool_unmark(unit);
        }
        if (unit == POOL_NONE && part != 0) return;
        take_part(part);
    }
    const size_t kv_row_bytes = (size_t)p.Hkv * HD * 2;
    const unsigned char *kg = (const unsigned char *)(p.k + ((size_t)b * p.Skv * p.Hkv + hkv) * HD);
    const unsigned char *vg = (const unsigned char *)(p.v + ((size_t)b * p.Skv * p.Hkv + hkv) * HD);

    const uint32_t kbase = wave * SPLIT_WAVE_BYTES, vbase = kbase + SPLIT_TILE_BYTES;
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    // One block = 8 requests of 1 KiB (4 rows): lane L's 16 bytes land at base + 16 L, and the lane
    // fetches the logical 16-byte unit that the swizzle of the main kernel puts there.
    uint32_t koff[8], voff[8];      // byte offset of this lane's 16 bytes from the first row of a full block
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 4 * i + (lane >> 4), unit = lane & 15;
        koff[i] = (uint32_t)(row * kv_row_bytes) + ((unit ^ (row & 15)) << 4);
        voff[i] = (uint32_t)(row * kv_row_bytes) + ((unit ^ ((row & 3) << 2)) << 4);
    }
    auto request = [&](int blk, bool is_v) __attribute__((always_inline)) {
        const unsigned char *g = uniform_ptr((is_v ? vg : kg) + (size_t)blk * SPLIT_KEYS * kv_row_bytes);
        const int last = p.Skv - 1 - blk * SPLIT_KEYS;      // rows past the end of K/V re-read the last row
        const uint32_t dst = lds0 + (is_v ? vbase : kbase);
        if (SHARED && last >= SPLIT_KEYS - 1 && p.once) {
#pragma unroll
            for (int i = 0; i < 8; ++i) lds_dma16_once(g, is_v ? voff[i] : koff[i], dst + i * 1024);
        } else if (last >= SPLIT_KEYS - 1) {
#pragma unroll
            for (int i = 0; i < 8; ++i) lds_dma16(g, is_v ? voff[i] : koff[i], dst + i * 1024);
        } else {
            int ln = lane;
            if (SHARED) PIN(ln);        // formed here, not kept in registers through all parts
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = 4 * i + (ln >> 4);
                const uint32_t o = (is_v ? voff[i] : koff[i]) - (uint32_t)(row * kv_row_bytes) + (uint32_t)(min(row, last) * kv_row_bytes);
                lds_dma16(g, o, dst + i * 1024);
            }
        }
    };
    // What the first MFMA needs goes out first, and before anything else is computed: the eight wavefronts'
    // first blocks are 128 KiB through a load path of 64 bytes a clock, the longest single stretch of a
    // small launch.  The item's 32 Q rows go through LDS as well, each wavefront requesting four of them
    // (rows past the end re-read the last row): fetched by every wavefront for itself they would be
    // another 64 KiB on that path, and as ordinary loads they would make the compiler's own count of
    // outstanding loads, which knows nothing of the requests around them, wait for V before the first MFMA.
    {
        const int r = 4 * wave + (lane >> 4), unit = lane & 15;
        const int row0 = min(q0, p.Sq - 1);
        const int drow = min(q0 + (r >> p.pack_log2), p.Sq - 1) - row0;         // 0 .. 31
        const int dhead = r & (p.pack - 1);
        const unsigned char *qg = (const unsigned char *)(p.q + ((size_t)((size_t)b * p.Sq + row0) * p.Hq + hkv * p.G + chunk * p.pack) * HD);
        // (at most 32 rows of at most 32768 heads of 256 bytes: the offset fits 32 bits)
        const uint32_t o = (uint32_t)(drow * p.Hq + dhead) * (uint32_t)(HD * 2) + ((unit ^ (r & 15)) << 4);
        lds_dma16(qg, o, lds0 + SPLIT_Q_BASE + wave * 1024);
    }
    int t = first + wave;
    if (t < nb) {
        request(t, false);
        request(t, true);
    }
    __builtin_amdgcn_sched_barrier(0);
    f32x16 acc[4];
    float m, l, lr;
    auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[dt][r] = 0.0f;
        m = -INFINITY;
        l = lr = 0.0f;
    };
    reset_state();
    // SHARED: what the parts of an item add up to, as far as they have been added, for the eight outputs of this thread.
    // Four parts at a time (fewer rescalings than one by one), and the same operations in the same order wherever the parts
    // come from, so that results do not depend on that.
    constexpr int GROUP = 4;
    struct Parts { float m[GROUP], l[GROUP], r[GROUP], x[GROUP][8]; };
    float M = -INFINITY, L = 0.0f, LR = 0.0f, o8[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) o8[j] = 0.0f;
    auto no_part = [&](Parts &g, int i) __attribute__((always_inline)) {        // adds nothing
        g.m[i] = -INFINITY;
        g.l[i] = g.r[i] = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) g.x[i][j] = 0.0f;
    };
    auto add_parts = [&](const Parts &g) __attribute__((always_inline)) {
        float mn = M;
#pragma unroll
        for (int i = 0; i < GROUP; ++i) mn = fmaxf(mn, g.m[i]);
        const float keep = (M == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(M - mn);
        M = mn;
        L *= keep;
        LR *= keep;
#pragma unroll
        for (int j = 0; j < 8; ++j) o8[j] *= keep;
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
            const float f = (g.m[i] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(g.m[i] - mn);
            L = __builtin_fmaf(f, g.l[i], L);
            LR = __builtin_fmaf(f, g.r[i], LR);
#pragma unroll
            for (int j = 0; j < 8; ++j) o8[j] = __builtin_fmaf(f, g.x[i][j], o8[j]);
        }
    };
    Parts group;        // of a workgroup that takes all parts: those not added yet
    int kaddr[8];
#pragma unroll
    for (int st = 0; st < 8; ++st) kaddr[st] = kbase + l32 * ROW_BYTES + (((2 * st + hh) ^ (l32 & 15)) << 4);
    int vaddr[4];
    {
        const int i16 = lane & 15, g = (lane >> 4) & 1;
        const int row = 4 * hh + (i16 >> 2);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const int d = 32 * dt + 16 * g + 4 * (i16 & 3);
            vaddr[dt] = vbase + row * ROW_BYTES + ((((d >> 3) ^ ((row & 3) << 2))) << 4) + (d & 7) * 2;
        }
    }

    // this wavefront's Q rows have landed (and K(t), if it has a block: both are older than V(t)'s
    // eight requests); the barrier publishes all 32 rows
    if (t < nb) __builtin_amdgcn_s_waitcnt(wait_vmcnt(8)); else __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    wg_barrier();
    bf16x8 qf[8];           // Q^T operand: query l32, d = 16 s + 8 hh .. + 7
#pragma unroll
    for (int s = 0; s < 8; ++s)
        qf[s] = *(const LDS_AS bf16x8 *)(lds + SPLIT_Q_BASE + l32 * ROW_BYTES + (((2 * s + hh) ^ (l32 & 15)) << 4));
    // a negative scale: the negated Q (exact) with the scale's absolute value
    const float c = fabsf(p.c);
    if (p.c < 0.0f) {
#pragma unroll
        for (int s = 0; s < 8; ++s) qf[s] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[s]) ^ 0x80008000u);
    }

    float mp, lp, rp, x[8];         // what the loop below leaves: this part's result for this thread's eight outputs
    // (one turn; where items are shared and no units were free, one for each part)
    for (;;) {
        // Blocks first + wave, first + wave + 8, ...: K(t) and V(t) were requested above (this wavefront's first block); K(t + 8) goes out as soon as the
        // score MFMAs have read K(t), V(t + 8) as soon as the PV MFMAs have read V(t), so that a wait is "all
        // but the newest eight requests have landed" while there is a next block and "all" at the last one.
        for (; t < nb; t += NWAVES) {
            const bool more = t + NWAVES < nb;
            __builtin_amdgcn_s_waitcnt(wait_vmcnt(8));          // K(t) has landed
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.0f;
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                bf16x8 a = *(const LDS_AS bf16x8 *)(lds + kaddr[st]);
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[st], s, 0, 0, 0);
            }
            // (the MFMAs above hold K(t) in registers: the compiler has waited for the LDS reads)
            __builtin_amdgcn_sched_barrier(0);
            if (more) request(t + NWAVES, false);
            // exact online softmax of the block, masked per key
            const int lim = min(p.Skv - 1, qpos + p.off);
            const int kidx = t * SPLIT_KEYS + 4 * hh;
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int key = kidx + 8 * (r >> 2) + (r & 3);
                mx = fmaxf(mx, key <= lim ? s[r] : -INFINITY);
            }
            mx = lane32_max(mx);
            mx = (mx == -INFINITY) ? -INFINITY : mx * c;
            if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
                const float mn = fmaxf(m, mx);
                const float alpha = (mn == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - mn);
                m = mn;
                l *= alpha;
                lr *= alpha;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[dt][r] *= alpha;
            }
            const float mu = (m == -INFINITY) ? 0.0f : m;
            uint32_t pb[8];
            float ls = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) {
                const int key = kidx + 8 * (r >> 2) + (r & 3);
                float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -mu));
                float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r + 1], c, -mu));
                e0 = (key <= lim) ? e0 : 0.0f;
                e1 = (key + 1 <= lim) ? e1 : 0.0f;
                ls += e0 + e1;
                pb[r >> 1] = pack_bf16(e0, e1);
                lr = add_bf16_pair(pb[r >> 1], lr);
            }
            l += ls;
            // V(t) has landed: behind it in the queue are the requests of K(t + 8), if there is such a block
            if (more) __builtin_amdgcn_s_waitcnt(wait_vmcnt(8)); else __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                u32x4 pw = {pb[4 * g], pb[4 * g + 1], pb[4 * g + 2], pb[4 * g + 3]};
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) {
                    const int ro = g * 16 * ROW_BYTES;
                    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + vaddr[dt] + ro));
                    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + vaddr[dt] + (ro + 8 * ROW_BYTES)));
                    s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av),
                                                                       __builtin_bit_cast(bf16x8, pw), acc[dt], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (more) request(t + NWAVES, true);
        }
        // nothing of this wavefront's is still on its way into LDS (the last block waited for everything),
        // and its MFMAs have read their operands
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);

        // ---- merge.  Each wavefront leaves its accumulator as FP32 [query][d] in its own 16 KiB (its blocks
        // are dead), the 16-byte units of a query's row swizzled by the query so that the 32 lanes of a
        // store or load touch 32 different units, and its m, l, lr in the state area; wavefront w then
        // combines d = 16 w .. 16 w + 15.
        typedef float f32x4 __attribute__((ext_vector_type(4)));
        int l32 = lane & 31, hh = lane >> 5;
        if (SHARED) { PIN(l32); PIN(hh); }      // what follows is formed here in every turn, not kept through the blocks
        {
            LDS_AS unsigned char *part = lds + wave * SPLIT_WAVE_BYTES + l32 * (HD * 4);
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int rg = 0; rg < 4; ++rg) {
                    const int u = 8 * dt + 2 * rg + hh;          // d = 4 u .. 4 u + 3
                    const f32x4 val = {acc[dt][4 * rg], acc[dt][4 * rg + 1], acc[dt][4 * rg + 2], acc[dt][4 * rg + 3]};
                    *(LDS_AS f32x4 *)(part + ((u ^ l32) << 4)) = val;
                }
            // every lane of a query holds the same m; l and lr are the lane's share: add the two halves
            const float lt = lane32_sum(l), lrt = lane32_sum(lr);
            LDS_AS float *state = (LDS_AS float *)(lds + SPLIT_STATE_BASE) + wave * 96;
            if (hh == 0) {
                state[l32] = m;
                state[32 + l32] = lt;
                state[64 + l32] = lrt;
            }
        }
        __syncthreads();
        mp = -INFINITY;
        lp = rp = 0.0f;
        {
            const LDS_AS float *state = (const LDS_AS float *)(lds + SPLIT_STATE_BASE);
            float mw[NWAVES];
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) {
                mw[w] = state[w * 96 + l32];
                mp = fmaxf(mp, mw[w]);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) x[j] = 0.0f;
#pragma unroll
            for (int w = 0; w < NWAVES; ++w) {
                const float f = (mw[w] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(mw[w] - mp);
                lp += f * state[w * 96 + 32 + l32];
                rp += f * state[w * 96 + 64 + l32];
                const LDS_AS unsigned char *part = lds + w * SPLIT_WAVE_BYTES + l32 * (HD * 4);
                const int u = 4 * wave + 2 * hh;
                const f32x4 lo = *(const LDS_AS f32x4 *)(part + ((u ^ l32) << 4));
                const f32x4 hi = *(const LDS_AS f32x4 *)(part + (((u + 1) ^ l32) << 4));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    x[j] += f * lo[j];
                    x[4 + j] += f * hi[j];
                }
            }
        }
        if (!SHARED || unit != POOL_NONE) break;
        // No units: all parts one after the other, added up like those that come from memory.
        const int k = part % GROUP;
#pragma unroll
        for (int i = 0; i < GROUP; ++i) {
            if (i == k) {
                group.m[i] = mp; group.l[i] = lp; group.r[i] = rp;
#pragma unroll
                for (int j = 0; j < 8; ++j) group.x[i][j] = x[j];
            } else if (i > k) {
                no_part(group, i);
            }
        }
        ++part;
        if (k == GROUP - 1 || part == p.splits) add_parts(group);
        if (part == p.splits) break;
        __syncthreads();            // the merge is done with the wavefronts' results, which lie where the blocks go
        take_part(part);
        t = first + wave;
        if (t < nb) {
            request(t, false);
            request(t, true);
        }
        reset_state();
    }
    {
        if (SHARED && unit < POOL_SOLO) {
            // Leave this part's result; every thread of the merging workgroup reads what the same thread of
            // the others wrote, so the accumulators lie in thread order.
            unsigned char *run = g_pool + (size_t)unit * POOL_UNIT_BYTES;
            uint32_t *header = (uint32_t *)run;
            const int item = tile * p.nrest + rest;
            unsigned char *mine = run + SPLIT_HEADER_BYTES + (size_t)item * p.splits * SPLIT_PART_BYTES;
            const bool valid = qpos < p.Sq;
            {
                unsigned char *out = mine + (size_t)part * SPLIT_PART_BYTES;
                if (valid) {
                    pool_store4(out + ((2 * wave) * 64 + lane) * 16, x[0], x[1], x[2], x[3]);
                    pool_store4(out + ((2 * wave + 1) * 64 + lane) * 16, x[4], x[5], x[6], x[7]);
                }
                if (wave == 0 && hh == 0) {
                    float *st = (float *)(out + 32 * HD * 4);
                    pool_store(st + l32, mp);
                    pool_store(st + 32 + l32, lp);
                    pool_store(st + 64 + l32, rp);
                }
            }
            __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);        // this thread's stores have arrived
            __syncthreads();                // (also: everyone is done with the state area)
            uint32_t *shared = (uint32_t *)(smem + SPLIT_STATE_BASE);
            if (tid == 0)
                shared[0] = __hip_atomic_fetch_add(&header[1 + item], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (shared[0] != (uint32_t)p.splits - 1) return;
            // eight parts at a time, all of their loads in flight together
            constexpr int BATCH = 2;
            for (int s0 = 0; s0 < p.splits; s0 += BATCH * GROUP) {
                Parts g[BATCH];
#pragma unroll
                for (int i = 0; i < BATCH * GROUP; ++i) {
                    const bool there = s0 + i < p.splits;
                    const unsigned char *in = mine + (size_t)(s0 + i) * SPLIT_PART_BYTES;
                    const float *st = (const float *)(in + 32 * HD * 4);
                    Parts &gi = g[i / GROUP];
                    no_part(gi, i % GROUP);
                    if (there) {
                        gi.m[i % GROUP] = pool_load(st + l32);
                        gi.l[i % GROUP] = pool_load(st + 32 + l32);
                        gi.r[i % GROUP] = pool_load(st + 64 + l32);
                    }
                    if (there && valid) {
                        pool_load4(in + ((2 * wave) * 64 + lane) * 16, gi.x[i % GROUP]);
                        pool_load4(in + ((2 * wave + 1) * 64 + lane) * 16, gi.x[i % GROUP] + 4);
                    }
                }
#pragma unroll
                for (int k = 0; k < BATCH; ++k)
                    if (s0 + k * GROUP < p.splits) add_parts(g[k]);
            }
            __syncthreads();                // everything of this item is read
            if (tid == 0) {
                pool_clear(unit, &header[1 + item]);
                if (!sets_counters_back(unit)) {        // (the region is not given back)
                    const uint32_t done = __hip_atomic_fetch_add(&header[0], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (done == (uint32_t)(p.nrest * p.ntile) - 1) pool_give(unit, p.units);
                }
            }
        } else if (!SHARED || unit == POOL_SOLO) {
            M = mp; L = lp; LR = rp;
            // (pinned in front of the branch on qpos: moved behind it, the compiler no longer keeps all LDS reads of the merge in
            // flight, 0.2 .. 0.4 us of 8)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                o8[j] = x[j];
                PIN(o8[j]);
            }
        }
        const float inv = LR > 0.0f ? 1.0f / LR : 0.0f;
        if (qpos < p.Sq) {
            u32x4 ww = {pack_bf16(o8[0] * inv, o8[1] * inv), pack_bf16(o8[2] * inv, o8[3] * inv),
                        pack_bf16(o8[4] * inv, o8[5] * inv), pack_bf16(o8[6] * inv, o8[7] * inv)};
            __bf16 *op = p.o + ((size_t)((size_t)b * p.Sq + qpos) * p.Hq + head) * HD + 16 * wave + 8 * hh;
            *(u32x4 *)op = ww;
            if (wave == 0 && hh == 0)
                p.lse[((size_t)b * p.Hq + head) * p.Sq + qpos] =
                    L > 0.0f ? (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f : -INFINITY;
        }
    }
#ifdef ATTN_CLOCKS
    if (bid == 0 && tid == 0) { g_clocks[1] = __builtin_readcyclecounter(); g_clocks[3] = wall_clock64(); }
#endif
}

// ---------------------------------------------------------------------------------------------------
// The kernel with workgroups of four wavefronts, for everything between the two others: calls of too few 256-row items to fill the
// chip evenly, and short sequences, whose items are mostly prologue and epilogue.  Two workgroups share a compute unit, with a barrier of their own
// each, so that one computes where the other starts, waits or ends; workgroups are handed out by the hardware as others end,
// longest first.  (One workgroup of eight wavefronts per compute unit, in an earlier form of the loop: 24 x 200 30.1 us instead of 22.4, 2 x 1500 56 instead of 45.)
//
// An item is 128 rows (KG = 1: each wavefront has 32 of them and all keys), or 64 (KG = 2: two pairs of wavefronts share the
// rows' keys, every other block of 32 each, and add their results up through LDS at the end).  64 rows make twice as many items, each of half
// as many turns, for twice the K/V traffic from L2 to LDS with half the stages to cover it: 8 x 4096, 16 heads 963 us in items of 128
// rows, 1242 in items of 64 (256-row kernel 890), where counters show 21 and 29 bytes per clock and compute unit, a read from L2 under way for 142 and 489
// clocks, wavefronts waiting 17 and 40 % of their time and the matrix pipe busy for 67 and 45 %; 1 x 1111, 32 heads on 8, causal 21.4 and 17.7 (29.5).
//
// A turn is 16 MFMAs per wavefront, as in the 256-row kernel: O += P(t-1) V(t-1) and S(t+1) = K(t+1) Q^T alternating, with the softmax of S(t)
// between them, one exponent ahead.  By its own clock a wavefront alone on its SIMD takes 890 cycles for one (512 of matrix pipe; 700 without the vector
// instructions), two of them 1500 together; whole launches against 8192 keys, start and memory included, 1090 and 1610 (KG = 1), 1600 and 1950 (KG = 2).  K and V stages: four (KG = 1) or two (KG = 2) of each, 64 KiB, requested that many
// turns before use less one.
struct RowsParams {
    const __bf16 *q, *k, *v;
    __bf16 *o;
    float *lse;
    int Hq, Hkv, Sq, Skv, G;
    int pack, pack_log2;    // as in SplitParams: row r of an item is head r % pack, position r / pack
    int chunks;             // G / pack
    int tile_pos;           // query positions per work item = 128 / KG / pack
    int ntile;              // ceil(Sq / tile_pos)
    int nrest;              // B * Hkv * chunks; items = ntile * nrest
    int window, window0;    // (group, K/V head, batch entry) units that are worked through together; in the first window there may be fewer
    Div d_per_win, d_window, d_window0, d_chunks, d_hkv;      // exact division by window * ntile, window, window0, chunks, Hkv
    int off;                // as in SplitParams
    float c;                // scale * log2(e)
};
constexpr int ROWS_BLOCK_BYTES = SPLIT_KEYS * ROW_BYTES;        // 8 KiB: 32 keys of K or V
constexpr int rows_stages(int KG) { return 4 / KG; }
constexpr int ROWS_LDS_BYTES = 8 * ROWS_BLOCK_BYTES + 3 * 4 * 32 * ROWS_WAVES;
static_assert(2 * ROWS_LDS_BYTES <= LDS_BYTES, "two workgroups fit a CU");

// R row groups of 32 rows, KG key groups; one wavefront for each pair of them.
template <int KG>
__global__ __launch_bounds__(64 * ROWS_WAVES) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_fwd_kernel_rows(const RowsParams p)
{
    constexpr int R = ROWS_WAVES / KG, NS = rows_stages(KG);
    constexpr int STAGE = KG * ROWS_BLOCK_BYTES;        // one block of each key group
    constexpr int VB = NS * STAGE, QB = VB;             // K stages, V stages (at first Q)
    constexpr int STATE = 2 * VB;                       // m, l, lr
    static_assert(R * 32 * ROW_BYTES <= NS * STAGE && STATE == 8 * ROWS_BLOCK_BYTES, "layout of LDS");
    constexpr int LPW = 8 / R;                          // requests of 1 KiB per block and wavefront
    constexpr int QPW = R * 8 / ROWS_WAVES;                 // and of Q
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    LDS_AS unsigned char *lds = (LDS_AS unsigned char *)smem;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;
    const int rg = wave % R, kgrp = wave / R;           // row group, key group
    // blockIdx.x -> (tile, rest): windows of `window` rests, tiles slowest in each, last tile first
    int in_win = blockIdx.x, rest = 0, tile_r;
    if (in_win < p.window0 * p.ntile) {
        tile_r = fast_div(in_win, p.d_window0);
        rest = in_win - tile_r * p.window0;
    } else {
        in_win -= p.window0 * p.ntile;
        const int win = fast_div(in_win, p.d_per_win);
        in_win -= win * (p.window * p.ntile);
        tile_r = fast_div(in_win, p.d_window);
        rest = p.window0 + win * p.window + in_win - tile_r * p.window;
    }
    const int tile = p.ntile - 1 - tile_r;
    const int bh = fast_div(rest, p.d_chunks), chunk = rest - bh * p.chunks;
    const int b = fast_div(bh, p.d_hkv), hkv = bh - b * p.Hkv;
    const int q0 = tile * p.tile_pos;
    const int row = 32 * rg + l32;                      // this lane's query: its row of the item
    // blocks of 32 keys: of the item, of this wavefront's rows, and of those the leading ones without masked keys
    const int klast = min(p.Skv - 1, min(q0 + p.tile_pos - 1, p.Sq - 1) + p.off);
    const int nb = klast < 0 ? 0 : klast / SPLIT_KEYS + 1;
    const int pos_lo = q0 + ((32 * rg) >> p.pack_log2), pos_hi = q0 + ((32 * rg + 31) >> p.pack_log2);
    const int klast_w = min(p.Skv - 1, min(pos_hi, p.Sq - 1) + p.off);
    const int n_w = klast_w < 0 ? 0 : klast_w / SPLIT_KEYS + 1;
    const int kfirst_w = min(p.Skv, pos_lo + p.off + 1);
    const int n_unm = kfirst_w <= 0 ? 0 : kfirst_w / SPLIT_KEYS;
    const int n = (nb + KG - 1) / KG;                   // turns of the loop
    const size_t pitch = (size_t)p.Hkv * HD * 2;
    const unsigned char *kg = uniform_ptr((const unsigned char *)(p.k + ((size_t)b * p.Skv * p.Hkv + hkv) * HD));
    const unsigned char *vg = uniform_ptr((const unsigned char *)(p.v + ((size_t)b * p.Skv * p.Hkv + hkv) * HD));
    const uint32_t lds0 = (uint32_t)(uintptr_t)lds;
    const uint32_t lds_wave = lds0 + kgrp * ROWS_BLOCK_BYTES + rg * (LPW * 1024);

    // ---- requests.  A key group's block is fetched by its R wavefronts.
    uint32_t koff[LPW], voff[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int r = 4 * (LPW * rg + i) + (lane >> 4), unit = lane & 15;
        koff[i] = (uint32_t)(r * pitch) + ((unit ^ (r & 15)) << 4);
        voff[i] = (uint32_t)(r * pitch) + ((unit ^ ((r & 3) << 2)) << 4);
    }
    // Block of turn t into its stage.  (In the last turn a key group may have no block: it reads the item's last one once more.)
    auto request = [&](int t, bool is_v) __attribute__((always_inline)) {
        const int blk = min(t * KG + kgrp, nb - 1);
        const unsigned char *g = uniform_ptr((is_v ? vg : kg) + (size_t)blk * SPLIT_KEYS * pitch);
        const int last = p.Skv - 1 - blk * SPLIT_KEYS;      // rows past the end of K/V re-read the last row
        const uint32_t dst = lds_wave + (is_v ? VB : 0) + (t & (NS - 1)) * STAGE;
        if (last >= SPLIT_KEYS - 1) {
#pragma unroll
            for (int i = 0; i < LPW; ++i) lds_dma16(g, is_v ? voff[i] : koff[i], dst + i * 1024);
        } else {
            int ln = lane;
            PIN(ln);
#pragma unroll
            for (int i = 0; i < LPW; ++i) {
                const int r = 4 * (LPW * rg + i) + (ln >> 4);
                lds_dma16(g, (is_v ? voff[i] : koff[i]) + (uint32_t)((min(r, last) - r) * (int)pitch), dst + i * 1024);
            }
        }
    };
    {
        const int row0 = min(q0, p.Sq - 1);
        const unsigned char *qg = uniform_ptr(
            (const unsigned char *)(p.q + ((size_t)((size_t)b * p.Sq + row0) * p.Hq + hkv * p.G + chunk * p.pack) * HD));
#pragma unroll
        for (int i = 0; i < QPW; ++i) {
            const int r = (wave * QPW + i) * 4 + (lane >> 4), unit = lane & 15;
            const int drow = min(q0 + (r >> p.pack_log2), p.Sq - 1) - row0;         // 0 .. 127
            const uint32_t o = (uint32_t)(drow * p.Hq + (r & (p.pack - 1))) * (uint32_t)(HD * 2) + ((unit ^ (r & 15)) << 4);
            lds_dma16(qg, o, lds0 + QB + (wave * QPW + i) * 1024);
        }
    }
    if (n > 0) {
#pragma unroll
        for (int t = 0; t < NS; ++t)
            if (t < n) request(t, false);
    }
    __builtin_amdgcn_sched_barrier(0);

    f32x16 acc[4], s[2];
    uint32_t pb[2][8];
    float m = -INFINITY, l = 0.0f, lr = 0.0f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[dt][r] = 0.0f;
    int kaddr[8], vaddr[4];
#pragma unroll
    for (int st = 0; st < 8; ++st) kaddr[st] = kgrp * ROWS_BLOCK_BYTES + l32 * ROW_BYTES + (((2 * st + hh) ^ (l32 & 15)) << 4);
    {
        const int i16 = lane & 15, g = (lane >> 4) & 1;
        const int r = 4 * hh + (i16 >> 2);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const int d = 32 * dt + 16 * g + 4 * (i16 & 3);
            vaddr[dt] = VB + kgrp * ROWS_BLOCK_BYTES + r * ROW_BYTES + ((((d >> 3) ^ ((r & 3) << 2))) << 4) + (d & 7) * 2;
        }
    }
    // (opaque from here on, so that the stage and the row stay immediate offsets)
#pragma unroll
    for (int st = 0; st < 8; ++st) PIN(kaddr[st]);
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) PIN(vaddr[dt]);

    auto fetch_k = [&](int st, int at) __attribute__((always_inline)) -> bf16x8 {
        return *(const LDS_AS bf16x8 *)(lds + kaddr[st] + at);
    };
    auto fetch_v = [&](int i, int at) __attribute__((always_inline)) -> bf16x8 {        // 16 keys i / 4, d tile i % 4
        const int ro = at + (i >> 2) * 16 * ROW_BYTES;
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + vaddr[i & 3] + ro));
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4 *)(lds + vaddr[i & 3] + (ro + 8 * ROW_BYTES)));
        s16x8 av = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, av);
    };
    bf16x8 qf[8];           // Q^T operand: query l32, d = 16 s + 8 hh .. + 7
    auto qk = [&](f32x16 &x, int at) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = 0.0f;
#pragma unroll
        for (int st = 0; st < 8; ++st) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fetch_k(st, at), qf[st], x, 0, 0, 0);
    };
    auto pv_mfma = [&](bf16x8 av, const uint32_t (&pp)[8], int i) __attribute__((always_inline)) {
        const int g = i >> 2;
        u32x4 pw = {pp[4 * g], pp[4 * g + 1], pp[4 * g + 2], pp[4 * g + 3]};
        acc[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8, pw), acc[i & 3], 0, 0, 0);
    };
    auto pv = [&](const uint32_t (&pp)[8], int at) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 8; ++i) pv_mfma(fetch_v(i, at), pp, i);
    };
    const float c = fabsf(p.c);
    auto key_room = [&](int blk) __attribute__((always_inline)) -> int {       // key 4 hh + k of the block is valid for this lane's row iff k <= room
        int ln = lane;
        PIN(ln);
        return min(p.Skv - 1, q0 + ((32 * rg + (ln & 31)) >> p.pack_log2) + p.off) - blk * SPLIT_KEYS - 4 * (ln >> 5);
    };
    // Exact online softmax of a block, masked per key.  (The reference is finite once there is a valid key.)  FIRST: against m as it stands.
    auto softmax_exact = [&](auto first, const f32x16 &x, uint32_t (&pn)[8], int blk) __attribute__((always_inline)) {
        constexpr bool FIRST = decltype(first)::value;
        const int room = key_room(blk);
        if (!FIRST) {
            float mx = -INFINITY;
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, 8 * (r >> 2) + (r & 3) <= room ? fmaxf(x[r] * c, -FLT_MAX) : -INFINITY);
            const float mn = fmaxf(m, lane32_max(mx));
            const float alpha = (mn == -INFINITY) ? 1.0f : __builtin_amdgcn_exp2f(m - mn);
            m = mn;
            l *= alpha;
            lr *= alpha;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[dt][r] *= alpha;
        }
        const float mu = (m == -INFINITY) ? 0.0f : m;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const int key = 8 * (r >> 2) + (r & 3);
            float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], c, -mu));
            float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r + 1], c, -mu));
            e0 = (key <= room) ? e0 : 0.0f;
            e1 = (key + 1 <= room) ? e1 : 0.0f;
            l += e0 + e1;
            pn[r >> 1] = pack_bf16(e0, e1);
            lr = add_bf16_pair(pn[r >> 1], lr);
        }
    };
    // Largest scaled score of block blk's valid keys per query, at least -FLT_MAX; minus infinity if none is valid.
    auto largest = [&](const f32x16 &x, int blk) __attribute__((always_inline)) -> float {
        const int room = key_room(blk);
        float mx = -INFINITY;
        if (blk < n_unm) {
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, x[r]);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) mx = fmaxf(mx, 8 * (r >> 2) + (r & 3) <= room ? x[r] : -INFINITY);
        }
        return lane32_max(room >= 0 ? fmaxf(mx * c, -FLT_MAX) : -INFINITY);
    };
    // Turn t: O += P(t-1) V(t-1) from stage vat, S(t+1) = K(t+1) Q^T from stage kat, and between the MFMAs P(t) from S(t) against the
    // running maximum as it stands.  LDS reads run four MFMAs ahead of their consumer, from one turn into the next: before the last four MFMAs,
    // when all of the turn's operands are in registers, come the turn's barrier (mid), which publishes the next turn's
    // stages and frees this turn's, and the first reads from stages vat_next and kat_next.
    constexpr int AHEAD = 4;
    bf16x8 frag[16 + AHEAD];        // [0, AHEAD): read by the turn before
    auto fetch = [&](int slot, int vat, int kat) __attribute__((always_inline)) -> bf16x8 {
        return (slot & 1) ? fetch_k(slot >> 1, kat) : fetch_v(slot >> 1, vat);
    };
    auto turn = [&](auto masked_, auto more_, const f32x16 &x, f32x16 &y, const uint32_t (&pp)[8], uint32_t (&pn)[8],
                    int vat, int kat, int vat_next, int kat_next, int blk, auto mid, auto after) __attribute__((always_inline)) {
        constexpr bool MASKED = decltype(masked_)::value, MORE = decltype(more_)::value;
        float ev[16], ls0 = 0.0f, ls1 = 0.0f, r0 = 0.0f, r1 = 0.0f, arg = 0.0f;
        uint32_t pw[8];
        const int room = MASKED ? key_room(blk) : 0;
#pragma unroll
        for (int slot = 0; slot < 16; ++slot) {
            if (MORE && slot + AHEAD == 16) {
                __builtin_amdgcn_s_waitcnt(WAIT_LGKMCNT0);
                mid();
            }
            if (slot + AHEAD < 16 && (MORE || !(slot & 1))) frag[slot + AHEAD] = fetch(slot + AHEAD, vat, kat);
            else if (MORE) frag[slot + AHEAD] = fetch(slot + AHEAD - 16, vat_next, kat_next);
            if ((slot & 1) == 0) {
                pv_mfma(frag[slot], pp, slot >> 1);
            } else if (MORE) {
                const int st = slot >> 1;
                f32x16 z;
#pragma unroll
                for (int r = 0; r < 16; ++r) z[r] = 0.0f;
                y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[slot], qf[st], st == 0 ? z : y, 0, 0, 0);
            }
            // probability `slot`; its argument was formed a slot before, its sum and its pair's rounding follow a slot later, so that
            // no instruction waits for the one in front of it
            ev[slot] = __builtin_amdgcn_exp2f(slot == 0 ? __builtin_fmaf(x[0], c, -m) : arg);
            if (MASKED) ev[slot] = 8 * (slot >> 2) + (slot & 3) <= room ? ev[slot] : 0.0f;
            if (slot < 15) {
                arg = __builtin_fmaf(x[slot + 1], c, -m);
                PIN(arg);
            }
            if (slot & 1) {
                ls0 += ev[slot - 1];
                PIN(ls0);
            } else if (slot > 0) {
                ls1 += ev[slot - 1];
                PIN(ls1);
                pw[(slot >> 1) - 1] = pack_bf16(ev[slot - 2], ev[slot - 1]);
                PIN(pw[(slot >> 1) - 1]);
            }
            if (MORE && slot + AHEAD >= 16) after(slot + AHEAD - 16);
            __builtin_amdgcn_sched_barrier(0);
        }
        ls1 += ev[15];
        pw[7] = pack_bf16(ev[14], ev[15]);
        if (MORE) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) frag[i] = frag[16 + i];
        }
#pragma unroll
        for (int k = 0; k < 8; k += 2) {
            r0 = add_bf16_pair(pw[k], r0);
            r1 = add_bf16_pair(pw[k + 1], r1);
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) pn[k] = pw[k];
        float ls = ls0 + ls1, lrn = r0 + r1;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(ls <= P_SUM_LIMIT)) != 0, 0)) {
            softmax_exact(std::false_type{}, x, pn, blk);
            ls = lrn = 0.0f;        // (it has added them)
        }
        l += ls;
        lr += lrn;
    };

    // (waits: everything, where the item is too short for the counts of the steady state)
    if (n >= NS) __builtin_amdgcn_s_waitcnt(wait_vmcnt((NS - 1) * LPW)); else __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    wg_barrier();           // Q and K(0) have landed
#pragma unroll
    for (int st = 0; st < 8; ++st) qf[st] = *(const LDS_AS bf16x8 *)(lds + QB + row * ROW_BYTES + (((2 * st + hh) ^ (l32 & 15)) << 4));
    // a negative scale: the negated Q (exact) with the scale's absolute value
    if (p.c < 0.0f) {
#pragma unroll
        for (int st = 0; st < 8; ++st) qf[st] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, qf[st]) ^ 0x80008000u);
    }
    if (n > 0) {
        qk(s[0], 0);
        if (n >= NS) __builtin_amdgcn_s_waitcnt(wait_vmcnt((NS - 2) * LPW)); else __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
        wg_barrier();                                           // K(1) has landed, and everyone has read K(0) and Q
#pragma unroll
        for (int t = 0; t < NS - 1; ++t)
            if (t < n) request(t, true);
        if (NS < n) request(NS, false);
        // Turn t requests K(t+1+NS) and V(t-1+NS) behind its barrier, into the stages that it has read; at the barrier what the next turn
        // reads has landed, K(t+2) and V(t), requested NS - 1 turns before.
        constexpr int IN_FLIGHT = (NS - 2) * 2 * LPW;
        m = largest(s[0], kgrp);
        if (n > 1) {
            // (the reference of the first turns is the largest of two blocks, 64 keys, as in the 256-row kernel: one block alone leaves
            // larger weights to rounding)
            qk(s[1], STAGE);
            m = fmaxf(m, largest(s[1], KG + kgrp));
        }
        softmax_exact(std::true_type{}, s[0], pb[0], kgrp);
        if (n > 1) {
            if (n > NS) __builtin_amdgcn_s_waitcnt(wait_vmcnt((NS - 1) / 2 * 3 * LPW)); else __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
            wg_barrier();                                       // K(2), V(0) have landed, and everyone has read K(1)
            if (1 + NS < n) request(1 + NS, false);
            if (NS - 1 < n) request(NS - 1, true);
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) frag[i] = fetch(i, 0, 2 % NS * STAGE);
        }
        const std::true_type yes = {};
        const std::false_type no = {};
        int t = 1;
        // turns below it see no masked key of this wavefront, and request full blocks
        const int fast_end = min(n - 1, (min(n_unm, min(nb, p.Skv / SPLIT_KEYS) - (NS + 1) * KG) - kgrp + KG - 1) / KG);
        const size_t step = (size_t)KG * SPLIT_KEYS * pitch;
        const unsigned char *kp = uniform_ptr(kg + (size_t)((NS + 2) * KG + kgrp) * SPLIT_KEYS * pitch);
        const unsigned char *vp = uniform_ptr(vg + (size_t)(NS * KG + kgrp) * SPLIT_KEYS * pitch);
        auto wait = [&]() __attribute__((always_inline)) {
            if (t + NS < n) __builtin_amdgcn_s_waitcnt(wait_vmcnt(IN_FLIGHT)); else __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
            wg_barrier();
        };
        auto more_requests = [&]() __attribute__((always_inline)) {
            if (t + 1 + NS < n) request(t + 1 + NS, false);
            if (t - 1 + NS < n) request(t - 1 + NS, true);
        };
        auto fast = [&](auto phase) __attribute__((always_inline)) {
            constexpr int T = decltype(phase)::value % NS;      // t % NS
            constexpr int VA = (T + NS - 1) % NS * STAGE, KA = (T + 1) % NS * STAGE, VN = T * STAGE, KN = (T + 2) % NS * STAGE;
            turn(no, yes, s[T & 1], s[1 - (T & 1)], pb[1 - (T & 1)], pb[T & 1], VA, KA, VN, KN, t * KG + kgrp,
                 [&]() __attribute__((always_inline)) {
                     __builtin_amdgcn_s_waitcnt(wait_vmcnt(IN_FLIGHT));
                     wg_barrier();
                 },
                 [&](int i) __attribute__((always_inline)) {
                     // (one of four: the first and the second half of K's requests, then of V's)
                     constexpr int H = LPW / 2;
                     if (i == 0) lds_dma16_imm<KA>(kp, koff[0], lds_wave);
                     if (i == 0 && H == 2) lds_dma16_imm<KA + 1024>(kp, koff[1], lds_wave);
                     if (i == 1) lds_dma16_imm<KA + H * 1024>(kp, koff[H], lds_wave);
                     if (i == 1 && H == 2) lds_dma16_imm<KA + 3072>(kp, koff[LPW - 1], lds_wave);
                     if (i == 2) lds_dma16_imm<VB + VA>(vp, voff[0], lds_wave);
                     if (i == 2 && H == 2) lds_dma16_imm<VB + VA + 1024>(vp, voff[1], lds_wave);
                     if (i == 3) lds_dma16_imm<VB + VA + H * 1024>(vp, voff[H], lds_wave);
                     if (i == 3 && H == 2) lds_dma16_imm<VB + VA + 3072>(vp, voff[LPW - 1], lds_wave);
                 });
            kp += step;
            vp += step;
            ++t;
        };
#pragma nounroll
        for (; t + NS - 1 < fast_end;) {
            fast(std::integral_constant<int, 1>{});
            fast(std::integral_constant<int, 2>{});
            if (NS == 4) {
                fast(std::integral_constant<int, 3>{});
                fast(std::integral_constant<int, 4>{});
            }
        }
        // The rest, masked, one after the other: s[1] holds S(t), pb[0] P(t-1).
#pragma nounroll
        for (; t < n - 1; ++t) {
            turn(yes, yes, s[1], s[0], pb[0], pb[0], (t - 1) % NS * STAGE, (t + 1) % NS * STAGE, t % NS * STAGE, (t + 2) % NS * STAGE,
                 t * KG + kgrp, wait, [](int) {});
            more_requests();
            s[1] = s[0];
        }
        // the last turn: no further scores
        if (n > 1 && (n - 2) * KG + kgrp < n_w) {
#pragma unroll
            for (int i = 0; i < AHEAD; i += 2) frag[i] = fetch(i, (n - 2) % NS * STAGE, 0);
            turn(yes, no, s[1], s[0], pb[0], pb[0], (n - 2) % NS * STAGE, 0, 0, 0, (n - 1) * KG + kgrp, []() {}, [](int) {});
        }
        __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);        // V(n-1) has landed
        wg_barrier();
        if ((n - 1) * KG + kgrp < n_w) pv(pb[0], (n - 1) % NS * STAGE);
    }
    __builtin_amdgcn_s_waitcnt(WAIT_VMCNT0);
    if (KG > 1) wg_barrier();       // the stages are read

    // ---- merge of the key groups: wavefront (rg, kgrp) finishes d tiles DT kgrp .. DT kgrp + DT - 1 of its rows
    constexpr int DT = 4 / KG;
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    auto part = [&](int to, int from) __attribute__((always_inline)) {
        return (LDS_AS f32x4 *)(lds + ((rg * KG + to) * KG + from) * (DT * 4096)) + lane;
    };
    LDS_AS float *state = (LDS_AS float *)(lds + STATE) + rg * KG * 96;
    if (KG > 1) {
        const float lt = lane32_sum(l), lrt = lane32_sum(lr);
        if (hh == 0) {
            state[kgrp * 96 + l32] = m;
            state[kgrp * 96 + 32 + l32] = lt;
            state[kgrp * 96 + 64 + l32] = lrt;
        }
    }
    const int head = hkv * p.G + chunk * p.pack + (row & (p.pack - 1));
    const int qpos = q0 + (row >> p.pack_log2);
    const bool valid = qpos < p.Sq;
    float M = -INFINITY, L = 0.0f;
    auto finish = [&](auto mine) __attribute__((always_inline)) {
        constexpr int ME = decltype(mine)::value;
#pragma unroll
        for (int to = 0; to < KG; ++to) {
            if (to == ME) continue;
#pragma unroll
            for (int i = 0; i < 4 * DT; ++i) {
                const f32x16 &a = acc[to * DT + (i >> 2)];
                part(to, ME)[64 * i] = f32x4{a[4 * (i & 3)], a[4 * (i & 3) + 1], a[4 * (i & 3) + 2], a[4 * (i & 3) + 3]};
            }
        }
        float f[KG], LR = 0.0f;
        if (KG == 1) {
            f[0] = 1.0f;
            M = m;
            L = lane32_sum(l);
            LR = lane32_sum(lr);
        } else {
            __syncthreads();
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                f[g] = state[g * 96 + l32];
                M = fmaxf(M, f[g]);
            }
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                f[g] = (f[g] == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f(f[g] - M);
                L += f[g] * state[g * 96 + 32 + l32];
                LR += f[g] * state[g * 96 + 64 + l32];
            }
        }
        const float inv = LR > 0.0f ? 1.0f / LR : 0.0f;
        unsigned char *op = (unsigned char *)(p.o + ((size_t)((size_t)b * p.Sq + qpos) * p.Hq + head) * HD + 32 * DT * ME + 8 * hh);
#pragma unroll
        for (int i = 0; i < 2 * DT; ++i) {      // 16 d: this lane's two pieces of four, then with its partner's one of eight
            float y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) y[j] = 0.0f;
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                const f32x16 &a = acc[ME * DT + (i >> 1)];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const int e = 8 * (i & 1) + 4 * k;
                    f32x4 z = {a[e], a[e + 1], a[e + 2], a[e + 3]};
                    if (g != ME) z = part(ME, g)[64 * (2 * i + k)];
#pragma unroll
                    for (int j = 0; j < 4; ++j) y[4 * k + j] = KG == 1 ? z[j] : y[4 * k + j] + f[g] * z[j];
                }
            }
            auto u = __builtin_amdgcn_permlane32_swap(pack_bf16(y[0] * inv, y[1] * inv), pack_bf16(y[4] * inv, y[5] * inv), false, false);
            auto w = __builtin_amdgcn_permlane32_swap(pack_bf16(y[2] * inv, y[3] * inv), pack_bf16(y[6] * inv, y[7] * inv), false, false);
            const u32x4 ww = {u[0], w[0], u[1], w[1]};
            if (valid) *(u32x4 *)(op + 32 * i) = ww;
        }
    };
    if (KG == 1 || kgrp == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, KG - 1>{});
    if (valid && kgrp == 0 && hh == 0)
        p.lse[((size_t)b * p.Hq + head) * p.Sq + qpos] = L > 0.0f ? (M + __builtin_amdgcn_logf(L)) * 0.6931471805599453f : -INFINITY;
}

}  // namespace

extern "C" {

int attn_fwd(const void *q, const void *k, const void *v, void *o, float *lse,
             int B, int Hq, int Hkv, int Sq, int Skv, int D,
             int causal, float scale, void *stream)
{
    if (!q || !k || !v || !o || !lse) return ATTN_E_NULL;
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || Sq <= 0 || Skv <= 0 || D <= 0) return ATTN_E_SHAPE;
    if (Hq % Hkv != 0) return ATTN_E_SHAPE;
    if (D != HD) return ATTN_E_UNSUPPORTED;
    if (!isfinite(scale)) return ATTN_E_SCALE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return ATTN_E_ALIGN;
    if ((uintptr_t)lse & 3) return ATTN_E_ALIGN;

    Route r = {};
    const int rc = make_shape(B, Hq, Hkv, Sq, Skv, r.shape, r.sched);
    if (rc != ATTN_OK) return rc;

    // Once per device: the CU count, and the opt-in that 160 KiB of dynamic LDS needs.
    static std::atomic<int> cus[64];          // zero-initialised; threads that race here store the same value
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return ATTN_E_LAUNCH;
    if (!cus[dev].load(std::memory_order_acquire)) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0 ||
            hipFuncSetAttribute((const void *)attn_fwd_kernel<true, false>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_kernel<true, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_kernel<false, false>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_kernel<false, true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_kernel_rows<1>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, ROWS_LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_kernel_rows<2>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, ROWS_LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_split_kernel<true>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, SPLIT_LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute((const void *)attn_fwd_split_kernel<false>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, SPLIT_LDS_BYTES) != hipSuccess)
            return ATTN_E_LAUNCH;
        cus[dev].store(n, std::memory_order_release);
    }
    const int ncu = cus[dev].load(std::memory_order_relaxed);
    make_route(B, Hkv, Skv, causal, ncu, r);
    const Shape &sh = r.shape;
    hipStream_t st = (hipStream_t)stream;

    Params p = {};
    p.q = (const __bf16 *)q; p.k = (const __bf16 *)k; p.v = (const __bf16 *)v;
    p.o = (__bf16 *)o; p.lse = lse;
    p.Hkv = Hkv; p.Skv = Skv;
    p.c = scale * 1.4426950408889634f;
    p.shape = sh; p.sched = r.sched; p.share = r.share;

    const bool region = ATTN_POOL && shares_items(r) && st == nullptr;
    p.unit = region ? REGION_SHARE_UNIT : POOL_NONE;

    SplitParams sp = {};
    sp.lse = lse;
    sp.unit = region ? REGION_SPLIT_UNIT : shares_items(r) ? POOL_NONE : POOL_SOLO;
    sp.Hq = Hq; sp.Hkv = Hkv; sp.Sq = Sq; sp.G = sh.G;
    sp.pack = sh.pack; sp.chunks = sh.chunks;
    sp.d_chunks = sh.d_chunks;
    sp.d_hkv = sh.d_hkv;
    if (r.kind == ROUTE_SPLIT) {
        sp.q = p.q; sp.k = p.k; sp.v = p.v; sp.o = p.o;
        sp.Skv = Skv;
        sp.pack_log2 = sh.pack_log2;
        sp.tile_pos = r.split.tile_pos; sp.ntile = r.split.ntile; sp.nrest = r.split.nrest;
        sp.splits = r.split.splits; sp.units = r.split.units;
        sp.d_nrs = make_div((uint32_t)(sp.nrest * sp.splits));
        sp.d_splits = make_div((uint32_t)sp.splits);
        // (i + INT32_MAX - Sq - 64 is above every key for i >= 0 and within 32 bits for the i < Sq + 32 of a tile)
        sp.off = causal ? Skv - Sq : INT32_MAX - Sq - 64;
        sp.c = p.c;
        sp.once = r.split.once || (region && r.split.once_region);
    } else {
        sp.tile_pos = sh.tile_pos;
        sp.ntile = r.sched.ntile;
        sp.nrest = r.share.groups;
        sp.units = r.share.units;
    }
    RowsParams rp = {};
    if (r.rows.kgroups != 0) {
        const Rows &rw = r.rows;
        rp.q = p.q; rp.k = p.k; rp.v = p.v; rp.o = p.o; rp.lse = lse;
        rp.Hq = Hq; rp.Hkv = Hkv; rp.Sq = Sq; rp.Skv = Skv; rp.G = sh.G;
        rp.pack = sh.pack; rp.pack_log2 = sh.pack_log2; rp.chunks = sh.chunks;
        rp.tile_pos = rw.tile_pos; rp.ntile = rw.ntile; rp.nrest = rw.nrest;
        rp.window = rw.window; rp.window0 = rw.window0;
        rp.d_per_win = make_div((uint32_t)(rw.window * rw.ntile));
        rp.d_window = make_div((uint32_t)rw.window);
        rp.d_window0 = make_div((uint32_t)rw.window0);
        rp.d_chunks = sh.d_chunks; rp.d_hkv = sh.d_hkv;
        // (i + INT32_MAX - Sq - 128 is above every key for i >= 0 and within 32 bits for the i < Sq + 128 of a tile)
        rp.off = causal ? Skv - Sq : INT32_MAX - Sq - 128;
        rp.c = p.c;
    }
    // Each launch is judged by its own status: the runtime's record of the thread's last error may hold an earlier
    // call's.  (One that fails is taken out of that record, as its report is the return value.)
    auto launch = [&](const void *kernel, unsigned wgs, int lds, void *params, int threads = NTHREADS) -> bool {
        if (hipLaunchKernel(kernel, dim3(wgs), dim3(threads), &params, lds, st) == hipSuccess) return true;
        (void)hipGetLastError();
        return false;
    };
    return enqueue(r, [&](Step step) -> bool {
        if (step != STEP_MAIN) {
            sp.reserve = step == STEP_GIVE ? -1 : r.kind == ROUTE_SHARED ? NWAVES : 1;
            return launch((const void *)attn_fwd_split_kernel<true>, 1, 1024, &sp);
        }
        sp.reserve = 0;
        if (r.kind == ROUTE_SPLIT)
            return launch(sp.splits > 1 || sp.once ? (const void *)attn_fwd_split_kernel<true> : (const void *)attn_fwd_split_kernel<false>,
                          (unsigned)sp.nrest * sp.ntile * sp.splits, SPLIT_LDS_BYTES, &sp);
        if (r.kind == ROUTE_SHARED)
            return launch(causal ? (const void *)attn_fwd_kernel<true, true> : (const void *)attn_fwd_kernel<false, true>,
                          r.share.wgs, LDS_BYTES, &p);
        if (r.rows.kgroups != 0)
            return launch(r.rows.kgroups == 1 ? (const void *)attn_fwd_kernel_rows<1> : (const void *)attn_fwd_kernel_rows<2>,
                          (unsigned)rp.nrest * rp.ntile, ROWS_LDS_BYTES, &rp, 64 * ROWS_WAVES);
        const void *whole = causal ? (const void *)attn_fwd_kernel<true, false> : (const void *)attn_fwd_kernel<false, false>;
        return launch(whole, (unsigned)(r.sched.slots * 8), LDS_BYTES, &p);
    }, region);
}

const char *attn_strerror(int code)
{
    switch (code) {
    case ATTN_OK:            return "success";
    case ATTN_E_NULL:        return "null pointer argument";
    case ATTN_E_SHAPE:       return "bad shape: every dimension must be positive and Hq a multiple of Hkv";
    case ATTN_E_UNSUPPORTED: return "unsupported: head dimension must be 128 and sizes must fit 32-bit indices";
    case ATTN_E_ALIGN:       return "misaligned pointer: q, k, v, o need 16-byte and lse 4-byte alignment";
    case ATTN_E_SCALE:       return "scale must be finite";
    case ATTN_E_LAUNCH:      return "kernel launch failed";
    default:                 return "unknown attn error code";
    }
}

int attn_version(void) { return 1001; }

#ifdef ATTN_CLOCKS
// Waits for the device, then copies the stamps of the last launch to the host (10 x 64-bit).
int attn_clocks_read(unsigned long long *out)
{
    if (!out) return ATTN_E_NULL;
    return hipMemcpyFromSymbol(out, HIP_SYMBOL(g_clocks), sizeof(g_clocks)) == hipSuccess ? ATTN_OK : ATTN_E_LAUNCH;
}
#if ATTN_CLOCKS >= 2
// Waits for the device, then copies the phase sums of the last launch to the host (2 x 12 x 64-bit).
int attn_phases_read(unsigned long long *out)
{
    if (!out) return ATTN_E_NULL;
    return hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phases), sizeof(g_phases)) == hipSuccess ? ATTN_OK : ATTN_E_LAUNCH;
}
#endif
#endif

}  // extern "C"
