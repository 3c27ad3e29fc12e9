// Batched plan-search dynamic program for gfx950 (MI355X): kernels + C ABI.
//
// Paper section 3.3 ("Dynamic Programming Search", Eq. 1): for every layer l,
// budget column e and strategy s,
//     C[l][e][s] = c(l,s) + min_{s'} ( C[l-1][e - m(l,s)][s'] + R(s', s) ).
//
// How the recurrence is laid out here
// -----------------------------------
// The inner minimum does not depend on the memory shift, so each layer is a
// min-plus product of the (E+1) x S table with the S x S transition matrix:
//     U_l[e'][s] = c(l,s) + min_{s'} ( C[l-1][e'][s'] + R_l(s', s) )
//     C[l][e][s] = U_l[e - m(l,s)][s]                (infinity when e < m(l,s))
// The tables are stored UN-shifted (U_l, and the argmin beside it), strategy
// major and budget minor, so a wavefront covers 64 consecutive budget columns of
// one strategy: m(l,s), c(l,s) and R(s',s) are wave-uniform scalars, every
// global access is a contiguous row segment, and the shift is applied when layer
// l+1 reads column s' at offset -m(l,s').  Each lane keeps the running minima of
// its budget columns for a group of strategies in registers, so the minimum over
// s' is a serial in-lane loop: no cross-lane reduction, and the lowest-index
// tie-break falls out of the key order.
//
// Exact arithmetic paths, chosen per instance on the device
// ---------------------------------------------------------
//  * 32-bit keys (small costs and transition costs: the common case): costs are taken
//    relative to the column's smallest former cost and clamped at R_max + 1, so that
//    key = (relative cost + R) * 2^k + s' fits 32 bits; two candidates cost two
//    v_add_u32 and one v_min3_u32.  A clamped former strategy can neither win nor tie, which
//    is also what lets the sweep PRUNE: a former-layer row that is clamped in every column of
//    a tile is left out of the inner loop, and (rows being non-increasing along the budget
//    axis) two of its cells tell whether it needs to be fetched at all.  With the usual spread
//    of layer costs some 90-95 % of the candidates fall away and the sweep is bound by the chain of memory
//    round trips of a tile.
//    The keys' width depends on the transition costs only; when the costs themselves outgrow
//    32-bit cells, the same body runs over 64-bit cells (up to 256 strategies).
//    Where a layer has many tiles, these instances keep argmins of one byte and what it takes to
//    rebuild the few cells the next layer reads, instead of cost rows (see the byte-table sweep);
//    so do the instances on 64-bit keys whose transition costs fit 32 bits.
//  * 64-bit keys: key = cost * 2^k + s' (k = ceil(log2 S)) lives in the mantissa of a double
//    whose exponent is pinned, K = 2^52 + key; one v_add_f64 + one v_min_f64 per candidate,
//    exact while K stays below 2^53.  Two storage widths: narrow (costs below 2^31 stored as
//    uint32, infinity = 2^31) and wide (the key itself stored as a double, infinity = +inf).
//  * int64: plain 64-bit integer add / compare / select with a separate index, for
//    instances whose value range does not fit a 52-bit key.
// In every packed form the minimum of keys is the minimum cost with the lowest s' among
// equals.  A preparation kernel bounds each instance's largest possible plan cost and picks
// the path; all paths produce bit-identical results.
//
// All kernels are plain VALU + LDS + global memory; there is no matrix-core work in a
// min-plus recurrence.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "../../include/galv_dp.h"

// Workspace of galv_dp_solve_static, the entry point that allocates nothing: it lives in the
// code object, one copy per GPU for as long as the process runs.  Host code never uses this
// name as an address; it asks the runtime for the device address once per device (see
// static_scratch()).
static __device__ __align__(256) unsigned char scratch[GALV_DP_STATIC_BYTES];

namespace {

constexpr int kThreads = 256;          // workgroup = 4 wavefronts of 64
constexpr int kPrepThreads = 1024;     // prep_kernel: one workgroup per instance, whose loops are chains of
                                       // load round trips: 16 wavefronts shorten each chain
constexpr int kWave = 64;
constexpr int kEAlign = 1024;          // budget columns are padded to this
constexpr int kMaxS = 1024;
constexpr int kSample = 64;            // byte-table sweep: absolute costs are kept of every 64th budget column
constexpr int kMaxSide = 16;          // internal streams per handle
constexpr int kMaxPp = 16;            // pipeline degrees per reduce call
constexpr int kWordStep = 16;         // chained sweep: 32-bit words from one flag to the next
constexpr int32_t kUnset = INT32_MIN; // chained sweep: the last column of a layer is not told yet
#ifndef GALV_P1_BATCH
#define GALV_P1_BATCH 8
#endif
#ifndef GALV_DEPTH
#define GALV_DEPTH 2
#endif
#ifndef GALV_XCD_MAP
#define GALV_XCD_MAP 1
#endif
constexpr int kDepth = GALV_DEPTH;      // previous-layer loads kept in flight per wave
constexpr int64_t kInf = GALV_INF;
constexpr uint32_t kInf32 = 0x80000000u;             // infinity of the narrow storage
constexpr uint64_t kBias = 0x4330000000000000ull;    // bit pattern of 2^52

thread_local char g_err[512] = "";

galv_status_t fail(galv_status_t code, const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr)                                                                  \
    do {                                                                               \
        hipError_t e_ = (expr);                                                        \
        if (e_ != hipSuccess)                                                          \
            return fail(GALV_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));  \
    } while (0)

inline size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Geometry of one sweep-kernel variant: TS strategies x TE budget columns of
// running minima per lane, NG strategy groups per workgroup.
struct Variant {
    int ts, te, ng, w, ux; // w: wavefronts per workgroup (w / ng budget sub-tiles); ux: see sweep_kernel
    int wpe;               // waves per SIMD the kernel is built for
    int share;             // 1: the row-sharing 32-bit-key body (one tile per workgroup, LDS for the kept rows)
};

enum : int32_t { kAllBytes = 1, kRowsIfAlive = 2, kChain = 3 };      // Layout::packed

// Everything the kernels need to find their data.  Passed by value.  (One more 4-byte field shifts the pointers behind
// it and costs every sweep launch 0.2 us.)
struct Layout {
    int32_t B, L, S, E_max, nR;
    int32_t S_pad;        // strategies rounded up to the variant's group size
    int32_t k_bits;       // index bits in a packed key
    int32_t tile_e;       // budget columns per workgroup
    int32_t n_tiles;      // workgroups along the budget axis
    int64_t lead;         // infinity columns in front of every cost row (fast paths)
    int64_t row;          // cells per cost row: lead + padded columns (8 bytes reserved each)
    int64_t e_pad;        // padded budget columns (multiple of kEAlign)
    char *U[2];           // rolling cost rows   [B][S_pad][row] of 8-byte slots
    void *bp;             // argmin, un-shifted  [B][L-1][S][e_pad] of int32, or of uint8 (0xFF = none)
    int32_t bp_u8;        // 1: one-byte back-pointers
    int32_t peek;         // 1: the row-sharing sweep looks at two cells of a row before it fetches the row
    int32_t packed;       // not 0: instances of byte_status() keep the byte table: argmins in one byte, and
                          //    instead of cost rows what it takes to rebuild a cell (see PackTables); kAllBytes,
                          //    or kRowsIfAlive: those on 64-bit keys not where most rows stay alive (see prep_kernel).
                          //    kChain: one launch for all layers (see the chained sweep): argmins in one byte, whole
                          //    cost rows of every layer at U[0], the workgroups' words at U[1]
    int32_t synth_l1;     // 1: the 32-bit-key sweep makes up layer 0's cells (a constant per strategy)
                          //    when it sweeps layer 1, so layer 0's row is never written nor read
    int32_t b_off, b_step; // a sweep launch covers instances b_off + z * b_step (dealt over streams)
    double *Rk;           // R * 2^k + s'        [B][nR][S][S_pad] (+inf in padded columns)
    uint64_t *ck;         // per-mode c(l,s)     [B][L][S_pad]
    uint64_t *vlist;      // usable strategies of each layer, ascending: shift << 32 | s'; the last one repeats
                          // up to the row's end  [B][L][S_pad]
    uint64_t *vcost;      // c(l, s') of the listed strategies, in the list's order (padded the same way)  [B][L][S_pad]
    int32_t *nvalid;      // how many of them    [B][L]
    uint32_t *dclamp;     // largest R + 1, the clamp of relative costs; 0 when it does not fit (or see byte_status)  [B]
    int32_t *hdr;         // what a sweep workgroup needs first, in one place: status, budget, usable strategies of
                          // the former layer, clamp, transition matrix of the layer, first reachable column,
                          // last column worth sweeping (byte table), smallest usable memory  [B][L][8]
    int32_t *status;      // per instance        [B]
    int32_t *last;        // best last strategy  [B]
    int32_t *lead_mode;   // whose infinity leads the rows hold (lead_kind), 0 none  [B]
    uint32_t *stats;      // 32-bit-key sweeps, per tile: rows reduced << 16 | rows listed; rows fetched  [B][L-1][n_tiles][2]
    int32_t *seen;        // pinned host word (or null): the budget tiles of all instances, as the last solve found them
    const int64_t *c;
    const int32_t *m;
    const int64_t *R;
    const int32_t *r_idx; // may be null
    const int32_t *budget;
};

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
// Position of the thread, without the thread-index register: the kernel reads that register
// once, at its top (wave number, a scalar), and the lane number is recomputed where it is
// needed, so no vector register stays occupied from the kernel's entry to the body it selects.
__device__ __forceinline__ int lane_id() { return (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }
// Lane `lane`'s value of v, as a wave-uniform scalar.
__device__ __forceinline__ uint32_t read_lane(uint32_t v, int lane) {
    return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}
__device__ __forceinline__ uint64_t read_lane(uint64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return (uint64_t)hi << 32 | lo;
}

// Read-only view through the constant address space: data that no thread writes
// while the kernel runs (inputs, tables packed by the preparation kernel).  With a
// wave-uniform address such loads go through the scalar cache into SGPRs.
template <class T>
using ConstPtr = const T __attribute__((address_space(4))) *;
template <class T>
__device__ __forceinline__ ConstPtr<T> as_const(const T *p) {
    return (ConstPtr<T>)(uintptr_t)p;
}

// Storage of the cost rows: 32-bit cells for both packed-key paths of small costs.
__device__ __forceinline__ bool narrow_cells(int st) {
    return st == GALV_INSTANCE_OK_FAST || st == GALV_INSTANCE_OK_FAST_U32;
}
// What the infinity lead in front of a cost row must hold: 1 uint32 2^31, 2 double +inf,
// 3 uint64 2^62, 0 no lead is read.
__device__ __forceinline__ int lead_kind(int st) {
    if (narrow_cells(st)) return 1;
    if (st == GALV_INSTANCE_OK_FAST_WIDE) return 2;
    if (st == GALV_INSTANCE_OK_U32_WIDE) return 3;
    return 0;
}

// Whether an instance of status st keeps the byte table (a handle-wide choice of kernels; one
// layer has no table at all).  That takes packed keys, and relative costs of 32 bits: clamp is
// R_max + 1, or 0 when that does not fit or does not pay.
__device__ __forceinline__ bool byte_status(int st, uint32_t clamp) {
    return st == GALV_INSTANCE_OK_FAST_U32 || st == GALV_INSTANCE_OK_U32_WIDE ||
           ((st == GALV_INSTANCE_OK_FAST || st == GALV_INSTANCE_OK_FAST_WIDE) && clamp != 0);
}
// The same in a handle that runs all layers in one launch: relative costs may have 64 bits there (KeyBig).
__device__ __forceinline__ bool byte_status(const Layout &a, int st, uint32_t clamp) {
    return a.packed == kChain ? st >= 0 && st != GALV_INSTANCE_OK_INT64 : byte_status(st, clamp);
}
__device__ __forceinline__ bool is_packed(const Layout &a, int st, int b) {
    return a.packed && a.L > 1 && byte_status(a, st, a.dclamp[b]);
}

// First row of layer l (>= 1) in the byte table.  An instance's bytes start where its 32-bit back-pointers
// would: the same batch may hold instances that keep those.
__device__ __forceinline__ uint8_t *byte_rows(const Layout &a, int b, int l) {
    return static_cast<uint8_t *>(a.bp) + ((int64_t)b * 4 * (a.L - 1) + (l - 1)) * a.S * a.e_pad;
}

// Back-pointer of un-shifted cell (layer l >= 1, strategy s, column x), whichever width the handle
// stores.  The byte table holds the columns [first, last] of the layer's header record: below is
// unreachable, above is constant.
__device__ __forceinline__ int32_t load_bp(const Layout &a, bool packed, int b, int l, int64_t s, int64_t x) {
    const int64_t row = (((int64_t)b * (a.L - 1) + (l - 1)) * a.S + s) * a.e_pad;
    if (packed) {
        const int32_t *h = a.hdr + ((int64_t)b * a.L + l) * 8;
        if (x < h[5]) return -1;
        return byte_rows(a, b, l)[s * a.e_pad + (x < h[6] ? x : h[6])];
    }
    if (a.bp_u8) {
        const uint8_t v = static_cast<const uint8_t *>(a.bp)[row + x];
        return v == 0xFF ? -1 : (int32_t)v;
    }
    return static_cast<const int32_t *>(a.bp)[row + x];
}
__device__ __forceinline__ void store_bp(const Layout &a, int64_t idx, int32_t v) {
    if (a.bp_u8)
        static_cast<uint8_t *>(a.bp)[idx] = (uint8_t)v;      // -1 becomes 0xFF
    else
        static_cast<int32_t *>(a.bp)[idx] = v;
}

// ------------------------------------------------------------- storage policies
//
// How a cost is kept in the rolling rows, and how it becomes the biased key
// K = 2^52 + cost * 2^k that the arithmetic works on (and back).
struct Narrow {
    using Cell = uint32_t;
    static __device__ __forceinline__ double dead_key(int k) {
        return __longlong_as_double((long long)(kBias | ((uint64_t)kInf32 << k)));
    }
    // K = 2^52 + x * 2^k, built from two 32-bit operations (1 <= k <= 10): the low word is
    // x << k; the high word is one funnel shift of {bias >> k, x} by 32 - k, which puts
    // the bias back in place above the top k bits of x.
    static __device__ __forceinline__ double to_key(Cell x, int k) {
        const uint32_t lo = x << k;
        const uint32_t hi = __builtin_amdgcn_alignbit((uint32_t)(kBias >> 32) >> k, x, 32 - k);
        return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
    }
    // From the reduced key: new cell = cost + c(l,s), argmin index (-1 if unreachable).
    static __device__ __forceinline__ void finish(double key, uint64_t cs, int k, uint32_t mask,
                                                  Cell &cell, int32_t &arg) {
        const uint64_t bits = (uint64_t)__double_as_longlong(key);
        const uint32_t cost = (uint32_t)(bits >> k);          // >= 2^31 exactly when unreachable
        const uint32_t sum = cost + (uint32_t)cs;             // < 2^32 by the range check
        cell = sum < kInf32 ? sum : kInf32;
        arg = (int32_t)((uint32_t)bits & mask) | ((int32_t)cost >> 31);
    }
    static __device__ __forceinline__ Cell first_layer(uint64_t cs) { return (Cell)cs; }
    static __device__ __forceinline__ Cell infinity() { return kInf32; }
    static __device__ __forceinline__ int64_t to_int64(Cell x, int) {
        return x >= kInf32 ? kInf : (int64_t)x;
    }
};

struct Wide {
    using Cell = double;
    static __device__ __forceinline__ double dead_key(int) { return INFINITY; }
    static __device__ __forceinline__ double to_key(Cell x, int) { return x; }
    static __device__ __forceinline__ void finish(double key, uint64_t cs, int, uint32_t mask,
                                                  Cell &cell, int32_t &arg) {
        const uint64_t bits = (uint64_t)__double_as_longlong(key);
        const uint32_t hi = (uint32_t)(bits >> 32);
        // strip the index, add c * 2^k (an unbiased double): the sum keeps the bias
        cell = __longlong_as_double((long long)(bits & ~(uint64_t)mask)) +
               __longlong_as_double((long long)cs);
        // bit 29 of the high word is set for +inf (0x7ff..) and clear for 2^52 <= K < 2^53
        arg = (int32_t)((uint32_t)bits & mask) | ((int32_t)(hi << 2) >> 31);
    }
    static __device__ __forceinline__ Cell first_layer(uint64_t cs) {
        return __longlong_as_double((long long)cs) + 0x1p52;
    }
    static __device__ __forceinline__ Cell infinity() { return INFINITY; }
    static __device__ __forceinline__ int64_t to_int64(Cell x, int k) {
        if (x == INFINITY) return kInf;
        return (int64_t)((((uint64_t)__double_as_longlong(x)) & 0x000fffffffffffffull) >> k);
    }
};

// Smallest value over the wave's lanes, in every lane.
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#define GALV_DPP_MIN(ctrl) v = min(v, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, ctrl, 0xf, 0xf, false))
    GALV_DPP_MIN(0x111);                           // row_shr 1, 2, 4, 8: minimum of each row of 16 in its last lane
    GALV_DPP_MIN(0x112);
    GALV_DPP_MIN(0x114);
    GALV_DPP_MIN(0x118);
#undef GALV_DPP_MIN
    return min(min(read_lane(v, 15), read_lane(v, 31)), min(read_lane(v, 47), read_lane(v, 63)));
}
__device__ __forceinline__ uint64_t wave_min(uint64_t v) {     // (the high words' minimum, then the low words' beside it)
    const uint32_t hi = wave_min((uint32_t)(v >> 32));
    return (uint64_t)hi << 32 | wave_min((uint32_t)(v >> 32) == hi ? (uint32_t)v : 0xffffffffu);
}

// Chained sweep, words that workgroups tell each other: the counter of places, then [B][n_tiles] the last layer finished, each in
// a line of its own (a line that many ask for answers them one after the other).  Behind them the clamps of 64-bit relative costs.
__device__ __forceinline__ int32_t *chain_words(const Layout &a) { return reinterpret_cast<int32_t *>(a.U[1]); }
__device__ __forceinline__ int32_t *chain_flags(const Layout &a, int b) {
    return chain_words(a) + kWave + (int64_t)b * a.n_tiles * kWordStep;
}
__device__ __forceinline__ uint64_t *chain_clamps(const Layout &a) { return reinterpret_cast<uint64_t *>(chain_flags(a, a.B)); }
constexpr size_t chain_word_bytes(int64_t B, int64_t n_tiles) { return (size_t)(kWave + B * n_tiles * kWordStep) * 4 + (size_t)B * 8; }

// ------------------------------------------------------------------ preparation
//
// One workgroup per instance.  Checks the value preconditions, bounds the
// largest cost any plan prefix can reach, picks the arithmetic path and, for the
// fast paths, packs R and c and lists the usable strategies of every layer.
__global__ __launch_bounds__(kPrepThreads) void prep_kernel(Layout a, uint32_t flags) {
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int64_t L = a.L, S = a.S, nR = a.nR;
    // (the inputs through the constant address space: their loads may then pass the stores of the lists)
    const ConstPtr<int64_t> c = as_const(a.c + (int64_t)b * L * S);
    const ConstPtr<int32_t> m = as_const(a.m + (int64_t)b * L * S);
    const ConstPtr<int64_t> R = as_const(a.R + (int64_t)b * nR * S * S);
    const int32_t *ridx = a.r_idx ? a.r_idx + (int64_t)b * L : nullptr;
    const unsigned long long cap = (unsigned long long)kInf;

    __shared__ int bad;
    __shared__ unsigned long long rmax[64];  // max of each transition matrix (64 at a time)
    __shared__ unsigned long long red[2][kPrepThreads / kWave], red4[4][kPrepThreads / kWave];
    __shared__ int m_top;                          // layer 0's largest usable memory
    if (tid == 0) bad = 0;
    __syncthreads();
    const int wave = tid >> 6, lane = tid & 63;
    // A value of every thread, reduced over the workgroup, in every thread: one barrier (a tree in LDS took ten; the
    // slots take turns, and nobody can be two reductions ahead of a barrier).
    int turn = 0;
    auto reduce = [&](unsigned long long v, auto op) {
#pragma unroll
        for (int w = kWave / 2; w > 0; w >>= 1) v = op(v, (unsigned long long)__shfl_xor((long long)v, w, kWave));
        if (lane == 0) red[turn][wave] = v;
        __syncthreads();
        v = red[turn][lane & (kPrepThreads / kWave - 1)];
#pragma unroll
        for (int w = kPrepThreads / kWave / 2; w > 0; w >>= 1)
            v = op(v, (unsigned long long)__shfl_xor((long long)v, w, kWave));
        turn ^= 1;
        return v;
    };
    auto largest = [](unsigned long long x, unsigned long long y) { return x > y ? x : y; };
    auto sum_to_cap = [](unsigned long long x, unsigned long long y) {     // each at most 2^62: no wrap
        return x + y > cap ? cap : x + y;
    };

    const int budget = uniform(a.budget[b]);
    if (tid == 0 && (budget < 0 || budget > a.E_max)) bad = 1;

    // What the batch's sweeps really cover: the budget tiles of all instances, told to the host (a
    // word of pinned memory that the NEXT solve reads when it sizes its launches; the budgets live
    // on the device, and a solve never waits for one).
    if (a.packed == kChain) {                      // nothing told yet (see chain_words)
        if (b == 0 && tid == 0) *chain_words(a) = 0;
        for (int i = tid; i < a.n_tiles; i += kPrepThreads) chain_flags(a, b)[(int64_t)i * kWordStep] = 0;
    }
    if (a.seen && b == 0) {
        unsigned long long tiles = 0;
        for (int i = tid; i < a.B; i += kPrepThreads) {
            const int e = a.budget[i];
            if (e >= 0 && e <= a.E_max) tiles += (unsigned)(e / a.tile_e + 1);
        }
        tiles = reduce(tiles, sum_to_cap);
        if (tid == 0)
            __hip_atomic_store(a.seen, (int32_t)(tiles < 0x7fffffffull ? tiles : 0x7fffffffull),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }

    // The largest entries of the first two matrices, and how many transitions use them; then the sum over layers of max_s c(l,s),
    // saturating at 2^62: a wave per layer, a lane per strategy (one thread walking a layer's strategies is a chain of loads,
    // and with few layers most of the workgroup would idle).  All loads are on their way before the first reduction, and
    // one barrier reduces all four: this kernel's time is its round trips (one by one, 37 layers x 29 strategies took 12.7 us).
    unsigned long long of[4] = {0, 0, 0, 0};       // sum of costs; matrix 0; matrix 1; transitions with 0 and, from bit 32, with 1
    bool off = false;                              // (kept in a register: a store to `bad` inside the loops
                                                   // would hold the next iteration's loads back)
    for (int64_t k = 0; k < 2 && k < nR; ++k) {
        const ConstPtr<int64_t> Rm = R + k * S * S;
#pragma unroll 4
        for (int64_t i = tid; i < S * S; i += kPrepThreads) {
            const int64_t v = Rm[i];
            off |= v < 0 || v >= kInf;
            of[1 + k] = largest(of[1 + k], (unsigned long long)v);
        }
    }
    for (int64_t l = 1 + tid; l < L; l += kPrepThreads) {
        const int64_t k = ridx ? ridx[l] : 0;
        off |= k < 0 || k >= nR;
        of[3] += (k == 0 ? 1ull : 0) + (k == 1 ? 1ull << 32 : 0);
    }
    for (int64_t l = wave; l < L; l += kPrepThreads / kWave) {
        unsigned long long mx = 0;
#pragma unroll 2
        for (int64_t s = lane; s < S; s += kWave) {
            const int64_t v = c[l * S + s];
            off |= v < 0 || v >= kInf || m[l * S + s] < 0;
            if ((unsigned long long)v > mx) mx = (unsigned long long)v;
        }
        mx = ~(unsigned long long)wave_min((uint64_t)~mx);
        if (lane == 0) of[0] = sum_to_cap(of[0], mx < cap ? mx : cap);
    }
    if (off) bad = 1;
    auto join = [&](int q, unsigned long long x, unsigned long long y) { return q == 0 ? sum_to_cap(x, y) : q == 3 ? x + y : largest(x, y); };
#pragma unroll
    for (int w = kWave / 2; w > 0; w >>= 1)
#pragma unroll
        for (int q = 0; q < 4; ++q) of[q] = join(q, of[q], (unsigned long long)__shfl_xor((long long)of[q], w, kWave));
    if (lane < 4) red4[lane][wave] = lane == 0 ? of[0] : lane == 1 ? of[1] : lane == 2 ? of[2] : of[3];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) of[q] = red4[q][lane & (kPrepThreads / kWave - 1)];
#pragma unroll
    for (int w = kPrepThreads / kWave / 2; w > 0; w >>= 1)
#pragma unroll
        for (int q = 0; q < 4; ++q) of[q] = join(q, of[q], (unsigned long long)__shfl_xor((long long)of[q], w, kWave));
    const unsigned long long bound_c = of[0];
    // the sum, over the layer transitions, of the largest entry of the matrix each uses
    auto times = [&](unsigned long long n, unsigned long long x) {
        return __umul64hi(n, x) != 0 || n * x > cap ? cap : n * x;
    };
    unsigned long long rmax_all = largest(of[1], of[2]);
    unsigned long long rsum = sum_to_cap(times(of[3] & 0xffffffffull, of[1] < cap ? of[1] : cap), times(of[3] >> 32, of[2] < cap ? of[2] : cap));
    for (int64_t k0 = 2; k0 < nR; k0 += 64) {
        const int64_t kn = (nR - k0 < 64) ? nR - k0 : 64;
        for (int64_t k = 0; k < kn; ++k) {
            unsigned long long mx = 0;
            const ConstPtr<int64_t> Rm = R + (k0 + k) * S * S;
            bool wrong = false;
#pragma unroll 4
            for (int64_t i = tid; i < S * S; i += kPrepThreads) {
                const int64_t v = Rm[i];
                wrong |= v < 0 || v >= kInf;
                if ((unsigned long long)v > mx) mx = (unsigned long long)v;
            }
            if (wrong) bad = 1;
            mx = reduce(mx, largest);
            if (tid == 0) rmax[k] = mx;
            rmax_all = largest(rmax_all, mx);
        }
        __syncthreads();
        // (every thread adds up the layers it owns, saturating; one thread walking all layers is
        // a chain of dependent loads that takes longer than the rest of this kernel)
        unsigned long long part_r = 0;
        for (int64_t l = 1 + tid; l < L; l += kPrepThreads) {
            const int64_t k = ridx ? ridx[l] : 0;
            if (k >= k0 && k < k0 + kn) {
                part_r += rmax[k - k0];
                if (part_r > cap) part_r = cap;
            }
        }
        rsum = sum_to_cap(rsum, reduce(part_r, sum_to_cap));
    }

    // (what was found wrong stands behind a barrier since; every thread works out the same status)
    int st;
    const unsigned long long bound = bound_c + rsum;       // each <= 2^62: no wrap
    {
        if (bad || bound >= cap) {
            st = GALV_INSTANCE_BAD_VALUE;
        } else if (flags & GALV_DP_FORCE_INT64) {
            st = GALV_INSTANCE_OK_INT64;
        } else if (bound + rmax_all < kInf32) {
            // costs, and infinity + R, fit 32 bits.  If, besides, twice the largest R still
            // leaves room for the index in a 32-bit key, the integer path applies.
            const bool u32 = !(flags & GALV_DP_NO_U32) &&
                             ((2 * rmax_all + 2) << a.k_bits) <= (1ull << 32);
            st = u32 ? GALV_INSTANCE_OK_FAST_U32 : GALV_INSTANCE_OK_FAST;
        } else if (a.synth_l1 && !(flags & GALV_DP_NO_U32) && rmax_all < (1ull << 32) &&
                   ((2 * rmax_all + 2) << a.k_bits) <= (1ull << 32)) {
            // costs need 64-bit cells, but only RELATIVE costs (clamped at R_max + 1) enter the keys:
            // the 32-bit-key arithmetic and its pruning apply all the same (row-sharing variants)
            st = GALV_INSTANCE_OK_U32_WIDE;
        } else if (bound + 1 <= (1ull << (52 - a.k_bits))) {
            st = GALV_INSTANCE_OK_FAST_WIDE;    // keys fit the 52-bit mantissa
        } else {
            st = GALV_INSTANCE_OK_INT64;
        }
    }
    uint32_t clamp = rmax_all < 0xffffffffull ? (uint32_t)(rmax_all + 1) : 0u;
    if (tid == 0) a.status[b] = st;
    // The byte table saves what the pruning lets it save.  Where transition costs dwarf the spread of the layer
    // costs, hardly a row is left out, and an instance on 64-bit keys rebuilds every cell that it could have read:
    // it keeps cost rows instead (clamp 0 says so, see byte_status), as long as these stay in the caches.  Rows of
    // a layer differ in cost by about what their strategies do there, so a strategy counts as alive that costs less
    // than the layer's cheapest plus the largest transition cost.  Whole solves of 10 layers over cost rows / with the
    // byte table, in us, share of alive strategies 1.0: 22 strategies x 1512 tiles 201 / 258, 44 x 1512 379 / 493, 14 x
    // 3760 250 / 374; 0.55: 34 x 582 97 / 101; 0.35: 22 x 1512 202 / 180, 44 x 1512 379 / 254.
    if (a.packed == kRowsIfAlive && (st == GALV_INSTANCE_OK_FAST || st == GALV_INSTANCE_OK_FAST_WIDE)) {
        unsigned long long seen = 0;               // usable << 32 | alive
        for (int64_t l = wave; l + 1 < L; l += kPrepThreads / kWave) {
            unsigned long long v[4], least = ~0ull;           // (the byte table has at most 256 strategies)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t s = q * kWave + lane, at = l * S + (s < S ? s : 0);
                const unsigned long long cost = (unsigned long long)c[at];
                v[q] = s < S && m[at] <= budget ? cost : ~0ull;
                least = v[q] < least ? v[q] : least;
            }
#pragma unroll
            for (int w = kWave / 2; w > 0; w >>= 1) {
                const unsigned long long o = (unsigned long long)__shfl_xor((long long)least, w, kWave);
                least = o < least ? o : least;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (v[q] != ~0ull) seen += (1ull << 32) + (v[q] - least <= rmax_all ? 1 : 0);
        }
        seen = reduce(seen, [](unsigned long long x, unsigned long long y) { return x + y; });
        if (4 * (seen & 0xffffffffull) > 3 * (seen >> 32)) clamp = 0;
    }
    // One record per layer with what a sweep workgroup needs before anything else, so that it
    // takes one load instead of a chain of them.  (The count of the former layer's usable
    // strategies is filled in below, by the wave that builds that layer's list, if any.)
    if (tid == 0) a.dclamp[b] = clamp;
    if (a.packed == kChain && tid == 0) chain_clamps(a)[b] = (rmax_all < bound ? rmax_all : bound) + 1;
    const bool lists = narrow_cells(st) || st == GALV_INSTANCE_OK_FAST_WIDE || st == GALV_INSTANCE_OK_U32_WIDE;
    const bool bytes = a.packed && L > 1 && byte_status(a, st, clamp);
    for (int64_t l = tid; l < L; l += kPrepThreads) {
        int32_t *h = a.hdr + ((int64_t)b * L + l) * 8;
        h[0] = st;
        h[1] = budget;
        if (!lists || l == 0) h[2] = 0;
        h[3] = (int32_t)clamp;
        h[4] = (ridx && l >= 1 && st >= 0) ? ridx[l] : 0;
        h[5] = 0;
        h[6] = a.packed == kChain && l > 1 && bytes ? kUnset : budget;
    }
    if (!lists) return;

    // R key = R * 2^k + s' (s' = row = former strategy); padded columns are +inf so
    // that they never win and never read past the caller's matrix.
    const double scale = (double)(1ull << a.k_bits);
    double *Rk = a.Rk + (int64_t)b * nR * S * a.S_pad;
    // (a wave per matrix row / per layer and a lane per column: no index arithmetic per element)
    constexpr int kWaves = kPrepThreads / kWave;
    const int S_pad = a.S_pad;
    const bool keys32 = st == GALV_INSTANCE_OK_FAST_U32 || st == GALV_INSTANCE_OK_U32_WIDE;
    for (int64_t k = 0; k < nR; ++k) {
        for (int sp = wave; sp < (int)S; sp += kWaves) {
            const ConstPtr<int64_t> src = R + (k * S + sp) * S;
            if (keys32) {
                // 32-bit keys in the first half of each matrix's slot: rows of S_pad words, one
                // matrix every S * S_pad doubles; padded columns hold the largest word.
                uint32_t *row = reinterpret_cast<uint32_t *>(Rk + k * S * S_pad) + (int64_t)sp * S_pad;
                for (int sx = lane; sx < S_pad; sx += kWave)
                    row[sx] = (sx < (int)S) ? (((uint32_t)src[sx]) << a.k_bits) | (uint32_t)sp : 0xffffffffu;
            } else {
                double *row = Rk + (k * S + sp) * S_pad;
                for (int sx = lane; sx < S_pad; sx += kWave)
                    row[sx] = (sx < (int)S) ? (double)src[sx] * scale + (double)sp : INFINITY;
            }
        }
    }
    // Per layer, the strategies whose memory fits the budget at all, in ascending
    // order, with their shift: the sweep of the next layer walks this list instead
    // of all S columns (a column that never fits is infinity everywhere).
    // (a wave per layer, a lane per strategy: the usable ones find their place in the list by
    // counting the usable lanes below them)
    // Beside it c(l,s) in the form the epilogue adds: the integer itself (integer cells) or the
    // double c * 2^k (cells that hold 64-bit keys).
    uint64_t *ck = a.ck + (int64_t)b * L * S_pad;
    const bool c_int = narrow_cells(st) || st == GALV_INSTANCE_OK_U32_WIDE || bytes;
    for (int64_t l = wave; l < L; l += kPrepThreads / kWave) {
        uint64_t *lst = a.vlist + ((int64_t)b * L + l) * a.S_pad;
        uint64_t *lc = a.vcost + ((int64_t)b * L + l) * a.S_pad;
        int n = 0, m_lo = budget + 1, m_hi = 0;    // usable strategies, their smallest and largest memory
        uint64_t last_ent = 0, last_c = 0;         // the list's last entry so far (wave-uniform)
        for (int s0 = 0; s0 < S_pad; s0 += kWave) {
            const int sx = s0 + lane;
            const bool in = sx < (int)S;
            const int sh = in ? m[l * S + sx] : 0;
            const uint64_t cv = in ? (uint64_t)c[l * S + sx] : 0;
            if (sx < S_pad) ck[l * S_pad + sx] = c_int ? cv : (uint64_t)__double_as_longlong((double)(int64_t)cv * scale);
            const bool ok = in && sh <= budget;
            if (ok) {
                m_lo = min(m_lo, sh);
                m_hi = max(m_hi, sh);
            }
            const uint64_t ent = ((uint64_t)(uint32_t)sh << 32) | (uint32_t)sx;
            const uint64_t votes = __builtin_amdgcn_ballot_w64(ok);
            if (ok) {
                const int pos = n + __builtin_popcountll(votes & ((1ull << lane) - 1ull));
                lst[pos] = ent;
                lc[pos] = cv;
            }
            if (votes != 0) {                      // wave-uniform
                const int top = 63 - __builtin_clzll(votes);
                last_ent = read_lane(ent, top);
                last_c = read_lane(cv, top);
                n += __builtin_popcountll(votes);
            }
        }
        m_lo = (int)wave_min((uint32_t)m_lo);      // (neither is negative)
        m_hi = (int)~wave_min(~(uint32_t)m_hi);
        if (lane == 0) {
            a.nvalid[(int64_t)b * L + l] = n;
            a.hdr[((int64_t)b * L + l) * 8 + 7] = m_lo;
            if (l + 1 < L) a.hdr[((int64_t)b * L + l + 1) * 8 + 2] = n;
            if (l == 0) m_top = m_hi;
        }
        // Past the list's end its last entry repeats (it changes no minimum: min(x, x) = x), so
        // a sweep that walks a fixed number of entries needs no bound check; an empty list is
        // never walked.
        if (n > 0)
            for (int i = n + lane; i < a.S_pad; i += kWave) {
                lst[i] = last_ent;
                lc[i] = last_c;
            }
    }
    if (!bytes) return;
    // Columns of each layer that are worth sweeping (see the byte-table sweep): from the sum of the
    // smallest memories before it, saturating above the budget (a wave's prefix sum, 64 layers at a
    // time); layer 1 up to layer 0's largest memory, later layers as live_step finds.
    __syncthreads();
    if (wave != 0) return;
    int64_t before = 0;
    for (int l0 = 0; l0 < (int)L; l0 += kWave) {
        const int l = l0 + lane;
        int32_t *h = a.hdr + ((int64_t)b * L + (l < L ? l : L - 1)) * 8;
        const int64_t mine = l < L ? h[7] : 0;
        int64_t sum = mine;
#pragma unroll
        for (int w = 1; w < kWave; w <<= 1) {
            const int64_t o = __shfl_up((long long)sum, w, kWave);
            if (lane >= w) sum += o;
        }
        if (l < L) {
            const int64_t y = before + sum - mine;
            h[5] = (int32_t)(y <= budget ? y : (int64_t)budget + 1);
            if (l == 1) h[6] = m_top < budget - (int)mine ? m_top : budget - (int)mine;
        }
        before += __shfl((long long)sum, kWave - 1, kWave);
    }
}

// Layer 0: U_0[e'][s] = c(0,s) for every e' (the shift by m(0,s) is applied by
// whoever reads it), and the infinity lead in front of both rolling rows of the
// strategy.  Grid: (a few blocks that stride over the row, S, B).
//
// The leads never change while an instance keeps its storage mode, and no sweep
// writes into them, so only the first solve of a handle (fresh != 0) and a solve
// that finds another mode than the one recorded in lead_mode[b] write them;
// final_kernel records the mode once the solve is through.
__global__ __launch_bounds__(kThreads) void init_kernel(Layout a, int fresh) {
    const int b = blockIdx.z, s = blockIdx.y;
    const int st = uniform(a.status[b]);
    if (st < 0) return;
    const int64_t base = ((int64_t)b * a.S_pad + s) * a.row * 8;
    const int64_t x0 = (int64_t)blockIdx.x * kThreads + threadIdx.x, step = (int64_t)gridDim.x * kThreads;
    if (st == GALV_INSTANCE_OK_INT64) {
        const int64_t c0 = a.c[((int64_t)b * a.L) * a.S + s];
        for (int64_t x = a.lead + x0; x < a.row; x += step) reinterpret_cast<int64_t *>(a.U[0] + base)[x] = c0;
        return;
    }
    if (is_packed(a, st, b)) return;               // no cost rows: layer 0 is made up, the sweeps test the shift
    const bool leads = fresh || a.lead_mode[b] != lead_kind(st);
    const bool u32_keys = st == GALV_INSTANCE_OK_FAST_U32 || st == GALV_INSTANCE_OK_U32_WIDE;
    const bool row0 = !(u32_keys && a.synth_l1 && a.L > 1);
    if (!leads && !row0) return;                   // the usual case after a handle's first solve
    const uint64_t cs = a.ck[((int64_t)b * a.L) * a.S_pad + s];
    if (narrow_cells(st)) {
        uint32_t *u0 = reinterpret_cast<uint32_t *>(a.U[0] + base);
        uint32_t *u1 = reinterpret_cast<uint32_t *>(a.U[1] + base);
        if (leads)
            for (int64_t x = x0; x < a.lead; x += step) {
                u0[x] = Narrow::infinity();
                u1[x] = Narrow::infinity();
            }
        if (row0)
            for (int64_t x = a.lead + x0; x < a.row; x += step) u0[x] = Narrow::first_layer(cs);
    } else if (st == GALV_INSTANCE_OK_U32_WIDE) {
        uint64_t *u0 = reinterpret_cast<uint64_t *>(a.U[0] + base);
        uint64_t *u1 = reinterpret_cast<uint64_t *>(a.U[1] + base);
        if (leads)
            for (int64_t x = x0; x < a.lead; x += step) {
                u0[x] = (uint64_t)kInf;
                u1[x] = (uint64_t)kInf;
            }
        if (row0)
            for (int64_t x = a.lead + x0; x < a.row; x += step) u0[x] = cs;
    } else {
        double *u0 = reinterpret_cast<double *>(a.U[0] + base);
        double *u1 = reinterpret_cast<double *>(a.U[1] + base);
        if (leads)
            for (int64_t x = x0; x < a.lead; x += step) {
                u0[x] = Wide::infinity();
                u1[x] = Wide::infinity();
            }
        for (int64_t x = a.lead + x0; x < a.row; x += step) u0[x] = Wide::first_layer(cs);
    }
}

// ---------------------------------------------------------------- layer sweep

// General 64-bit integer body: one budget column per thread at a time, strategy
// columns in chunks of CH running (min, argmin) pairs.
template <int CH>
__device__ __forceinline__ void sweep_int64(const Layout &a, int wave, int l, int b, int budget,
                                            int64_t tile_start) {
    const int64_t S = a.S;
    const int64_t *Uprev = reinterpret_cast<const int64_t *>(a.U[(l - 1) & 1]) +
                           (int64_t)b * a.S_pad * a.row + a.lead;
    int64_t *Unew = reinterpret_cast<int64_t *>(a.U[l & 1]) + (int64_t)b * a.S_pad * a.row + a.lead;
    const int64_t bp0 = ((int64_t)b * (a.L - 1) + (l - 1)) * S * a.e_pad;
    const int32_t *mprev = a.m + ((int64_t)b * a.L + (l - 1)) * S;
    const int64_t *cl = a.c + ((int64_t)b * a.L + l) * S;
    const int r = a.r_idx ? a.r_idx[(int64_t)b * a.L + l] : 0;
    const int64_t *R = a.R + ((int64_t)b * a.nR + r) * S * S;

    for (int64_t e = tile_start + wave * kWave + lane_id(); e < tile_start + a.tile_e; e += blockDim.x) {
        if (e > budget) continue;
        for (int64_t s0 = 0; s0 < S; s0 += CH) {
            int64_t best[CH];
            int32_t arg[CH];
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                best[q] = kInf;
                arg[q] = -1;
            }
            for (int64_t sp = 0; sp < S; ++sp) {
                const int64_t shift = mprev[sp];
                if (shift > budget) continue;             // whole column is infinity
                const int64_t es = e - shift;
                const int64_t v = (es >= 0) ? Uprev[sp * a.row + es] : kInf;
                const int64_t *Rrow = R + sp * S;
#pragma unroll
                for (int q = 0; q < CH; ++q) {
                    const int64_t col = (s0 + q < S) ? s0 + q : S - 1;
                    const int64_t cand = v + Rrow[col];
                    if (cand < best[q]) {                 // strict: lowest s' keeps ties
                        best[q] = cand;
                        arg[q] = (int32_t)sp;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < CH; ++q) {
                if (s0 + q < S) {
                    const bool dead = best[q] >= kInf;
                    Unew[(s0 + q) * a.row + e] = dead ? kInf : best[q] + cl[s0 + q];
                    store_bp(a, bp0 + (s0 + q) * a.e_pad + e, dead ? -1 : arg[q]);
                }
            }
        }
    }
}

// acc[j] = min(acc[j], v[j] + rk) on packed keys: one v_add_f64 and one v_min_f64
// per candidate, rk a wave-uniform SGPR pair.  Written as one asm block per
// strategy so that each needs only TE temporaries (left to itself the scheduler
// hoists every add of a row above the minima and spills), with the adds ahead of
// the minima so that no instruction waits on the one just issued.
typedef double double8 __attribute__((ext_vector_type(8)));

// `keep0`, `keep1` are the registers of the R group that is still being loaded while this
// statement runs: naming them as (unused) inputs keeps their next use close, so the
// register allocator has no reason to spill or move them while the load is in flight.
template <int TE, class K0, class K1>
__device__ __forceinline__ void minplus(double (&acc)[TE], const double (&v)[TE], double rk,
                                        const K0 &keep0, const K1 &keep1) {
    static_assert(TE == 1 || TE == 2 || TE == 4, "budget columns per lane");
    if constexpr (TE == 1) {
        double t0;
        asm("v_add_f64 %1, %2, %3\n\tv_min_f64 %0, %0, %1"
            : "+v"(acc[0]), "=&v"(t0)
            : "v"(v[0]), "s"(rk), "s"(keep0), "s"(keep1));
    } else if constexpr (TE == 2) {
        double t0, t1;
        asm("v_add_f64 %2, %4, %6\n\tv_add_f64 %3, %5, %6\n\t"
            "v_min_f64 %0, %0, %2\n\tv_min_f64 %1, %1, %3"
            : "+v"(acc[0]), "+v"(acc[1]), "=&v"(t0), "=&v"(t1)
            : "v"(v[0]), "v"(v[1]), "s"(rk), "s"(keep0), "s"(keep1));
    } else {
        double t0, t1, t2, t3;
        asm("v_add_f64 %4, %8, %12\n\tv_add_f64 %5, %9, %12\n\t"
            "v_add_f64 %6, %10, %12\n\tv_add_f64 %7, %11, %12\n\t"
            "v_min_f64 %0, %0, %4\n\tv_min_f64 %1, %1, %5\n\t"
            "v_min_f64 %2, %2, %6\n\tv_min_f64 %3, %3, %7"
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "=&v"(t0), "=&v"(t1),
              "=&v"(t2), "=&v"(t3)
            : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(rk), "s"(keep0), "s"(keep1));
    }
}

// A group of R keys in SGPRs: 8 * NCH doubles fetched by NCH scalar loads of 16
// dwords.  The loads are issued by hand (the compiler would wait for each right
// where it issues it); rgroup_await makes every later use depend on the wait.
// Between request and await the compiler believes the destination registers are
// already defined; were it to spill or reuse them there (it does under heavy SGPR
// pressure, e.g. a deeper prefetch with an unsuitable tile shape), late-arriving
// data would overwrite whatever it put there.  The build refuses such code: it
// scans the produced assembly for any use of a destination register, any label or
// any branch between a request and its wait (paper_2211_13878_amd/isa_check.py).
template <int NCH>
struct RGroup {
    double8 c[NCH];
};
__device__ __forceinline__ void rgroup_request(RGroup<1> &g, ConstPtr<double> p) {
    asm volatile("s_load_dwordx16 %0, %1, 0x0" : "=&s"(g.c[0]) : "s"(p));
}
__device__ __forceinline__ void rgroup_request(RGroup<2> &g, ConstPtr<double> p) {
    asm volatile("s_load_dwordx16 %0, %2, 0x0\n\ts_load_dwordx16 %1, %2, 0x40"
                 : "=&s"(g.c[0]), "=&s"(g.c[1])
                 : "s"(p));
}
__device__ __forceinline__ void rgroup_await(RGroup<1> &g) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(g.c[0]));
}
__device__ __forceinline__ double rgroup_key(const RGroup<1> &g, int x) { return g.c[0][x]; }
__device__ __forceinline__ double rgroup_key(const RGroup<2> &g, int x) { return g.c[x / 8][x % 8]; }
__device__ __forceinline__ const double8 &rgroup_keep0(const RGroup<1> &g) { return g.c[0]; }
__device__ __forceinline__ const double8 &rgroup_keep1(const RGroup<1> &g) { return g.c[0]; }
__device__ __forceinline__ const double8 &rgroup_keep0(const RGroup<2> &g) { return g.c[0]; }
__device__ __forceinline__ const double8 &rgroup_keep1(const RGroup<2> &g) { return g.c[1]; }
// 9 to 12 keys: 8 + 4 doubles.  (Two buffers of 16 would take 64 of the ~100 scalar registers;
// the compiler then moves or spills registers that a load in flight still targets, which the
// build refuses.)
typedef double double4 __attribute__((ext_vector_type(4)));
struct RGroupMid {
    double8 lo;
    double4 hi;
};
__device__ __forceinline__ void rgroup_request(RGroupMid &g, ConstPtr<double> p) {
    asm volatile("s_load_dwordx16 %0, %2, 0x0\n\ts_load_dwordx8 %1, %2, 0x40"
                 : "=&s"(g.lo), "=&s"(g.hi)
                 : "s"(p));
}
__device__ __forceinline__ void rgroup_await(RGroupMid &g) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(g.lo), "+s"(g.hi));
}
__device__ __forceinline__ double rgroup_key(const RGroupMid &g, int x) { return x < 8 ? g.lo[x] : g.hi[x - 8]; }
__device__ __forceinline__ const double8 &rgroup_keep0(const RGroupMid &g) { return g.lo; }
__device__ __forceinline__ const double4 &rgroup_keep1(const RGroupMid &g) { return g.hi; }
__device__ __forceinline__ void rgroup_await(RGroup<2> &g) {
    asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(g.c[0]), "+s"(g.c[1]));
}

// Fast body.  Lane owns TE budget columns (64 apart) and TS strategy columns; per
// usable s' it loads its TE shifted previous-layer cells once and reuses them for
// all TS strategies, with the R keys as wave-uniform scalars.
// The wave's position is explicit: its first budget column e_wave and its first strategy s0.
template <int TS, int TE, class Store, class BP>
__device__ __forceinline__ void sweep_fast_at(const Layout &a, int l, int b, int budget,
                                              int64_t e_wave, int64_t s0) {
    using Cell = typename Store::Cell;
    constexpr int64_t kPerSlot = 8 / sizeof(Cell);     // cells per reserved 8-byte slot
    const int lane = lane_id();
    const int64_t e0 = e_wave + lane;
    if (s0 >= a.S) return;
    if (e_wave > budget) return;

    const int64_t S = a.S;
    const int k = a.k_bits;
    const int64_t pitch = a.row * kPerSlot;        // cells between rows of two strategies
    // wave-uniform base of the previous layer's rows; the lane adds only its own column, so
    // that the shifted addresses are a scalar base plus a loop-invariant lane offset
    const Cell *Up = reinterpret_cast<const Cell *>(a.U[(l - 1) & 1]) +
                     (int64_t)b * a.S_pad * pitch + a.lead + (e0 - lane);
    Cell *Un = reinterpret_cast<Cell *>(a.U[l & 1]) + ((int64_t)b * a.S_pad + s0) * pitch +
               a.lead + e0;
    BP *bp = static_cast<BP *>(a.bp) + (((int64_t)b * (a.L - 1) + (l - 1)) * S + s0) * a.e_pad + e0;
    const int r = a.r_idx ? a.r_idx[(int64_t)b * a.L + l] : 0;
    const ConstPtr<double> Rk = as_const(a.Rk + ((int64_t)b * a.nR + r) * S * a.S_pad + s0);
    const ConstPtr<uint64_t> ck = as_const(a.ck + ((int64_t)b * a.L + l) * a.S_pad + s0);

    double acc[TS][TE];
    const double dead = Store::dead_key(k);
#pragma unroll
    for (int s = 0; s < TS; ++s)
#pragma unroll
        for (int j = 0; j < TE; ++j) acc[s][j] = dead;

    // Walk the usable former-layer strategies (list built by the preparation
    // kernel; entries are wave-uniform scalars).  Two software pipelines run
    // under the arithmetic:
    //  * the shifted previous-layer cells of entry i + kDepth are requested
    //    while entry i is reduced (vector loads, kDepth - 1 entries of cover);
    //  * the R keys of a row arrive in groups of up to 16 doubles through explicit
    //    scalar loads into one of two SGPR buffers: the next group is requested
    //    before the current one is consumed and awaited after it.
    const ConstPtr<uint64_t> vl = as_const(a.vlist + ((int64_t)b * a.L + (l - 1)) * a.S_pad);
    const int n = as_const(a.nvalid)[(int64_t)b * a.L + (l - 1)];
    if (n > 0) {
        constexpr int kChunks = TS > 8 ? 2 : 1;            // scalar loads per group
        constexpr int kGroup = 8 * kChunks;                // doubles per group
        constexpr int kGroups = (TS + kGroup - 1) / kGroup;
        static_assert((kDepth * kGroups) % 2 == 0, "buffer roles must repeat every loop trip");
        Cell v[kDepth][TE];
        int sps[kDepth];
        using Group = std::conditional_t<(TS > 8 && TS <= 12), RGroupMid, RGroup<kChunks>>;
        Group buf[2];
        // Requests are never conditional (past the end they repeat the last entry,
        // which is cached) so that no wait is needed where control flow joins.
        auto request = [&](int q, int i) {
            const uint64_t ent = vl[i < n ? i : n - 1];
            sps[q] = (int)(uint32_t)ent;
            const Cell *p = Up + (int64_t)(uint32_t)ent * pitch - (int64_t)(ent >> 32);
#pragma unroll
            for (int j = 0; j < TE; ++j) v[q][j] = p[(uint32_t)lane + j * kWave];
        };
        // One entry: for each group, request the following group (of this entry or
        // of the next entry's row), reduce the current one, then await the request.
        auto reduce_entry = [&](int q) {
            double key[TE];
#pragma unroll
            for (int j = 0; j < TE; ++j) key[j] = Store::to_key(v[q][j], k);
#pragma unroll
            for (int gr = 0; gr < kGroups; ++gr) {
                const int t = q * kGroups + gr;
                const int qn = (gr + 1 < kGroups) ? q : (q + 1) % kDepth;
                const int gn = (gr + 1 < kGroups) ? gr + 1 : 0;
                rgroup_request(buf[(t + 1) & 1], Rk + (int64_t)sps[qn] * a.S_pad + gn * kGroup);
#pragma unroll
                for (int x = 0; x < kGroup; ++x)
                    if (gr * kGroup + x < TS)
                        minplus<TE>(acc[gr * kGroup + x], key, rgroup_key(buf[t & 1], x),
                                    rgroup_keep0(buf[(t + 1) & 1]), rgroup_keep1(buf[(t + 1) & 1]));
                rgroup_await(buf[(t + 1) & 1]);
            }
        };
#pragma unroll
        for (int q = 0; q < kDepth; ++q) request(q, q);
        rgroup_request(buf[0], Rk + (int64_t)sps[0] * a.S_pad);
        rgroup_await(buf[0]);
        int i = 0;
        for (; i + kDepth <= n; i += kDepth) {
#pragma unroll
            for (int q = 0; q < kDepth; ++q) {
                reduce_entry(q);
                request(q, i + q + kDepth);
            }
        }
#pragma unroll
        for (int q = 0; q < kDepth - 1; ++q)
            if (i + q < n) reduce_entry(q);
    }

    const uint32_t mask = (1u << k) - 1u;
#pragma unroll
    for (int s = 0; s < TS; ++s) {
        if (s0 + s < S) {
            const uint64_t cs = ck[s];
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                Cell cell;
                int32_t arg;
                Store::finish(acc[s][j], cs, k, mask, cell, arg);
                Un[(int64_t)s * pitch + j * kWave] = cell;
                // Back-pointers are written once and read again only by the backtrack: a
                // streaming store keeps them from pushing the cost rows, which the next
                // layer reads back, out of the caches.  (-1 becomes 0xFF in one byte.)
                __builtin_nontemporal_store((BP)arg, &bp[(int64_t)s * a.e_pad + j * kWave]);
            }
        }
    }
}

// Position of a wave in a workgroup of NG strategy groups x (waves / NG) budget sub-tiles.
template <int TS, int TE, int NG, class Store, class BP>
__device__ __forceinline__ void sweep_fast(const Layout &a, int wave, int l, int b, int budget,
                                           int64_t tile_start) {
    const int g = wave % NG;                       // strategy group of this wave
    const int esub = wave / NG;                    // budget sub-tile of this wave
    sweep_fast_at<TS, TE, Store, BP>(a, l, b, budget, tile_start + (int64_t)esub * (kWave * TE),
                                     ((int64_t)blockIdx.y * NG + g) * TS);
}

// ------------------------------------------------------- 32-bit integer keys
//
// When costs fit 32 bits and twice the largest transition cost R_max still leaves
// room for the index, the inner minimum runs on 32-bit integers, two candidates per
// three instructions (two adds and one three-way minimum) instead of two per four.
// Costs are taken RELATIVE to the column's smallest former cost Cmin(e') =
// min_{s'} C[l-1][e'][s'] and clamped at D = R_max + 1:
//     key(s') = (min(C[l-1][e'][s'] - Cmin, D) + R(s', s)) * 2^k + s'   <  2^32.
// Clamping changes no result: the former strategy that attains Cmin gives a
// candidate of at most Cmin + R_max, while a clamped one costs at least
// Cmin + R_max + 1, so it neither wins nor ties.  Cmin comes from a first pass over
// the same shifted cells (they are then read again from the caches).  The new cell
// is Cmin + (key >> k) + c(l, s); a column without any reachable former cell
// (Cmin = infinity) stays infinity.
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint8v __attribute__((ext_vector_type(8)));
typedef uint32_t uint16v __attribute__((ext_vector_type(16)));
typedef uint16v uint16v_u __attribute__((aligned(8)));      // 16 words at any 8-byte boundary

// The R keys of one former strategy for TS strategy columns, in as few scalar registers as
// the loads allow (8, 8 + 4 or 16): four such rows are live at a time.
template <int TS, class = void>
struct R32Row;
template <int TS>
struct R32Row<TS, std::enable_if_t<(TS <= 8)>> {
    uint8v lo;
    uint32_t hi = 0;       // (unused; keeps the three shapes alike)
    __device__ __forceinline__ uint32_t at(int s) const { return lo[s]; }
    __device__ __forceinline__ void request(ConstPtr<uint32_t> p) {
        asm volatile("s_load_dwordx8 %0, %1, 0x0" : "=&s"(lo) : "s"(p));
    }
    __device__ __forceinline__ void tie() { asm volatile("" : "+s"(lo)); }
};
template <int TS>
struct R32Row<TS, std::enable_if_t<(TS > 8 && TS <= 12)>> {
    uint8v lo;
    uint4v hi;
    __device__ __forceinline__ uint32_t at(int s) const { return s < 8 ? lo[s] : hi[s - 8]; }
    __device__ __forceinline__ void request(ConstPtr<uint32_t> p) {
        asm volatile("s_load_dwordx8 %0, %2, 0x0\n\ts_load_dwordx4 %1, %2, 0x20"
                     : "=&s"(lo), "=&s"(hi)
                     : "s"(p));
    }
    __device__ __forceinline__ void tie() { asm volatile("" : "+s"(lo), "+s"(hi)); }
};
template <int TS>
struct R32Row<TS, std::enable_if_t<(TS > 12)>> {
    uint16v lo;
    uint32_t hi = 0;       // (unused; keeps the three shapes alike)
    __device__ __forceinline__ uint32_t at(int s) const { return lo[s]; }
    __device__ __forceinline__ void request(ConstPtr<uint32_t> p) {
        asm volatile("s_load_dwordx16 %0, %1, 0x0" : "=&s"(lo) : "s"(p));
    }
    __device__ __forceinline__ void tie() { asm volatile("" : "+s"(lo)); }
};
// Wait for every outstanding scalar load; the rows passed in become usable only after it.
template <class Row>
__device__ __forceinline__ void r32_await(Row &g0, Row &g1) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    g0.tie();
    g1.tie();
}

// acc = min(acc, va + ra, vb + rb) per budget column.  `keep...` are the registers of the
// rows still being loaded: naming them as (unused) inputs of every statement between their
// request and their wait keeps their next use close, so the register allocator has no
// reason to spill or move them while the loads are in flight.
template <int TE, class Row>
__device__ __forceinline__ void minplus_u32x2(uint32_t (&acc)[TE], const uint32_t (&va)[TE],
                                              const uint32_t (&vb)[TE], uint32_t ra, uint32_t rb,
                                              const Row &ka, const Row &kb) {
    static_assert(TE == 1 || TE == 2 || TE == 4, "budget columns per lane");
    if constexpr (TE == 1) {
        uint32_t t0, t1;
        asm("v_add_u32 %1, %5, %3\n\tv_add_u32 %2, %6, %4\n\tv_min3_u32 %0, %0, %1, %2"
            : "+v"(acc[0]), "=&v"(t0), "=&v"(t1)
            : "v"(va[0]), "v"(vb[0]), "s"(ra), "s"(rb), "s"(ka.lo), "s"(ka.hi), "s"(kb.lo), "s"(kb.hi));
    } else if constexpr (TE == 2) {
        uint32_t t0, t1, t2, t3;
        asm("v_add_u32 %2, %10, %6\n\tv_add_u32 %3, %11, %8\n\t"
            "v_add_u32 %4, %10, %7\n\tv_add_u32 %5, %11, %9\n\t"
            "v_min3_u32 %0, %0, %2, %3\n\tv_min3_u32 %1, %1, %4, %5"
            : "+v"(acc[0]), "+v"(acc[1]), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3)
            : "v"(va[0]), "v"(va[1]), "v"(vb[0]), "v"(vb[1]), "s"(ra), "s"(rb), "s"(ka.lo), "s"(ka.hi),
              "s"(kb.lo), "s"(kb.hi));
    } else {
        uint32_t t0, t1, t2, t3, t4, t5, t6, t7;
        asm("v_add_u32 %4, %20, %12\n\tv_add_u32 %5, %21, %16\n\t"
            "v_add_u32 %6, %20, %13\n\tv_add_u32 %7, %21, %17\n\t"
            "v_add_u32 %8, %20, %14\n\tv_add_u32 %9, %21, %18\n\t"
            "v_add_u32 %10, %20, %15\n\tv_add_u32 %11, %21, %19\n\t"
            "v_min3_u32 %0, %0, %4, %5\n\tv_min3_u32 %1, %1, %6, %7\n\t"
            "v_min3_u32 %2, %2, %8, %9\n\tv_min3_u32 %3, %3, %10, %11"
            : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "=&v"(t0), "=&v"(t1),
              "=&v"(t2), "=&v"(t3), "=&v"(t4), "=&v"(t5), "=&v"(t6), "=&v"(t7)
            : "v"(va[0]), "v"(va[1]), "v"(va[2]), "v"(va[3]), "v"(vb[0]), "v"(vb[1]), "v"(vb[2]),
              "v"(vb[3]), "s"(ra), "s"(rb), "s"(ka.lo), "s"(ka.hi), "s"(kb.lo), "s"(kb.hi));
    }
}

// Dynamic LDS of the row-sharing body below.
extern __shared__ __align__(16) uint32_t lds_cells[];

// Plain form: NG strategy groups x (waves / NG) budget sub-tiles per workgroup, every wave
// reads the rows it needs through the caches, twice (a first pass for the column minima, a
// second for the minimum over s'), and reduces every usable row.  It serves strategy counts
// beyond what one workgroup of the row-sharing body covers (several strategy-group blocks along
// grid.y).
template <int TS, int TE, int NG, class BP>
__device__ __forceinline__ void sweep_u32(const Layout &a, int wave, int l, int b, int budget,
                                          int64_t tile_start) {
    static_assert(TS <= 16, "one scalar load fetches the R keys of a row");
    const int lane = lane_id();
    const int g = wave % NG;
    const int esub = wave / NG;
    const int64_t e0 = tile_start + (int64_t)esub * (kWave * TE) + lane;
    const int64_t s0 = ((int64_t)blockIdx.y * NG + g) * TS;
    if (s0 >= a.S) return;
    if (tile_start + (int64_t)esub * (kWave * TE) > budget) return;      // wave-uniform

    const int64_t S = a.S;
    const int k = a.k_bits;
    const int64_t pitch = a.row * 2;               // 32-bit cells between the rows of two strategies
    const uint32_t *Up = reinterpret_cast<const uint32_t *>(a.U[(l - 1) & 1]) +
                         (int64_t)b * a.S_pad * pitch + a.lead + (e0 - lane);
    uint32_t *Un = reinterpret_cast<uint32_t *>(a.U[l & 1]) + ((int64_t)b * a.S_pad + s0) * pitch +
                   a.lead + e0;
    BP *bp = static_cast<BP *>(a.bp) + (((int64_t)b * (a.L - 1) + (l - 1)) * S + s0) * a.e_pad + e0;
    const int r = a.r_idx ? a.r_idx[(int64_t)b * a.L + l] : 0;
    const ConstPtr<uint32_t> Rk =
        as_const(reinterpret_cast<const uint32_t *>(a.Rk + ((int64_t)b * a.nR + r) * S * a.S_pad) + s0);
    const ConstPtr<uint64_t> ck = as_const(a.ck + ((int64_t)b * a.L + l) * a.S_pad + s0);
    const ConstPtr<uint64_t> vl = as_const(a.vlist + ((int64_t)b * a.L + (l - 1)) * a.S_pad);
    const int n = as_const(a.nvalid)[(int64_t)b * a.L + (l - 1)];
    const uint32_t dmax = as_const(a.dclamp)[b];

    uint32_t acc[TS][TE];
#pragma unroll
    for (int s = 0; s < TS; ++s)
#pragma unroll
        for (int j = 0; j < TE; ++j) acc[s][j] = 0xffffffffu;
    uint32_t cmin[TE];
#pragma unroll
    for (int j = 0; j < TE; ++j) cmin[j] = 0xffffffffu;

    auto cells = [&](int i) {            // shifted row of list entry i (clamped to the list)
        const uint64_t ent = vl[i < n ? i : n - 1];
        return Up + (int64_t)(uint32_t)ent * pitch - (int64_t)(ent >> 32);
    };

    if (s0 == 0 && esub == 0 && lane == 0) {       // statistics: this body reads and reduces every listed row
        uint32_t *st = a.stats + 2 * (((int64_t)b * (a.L - 1) + (l - 1)) * a.n_tiles +
                                      (uint32_t)tile_start / (uint32_t)a.tile_e);
        st[0] = (uint32_t)n << 16 | (uint32_t)n;
        st[1] = (uint32_t)n;
    }
    if (n > 0) {
        // Pass 1: the column minima of the former layer.  Pure loads: batches of kBatch list
        // entries, the next batch requested before the current one is reduced.
        constexpr int kBatch = GALV_P1_BATCH;
        uint32_t t[2][kBatch][TE];
        auto fetch = [&](int h, int i0) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const uint32_t *p = cells(i0 + u);
#pragma unroll
                for (int j = 0; j < TE; ++j) t[h][u][j] = p[(uint32_t)lane + j * kWave];
            }
        };
        auto fold = [&](int h) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
#pragma unroll
                for (int j = 0; j < TE; ++j) cmin[j] = min(cmin[j], t[h][u][j]);
        };
        fetch(0, 0);
        int i = 0;
        for (; i + 2 * kBatch < n; i += 2 * kBatch) {
            fetch(1, i + kBatch);
            fold(0);
            fetch(0, i + 2 * kBatch);
            fold(1);
        }
        if (i + kBatch < n) {
            fetch(1, i + kBatch);
            fold(0);
            fold(1);
        } else {
            fold(0);
        }

        // Pass 2: pairs of list entries.  The cells of the next pair and the R rows of the
        // next pair are requested before the current pair is reduced.
        const int npair = (n + 1) / 2;             // an odd tail repeats its entry: min(x, x) = x
        uint32_t va[2][TE], vb[2][TE];
        int spa[2], spb[2];
        R32Row<TS> ra[2], rb[2];
        auto request = [&](int q, int pr) {
            const int ia = 2 * pr < n ? 2 * pr : n - 1;
            const int ib = 2 * pr + 1 < n ? 2 * pr + 1 : n - 1;
            const uint64_t ea = vl[ia], eb = vl[ib];
            spa[q] = (int)(uint32_t)ea;
            spb[q] = (int)(uint32_t)eb;
            const uint32_t *pa = Up + (int64_t)(uint32_t)ea * pitch - (int64_t)(ea >> 32);
            const uint32_t *pb = Up + (int64_t)(uint32_t)eb * pitch - (int64_t)(eb >> 32);
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                va[q][j] = pa[(uint32_t)lane + j * kWave];
                vb[q][j] = pb[(uint32_t)lane + j * kWave];
            }
        };
        auto reduce_pair = [&](int q) {
            // keys of the next pair's rows, in flight under this pair's arithmetic
            ra[q ^ 1].request(Rk + (int64_t)spa[q ^ 1] * a.S_pad);
            rb[q ^ 1].request(Rk + (int64_t)spb[q ^ 1] * a.S_pad);
            uint32_t da[TE], db[TE];
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                da[j] = min(va[q][j] - cmin[j], dmax) << k;
                db[j] = min(vb[q][j] - cmin[j], dmax) << k;
            }
#pragma unroll
            for (int s = 0; s < TS; ++s)
                minplus_u32x2<TE>(acc[s], da, db, ra[q].at(s), rb[q].at(s), ra[q ^ 1], rb[q ^ 1]);
            r32_await(ra[q ^ 1], rb[q ^ 1]);
        };
        request(0, 0);
        request(1, 1);
        ra[0].request(Rk + (int64_t)spa[0] * a.S_pad);
        rb[0].request(Rk + (int64_t)spb[0] * a.S_pad);
        r32_await(ra[0], rb[0]);
        int pr = 0;
        for (; pr + 2 <= npair; pr += 2) {
            reduce_pair(0);
            request(0, pr + 2);
            reduce_pair(1);
            request(1, pr + 3);
        }
        if (pr < npair) reduce_pair(0);
    }

    const uint32_t mask = (1u << k) - 1u;
#pragma unroll
    for (int s = 0; s < TS; ++s) {
        if (s0 + s < S) {
            const uint32_t cs = (uint32_t)ck[s];
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                const bool alive = cmin[j] < kInf32;
                const uint32_t key = acc[s][j];
                Un[(int64_t)s * pitch + j * kWave] = alive ? cmin[j] + (key >> k) + cs : kInf32;
                // Back-pointers are written once and read again only by the backtrack: a
                // streaming store keeps them from pushing the cost rows, which the next
                // layer reads back, out of the caches.  (-1 becomes 0xFF in one byte.)
                __builtin_nontemporal_store((BP)(alive ? (int32_t)(key & mask) : -1),
                                            &bp[(int64_t)s * a.e_pad + j * kWave]);
            }
        }
    }
}

// How many surviving rows the row-sharing body below keeps in LDS for a workgroup that covers
// `cap` strategies (host and device agree through this one function).
// As many as the LDS holds without costing a resident workgroup: a CU holds wpe * 4 / ng
// workgroups by registers, each may take that share of the 160 KB (at most 128 KB); what the
// partial minima and counters leave goes to the list, in whole rows per wave and pass.  With
// 128-column tiles 8, 11, 16, 22, 32, 48, 96 and 224 rows for the eight variants below; with
// 256-column tiles 12, 16, 24, 32, 64 and 96.
constexpr int keep_rows(int ts, int ng, int wpe, int cols) {       // cols: budget columns of a tile
    const int wgs = wpe * 4 / ng > 0 ? wpe * 4 / ng : 1;
    const int share = 160 * 1024 / wgs < 128 * 1024 ? 160 * 1024 / wgs : 128 * 1024;
    const int fixed = ng * cols * 4 + ng * 8 + 16 + 256;
    int rows = (share - fixed) / (cols * 4 + 4);
    if (rows > ts * ng) rows = ts * ng;
    rows -= rows % ng;
    return rows < ng ? ng : rows;
}

// Row-sharing form of the 32-bit-key body, for S <= TS * NG (up to 256) with one budget tile of
// 64 * TE columns per workgroup of NG waves.  Wave g owns the former-layer rows g, g + NG, ...
// (TS of them, in registers) AND the strategy group g of the output.
//   1. Every wave loads its rows once (shifted, coalesced) and reduces them to partial column
//      minima; the partial minima meet in LDS (one barrier).
//   2. With the column minimum known, a wave tests each of its rows: a row whose relative cost
//      is clamped (>= dmax = R_max + 1) in every reachable column of the tile can neither win nor
//      tie any minimum of the tile (the strategy that attains the column minimum offers at most
//      Cmin + R_max) and is dropped.  The other rows are appended, as ready keys, to a short
//      list in LDS together with their strategy index (second barrier).  The order of the list
//      is whatever the appends make it: the minimum does not depend on it, and the lowest-index
//      tie-break rides in the low bits of the keys.
//   3. The inner loop runs over the surviving rows only, reading keys from LDS and R keys by
//      scalar loads.  Should more rows survive than the list holds (transition costs that dwarf
//      the spread of the layer costs), the rows go through the list in passes, a few rows of
//      every wave at a time: each wave reads its rows of the pass again, appends the live ones,
//      and every wave reduces that list.
// Only the survivors' keys live in LDS, as many rows as fit without costing a resident workgroup
// (keep_rows), which is what lets three 8-wave workgroups share a CU at S = 128.
template <int TS, int TE, int NG, class BP, class Cell, int KEEP>
__device__ __forceinline__ void sweep_u32_shared(const Layout &a, int g, int l, int b, int budget,
                                                 int64_t tile_start, bool add_stats, int n, uint32_t dmax,
                                                 int r_sel, uint64_t my_ent, uint64_t my_c0_64) {
    // n, dmax, r_sel: the former layer's usable strategies, the clamp and the layer's transition
    // matrix, from the header record.  my_ent, my_c0_64: lane r (and lane 32 + r) holds the list
    // entry of this wave's row g + NG * r and that strategy's c(l-1, s'), which made-up
    // cells hold; the kernel requests them before it knows anything else (their addresses
    // depend on the workgroup's position only), so that they arrive together with the header.
    // Fetched as scalars where they are used, one row at a time, they form a chain of dependent
    // round trips (entry, then c, then the cells) that costs more than everything else a tile
    // does.  Rows that turn out to be needed get their entry broadcast from its lane.
    // Cell: uint32_t (costs below 2^31, infinity = 2^31) or uint64_t (any cost up to the 2^62
    // precondition, infinity = 2^62).  Only RELATIVE costs enter the 32-bit keys, so the wide form
    // runs the same arithmetic and the same pruning; it moves 8-byte cells.
    constexpr bool kWide = sizeof(Cell) == 8;
    constexpr Cell kInfCell = kWide ? (Cell)kInf : (Cell)kInf32;
    constexpr Cell kAllOnes = ~(Cell)0;
    static_assert(TS <= 16, "one scalar load fetches the R keys of a row");
    constexpr int kCols = kWave * TE;
    constexpr int kKeep = KEEP;                    // rows the list holds (keep_rows of the variant)
    (void)budget;
    // A wave that has loads to issue goes before the waves that are in their arithmetic: the sooner a
    // tile's requests are out, the shorter its chain of round trips, and the arithmetic of the other
    // waves fills the time the requests take either way.  (Priority drops again before the inner loop.)
    __builtin_amdgcn_s_setprio(3);
    const int lane = lane_id();                    // (g: the wave = owner of rows g + NG * r = strategy group)
    const int64_t e0 = tile_start + lane;
    const int64_t s0 = (int64_t)g * TS;

    const int64_t S = a.S;
    const int k = a.k_bits;
    const int64_t pitch = a.row * (8 / (int64_t)sizeof(Cell));   // cells between the rows of two strategies
    const Cell *Up = reinterpret_cast<const Cell *>(a.U[(l - 1) & 1]) +
                     (int64_t)b * a.S_pad * pitch + a.lead + tile_start;
    // (wave-uniform: the first column of the tile in this wave's first output row)
    Cell *Un_tile = reinterpret_cast<Cell *>(a.U[l & 1]) + ((int64_t)b * a.S_pad + s0) * pitch +
                    a.lead + tile_start;
    BP *bp_tile = static_cast<BP *>(a.bp) + (((int64_t)b * (a.L - 1) + (l - 1)) * S + s0) * a.e_pad + tile_start;
    const ConstPtr<uint32_t> Rk =
        as_const(reinterpret_cast<const uint32_t *>(a.Rk + ((int64_t)b * a.nR + r_sel) * S * a.S_pad) + s0);
    const ConstPtr<uint64_t> ck = as_const(a.ck + ((int64_t)b * a.L + l) * a.S_pad + s0);
    const Cell my_c0 = (Cell)my_c0_64;

    // The shifted cells of one usable former strategy for this lane's columns.  Layer 0's table
    // is a constant per strategy, U_0[e'][s'] = c(0, s'), so when layer 1 is swept its cells are
    // made up here (infinity below the shift) instead of being read.
    const bool first = l == 1;                     // uniform
    // (cp = c(l-1, s'): what a made-up cell holds; unused for stored cells)
    auto load_row = [&](uint64_t ent, Cell cp, Cell (&out)[TE]) {
        const uint32_t sp = (uint32_t)ent, shift = (uint32_t)(ent >> 32);
        if (first) {
#pragma unroll
            for (int j = 0; j < TE; ++j) out[j] = e0 + j * kWave >= (int64_t)shift ? cp : kInfCell;
        } else {
            const Cell *p = Up + (int64_t)sp * pitch - (int64_t)shift;
#pragma unroll
            for (int j = 0; j < TE; ++j) out[j] = p[(uint32_t)lane + j * kWave];
        }
    };

    Cell *part = reinterpret_cast<Cell *>(lds_cells);               // [NG][kCols] partial column minima
    Cell *wave_min = part + NG * kCols;                             // [NG] the waves' minima of the peek
    uint32_t *count = reinterpret_cast<uint32_t *>(wave_min + NG);  // [0] surviving rows, [2] rows fetched
    uint32_t *meta = count + 4;                    // [kKeep] strategy index of a kept row
    uint32_t *keys = meta + kKeep;                 // [kKeep][kCols] its keys

    uint32_t acc[TS][TE];
#pragma unroll
    for (int s = 0; s < TS; ++s)
#pragma unroll
        for (int j = 0; j < TE; ++j) acc[s][j] = 0xffffffffu;
    Cell cmin[TE];
#pragma unroll
    for (int j = 0; j < TE; ++j) cmin[j] = kAllOnes;

    if (g == 0 && lane == 0) count[0] = 0;

    // Peek.  Every stored row is non-increasing along the budget axis (more memory never costs
    // more), so a row's cells in this tile are at least its cell in the tile's last column, and
    // every column minimum of the tile is at most Cmin_before = the minimum over the rows' cells
    // in the column just BEFORE the tile.  A row whose last-column cell is at least
    // Cmin_before + dmax is therefore clamped in every column of the tile and need not be read at
    // all: two cells per row decide whether its 64 * TE cells are fetched.  (The column before the
    // tile rather than its first column: that is the last column of the neighbouring tile, whose
    // workgroup probes the same cell, so the two probes meet in the L2.)  The row that attains a
    // column's minimum always passes (its cell there is at most Cmin_before), so the minima over
    // the rows that are read are the true column minima.
    uint32_t keep = 0;                             // bit r: row g + NG * r is read (wave-uniform)
    if (n > 0 && !a.peek) {
        // (a launch that does not fill the chip is bound by latency, not by bytes: there the two
        // extra dependent steps of the peek cost more than the rows it saves)
#pragma unroll
        for (int r = 0; r < TS; ++r)
            if (g + NG * r < n) keep |= 1u << r;
        if (g == 0 && lane == 0) count[2] = (uint32_t)n;
    }
    if (n > 0 && a.peek) {
        // One gather for the whole wave: lane r (r < TS) fetches row r's cell in the column before
        // the tile (below the shift: infinity), lane 32 + r its cell in the tile's last column.
        Cell first_min = kAllOnes;
        const bool my_last = lane >= 32;
        const uint32_t my_sp = (uint32_t)my_ent, my_shift = (uint32_t)(my_ent >> 32);
        Cell mine;
        const int64_t idx = tile_start + (my_last ? kCols - 1 : -1) - (int64_t)my_shift;
        if (first) {
            mine = idx < 0 ? kInfCell : my_c0;     // this lane's column lies below the row's shift
        } else {
            mine = Up[(int64_t)my_sp * pitch + (idx - tile_start)];   // (the lead holds infinity below the shift)
        }
#pragma unroll
        for (int r = 0; r < TS; ++r) first_min = min(first_min, read_lane(mine, r));
        uint32_t *peek = count + 2;                // rows fetched by the workgroup
        if (lane == 0) wave_min[g] = first_min;
        if (g == 0 && lane == 0) peek[0] = 0;
        __syncthreads();
        Cell cmin_first = kAllOnes;
#pragma unroll
        for (int w = 0; w < NG; ++w) cmin_first = min(cmin_first, read_lane(wave_min[w], 0));
        // an unreachable column before the tile (Cmin_before = infinity) bounds nothing: read every row
        const Cell limit = cmin_first < kInfCell ? cmin_first + (Cell)dmax : kAllOnes;
        // lane 32 + r holds row r's last-column cell and votes for its row
        const bool my_keep = my_last && lane - 32 < TS && g + NG * (lane - 32) < n && mine < limit;
        keep = (uint32_t)(__builtin_amdgcn_ballot_w64(my_keep) >> 32);
        const int mine_read = __builtin_popcount(keep);
        if (lane == 0 && mine_read) atomicAdd(&peek[0], (uint32_t)mine_read);
    }

    Cell rowc[TS][TE];
    if (n > 0) {                                   // workgroup-uniform
        Cell pm[TE];
#pragma unroll
        for (int j = 0; j < TE; ++j) pm[j] = kAllOnes;
#pragma unroll
        for (int r = 0; r < TS; ++r) {
            if (keep >> r & 1) {
                load_row(read_lane(my_ent, r), read_lane(my_c0, r), rowc[r]);
            } else {
#pragma unroll
                for (int j = 0; j < TE; ++j) rowc[r][j] = kAllOnes;          // leaves every minimum alone
            }
        }
#pragma unroll
        for (int r = 0; r < TS; ++r)
#pragma unroll
            for (int j = 0; j < TE; ++j) pm[j] = min(pm[j], rowc[r][j]);     // a repeated row changes nothing
#pragma unroll
        for (int j = 0; j < TE; ++j) part[g * kCols + j * kWave + lane] = pm[j];
    }
    __syncthreads();
    // With the column minimum known, a row's relative costs, clamped: all that its keys need.  A
    // row that is clamped in every reachable column of the tile is dropped; the others go on the
    // list (keys and strategy index), at the slot `counter` hands out.
    auto append_row = [&](int r, const Cell (&cells)[TE], uint32_t *counter) {
        uint32_t d[TE];
        bool live = false;
#pragma unroll
        for (int j = 0; j < TE; ++j) {
            const Cell rel = cells[j] - cmin[j];
            d[j] = (uint32_t)min(rel, (Cell)dmax);
            live |= rel < (Cell)dmax && cmin[j] < kInfCell;
        }
        if (__builtin_amdgcn_ballot_w64(live) != 0) {        // wave-uniform
            uint32_t slot = 0;
            if (lane == 0) slot = atomicAdd(counter, 1u);
            slot = (uint32_t)uniform((int)slot);
            if (slot < (uint32_t)kKeep) {
#pragma unroll
                for (int j = 0; j < TE; ++j) keys[slot * kCols + j * kWave + lane] = d[j] << k;
                // (broadcast with every lane active, not under the test for lane 0: a register
                // reloaded from a spill there holds lane 0's value only)
                const uint32_t sp_r = (uint32_t)read_lane(my_ent, r);
                if (lane == 0) meta[slot] = sp_r;
            }
        }
    };
    if (n > 0) {
#pragma unroll
        for (int w = 0; w < NG; ++w)
#pragma unroll
            for (int j = 0; j < TE; ++j) cmin[j] = min(cmin[j], part[w * kCols + j * kWave + lane]);
#pragma unroll
        for (int r = 0; r < TS; ++r)
            if (keep >> r & 1) append_row(r, rowc[r], count);   // listed (the padding repeats a listed row) and read
        if (g == 0 && lane == 0) count[1] = 0;     // the counter of the pass after this one
    }
    __syncthreads();

    // The list holds the rows that matter, or it has overflowed (transition costs that dwarf the
    // spread of the layer costs: few rows are clamped everywhere).  Then the rows go through the
    // list in passes, kRpw rows of every wave at a time, which always fit: each wave reads its
    // own rows of the pass again (once per workgroup, not once per wave), appends the live ones,
    // and every wave reduces that list.  Three counters take turns, so that the one a pass uses
    // was cleared while the pass before it was under way and after its last reader had gone.
    constexpr int kRpw = kKeep / NG;
    static_assert(kRpw >= 1, "one pass holds at least one row of every wave");
    __builtin_amdgcn_s_setprio(0);                 // from here on arithmetic: let the waves that fetch go first
    int cnt = n > 0 ? uniform((int)count[0]) : 0;
    int r_next = TS;                               // first row of the next pass; TS: no further pass
    if (cnt > kKeep) {
        r_next = 0;
        cnt = -1;                                  // nothing to reduce yet
    }
    uint32_t rows_reduced = 0;
    int pass = 0;
    for (;;) {
        if (cnt < 0) {                             // workgroup-uniform
            ++pass;
            uint32_t *counter = count + (pass % 3 == 2 ? 3 : pass % 3);
            if (g == 0 && lane == 0) count[(pass + 1) % 3 == 2 ? 3 : (pass + 1) % 3] = 0;
#pragma unroll
            for (int r = 0; r < TS; ++r)
                if (r >= r_next && r < r_next + kRpw && (keep >> r & 1)) {
                    Cell cells[TE];
                    load_row(read_lane(my_ent, r), read_lane(my_c0, r), cells);
                    append_row(r, cells, counter);
                }
            __syncthreads();
            cnt = uniform((int)counter[0]);        // at most NG * kRpw = kKeep
            r_next += kRpw;
        }
        rows_reduced += (uint32_t)cnt;
        if (s0 < S && cnt > 0) {                   // (an idle strategy group only contributes its rows)
            const int npair = (cnt + 1) / 2;       // an odd tail repeats its entry: min(x, x) = x
            uint32_t va[2][TE], vb[2][TE];
            int spa[2], spb[2];
            R32Row<TS> ra[2], rb[2];
            auto request = [&](int q, int pr) {
                const int ia = 2 * pr < cnt ? 2 * pr : cnt - 1;
                const int ib = 2 * pr + 1 < cnt ? 2 * pr + 1 : cnt - 1;
                spa[q] = uniform((int)meta[ia]);
                spb[q] = uniform((int)meta[ib]);
#pragma unroll
                for (int j = 0; j < TE; ++j) {
                    va[q][j] = keys[ia * kCols + j * kWave + lane];
                    vb[q][j] = keys[ib * kCols + j * kWave + lane];
                }
            };
            auto reduce_pair = [&](int q) {
                // keys of the next pair's rows, in flight under this pair's arithmetic
                ra[q ^ 1].request(Rk + (int64_t)uniform(spa[q ^ 1]) * a.S_pad);
                rb[q ^ 1].request(Rk + (int64_t)uniform(spb[q ^ 1]) * a.S_pad);
#pragma unroll
                for (int s = 0; s < TS; ++s)
                    minplus_u32x2<TE>(acc[s], va[q], vb[q], ra[q].at(s), rb[q].at(s), ra[q ^ 1], rb[q ^ 1]);
                r32_await(ra[q ^ 1], rb[q ^ 1]);
            };
            request(0, 0);
            request(1, 1);
            ra[0].request(Rk + (int64_t)uniform(spa[0]) * a.S_pad);
            rb[0].request(Rk + (int64_t)uniform(spb[0]) * a.S_pad);
            r32_await(ra[0], rb[0]);
            int pr = 0;
            for (; pr + 2 <= npair; pr += 2) {
                reduce_pair(0);
                request(0, pr + 2);
                reduce_pair(1);
                request(1, pr + 3);
            }
            if (pr < npair) reduce_pair(0);
        }
        if (r_next >= TS) break;
        __syncthreads();                           // the list is free again
        cnt = -1;
    }
    if (g == 0 && lane == 0) {                     // statistics: how much the pruning removed
        uint32_t *st = a.stats + 2 * (((int64_t)b * (a.L - 1) + (l - 1)) * a.n_tiles +
                                      (uint32_t)tile_start / (uint32_t)a.tile_e);
        const uint32_t rows = rows_reduced << 16 | (uint32_t)n;
        const uint32_t fetched = n > 0 ? count[2] : 0u;
        st[0] = add_stats ? st[0] + rows : rows;   // (a tile swept in several parts adds them up)
        st[1] = add_stats ? st[1] + fetched : fetched;
    }
    if (s0 >= S) return;                           // an idle strategy group has done its share of the rows

    const uint32_t mask = (1u << k) - 1u;
#pragma unroll
    for (int s = 0; s < TS; ++s) {
        if (s0 + s < S) {
            const Cell cs = (Cell)ck[s];
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                const bool alive = cmin[j] < kInfCell;
                const uint32_t key = acc[s][j];
                // (wave-uniform row address + the lane's offset: no per-store address arithmetic)
                BP *bp_row = bp_tile + (int64_t)s * a.e_pad;
                Cell *un_row = Un_tile + (int64_t)s * pitch;
                un_row[(uint32_t)lane + j * kWave] = alive ? cmin[j] + (Cell)(key >> k) + cs : kInfCell;
                __builtin_nontemporal_store((BP)(alive ? (int32_t)(key & mask) : -1),
                                            &bp_row[(uint32_t)lane + j * kWave]);
            }
        }
    }
}

// UX: the 32-bit-key body keeps half-size accumulators, so it may take UX (1 or 2) times
// the budget columns per lane; the 64-bit-key bodies then cover the same tile in UX steps.
template <int TS, int TE, int NG, int WPE, class BP, int W, int UX, int SHARE>
__global__ __launch_bounds__(W * kWave, WPE) void sweep_kernel(Layout a, int l) {
    const int wave = uniform(threadIdx.x >> 6);    // the only use of the thread-index register (see lane_id)
    const int b = a.b_off + blockIdx.z * a.b_step;
    // The row-sharing body's list entries (see there): requested first, ahead of the header.
    uint64_t my_ent = 0, my_c0 = 0;
    if constexpr (SHARE != 0) {
        const int lane = lane_id();
        const int my_row = (lane & 31) < TS ? (lane & 31) : TS - 1;      // (idle lanes repeat the last row)
        const int64_t at = ((int64_t)b * a.L + (l - 1)) * a.S_pad + wave + NG * my_row;
        my_ent = a.vlist[at];
        my_c0 = a.vcost[at];
    }
    // One record holds what the workgroup needs to begin with.
    const ConstPtr<int32_t> hdr = as_const(a.hdr + ((int64_t)b * a.L + l) * 8);
    const int st = hdr[0];
    const int budget = hdr[1];
    const int n_prev = hdr[2];
    const uint32_t dmax = (uint32_t)hdr[3];
    const int r_sel = hdr[4];
    (void)n_prev, (void)dmax, (void)r_sel, (void)my_ent, (void)my_c0;
    if (st < 0) return;
#if GALV_XCD_MAP
    // Workgroups go round-robin to the 8 XCDs in the order of their linear index, and grid.x is
    // a multiple of 8, so blockIdx.x & 7 names the XCD.  Each XCD takes a contiguous eighth of
    // the tiles the instance needs: neighbouring tiles read overlapping cache lines of the
    // shifted former-layer rows, which then meet in one XCD's L2.
    const int nt = budget / a.tile_e + 1;
    const int per = (nt + 7) >> 3;
    if ((int)(blockIdx.x >> 3) >= per) return;
    const int64_t tile_start = (int64_t)((blockIdx.x & 7) * per + (blockIdx.x >> 3)) * a.tile_e;
#else
    const int64_t tile_start = (int64_t)blockIdx.x * a.tile_e;
#endif
    if (tile_start > budget) return;
    if (st == GALV_INSTANCE_OK_FAST_U32) {
        if constexpr (SHARE)
            sweep_u32_shared<TS, TE * UX, NG, BP, uint32_t, keep_rows(TS, NG, WPE, kWave * TE * UX)>(a, wave, l, b, budget, tile_start, false, n_prev, dmax, r_sel, my_ent, my_c0);
        else
            sweep_u32<TS, TE * UX, NG, BP>(a, wave, l, b, budget, tile_start);
    } else if (st == GALV_INSTANCE_OK_U32_WIDE) {
        // 8-byte cells: half the tile's columns at a time keep the rows within the registers the narrow
        // form uses (the preparation kernel grants this path to row-sharing variants only)
        if constexpr (SHARE) {
            for (int h = 0; h < TE; ++h) {
                if (tile_start + h * (kWave * UX) > budget) break;   // workgroup-uniform
                if (h) __syncthreads();                              // the LDS of the part before is free again
                sweep_u32_shared<TS, UX, NG, BP, uint64_t, keep_rows(TS, NG, WPE, kWave * TE * UX)>(a, wave, l, b, budget, tile_start + h * (kWave * UX), h > 0, n_prev, dmax, r_sel, my_ent, my_c0);
            }
        }
    } else if (st == GALV_INSTANCE_OK_FAST) {
        for (int h = 0; h < UX; ++h)
            sweep_fast<TS, TE, NG, Narrow, BP>(a, wave, l, b, budget, tile_start + h * (a.tile_e / UX));
    } else if (st == GALV_INSTANCE_OK_FAST_WIDE) {
        for (int h = 0; h < UX; ++h)
            sweep_fast<TS, TE, NG, Wide, BP>(a, wave, l, b, budget, tile_start + h * (a.tile_e / UX));
    } else {
        if (blockIdx.y == 0) sweep_int64<8>(a, wave, l, b, budget, tile_start);
    }
}

// ------------------------------------------------------------ byte-table sweep
//
// The packed form of the pruning sweep, for handles whose layers have many tiles.  There the
// sweep is bound by what it writes and by its chain of round trips, so it keeps little per state:
//   * the argmin, one byte: the only table that lives on after the next layer;
//   * and, per budget column, the former minimum Cmin and the clamped relative costs
//     rel(s') = C[l-1][e'][s'] - Cmin of those former strategies that are alive in the tile (a few
//     of S when the pruning bites).
// That is enough to rebuild any cell, because its argmin is always one of the alive strategies:
//     U_l[e'][s] = Cmin_l[e'] + rel_l(s')[e'] + R_l(s', s) + c(l, s)   with s' = argmin byte.
// The next layer fetches few rows, so rebuilding them (two dependent loads) costs less than
// writing every cell: 1 byte + 4 bytes x (share of rows alive) are written per state, where a
// 32-bit key per state was 4.  A lane owns TE consecutive columns, so the bytes of a row leave as
// one word per lane.  For the peek, absolute costs of every 64th column are kept too ("samples",
// 1/16 byte per state): rows are non-increasing along the budget axis, so the sample at or after a
// tile's last column bounds the row's cells in the tile from below and the one at or before the
// column in front of the tile bounds every column minimum of the tile from above, in one load each.
//
// Only the columns [Y_l, X_l] of layer l are swept and stored:
//   * below Y_l = sum of the smallest memories of the layers before l nothing is reachable;
//   * from X_l = max_s (memory of the best plan without any memory limit that ends in s) on, every
//     row is constant, costs and argmins alike: the unlimited optimum fits, no column offers a
//     candidate below it, and the lowest-index minimiser is the same.  Readers clamp to X_l.
//     (And columns beyond budget - min_s m(l, s) are read by nobody.)
// 55-65 % of the columns of 22 strategies x 32-48 layers fall away, 35-40 % of 44 x 96, 16 % of
// 128 x 128.  live_step() runs the unlimited recurrence one layer ahead of the sweep.
//
// Measured, before (a 32-bit key per state, all columns, 2 / 6 / 16 streams) and after (1 / 2 / 2), whole
// solves: 22 strategies x 24576 columns x 48 layers x 32 instances 1.30 -> 0.82 ms, 44 x 32768 x 96 x 64
// (budgets of a quarter up) 6.7 -> 3.6 ms, 128 x 65536 x 128 x 16 20.7 -> 12.4 ms.
struct PackTables {                                // of one instance, in the space of the cost rows
    uint32_t *rel;                                 // [S_pad][e_pad]
    char *cost;                                    // samples [S_pad][e_pad / 64] of Cell
    char *cmin;                                    // [e_pad] of Cell
    uint64_t *V;                                   // [S_pad] unlimited optimum ending in s
    int32_t *mem;                                  // [S_pad] its memory in the layers before
};
__device__ __forceinline__ PackTables pack_tables(const Layout &a, int parity, int b) {
    char *base = a.U[parity] + (int64_t)b * a.S_pad * a.row * 8;
    PackTables t;
    t.rel = reinterpret_cast<uint32_t *>(base);
    t.cost = base + (int64_t)a.S_pad * a.e_pad * 4;
    t.cmin = t.cost + (int64_t)a.S_pad * (a.e_pad / kSample) * 8;
    t.V = reinterpret_cast<uint64_t *>(t.cmin + a.e_pad * 8);
    t.mem = reinterpret_cast<int32_t *>(t.V + a.S_pad);
    return t;                                      // (rows reserve 8 bytes per column, leads included: ample)
}
template <class T>
__device__ __forceinline__ const T *rkeys(const Layout &a, int b, int r) {
    return reinterpret_cast<const T *>(a.Rk + ((int64_t)b * a.nR + r) * a.S * a.S_pad);
}

// The two kinds of keys, (relative cost + R) * 2^k + s': 32-bit words where twice the largest
// relative cost fits them, else whole numbers below 2^42 held in doubles (the add and the minimum
// of doubles run at the same rate as two 32-bit ones, and there is no 64-bit integer minimum).
// Costs outgrow the 32-bit key with the unit of time: 44 strategies and transitions of 0.1 s,
// counted in nanoseconds.  Over cost rows such instances take every candidate of every column: 44
// strategies x 16384 columns x 48 layers x 16 instances 3.06 ms, and with the byte table 1.27 ms.
struct Key32 {
    using T = uint32_t;
    using Rel = uint32_t;      // a relative cost
    using Stored = uint32_t;   // and how the chained sweep keeps it: as it is
    static constexpr bool kKeysInLds = true;       // chained sweep: the transition keys are kept there
    static __device__ __forceinline__ Stored stored(Rel rel, int) { return rel; }
    static __device__ __forceinline__ T from(Stored rel, int k) { return make(rel, k); }
    static __device__ __forceinline__ T none() { return 0xffffffffu; }
    static __device__ __forceinline__ T make(uint32_t rel, int k) { return rel << k; }
    static __device__ __forceinline__ uint32_t low(T key) { return key; }
    static __device__ __forceinline__ uint64_t cost(T key, int k) { return key >> k; }
    static __device__ __forceinline__ T least(T x, T y) { return min(x, y); }
};
struct Key64 {
    using T = double;
    using Rel = uint32_t;
    using Stored = uint32_t;
    static constexpr bool kKeysInLds = true;
    static __device__ __forceinline__ Stored stored(Rel rel, int) { return rel; }
    static __device__ __forceinline__ T from(Stored rel, int k) { return make(rel, k); }
    static __device__ __forceinline__ T none() { return 0x1p51; }
    static __device__ __forceinline__ T make(uint32_t rel, int k) { return __builtin_ldexp((double)rel, k); }
    static __device__ __forceinline__ uint64_t bits(T key) {     // (below 2^52: the sum's mantissa is the number)
        return (uint64_t)__double_as_longlong(key + 0x1p52) & 0x000fffffffffffffull;
    }
    static __device__ __forceinline__ uint32_t low(T key) { return (uint32_t)bits(key); }
    static __device__ __forceinline__ uint64_t cost(T key, int k) { return bits(key) >> k; }
    static __device__ __forceinline__ T least(T x, T y) { return __builtin_fmin(x, y); }
};
// The same with relative costs of 64 bits, for transition costs of 2^32 - 1 and more (chained sweep only).  The clamp is at most
// the largest plan cost + 1, so a clamped key is at most 2^52 and with a transition cost 2^53; a minimum is below 2^52.  (The keys
// themselves are kept, as bits; they take the room that the transition keys have in LDS otherwise.)
struct KeyBig {
    using T = double;
    using Rel = uint64_t;
    using Stored = uint64_t;
    static constexpr bool kKeysInLds = false;
    static __device__ __forceinline__ T none() { return INFINITY; }
    static __device__ __forceinline__ Stored stored(Rel rel, int k) {
        return (uint64_t)__double_as_longlong(__longlong_as_double((long long)(kBias + (rel << k))) - 0x1p52);
    }
    static __device__ __forceinline__ T from(Stored key, int) { return __longlong_as_double((long long)key); }
    static __device__ __forceinline__ uint32_t low(T key) { return Key64::low(key); }
    static __device__ __forceinline__ uint64_t cost(T key, int k) { return Key64::cost(key, k); }
    static __device__ __forceinline__ T least(T x, T y) { return __builtin_fmin(x, y); }
};

// One step of the recurrence without a memory limit, for layer l of instance b: V_l(s) and the
// memory its plan takes before layer l, from those of layer l - 1; then (tell) the last column of
// layer l that has to be swept.  Same keys, same tie-break as the sweep.  One workgroup; S <= 16 * NG.
template <int NG, class Key>
__device__ __forceinline__ void live_step(const Layout &a, int wave, int b, int l, bool tell) {
    int32_t *h = a.hdr + ((int64_t)b * a.L + l) * 8;
    const int lane = lane_id(), tid = wave * kWave + lane;
    const int S = a.S, k = a.k_bits;
    const int budget = h[1], n = h[2];
    const uint32_t dmax = (uint32_t)h[3];
    const PackTables from = pack_tables(a, (l - 1) & 1, b), to = pack_tables(a, l & 1, b);
    const uint64_t *list = a.vlist + ((int64_t)b * a.L + (l - 1)) * a.S_pad;
    const uint64_t *lcost = a.vcost + ((int64_t)b * a.L + (l - 1)) * a.S_pad;
    using KeyT = typename Key::T;
    KeyT *part = reinterpret_cast<KeyT *>(lds_cells);               // [NG][S_pad]
    uint32_t *dv = reinterpret_cast<uint32_t *>(part + NG * a.S_pad), *sp = dv + a.S_pad, *mem = sp + a.S_pad;
    uint32_t *top = mem + a.S_pad;
    if (n == 0) {                                  // nothing reachable from here on
        if (tid == 0 && tell) h[6] = -1;
        return;
    }
    // (list entry i belongs to thread i of every wave's view: each wave takes the minimum itself)
    uint64_t vmin = ~0ull;
    for (int i = lane; i < n; i += kWave) {
        const uint32_t s = (uint32_t)list[i];
        const uint64_t v = l == 1 ? lcost[i] : from.V[s];
        vmin = v < vmin ? v : vmin;
    }
    vmin = wave_min(vmin);
    if (tid < n) {
        const uint64_t ent = list[tid];
        const uint32_t s = (uint32_t)ent;
        const uint64_t rel = (l == 1 ? lcost[tid] : from.V[s]) - vmin;
        dv[tid] = rel < dmax ? (uint32_t)rel : dmax;
        sp[tid] = s;
        // (memories saturate just above the budget)
        const int64_t x = (int64_t)(l == 1 ? 0 : from.mem[s]) + (int64_t)(ent >> 32);
        mem[s] = (uint32_t)(x <= budget ? x : (int64_t)budget + 1);
    }
    if (tid == 0) *top = 0;
    __syncthreads();
    const KeyT *Rk = rkeys<KeyT>(a, b, h[4]);
    constexpr int kQ = (16 * NG + kWave - 1) / kWave;
    KeyT best[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) best[q] = Key::none();
#pragma unroll 4
    for (int i = wave; i < n; i += NG) {
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
            const int s = q * kWave + lane;
            const KeyT key = Key::make(dv[i], k) + Rk[(int64_t)sp[i] * a.S_pad + (s < S ? s : S - 1)];
            best[q] = key < best[q] ? key : best[q];
        }
    }
#pragma unroll
    for (int q = 0; q < kQ; ++q)
        if (q * kWave + lane < S) part[wave * a.S_pad + q * kWave + lane] = best[q];
    __syncthreads();
    if (tid < S) {
        KeyT key = Key::none();
        for (int w = 0; w < NG && w < n; ++w) {
            const KeyT o = part[w * a.S_pad + tid];
            key = o < key ? o : key;
        }
        const uint32_t x = mem[Key::low(key) & ((1u << k) - 1u)];
        to.V[tid] = vmin + Key::cost(key, k) + (uint64_t)a.c[((int64_t)b * a.L + l) * S + tid];
        to.mem[tid] = (int32_t)x;
        if (a.m[((int64_t)b * a.L + l) * S + tid] <= budget) atomicMax(top, x);
    }
    __syncthreads();
    if (tid == 0 && tell) {
        const int64_t fits = (int64_t)budget - h[7];         // beyond it nobody reads layer l
        h[6] = (int32_t)((int64_t)*top < fits ? (int64_t)*top : fits);
    }
}

// Rows of cells a tile keeps in LDS, out of a resident workgroup's share of the 160 KB.
constexpr int byte_keep_rows(int ts, int ng, int wpe, int cols) {
    const int wgs = wpe * 4 / ng > 0 ? wpe * 4 / ng : 1;
    const int share = 160 * 1024 / wgs < 128 * 1024 ? 160 * 1024 / wgs : 128 * 1024;
    int rows = (share - ng * cols * 4 - ts * ng * 16 - 512) / (cols * 4 + 4);
    if (rows > ts * ng) rows = ts * ng;
    rows -= rows % ng;
    return rows < ng ? ng : rows;
}
constexpr unsigned byte_lds(int ts, int ng, int wpe, int cols) {
    // (the two halves of an overfull tile take no more: half the columns, and twice the rows of half the size)
    const int keep = byte_keep_rows(ts, ng, wpe, cols);
    const unsigned tile = (unsigned)(ng * cols * 4 + keep * cols * 4 + ts * ng * 16 + keep * 4 + 16);
    const unsigned live = (unsigned)((3 + 2 * ng) * ts * ng * 4 + 4);   // live_step
    return tile > live ? tile : live;
}

// How a part of a tile enters the tile's statistics: alone, added to the part before, or, for the second half of
// an overfull tile, which otherwise counts as one, as the mean of the two.
enum PartStats { kSetStats, kAddStats, kMeanStats };

// What a tile needs to know of its layer and of the former one.
struct TileHdr {
    int n;                                         // usable strategies of the former layer
    uint32_t dmax;
    int r, r_prev;                                 // transition matrices of this layer and of the former
    int y_prev, x_prev;                            // reachable from / stored up to, former layer
};

// The kernel's Layout argument, read again from the argument segment: pointers derived from this
// copy are computed where they are used.  (Derived once at the top they would outlive the
// min-plus loop, whose transition keys take 64 of the scalar registers, and be spilled around it.)
__device__ __forceinline__ const Layout &layout_again() {
    ConstPtr<Layout> p = (ConstPtr<Layout>)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const Layout *)p;
}

// What rebuilding the former layer's cells takes.
template <class Cell, class Key>
struct Former {
    const uint8_t *bp;
    const Cell *cmin;
    const uint32_t *rel;
    const typename Key::T *R;
    int64_t e_pad;
    int S_pad, k;
    __device__ __forceinline__ Former(const Layout &a, int b, int l, int r) {
        const PackTables t = pack_tables(a, (l - 1) & 1, b);
        bp = byte_rows(a, b, l == 1 ? 1 : l - 1);
        cmin = reinterpret_cast<const Cell *>(t.cmin);
        rel = t.rel;
        R = rkeys<typename Key::T>(a, b, r);
        e_pad = a.e_pad;
        S_pad = a.S_pad;
        k = a.k_bits;
    }
};

// Returns true when the tile has been swept.  With MAY_REFUSE a tile that keeps more rows than the list
// holds is left untouched instead (all waves agree; nothing but LDS has been written).
template <int TS, int TE, int NG, class Cell, class Key, int KEEP, int TILE, bool MAY_REFUSE = false>
__device__ __forceinline__ bool sweep_bytes(const Layout &a, int g, int l, int b, int tile_start, PartStats part_stats,
                                            const TileHdr &h, const uint64_t (&ent)[(TS * NG + kWave - 1) / kWave],
                                            const uint64_t (&c0_64)[(TS * NG + kWave - 1) / kWave]) {
    constexpr Cell kInfCell = sizeof(Cell) == 8 ? (Cell)kInf : (Cell)kInf32;
    constexpr Cell kAllOnes = ~(Cell)0;
    constexpr int kCols = kWave * TE;
    constexpr int kQ = (TS * NG + kWave - 1) / kWave;
    static_assert(TS <= 16, "one scalar load fetches the R keys of a row");
    using KeyT = typename Key::T;
    constexpr bool kDouble = sizeof(KeyT) == 8;
    typedef uint32_t relv __attribute__((ext_vector_type(TE)));
    typedef Cell cellv __attribute__((ext_vector_type(TE)));
    __builtin_amdgcn_s_setprio(3);                 // (a wave with loads to issue goes first, as in sweep_u32_shared)
    const int lane = lane_id();
    const int e0 = tile_start + lane * TE;
    const int s0 = g * TS;
    const bool first = l == 1;

    Cell *part = reinterpret_cast<Cell *>(lds_cells);                   // [NG][kCols] partial column minima
    Cell *cells = part + NG * kCols;                                    // [KEEP][kCols] fetched rows, then their keys
    uint64_t *row_ent = reinterpret_cast<uint64_t *>(cells + KEEP * kCols);   // [TS * NG] kept rows: list entry
    uint64_t *row_c0 = row_ent + TS * NG;                               // [TS * NG] and c(l-1, s')
    uint32_t *live = reinterpret_cast<uint32_t *>(row_c0 + TS * NG);    // [KEEP] slot << 16 | strategy
    uint32_t *count = live + KEEP;                                      // [3] live rows, by pass modulo 3
    if (g == 0 && lane == 0) count[0] = 0;

    // Peek.  Lane i holds list entry i (and i + 64, ...): every wave does all rows itself, so no
    // exchange is needed and all waves agree on which rows are fetched and who fetches them.
    const int64_t n_samples = a.e_pad / kSample;
    const Cell *prev_cost = reinterpret_cast<const Cell *>(pack_tables(a, (l - 1) & 1, b).cost);
    Cell lower[kQ], upper = kAllOnes;
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int shift = (int)(uint32_t)(ent[q] >> 32);
        const int last = tile_start + kCols - 1 - shift, before = tile_start - 1 - shift;
        const bool listed = q * kWave + lane < h.n;
        Cell lo, up;
        if (first) {
            lo = last >= 0 ? (Cell)c0_64[q] : kInfCell;
            up = before >= 0 ? (Cell)c0_64[q] : kInfCell;
        } else {
            const Cell *row = prev_cost + (int64_t)(uint32_t)ent[q] * n_samples;
            const int at_last = min(last, h.x_prev) / kSample;                  // (ends at or after the column)
            const int at_before = (min(before, h.x_prev) + 1) / kSample - 1;    // (ends at or before it)
            const bool lo_ok = last >= h.y_prev;
            const bool up_ok = before >= 0 && at_before >= h.y_prev / TILE * (TILE / kSample);
            const int last_stored = h.x_prev / kSample;
            const Cell v_lo = row[lo_ok ? at_last : last_stored], v_up = row[up_ok ? at_before : last_stored];
            lo = lo_ok ? v_lo : kInfCell;
            up = up_ok ? v_up : kInfCell;
        }
        lower[q] = listed ? lo : kAllOnes;
        upper = min(upper, listed ? up : kAllOnes);
    }
    const Cell bound = wave_min(upper);
    // (no bound without a reachable column in front of the tile; rows without a reachable cell are out either way)
    const Cell limit = a.peek && bound < kInfCell ? bound + (Cell)h.dmax : kInfCell;
    int nk = 0;                                    // rows to fetch
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const bool kept = lower[q] < limit;
        const uint64_t votes = __builtin_amdgcn_ballot_w64(kept);
        if (kept) {                                // (all waves write the same words)
            const int at = nk + __builtin_popcountll(votes & ((1ull << lane) - 1ull));
            row_ent[at] = ent[q];
            row_c0[at] = c0_64[q];
        }
        nk += __builtin_popcountll(votes);
    }
    if (MAY_REFUSE && nk > KEEP) return false;

    // The shifted cells of kept row i for this lane's columns.
    struct Fetch {
        uint32_t sp[TE];                           // argmin bytes
        Cell cmin[TE];
        bool ok[TE];
        int x[TE];
    };
    auto row_entry = [&](int i, uint32_t &sp, int &shift, Cell &cp) {
        const uint64_t en = row_ent[i], cv = row_c0[i];
        sp = (uint32_t)uniform((int)(uint32_t)en);
        shift = uniform((int)(uint32_t)(en >> 32));
        cp = (Cell)((uint64_t)(uint32_t)uniform((int)(uint32_t)(cv >> 32)) << 32 | (uint32_t)uniform((int)(uint32_t)cv));
    };
    auto fetch_row = [&](const Former<Cell, Key> &t, uint32_t sp, int shift, Fetch &f) {
        const uint8_t *w = t.bp + (int64_t)sp * t.e_pad;
#pragma unroll
        for (int j = 0; j < TE; ++j) {
            const int idx = e0 + j - shift;
            f.ok[j] = idx >= h.y_prev;
            f.x[j] = f.ok[j] ? min(idx, h.x_prev) : h.x_prev;
            f.sp[j] = w[(uint32_t)f.x[j]];
            f.cmin[j] = t.cmin[(uint32_t)f.x[j]];
        }
    };
    auto finish_row = [&](const Former<Cell, Key> &t, uint32_t sp, Cell cp, const Fetch &f, Cell (&out)[TE]) {
        uint32_t rel[TE];
        KeyT r[TE];
#pragma unroll
        for (int j = 0; j < TE; ++j) {
            rel[j] = t.rel[(int64_t)f.sp[j] * t.e_pad + f.x[j]];
            r[j] = t.R[f.sp[j] * (uint32_t)t.S_pad + sp];
        }
#pragma unroll
        for (int j = 0; j < TE; ++j) {
            const Cell v = f.cmin[j] + (Cell)rel[j] + (Cell)Key::cost(r[j], t.k) + cp;
            out[j] = f.ok[j] ? v : kInfCell;
        }
    };
    auto made_up = [&](int shift, Cell cp, Cell (&out)[TE]) {
#pragma unroll
        for (int j = 0; j < TE; ++j) out[j] = e0 + j >= shift ? cp : kInfCell;
    };

    // Wave g fetches kept rows g, g + NG, ...: two at a time, so that their round trips overlap.
    Cell cmin[TE];
    {
        const Former<Cell, Key> former(a, b, l, h.r_prev);
        Cell pm[TE];
#pragma unroll
        for (int j = 0; j < TE; ++j) pm[j] = kAllOnes;
        auto take = [&](int i, const Cell (&v)[TE]) {
            cellv out;
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                pm[j] = min(pm[j], v[j]);
                out[j] = v[j];
            }
            if (i < KEEP) *reinterpret_cast<cellv *>(cells + i * kCols + lane * TE) = out;
        };
        for (int i = g; i < nk; i += 2 * NG) {
            uint32_t spa, spb;
            int sha, shb;
            Cell ca, cb, va[TE], vb[TE];
            row_entry(i, spa, sha, ca);
            const bool two = i + NG < nk;
            if (two) row_entry(i + NG, spb, shb, cb);
            if (first) {
                made_up(sha, ca, va);
                if (two) made_up(shb, cb, vb);
            } else if (two) {
                Fetch fa, fb;
                fetch_row(former, spa, sha, fa);
                fetch_row(former, spb, shb, fb);
                finish_row(former, spa, ca, fa, va);
                finish_row(former, spb, cb, fb, vb);
            } else {
                Fetch fa;
                fetch_row(former, spa, sha, fa);
                finish_row(former, spa, ca, fa, va);
            }
            take(i, va);
            if (two) take(i + NG, vb);
        }
        if (g < nk) {
            cellv out;
#pragma unroll
            for (int j = 0; j < TE; ++j) out[j] = pm[j];
            *reinterpret_cast<cellv *>(part + g * kCols + lane * TE) = out;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < TE; ++j) cmin[j] = kAllOnes;
#pragma unroll
        for (int w = 0; w < NG; ++w)
            if (w < nk) {
                const cellv v = *reinterpret_cast<const cellv *>(part + w * kCols + lane * TE);
#pragma unroll
                for (int j = 0; j < TE; ++j) cmin[j] = min(cmin[j], v[j]);
            }
    }

    // Keys of the alive rows, and the min-plus product over them, KEEP kept rows at a time (one
    // pass unless transition costs dwarf the spread of the layer costs).
    KeyT acc[TS][TE];
#pragma unroll
    for (int s = 0; s < TS; ++s)
#pragma unroll
        for (int j = 0; j < TE; ++j) acc[s][j] = Key::none();
    const Layout &a1 = layout_again();
    const int S_pad = a1.S_pad, k = a1.k_bits;
    const bool idle = s0 >= a1.S;                  // an idle strategy group only fetches rows
    const ConstPtr<KeyT> Rk = as_const(rkeys<KeyT>(a1, b, h.r) + s0);
    uint32_t rows_reduced = 0;
    int pass = 0;
    for (int base = 0; base < nk; base += KEEP) {
        uint32_t *counter = count + pass % 3;
        for (int i = base + g; i < nk && i < base + KEEP; i += NG) {
            uint32_t sp;
            int shift;
            Cell cp, v[TE];
            row_entry(i, sp, shift, cp);
            const int slot = i - base;
            if (base == 0) {
                const cellv in = *reinterpret_cast<const cellv *>(cells + slot * kCols + lane * TE);
#pragma unroll
                for (int j = 0; j < TE; ++j) v[j] = in[j];
            } else if (first) {
                made_up(shift, cp, v);
            } else {
                const Former<Cell, Key> former(layout_again(), b, l, h.r_prev);
                Fetch f;
                fetch_row(former, sp, shift, f);
                finish_row(former, sp, cp, f, v);
            }
            relv d, key;
            bool alive = false;
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                const Cell rel = v[j] - cmin[j];
                d[j] = (uint32_t)min(rel, (Cell)h.dmax);
                key[j] = kDouble ? d[j] : d[j] << k;
                alive |= rel < (Cell)h.dmax && cmin[j] < kInfCell;
            }
            if (__builtin_amdgcn_ballot_w64(alive) != 0) {   // wave-uniform
                // (keys take the first words of the slot; wide cells leave the rest unused)
                *reinterpret_cast<relv *>(reinterpret_cast<uint32_t *>(cells + slot * kCols) + lane * TE) = key;
                const Layout &ar = layout_again();
                *reinterpret_cast<relv *>(pack_tables(ar, l & 1, b).rel + (int64_t)sp * ar.e_pad + e0) = d;
                if (lane == 0) live[atomicAdd(counter, 1u)] = (uint32_t)slot << 16 | sp;
            }
        }
        if (g == 0 && lane == 0) count[(pass + 1) % 3] = 0;
        __syncthreads();
        if (pass == 0) __builtin_amdgcn_s_setprio(0);
        const int cnt = uniform((int)*counter);
        rows_reduced += (uint32_t)cnt;
        if constexpr (kDouble) {
            if (!idle && cnt > 0) {
                using Group = std::conditional_t<(TS > 8 && TS <= 12), RGroupMid, RGroup<(TS > 8 ? 2 : 1)>>;
                uint32_t rel[2][TE];
                uint32_t sp[2];
                Group buf[2];
                auto request = [&](int q, int i) {
                    const uint32_t row = (uint32_t)uniform((int)live[i < cnt ? i : cnt - 1]);
                    sp[q] = row & 0xffffu;
                    const relv in = *reinterpret_cast<const relv *>(reinterpret_cast<const uint32_t *>(cells + (row >> 16) * kCols) + lane * TE);
#pragma unroll
                    for (int j = 0; j < TE; ++j) rel[q][j] = in[j];
                };
                auto reduce_row = [&](int q) {     // the next row's transition keys in flight under this one's arithmetic
                    rgroup_request(buf[q ^ 1], Rk + (int64_t)uniform((int)sp[q ^ 1]) * S_pad);
                    double key[TE];
#pragma unroll
                    for (int j = 0; j < TE; ++j) key[j] = Key::make(rel[q][j], k);
#pragma unroll
                    for (int s = 0; s < TS; ++s)
                        minplus<TE>(acc[s], key, rgroup_key(buf[q], s), rgroup_keep0(buf[q ^ 1]), rgroup_keep1(buf[q ^ 1]));
                    rgroup_await(buf[q ^ 1]);
                };
                request(0, 0);
                request(1, 1);
                rgroup_request(buf[0], Rk + (int64_t)uniform((int)sp[0]) * S_pad);
                rgroup_await(buf[0]);
                int i = 0;
                for (; i + 2 <= cnt; i += 2) {
                    reduce_row(0);
                    request(0, i + 2);
                    reduce_row(1);
                    request(1, i + 3);
                }
                if (i < cnt) reduce_row(0);
            }
        } else if (!idle && cnt > 0) {
            const int npair = (cnt + 1) / 2;       // an odd tail repeats its entry: min(x, x) = x
            uint32_t va[2][TE], vb[2][TE];
            uint32_t spa[2], spb[2];
            R32Row<TS> ra[2], rb[2];
            auto request = [&](int q, int pr) {
                const uint32_t la = (uint32_t)uniform((int)live[2 * pr < cnt ? 2 * pr : cnt - 1]);
                const uint32_t lb = (uint32_t)uniform((int)live[2 * pr + 1 < cnt ? 2 * pr + 1 : cnt - 1]);
                spa[q] = la & 0xffffu;
                spb[q] = lb & 0xffffu;
                const relv ka = *reinterpret_cast<const relv *>(reinterpret_cast<const uint32_t *>(cells + (la >> 16) * kCols) + lane * TE);
                const relv kb = *reinterpret_cast<const relv *>(reinterpret_cast<const uint32_t *>(cells + (lb >> 16) * kCols) + lane * TE);
#pragma unroll
                for (int j = 0; j < TE; ++j) {
                    va[q][j] = ka[j];
                    vb[q][j] = kb[j];
                }
            };
            auto reduce_pair = [&](int q) {
                // keys of the next pair's rows, in flight under this pair's arithmetic
                ra[q ^ 1].request(Rk + (int64_t)uniform((int)spa[q ^ 1]) * S_pad);
                rb[q ^ 1].request(Rk + (int64_t)uniform((int)spb[q ^ 1]) * S_pad);
#pragma unroll
                for (int s = 0; s < TS; ++s)
                    minplus_u32x2<TE>(acc[s], va[q], vb[q], ra[q].at(s), rb[q].at(s), ra[q ^ 1], rb[q ^ 1]);
                r32_await(ra[q ^ 1], rb[q ^ 1]);
            };
            request(0, 0);
            request(1, 1);
            ra[0].request(Rk + (int64_t)uniform((int)spa[0]) * S_pad);
            rb[0].request(Rk + (int64_t)uniform((int)spb[0]) * S_pad);
            r32_await(ra[0], rb[0]);
            int pr = 0;
            for (; pr + 2 <= npair; pr += 2) {
                reduce_pair(0);
                request(0, pr + 2);
                reduce_pair(1);
                request(1, pr + 3);
            }
            if (pr < npair) reduce_pair(0);
        }
        ++pass;
        if (base + KEEP < nk) __syncthreads();     // the slots and the list are free again
    }
    const Layout &a2 = layout_again();
    const PackTables now = pack_tables(a2, l & 1, b);
    const int64_t e_pad = a2.e_pad;
    if (g == 0 && lane == 0) {                     // statistics: how much the pruning removed
        uint32_t *st = a2.stats + 2 * (((int64_t)b * (a2.L - 1) + (l - 1)) * a2.n_tiles + tile_start / TILE);
        if (part_stats == kMeanStats) {
            st[0] = ((st[0] >> 16) + rows_reduced + 1) / 2 << 16 | (uint32_t)h.n;
            st[1] = (st[1] + (uint32_t)nk + 1) / 2;
        } else {
            const uint32_t rows = rows_reduced << 16 | (uint32_t)h.n;
            st[0] = part_stats == kAddStats ? st[0] + rows : rows;
            st[1] = part_stats == kAddStats ? st[1] + (uint32_t)nk : (uint32_t)nk;
        }
    }
    if (g == 0) {
        cellv out;
#pragma unroll
        for (int j = 0; j < TE; ++j) out[j] = cmin[j];
        *reinterpret_cast<cellv *>(reinterpret_cast<Cell *>(now.cmin) + e0) = out;
    }
    if (idle) return true;
    const int S = a2.S;
    uint8_t *bp = byte_rows(a2, b, l) + (int64_t)s0 * e_pad + tile_start;

    // (of an unreachable column the bytes are never used: readers compare with Y_l)
    const uint32_t mask = ((1u << k) - 1u) * 0x01010101u;
    auto store = [&](auto full) {                  // (whole groups of strategies: no test per row)
#pragma unroll
        for (int s = 0; s < TS; ++s)
            if (full || s0 + s < S) {
                uint8_t *row = bp + (int64_t)s * e_pad;
                uint32_t low[TE];
#pragma unroll
                for (int j = 0; j < TE; ++j) low[j] = Key::low(acc[s][j]);
                if constexpr (TE == 4) {
                    const uint32_t p01 = __builtin_amdgcn_perm(low[1], low[0], 0x0c0c0400u);
                    const uint32_t p23 = __builtin_amdgcn_perm(low[3], low[2], 0x0c0c0400u);
                    reinterpret_cast<uint32_t *>(row)[lane] = __builtin_amdgcn_perm(p23, p01, 0x05040100u) & mask;
                } else if constexpr (TE == 2) {
                    reinterpret_cast<uint16_t *>(row)[lane] =
                        (uint16_t)(__builtin_amdgcn_perm(low[1], low[0], 0x0c0c0400u) & mask);
                } else {
                    row[lane] = (uint8_t)(low[0] & mask);
                }
            }
        // the last column of every 64: samples for the next layer's peek
        constexpr int kLanes = kSample / TE;
        if ((lane & (kLanes - 1)) == kLanes - 1) {
            const ConstPtr<uint64_t> ck = as_const(a2.ck + ((int64_t)b * a2.L + l) * S_pad + s0);
            const uint32_t n_samples = (uint32_t)(e_pad / kSample);
            Cell *out = reinterpret_cast<Cell *>(now.cost) + (int64_t)s0 * n_samples + e0 / kSample;
#pragma unroll
            for (int s = 0; s < TS; ++s)
                if (full || s0 + s < S)
                    out[(uint32_t)s * n_samples] =
                        cmin[TE - 1] < kInfCell ? cmin[TE - 1] + (Cell)Key::cost(acc[s][TE - 1], k) + (Cell)ck[s] : kInfCell;
        }
    };
    if (s0 + TS <= S)
        store(std::true_type{});
    else
        store(std::false_type{});
    return true;
}

// The sweep of handles that keep the byte table (Layout::packed).  Grid: (8 + tiles, 1, instances);
// the first workgroup of an instance runs live_step for the layer after this one.
template <int TS, int TE, int NG, int WPE, int W, int UX>
__global__ __launch_bounds__(W * kWave, WPE) void sweep_bytes_kernel(Layout a, int l) {
    constexpr int kTile = kWave * TE * UX;
    constexpr int kQ = (TS * NG + kWave - 1) / kWave;
    constexpr int kKeep = byte_keep_rows(TS, NG, WPE, kTile);
    const int wave = uniform(threadIdx.x >> 6);    // the only use of the thread-index register (see lane_id)
    const int b = a.b_off + blockIdx.z * a.b_step;
    // List entries of the former layer, lane i those of entry i, i + 64, ...: requested ahead of the header.
    uint64_t ent[kQ], c0[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
        const int i = q * kWave + lane_id();
        const int64_t at = ((int64_t)b * a.L + (l - 1)) * a.S_pad + (i < TS * NG ? i : TS * NG - 1);
        ent[q] = a.vlist[at];
        c0[q] = a.vcost[at];
    }
    const ConstPtr<int32_t> hdr = as_const(a.hdr + ((int64_t)b * a.L + l) * 8);
    const int st = hdr[0], budget = hdr[1];
    if (st < 0) return;
    const bool keys32 = st == GALV_INSTANCE_OK_FAST_U32 || st == GALV_INSTANCE_OK_U32_WIDE;
    const bool packed = byte_status(st, (uint32_t)hdr[3]);
    const int slot = (int)(blockIdx.x >> 3) - 1;
    if (slot < 0) {
        if ((blockIdx.x & 7) == 0 && packed) {
            auto step = [&](auto key) {
                using Key = decltype(key);
                if (l == 1) {                      // (layer 1 itself is being swept, up to prep_kernel's bound)
                    live_step<NG, Key>(layout_again(), wave, b, 1, false);
                    __syncthreads();
                }
                if (l + 1 < a.L) live_step<NG, Key>(layout_again(), wave, b, l + 1, true);
            };
            if (keys32)
                step(Key32{});
            else
                step(Key64{});
        }
        return;
    }
    const TileHdr h = {hdr[2], (uint32_t)hdr[3], hdr[4], hdr[4 - 8], hdr[5 - 8], hdr[6 - 8]};
    const int y = packed ? hdr[5] : 0, x = packed ? hdr[6] : budget;
    if (y > x) return;
    // Each XCD takes a contiguous eighth of the tiles to sweep (see sweep_kernel).
    const int lo = y / kTile, nt = x / kTile - lo + 1;
    const int per = (nt + 7) >> 3;
    const int t = (int)(blockIdx.x & 7) * per + slot;
    if (slot >= per || t >= nt) return;
    const int tile_start = (lo + t) * kTile;
    if (st == GALV_INSTANCE_OK_FAST_U32) {
        // A tile of 256 columns that keeps more rows than its list holds (24 of 44, 32 of 64) would rebuild the rest
        // twice, in further passes: it is swept as two halves, for which the same LDS holds twice the rows.  Passes /
        // halves, in us, where a third to a half of the rows is kept: 44 strategies x 4805 tiles x 32 layers 1056 / 897,
        // 35 x 4805 x 96 3135 / 2880, 64 x 3768 x 20 610 / 572; a list that overflows by little pays more for the
        // second half than for the pass (56 x 2893 x 15 949 / 979).
        const bool done = sweep_bytes<TS, TE * UX, NG, uint32_t, Key32, kKeep, kTile, (UX > 1)>(
            layout_again(), wave, l, b, tile_start, kSetStats, h, ent, c0);
        if constexpr (UX > 1)
            for (int p = 0; p < UX && !done; ++p) {
                const int part = tile_start + p * (kTile / UX);
                if (part > x) break;                             // workgroup-uniform
                __syncthreads();                                 // the LDS of the part before is free again
                sweep_bytes<TS, TE, NG, uint32_t, Key32, UX * kKeep, kTile>(
                    layout_again(), wave, l, b, part, p ? kMeanStats : kSetStats, h, ent, c0);
            }
    } else if (packed) {
        // 8-byte cells: a part of the tile at a time keeps registers and LDS within what the narrow form uses
        for (int p = 0; p < TE; ++p) {
            if (tile_start + p * (kWave * UX) > x) break;    // workgroup-uniform
            if (p) __syncthreads();                          // the LDS of the part before is free again
            if (keys32)
                sweep_bytes<TS, UX, NG, uint64_t, Key32, kKeep, kTile>(layout_again(), wave, l, b, tile_start + p * (kWave * UX), p ? kAddStats : kSetStats, h, ent, c0);
            else
                sweep_bytes<TS, UX, NG, uint64_t, Key64, kKeep, kTile>(layout_again(), wave, l, b, tile_start + p * (kWave * UX), p ? kAddStats : kSetStats, h, ent, c0);
        }
    } else if (st == GALV_INSTANCE_OK_FAST) {
        for (int u = 0; u < UX; ++u)
            sweep_fast<TS, TE, NG, Narrow, int32_t>(layout_again(), wave, l, b, budget, tile_start + u * (kTile / UX));
    } else if (st == GALV_INSTANCE_OK_FAST_WIDE) {
        for (int u = 0; u < UX; ++u)
            sweep_fast<TS, TE, NG, Wide, int32_t>(layout_again(), wave, l, b, budget, tile_start + u * (kTile / UX));
    } else {
        sweep_int64<8>(layout_again(), wave, l, b, budget, tile_start);
    }
}

// ------------------------------------------------------------- chained sweep
//
// All layers of a search in one launch, for launches whose layers are too small to hide what a launch per layer costs
// (2.5 us from one empty launch to the next, 4 us with a kernel's first loads).  A workgroup owns 128
// budget columns of one instance and takes them through the layers; layer l of its columns needs layer l - 1 of
// columns at or below them only, so a workgroup waits for its left neighbours and never for a right one.
//   * Workgroups take their places in the order in which they start (a counter, cleared by prep_kernel), columns
//     ascending.  Whoever waits, waits for a place below its own, that is for a workgroup that runs already: the wait
//     ends however few workgroups the GPU holds at a time, whatever else runs on it.
//   * Costs pass between workgroups at agent scope, past the caches that other XCDs do not see; when all of a
//     workgroup's stores have arrived it writes its word of the flags, and a reader reads its cells after it has
//     seen the words of the blocks it needs.  (A fence per layer would write back and invalidate whole caches: 5 us
//     with 64 workgroups, 18 with 256, against 1.3 for the words.)  One wave asks for all, and every word has a line
//     of its own: with a word per wave and every wave asking, a layer of `single` below took 4.9 us instead of 3.6.
//   * Every layer has rows of its own (no two layers share memory): nobody has to wait until others have read.
// Rows are whole costs, [B][L][S_pad][e_pad], argmins one byte as in the byte table, and as there only the columns
// [Y_l, X_l] are swept and stored: the first places of the order belong to one wave per instance that runs the
// recurrence without a memory limit ahead of the sweep and tells each layer's X_l.
//
// What bounds it is the latency of a layer's chain: words 0.6 us, rows 0.8, column minima and alive rows 0.6, min-plus and
// new cells 0.5, until the cells have arrived 0.5.  Whole searches, a launch per layer / chained, in us: 29 strategies x 78 tiles
// x 37 layers (`single`) 250 / 156, 22 x 1032 x 32 282 / 186, 22 x 1256 x 24 with all budgets 249 / 192, 44 x 272 x 48 479 / 294.
constexpr int kChainCols = 128;
// Polls of some 0.6 us after which a wait is given up, so that no error in the memory order could hang the GPU.  A correct solve
// must never get there, and the longest wait spans a whole search: the wave with an instance's last place may start with the
// first layer, and blocks may run ahead of their neighbours over layers whose memories are small.  Hence the limit on layers:
// at the slowest rate measured (100 us a layer: 60 strategies, 64-bit integers) that many take some 170000 polls, a twelfth of these.
constexpr int kSpins = 1 << 21;
constexpr int kChainLayers = 1024;

template <class T>
__device__ __forceinline__ T agent_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void agent_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class Cell>
__device__ __forceinline__ Cell *chain_rows(const Layout &a, int b, int l) {
    return reinterpret_cast<Cell *>(a.U[0] + ((int64_t)b * a.L + l) * a.S_pad * a.e_pad * 8);
}

// Until the blocks from `lo` to `hi` have finished layer `want`.
__device__ __forceinline__ bool chain_wait(const int32_t *flags, int lo, int hi, int32_t want) {
    const int lane = lane_id();
    for (; lo <= hi; lo += kWave) {
        bool waits = lo + lane <= hi;
        for (int n = 0;; ++n) {
            if (waits) waits = agent_load(flags + (int64_t)(lo + lane) * kWordStep) < want;   // (not asked for again)
            if (__builtin_amdgcn_ballot_w64(waits) == 0) break;
            if (n == kSpins) return false;
            if (n >= 64)
                __builtin_amdgcn_s_sleep(8);
            else if (n >= 16)
                __builtin_amdgcn_s_sleep(2);
        }
    }
    asm volatile("" ::: "memory");
    return true;
}
// X_l, once it is told.
__device__ __forceinline__ bool chain_last_column(const int32_t *p, int32_t &x) {
    for (int n = 0; x == kUnset; ++n) {
        if (n == kSpins) return false;
        __builtin_amdgcn_s_sleep(4);
        x = uniform(agent_load(p));
    }
    return true;
}

// The recurrence without a memory limit for instance b, all layers (see live_step), by one wave with a lane per strategy:
// no exchange, the transition keys in LDS.  (1.7 us a layer at 29 strategies, half of what the sweep takes.)  It keeps several
// matrices: fetched anew for each of 82 layers whose matrices alternate, the keys of 60 strategies made the sweep wait for it (539
// tiles, layers alike: 727 us, now 598; where the sweep's layers are longer, or a matrix smaller, no difference).
template <int ROWS, class Key>
__device__ __forceinline__ void chain_live(const Layout &a, int b, typename Key::Rel dmax, int budget) {
    using KeyT = typename Key::T;
    const int lane = lane_id();
    const int S = a.S, k = a.k_bits, L = a.L;
    // [slots][S][ROWS], matrix r in slot r modulo their number: as many as the keys of a block's rows take (see chain_lds)
    constexpr int kSlots = kChainCols * 8 / (ROWS * (int)sizeof(KeyT));
    static_assert(kSlots >= 1 && kSlots <= kWave, "the matrix of each slot by lane");
    KeyT *slots = reinterpret_cast<KeyT *>(lds_cells);
    int held = -1;                                 // lane i: the matrix in slot i
    int32_t *hdr = a.hdr + (int64_t)b * L * 8;
    const uint64_t *costs = a.ck + (int64_t)b * L * ROWS;
    const int32_t *mems = a.m + (int64_t)b * L * S;
    const bool in = lane < S;
    const uint32_t at = (uint32_t)(in ? lane : S - 1);         // this lane's strategy
    struct Step {                                  // a layer's inputs, requested a layer ahead
        uint64_t c;
        int32_t m, r, least;
    };
    auto load = [&](int l, Step &to) {
        l = l < L ? l : L - 1;
        to.c = (costs + (int64_t)l * ROWS)[at];
        to.m = (mems + (int64_t)l * S)[at];
        to.r = (hdr + l * 8)[4];
        to.least = (hdr + l * 8)[7];
    };
    Step now, next;
    load(0, now);
    load(1, next);
    uint64_t V = now.c;
    int32_t mem = 0, m = now.m;                    // memory in the layers before; of the layer at hand
    for (int l = 1; l < L; ++l) {
        now = next;
        const int r = uniform(now.r), slot = r % kSlots;
        KeyT *Rl = slots + slot * (ROWS * ROWS);
        if ((int)read_lane((uint32_t)held, slot) != r) {
            const KeyT *Rk = rkeys<KeyT>(a, b, r);
            for (int i0 = 0; i0 < S; i0 += 8) {    // (eight rows under way at a time, the last one repeated)
                KeyT row[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) row[u] = (Rk + (i0 + u < S ? i0 + u : S - 1) * ROWS)[at];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (i0 + u < S && in) Rl[(i0 + u) * ROWS + lane] = row[u];
            }
            if (lane == slot) held = r;
        }
        load(l + 1, next);
        const bool usable = in && m <= budget;
        const uint64_t vmin = wave_min(usable ? V : ~(uint64_t)0);
        if (vmin == ~(uint64_t)0) {                // nothing reachable from here on
            if (lane == 0)
                for (int q = l > 1 ? l : 2; q < L; ++q) agent_store(hdr + q * 8 + 6, -1);
            return;
        }
        const int64_t with = (int64_t)mem + m;     // memory with the former layer, saturating just above the budget
        const int32_t upto = (int32_t)(with <= budget ? with : (int64_t)budget + 1);
        // (an unusable strategy costs as much as one that is ruled out)
        const uint64_t rel = V - vmin;
        const typename Key::Stored dv = Key::stored(usable && rel < dmax ? (typename Key::Rel)rel : dmax, k);
        KeyT best = Key::none();
        for (int i0 = 0; i0 < S; i0 += 8) {
            KeyT row[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) row[u] = Rl[(i0 + u < S ? i0 + u : S - 1) * ROWS + at];
#pragma unroll
            for (int u = 0; u < 8; ++u) best = Key::least(best, Key::from(read_lane(dv, i0 + u < S ? i0 + u : S - 1), k) + row[u]);
        }
        const int32_t x = __shfl(upto, (int)(Key::low(best) & ((1u << k) - 1u)), kWave);
        V = vmin + Key::cost(best, k) + now.c;
        mem = x;
        m = now.m;
        const uint32_t top = ~wave_min(~(in && m <= budget ? (uint32_t)x : 0u));
        const int64_t fits = (int64_t)budget - uniform(now.least);       // beyond it nobody reads layer l
        // (layer 1 is being swept up to prep_kernel's bound: every wave has to see the same one)
        if (l > 1 && lane == 0) agent_store(hdr + l * 8 + 6, (int32_t)((int64_t)top < fits ? (int64_t)top : fits));
    }
}

// A buffer over the rows of one layer, for loads and stores at agent scope of several cells at once: a wave-uniform offset
// and one that no row changes per lane cost no address arithmetic.
constexpr int kAgent = 16;                         // (the sc1 bit: what relaxed atomics at agent scope carry)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t chain_buffer(void *rows) {
    return __builtin_amdgcn_make_buffer_rsrc(rows, 0, 0xffffffffu, 0x00020000);
}
template <class Cell>
__device__ __forceinline__ void buffer_cells(__amdgpu_buffer_rsrc_t rows, uint32_t lane_off, uint32_t off, Cell (&out)[2]) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    if constexpr (sizeof(Cell) == 4) {
        const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rows, (int)lane_off, (int)off, kAgent));
        out[0] = v[0];
        out[1] = v[1];
    } else {
        const u32x4 v = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rows, (int)lane_off, (int)off, kAgent));
        out[0] = (uint64_t)v[1] << 32 | v[0];
        out[1] = (uint64_t)v[3] << 32 | v[2];
    }
}
template <class Cell>
__device__ __forceinline__ void buffer_store_cells(__amdgpu_buffer_rsrc_t rows, uint32_t lane_off, uint32_t off, const Cell (&in)[2]) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    if constexpr (sizeof(Cell) == 4) {
        const u32x2 v = {in[0], in[1]};
        __builtin_amdgcn_raw_buffer_store_b64(v, rows, (int)lane_off, (int)off, kAgent);
    } else {
        // (the whole offset per lane: behind a store of 16 bytes with a scalar offset the compiler leaves no wait states
        // before the data registers are written again, and the first cell of some lanes was then lost; the build refuses that form)
        const u32x4 v = {(uint32_t)in[0], (uint32_t)(in[0] >> 32), (uint32_t)in[1], (uint32_t)(in[1] >> 32)};
        __builtin_amdgcn_raw_buffer_store_b128(v, rows, (int)(lane_off + off), 0, kAgent);
    }
}

// What a layer's sweep needs to know, requested a layer ahead.
struct ChainIn {
    uint64_t ent;                                  // list entry `lane` of the former layer
    int32_t h;                                     // header record, lane i word i
    uint64_t ck;                                   // c(l, first strategy of the wave + lane)
    int32_t x;                                     // X_l as far as told (wave 0)
};
template <int TS, int NG>
__device__ __forceinline__ void chain_load(const Layout &a, int wave, int b, int l, ChainIn &in) {
    const int lane = lane_id();
    const int64_t row = (int64_t)b * a.L + l;
    const uint64_t *list = a.vlist + (row - 1) * (TS * NG), *cost = a.ck + row * (TS * NG) + wave * TS;
    int32_t *record = a.hdr + row * 8;
    in.ent = list[(uint32_t)(lane < TS * NG ? lane : TS * NG - 1)];
    in.h = record[(uint32_t)lane & 7];
    in.ck = cost[(uint32_t)(lane < TS ? lane : TS - 1)];
    in.x = 0;
    if (wave == 0) in.x = agent_load(record + 6);
}

// One workgroup's columns, layers 1 to L - 1: byte_status() instances.  As in sweep_u32_shared a wave owns the rows
// g, g + NG, ... of the former layer's list and the strategies g * TS on; the column minima meet in LDS, and the rows
// that are alive in the tile, all of which fit, are reduced by every wave, with the transition keys from LDS.  Wave 0 does the waiting for all.
template <int TS, int NG, class Cell, class Key>
__device__ __forceinline__ void chain_tiles(const Layout &a, int wave, int b, int t, typename Key::Rel dmax, ChainIn &in, uint64_t c0) {
    constexpr Cell kInfCell = sizeof(Cell) == 8 ? (Cell)kInf : (Cell)kInf32;
    constexpr Cell kAllOnes = ~(Cell)0;
    constexpr int kCols = kChainCols, TE = kCols / kWave, kRows = TS * NG;
    static_assert(kRows <= kWave, "list positions by lane");
    using KeyT = typename Key::T;
    using Word = std::conditional_t<sizeof(Cell) == 8, unsigned long long, uint32_t>;
    using Rel = typename Key::Rel;
    using Stored = typename Key::Stored;
    typedef Stored relv __attribute__((ext_vector_type(TE)));
    const int lane = lane_id();
    const int S = a.S, S_pad = kRows, L = a.L, k = a.k_bits;
    const int start = t * kCols, e0 = start + lane * TE;
    const uint32_t lane_off = (uint32_t)lane * TE * (uint32_t)sizeof(Cell);
    int32_t *flags = chain_flags(a, b);
    Word *minima = reinterpret_cast<Word *>(lds_cells);                     // [2][kCols] of the columns, in turns
    unsigned long long *alive_of = reinterpret_cast<unsigned long long *>(minima + 2 * kCols);   // [2] list positions
    KeyT *Rl = reinterpret_cast<KeyT *>(alive_of + 2);                      // [kRows][kRows] transition keys, where they are kept
    Stored *keys = reinterpret_cast<Stored *>(Rl + (Key::kKeysInLds ? kRows * kRows : 0));      // [kRows][kCols] relative costs by list position
    int32_t *last_of = reinterpret_cast<int32_t *>(keys + kRows * kCols);   // [2] X_l, by layer modulo 2
    uint64_t *kept_ent = reinterpret_cast<uint64_t *>(last_of + 2);         // [kRows] entries of the rows to read, and how many
    int32_t *kept_n = reinterpret_cast<int32_t *>(kept_ent + kRows);

    auto load = [&](int l, ChainIn &in) { chain_load<TS, NG>(layout_again(), wave, b, l < L ? l : L - 1, in); };
    // (Here the loads have arrived.  Left to itself the compiler waits for them at the top of the loop, where it cannot
    // tell them from the stores behind them and waits for those too.)
    auto settle = [&](ChainIn &in) { asm volatile("" : "+v"(in.ent), "+v"(in.h), "+v"(in.ck), "+v"(in.x)); };
    settle(in);
    int32_t *records = a.hdr + (int64_t)b * L * 8;
    int r_now = -1;
    int y_prev = 0, x_prev = 0;
    int turn = 0;
    auto clear = [&](int h) {
        Word *p = minima + h * kCols + lane * TE;
#pragma unroll
        for (int j = 0; j < TE; ++j) p[j] = kAllOnes;
        if (lane == 0) alive_of[h] = 0;
    };
    if (wave == 0) {                               // (the first layer's barrier is ahead)
        clear(0);
        clear(1);
    }
    uint32_t bytes[TS];                            // the former layer's argmins, not stored yet
    int unstored = 0;                              // of which layer (0: none)
    auto store_bytes = [&] {
        const Layout &al = layout_again();
        const uint32_t pitch = (uint32_t)al.e_pad;
        const int s0 = wave * TS;
        const __amdgpu_buffer_rsrc_t to = chain_buffer(byte_rows(al, b, unstored) + (int64_t)s0 * pitch + start);
#pragma unroll
        for (int s = 0; s < TS; ++s)
            if (s0 + s < S) __builtin_amdgcn_raw_buffer_store_b16((short)bytes[s], to, lane * 2, (int)(s * pitch), 0);
    };
    for (int l = 1; l < L; ++l) {
        // (What follows from these is worked out where it is used: kept from before the loop it would fill the scalar
        // registers and be spilled into vector lanes.)
        int g = wave;
        uint32_t pitch = (uint32_t)a.e_pad;        // (a layer's rows are below 4 GB, see make_plan)
        asm volatile("" : "+s"(g), "+s"(pitch));
        const int s0 = g * TS;
        const int n = (int)read_lane((uint32_t)in.h, 2), r_sel = (int)read_lane((uint32_t)in.h, 4);
        const int y = (int)read_lane((uint32_t)in.h, 5);
        if (start + kCols - 1 < y) break;          // nothing reachable here, in this layer and from it on
        // Another matrix than before: its keys, fetched by the waves that would only wait for wave 0.  (Read two barriers on, last
        // read before the latest one.  Fetched by all waves in front of the rows, deep stacks whose matrices alternate from layer to
        // layer took, in us: 60 strategies x 539 tiles x 82 layers 1053, now 1003; 18 x 1440 x 54 544, 499; 44 x 1032 x 24 311, 281.)
        const KeyT *Rk = rkeys<KeyT>(layout_again(), b, r_sel);
        if (Key::kKeysInLds && r_sel != r_now) {
            if (g != 0)
                for (int i = g - 1; i < S; i += NG - 1)
                    if (lane < kRows) Rl[i * kRows + lane] = (Rk + (int64_t)i * S_pad)[lane];
            r_now = r_sel;
        }
        if (g == 0) {
            int x = uniform(in.x);
            bool told = chain_last_column(records + l * 8 + 6, x);
            if (told && l > 1 && start <= x && y <= x) {
                // the former layer's blocks from the largest memory's shift to the smallest one's, but for the own one
                const uint32_t shift = (uint32_t)(in.ent >> 32);
                const int sh_lo = (int)wave_min(shift), sh_hi = (int)~wave_min(~shift);
                const int lo = min(max(start - sh_hi, y_prev), x_prev) / kCols;
                const int hi = start + kCols - 1 - sh_lo < y_prev ? -1 : min(min(start + kCols - 1 - sh_lo, x_prev) / kCols, t - 1);
                told = chain_wait(flags, lo, hi, l - 1);
                if (a.peek && told) {
                    // Rows are non-increasing: a row's cells here are at least its cell in the last column, every column
                    // minimum is at most the one in the first column (see sweep_u32_shared).
                    const __amdgpu_buffer_rsrc_t rows = chain_buffer(chain_rows<Cell>(a, b, l - 1));
                    const int first = start - (int)shift, last = first + kCols - 1;
                    const uint32_t row = (uint32_t)in.ent * pitch;
                    auto cell = [&](int at) -> Cell {
                        const uint32_t off = (row + (uint32_t)min(max(at, y_prev), x_prev)) * (uint32_t)sizeof(Cell);
                        if constexpr (sizeof(Cell) == 4)
                            return (Cell)__builtin_amdgcn_raw_buffer_load_b32(rows, (int)off, 0, kAgent);
                        else
                            return __builtin_bit_cast(Cell, __builtin_amdgcn_raw_buffer_load_b64(rows, (int)off, 0, kAgent));
                    };
                    const Cell at_first = cell(first), at_last = cell(last);
                    const bool listed = lane < n;
                    const Cell upper = listed && first >= y_prev ? at_first : kInfCell;
                    const Cell lower = listed && last >= y_prev ? at_last : kInfCell;
                    const Cell bound = wave_min(upper);
                    const bool kept = lower < (bound < kInfCell ? bound + (Cell)dmax : kInfCell);
                    const uint64_t votes = __builtin_amdgcn_ballot_w64(kept);
                    if (kept) kept_ent[__builtin_popcountll(votes & ((1ull << lane) - 1ull))] = in.ent;
                    if (lane == 0) *kept_n = __builtin_popcountll(votes);
                }
            }
            if (lane == 0) last_of[l & 1] = told ? x : kUnset;
        }
        __syncthreads();
        const int x = uniform(last_of[l & 1]);
        if (x == kUnset) {
            a.status[b] = GALV_INSTANCE_GAVE_UP;
            return;
        }
        if (y > x) break;                          // nothing reachable anywhere
        if (start > x) {                           // constant here: nothing to store
            load(l + 1, in);
            settle(in);
            y_prev = y;
            x_prev = x;
            continue;
        }
        uint64_t ent = in.ent;
        int nk = n;
        if (a.peek && l > 1) {
            nk = uniform(*kept_n);
            ent = kept_ent[lane < nk ? lane : 0];  // (beyond the list's end: not used)
        }
        Cell row[TS][TE];
        if (l == 1) {
#pragma unroll
            for (int r = 0; r < TS; ++r) {
                const int shift = (int)read_lane((uint32_t)(ent >> 32), g + NG * r);
                const Cell cp = (Cell)read_lane(c0, g + NG * r);
#pragma unroll
                for (int j = 0; j < TE; ++j) row[r][j] = e0 + j >= shift ? cp : kInfCell;
            }
        } else {
            // which rows lie inside the stored columns, and which nowhere reachable; where they begin
            const int shift_of = (int)(uint32_t)(ent >> 32);
            const uint64_t inside = __builtin_amdgcn_ballot_w64(start - shift_of >= y_prev && start + kCols - 1 - shift_of <= x_prev);
            const uint64_t dead = __builtin_amdgcn_ballot_w64(start + kCols - 1 - shift_of < y_prev || lane >= nk);
            const uint32_t off = ((uint32_t)ent * pitch + (uint32_t)(start - shift_of)) * (uint32_t)sizeof(Cell);
            const __amdgpu_buffer_rsrc_t rows = chain_buffer(chain_rows<Cell>(a, b, l - 1));
#pragma unroll
            for (int r = 0; r < TS; ++r) {
                const int i = g + NG * r;
                if (dead >> i & 1) {
#pragma unroll
                    for (int j = 0; j < TE; ++j) row[r][j] = kInfCell;
                } else if (inside >> i & 1) {
                    buffer_cells(rows, lane_off, read_lane(off, i), row[r]);
                } else {
                    const uint64_t en = read_lane(ent, i);
                    const uint32_t first = (uint32_t)en * pitch * (uint32_t)sizeof(Cell);
                    const int at = e0 - (int)(uint32_t)(en >> 32);
#pragma unroll
                    for (int j = 0; j < TE; ++j) {
                        const uint32_t cell = (uint32_t)(at + j >= y_prev ? min(at + j, x_prev) : x_prev) * (uint32_t)sizeof(Cell);
                        if constexpr (sizeof(Cell) == 4)
                            row[r][j] = (Cell)__builtin_amdgcn_raw_buffer_load_b32(rows, (int)cell, (int)first, kAgent);
                        else
                            row[r][j] = __builtin_bit_cast(Cell, __builtin_amdgcn_raw_buffer_load_b64(rows, (int)cell, (int)first, kAgent));
                    }
#pragma unroll
                    for (int j = 0; j < TE; ++j)
                        if (at + j < y_prev) row[r][j] = kInfCell;
                }
            }
            if (unstored) store_bytes();           // (behind the loads: nobody waits for them)
            unstored = 0;
        }
        const uint32_t list = (uint32_t)ent;
        const uint64_t ck = in.ck;
        load(l + 1, in);
        Word *now = minima + turn * kCols + lane * TE;
#pragma unroll
        for (int j = 0; j < TE; ++j) {
            Cell v = row[0][j];
#pragma unroll
            for (int r = 1; r < TS; ++r) v = min(v, row[r][j]);
            atomicMin(now + j, (Word)v);
        }
        __syncthreads();
        // (an unreachable column's rows are far above 0, so that none of them counts as alive there)
        Cell cmin[TE], from[TE];
#pragma unroll
        for (int j = 0; j < TE; ++j) {
            cmin[j] = (Cell)now[j];
            from[j] = cmin[j] < kInfCell ? cmin[j] : 0;
        }
        unsigned long long mine = 0;
#pragma unroll
        for (int r = 0; r < TS; ++r) {
            relv d;
            Rel least = dmax;
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                const Rel rel = (Rel)min(row[r][j] - from[j], (Cell)dmax);
                least = min(least, rel);
                d[j] = Key::stored(rel, k);
            }
            *reinterpret_cast<relv *>(keys + (g + NG * r) * kCols + lane * TE) = d;
            if (__builtin_amdgcn_ballot_w64(least < dmax) != 0 && g + NG * r < nk)     // wave-uniform
                mine |= 1ull << (g + NG * r);
        }
        if (lane == 0 && mine) atomicOr(alive_of + turn, mine);
        __syncthreads();
        const uint64_t alive = read_lane((uint64_t)alive_of[turn], 0);
        KeyT acc[TS][TE];
#pragma unroll
        for (int s = 0; s < TS; ++s)
#pragma unroll
            for (int j = 0; j < TE; ++j) acc[s][j] = Key::none();
        for (uint64_t left = alive; left;) {       // two rows at a time; an odd one twice
            const int i = __builtin_ctzll(left);
            left &= left - 1;
            const int i2 = left ? __builtin_ctzll(left) : i;
            left &= left - 1;                      // (0 stays 0)
            const relv da = *reinterpret_cast<const relv *>(keys + i * kCols + lane * TE);
            const relv db = *reinterpret_cast<const relv *>(keys + i2 * kCols + lane * TE);
            const int at_a = (int)read_lane(list, i) * kRows + s0, at_b = (int)read_lane(list, i2) * kRows + s0;
            KeyT va[TE], vb[TE], ra[TS], rb[TS];
#pragma unroll
            for (int s = 0; s < TS; ++s) {
                ra[s] = Key::kKeysInLds ? Rl[at_a + s] : as_const(Rk)[at_a + s];
                rb[s] = Key::kKeysInLds ? Rl[at_b + s] : as_const(Rk)[at_b + s];
            }
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                va[j] = Key::from(da[j], k);
                vb[j] = Key::from(db[j], k);
            }
#pragma unroll
            for (int s = 0; s < TS; ++s)
#pragma unroll
                for (int j = 0; j < TE; ++j) acc[s][j] = Key::least(Key::least(acc[s][j], va[j] + ra[s]), vb[j] + rb[s]);
        }
        if (s0 < S) {
            const __amdgpu_buffer_rsrc_t out = chain_buffer(chain_rows<Cell>(a, b, l) + (int64_t)s0 * pitch + start);
            const uint32_t mask = ((1u << k) - 1u) * 0x0101u;
#pragma unroll
            for (int s = 0; s < TS; ++s)
                if (s0 + s < S) {
                    const Cell cs = (Cell)read_lane(ck, s);
                    Cell v[TE];
#pragma unroll
                    for (int j = 0; j < TE; ++j) v[j] = cmin[j] < kInfCell ? cmin[j] + (Cell)Key::cost(acc[s][j], k) + cs : kInfCell;
                    buffer_store_cells(out, lane_off, (uint32_t)s * pitch * (uint32_t)sizeof(Cell), v);
                }
#pragma unroll
            for (int s = 0; s < TS; ++s)
                bytes[s] = __builtin_amdgcn_perm(Key::low(acc[s][1]), Key::low(acc[s][0]), 0x0c0c0400u) & mask;
            unstored = l;
        }
        if (g == NG - 1 && lane == 0) {            // statistics
            const Layout &al = layout_again();
            uint32_t *st = al.stats + 2 * (((int64_t)b * (L - 1) + (l - 1)) * al.n_tiles + t);
            st[0] = (uint32_t)__builtin_popcountll(alive) << 16 | (uint32_t)n;
            st[1] = (uint32_t)nk;
        }
        turn ^= 1;
        if (g == NG / 2) clear(turn);              // (read a layer ago; the barrier below is before its next use)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the cells have arrived
        settle(in);
        __syncthreads();
        if (g == 0 && lane == 0) agent_store(flags + (int64_t)t * kWordStep, l);
        y_prev = y;
        x_prev = x;
    }
    if (unstored) store_bytes();
}

// The same for the other instances, whose costs do not fit a key: 64-bit integers, every candidate, plain back-pointers, all columns
// up to the budget.  The waves share the rows that reach into the block through LDS, all of them under way at once.  (With every
// wave reading every row for itself a layer was a chain of as many trips as there are strategies.  Whole searches in us, a launch
// per layer / that / shared rows: 29 strategies x 78 tiles x 37 layers 3115 / 764 / 401, 44 x 1032 x 24 9200 / 5860 / 1640, 6 x 4104 x 24
// 831 / 1057 / 504.)
template <int TS, int NG>
__device__ __forceinline__ void chain_int64(const Layout &a, int wave, int b, int t, int budget) {
    constexpr int kCols = kChainCols, TE = kCols / kWave;
    static_assert(TS * NG <= kWave && TE == 2, "strategies by lane, two columns a lane");
    typedef uint64_t cell2 __attribute__((ext_vector_type(TE)));
    typedef int32_t arg2 __attribute__((ext_vector_type(TE)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const int lane = lane_id();
    const int S = a.S, L = a.L;
    const uint32_t pitch = (uint32_t)a.e_pad;      // (a layer's rows are below 4 GB, see make_plan)
    const int start = t * kCols, e0 = start + lane * TE, s0 = wave * TS;
    if (start > budget) return;
    const uint32_t lane_off = (uint32_t)lane * TE * 8;
    int32_t *flags = chain_flags(a, b);
    int32_t *ready = reinterpret_cast<int32_t *>(lds_cells);   // [2] by layer modulo 2
    cell2 *shared = reinterpret_cast<cell2 *>(lds_cells + 4);  // [TS * NG][kWave] the rows that reach into the block
    for (int l = 1; l < L; ++l) {
        // the former layer's strategies that reach into these columns, in ascending order, by lane: index and memory
        const int64_t row0 = (int64_t)b * L + l - 1;
        const int shift_of = a.m[row0 * S + (lane < S ? lane : S - 1)];
        const bool ok = lane < S && shift_of <= budget && shift_of <= start + kCols - 1;
        const uint64_t votes = __builtin_amdgcn_ballot_w64(ok);
        const int n = __builtin_popcountll(votes), below = __builtin_popcountll(votes & ((1ull << lane) - 1ull));
        const int to = (ok ? below : n + lane - below) * 4;    // (every lane has a place of its own)
        const int id = __builtin_amdgcn_ds_permute(to, lane), shift = __builtin_amdgcn_ds_permute(to, shift_of);
        const int64_t c_of = l == 1 ? a.c[row0 * S + (id < S ? id : S - 1)] : 0;
        if (wave == 0) {
            bool there = true;
            if (l > 1 && n > 0) {
                // the blocks from the largest memory's shift to the smallest one's, but for the own one
                const int sh_lo = (int)wave_min(ok ? (uint32_t)shift_of : ~0u), sh_hi = (int)~wave_min(ok ? ~(uint32_t)shift_of : ~0u);
                there = chain_wait(flags, max(start - sh_hi, 0) / kCols, min((start + kCols - 1 - sh_lo) / kCols, t - 1), l - 1);
            }
            if (lane == 0) ready[l & 1] = there ? 1 : 0;
        }
        __syncthreads();
        if (uniform(ready[l & 1]) == 0) {
            a.status[b] = GALV_INSTANCE_GAVE_UP;
            return;
        }
        uint64_t row[TS][TE];
        const __amdgpu_buffer_rsrc_t rows = chain_buffer(chain_rows<uint64_t>(a, b, l - 1));
#pragma unroll
        for (int r = 0; r < TS; ++r) {
            const int i = wave + NG * r;
            if (i >= n) continue;
            const int sh = (int)read_lane((uint32_t)shift, i);
            const uint32_t first = read_lane((uint32_t)id, i) * pitch;
            if (l == 1) {
                const uint64_t cp = read_lane((uint64_t)c_of, i);
#pragma unroll
                for (int j = 0; j < TE; ++j) row[r][j] = e0 + j >= sh ? cp : (uint64_t)kInf;
            } else if (start >= sh) {
                buffer_cells(rows, lane_off, (first + (uint32_t)(start - sh)) * 8, row[r]);
            } else {
#pragma unroll
                for (int j = 0; j < TE; ++j)
                    row[r][j] = __builtin_bit_cast(uint64_t, __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(
                                    rows, max(e0 + j - sh, 0) * 8, (int)(first * 8), kAgent)));
#pragma unroll
                for (int j = 0; j < TE; ++j)
                    if (e0 + j < sh) row[r][j] = (uint64_t)kInf;
            }
        }
#pragma unroll
        for (int r = 0; r < TS; ++r)
            if (wave + NG * r < n) shared[(wave + NG * r) * kWave + lane] = cell2{row[r][0], row[r][1]};
        __syncthreads();
        int64_t best[TS][TE];
        int32_t arg[TS][TE];
#pragma unroll
        for (int s = 0; s < TS; ++s)
#pragma unroll
            for (int j = 0; j < TE; ++j) {
                best[s][j] = kInf;
                arg[s][j] = -1;
            }
        const int r_sel = a.r_idx ? a.r_idx[row0 + 1] : 0;
        const ConstPtr<int64_t> R = as_const(a.R + ((int64_t)b * a.nR + r_sel) * S * S);
        constexpr int kAhead = 4;                  // (the last row repeated: that changes no minimum)
        for (int i0 = 0; i0 < (s0 < S ? n : 0); i0 += kAhead) {
            int64_t rk[kAhead][TS];
            cell2 v[kAhead];
            int sp[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int i = min(i0 + u, n - 1);
                sp[u] = (int)read_lane((uint32_t)id, i);
                v[u] = shared[i * kWave + lane];
#pragma unroll
                for (int s = 0; s < TS; ++s) rk[u][s] = R[sp[u] * S + min(s0 + s, S - 1)];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int s = 0; s < TS; ++s)
#pragma unroll
                    for (int j = 0; j < TE; ++j) {
                        const int64_t x = (int64_t)v[u][j] + rk[u][s];
                        if (x < best[s][j]) {      // strict: lowest s' keeps ties
                            best[s][j] = x;
                            arg[s][j] = sp[u];
                        }
                    }
        }
        const __amdgpu_buffer_rsrc_t out = chain_buffer(chain_rows<uint64_t>(a, b, l) + (int64_t)s0 * pitch + start);
        int32_t *bp = static_cast<int32_t *>(a.bp) + (((int64_t)b * (L - 1) + (l - 1)) * S + s0) * pitch + e0;
#pragma unroll
        for (int s = 0; s < TS; ++s)
            if (s0 + s < S) {
                const int64_t cs = a.c[(row0 + 1) * S + s0 + s];
                uint64_t cell[TE];
                arg2 from;
#pragma unroll
                for (int j = 0; j < TE; ++j) {
                    const bool dead = best[s][j] >= kInf;
                    cell[j] = (uint64_t)(dead ? kInf : best[s][j] + cs);
                    from[j] = dead ? -1 : arg[s][j];
                }
                buffer_store_cells(out, lane_off, (uint32_t)s * pitch * 8, cell);
                *reinterpret_cast<arg2 *>(bp + (int64_t)s * pitch) = from;
            }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the cells have arrived
        __syncthreads();
        if (wave == 0 && lane == 0) agent_store(flags + (int64_t)t * kWordStep, l);
    }
}

// min over s at e = budget, lowest s first, by the wave that has an instance's last place: a lane per strategy.
__device__ __forceinline__ void chain_final(const Layout &a, int b, int st, bool packed, int budget, int64_t *best_cost, int32_t *best_last) {
    const int lane = lane_id();
    const int L = a.L, S = a.S;
    const int32_t *h = a.hdr + ((int64_t)b * L + (L - 1)) * 8;
    uint64_t v = (uint64_t)kInf;                   // this lane's cost
    if (st >= 0) {
        const int e = budget - a.m[((int64_t)b * L + (L - 1)) * S + (lane < S ? lane : S - 1)];
        int y = 0, x = budget;
        bool there = true;
        if (packed) {
            y = uniform(h[5]);
            x = uniform(agent_load(h + 6));
            there = chain_last_column(h + 6, x);
        }
        const bool ok = there && lane < S && e >= y && y <= x;
        const int at = min(e, x);
        if (__builtin_amdgcn_ballot_w64(ok) != 0) {
            const int lo = (int)wave_min(ok ? (uint32_t)at : ~0u), hi = (int)~wave_min(ok ? ~(uint32_t)at : ~0u);
            there = chain_wait(chain_flags(a, b), lo / kChainCols, hi / kChainCols, L - 1);
            const int64_t cell = (int64_t)(lane < S ? lane : 0) * a.e_pad + (ok ? at : lo);
            if (packed && st == GALV_INSTANCE_OK_FAST_U32) {
                const uint32_t narrow = agent_load(chain_rows<uint32_t>(a, b, L - 1) + cell);
                if (ok && there && narrow < kInf32) v = narrow;
            } else {
                const uint64_t wide = agent_load(chain_rows<uint64_t>(a, b, L - 1) + cell);
                if (ok && there && wide < (uint64_t)kInf) v = wide;
            }
        }
        if (!there) a.status[b] = GALV_INSTANCE_GAVE_UP;
    }
    const uint64_t least = wave_min(v);
    const int last = least < (uint64_t)kInf ? __builtin_ctzll(__builtin_amdgcn_ballot_w64(v == least)) : -1;
    if (lane == 0) {
        best_cost[b] = (int64_t)least;
        best_last[b] = last;
        a.last[b] = last;
    }
}

// (4 waves per SIMD at least: no vector register is spilled)
template <int TS, int NG>
__global__ __launch_bounds__(NG * kWave, 4) void chain_kernel(Layout a, int64_t *best_cost, int32_t *best_last) {
    const int wave = uniform(threadIdx.x >> 6);
    if (wave == 0 && lane_id() == 0) lds_cells[0] = (uint32_t)atomicAdd(chain_words(a), 1);
    __syncthreads();
    const int place = uniform((int)lds_cells[0]);
    __syncthreads();
    // (block -1: the places of the unlimited recurrence; block n_tiles: those of the final minimum)
    const int b = place % a.B, t = place / a.B - 1;
    // (all that is needed first in one round trip)
    ChainIn in;
    chain_load<TS, NG>(a, wave, b, 1, in);
    // layer 0's costs, in the order of its list
    const uint64_t c0 = (a.vcost + (int64_t)b * a.L * (TS * NG))[(uint32_t)(lane_id() < TS * NG ? lane_id() : TS * NG - 1)];
    const int st = (int)read_lane((uint32_t)in.h, 0), budget = (int)read_lane((uint32_t)in.h, 1);
    const uint32_t dmax = read_lane((uint32_t)in.h, 3);
    const bool keys32 = st == GALV_INSTANCE_OK_FAST_U32 || st == GALV_INSTANCE_OK_U32_WIDE;
    const bool packed = byte_status(a, st, dmax);
    if (t == a.n_tiles) {
        if (wave == 0) chain_final(layout_again(), b, st, packed, budget, best_cost, best_last);
        return;
    }
    if (st < 0 || t * kChainCols > budget) return;
    if (t < 0) {
        if (!packed || wave != 0) return;
        if (keys32)
            chain_live<TS * NG, Key32>(layout_again(), b, dmax, budget);
        else if (dmax != 0)
            chain_live<TS * NG, Key64>(layout_again(), b, dmax, budget);
        else
            chain_live<TS * NG, KeyBig>(layout_again(), b, chain_clamps(layout_again())[b], budget);
    } else if (st == GALV_INSTANCE_OK_FAST_U32) {
        chain_tiles<TS, NG, uint32_t, Key32>(layout_again(), wave, b, t, dmax, in, c0);
    } else if (packed && keys32) {
        chain_tiles<TS, NG, uint64_t, Key32>(layout_again(), wave, b, t, dmax, in, c0);
    } else if (packed && dmax != 0) {
        chain_tiles<TS, NG, uint64_t, Key64>(layout_again(), wave, b, t, dmax, in, c0);
    } else if (packed) {
        chain_tiles<TS, NG, uint64_t, KeyBig>(layout_again(), wave, b, t, chain_clamps(layout_again())[b], in, c0);
    } else {
        chain_int64<TS, NG>(layout_again(), wave, b, t, budget);
    }
}
constexpr unsigned chain_lds(int ts, int ng) {
    // minima of 8-byte cells, alive rows, transition keys of 8 bytes and relative costs, or keys of relative costs, X_l, rows to
    // read.  (More than the whole rows of chain_int64.)
    const int rows = ts * ng, cols = kChainCols;
    const int small = rows * rows * 8 + rows * cols * 4, big = rows * cols * 8;
    return (unsigned)(2 * cols * 8 + 2 * 8 + (small > big ? small : big) + 8 + rows * 8 + 8);
}

// ------------------------------------------------- final minimum and backtrack

// C[L-1][e][s] from the un-shifted last row, as an integer (GALV_INF if none).
__device__ __forceinline__ int64_t last_layer_cost(const Layout &a, int b, int st, int64_t e,
                                                   int64_t s) {
    const int64_t shift = a.m[((int64_t)b * a.L + (a.L - 1)) * a.S + s];
    if (shift > e) return kInf;
    if (a.packed == kChain && !is_packed(a, st, b)) return chain_rows<int64_t>(a, b, a.L - 1)[s * a.e_pad + e - shift];
    if (is_packed(a, st, b)) {
        const int32_t *h = a.hdr + ((int64_t)b * a.L + (a.L - 1)) * 8;
        if (e - shift < h[5]) return kInf;
        const int64_t x = e - shift < h[6] ? e - shift : h[6];
        if (a.packed == kChain) {
            const int64_t at = s * a.e_pad + x;
            if (st == GALV_INSTANCE_OK_FAST_U32) return Narrow::to_int64(chain_rows<uint32_t>(a, b, a.L - 1)[at], a.k_bits);
            const uint64_t v = chain_rows<uint64_t>(a, b, a.L - 1)[at];
            return v >= (uint64_t)kInf ? kInf : (int64_t)v;
        }
        const PackTables t = pack_tables(a, (a.L - 1) & 1, b);
        const uint32_t sp = byte_rows(a, b, a.L - 1)[(int64_t)s * a.e_pad + x];
        const bool keys32 = st == GALV_INSTANCE_OK_FAST_U32 || st == GALV_INSTANCE_OK_U32_WIDE;
        const int64_t cmin = st == GALV_INSTANCE_OK_FAST_U32 ? (int64_t)reinterpret_cast<const uint32_t *>(t.cmin)[x]
                                                             : (int64_t)reinterpret_cast<const uint64_t *>(t.cmin)[x];
        const uint64_t at = (uint64_t)sp * (uint32_t)a.S_pad + (uint32_t)s;
        const uint64_t r = keys32 ? Key32::cost(rkeys<uint32_t>(a, b, h[4])[at], a.k_bits)
                                  : Key64::cost(rkeys<double>(a, b, h[4])[at], a.k_bits);
        // (c(l, s) from the solve's own copy: the caller's costs may be gone by the time an optimum is asked for)
        const uint64_t cs = a.ck[((int64_t)b * a.L + (a.L - 1)) * a.S_pad + s];
        return cmin + (int64_t)t.rel[(int64_t)sp * a.e_pad + x] + (int64_t)r + (int64_t)cs;
    }
    const char *U = a.U[(a.L - 1) & 1] + ((int64_t)b * a.S_pad + s) * a.row * 8;
    const int64_t x = a.lead + e - shift;
    if (narrow_cells(st))
        return Narrow::to_int64(reinterpret_cast<const uint32_t *>(U)[x], a.k_bits);
    if (st == GALV_INSTANCE_OK_FAST_WIDE)
        return Wide::to_int64(reinterpret_cast<const double *>(U)[x], a.k_bits);
    if (st == GALV_INSTANCE_OK_U32_WIDE) {
        const uint64_t v = reinterpret_cast<const uint64_t *>(U)[x];
        return v >= (uint64_t)kInf ? kInf : (int64_t)v;
    }
    return reinterpret_cast<const int64_t *>(U)[x];
}

// min_s C[L-1][e][s] and the lowest minimising s for one (instance, budget column), by a whole wave:
// a lane per strategy, so that the dependent loads of a cell (argmin, relative cost) are waited for once.
__device__ __forceinline__ void best_at_wave(const Layout &a, int b, int st, int64_t e, int64_t &opt, int32_t &last) {
    opt = kInf;
    last = -1;
    for (int s = lane_id(); s < a.S; s += kWave) {
        const int64_t v = last_layer_cost(a, b, st, e, s);
        if (v < opt) {
            opt = v;
            last = s;
        }
    }
#pragma unroll
    for (int w = kWave / 2; w > 0; w >>= 1) {
        const int64_t v = (int64_t)__shfl_xor((long long)opt, w, kWave);
        const int32_t s = __shfl_xor(last, w, kWave);
        if (v < opt || (v == opt && (uint32_t)s < (uint32_t)last)) {   // (-1, nothing reachable, is the largest)
            opt = v;
            last = s;
        }
    }
}

// One wave per instance: min over s at e = budget, lowest s first.
__global__ __launch_bounds__(kWave) void final_kernel(Layout a, int64_t *best_cost, int32_t *best_last) {
    const int b = blockIdx.x;
    const int st = uniform(a.status[b]);
    int64_t opt = kInf;
    int32_t last = -1;
    if (st >= 0) best_at_wave(a, b, st, uniform(a.budget[b]), opt, last);
    if (threadIdx.x == 0) {
        best_cost[b] = opt;
        best_last[b] = last;
        a.last[b] = last;
        // every block of init_kernel has long finished: safe to record what the leads hold
        // (an instance with the byte table keeps other things there)
        a.lead_mode[b] = st < 0 || is_packed(a, st, b) ? 0 : lead_kind(st);
    }
}

// Walk the un-shifted argmin table of instance b from (L-1, e, s) down to layer 0, where
// there are more strategies than walk_wave takes: L dependent loads.  Writes the plan, or
// all -1 when s < 0.
__device__ __forceinline__ void walk_plan(const Layout &a, int b, int64_t e, int s, int32_t *out) {
    if (s < 0) {
        for (int l = 0; l < a.L; ++l) out[l] = -1;
        return;
    }
    for (int l = a.L - 1; l >= 1; --l) {
        out[l] = s;
        e -= a.m[((int64_t)b * a.L + l) * a.S + s];
        // A reachable cell always points at a reachable cell; the guard only keeps
        // the walk inside the table if that invariant were ever broken.
        if (e < 0 || e > a.E_max) {
            for (int q = 0; q < a.L; ++q) out[q] = -1;
            return;
        }
        s = load_bp(a, false, b, l, s, e);         // (more strategies than a byte table has)
        if (s < 0 || s >= a.S) {
            for (int q = 0; q < a.L; ++q) out[q] = -1;
            return;
        }
    }
    out[0] = s;
}

// The same walk by a whole wave, two layers per round trip.  The column that layer l - 1 is left at
// depends on layer l's choice but not on layer l - 1's own, so while the argmin that names strategy
// s' of layer l - 1 is under way, lane s' already fetches the argmin that s' would lead to; memories and
// column ranges of the next two layers are fetched meanwhile.  S <= 64 * Q.
// (Before, one dependent load per layer after a copy of the memory table to LDS: 29 strategies x 37 layers
// 22 -> 21 us, 44 x 48 x 16 instances 37 -> 30 us; 32 queries of 22 x 24, once a thread each, 37 -> 15 us.)
template <int Q>
__device__ __forceinline__ void walk_wave(const Layout &a, bool packed, int b, int64_t e0, int s, int32_t *out) {
    const int lane = lane_id();
    const int S = a.S, L = a.L;
    const int32_t *m = a.m + (int64_t)b * L * S;
    const int32_t *hdr = a.hdr + (int64_t)b * L * 8;
    const int64_t bp0 = (int64_t)b * (L - 1) * S * a.e_pad;
    struct Row {                                   // of one layer: memories, and the columns the byte table holds
        int m[Q];
        int y, x;
    };
    auto load = [&](int l, Row &r) {
        l = l > 0 ? l : 0;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int sx = q * kWave + lane;
            r.m[q] = m[(int64_t)l * S + (sx < S ? sx : S - 1)];
        }
        r.y = packed ? hdr[l * 8 + 5] : 0;
        r.x = packed ? hdr[l * 8 + 6] : 0x7fffffff;
    };
    auto cell = [&](int l, const Row &r, int sx, int x) -> int {   // layer l >= 1, a column of the table
        const int64_t at = bp0 + ((int64_t)(l - 1) * S + sx) * a.e_pad;
        if (packed) return x < r.y ? -1 : (int)byte_rows(a, b, l)[(int64_t)sx * a.e_pad + (x < r.x ? x : r.x)];
        if (a.bp_u8) {
            const uint8_t v = static_cast<const uint8_t *>(a.bp)[at + x];
            return v == 0xFF ? -1 : (int)v;
        }
        return static_cast<const int32_t *>(a.bp)[at + x];
    };
    auto pick = [&](const int (&v)[Q], int sx) {   // strategy sx's value, wave-uniform
        int r = __builtin_amdgcn_readlane(v[0], sx & (kWave - 1));
#pragma unroll
        for (int q = 1; q < Q; ++q) {
            const int o = __builtin_amdgcn_readlane(v[q], sx & (kWave - 1));
            if (sx >> 6 == q) r = o;
        }
        return r;
    };
    int e = uniform((int)e0);
    s = uniform(s);
    int l = L - 1;
    Row now, below;
    load(l, now);
    load(l - 1, below);
    // A reachable cell always points at a reachable cell; the guards only keep the walk inside the
    // table if that invariant were ever broken.
    while (s >= 0 && l >= 1) {
        const int x = e - pick(now.m, s);
        if (x < 0 || x > a.E_max) {
            s = -1;
            break;
        }
        const int first = cell(l, now, s, x);
        int second[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int sx = q * kWave + lane, x2 = x - below.m[q];
            second[q] = l >= 2 && sx < S && x2 >= 0 && x2 <= a.E_max ? cell(l - 1, below, sx, x2) : -1;
        }
        Row next, next_below;
        load(l - 2, next);
        load(l - 3, next_below);
        if (lane == 0) out[l] = s;
        s = uniform(first);
        if (s < 0 || s >= S) {
            s = -1;
            break;
        }
        if (--l == 0) break;
        if (lane == 0) out[l] = s;
        e = x - pick(below.m, s);
        s = pick(second, s);
        if (s < 0 || s >= S) {
            s = -1;
            break;
        }
        --l;
        now = next;
        below = next_below;
    }
    if (s < 0)
        for (int q = lane; q < L; q += kWave) out[q] = -1;
    else if (lane == 0)
        out[0] = s;
}
__device__ __forceinline__ void walk_any(const Layout &a, int b, int64_t e, int s, int32_t *out) {
    const int st = uniform(a.status[b]);
    const bool packed = is_packed(a, st, b);
    if (st < 0) s = -1;                            // (no table to walk)
    if (a.S <= kWave)
        walk_wave<1>(a, packed, b, e, s, out);
    else if (a.S <= 4 * kWave)
        walk_wave<4>(a, packed, b, e, s, out);
    else if (lane_id() == 0)
        walk_plan(a, b, e, s, out);
}

// Per instance: the tiles' (rows reduced, rows listed) summed over the tiles within the budget
// and the layers; zeros for an instance that is not on the 32-bit-key path.
__global__ __launch_bounds__(kThreads) void stats_kernel(Layout a, int64_t *out) {
    const int b = blockIdx.x;
    __shared__ unsigned long long red[3][kThreads];
    unsigned long long done = 0, listed = 0, fetched = 0;
    if (a.status[b] == GALV_INSTANCE_OK_FAST_U32 || a.status[b] == GALV_INSTANCE_OK_U32_WIDE) {
        const int nt = a.budget[b] / a.tile_e + 1;
        for (int64_t i = threadIdx.x; i < (int64_t)(a.L - 1) * nt; i += kThreads) {
            if (a.packed) {                        // only the layer's tiles in its header's range are swept
                const int32_t *h = a.hdr + ((int64_t)b * a.L + i / nt + 1) * 8;
                if (h[5] > h[6] || i % nt < h[5] / a.tile_e || i % nt > h[6] / a.tile_e) continue;
            }
            const uint32_t *v = a.stats + 2 * (((int64_t)b * (a.L - 1) + i / nt) * a.n_tiles + i % nt);
            done += v[0] >> 16;
            listed += v[0] & 0xffffu;
            fetched += v[1];
        }
    }
    red[0][threadIdx.x] = done;
    red[1][threadIdx.x] = listed;
    red[2][threadIdx.x] = fetched;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) out[3 * b + q] = (int64_t)red[q][0];
}

// One wave per instance, from the full budget and the stored best last strategy.
__global__ __launch_bounds__(kWave) void backtrack_kernel(Layout a, int32_t *plan) {
    const int b = blockIdx.x;
    walk_any(a, b, a.budget[b], a.last[b], plan + (int64_t)b * a.L);
}

// min_s C[L-1][e][s] and the lowest minimising s for one (instance, budget column).
__device__ __forceinline__ void best_at(const Layout &a, int b, int st, int64_t e, int64_t &opt,
                                        int32_t &last) {
    opt = kInf;
    last = -1;
    for (int s = 0; s < a.S; ++s) {
        const int64_t v = last_layer_cost(a, b, st, e, s);
        if (v < opt) {
            opt = v;
            last = s;
        }
    }
}
// The same from the byte table: no branch per strategy, so that the two dependent loads of several cells are
// under way together (8 x 20002 columns x 22 strategies took 27 us with the branches).
template <class Cell, class Key>
__device__ __forceinline__ void best_at_bytes(const Layout &a, int b, int e, int64_t &opt, int32_t &last) {
    const int32_t *h = a.hdr + ((int64_t)b * a.L + (a.L - 1)) * 8;
    const int y = h[5], top = h[6];
    opt = kInf;
    last = -1;
    if (y > top) return;                           // nothing reachable, nothing stored
    const PackTables t = pack_tables(a, (a.L - 1) & 1, b);
    const uint8_t *bp = byte_rows(a, b, a.L - 1);
    const Cell *cmin = reinterpret_cast<const Cell *>(t.cmin);
    const typename Key::T *R = rkeys<typename Key::T>(a, b, h[4]);
    const int32_t *m = a.m + ((int64_t)b * a.L + (a.L - 1)) * a.S;
    const uint64_t *c = a.ck + ((int64_t)b * a.L + (a.L - 1)) * a.S_pad;    // (not the caller's: see last_layer_cost)
    const int mask = (1 << a.k_bits) - 1;
#pragma unroll 4
    for (int s = 0; s < a.S; ++s) {
        const int at = e - m[s];
        const bool ok = at >= y;                   // (memories are not negative, and y is not)
        const int x = ok && at < top ? at : top;
        const uint32_t sp = bp[(int64_t)s * a.e_pad + x] & (uint32_t)mask;
        const uint32_t in = sp < (uint32_t)a.S ? sp : 0;        // (bytes of unreachable columns may be anything)
        const int64_t v = (int64_t)cmin[x] + (int64_t)t.rel[(int64_t)in * a.e_pad + x] +
                          (int64_t)Key::cost(R[(int64_t)in * a.S_pad + s], a.k_bits) + (int64_t)c[s];
        if (ok && v < opt) {
            opt = v;
            last = s;
        }
    }
}

// The same from the rows of the chained sweep.
template <class Cell>
__device__ __forceinline__ void best_at_rows(const Layout &a, int b, int e, int64_t &opt, int32_t &last) {
    constexpr Cell kInfCell = sizeof(Cell) == 8 ? (Cell)kInf : (Cell)kInf32;
    const int32_t *h = a.hdr + ((int64_t)b * a.L + (a.L - 1)) * 8;
    const int y = h[5], top = h[6];
    opt = kInf;
    last = -1;
    if (y > top) return;                           // nothing reachable, nothing stored
    const Cell *rows = chain_rows<Cell>(a, b, a.L - 1);
    const int32_t *m = a.m + ((int64_t)b * a.L + (a.L - 1)) * a.S;
    Cell least = kInfCell;
#pragma unroll 4
    for (int s = 0; s < a.S; ++s) {
        const int at = e - m[s];
        const bool ok = at >= y;                   // (memories are not negative, and y is not)
        const Cell v = rows[(int64_t)s * a.e_pad + (ok && at < top ? at : top)];
        if (ok && v < least) {
            least = v;
            last = s;
        }
    }
    if (last >= 0) opt = (int64_t)least;
}

// The optimum of every budget column.  Grid: (column tiles, B).
__global__ __launch_bounds__(kThreads) void best_per_budget_kernel(Layout a, int64_t *best_cost,
                                                                   int32_t *best_last) {
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e > a.E_max) return;
    const int b = blockIdx.y;
    const int st = uniform(a.status[b]);
    int64_t opt = kInf;
    int32_t last = -1;
    if (st >= 0 && e <= a.budget[b]) {
        if (!is_packed(a, st, b))
            best_at(a, b, st, e, opt, last);
        else if (a.packed == kChain && st == GALV_INSTANCE_OK_FAST_U32)
            best_at_rows<uint32_t>(a, b, (int)e, opt, last);
        else if (a.packed == kChain)
            best_at_rows<uint64_t>(a, b, (int)e, opt, last);
        else if (st == GALV_INSTANCE_OK_FAST_U32)
            best_at_bytes<uint32_t, Key32>(a, b, (int)e, opt, last);
        else if (st == GALV_INSTANCE_OK_U32_WIDE)
            best_at_bytes<uint64_t, Key32>(a, b, (int)e, opt, last);
        else
            best_at_bytes<uint64_t, Key64>(a, b, (int)e, opt, last);
    }
    best_cost[(int64_t)b * (a.E_max + 1) + e] = opt;
    if (best_last) best_last[(int64_t)b * (a.E_max + 1) + e] = last;
}

// One wave per (instance, budget) query: final minimum at that column, then the walk.
__global__ __launch_bounds__(kWave) void backtrack_queries_kernel(Layout a, int n, const int32_t *inst,
                                                                  const int32_t *budgets, int64_t *cost,
                                                                  int32_t *plan) {
    for (int64_t q = blockIdx.x; q < n; q += gridDim.x) {
        const int b = uniform(inst[q]);
        const int64_t e = uniform(budgets[q]);
        int64_t opt = kInf;
        int32_t last = -1;
        if (b >= 0 && b < a.B) {
            const int st = uniform(a.status[b]);
            if (st >= 0 && e >= 0 && e <= a.budget[b]) best_at_wave(a, b, st, e, opt, last);
        }
        if (cost && threadIdx.x == 0) cost[q] = opt;
        walk_any(a, b < 0 || b >= a.B ? 0 : b, e, last, plan + q * a.L);
    }
}

// Canonical-order tables of one instance.  Grid: (e tiles, L + 1); row L of the
// grid writes C_last, rows 0..L-1 write the back-pointers of that layer.
__global__ __launch_bounds__(kThreads) void export_kernel(Layout a, int b, int64_t *C_last,
                                                          int32_t *bp_out) {
    const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (e > a.E_max) return;
    const int l = blockIdx.y;
    const int st = uniform(a.status[b]);
    const int budget = uniform(a.budget[b]);
    const bool live = st >= 0 && e <= budget;
    const bool packed = is_packed(a, st, b);
    if (l == a.L) {
        for (int s = 0; s < a.S; ++s)
            C_last[e * a.S + s] = live ? last_layer_cost(a, b, st, e, s) : kInf;
        return;
    }
    if (!bp_out) return;
    int32_t *dst = bp_out + ((int64_t)l * (a.E_max + 1) + e) * a.S;
    for (int s = 0; s < a.S; ++s) {
        int32_t v = -1;
        if (live && l >= 1) {
            const int64_t shift = a.m[((int64_t)b * a.L + l) * a.S + s];
            if (shift <= e)
                v = load_bp(a, packed, b, l, s, e - shift);
        }
        dst[s] = v;
    }
}

// -------------------------------------------------------------------- host side

// Sweep variants, in ascending order of the strategies one workgroup covers
// (TS * NG).  The first one that covers S is used; larger S use the last one with
// several strategy groups along grid.y.  <TS, TE, NG, WPE, W, UX, SHARE>: TS * TE running
// minima per lane (2 VGPRs each with 64-bit keys, 1 with 32-bit keys) for WPE resident
// waves per SIMD (512 VGPRs / WPE each), W waves per workgroup, UX times the columns for
// the 32-bit-key body, SHARE = 1 for the row-sharing 32-bit-key body (W == NG waves, each
// owning TS rows and TS strategies of one tile of 64 * TE * UX columns; it needs
// TS * NG >= S, so the last variant, which serves any S, uses the plain body; the one before
// it covers up to 256 strategies with 16-wave workgroups).
// Measured over cost rows: tiles of 128 columns beat 64 (longer contiguous row segments) while larger register
// tiles gain nothing; 8 waves per SIMD do not build for TS = 16 (the compiler then spills scalar
// registers that a hand-issued load still targets, which the build refuses).
#ifndef GALV_V0
#define GALV_V0 8, 2, 1, 8, 1, 1, 1
#endif
#ifndef GALV_V1
#define GALV_V1 16, 2, 1, 6, 1, 1, 1
#endif
#ifndef GALV_V2
#define GALV_V2 11, 2, 2, 8, 2, 1, 1
#endif
#ifndef GALV_V3
#define GALV_V3 16, 2, 2, 6, 2, 1, 1
#endif
#ifndef GALV_V4
#define GALV_V4 11, 2, 4, 8, 4, 1, 1
#endif
#ifndef GALV_V5
#define GALV_V5 16, 2, 4, 6, 4, 1, 1
#endif
#ifndef GALV_V6
#define GALV_V6 16, 2, 8, 6, 8, 1, 1
#endif
#ifndef GALV_V7
#define GALV_V7 16, 2, 16, 4, 16, 1, 1
#endif
#ifndef GALV_V8
#define GALV_V8 16, 2, 8, 6, 8, 1, 0
#endif
// Twins with tiles of 256 budget columns (UX = 2: four columns per lane) and fewer, fatter waves,
// for launches that fill the chip anyway: what a tile costs beside its min-plus arithmetic (its
// chain of round trips, its addresses and bookkeeping) is spread over twice the states, for half the
// rows in its list.  Which launches take them, and what both shapes measured, stands in make_plan.  (Up to 32
// strategies only cost rows take them by themselves; over the byte table they have to be asked for.)
#ifndef GALV_V2X
#define GALV_V2X 11, 2, 2, 5, 2, 2, 1
#endif
#ifndef GALV_V3X
#define GALV_V3X 16, 2, 2, 4, 2, 2, 1
#endif
#ifndef GALV_V4X
#define GALV_V4X 11, 2, 4, 5, 4, 2, 1
#endif
#ifndef GALV_V5X
#define GALV_V5X 16, 2, 4, 4, 4, 2, 1
#endif
#ifndef GALV_V6X
#define GALV_V6X 16, 2, 8, 4, 8, 2, 1
#endif
#ifndef GALV_V7X
#define GALV_V7X 16, 2, 16, 4, 16, 2, 1
#endif
// Twins with the plain shape's tiles and more, thinner waves, for launches that leave wavefront slots idle: a
// tile's time is then a chain of round trips, two per row that a wave rebuilds or one per row that it
// loads, and of the additions of the strategies it owns, and more waves shorten both.
#ifndef GALV_S0
#define GALV_S0 2, 2, 4, 8, 4, 1, 1
#endif
#ifndef GALV_S1
#define GALV_S1 4, 2, 4, 8, 4, 1, 1
#endif
#ifndef GALV_S2
#define GALV_S2 6, 2, 4, 8, 4, 1, 1
#endif
#ifndef GALV_S3
#define GALV_S3 8, 2, 4, 8, 4, 1, 1
#endif
#ifndef GALV_S4
#define GALV_S4 6, 2, 8, 8, 8, 1, 1
#endif
#ifndef GALV_S5
#define GALV_S5 8, 2, 8, 8, 8, 1, 1
#endif
#ifndef GALV_S6
#define GALV_S6 8, 2, 16, 8, 16, 1, 1
#endif
#ifndef GALV_F2
#define GALV_F2 3, 2, 8, 8, 8, 1, 1
#endif
#ifndef GALV_F3
#define GALV_F3 4, 2, 8, 8, 8, 1, 1
#endif

// ---------------------------------------------------------------------------------------------
// Outer loop of Algorithm 1 over a window of batch sizes: per (batch size, pipeline degree) the
// stage optima are summed, the minimum over pipeline degrees is C_opt, and the scan over batch
// sizes keeps the largest B / C_opt until the first batch size that fits under no degree.
// One workgroup: the sums in parallel, the scan by one lane (it is a dependent chain).
struct PpList {
    int n;
    int degree[kMaxPp];
};

__global__ __launch_bounds__(kThreads) void alg1_reduce_kernel(
    int n_batch, PpList pp, const int64_t *__restrict__ stage_cost,
    const int64_t *__restrict__ batch_size, int batch_index_base, int first_window,
    int64_t *__restrict__ c_p, galv_alg1_state_t *__restrict__ state) {
    for (int i = threadIdx.x; i < n_batch * pp.n; i += kThreads) {
        const int ib = i / pp.n, ip = i % pp.n;
        size_t off = 0;
        for (int j = 0; j < ip; ++j) off += (size_t)n_batch * pp.degree[j];
        const int64_t *x = stage_cost + off + (size_t)ib * pp.degree[ip];
        int64_t acc = 0;
        for (int st = 0; st < pp.degree[ip]; ++st) {
            const int64_t v = x[st];
            acc = (acc >= kInf || v < 0 || v >= kInf - acc) ? kInf : acc + v;
        }
        c_p[i] = acc;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    galv_alg1_state_t s;
    if (first_window) {
        s.batch_size = 0; s.cost = 1; s.pp_index = -1; s.batch_index = -1;
        s.stopped = 0; s.n_explored = 0;
    } else {
        s = *state;
    }
    for (int ib = 0; ib < n_batch && !s.stopped; ++ib) {
        int64_t c_opt = kInf;
        int arg = -1;
        for (int ip = 0; ip < pp.n; ++ip) {
            const int64_t v = c_p[(size_t)ib * pp.n + ip];
            if (v < c_opt) { c_opt = v; arg = ip; }
        }
        if (arg < 0) { s.stopped = 1; break; }          // Out-Of-Memory under every degree
        ++s.n_explored;
        const int64_t bsz = batch_size[ib];
        // bsz / c_opt > s.batch_size / s.cost, compared exactly as cross products
        const unsigned __int128 lhs = (unsigned __int128)(uint64_t)bsz * (uint64_t)s.cost;
        const unsigned __int128 rhs = (unsigned __int128)(uint64_t)s.batch_size * (uint64_t)c_opt;
        if (bsz > 0 && lhs > rhs) {
            s.batch_size = bsz; s.cost = c_opt; s.pp_index = arg;
            s.batch_index = batch_index_base + ib;
        }
    }
    *state = s;
}


// ---------------------------------------------------------------------------------------------
// Coarse-grained exploration (complexity remark at the end of section 3.3): `fuse` consecutive
// layers become one layer that runs a single strategy, and memory is counted in units `gran`
// times larger.  One thread per (instance, fused layer, strategy).
__global__ __launch_bounds__(kThreads) void coarsen_kernel(
    int B, int L, int S, int nR, int fuse, int gran, int Lc, const int64_t *__restrict__ c,
    const int32_t *__restrict__ m, const int64_t *__restrict__ R, const int32_t *__restrict__ r_idx,
    const int32_t *__restrict__ budget, int64_t *__restrict__ c_out, int32_t *__restrict__ m_out,
    int32_t *__restrict__ r_idx_out, int32_t *__restrict__ budget_out) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= (int64_t)B * Lc * S) return;
    const int s = (int)(i % S);
    const int j = (int)((i / S) % Lc);
    const int b = (int)(i / ((int64_t)S * Lc));
    const int lo = j * fuse, hi = min(L, lo + fuse);
    const int E = budget[b];
    int64_t cost = 0, mem = 0;
    bool unusable = false, bad_c = false, bad_m = false;   // invalid inputs stay invalid for the solver
    for (int l = lo; l < hi; ++l) {
        const int64_t at = ((int64_t)b * L + l) * S + s;
        const int64_t cl = c[at];
        bad_c |= cl < 0 || cl >= kInf;
        cost += bad_c ? 0 : cl;
        if (l > lo) {
            const int r = r_idx ? r_idx[(int64_t)b * L + l] : 0;
            const int64_t rr = (r < 0 || r >= nR) ? -1 : R[(((int64_t)b * nR + r) * S + s) * S + s];
            bad_c |= rr < 0 || rr >= kInf;
            cost += bad_c ? 0 : rr;
        }
        bad_c |= cost >= kInf;
        const int32_t ml = m[at];
        bad_m |= ml < 0;
        unusable |= ml > E;
        mem += ml;
    }
    const int64_t units = (mem + gran - 1) / gran;       // rounded up: a coarse plan that fits, fits
    const int32_t Ec = E < 0 ? -1 : E / gran;
    const int32_t over = Ec < INT32_MAX ? Ec + 1 : INT32_MAX;
    c_out[i] = bad_c ? -1 : cost;
    m_out[i] = bad_m ? -1 : ((unusable || units > Ec) ? over : (int32_t)units);
    if (s == 0) {
        r_idx_out[(int64_t)b * Lc + j] = r_idx ? r_idx[(int64_t)b * L + lo] : 0;
        if (j == 0) budget_out[b] = Ec;
    }
}

__global__ __launch_bounds__(kThreads) void expand_plan_kernel(int B, int L, int fuse, int Lc,
                                                               const int32_t *__restrict__ coarse,
                                                               int32_t *__restrict__ plan) {
    const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= (int64_t)B * L) return;
    const int b = (int)(i / L), l = (int)(i % L);
    plan[i] = coarse[(int64_t)b * Lc + l / fuse];
}

using SweepFn = void (*)(Layout, int);
using ChainFn = void (*)(Layout, int64_t *, int32_t *);
struct VariantEntry {
    Variant v;
    SweepFn fn, fn_u8;     // int32 and one-byte back-pointers
    SweepFn fn_pack;       // byte table (row-sharing variants; else null)
};
template <int TS, int TE, int NG, int WPE, int W, int UX, int SHARE>
VariantEntry variant_entry() {
    static_assert((W == 1 || W == 2 || W == 3 || W == 4 || W == 6 || W == 8 || W == 16) && W % NG == 0,
                  "strategy groups must divide the workgroup's waves");
    static_assert(!SHARE || W == NG, "the row-sharing body has one budget tile per workgroup");
    static_assert((UX == 1 || UX == 2) && TE * UX <= 4, "budget columns per lane");
    SweepFn pack = nullptr;
    if constexpr (SHARE != 0) pack = sweep_bytes_kernel<TS, TE, NG, WPE, W, UX>;
    return {{TS, TE, NG, W, UX, WPE, SHARE},
            sweep_kernel<TS, TE, NG, WPE, int32_t, W, UX, SHARE>,
            sweep_kernel<TS, TE, NG, WPE, uint8_t, W, UX, SHARE>,
            pack};
}

enum class Tiles { wide, normal, split, fine, chain };

// Shapes of the chained sweep: strategies and rows per wave, waves.  Few tiles take more, thinner waves: their time is a
// layer's latency.  Many take fewer: what a wave does beside its rows and strategies (words, list, scalars) then keeps the
// SIMDs busy, and the more workgroups are resident the sooner a block to the right begins.  Whole searches over the
// time with a launch per layer, thin / fat, layers alike - deep stacks - deep stacks in nanoseconds: 12 strategies x 504 tiles
// 0.66 0.64 0.42 / 0.70 0.66 0.46, x 2064 0.85 0.89 0.57 / 0.74 0.75 0.51; 22 x 504 0.65 0.65 0.43 / 0.74 0.70 0.48, x 1032 0.86 0.91
// 0.64 / 0.82 0.75 0.54; 30 x 700 0.84 0.87 0.63 / 0.88 0.76 0.56; 44 x 252 0.67 0.71 0.49 / 0.77 0.76 0.55, x 504 0.85 0.86 0.65 /
// 0.80 0.70 0.52; 60 x 252 0.75 0.69 0.49 / 0.90 0.75 0.54, x 504 0.87 0.92 0.71 / 0.85 0.76 0.58.
struct ChainEntry {
    int ts, ng;
    int64_t tiles;         // up to so many tiles in a layer of the whole batch
    int peek;              // the fat shapes from 17 strategies on look at two cells of a row before they read it: one more round trip,
                           // fewer rows.  Without / with, layers alike - deep stacks - the latter with tenfold transition costs, over the
                           // time with a launch per layer: 22 x 2244 0.86 0.92 0.71 / 0.85 0.92 0.73, x 3432 0.89 1.01 0.77 / 0.89 0.94 0.77; 30 x
                           // 1452 0.90 0.98 0.67 / 0.90 0.97 0.69; 44 x 1056 0.96 1.04 0.66 / 0.94 1.00 0.67; 12 x 5016 0.83 0.96 0.71 / 0.88 1.00 0.76
    ChainFn fn;
};
template <int TS, int NG>
ChainEntry chain_entry(int64_t tiles, int peek = 0) {
    return {TS, NG, tiles, peek, chain_kernel<TS, NG>};
}
const ChainEntry *pick_chain(int S, int64_t tiles) {
    constexpr int64_t any = INT64_MAX;
    static const ChainEntry table[] = {chain_entry<2, 4>(any),  chain_entry<2, 8>(768),  chain_entry<4, 4>(any), chain_entry<3, 8>(768),
                                       chain_entry<6, 4>(any, 1), chain_entry<4, 8>(704), chain_entry<8, 4>(any, 1), chain_entry<3, 16>(352),
                                       chain_entry<6, 8>(any, 1), chain_entry<4, 16>(352), chain_entry<8, 8>(any, 1)};
    for (const ChainEntry &t : table)
        if (S <= t.ts * t.ng && tiles <= t.tiles) return &t;
    return nullptr;
}

// wide: the launch fills the chip; take the 256-column twin where there is one.  split, fine: it
// leaves wavefront slots idle; take the twin with more waves per tile.
const VariantEntry &pick_variant(int S, Tiles tiles) {
    static const VariantEntry splits[] = {
        variant_entry<GALV_S0>(), variant_entry<GALV_S1>(), variant_entry<GALV_S2>(), variant_entry<GALV_S3>(),
        variant_entry<GALV_S4>(), variant_entry<GALV_S5>(), variant_entry<GALV_S6>()};
    static const VariantEntry fines[] = {variant_entry<GALV_F2>(), variant_entry<GALV_F3>()};
    if (tiles == Tiles::fine)
        for (const VariantEntry &t : fines)
            if (S > 16 && S <= t.v.ts * t.v.ng) return t;
    if (tiles == Tiles::split || tiles == Tiles::fine)
        for (const VariantEntry &t : splits)
            if (S <= t.v.ts * t.v.ng) return t;
    static const VariantEntry table[] = {
        variant_entry<GALV_V0>(), variant_entry<GALV_V1>(), variant_entry<GALV_V2>(),
        variant_entry<GALV_V3>(), variant_entry<GALV_V4>(), variant_entry<GALV_V5>(),
        variant_entry<GALV_V6>(), variant_entry<GALV_V7>(), variant_entry<GALV_V8>()};
    static const VariantEntry twins[] = {
        variant_entry<GALV_V2X>(), variant_entry<GALV_V3X>(), variant_entry<GALV_V4X>(),
        variant_entry<GALV_V5X>(), variant_entry<GALV_V6X>(), variant_entry<GALV_V7X>()};
    constexpr int n = sizeof table / sizeof table[0];
    for (int i = 0; i < n; ++i)
        if (S <= table[i].v.ts * table[i].v.ng) {
            if (tiles == Tiles::wide)
                for (const VariantEntry &t : twins)
                    if (t.v.ts == table[i].v.ts && t.v.ng == table[i].v.ng) return t;
            return table[i];
        }
    return table[n - 1];
}

}  // namespace

struct galv_dp {
    galv_dp_desc_t desc;
    Variant var;
    SweepFn sweep;
    ChainFn chain;     // the chained sweep, or null
    Layout lay;        // workspace pointers filled, input pointers set per solve
    size_t ws_bytes;
    int groups_y;      // grid.y of the sweep
    unsigned lds_bytes; // dynamic LDS of a sweep workgroup (staging variants only)
    bool lds_allowed;   // the kernel has been told that it may use that much
    bool solved;
    bool fresh;         // no solve has run over this workspace yet: the infinity leads are unwritten
    int n_side;                    // side streams the handle owns (0 or >= 2); a solve uses some or all of them
    bool auto_streams;             // the solve picks how many (else: all of them, as the caller asked)
    int n_used;                    // how many the last solve used (0: none has run)
    int resident;                  // sweep workgroups the GPU holds at a time
    int32_t *seen_host;            // pinned: budget tiles of the batch as the last solve's prep_kernel found them
    hipStream_t side[kMaxSide];
    hipEvent_t fork, join[kMaxSide];
};

namespace {

struct Plan {
    Variant var;
    SweepFn sweep;
    ChainFn chain;
    Layout lay;
    size_t off_U[2], off_bp, off_Rk, off_ck, off_vlist, off_vcost, off_nvalid, off_hdr, off_status, off_last, off_dclamp,
        off_lead_mode, off_stats, total;
    int groups_y;
    unsigned lds_bytes;
};

// Tiles of 128 columns in one layer of the whole batch; from kFullChip on they fill the chip several times over.
int64_t launch_tiles(const galv_dp_desc_t &d) { return ((int64_t)d.max_budget / 128 + 1) * d.n_instances; }
constexpr int64_t kFullChip = 3072;

// `only`: the shape to take instead of the one the rules below choose (the flags still override it); `chain`: the chained
// sweep may be chosen.
galv_status_t make_plan(const galv_dp_desc_t *d, const Tiles *only, bool chain, Plan *p) {
    if (!d) return fail(GALV_ERR_INVALID_ARG, "desc is NULL");
    if (d->n_instances < 1 || d->n_layers < 1 || d->n_strategies < 1 || d->max_budget < 0 ||
        d->n_transition < 1)
        return fail(GALV_ERR_INVALID_ARG,
                    "desc: need n_instances>=1, n_layers>=1, n_strategies>=1, max_budget>=0, "
                    "n_transition>=1 (got %d %d %d %d %d)",
                    d->n_instances, d->n_layers, d->n_strategies, d->max_budget, d->n_transition);
    if (d->n_strategies > kMaxS)
        return fail(GALV_ERR_INVALID_ARG, "n_strategies %d exceeds the limit %d", d->n_strategies,
                    kMaxS);
    if (d->flags & ~(GALV_DP_FORCE_INT64 | GALV_DP_BP_U8 | GALV_DP_NO_U32 | GALV_DP_NO_PEEK | GALV_DP_FORCE_PEEK |
                     GALV_DP_NO_PACK | GALV_DP_FORCE_PACK | GALV_DP_FORCE_WIDE_TILES | GALV_DP_NO_WIDE_TILES |
                     GALV_DP_STREAMS_MASK))
        return fail(GALV_ERR_INVALID_ARG, "unknown flag bits");
    if (((d->flags & GALV_DP_STREAMS_MASK) >> GALV_DP_STREAMS_SHIFT) > (uint32_t)kMaxSide)
        return fail(GALV_ERR_INVALID_ARG, "at most %d internal streams", kMaxSide);
    const bool u8 = (d->flags & GALV_DP_BP_U8) != 0;
    if (u8 && d->n_strategies > 255)
        return fail(GALV_ERR_INVALID_ARG, "one-byte back-pointers need n_strategies <= 255 (got %d)",
                    d->n_strategies);
    if (d->n_instances > 65535)
        return fail(GALV_ERR_RANGE, "n_instances %d exceeds the grid limit 65535", d->n_instances);
    if (d->max_budget > (1 << 30))
        return fail(GALV_ERR_RANGE, "max_budget %d exceeds 2^30", d->max_budget);

    memset(p, 0, sizeof *p);
    const int64_t tiles = launch_tiles(*d);
    const int S = d->n_strategies;
    const bool fills_chip = tiles >= kFullChip;
    const int64_t share = d->max_budget / d->n_layers;
    const bool rows_asked = u8 || (d->flags & GALV_DP_NO_PACK);
    // Byte table or cost rows.  The byte table sweeps half the columns and writes a quarter of the bytes or less,
    // but rebuilds every cell it reads in two dependent steps, so a tile takes longer: it pays where a layer has
    // many states, and where its share of the budget spans a tile (rows otherwise fall steeply within one and the
    // peek leaves too many).  Whole solves of 12 layers over cost rows / with the byte table, in us:
    //   14 strategies:  504 tiles  96 / 100   1008 tiles 114 / 105      44:   94 tiles  98 / 100    252 tiles 115 / 108
    //   22:             252 tiles  87 /  93    504 tiles 108 / 103      64:   94 tiles 111 / 106
    //   29:             252 tiles  96 / 104    504 tiles 119 / 111     120:   94 tiles 158 / 140
    //   140, 200, 256:  126 tiles 179 / 169, 247 / 241, 246 / 228 on deep stacks of layers, 255 / 272, 357 / 374, 417 / 433
    //                   on independent layers; 752 tiles 474 / 416, 610 / 564, 748 / 564 and 655 / 444, 892 / 663, 1102 / 798
    // (costs in nanoseconds, that is 64-bit keys: 44 x 504 260 / 196, 120 x 504 917 / 357).  Between the two, the kind
    // of input decides: time with the byte table over that with cost rows, each in its better shape, on independent
    // layers / layers alike / deep stacks, at a share of 140: 32 x 352 1.38 1.20 0.96, x 1080 1.08 1.01 0.83, 100 x 352
    // 0.99 0.99 0.85; of 700: 32 x 657 1.00 0.90 0.80.
    // Below a share of 128, 22 x 512 tiles of 1000 columns 120 / 131, of 2040 columns 116 / 115; 120 x 512 of 1000 258 /
    // 362, of 2040 261 / 238.  Where the chip is full, down to half a tile, beyond 16 strategies: 3200 to 4000 tiles, in
    // ms, share 49: 22 2.41 / 2.84, 44 3.70 / 4.03; share 83 to 98: 14 0.90 / 1.11, 22 1.19 / 1.10 and 1.94 / 2.02, 44
    // 3.60 / 2.54.
    const bool pays = !rows_asked && tiles * S >= 10000 && (S > 8 || fills_chip) && (share >= 128 || (fills_chip && S > 16 && share >= 64));
    // Tiles of 256 columns where the launch fills the chip with them (normal / wide, in us: 44 x 16448 tiles 4190 /
    // 3440, 128 x 8208 3136 / 2263; with 64-bit keys, which sweep a tile in two parts, from 80000 tile-strategies on: 44 x
    // 2064 1205 / 1077, 64 x 2064 1556 / 1282).  Where many rows are kept they lose (44 x 4805 613 / 897), all the more where
    // their list holds 12 or 16: not for up to 32 strategies over the byte table (a third of the rows kept: 22 x 4240 221
    // / 510, 32 x 4240 279 / 601; a seventh: 22 x 6176 263 / 256, 29 x 10048 669 / 669), nor where a layer's share
    // is small (22 x 4032 tiles at 83 columns 2.02 / 3.08 ms).  Cost rows: 140 strategies x 3528 tiles 1907 / 1551; at a
    // share of 48 to 63, 3200 tiles, 22 strategies 1839 / 1972, 44 2876 / 3181, 100 8109 / 8761.
    const bool wide = pays ? S > 32 && (fills_chip ? share >= 128 : tiles * S >= 80000 && share >= 256)
                           : fills_chip && share >= 64;
    // More waves per tile where the normal shape would leave wavefront slots idle.  Normal / split over cost rows,
    // relative: 6 strategies x 1520 tiles 1.00 / 0.98, x 1752 1.00 / 1.02, x 1980 1.00 / 1.15
    // (64-bit keys, which take every row in every wave: 8 x 1128 1.00 / 0.77, x 1407 1.00 / 1.17); 16 and 32 x 1752 1.00 / 0.88,
    // x 2120 1.00 / 1.02; 44 and 64 x 760 1.00 / 0.96, x 1060 1.00 / 1.09; 100 x 352 1.00 / 0.96, x 540 1.00 / 1.15.  Over the
    // byte table, in us, on independent layers / layers alike / deep stacks: 11 x 3080 166 145 153 / 124 139 156, x 3520 172
    // 145 156 / 129 142 168, x 4400 174 160 167 / 137 168 186; 24 x 2640 0.79 0.77 0.82 / 0.62 0.66 0.80 of the time over cost
    // rows, x 3960 0.84 0.77 0.82 / 0.66 0.75 0.81, x 5640 0.77 0.72 0.83 / 0.61 0.74 0.88; 44 x 1080 1.14 0.88 0.79 / 0.97 0.92
    // 0.95; 100 x 760 1.04 0.83 0.90 / 0.87 0.86 0.89, x 882 287 - 289 / 256 - 285 (64-bit keys: x 564 310 / 336 on deep stacks).
    // Very few tiles of 17 to 32 strategies take eight waves each (split / fine, cost rows: 22 x 94 88 / 82 us, 29 x 252
    // 106 / 96, 22 x 1008 142 / 152).
    const int64_t split_to = S <= 32 ? (pays && S > 8 ? 3584 : 1792) : S <= 64 || pays ? 896 : 448;
    Tiles shape = Tiles::normal;
    if (wide)
        shape = Tiles::wide;
    else if (S > 16 && S <= 32 && tiles <= 256)
        shape = Tiles::fine;
    else if (tiles <= split_to)
        shape = Tiles::split;
    // All layers in one launch (the chained sweep), up to 64 strategies.  It wins by what a launch per layer costs, and loses
    // where the byte table writes and reads less than whole rows: where a layer has many tiles and its share of the budget
    // spans several.  Where the share is below a tile the other side keeps cost rows, and the line lies further out.  Whole
    // searches over the time with a launch per layer, layers alike - deep stacks - independent layers - deep stacks in nanoseconds
    // - layers alike in nanoseconds with tenfold transition costs - deep stacks with tenfold transition costs:
    //   share 700:  6 x 5940 0.77 0.77 0.64 0.52 0.47 0.68, x 15972 1.10 1.09 0.92 0.85 0.71 0.98; 12 x 5016 0.83 0.96 0.50 0.78 0.48 0.71, x 8976 1.17 1.39
    //   0.66 1.12 0.72 0.95; 22 x 3432 0.89 0.94 0.66 0.80 0.58 0.77, x 6204 1.10 1.34 0.67 1.16 0.68 0.88; 30 x 1452 0.90 0.97 0.68 0.77 0.55 0.69,
    //   x 2244 0.90 1.03 0.65 0.88 0.59 0.77; 44 x 1056 0.94 1.00 0.58 0.81 0.57 0.67, x 1584 1.03 1.24 0.63 1.04 0.62 0.79; 60 x 792 0.89 1.01 0.71 0.81
    //   0.59 0.73, x 1452 0.91 1.13 0.39 1.07 0.51 0.56
    //   share 100:  12 x 4940 0.78 0.94 0.49 0.67 0.59 0.69; 22 x 3458 0.64 0.79 0.46 0.68 0.49 0.66, x 6080 0.68 1.14 0.39 1.02 0.62 0.77; 30 x 2166 0.60
    //   0.73 0.40 0.50 0.44 0.56; 44 x 2166 0.61 0.83 0.36 0.47 0.42 0.79; 60 x 1482 0.60 0.76 0.36 0.31 0.34 0.72.
    // Transition costs of 2^32 and more (layers alike in nanoseconds, hundredfold, every row alive) - 64-bit integers:
    //   6 x 4104 share 2730 0.80 0.61; 12 x 4112 share 1024 0.70 0.37; 22 x 1032 share 512 0.65 0.25, x 576 share 75 0.71 0.25; 29 x 78 share 269
    //   0.85 0.13; 44 x 1032 share 682 0.82 0.18, x 272 share 42 0.60 0.16; 60 x 715 share 341 0.77 0.17.
    // (Beyond 64 strategies, two waves' worth of list entries: 100 x 252 1.02 0.96 0.80 0.72, x 1032 1.43 1.79 0.56 1.87.)
    const uint32_t other = GALV_DP_BP_U8 | GALV_DP_NO_U32 | GALV_DP_NO_PEEK | GALV_DP_FORCE_PEEK | GALV_DP_NO_PACK | GALV_DP_FORCE_PACK |
                           GALV_DP_FORCE_WIDE_TILES | GALV_DP_NO_WIDE_TILES;        // (what these ask for is a launch per layer)
    // Where a layer's share of the budget is very large the other side sweeps few columns: share 6250: 16 x 3128 1.04, 22 x 3128 1.06, 44 x
    // 782 1.11 on deep stacks; share 14000 to 25000: 13 x 929 1.11, 24 x 1203 1.08, 27 x 1166 1.14, 44 x 782 1.20; up to 8 strategies 0.70 to 0.84.
    const int64_t chain_to = share < 128 ? 90000 : share >= 4096 ? 10000 : S <= 16 ? 60000 : S <= 24 ? 70000 : 46000;
    // What the launches of all layers but the first cost has to pay for one workgroup per tile, which takes its place from a counter
    // (12 ns each, one after the other) and then starts (a thousand or two at a time, 3 us).  Few strategies, many tiles, over the
    // time with a launch per layer for 2 - 4 - 8 - 16 - 32 layers: 1 x 3000 columns of 2000 2.29 1.52 1.02 0.72 0.53, 1 x 15000 of 16384 7.2 4.2
    // 2.5 1.4 0.76, 1 x 60000 of 100000 19 10 5.0 2.5 -; 6 x 10000 of 2000 3.1 1.8 1.04 0.81 0.76, of 16384 4.0 2.3 1.3 1.08 0.98; 16 x 3750 of 2000 2.1
    // 1.06 0.70 0.71 0.69.  Up to 300 workgroups a layer, 593 searches of seven kinds took 0.07 to 1.04, but for two whose transition
    // matrices alternate (1.13, 1.15, before chain_live kept several; 260 such searches since 0.17 to 1.03); from there to 640 one
    // strategy 0.55 to 1.06, 2 to 8 0.52 to 1.21, more 0.50 to 1.01.  Below a share of 128 cost rows are the other side, and the line lies
    // further out: up to 1000 workgroups a layer 0.13 to 1.00, up to 2000 0.13 to 1.32.
    const int64_t chain_groups = (int64_t)(share < 128 ? 1000 : share < 4096 && (S == 1 || S > 8) ? 640 : 300) * (d->n_layers - 1);
    const ChainEntry *ce = S <= kWave ? pick_chain(S, tiles) : nullptr;
    // Near the line two kinds of inputs lose and all others gain: deep stacks and independent layers with a wide memory range (the
    // peek rules out most of their rows, and the byte table writes one byte where the chain writes eight), the more the larger the
    // share and the more strategies the shape adds to fill its rows.  Deep stacks, those layers - the mean of seven kinds of inputs: 44 x 930
    // share 258 0.93 0.98 - 0.69, share 901 1.08 1.08 - 0.86; 36 x 1134 share 343 1.10 1.05 - 0.82, 34 x 1204 share 895 1.14 1.19 - 0.90, 33 x 1350
    // share 909 1.29 1.27 - 0.97, 17 x 3990 share 889 1.10 1.15 - 0.92, 9 x 6463 share 899 1.08 0.86 - 0.87, 9 x 6454 share 2458 1.19 1.03 - 0.97.
    // The rule knows sizes only, which do not tell these kinds from the others, so the line stays where the mean is below 1.  It is not
    // with shares of 2048 and more and many rows to fill: 35 x 1272 1.35 1.25 - 1.05, 33 x 1350 1.22 1.30 - 1.01, 17 x 3987 1.21 1.24 - 1.00; inside
    // the line that follows 33 x 1044 1.12 1.18 - 0.88, 17 x 3087 0.99 0.96 - 0.86.
    if (ce && S > 16 && share >= 2048 && share < 4096 && tiles * ce->ts * ce->ng > chain_to + chain_to / 4) ce = nullptr;
    // (rows of every layer: at most 8 GB of them, and a layer's of one instance within 32 bits of offset; at most kChainLayers
    // layers, see there)
    const long double chain_bytes = ce ? 8.0L * ce->ts * ce->ng * ((int64_t)d->max_budget + kChainCols) : 0;
    if (chain && ce && !(d->flags & other) && ((d->flags & GALV_DP_STREAMS_MASK) >> GALV_DP_STREAMS_SHIFT) <= 1 && d->n_layers > 1 &&
        d->n_layers <= kChainLayers && tiles * S <= chain_to && tiles + 2ll * d->n_instances <= chain_groups && chain_bytes < 4.0e9L && chain_bytes * d->n_instances * d->n_layers <= 8.0e9L)
        shape = Tiles::chain;
    if (only) shape = *only;
    if (d->flags & GALV_DP_FORCE_WIDE_TILES) shape = Tiles::wide;
    if (d->flags & GALV_DP_NO_WIDE_TILES) shape = Tiles::normal;
    if (shape != Tiles::chain) ce = nullptr;
    const VariantEntry &ve = pick_variant(S, shape);
    const Variant v = ce ? Variant{ce->ts, kChainCols / kWave, ce->ng, ce->ng, 1, 4, 0} : ve.v;
    Layout &a = p->lay;
    a.B = d->n_instances;
    a.L = d->n_layers;
    a.S = d->n_strategies;
    a.E_max = d->max_budget;
    a.nR = d->n_transition;
    a.bp_u8 = u8 ? 1 : 0;
    a.synth_l1 = v.share || ce ? 1 : 0;
    const int group = v.ts * v.ng;
    p->groups_y = (a.S + group - 1) / group;
    a.S_pad = p->groups_y * group;
    int k = 1;               // at least one index bit: the key builders shift by 32 - k
    while ((1 << k) < a.S) ++k;
    a.k_bits = k;
    a.tile_e = kWave * v.te * v.ux * (v.w / v.ng);
    // row-sharing body: partial minima [NG][columns], counters, keep_rows rows of (strategy index, keys), [NG] minima
    p->lds_bytes = 0;
    if (v.share) {
        const size_t cols = (size_t)kWave * v.te * v.ux, keep = keep_rows(v.ts, v.ng, v.wpe, (int)cols);
        const size_t narrow = ((size_t)v.ng * cols + v.ng + 4 + keep + keep * cols) * sizeof(uint32_t);
        // the 8-byte-cell form works on a part of the tile (64 x ux columns) at a time
        const size_t wcols = (size_t)kWave * v.ux;
        const size_t wide = ((size_t)v.ng * wcols + v.ng) * sizeof(uint64_t) + (4 + keep + keep * wcols) * sizeof(uint32_t);
        p->lds_bytes = (unsigned)(narrow > wide ? narrow : wide);
    }
    const unsigned lds_packed = v.share ? byte_lds(v.ts, v.ng, v.wpe, kWave * v.te * v.ux) : 0;
    if (p->lds_bytes > 160u * 1024u || lds_packed > 160u * 1024u)
        return fail(GALV_ERR_RANGE, "internal: staging variant needs %u bytes of LDS", p->lds_bytes);
    a.e_pad = (int64_t)round_up((size_t)a.E_max + 1, kEAlign);
    a.n_tiles = (int32_t)((a.E_max + a.tile_e) / a.tile_e);   // ceil((E_max+1)/tile_e)
    // measured over cost rows: with ~1000 workgroups per layer the peek costs 9 %, with ~6000 it gains 14 %
    a.peek = fills_chip || pays ? 1 : 0;
    if (d->flags & GALV_DP_NO_PEEK) a.peek = 0;
    if (d->flags & GALV_DP_FORCE_PEEK) a.peek = 1;
    bool packed = v.share && pays;
    if (ce) {
        p->lds_bytes = chain_lds(v.ts, v.ng);
        a.peek = ce->peek;
        a.e_pad = (int64_t)round_up((size_t)a.E_max + 1, (size_t)a.tile_e);
    }
    if ((d->flags & GALV_DP_FORCE_PACK) && v.share && !u8) packed = true;
    if (packed) p->lds_bytes = lds_packed;
    p->sweep = packed ? ve.fn_pack : (u8 ? ve.fn_u8 : ve.fn);
    p->chain = ce ? ce->fn : nullptr;
    // (up to 30 strategies x 3000 tiles: two tables of 8-byte cells take 184 MB, and the caches hold 256.  With all
    // rows alive, cost rows / byte table: 30 x 3760 tiles 904 / 658 us, 34 x 3760 957 / 675, 64 x 1512 919 / 833)
    a.packed = ce ? kChain : !packed ? 0 : !(d->flags & GALV_DP_FORCE_PACK) && tiles * S < 90000 ? kRowsIfAlive : kAllBytes;
    a.seen = nullptr;
    a.lead = (int64_t)round_up((size_t)a.E_max + 1, 64);
    a.row = a.lead + a.e_pad;
    p->var = v;

    // Sizes in long double first, to reject anything that would overflow size_t math.
    const long double approx = (long double)a.B * a.S_pad * (ce ? a.L * a.e_pad * 8 : a.row * 16) +
                               (long double)a.B * (a.L - 1) * a.S * a.e_pad * (u8 ? 1 : 4) +
                               (long double)a.B * a.nR * a.S * a.S_pad * 8;
    if (approx > 1e15L) return fail(GALV_ERR_RANGE, "tables of %.3Lg bytes cannot be indexed", approx);

    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t at = off;
        off = round_up(off + bytes, 256);
        return at;
    };
    const size_t u_bytes = ce ? (size_t)a.B * a.L * a.S_pad * a.e_pad * 8 : (size_t)a.B * a.S_pad * a.row * 8;
    p->off_U[0] = take(u_bytes);
    p->off_U[1] = take(ce ? chain_word_bytes(a.B, a.n_tiles) : u_bytes);
    p->off_bp = take((size_t)a.B * (a.L - 1) * a.S * a.e_pad * (u8 ? 1 : sizeof(int32_t)));
    // + slack: a group of R keys is fetched whole even when it straddles the row end
    p->off_Rk = take((size_t)a.B * a.nR * a.S * a.S_pad * sizeof(double) + 1024);
    p->off_ck = take((size_t)a.B * a.L * a.S_pad * sizeof(uint64_t));
    p->off_vlist = take((size_t)a.B * a.L * a.S_pad * sizeof(uint64_t) + 64);   // + slack: entries are fetched eight at a time
    p->off_vcost = take((size_t)a.B * a.L * a.S_pad * sizeof(uint64_t) + 64);
    p->off_nvalid = take((size_t)a.B * a.L * sizeof(int32_t));
    p->off_status = take((size_t)a.B * sizeof(int32_t));
    p->off_last = take((size_t)a.B * sizeof(int32_t));
    p->off_dclamp = take((size_t)a.B * sizeof(uint32_t));
    p->off_hdr = take((size_t)a.B * a.L * 8 * sizeof(int32_t));
    p->off_lead_mode = take((size_t)a.B * sizeof(int32_t));
    p->off_stats = take((size_t)a.B * (a.L > 1 ? a.L - 1 : 1) * a.n_tiles * 2 * sizeof(uint32_t));
    p->total = off;
    return GALV_OK;
}

// The plan for a launch per layer: the shape that the rules choose, or, where it does not fit `bytes` of workspace, the plain
// one, and where the launch fills the chip the wide one, if that does.  (The twins with more waves pad the strategies
// to a little more, and narrow tiles take more statistics: a workspace of the size that these shapes need, which
// were once all there were, stays large enough.)
galv_status_t make_plan(const galv_dp_desc_t *d, size_t bytes, Plan *p) {
    const galv_status_t st = make_plan(d, nullptr, false, p);
    if (st != GALV_OK || p->total <= bytes) return st;
    const bool fills_chip = launch_tiles(*d) >= kFullChip;
    for (Tiles only : {Tiles::normal, Tiles::wide}) {
        if (only == Tiles::wide && !fills_chip) continue;
        Plan q;
        if (make_plan(d, &only, false, &q) == GALV_OK && q.total <= bytes) {
            *p = q;
            break;
        }
    }
    return GALV_OK;
}

// The plan of a handle: the chained sweep, which keeps every layer's rows, where the rules choose it and the workspace
// holds it.  (What it takes decides nothing else: a workspace is too small or a shape too large when a launch per layer
// would not fit.)
galv_status_t choose_plan(const galv_dp_desc_t *d, size_t bytes, Plan *p) {
    const galv_status_t st = make_plan(d, bytes, p);
    if (st != GALV_OK || p->total > bytes) return st;
    Plan q;
    if (make_plan(d, nullptr, true, &q) == GALV_OK && q.total <= bytes) *p = q;
    return GALV_OK;
}

// grid.x of a sweep launch for n budget tiles.
// (the byte-table sweep's first eight workgroups are not for tiles)
inline unsigned kGridTiles(const Layout &a) {
    const unsigned n = (unsigned)a.n_tiles;
    if (a.packed == kChain) return (unsigned)((n + 2) * a.B);     // (and two places more per instance)
    return (GALV_XCD_MAP || a.packed ? (n + 7) / 8 * 8 : n) + (a.packed ? 8 : 0);
}

// Point a layout's table pointers into a workspace laid out by make_plan.
void bind_workspace(Layout &a, const Plan &p, char *ws) {
    a.U[0] = ws + p.off_U[0];
    a.U[1] = ws + p.off_U[1];
    a.bp = ws + p.off_bp;
    a.Rk = reinterpret_cast<double *>(ws + p.off_Rk);
    a.ck = reinterpret_cast<uint64_t *>(ws + p.off_ck);
    a.vlist = reinterpret_cast<uint64_t *>(ws + p.off_vlist);
    a.vcost = reinterpret_cast<uint64_t *>(ws + p.off_vcost);
    a.nvalid = reinterpret_cast<int32_t *>(ws + p.off_nvalid);
    a.status = reinterpret_cast<int32_t *>(ws + p.off_status);
    a.last = reinterpret_cast<int32_t *>(ws + p.off_last);
    a.dclamp = reinterpret_cast<uint32_t *>(ws + p.off_dclamp);
    a.hdr = reinterpret_cast<int32_t *>(ws + p.off_hdr);
    a.lead_mode = reinterpret_cast<int32_t *>(ws + p.off_lead_mode);
    a.stats = reinterpret_cast<uint32_t *>(ws + p.off_stats);
}

// How many internal streams a solve deals its instances over, given the budget tiles (sweep
// workgroups per strategy group and layer) of the whole batch.  Measured on MI355X with 4 hardware
// queues: the sweeps run fastest when one launch holds about two thirds of the workgroups the GPU
// can keep resident, so that launches of different streams overlap in different phases (loads of
// one under the arithmetic and stores of another) -- 64 instances of 44 strategies: 5-6 streams
// for 4096 tiles, 6 for 5150, 9-10 for 8192, each 5-15 % ahead of two streams more or fewer; as
// long as a launch still takes ~12 us (shorter ones are bound by the launch rate: 32 instances of
// 22 strategies x 24576 columns take 1.16 / 1.20 / 1.70 ms with 2 / 3 / 4 streams).  A stream that
// holds two instances where others hold one sets the pace, so when most streams would hold a
// single instance every instance gets its own (16 instances of 128 strategies x 65536 columns:
// 20.3 ms with 16 streams, 21.2 with 12, 22.1 with 11).
int pick_streams(const galv_dp *h, int64_t tiles) {
    if (h->n_side <= 1 || h->lay.packed == kChain) return 1;
    if (!h->auto_streams) return h->n_side;
    const Layout &a = h->lay;
    // The byte-table sweep: every launch costs ~4 us on the host and the same again on the queue, so
    // one stream, or two where a layer holds enough states for the overlap of two launches to pay:
    // 17 M states (22 x 24576 columns x 32 instances) 0.82 / 0.94 ms with 1 / 2 streams, 58 M (44 x
    // 20480 x 64) 4.05 / 3.59 / 3.72 / 4.5 ms with 1 / 2 / 3 / 6, 134 M (128 x 65536 x 16) 13.3 / 12.4 /
    // 12.5 / 16.3 ms with 1 / 2 / 3 / 16.
    if (a.packed) return (double)tiles * a.tile_e * a.S >= 20e6 && a.B > 1 ? 2 : 1;
    const double wgs = (double)tiles * h->groups_y;
    int n = (int)(wgs / (0.66 * h->resident) + 0.5);
    const double us = (double)tiles * a.tile_e * a.S * 8.0 / 5.5e12 * 1e6;   // a layer at 8 B per state
    if (n > (int)(us / 12.0)) n = (int)(us / 12.0);
    if (2 * n > a.B) n = a.B;
    if (n > h->n_side) n = h->n_side;
    return n < 1 ? 1 : n;
}
int64_t tiles_at_most(const galv_dp *h) { return (int64_t)h->lay.B * (h->lay.E_max / h->lay.tile_e + 1); }

// The kernel that sweeps, as the runtime knows it.
const void *sweep_function(const galv_dp *h) {
    return h->chain ? reinterpret_cast<const void *>(h->chain) : reinterpret_cast<const void *>(h->sweep);
}

// Enqueue one whole solve (preparation, layer 0, the L-1 sweeps, final minimum) of handle h on
// stream st.  Shared by every entry point that solves.
galv_status_t enqueue_solve(galv_dp *h, const int64_t *c_dev, const int32_t *m_dev,
                            const int64_t *R_dev, const int32_t *r_idx_dev,
                            const int32_t *budget_dev, int64_t *best_cost_dev,
                            int32_t *best_last_dev, hipStream_t st) {
    Layout &a = h->lay;
    a.c = c_dev;
    a.m = m_dev;
    a.R = R_dev;
    a.r_idx = r_idx_dev;
    a.budget = budget_dev;
    h->solved = false;

    if (!h->lds_allowed) {     // more than the default 64 KB of dynamic LDS: say so before any launch
        HIP_TRY(hipFuncSetAttribute(sweep_function(h),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)h->lds_bytes));
        h->lds_allowed = true;
    }
    // (the budgets are on the device: what an earlier solve's preparation reported stands in for
    // them, and the largest possible count before any has; read before this solve's own
    // preparation is launched, so that the choice does not depend on how fast that one runs)
    const int32_t seen = h->seen_host ? *static_cast<volatile int32_t *>(h->seen_host) : 0;
    const int n_use = a.L < 2 ? 1 : pick_streams(h, seen > 0 ? seen : tiles_at_most(h));
    h->n_used = n_use;
    prep_kernel<<<a.B, kPrepThreads, 0, st>>>(a, h->desc.flags);
    if (a.packed != kChain) {
        // at most 16 cells per thread: enough blocks to write a row at full rate, few enough to cost
        // nothing when, as usual after a handle's first solve, there is nothing to write
        const int64_t blocks = (a.row + 16 * kThreads - 1) / (16 * kThreads);
        init_kernel<<<dim3((unsigned)blocks, a.S, a.B), kThreads, 0, st>>>(a, h->fresh ? 1 : 0);
    }
    a.b_off = 0;
    a.b_step = 1;
    if (a.packed == kChain) {
        h->chain<<<kGridTiles(a), h->var.w * kWave, h->lds_bytes, st>>>(a, best_cost_dev, best_last_dev);
    } else if (n_use <= 1) {
        const dim3 grid(kGridTiles(a), h->groups_y, a.B);
        for (int l = 1; l < a.L; ++l) h->sweep<<<grid, h->var.w * kWave, h->lds_bytes, st>>>(a, l);
    } else {
        // Instances are independent, so their layer chains need no common barrier: each
        // side stream sweeps its own share of the instances (dealt round-robin, which balances
        // unequal budgets) and the shares overlap freely.
        HIP_TRY(hipEventRecord(h->fork, st));
        // A failure after the fork must not leave side streams running behind the caller's
        // back: whatever was started is still joined into `st` before the error is returned.
        hipError_t err = hipSuccess;
        for (int g = 0; g < n_use && err == hipSuccess; ++g) {
            const int count = (a.B - g + n_use - 1) / n_use;            // instances g, g + n, g + 2n, ...
            if (count <= 0) continue;
            err = hipStreamWaitEvent(h->side[g], h->fork, 0);
            if (err != hipSuccess) break;                 // nothing enqueued on this side stream
            Layout ag = a;
            ag.b_off = g;
            ag.b_step = n_use;
            const dim3 grid(kGridTiles(a), h->groups_y, count);
            for (int l = 1; l < a.L; ++l) h->sweep<<<grid, h->var.w * kWave, h->lds_bytes, h->side[g]>>>(ag, l);
            err = hipEventRecord(h->join[g], h->side[g]);
            const hipError_t e2 = err == hipSuccess ? hipStreamWaitEvent(st, h->join[g], 0) : err;
            if (e2 != hipSuccess) {
                // could not order `st` after this side stream: wait for it on the host instead
                (void)hipStreamSynchronize(h->side[g]);
                err = e2;
            }
        }
        if (err != hipSuccess)
            return fail(GALV_ERR_HIP, "forking the layer sweeps over internal streams failed: %s",
                        hipGetErrorString(err));
    }
    if (a.packed != kChain) final_kernel<<<a.B, kWave, 0, st>>>(a, best_cost_dev, best_last_dev);
    HIP_TRY(hipGetLastError());
    h->solved = true;
    h->fresh = false;
    return GALV_OK;
}

constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];       // device address of `scratch` on each GPU, once known
std::mutex g_scratch_mutex;

// Device address of the current GPU's copy of `scratch`, looked up on the first call per device.
galv_status_t static_scratch(void **out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(GALV_ERR_RANGE, "device ordinal %d is outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 256 != 0)
            return fail(GALV_ERR_HIP, "the static workspace has no usable device address (%p)", ptr);
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return GALV_OK;
}


}  // namespace

extern "C" {

galv_status_t galv_dp_workspace_bytes(const galv_dp_desc_t *desc, size_t *bytes) {
    if (!bytes) return fail(GALV_ERR_INVALID_ARG, "bytes is NULL");
    Plan p;
    galv_status_t st = make_plan(desc, (size_t)GALV_DP_STATIC_BYTES, &p);
    if (st != GALV_OK) return st;
    *bytes = p.total;
    return GALV_OK;
}

galv_status_t galv_dp_workspace_bytes_preferred(const galv_dp_desc_t *desc, size_t *bytes) {
    if (!bytes) return fail(GALV_ERR_INVALID_ARG, "bytes is NULL");
    Plan p, q;
    galv_status_t st = make_plan(desc, nullptr, false, &p);
    if (st == GALV_OK) st = make_plan(desc, nullptr, true, &q);
    if (st != GALV_OK) return st;
    *bytes = p.total > q.total ? p.total : q.total;
    return GALV_OK;
}

galv_status_t galv_dp_create(const galv_dp_desc_t *desc, void *workspace_dev,
                             size_t workspace_bytes, galv_dp_t **out) {
    if (!out) return fail(GALV_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    Plan p;
    galv_status_t st = choose_plan(desc, workspace_bytes, &p);
    if (st != GALV_OK) return st;
    if (!workspace_dev) return fail(GALV_ERR_WORKSPACE, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace_dev) % 256 != 0)
        return fail(GALV_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    if (workspace_bytes < p.total)
        return fail(GALV_ERR_WORKSPACE, "workspace of %zu bytes is smaller than the %zu needed",
                    workspace_bytes, p.total);

    galv_dp *h = new (std::nothrow) galv_dp;
    if (!h) return fail(GALV_ERR_INVALID_ARG, "out of host memory");
    h->desc = *desc;
    h->var = p.var;
    h->sweep = p.sweep;
    h->chain = p.chain;
    h->lay = p.lay;
    h->ws_bytes = p.total;
    h->groups_y = p.groups_y;
    h->lds_bytes = p.lds_bytes;
    h->lds_allowed = p.lds_bytes <= 64u * 1024u;
    if (!h->lds_allowed) {
        // More than the default 64 KB of dynamic LDS: the kernel is told here, once, rather than at
        // the first solve, which a caller may be capturing into a graph.  (Should this fail, the
        // solve tries again and reports it.)
        if (hipFuncSetAttribute(sweep_function(h), hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)h->lds_bytes) == hipSuccess)
            h->lds_allowed = true;
        else
            (void)hipGetLastError();
    }
    h->solved = false;
    h->fresh = true;
    h->n_side = 0;
    h->n_used = 0;
    h->seen_host = nullptr;
    h->lay.seen = nullptr;
    {
        // workgroups of the sweep that the GPU holds at a time (by registers and LDS)
        int per_cu = 0, cus = 0, dev = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 256;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, sweep_function(h),
                                                         h->var.w * kWave, h->lds_bytes) != hipSuccess || per_cu < 1)
            per_cu = h->var.wpe * 4 / h->var.w > 0 ? h->var.wpe * 4 / h->var.w : 1;
        (void)hipGetLastError();
        h->resident = per_cu * cus;
    }
    int n = (int)((desc->flags & GALV_DP_STREAMS_MASK) >> GALV_DP_STREAMS_SHIFT);
    h->auto_streams = n == 0;
    if (n == 0) {
        // Automatic: the handle owns as many streams as its largest batch could use (pick_streams
        // with every budget at the maximum), and every solve picks from the budgets the solve
        // before it met.
        h->n_side = kMaxSide;                      // (lets pick_streams answer for the cap below)
        n = pick_streams(h, tiles_at_most(h));
        h->n_side = 0;
        if (n > 1 && hipHostMalloc(reinterpret_cast<void **>(&h->seen_host), 64, hipHostMallocDefault) == hipSuccess) {
            *h->seen_host = 0;
            void *dptr = nullptr;
            if (hipHostGetDevicePointer(&dptr, h->seen_host, 0) == hipSuccess && dptr) {
                h->lay.seen = static_cast<int32_t *>(dptr);
            } else {
                (void)hipHostFree(h->seen_host);
                h->seen_host = nullptr;
            }
        }
        (void)hipGetLastError();
    }
    if (n > desc->n_instances) n = desc->n_instances;
    if (n > 1 && desc->n_layers > 1) {
        hipError_t e = hipEventCreateWithFlags(&h->fork, hipEventDisableTiming);
        const bool have_fork = e == hipSuccess;
        int made_s = 0, made_e = 0;
        for (int g = 0; g < n && e == hipSuccess; ++g) {
            e = hipStreamCreateWithFlags(&h->side[g], hipStreamNonBlocking);   // default priority
            if (e != hipSuccess) break;
            ++made_s;
            e = hipEventCreateWithFlags(&h->join[g], hipEventDisableTiming);
            if (e == hipSuccess) ++made_e;
        }
        if (e != hipSuccess) {
            for (int g = 0; g < made_s; ++g) (void)hipStreamDestroy(h->side[g]);
            for (int g = 0; g < made_e; ++g) (void)hipEventDestroy(h->join[g]);
            if (have_fork) (void)hipEventDestroy(h->fork);
            if (h->seen_host) (void)hipHostFree(h->seen_host);
            delete h;
            return fail(GALV_ERR_HIP, "creating internal streams failed: %s", hipGetErrorString(e));
        }
        h->n_side = n;
    }
    bind_workspace(h->lay, p, static_cast<char *>(workspace_dev));
    *out = h;
    return GALV_OK;
}

galv_status_t galv_dp_solve_batched(galv_dp_t *h, const int64_t *c_dev, const int32_t *m_dev,
                                    const int64_t *R_dev, const int32_t *r_idx_dev,
                                    const int32_t *budget_dev, int64_t *best_cost_dev,
                                    int32_t *best_last_dev, void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!c_dev || !m_dev || !R_dev || !budget_dev || !best_cost_dev || !best_last_dev)
        return fail(GALV_ERR_INVALID_ARG, "a required device pointer is NULL");
    return enqueue_solve(h, c_dev, m_dev, R_dev, r_idx_dev, budget_dev, best_cost_dev, best_last_dev,
                         static_cast<hipStream_t>(stream));
}

galv_status_t galv_dp_backtrack(galv_dp_t *h, int32_t *plan_dev, void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!plan_dev) return fail(GALV_ERR_INVALID_ARG, "plan_dev is NULL");
    if (!h->solved) return fail(GALV_ERR_STATE, "backtrack before a successful solve");
    const Layout &a = h->lay;
    backtrack_kernel<<<a.B, kWave, 0, static_cast<hipStream_t>(stream)>>>(a, plan_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_solve_static(const galv_dp_desc_t *desc, const int64_t *c_dev,
                                   const int32_t *m_dev, const int64_t *R_dev,
                                   const int32_t *r_idx_dev, const int32_t *budget_dev,
                                   int64_t *best_cost_dev, int32_t *best_last_dev, int32_t *plan_dev,
                                   void *stream) {
    Plan p;
    galv_status_t rc = choose_plan(desc, (size_t)GALV_DP_STATIC_BYTES, &p);
    if (rc != GALV_OK) return rc;
    if (((desc->flags & GALV_DP_STREAMS_MASK) >> GALV_DP_STREAMS_SHIFT) > 1u)
        return fail(GALV_ERR_INVALID_ARG, "galv_dp_solve_static runs on the caller's stream only "
                                          "(GALV_DP_STREAMS must be 0 or 1)");
    if (p.total > (size_t)GALV_DP_STATIC_BYTES)
        return fail(GALV_ERR_WORKSPACE,
                    "this shape needs %zu bytes of workspace; galv_dp_solve_static holds %zu "
                    "(use galv_dp_create with a workspace of your own)",
                    p.total, (size_t)GALV_DP_STATIC_BYTES);
    if (!c_dev || !m_dev || !R_dev || !budget_dev || !best_cost_dev || !best_last_dev || !plan_dev)
        return fail(GALV_ERR_INVALID_ARG, "a required device pointer is NULL");
    void *ws = nullptr;
    rc = static_scratch(&ws);
    if (rc != GALV_OK) return rc;

    // A handle on the stack: host memory only, no internal streams, nothing to destroy.
    galv_dp h;
    h.desc = *desc;
    h.var = p.var;
    h.sweep = p.sweep;
    h.chain = p.chain;
    h.lay = p.lay;
    h.ws_bytes = p.total;
    h.groups_y = p.groups_y;
    h.lds_bytes = p.lds_bytes;
    h.lds_allowed = p.lds_bytes <= 64u * 1024u;
    h.solved = false;
    h.fresh = true;            // the array keeps the last call's contents: write the leads anew
    h.n_side = 0;              // the caller's stream only: nothing to create, nothing to adapt
    h.auto_streams = false;
    h.n_used = 0;
    h.resident = 1;
    h.seen_host = nullptr;
    h.lay.seen = nullptr;
    bind_workspace(h.lay, p, static_cast<char *>(ws));
    hipStream_t st = static_cast<hipStream_t>(stream);
    rc = enqueue_solve(&h, c_dev, m_dev, R_dev, r_idx_dev, budget_dev, best_cost_dev, best_last_dev, st);
    if (rc != GALV_OK) return rc;
    backtrack_kernel<<<h.lay.B, kWave, 0, st>>>(h.lay, plan_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_best_per_budget(galv_dp_t *h, int64_t *best_cost_dev, int32_t *best_last_dev,
                                      void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!best_cost_dev) return fail(GALV_ERR_INVALID_ARG, "best_cost_dev is NULL");
    if (!h->solved) return fail(GALV_ERR_STATE, "best_per_budget before a successful solve");
    const Layout &a = h->lay;
    const dim3 grid((unsigned)((a.E_max + kThreads) / kThreads), a.B);
    best_per_budget_kernel<<<grid, kThreads, 0, static_cast<hipStream_t>(stream)>>>(a, best_cost_dev,
                                                                                  best_last_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_backtrack_queries(galv_dp_t *h, int32_t n_queries, const int32_t *instance_dev,
                                        const int32_t *budget_dev, int64_t *cost_dev,
                                        int32_t *plan_dev, void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (n_queries < 0) return fail(GALV_ERR_INVALID_ARG, "n_queries %d is negative", n_queries);
    if (n_queries == 0) return GALV_OK;
    if (!instance_dev || !budget_dev || !plan_dev)
        return fail(GALV_ERR_INVALID_ARG, "a required device pointer is NULL");
    if (!h->solved) return fail(GALV_ERR_STATE, "backtrack_queries before a successful solve");
    const unsigned blocks = (unsigned)(n_queries < 1 << 20 ? n_queries : 1 << 20);
    backtrack_queries_kernel<<<blocks, kWave, 0, static_cast<hipStream_t>(stream)>>>(h->lay, n_queries, instance_dev,
                                                                                     budget_dev, cost_dev, plan_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_export_tables(galv_dp_t *h, int32_t instance, int64_t *C_last_dev,
                                    int32_t *bp_dev, void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!C_last_dev) return fail(GALV_ERR_INVALID_ARG, "C_last_dev is NULL");
    if (!h->solved) return fail(GALV_ERR_STATE, "export before a successful solve");
    const Layout &a = h->lay;
    if (instance < 0 || instance >= a.B)
        return fail(GALV_ERR_INVALID_ARG, "instance %d out of range [0, %d)", instance, a.B);
    if (a.L + 1 > 65535) return fail(GALV_ERR_RANGE, "too many layers to export");
    const dim3 grid((unsigned)((a.E_max + kThreads) / kThreads), a.L + 1);
    export_kernel<<<grid, kThreads, 0, static_cast<hipStream_t>(stream)>>>(a, instance, C_last_dev,
                                                                          bp_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_get_status(galv_dp_t *h, int32_t *status_dev, void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!status_dev) return fail(GALV_ERR_INVALID_ARG, "status_dev is NULL");
    if (!h->solved) return fail(GALV_ERR_STATE, "status before a successful solve");
    HIP_TRY(hipMemcpyAsync(status_dev, h->lay.status, (size_t)h->lay.B * sizeof(int32_t),
                           hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream)));
    return GALV_OK;
}

galv_status_t galv_dp_get_stats(galv_dp_t *h, int64_t *stats_dev, void *stream) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!stats_dev) return fail(GALV_ERR_INVALID_ARG, "stats_dev is NULL");
    if (!h->solved) return fail(GALV_ERR_STATE, "statistics before a successful solve");
    stats_kernel<<<h->lay.B, kThreads, 0, static_cast<hipStream_t>(stream)>>>(h->lay, stats_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_get_config(const galv_dp_t *h, int32_t *config) {
    if (!h) return fail(GALV_ERR_INVALID_ARG, "handle is NULL");
    if (!config) return fail(GALV_ERR_INVALID_ARG, "config is NULL");
    config[0] = h->lay.packed == kChain ? 2 : h->lay.packed ? 1 : 0;
    config[1] = h->lay.peek && (h->chain || h->var.share) ? 1 : 0;
    config[2] = h->n_used > 0 ? h->n_used : (h->lay.L < 2 ? 1 : pick_streams(h, tiles_at_most(h)));
    config[3] = h->lay.tile_e;
    return GALV_OK;
}

galv_status_t galv_alg1_reduce(int32_t n_batch, int32_t n_pp, const int32_t *pp_degree,
                               const int64_t *stage_cost_dev, const int64_t *batch_size_dev,
                               int32_t batch_index_base, int32_t first_window, int64_t *c_p_dev,
                               galv_alg1_state_t *state_dev, void *stream) {
    if (n_batch < 1 || n_batch > (1 << 20))
        return fail(GALV_ERR_INVALID_ARG, "n_batch %d out of range [1, 2^20]", n_batch);
    if (n_pp < 1 || n_pp > kMaxPp)
        return fail(GALV_ERR_INVALID_ARG, "n_pp %d out of range [1, %d]", n_pp, kMaxPp);
    if (!pp_degree || !stage_cost_dev || !batch_size_dev || !c_p_dev || !state_dev)
        return fail(GALV_ERR_INVALID_ARG, "a required pointer is NULL");
    PpList pp;
    pp.n = n_pp;
    for (int i = 0; i < kMaxPp; ++i) pp.degree[i] = 0;
    for (int i = 0; i < n_pp; ++i) {
        if (pp_degree[i] < 1 || pp_degree[i] > (1 << 16))
            return fail(GALV_ERR_INVALID_ARG, "pp_degree[%d] = %d out of range [1, 65536]", i,
                        pp_degree[i]);
        pp.degree[i] = pp_degree[i];
    }
    alg1_reduce_kernel<<<1, kThreads, 0, static_cast<hipStream_t>(stream)>>>(
        n_batch, pp, stage_cost_dev, batch_size_dev, batch_index_base, first_window, c_p_dev,
        state_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_coarsen(int32_t n_instances, int32_t n_layers, int32_t n_strategies,
                              int32_t n_transition, int32_t fuse, int32_t granularity,
                              const int64_t *c_dev, const int32_t *m_dev, const int64_t *R_dev,
                              const int32_t *r_idx_dev, const int32_t *budget_dev, int64_t *c_out_dev,
                              int32_t *m_out_dev, int32_t *r_idx_out_dev, int32_t *budget_out_dev,
                              void *stream) {
    if (n_instances < 1 || n_layers < 1 || n_strategies < 1 || n_transition < 1)
        return fail(GALV_ERR_INVALID_ARG, "coarsen: sizes must be >= 1");
    if (fuse < 1 || granularity < 1)
        return fail(GALV_ERR_INVALID_ARG, "coarsen: fuse %d and granularity %d must be >= 1", fuse,
                    granularity);
    if (!c_dev || !m_dev || !R_dev || !budget_dev || !c_out_dev || !m_out_dev || !r_idx_out_dev ||
        !budget_out_dev)
        return fail(GALV_ERR_INVALID_ARG, "a required device pointer is NULL");
    const int Lc = (n_layers + fuse - 1) / fuse;
    const long double cells = (long double)n_instances * Lc * n_strategies;
    if (cells > 2.0e12L) return fail(GALV_ERR_RANGE, "coarsen: %.3Lg cells cannot be indexed", cells);
    const int64_t n = (int64_t)n_instances * Lc * n_strategies;
    coarsen_kernel<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0,
                     static_cast<hipStream_t>(stream)>>>(
        n_instances, n_layers, n_strategies, n_transition, fuse, granularity, Lc, c_dev, m_dev, R_dev,
        r_idx_dev, budget_dev, c_out_dev, m_out_dev, r_idx_out_dev, budget_out_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_expand_plan(int32_t n_instances, int32_t n_layers, int32_t fuse,
                                  const int32_t *coarse_plan_dev, int32_t *plan_dev, void *stream) {
    if (n_instances < 1 || n_layers < 1 || fuse < 1)
        return fail(GALV_ERR_INVALID_ARG, "expand_plan: sizes must be >= 1");
    if (!coarse_plan_dev || !plan_dev) return fail(GALV_ERR_INVALID_ARG, "a required device pointer is NULL");
    const int Lc = (n_layers + fuse - 1) / fuse;
    const int64_t n = (int64_t)n_instances * n_layers;
    expand_plan_kernel<<<(unsigned)((n + kThreads - 1) / kThreads), kThreads, 0,
                         static_cast<hipStream_t>(stream)>>>(n_instances, n_layers, fuse, Lc,
                                                             coarse_plan_dev, plan_dev);
    HIP_TRY(hipGetLastError());
    return GALV_OK;
}

galv_status_t galv_dp_destroy(galv_dp_t *h) {
    if (h && h->n_side > 1) {
        for (int g = 0; g < h->n_side; ++g) {
            (void)hipStreamDestroy(h->side[g]);
            (void)hipEventDestroy(h->join[g]);
        }
        (void)hipEventDestroy(h->fork);
    }
    if (h && h->seen_host) (void)hipHostFree(h->seen_host);
    delete h;
    return GALV_OK;
}

const char *galv_dp_last_error(void) { return g_err; }

#ifndef GALV_DP_BUILD_STAMP
#define GALV_DP_BUILD_STAMP "unchecked"
#endif
const char *galv_dp_build_stamp(void) { return GALV_DP_BUILD_STAMP; }

}  // extern "C"
