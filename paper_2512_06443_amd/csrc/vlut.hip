// Vector-LUT ternary x INT8 mpGeMM for MI355X (gfx950): kernels and C ABI.
//
// Data layout in LDS (one "slot" = one 81-row table whose rows are 256 bytes):
//   a 256-byte row is 16 slices of 16 bytes; slice l belongs to LDS banks 4l..4l+3,
//   so 16 lanes that each read "their" slice of 16 different rows never conflict.
//   A slice holds 8 INT16 table entries (8 tokens) of ONE sub-table.  With
//   J = 1,2,4,8,16 sub-tables interleaved per row, a slot serves J sub-tables x
//   (128/J) tokens: slice l = j * (16/J) + t  (j = sub-table selector, t = 8-token chunk).
//   Lane (grp = lane/16, l = lane%16) of a wave looks up row idx of slice l for
//   output row 4*rowgroup + grp, so one ds_read_b128 serves 4 output rows x 128
//   (sub-table, token) pairs; the J partial sums of a token are added across lanes
//   once, after the K loop.
//
// Paper references: Alg. 1 (lookup/accumulate and Precompute), Eq. 1-2, Sec. 3.3
// (token-contiguous tables, tile-contiguous packed weights), Sec. 3.4 (tiling,
// streamed precompute-lookup, INT16->INT32 hierarchy, block size 64), Sec. 4
// (topological precompute).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstring>
#include <algorithm>
#include <atomic>
#include <mutex>
#include <type_traits>

#include "vlut.h"


// The kernels, one header per kernel family; this file holds the host side (launch plans, launches, the C ABI).
#include "common.hip.h"
#include "prepare_kernels.hip.h"
#include "lookup_kernel.hip.h"
#include "mfma_kernel.hip.h"
#include "lookup5_kernel.hip.h"
#include "gemm_kernel.hip.h"
#include "gemm_ring_kernel.hip.h"
#include "gemm_private_kernel.hip.h"
#include "decode_kernel.hip.h"
#include "narrow_kernel.hip.h"
#include "small_kernels.hip.h"

// Scratch of vlut_mpgemm_static (split-K partial sums, INT32 [S][N][M]): device memory owned by the library, one
// copy per GPU, held until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; every use of the memory goes through the per-device pointer kept below.
static __device__ __align__(256) unsigned char scratch[VLUT_STATIC_SCRATCH_BYTES];

namespace {

// ---------------------------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per device (with that device current).
int static_scratch_ptr(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return VLUT_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return VLUT_ERR_DEVICE;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return VLUT_OK;
}

// Raises a kernel's dynamic LDS limit once per device (the limit is a property of the kernel on one device).
// The table kernels form LDS addresses as idx*256 + slice*16 and so need their dynamic LDS segment to start at LDS
// address 0, i.e. a kernel without static LDS: checked here, once per device, before the first launch (a kernel
// that fails the check is never launched and the call returns VLUT_ERR_DEVICE).
bool allow_dynamic_lds(const void* kfn, int bytes, std::atomic<unsigned>& done_mask) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    const unsigned bit = (dev >= 0 && dev < 32) ? (1u << dev) : 0u;
    if (bit && (done_mask.load(std::memory_order_relaxed) & bit)) return true;
    hipFuncAttributes attr;
    if (hipFuncGetAttributes(&attr, kfn) != hipSuccess || attr.sharedSizeBytes != 0) return false;
    if (hipFuncSetAttribute(kfn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) != hipSuccess) return false;
    done_mask.fetch_or(bit, std::memory_order_relaxed);
    return true;
}

// A launch by the runtime's call itself: <<< >>> (hipLaunchKernelGGL) hands the same arguments over through a thread's stack of
// configurations first, 2.35 us of the host against 2.15.
template <class T>
struct AsIs { using type = T; };
template <class... Args>
int launch(void (*kfn)(Args...), dim3 grid, int threads, int lds, hipStream_t stream, typename AsIs<Args>::type... args) {
    void* list[] = {(void*)&args...};
    if (hipLaunchKernel((const void*)kfn, grid, dim3((unsigned)threads), list, (size_t)lds, stream) == hipSuccess) return VLUT_OK;
    (void)hipGetLastError();                     // (reported here: not once more to whoever asks next)
    return VLUT_ERR_DEVICE;
}

struct Plan {
    int Jlog, R, S;
    int BW;      // build waves of the 16-wave workgroup (4, 2 or 1); the other 16 - BW waves look up
};

thread_local Plan t_forced = {-1, 0, 0, 0};
bool lookup_plan_forced() { return t_forced.Jlog >= 0 || t_forced.R != 0 || t_forced.S != 0 || t_forced.BW != 0; }

const int kSupportedR[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16};

bool r_supported(int R) {
    for (int v : kSupportedR)
        if (v == R) return true;
    return false;
}

bool shape_ok(int64_t M, int64_t K, int64_t N) {
    return M >= 1 && N >= 1 && K >= 4 && (K % 4) == 0 && M < kMaxDim && K < kMaxDim && N < kMaxDim;
}

struct Derived {
    int G, KCn, RGtotal, n_tile, tiles_n, tiles_m, RGW, stages_total, stages_per_split, total, per_xcd;
    bool need32;
};

Derived derive(const Plan& pl, int64_t M, int64_t K, int64_t N) {
    Derived d;
    d.G = (int)(K / 4);
    d.KCn = (d.G + 15) / 16;
    d.RGtotal = (int)((M + 3) / 4);
    int J = 1 << pl.Jlog;
    d.n_tile = 128 >> pl.Jlog;
    d.tiles_n = (int)((N + d.n_tile - 1) / d.n_tile);
    int cap = (kWaves - pl.BW) * pl.R;                // row groups a workgroup can hold
    d.tiles_m = (d.RGtotal + cap - 1) / cap;
    d.RGW = (d.RGtotal + d.tiles_m - 1) / d.tiles_m;  // balanced rows per workgroup
    d.stages_total = (d.G + 4 * J - 1) / (4 * J);
    d.stages_per_split = (d.stages_total + pl.S - 1) / pl.S;
    d.total = d.tiles_m * d.tiles_n * pl.S;
    d.per_xcd = (d.total + 7) / 8;
    d.need32 = d.stages_per_split * 4 > kBlockLookups;
    return d;
}

// Cost model in nanoseconds, fitted to K-scans and in-kernel timestamps on this chip.  A stage (4 slots = 64
// k-groups at 16 sub-tables per table row) costs a fixed part (the table build and its LDS writes, which share the LDS
// pipe with the table reads) plus a part per row group of the slowest lookup wave (two table reads, two address
// permutes and four three-operand adds per slot pair); with two build waves the fixed part is smaller and every
// workgroup holds 7/6 of the rows, but the build itself takes ~1.37 us per stage, which only R >= 7 hides.  Per tile,
// outside the K loop: the cross-lane reduction and the stores of every row group (bound by the SIMD that holds the
// most lookup waves: four of 14, three of 12) and the hand-over to the next tile; once per workgroup: the argument
// fetch, the first activations and the first table.
double plan_cost(const Plan& pl, int64_t M, int64_t K, int64_t N) {
    Derived d = derive(pl, M, K, N);
    const int lookup_waves = kWaves - pl.BW;
    const double rw = (double)((d.RGW + lookup_waves - 1) / lookup_waves);   // row groups of the slowest lookup wave
    double stage, outside;
    if (pl.BW == 4) {
        stage = 867.0 + 90.0 * rw;
        outside = 600.0 + 190.0 * rw;
    } else {
        stage = 745.0 + 106.0 * rw;
        if (stage < 1370.0) stage = 1370.0;
        outside = 600.0 + 250.0 * rw;
    }
    double wg = d.stages_per_split * stage * (d.need32 ? 1.05 : 1.0) + outside;
    double rounds = (double)((d.total + 255) / 256);          // tiles of the busiest workgroup
    double t = 2000.0 + 2100.0 + rounds * wg;
    if (pl.S > 1) t += 2400.0 + 290.0 * pl.S + (double)pl.S * (double)M * (double)N * 8.0 / (256.0 * 16.0 * 2.1);   // second kernel
    // weight bytes pulled from L2 by all token tiles (256 CUs x ~24 B/clk)
    double traffic = (double)d.tiles_n * (double)d.RGtotal * d.KCn * 64.0 / (256.0 * 24.0 * 2.1);
    return t > traffic ? t : traffic;
}

bool plan_valid(const Plan& pl, int64_t M, int64_t K, int64_t N) {
    if (pl.Jlog < 0 || pl.Jlog > 4 || !r_supported(pl.R) || pl.S < 1 || pl.S > 16) return false;
    if (pl.BW != 4 && pl.BW != 2 && pl.BW != 1) return false;
    Derived d = derive(pl, M, K, N);
    if (d.need32 && pl.R > 6) return false;      // register budget of the INT32 variant
    if (pl.S > d.stages_total) return false;
    return true;
}

// A plan with R == 0 means: the override of vlut_set_plan fits this shape with no value of the free parameters
// (callers report VLUT_ERR_UNSUPPORTED).  Without an override there is always a valid plan (R = 1, S = 1).
const int kBuildWaveChoices[] = {4, 2};
Plan search_plan(int64_t M, int64_t K, int64_t N, int max_S = 16, bool four_build_waves_only = false) {
    Plan best = {0, 0, 0, 0};
    double best_cost = 1e300;
    const int Ss[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    for (int Jlog = 0; Jlog <= 4; ++Jlog)
        for (int R : kSupportedR)
            for (int S : Ss) {
                if (S > max_S) continue;
                for (int BW : kBuildWaveChoices) {
                    if (four_build_waves_only && BW != 4) continue;
                    Plan pl = {t_forced.Jlog >= 0 ? t_forced.Jlog : Jlog, t_forced.R > 0 ? t_forced.R : R,
                               t_forced.S > 0 ? t_forced.S : S, t_forced.BW > 0 ? t_forced.BW : BW};
                    if (!plan_valid(pl, M, K, N)) continue;
                    double c = plan_cost(pl, M, K, N);
                    if (c < best_cost) { best_cost = c; best = pl; }
                }
            }
    return best;
}

// Fused quantisation needs 8-token tiles (16 sub-tables per row) and the codes of the workgroup's K range in LDS.
bool fused_plan_valid(const Plan& pl, int64_t M, int64_t K, int64_t N) {
    if (pl.Jlog != 4 || pl.R > kFusedMaxR || !plan_valid(pl, M, K, N)) return false;
    return derive(pl, M, K, N).stages_per_split <= kFusedMaxStages;
}

bool search_fused_plan(int64_t M, int64_t K, int64_t N, Plan* out) {
    if ((t_forced.Jlog >= 0 && t_forced.Jlog != 4) || (t_forced.BW != 0 && t_forced.BW != 4)) return false;
    bool found = false;
    double best_cost = 1e300;
    const int Ss[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    for (int R : kSupportedR)
        for (int S : Ss) {
            Plan pl = {4, t_forced.R > 0 ? t_forced.R : R, t_forced.S > 0 ? t_forced.S : S, 4};
            if (!fused_plan_valid(pl, M, K, N)) continue;
            double c = plan_cost(pl, M, K, N);
            if (c < best_cost) { best_cost = c; *out = pl; found = true; }
        }
    return found;
}

// The search above costs microseconds of host time; a launch-bound caller repeats a handful of shapes, so the
// last few answers are kept per thread (invalidated by vlut_set_plan).
struct PlanCacheEntry {
    int64_t M, K, N;
    Plan plan;
};
thread_local PlanCacheEntry t_cache[8];
thread_local int t_cache_used = 0, t_cache_next = 0;

Plan choose_plan(int64_t M, int64_t K, int64_t N) {
    for (int i = 0; i < t_cache_used; ++i)
        if (t_cache[i].M == M && t_cache[i].K == K && t_cache[i].N == N) return t_cache[i].plan;
    Plan pl = search_plan(M, K, N);
    t_cache[t_cache_next] = {M, K, N, pl};
    t_cache_next = (t_cache_next + 1) % 8;
    if (t_cache_used < 8) ++t_cache_used;
    return pl;
}

struct FusedCacheEntry {
    int64_t M, K, N;
    Plan plan;
    bool found;
};
thread_local FusedCacheEntry t_fcache[8];
thread_local int t_fcache_used = 0, t_fcache_next = 0;

bool choose_fused_plan(int64_t M, int64_t K, int64_t N, Plan* out) {
    for (int i = 0; i < t_fcache_used; ++i)
        if (t_fcache[i].M == M && t_fcache[i].K == K && t_fcache[i].N == N) {
            *out = t_fcache[i].plan;
            return t_fcache[i].found;
        }
    Plan pl = {4, 1, 1, 4};
    const bool found = search_fused_plan(M, K, N, &pl);
    t_fcache[t_fcache_next] = {M, K, N, pl, found};
    t_fcache_next = (t_fcache_next + 1) % 8;
    if (t_fcache_used < 8) ++t_fcache_used;
    *out = pl;
    return found;
}

// Compute units of the current device (cached per device; 0 if the query fails).
int compute_units() {
    static std::atomic<int> cached[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    int v = cached[dev].load(std::memory_order_relaxed);
    if (v > 0) return v;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0) return 0;
    cached[dev].store(v, std::memory_order_relaxed);
    return v;
}

// The lookup kernel's workgroups are persistent: at most one per compute unit (a workgroup needs more than half of a
// unit's LDS), spread evenly over the 8 XCDs; each walks through its share of the tile list.
template <int R, bool NEED32, int MODE, int BW>
int launch_lookup_t(const LookupParams& p, hipStream_t stream) {
    const int cus = compute_units();
    if (cus < 8) return VLUT_ERR_DEVICE;
    const int grid = 8 * std::min(p.per_xcd, cus / 8);
    auto kfn = lookup_kernel<R, NEED32, MODE, BW>;
    constexpr int max_lds = MODE == kFusedQuant ? kFusedMaxLds : kLdsBytes;
    const int lds = MODE == kFusedQuant ? kFusedAqBase + p.stages_per_split * kFusedStageBytes : kLdsBytes;
    if (lds > max_lds) return VLUT_ERR_UNSUPPORTED;
    static std::atomic<unsigned> attr_done{0};   // one bit per device: the attribute belongs to the device's copy
    if (!allow_dynamic_lds((const void*)kfn, max_lds, attr_done)) return VLUT_ERR_DEVICE;
    LookupParams q = p;
    if (q.S > 1 || q.partial) q.out_vec = ((uintptr_t)q.ws % 16 == 0) && (q.M % 4 == 0);
    else q.out_vec = !q.y || (((uintptr_t)q.y % 16 == 0) && (q.ldy % 4 == 0));
    q.magic_S = q.S > 1 ? (unsigned)((1ull << 32) / (unsigned)q.S) : 0xffffffffu;
    q.magic_tiles_n = q.tiles_n > 1 ? (unsigned)((1ull << 32) / (unsigned)q.tiles_n) : 0xffffffffu;
    return launch(kfn, dim3(grid), kThreads, lds, stream, q);
}

// Which instances of the lookup kernel are compiled: the streamed kernels for every supported R (the INT32-widening
// and the quantising variants hold more state per wave and stop earlier), the variant that reads a materialised
// table for a few small R only (the launcher maps R down).  VLUT_ONLY_R (a build-time macro for experiments)
// restricts the streamed instances to one R.
constexpr bool lookup_instance_built(int R, bool need32, int mode) {
#ifdef VLUT_ONLY_R
    if (mode != kFromGlobal && R != (VLUT_ONLY_R)) return false;
#endif
    if (mode == kFromGlobal) return R == 1 || R == 2 || R == 4;
    if (need32) return R <= 6;
    if (mode == kFusedQuant) return R <= kFusedMaxR;
    return R <= 16;
}

constexpr bool lookup_bw_built(int BW, int mode) { return BW == 4 || (BW == 2 && mode == kFast); }

template <bool NEED32, int MODE, int BW, int R = 1>
int launch_lookup_by_r(int r, const LookupParams& p, hipStream_t stream) {
    if constexpr (R > 16) {
        return VLUT_ERR_UNSUPPORTED;
    } else {
        if constexpr (lookup_instance_built(R, NEED32, MODE)) {
            if (r == R) return launch_lookup_t<R, NEED32, MODE, BW>(p, stream);
        }
        return launch_lookup_by_r<NEED32, MODE, BW, R + 1>(r, p, stream);
    }
}

template <bool NEED32>
int launch_lookup_r(int R, int BW, int mode, const LookupParams& p, hipStream_t stream) {
    if (mode == kFusedQuant && BW == 4) return launch_lookup_by_r<NEED32, kFusedQuant, 4>(R, p, stream);
    if (mode == kFast && BW == 4) return launch_lookup_by_r<NEED32, kFast, 4>(R, p, stream);
    if (mode == kFast && BW == 2) return launch_lookup_by_r<NEED32, kFast, 2>(R, p, stream);
    if (mode == kFromGlobal && BW == 4) return launch_lookup_by_r<NEED32, kFromGlobal, 4>(R, p, stream);
    return VLUT_ERR_UNSUPPORTED;
}

// Second kernel of a split-K (or mixed-packing) launch: four rows per thread when everything is aligned for it.
int launch_splitk_reduce(const int32_t* ws, int S, int64_t M, int64_t N, float w_scale, const float* w_rows,
                         const float* a_scale, float* y, int64_t ldy, int32_t* acc, hipStream_t s) {
    const bool vec = (M % 4 == 0) && ((uintptr_t)ws % 16 == 0) && (!y || ((uintptr_t)y % 16 == 0 && ldy % 4 == 0)) &&
                     (!w_rows || (uintptr_t)w_rows % 16 == 0);
    const size_t total = (size_t)(vec ? M / 4 : M) * (size_t)N;
    const dim3 grid((unsigned)((total + 255) / 256));
    return launch(vec ? splitk_reduce_kernel<4> : splitk_reduce_kernel<1>, grid, 256, 0, s, ws, S, (int)M, (int)N, w_scale, w_rows, a_scale, y, ldy, acc);
}

int check_mpgemm_args(const uint8_t* packed, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K,
                      int64_t N, float* y, int64_t ldy, int32_t* acc) {
    if (!shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (!packed || !a_q || !a_scale) return VLUT_ERR_NULL;
    if (!y && !acc) return VLUT_ERR_NULL;
    if (y && (ldy < M || ldy > INT32_MAX)) return VLUT_ERR_SHAPE;
    return VLUT_OK;
}

// ---- few-token kernel: one copy of the row tiles per token pair.  Measured (K = 2560..6912, 40..250 workgroups):
//      the time of a launch depends on the rows per workgroup, hardly on the number of workgroups while they all
//      fit the device at once (16 rows with four lanes per row were never the best), against 12-16 us for quantiser
//      + general kernel + split-K sum at 3..32 tokens.  So: the fewest rows (from 32) whose grid is one round of
//      workgroups, and narrow_applies weighs that against the general path.
constexpr int kNarrowMaxN = 32;
struct NarrowPlan {
    int parts, rr, rows, gridx, chunks, pairs, gx8, grid;
};

NarrowPlan narrow_plan(int64_t M, int64_t K, int64_t N) {
    NarrowPlan np;
    np.pairs = (int)((N + 1) / 2);
    for (int rows = 32; rows <= 256; rows *= 2) {
        np.rows = rows;
        np.gridx = (int)((M + rows - 1) / rows);
        np.gx8 = np.pairs > 1 ? (np.gridx + 7) / 8 * 8 : np.gridx;
        const int64_t grid = (int64_t)np.gx8 * (np.pairs - 1) + np.gridx;
        np.grid = (int)(grid < INT32_MAX ? grid : INT32_MAX);
        if (grid <= 256) break;
    }
    np.parts = np.rows == 32 ? 2 : 1;
    np.rr = np.rows <= 64 ? 1 : np.rows / 64;
    np.chunks = (int)((K / 4 + kNarrowChunk - 1) / kNarrowChunk);
    return np;
}

// One or two tokens always take this kernel; more tokens while its workgroups fit the device at once and a cost
// estimate fitted to measurements at N <= 32 (2B-model shapes) favours it by 10 % over the lookup kernel.  In us, with c = K / 1024:
//   this kernel   4.6 from fp32 activations (3.6 from INT8 ones) + c x {0.9, 1.35, 2.0, 3.4} for 32, 64, 128, 256 rows
//                 per workgroup;
//   lookup kernel 5.8 + 0.94 c + 0.41 x M N / 10^4 with its split-K sum, + 3.5 for the quantiser from fp32.
// The estimate is older than the matrix-core kernels.  From INT8 codes decode_codes_kernel takes every call that this rule accepts and
// whose K it holds (codes_plan_if_taken); beyond that the table kernel keeps what it had (2560 x 30000 x 2 33.0 us, gemm_kernel 17.7):
// workspace sizes and reported plans follow the rule, so callers know where it lies.
bool narrow_applies(int64_t M, int64_t K, int64_t N, const void* lut, bool from_f32) {
    if (N > kNarrowMaxN || lut != nullptr || lookup_plan_forced()) return false;
    if (N <= 2) return true;
    const NarrowPlan np = narrow_plan(M, K, N);
    if (np.grid > 256) return false;
    const double c = (double)K / 1024.0;
    const double per_chunk = np.rows <= 32 ? 0.9 : (np.rows <= 64 ? 1.35 : (np.rows <= 128 ? 2.0 : 3.4));
    const double narrow_us = (from_f32 ? 4.6 : 3.6) + c * per_chunk;
    const double general_us = 5.8 + 0.94 * c + 0.41 * (double)M * (double)N / 1e4 + (from_f32 ? 3.5 : 0.0);
    return narrow_us * 1.1 < general_us;
}

template <int NTOK, int PARTS, int RR, bool FUSED>
int launch_narrow_t(const NarrowParams& p, int grid, hipStream_t stream) {
    auto kfn = narrow_kernel<NTOK, PARTS, RR, FUSED>;
    constexpr int max_lds = FUSED ? 160 * 1024 : narrow_tab_bytes(NTOK);
    const int lds = FUSED ? narrow_fused_lds_bytes(NTOK, p.chunks) : narrow_tab_bytes(NTOK);
    if (lds > max_lds) return VLUT_ERR_UNSUPPORTED;
    static std::atomic<unsigned> attr_done{0};   // one bit per device: the attribute belongs to the device's copy
    if (!allow_dynamic_lds((const void*)kfn, max_lds, attr_done)) return VLUT_ERR_DEVICE;
    return launch(kfn, dim3(grid), kThreads, lds, stream, p);
}

template <int NTOK, bool FUSED>
int launch_narrow_n(const NarrowPlan& np, const NarrowParams& p, hipStream_t stream) {
    if constexpr (NTOK == 1 && FUSED) {          // fewer rows are decode_kernel's: not built
        if (np.rows < 128) return VLUT_ERR_UNSUPPORTED;
    } else {
        if (np.parts == 2) return launch_narrow_t<NTOK, 2, 1, FUSED>(p, np.grid, stream);
        if (np.rr == 1) return launch_narrow_t<NTOK, 1, 1, FUSED>(p, np.grid, stream);
    }
    if (np.rr == 2) return launch_narrow_t<NTOK, 1, 2, FUSED>(p, np.grid, stream);
    return launch_narrow_t<NTOK, 1, 4, FUSED>(p, np.grid, stream);
}

template <bool FUSED>
int launch_narrow(const NarrowPlan& np, const NarrowParams& p, hipStream_t stream) {
    NarrowParams q = p;
    q.gridx = np.gridx;
    q.gx8 = np.gx8;
    q.chunks = np.chunks;
    return q.N == 1 ? launch_narrow_n<1, FUSED>(np, q, stream) : launch_narrow_n<2, FUSED>(np, q, stream);
}

std::mutex g_pack_mutex;
int* g_pack_flag = nullptr;                // pinned host memory, one int, kept until the process ends (guarded by the mutex)

template <int GW>
int launch_pack(const int8_t* w, int64_t M, int64_t ldw, int64_t K, uint8_t* packed, hipStream_t s) {
    const int G = (int)(K / GW), KCn = (G + 15) / 16, RGtotal = (int)((M + 3) / 4);
    const size_t threads = (size_t)RGtotal * KCn * 16;
    return launch(pack_kernel<GW>, dim3((unsigned)((threads + 255) / 256)), 256, 0, s, w, (int)M, ldw, G, KCn, RGtotal, (unaligned_u32*)packed, g_pack_flag);
}

// The first K5 values of every row five to a byte, the others four to a byte behind them; then waits for the flag of the
// value check.  The kernels raise it in pinned host memory, so that an ordinary call copies nothing (a device flag that is
// cleared and read back by two copies of four bytes costs about 25 us).
int pack_parts(const int8_t* w, int64_t M, int64_t K, int64_t K5, uint8_t* packed, void* stream) {
    hipStream_t s = (hipStream_t)stream;
    std::lock_guard<std::mutex> lock(g_pack_mutex);
    if (!g_pack_flag && hipHostMalloc((void**)&g_pack_flag, sizeof(int), hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
        g_pack_flag = nullptr;
        return VLUT_ERR_DEVICE;
    }
    volatile int* flag = g_pack_flag;
    *flag = 0;
    int rc = K5 > 0 ? launch_pack<5>(w, M, K, K5, packed, s) : VLUT_OK;
    if (rc == VLUT_OK && K > K5)
        rc = launch_pack<4>(w + K5, M, K, K - K5, packed + (K5 > 0 ? (size_t)((M + 3) / 4) * (size_t)((K5 / 5 + 15) / 16) * 64 : 0), s);
    // (waits also when the second launch failed: the flag must not be raised into a later call)
    if (hipStreamSynchronize(s) != hipSuccess) return VLUT_ERR_DEVICE;
    return rc != VLUT_OK ? rc : (*flag ? VLUT_ERR_VALUE : VLUT_OK);
}

// ---- up to sixteen tokens from fp32 (decode_kernel): one launch, every workgroup quantises all tokens.  Measured against
//      quantiser + gemm_kernel, launches back to back: 13824 x 2560 x 16 8.8 us (3.3 + 6.9 us as two), but 2560 x 6912 x 16 13.9 us
//      (11.6 us): the rows of x are read by every workgroup, so N * K is bounded; beyond 128 rows for
//      each of 256 workgroups that work is repeated (128256 x 4096 x 1 45 us, the table kernel 30 us), so M is bounded too.
//      One token and more than 64 rows for each of 256 workgroups: unpacking twice as many bytes per workgroup costs more than the
//      table kernel's lookups, where its one launch from fp32 covers K (decode / table: 32768 x 4096 11.7 / 9.9 us, 32768 x 14336
//      30.1 / 24.9; 16384 x 4096 8.2 / 8.0, 16384 x 6912 10.3 / 10.7; below K = 1024 level; two tokens, 32768 x 4096 12.0 / 12.6).
//      9 to 16 tokens: a wave quantises a whole row, so the time grows with N * K, while the table kernel with 32 rows per workgroup
//      spreads the tokens over workgroups; its time grows with their number, hence with M.  The line between them is fitted to
//      M = 4 to 1000 (decode / table: 100 x 4096 x 12 8.2 / 8.7 us, 100 x 4680 x 14 10.3 / 9.5, 4 x 6552 x 9 11.5 / 10.6; 1000 x 4096 x 16
//      level): within 3 % of the faster one, 5 % at M = 4.
//      All of this is older than decode_codes_kernel behind the quantiser, which these rules don't weigh, and than the shorter quantisation in
//      decode_kernel.  Graph replays, one launch / two, now: table kernel 100 x 4680 x 14 8.5 / 6.3 us, 1000 x 4680 x 14 8.8 / 6.3; decode_kernel
//      100 x 4096 x 12 5.7 / 5.65, 2560 x 6912 x 8 7.1 / 6.9, but 2560 x 2560 x 16 5.0 / 5.8, 13824 x 2560 x 16 6.2 / 6.9, 640 x 2560 x 8
//      4.1 / 5.3, 13824 x 2560 x 1 4.5 / 6.2.
constexpr int64_t kDecodeMaxValues = 65536;
bool decode_applies(int64_t M, int64_t K, int64_t N) {
    if (lookup_plan_forced() || N > 16 || N * K > kDecodeMaxValues || M > 256 * 128) return false;
    if (N == 1 && M > 256 * 64 && K >= 1024 && narrow_plan(M, K, N).chunks <= narrow_fused_max_chunks(1)) return false;
    if (N > 8 && N * K >= 49152 + 12 * M && narrow_applies(M, K, N, nullptr, true) && narrow_plan(M, K, N).rows == 32) return false;
    return true;
}
int decode_token_slots(int64_t N) { return N <= 2 ? (int)N : (N <= 4 ? 4 : (N <= 8 ? 8 : 16)); }
// Row tiles of 16 per workgroup: the fewest whose grid is one round of workgroups (more waves per row tile split K finer).
int decode_row_tiles(int64_t M) { return M <= 256 * 16 ? 1 : (M <= 256 * 32 ? 2 : (M <= 256 * 64 ? 4 : 8)); }

// ---- vlut_mpgemm_f32: which kernels run and how the caller's workspace is divided
enum { kF32Narrow = 0, kF32Fused = 1, kF32TwoLaunches = 2 };
struct F32Layout {
    int kind;                                    // also the division of the workspace where decode_kernel takes the call
    bool decode;                                 // decode_kernel takes the call (and leaves the workspace alone)
    Plan plan;                                   // kF32Fused
    size_t off_scale, off_aq, off_ws, total;     // byte offsets into the workspace
};

size_t round256(size_t v) { return (v + 255) & ~(size_t)255; }

F32Layout work_out_f32_layout(int64_t M, int64_t K, int64_t N) {
    F32Layout L;
    std::memset(&L, 0, sizeof(L));
    L.decode = decode_applies(M, K, N);
    const size_t scale_bytes = round256((size_t)N * sizeof(float));
    if (narrow_applies(M, K, N, nullptr, true) && narrow_plan(M, K, N).chunks <= narrow_fused_max_chunks(N == 1 ? 1 : 2)) {
        L.kind = kF32Narrow;
        return L;
    }
    // More than two tokens: measured, quantising inside the lookup kernel loses against a kernel of its own ahead of
    // it (every workgroup reads the whole rows of its 8 tokens and 16 row tiles repeat the work: +5.6 us on the
    // lookup kernel at M = 6912, K = 2560, N = 128, against 3.2 us + the gap between two kernels).  The fused form
    // is therefore only taken when a launch plan is forced (an override selects the kernel too).
    const bool fused = lookup_plan_forced() && choose_fused_plan(M, K, N, &L.plan);
    if (fused) {
        L.kind = kF32Fused;
        if (L.plan.S > 1) {                      // the second kernel reads the scales from memory
            L.off_ws = scale_bytes;
            L.total = L.off_ws + (size_t)L.plan.S * (size_t)M * (size_t)N * sizeof(int32_t);
        }
        return L;
    }
    L.kind = kF32TwoLaunches;                    // quantise into the workspace, then the ordinary path
    // (N unused floats ahead of the codes of a large input: callers may hold a workspace of the size this call has always had)
    L.off_aq = scale_bytes + ((N * K >= ((int64_t)1 << 22) && N >= 64) ? scale_bytes : 0);
    L.off_ws = L.off_aq + round256((size_t)((N + 7) / 8) * (size_t)K * 8);
    const bool narrow = narrow_applies(M, K, N, nullptr, false);
    const Plan pl = narrow ? Plan{4, 1, 1, 4} : choose_plan(M, K, N);
    L.plan = pl;
    L.total = L.off_ws + (pl.S > 1 ? (size_t)pl.S * (size_t)M * (size_t)N * sizeof(int32_t) : 0);
    return L;
}

// (kept like the routes from codes, in a smaller table with the same kind of places; asked for twice per call)
struct F32Entry {
    int64_t M, K, N;
    F32Layout layout;
};
constexpr int kF32Entries = 16;
thread_local F32Entry t_f32[kF32Entries];
const F32Layout& f32_layout(int64_t M, int64_t K, int64_t N) {
    F32Entry& e = t_f32[(unsigned)(M * 5 + K * 3 + N * 7 + (M >> 5) + (K >> 5)) % kF32Entries];
    if (e.M != M || e.K != K || e.N != N) e = {M, K, N, work_out_f32_layout(M, K, N)};
    return e.layout;
}

// ---- 1.60-bit (g = 5) host side
struct Plan5 {
    int R, S;
};
thread_local Plan5 t_forced5 = {0, 0};
constexpr int kSupportedR5[] = {1, 2, 4, 6, 9, 12, 14};

bool shape5_ok(int64_t M, int64_t K, int64_t N) {
    return M >= 1 && N >= 1 && K >= 5 && (K % 5) == 0 && M < kMaxDim && K < kMaxDim && N < kMaxDim;
}

struct Derived5 {
    int G, KCn, RGtotal, tiles_n, tiles_m, RGW, dstages_total, dstages_per_split, total, per_xcd;
    bool need32;
};

Derived5 derive5(const Plan5& pl, int64_t M, int64_t K, int64_t N) {
    Derived5 d;
    d.G = (int)(K / 5);
    d.KCn = (d.G + 15) / 16;
    d.RGtotal = (int)((M + 3) / 4);
    d.tiles_n = (int)((N + 7) / 8);
    int cap = kLookupWaves5 * pl.R;
    d.tiles_m = (d.RGtotal + cap - 1) / cap;
    d.RGW = (d.RGtotal + d.tiles_m - 1) / d.tiles_m;
    d.dstages_total = (d.G + 63) / 64;
    d.dstages_per_split = (d.dstages_total + pl.S - 1) / pl.S;
    d.total = d.tiles_m * d.tiles_n * pl.S;
    d.per_xcd = (d.total + 7) / 8;
    d.need32 = d.dstages_per_split * 4 > kBlockLookups5;
    return d;
}

bool plan5_valid(const Plan5& pl, int64_t M, int64_t K, int64_t N) {
    bool ok = false;
    for (int v : kSupportedR5) ok = ok || v == pl.R;
    if (!ok || pl.S < 1 || pl.S > 16) return false;
    Derived5 d = derive5(pl, M, K, N);
    if (d.need32 && pl.R > 6) return false;
    return pl.S <= d.dstages_total;
}

// R == 0 in the result: the override of vlut_set_plan_g5 fits this shape with no value of the free parameter
// (plan5_valid is then false and the callers report VLUT_ERR_UNSUPPORTED).
Plan5 choose_plan5(int64_t M, int64_t K, int64_t N) {
    Plan5 best = {0, 0};
    double best_cost = 1e300;
    const int Ss[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
    for (int R : kSupportedR5)
        for (int S : Ss) {
            Plan5 pl = {t_forced5.R > 0 ? t_forced5.R : R, t_forced5.S > 0 ? t_forced5.S : S};
            if (!plan5_valid(pl, M, K, N)) continue;
            Derived5 d = derive5(pl, M, K, N);
            double rw = (double)((d.RGW + kLookupWaves5 - 1) / kLookupWaves5);
            // a dword stage = four half-stages; each writes a 62 KB slot and reads it rw times per lookup wave
            double wg = d.dstages_per_split * 4.0 * (1900.0 + 75.0 * rw) + 5900.0 + 840.0 * rw;
            double t = (double)((d.total + 255) / 256) * wg;
            if (pl.S > 1) t += 5000.0 + 600.0 * pl.S;
            if (t < best_cost) { best_cost = t; best = pl; }
        }
    return best;
}

template <int R, bool NEED32>
int launch_lookup5_t(const Lookup5Params& p, int grid, hipStream_t stream) {
    auto kfn = lookup5_kernel<R, NEED32>;
    static std::atomic<unsigned> attr_done{0};   // one bit per device: the attribute belongs to the device's copy
    if (!allow_dynamic_lds((const void*)kfn, kLds5Bytes, attr_done)) return VLUT_ERR_DEVICE;
    Lookup5Params q = p;
    if (q.S > 1 || q.partial) q.out_vec = ((uintptr_t)q.ws % 16 == 0) && (q.M % 4 == 0);
    else q.out_vec = !q.y || (((uintptr_t)q.y % 16 == 0) && (q.ldy % 4 == 0));
    return launch(kfn, dim3(grid), kThreads, kLds5Bytes, stream, q);
}

template <bool NEED32>
int launch_lookup5_r(int R, const Lookup5Params& p, int grid, hipStream_t stream);

constexpr bool lookup5_instance_built(int R, bool need32) {
    for (int v : kSupportedR5)
        if (v == R) return !need32 || R <= 6;
    return false;
}

template <bool NEED32, int R = 1>
int launch_lookup5_by_r(int r, const Lookup5Params& p, int grid, hipStream_t stream) {
    if constexpr (R > 14) {
        return VLUT_ERR_UNSUPPORTED;
    } else {
        if constexpr (lookup5_instance_built(R, NEED32)) {
            if (r == R) return launch_lookup5_t<R, NEED32>(p, grid, stream);
        }
        return launch_lookup5_by_r<NEED32, R + 1>(r, p, grid, stream);
    }
}

template <bool NEED32>
int launch_lookup5_r(int R, const Lookup5Params& p, int grid, hipStream_t stream) {
    return launch_lookup5_by_r<NEED32>(R, p, grid, stream);
}

// ---- quantiser: tokens per workgroup and threads by the shape, rows in registers whether they are aligned or not (reading
//      unaligned ones twice, eight loads at a time, costs 21 us instead of 5.6 at N = 4096, K = 1024).  Measured, us:
//        one token per workgroup up to K = 1024 (K = 768, N = 4096: 5.2; four tokens 6.7), up to N = 1536 while K <= 3072 (K = 2560,
//        N = 1024 / 2000: 4.7 / 7.0; four tokens 4.9 / 6.5), up to N = 768 beyond (K = 6912, N = 512 / 1024: 5.7 / 8.9; four tokens 7.4 / 8.4)
//        eight tokens from N = 3584 on while K <= 3072 (K = 2560, N = 3000 / 4096: 9.6 / 11.2; four tokens 9.3 / 12.1)
template <bool VEC>
int launch_quantize(const float* x, int64_t N, int64_t K, int64_t ldx, int8_t* a_q, float* a_scale, int chunks, hipStream_t s) {
    const unsigned blocks8 = (unsigned)((chunks + 7) / 8);       // groups of eight chunks, one per XCD
    auto run = [&](auto kfn, unsigned grid, int threads) { return launch(kfn, dim3(grid), threads, 0, s, x, (int)N, (int)K, ldx, a_q, a_scale, chunks); };
    if (K <= 256) return run(quantize_token_kernel<64, 1, VEC>, blocks8 * 64, 64);
    if (K <= 1024) return run(quantize_token_kernel<256, 1, VEC>, blocks8 * 64, 256);
    if (N < (K <= 3072 ? 1536 : 768)) {
        constexpr int T = kTokThreads;
        if (K <= 4096) return run(quantize_token_kernel<T, 2, VEC>, blocks8 * 64, T);
        if (K <= 8192) return run(quantize_token_kernel<T, 4, VEC>, blocks8 * 64, T);
        if (K <= 16384) return run(quantize_token_kernel<T, 8, VEC>, blocks8 * 64, T);
        return run(quantize_token_kernel<T, 0, VEC>, blocks8 * 64, T);
    }
    if (N >= 3584 && K <= 3072) {
        if (K <= 1536) return run(quantize_kernel<8, 3, VEC>, (unsigned)chunks, kQuantThreads);
        if (K <= 2048) return run(quantize_kernel<8, 4, VEC>, (unsigned)chunks, kQuantThreads);
        return run(quantize_kernel<8, 6, VEC>, (unsigned)chunks, kQuantThreads);
    }
    if (K <= 2048) return run(quantize_kernel<4, 2, VEC>, blocks8 * 16, kQuantThreads);
    if (K <= 3072) return run(quantize_kernel<4, 3, VEC>, blocks8 * 16, kQuantThreads);
    if (K <= 4096) return run(quantize_kernel<4, 4, VEC>, blocks8 * 16, kQuantThreads);
    if (K <= 8192) return run(quantize_kernel<4, 8, VEC>, blocks8 * 16, kQuantThreads);
    if (K <= 14336) return run(quantize_kernel<4, 14, VEC>, blocks8 * 16, kQuantThreads);
    return run(quantize_kernel<4, 0, VEC>, blocks8 * 16, kQuantThreads);
}

// ---- matrix-core path (gemm_kernel): products with streamed tables, unless a plan of the lookup kernels is forced or a rule below says otherwise
double gemm_cost(int gw, int tile, int64_t M, int64_t macros, int64_t N) {
    const GemmTile t = gemm_tile(tile);
    const int g = gw - 4;
    const int64_t tiles = ((M + t.rows() - 1) / t.rows()) * ((N + t.tokens() - 1) / t.tokens());
    const double n = (double)((tiles + 255) / 256), passes = (double)((macros + t.wk - 1) / t.wk);
    return t.base[g] + (double)((tiles + 256 * t.per_unit[g] - 1) / (256 * t.per_unit[g])) * t.fixed[g] + 1e-6 * (double)M * (double)N * t.store[g] + passes * (t.lat[g] + n * t.pass[g]);
}

int choose_gemm_tile(int gw, int64_t M, int64_t macros, int64_t N) {
    int best = -1;
    double best_cost = 1e300;
    for (int i = 0; i < kGemmTileCount + kGemmTilesLongCount; ++i) {
        if (!gemm_tile_considered(gw, i, macros)) continue;
        const double c = gemm_cost(gw, i, M, macros, N);
        if (c < best_cost) { best_cost = c; best = i; }
    }
    return best;
}

int gemm_macros(int gw, int64_t K) { return (int)(((K / gw + 15) / 16 + 1) / 2); }

double gemm_best_cost(int gw, int64_t M, int64_t K, int64_t N) {
    const int macros = gemm_macros(gw, K);
    return gemm_cost(gw, choose_gemm_tile(gw, M, macros, N), M, macros, N);
}

// decode_codes_kernel for a few tokens: eight or sixteen per workgroup (ch chunks) and 16 * mt rows; ch = 0: not this kernel.  Its time in
// us, launches back to back in a stream (graph replays: 0.5 to 0.9 less), fitted (rms 3.7 %) to 18000 launches over 4100 shapes of 200 to 14336
// rows, K = 256 to 14336 and 16 to 1024 tokens: a launch and two trips to memory, then K times what a workgroup copies and unpacks,
// weights beyond 27 MB from further away, the store; beyond one workgroup per compute unit further rounds, shorter where two of them share a unit: their LDS fits and
// their 16 waves each take at most 64 registers (four weights per byte: 60 to 62; five: 75 to 77, never two).  Five weights per byte cost the
// same otherwise (us, gemm_kernel / this one: 4096 x 4096 x 32 mixed 6.6 / 5.8, 4096 x 4000 x 16 6.5 / 4.8, 2560 x 6900 x 8 7.7 / 4.8, but
// 13820 x 2560 x 64 7.7 / 11.9, 3079 x 360 x 233 4.8 / 6.7, 8624 x 1640 x 170 11.0 / 13.9, 12659 x 2020 x 98 12.0 / 15.0).
struct CodesPlan {
    int ch, mt;
    double us;
};
CodesPlan codes_plan(int gw, int64_t M, int64_t K, int64_t N) {
    CodesPlan best = {0, 0, 1e300};
    if (gw == 4 && lookup_plan_forced()) return best;
    const double mb = (double)M * (double)K / (gw * 1e6);
    for (int ch = 1; ch <= 2; ++ch) {
        if (!decode_codes_fits(gw, ch, K) || (ch == 2 && N <= 8)) continue;
        const bool two_per_unit = gw == 4 && decode_codes_lds_bytes(gw, ch, K) <= 80 * 1024;
        for (int mt = 1; mt <= 8; mt *= 2) {
            const int64_t wgs = ((M + 16 * mt - 1) / (16 * mt)) * ((N + 8 * ch - 1) / (8 * ch)), rounds = (wgs + 255) / 256;
            double us = 3.45 + (double)K * (ch == 1 ? 0.51e-4 + 1.31e-4 * mt : 1.29e-4 + 1.34e-4 * mt) + 0.00073 * (double)std::min<int64_t>(wgs, 256);
            us += 0.024 * std::max(0.0, mb - 27.5) + 0.52e-6 * (double)M * (double)N;
            if (rounds > 1) us = 3.06 + (double)rounds * (us - 3.06) * (two_per_unit ? 0.9 : 1.18);
            if (us < best.us) best = {ch, mt, us};
        }
    }
    return best;
}
// Where the few-token table kernel would run: always (beyond 32768 rows workgroups of 128 rows repeat the copy: left to that kernel).  us, table
// kernel / this one: 256 x 256 x 1 3.43 / 3.36, 640 x 2560 x 4 5.5 / 3.7, 2560 x 6912 x 2 9.8 / 4.4, 14336 x 14336 x 1 16.3 / 14.0.
// Else against the tiles of gemm_kernel (us, gemm_kernel / this one: 2560 x 2560 x 16 5.5 / 4.05, 2560 x 6912 x 16 7.5 / 5.3,
// 6912 x 2560 x 32 5.6 / 5.1, but 6912 x 2560 x 64 5.9 / 6.7, 13824 x 2560 x 32 5.9 / 6.7).
CodesPlan codes_plan_if_taken(int gw, int64_t M, int64_t K, int64_t N, bool narrow) {
    CodesPlan pl = codes_plan(gw, M, K, N);
    if (narrow ? M > 256 * 128 : pl.us >= gemm_best_cost(gw, M, K, N)) pl.ch = 0;
    return pl;
}

// Time of a lookup plan (with its split-K sum) in us, in the units of gemm_cost: least squares over 869 shapes of 4 to 4096 rows,
// K = 1024 to 65532 and 3 to 400 tokens, launches back to back (standard deviation 2.6 %, worst 12 % at 4 rows).  plan_cost above ranks plans
// and overstates the time, by 6 % where a workgroup has several tiles and by 20 to 57 % where it has one.
double lookup_us(const Plan& pl, int64_t M, int64_t K, int64_t N) {
    const Derived d = derive(pl, M, K, N);
    const int lookup_waves = kWaves - pl.BW;
    const double rw = (double)((d.RGW + lookup_waves - 1) / lookup_waves);   // row groups of the slowest lookup wave
    double stage = pl.BW == 4 ? 0.99 + 0.07 * rw : std::max(1.32, 0.72 + 0.102 * rw);
    if (d.need32) stage *= 1.05;
    double t = 3.8 + (double)((d.total + 255) / 256) * (d.stages_per_split * stage + 0.058 * rw);
    if (pl.S > 1) t += 1.65 + 0.07 * pl.S + 3.8e-6 * (double)pl.S * (double)M * (double)N;
    return std::max(t, (double)d.tiles_n * (double)d.RGtotal * d.KCn * 64.0 / (256.0 * 24.0 * 2100.0));   // weights from L2
}

// Few rows and tokens with a K that decode_codes_kernel does not hold leave the matrix-core path a handful of workgroups, while the lookup
// kernel can split K over many (with the partial sums in the workspace).  us, lookup / gemm_kernel: 16 x 65532 x 33 23.3 / 33.5, 16 x 32768
// x 33 14.3 / 18.4, 64 x 16384 x 128 10.3 / 10.7, 100 x 24000 x 72 13.4 / 14.7; but 640 x 30000 x 33 18.5 / 17.9, 2048 x 36000 x 20 22.8 / 20.8,
// 1280 x 65532 x 64 43.3 / 39.0, 2560 x 20480 x 16 15.0 / 12.6.  The lookup kernel keeps a call up to 1.25 times gemm_kernel's fitted time: that
// is where the line was before gemm_kernel unpacked by permutes, and from about 500 rows on it is now up to a fifth too far out.
bool matrix_cores_take(const Plan& pl, int64_t M, int64_t K, int64_t N) {
    if (lookup_plan_forced()) return false;
    return decode_codes_fits(4, 1, K) || lookup_us(pl, M, K, N) >= 1.25 * gemm_best_cost(4, M, K, N);
}
bool matrix_cores_take_g5(int64_t K) { return t_forced5.R == 0 && t_forced5.S == 0 && K % 4 == 0; }
bool matrix_cores_take_mixed() { return t_forced5.R == 0 && t_forced5.S == 0 && !lookup_plan_forced(); }

template <int GW, int I>
int launch_gemm_t(const GemmParams& p, hipStream_t stream) {
    constexpr GemmTile t = gemm_tile(I);
    constexpr bool own = gemm_private_built(GW, t.wm, t.wk), ring = gemm_ring_built(GW, t.rt, t.ct, t.wm, t.wk);
    void (*kfn)(GemmParams);
    if constexpr (own) kfn = gemm_private_kernel<t.rt, t.ct, t.wk>;
    else if constexpr (ring) kfn = gemm_ring_kernel<t.rt, t.ct, t.wm, t.wk>;
    else kfn = gemm_kernel<GW, t.rt, t.ct, t.wm, t.wk>;
    constexpr int lds = own ? PrivateShape<t.rt, t.ct, t.wk>::kLds : ring ? ring_lds_bytes<t.rt, t.ct, t.wm, t.wk>() : gemm_lds_bytes<GW, t.rt, t.ct, t.wm, t.wk>();
    static_assert(lds <= 160 * 1024, "LDS of a workgroup");
    static std::atomic<unsigned> attr_done{0};   // one bit per device: the attribute belongs to the device's copy
    if (!allow_dynamic_lds((const void*)kfn, lds, attr_done)) return VLUT_ERR_DEVICE;
    GemmParams q = p;
    q.tiles_n = (q.N + t.tokens() - 1) / t.tokens();
    q.tiles = (q.M + t.rows() - 1) / t.rows() * q.tiles_n;
    q.per_xcd = (q.tiles + 7) / 8;
    return launch(kfn, dim3(8 * q.per_xcd), 64 * t.wm * t.wk, lds, stream, q);
}

template <int GW, int I = 0>
int launch_gemm_tile(int tile, const GemmParams& p, hipStream_t stream) {
    if constexpr (I >= kGemmTileCount + kGemmTilesLongCount) {
        return VLUT_ERR_UNSUPPORTED;
    } else {
        if constexpr (gemm_tile_built(GW, I)) {
            if (tile == I) return launch_gemm_t<GW, I>(p, stream);
        }
        return launch_gemm_tile<GW, I + 1>(tile, p, stream);
    }
}

// K5 values of K five to a byte (0: none), the rest of K four to a byte behind them (at most 16 values if K5 > 0).
int launch_gemm(const uint8_t* packed, float w_scale, const float* w_rows, const int8_t* a_q, const float* a_scale, int64_t M,
                int64_t K, int64_t K5, int64_t N, float* y, int64_t ldy, int32_t* acc, hipStream_t stream, int tile) {
    GemmParams p;
    std::memset(&p, 0, sizeof(p));
    const int gw = K5 > 0 ? 5 : 4;
    p.packed = packed; p.a_q = a_q; p.a_scale = a_scale; p.w_rows = w_rows; p.y = y; p.acc = acc; p.w_scale = w_scale;
    p.M = (int)M; p.N = (int)N; p.Ka = (int)K; p.ldy = (int)ldy; p.RGtotal = (int)((M + 3) / 4); p.chunks = (int)((N + 7) / 8);
    p.Kmain = (int)(K5 > 0 ? K5 : K);
    p.KCn = (p.Kmain / gw + 15) / 16;
    p.macros = gemm_macros(gw, p.Kmain);
    // an output beyond half of the L2s (32 MB) is not kept there: 14336 x 4096 x 512 37.4 -> 35.4 us.  Who reads y next pays about what
    // the store saves: with quantise, clamp or sigmoid behind it 47.5, 48.0, 54.1 us, 47.5, 47.9, 53.8 with ordinary stores; nine
    // shapes from 17 to 84 MB with a reader are within 2 % either way
    p.stream_out = M * N * 4 >= ((int64_t)16 << 20);
    if (K5 > 0 && K > K5) {
        p.packed4 = packed + (size_t)p.RGtotal * p.KCn * 64;
        p.KCn4 = (int)(((K - K5) / 4 + 15) / 16);
    }
    return gw == 5 ? launch_gemm_tile<5>(tile, p, stream) : launch_gemm_tile<4>(tile, p, stream);
}

template <int T, int MT>
int launch_decode_t(const DecodeParams& p, hipStream_t stream) {
    auto kfn = decode_kernel<T, MT>;
    const int lds = decode_lds_bytes(T, p.macros);
    if (lds > 160 * 1024) return VLUT_ERR_UNSUPPORTED;      // (cannot happen within decode_applies)
    static std::atomic<unsigned> attr_done{0};   // one bit per device: the attribute belongs to the device's copy
    if (!allow_dynamic_lds((const void*)kfn, 160 * 1024, attr_done)) return VLUT_ERR_DEVICE;
    return launch(kfn, dim3((unsigned)((p.M + 16 * MT - 1) / (16 * MT))), 64 * kDecodeWaves, lds, stream, p);
}

template <int T>
int launch_decode(const DecodeParams& p, hipStream_t stream) {
    switch (decode_row_tiles(p.M)) {
    case 1: return launch_decode_t<T, 1>(p, stream);
    case 2: return launch_decode_t<T, 2>(p, stream);
    case 4: return launch_decode_t<T, 4>(p, stream);
    default: return launch_decode_t<T, 8>(p, stream);
    }
}

// ---- a few tokens from INT8 codes (decode_codes_kernel)
template <int GW, int CH, int MT>
int launch_codes_t(const DecodeParams& p, hipStream_t stream) {
    auto kfn = decode_codes_kernel<GW, CH, MT>;
    if (!decode_codes_fits(GW, CH, p.K)) return VLUT_ERR_UNSUPPORTED;      // (cannot happen: codes_plan)
    static std::atomic<unsigned> attr_done{0};   // one bit per device: the attribute belongs to the device's copy
    if (!allow_dynamic_lds((const void*)kfn, 160 * 1024, attr_done)) return VLUT_ERR_DEVICE;
    DecodeParams q = p;
    q.chunks = (q.N + 7) / 8;
    q.pitch = decode_codes_pitch(GW, q.K);
    q.tiles_n = (q.chunks + CH - 1) / CH;
    q.magic_n = q.tiles_n > 1 ? (unsigned)(((uint64_t)1 << 32) / (unsigned)q.tiles_n) + 1u : 0u;      // exact while tiles * tiles_n < 2^32
    const int64_t tiles = (int64_t)((q.M + 16 * MT - 1) / (16 * MT)) * q.tiles_n;
    if (tiles * q.tiles_n >= ((int64_t)1 << 32) || tiles > INT32_MAX / 2) return VLUT_ERR_UNSUPPORTED;     // (cannot happen: codes_plan)
    q.tiles = (int)tiles;
    q.per_xcd = (q.tiles + 7) / 8;
    return launch(kfn, dim3((unsigned)(8 * q.per_xcd)), 64 * kDecodeWaves, decode_codes_lds_bytes(GW, CH, q.K), stream, q);
}

template <int GW, int CH>
int launch_codes_mt(int mt, const DecodeParams& p, hipStream_t stream) {
    switch (mt) {
    case 1: return launch_codes_t<GW, CH, 1>(p, stream);
    case 2: return launch_codes_t<GW, CH, 2>(p, stream);
    case 4: return launch_codes_t<GW, CH, 4>(p, stream);
    default: return launch_codes_t<GW, CH, 8>(p, stream);
    }
}

// K5 values of K five to a byte (0: none), the rest of K four to a byte behind them (at most 16 values if K5 > 0).
int launch_codes(const CodesPlan& pl, const uint8_t* packed, float w_scale, const float* w_rows, const int8_t* a_q, const float* a_scale, int64_t M,
                 int64_t K, int64_t K5, int64_t N, float* y, int64_t ldy, int32_t* acc, hipStream_t stream) {
    DecodeParams q;
    std::memset(&q, 0, sizeof(q));
    const int gw = K5 > 0 ? 5 : 4;
    q.packed = packed; q.a_q = a_q; q.a_scale = a_scale; q.w_rows = w_rows; q.y = y; q.acc = acc; q.w_scale = w_scale;
    q.M = (int)M; q.N = (int)N; q.K = (int)K; q.RGtotal = (int)((M + 3) / 4); q.ldy = (int)ldy;
    q.Kmain = (int)(K5 > 0 ? K5 : K);
    q.KCn = (q.Kmain / gw + 15) / 16;
    q.macros = (q.KCn + 3) / 4;
    if (gw == 4) return pl.ch == 1 ? launch_codes_mt<4, 1>(pl.mt, q, stream) : launch_codes_mt<4, 2>(pl.mt, q, stream);
    if (K > K5) {
        q.packed4 = packed + (size_t)q.RGtotal * q.KCn * 64;
        q.KCn4 = (int)(((K - K5) / 4 + 15) / 16);
    }
    return pl.ch == 1 ? launch_codes_mt<5, 1>(pl.mt, q, stream) : launch_codes_mt<5, 2>(pl.mt, q, stream);
}

// ---- what a product from INT8 codes runs and demands: the rules above and the plans of the lookup kernels, which a call asks for twice (the
// size of the workspace, then the launch).  The last answers are kept per thread until a plan is forced or released, in a table where every
// shape has one place.  Shapes that fall on the same place replace each other: of a layer's four stacked matrices (3840, 2560, 13824 x 2560 and
// 2560 x 6912) the first and the last share one and the others another, so that in turn each is worked out once per call, which
// costs 0.03 to 0.2 us (2-bit), 0.6 (mixed) or 0.9 (1.60-bit, whose plans are searched anew) of a call of 4 to 5; repeated shapes are found.
enum { kRouteTables = 0, kRouteCodes = 1, kRouteGemm = 2 };
struct Route {
    int64_t M, K, N;                             // M = 0: none kept here
    int form, status;                            // status: VLUT_ERR_UNSUPPORTED where an override does not fit the shape
    int kernel, tile;                            // tile of gemm_kernel
    bool narrow;                                 // (2-bit) the few-token rule holds
    CodesPlan codes;
    Plan plan;                                   // of the lookup kernel (mixed: of the 2-bit part)
    Plan5 plan5;
    size_t demanded;                             // bytes of workspace that the call wants to see
    size_t used() const { return kernel == kRouteTables ? demanded : 0; }
};
constexpr int kRoutes = 32;
thread_local Route t_routes[kRoutes];
void forget_routes() {
    for (Route& r : t_routes) r.M = 0;
    for (F32Entry& e : t_f32) e.M = 0;
}

bool mixed_plans(int64_t M, int64_t K, int64_t N, Plan5* p5, Plan* p4);

// gw weights per byte in the main blob of Kmain values
void matrix_route(Route& r, int gw, int64_t Kmain) {
    r.codes = codes_plan_if_taken(gw, r.M, r.K, r.N, false);
    r.kernel = r.codes.ch ? kRouteCodes : kRouteGemm;
    if (!r.codes.ch) r.tile = choose_gemm_tile(gw, r.M, gemm_macros(gw, Kmain), r.N);
}

const Route& find_route(int form, int64_t M, int64_t K, int64_t N) {
    Route& r = t_routes[(unsigned)(M * 5 + K * 3 + N * 7 + form + (M >> 5) + (K >> 5)) % kRoutes];
    if (r.M == M && r.K == K && r.N == N && r.form == form) return r;
    r = Route{};
    r.M = M; r.K = K; r.N = N; r.form = form;
    const size_t sums = (size_t)M * (size_t)N * sizeof(int32_t);
    if (form == VLUT_FORM_CODES) {
        r.narrow = narrow_applies(M, K, N, nullptr, false);
        if (r.narrow) {
            r.codes = codes_plan_if_taken(4, M, K, N, true);
            r.kernel = r.codes.ch ? kRouteCodes : kRouteTables;
            return r;
        }
        r.plan = choose_plan(M, K, N);
        if (r.plan.R == 0) r.status = VLUT_ERR_UNSUPPORTED;
        else if (matrix_cores_take(r.plan, M, K, N)) matrix_route(r, 4, K);
        r.demanded = r.plan.S > 1 ? (size_t)r.plan.S * sums : 0;
    } else if (form == VLUT_FORM_G5) {
        r.plan5 = choose_plan5(M, K, N);
        if (!plan5_valid(r.plan5, M, K, N)) r.status = VLUT_ERR_UNSUPPORTED;
        else if (matrix_cores_take_g5(K)) matrix_route(r, 5, K);
        r.demanded = r.plan5.S > 1 ? (size_t)r.plan5.S * sums : 0;
    } else {
        const int64_t K5 = (K / 20) * 20;
        if (!mixed_plans(M, K, N, &r.plan5, &r.plan)) {
            r.status = VLUT_ERR_UNSUPPORTED;
            return r;
        }
        r.demanded = (size_t)(r.plan5.S + r.plan.S) * sums;
        if (matrix_cores_take_mixed()) matrix_route(r, K5 > 0 ? 5 : 4, K5 > 0 ? K5 : K);
    }
    return r;
}

// The mixed packing as launches of the lookup kernels in partial-sum mode, then one exact INT32 sum + scale step.
// Workspace: [S5 + S4][N][M] INT32.
bool mixed_plans(int64_t M, int64_t K, int64_t N, Plan5* p5, Plan* p4) {
    const int64_t K5 = (K / 20) * 20, K4 = K - K5;
    if (K5 > 0) {
        *p5 = choose_plan5(M, K5, N);
        if (!plan5_valid(*p5, M, K5, N)) return false;
    } else {
        *p5 = Plan5{0, 0};
    }
    *p4 = K4 > 0 ? choose_plan(M, K4, N) : Plan{0, 0, 0, 0};
    if (K4 > 0 && p4->R == 0) return false;              // the override of vlut_set_plan does not fit the 2-bit part
    return true;
}

// The workspace of a call that demands r.demanded bytes (lean: r.used() if none is handed over)
int check_workspace(const Route& r, const void* workspace, size_t bytes, bool lean) {
    const size_t need = lean && !workspace ? r.used() : r.demanded;
    if (need == 0) return VLUT_OK;
    return !workspace ? VLUT_ERR_NULL : bytes < need ? VLUT_ERR_SMALL_BUFFER : VLUT_OK;
}

int launch_matrix_route(const Route& r, const uint8_t* packed, float w_scale, const float* w_rows, const int8_t* a_q, const float* a_scale, int64_t K5,
                        float* y, int64_t ldy, int32_t* acc, hipStream_t s) {
    if (r.kernel == kRouteCodes) return launch_codes(r.codes, packed, w_scale, w_rows, a_q, a_scale, r.M, r.K, K5, r.N, y, ldy, acc, s);
    return launch_gemm(packed, w_scale, w_rows, a_q, a_scale, r.M, r.K, K5, r.N, y, ldy, acc, s, r.tile);
}

// ---- comparison path: tokens per workgroup from N, K split so that few tiles still give every CU a few workgroups
struct MfmaPlan {
    int BN, tiles_m, tiles_n, S, steps_per_split, grid;
};

MfmaPlan mfma_plan(int64_t M, int64_t K, int64_t N) {
    MfmaPlan mp;
    mp.BN = N > 64 ? 128 : (N > 32 ? 64 : (N > 16 ? 32 : 16));
    mp.tiles_m = (int)((M + kMfRows - 1) / kMfRows);
    // the kernel hides latency with resident waves only: narrower token tiles while the wide ones give a CU fewer
    // than about three workgroups
    if (mp.BN == 128 && (int64_t)mp.tiles_m * ((N + 127) / 128) < 768) mp.BN = 64;
    mp.tiles_n = (int)((N + mp.BN - 1) / mp.BN);
    const int steps = (int)((K / 4 + 15) / 16);
    const int64_t tiles = (int64_t)mp.tiles_m * mp.tiles_n;
    int S = 1;
    if (tiles < 512) {
        S = (int)((768 + tiles - 1) / tiles);                // about three workgroups per CU
        if (S > 16) S = 16;
        if (S > steps / 4) S = steps / 4 > 0 ? steps / 4 : 1;  // at least four K steps per split
    }
    mp.steps_per_split = (steps + S - 1) / S;
    mp.S = (steps + mp.steps_per_split - 1) / mp.steps_per_split;
    mp.grid = (int)(tiles * mp.S);
    return mp;
}

}  // namespace

extern "C" {

const char* vlut_status_string(int status) {
    switch (status) {
    case VLUT_OK: return "VLUT_OK";
    case VLUT_ERR_NULL: return "VLUT_ERR_NULL: a required pointer is NULL";
    case VLUT_ERR_SHAPE: return "VLUT_ERR_SHAPE: shape or leading dimension out of range";
    case VLUT_ERR_SMALL_BUFFER: return "VLUT_ERR_SMALL_BUFFER: buffer smaller than required";
    case VLUT_ERR_VALUE: return "VLUT_ERR_VALUE: weight outside {-1,0,+1}";
    case VLUT_ERR_DEVICE: return "VLUT_ERR_DEVICE: HIP call or kernel launch failed";
    case VLUT_ERR_UNSUPPORTED: return "VLUT_ERR_UNSUPPORTED: request not supported by this build";
    default: return "VLUT_ERR_UNKNOWN";
    }
}

int vlut_version(void) { return 100; }

size_t vlut_packed_weight_bytes(int64_t M, int64_t K) {
    if (!shape_ok(M, K, 1)) return 0;
    return (size_t)((M + 3) / 4) * (size_t)((K / 4 + 15) / 16) * 64;
}

size_t vlut_packed_offset(int64_t M, int64_t K, int64_t m, int64_t kg) {
    if (!shape_ok(M, K, 1) || m < 0 || m >= M || kg < 0 || kg >= K / 4) return (size_t)-1;
    size_t KCn = (size_t)((K / 4 + 15) / 16);
    return (((size_t)(m / 4) * KCn + (size_t)(kg / 16)) * 64) + (size_t)(m % 4) * 16 + (size_t)(kg % 16);
}

size_t vlut_act_bytes(int64_t K, int64_t N) {
    if (!shape_ok(1, K, N)) return 0;
    return (size_t)((N + 7) / 8) * (size_t)K * 8;
}

size_t vlut_lut_bytes(int64_t K, int64_t N) {
    if (!shape_ok(1, K, N)) return 0;
    return (size_t)(K / 4) * kRows * (size_t)N * sizeof(int16_t);
}

size_t vlut_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    if (!shape_ok(M, K, N)) return 0;
    // Where the few-token kernel serves the streamed path (no workspace), the materialised-table variant runs a
    // plan without split-K, so this one size serves both variants.
    return find_route(VLUT_FORM_CODES, M, K, N).demanded;
}

size_t vlut_workspace_used(int64_t M, int64_t K, int64_t N) {
    return shape_ok(M, K, N) ? find_route(VLUT_FORM_CODES, M, K, N).used() : 0;
}

int vlut_set_plan(int J, int R, int waves, int split_k) {
    int Jlog = -1;
    if (J != 0) {
        for (int e = 0; e <= 4; ++e)
            if ((1 << e) == J) Jlog = e;
        if (Jlog < 0) return VLUT_ERR_UNSUPPORTED;
    }
    if (R != 0 && !r_supported(R)) return VLUT_ERR_UNSUPPORTED;
    if (waves != 0 && waves != kWaves && waves != 12 && waves != 14) return VLUT_ERR_UNSUPPORTED;
    if (split_k < 0 || split_k > 16) return VLUT_ERR_UNSUPPORTED;
    t_forced = {Jlog, R, split_k, (waves == 12 || waves == 14) ? kWaves - waves : 0};
    t_cache_used = 0;
    t_cache_next = 0;
    t_fcache_used = 0;
    t_fcache_next = 0;
    forget_routes();
    return VLUT_OK;
}

int vlut_query_plan(int64_t M, int64_t K, int64_t N, int* out4) {
    if (!out4) return VLUT_ERR_NULL;
    if (!shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (narrow_applies(M, K, N, nullptr, false)) {   // the few-token kernel: J reported as 0, R = rows per workgroup
        const NarrowPlan np = narrow_plan(M, K, N);
        out4[0] = 0; out4[1] = np.rows; out4[2] = 1; out4[3] = np.gridx * np.pairs;
        return VLUT_OK;
    }
    Plan pl = choose_plan(M, K, N);
    if (pl.R == 0) return VLUT_ERR_UNSUPPORTED;          // the override does not fit this shape
    Derived d = derive(pl, M, K, N);
    out4[0] = 1 << pl.Jlog;
    out4[1] = pl.R;
    out4[2] = pl.S;
    out4[3] = d.total;
    return VLUT_OK;
}

int vlut_query_lookup_waves(int64_t M, int64_t K, int64_t N) {
    if (!shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (narrow_applies(M, K, N, nullptr, false)) return 0;
    const Plan pl = choose_plan(M, K, N);
    if (pl.R == 0) return VLUT_ERR_UNSUPPORTED;
    return kWaves - pl.BW;
}

int vlut_pack_weights(const int8_t* w_ternary, int64_t M, int64_t K, uint8_t* packed, size_t packed_bytes,
                      void* stream) {
    if (!shape_ok(M, K, 1)) return VLUT_ERR_SHAPE;
    if (!w_ternary || !packed) return VLUT_ERR_NULL;
    size_t need = vlut_packed_weight_bytes(M, K);
    if (packed_bytes < need) return VLUT_ERR_SMALL_BUFFER;
    return pack_parts(w_ternary, M, K, 0, packed, stream);
}

static int quantize_impl(const float* x, int64_t N, int64_t K, int64_t ldx, int8_t* a_q, float* a_scale, void* stream) {
    if (!shape_ok(1, K, N)) return VLUT_ERR_SHAPE;
    if (ldx < K) return VLUT_ERR_SHAPE;
    if (!x || !a_q || !a_scale) return VLUT_ERR_NULL;
    if (((uintptr_t)a_q) % 16 != 0) return VLUT_ERR_UNSUPPORTED;
    hipStream_t s = (hipStream_t)stream;
    const int chunks = (int)((N + 7) / 8);
    const bool vec = (((uintptr_t)x) % 16 == 0) && (ldx % 4 == 0);
    return vec ? launch_quantize<true>(x, N, K, ldx, a_q, a_scale, chunks, s) : launch_quantize<false>(x, N, K, ldx, a_q, a_scale, chunks, s);
}

int vlut_quantize_act(const float* x, int64_t N, int64_t K, int64_t ldx, int8_t* a_q, float* a_scale,
                      void* stream) {
    return quantize_impl(x, N, K, ldx, a_q, a_scale, stream);
}

int vlut_build_lut(const int8_t* a_q, int64_t K, int64_t N, int16_t* lut, size_t lut_bytes, void* stream) {
    if (!shape_ok(1, K, N)) return VLUT_ERR_SHAPE;
    if (!a_q || !lut) return VLUT_ERR_NULL;
    if (lut_bytes < vlut_lut_bytes(K, N)) return VLUT_ERR_SMALL_BUFFER;
    size_t total = (size_t)(K / 4) * (size_t)N;
    hipLaunchKernelGGL(build_lut_kernel<false>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       a_q, (int)(K / 4), (int)N, lut);
    return hipGetLastError() == hipSuccess ? VLUT_OK : VLUT_ERR_DEVICE;
}

int vlut_build_lut_token_outer(const int8_t* a_q, int64_t K, int64_t N, int16_t* lut, size_t lut_bytes, void* stream) {
    if (!shape_ok(1, K, N)) return VLUT_ERR_SHAPE;
    if (!a_q || !lut) return VLUT_ERR_NULL;
    if (lut_bytes < vlut_lut_bytes(K, N)) return VLUT_ERR_SMALL_BUFFER;
    size_t total = (size_t)(K / 4) * (size_t)N;
    hipLaunchKernelGGL(build_lut_kernel<true>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       a_q, (int)(K / 4), (int)N, lut);
    return hipGetLastError() == hipSuccess ? VLUT_OK : VLUT_ERR_DEVICE;
}

int vlut_mpgemm_token_outer(const uint8_t* packed, float w_scale, const float* a_scale, const int16_t* lut, int64_t M,
                            int64_t K, int64_t N, float* y, int64_t ldy, int32_t* acc_or_null, void* stream) {
    if (!shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (!packed || !a_scale || !lut) return VLUT_ERR_NULL;
    if (!y && !acc_or_null) return VLUT_ERR_NULL;
    if (y && (ldy < M || ldy > INT32_MAX)) return VLUT_ERR_SHAPE;
    const int G = (int)(K / 4), KCn = (G + 15) / 16;
    const dim3 grid((unsigned)((M + 63) / 64), (unsigned)((N + 3) / 4));
    if (grid.y > 65535u) return VLUT_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(token_outer_lookup_kernel, grid, dim3(256), 0, (hipStream_t)stream, packed, lut, (int)M, (int)N, G,
                       KCn, w_scale, a_scale, y, ldy, acc_or_null);
    return hipGetLastError() == hipSuccess ? VLUT_OK : VLUT_ERR_DEVICE;
}

static int mpgemm_impl(const uint8_t* packed, float w_scale, const float* w_rows, const int8_t* a_q, const float* a_scale,
                       const int16_t* lut_or_null, int64_t M, int64_t K, int64_t N, float* y, int64_t ldy,
                       int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream, bool lean = false) {
    int rc = check_mpgemm_args(packed, a_q, a_scale, M, K, N, y, ldy, acc_or_null);
    if (rc != VLUT_OK) return rc;
    if (((uintptr_t)a_q) % 16 != 0) return VLUT_ERR_UNSUPPORTED;      // the [N/8][K][8] blocks are read 16 bytes at a time
    if (((uintptr_t)packed) % 16 != 0) return VLUT_ERR_UNSUPPORTED;   // packed tiles are read up to 16 bytes at a time
    hipStream_t s = (hipStream_t)stream;
    Plan pl;
    if (!lut_or_null) {
        const Route& r = find_route(VLUT_FORM_CODES, M, K, N);
        if (r.status != VLUT_OK) return r.status;                     // the override of vlut_set_plan does not fit this shape
        rc = check_workspace(r, workspace, workspace_bytes, lean);
        if (rc != VLUT_OK) return rc;
        if (r.kernel != kRouteTables) return launch_matrix_route(r, packed, w_scale, w_rows, a_q, a_scale, 0, y, ldy, acc_or_null, s);
        if (r.narrow) {                                  // a few tokens: the workgroups sweep all of K, no workspace
            const NarrowPlan np = narrow_plan(M, K, N);
            NarrowParams q;
            std::memset(&q, 0, sizeof(q));
            q.packed = packed; q.a_q = a_q; q.a_scale = a_scale; q.w_rows = w_rows; q.y = y; q.acc = acc_or_null;
            q.w_scale = w_scale; q.M = (int)M; q.K = (int)K; q.N = (int)N; q.G = (int)(K / 4);
            q.KCn = (int)((K / 4 + 15) / 16); q.RGtotal = (int)((M + 3) / 4); q.ldy = (int)ldy; q.chunks = np.chunks;
            return launch_narrow<false>(np, q, s);
        }
        pl = r.plan;
    } else {
        // A materialised table where the streamed path would take the few-token kernel (and vlut_workspace_bytes says
        // 0): a plan without split-K, so that no workspace is needed here either.
        const int max_S = narrow_applies(M, K, N, nullptr, false) ? 1 : 16;
        pl = max_S == 1 ? search_plan(M, K, N, 1) : choose_plan(M, K, N);
        if (pl.R != 0 && pl.BW != 4) pl = search_plan(M, K, N, max_S, true);
        if (pl.R == 0) return VLUT_ERR_UNSUPPORTED;      // the override of vlut_set_plan does not fit this shape
        pl.R = pl.R >= 4 ? 4 : (pl.R >= 2 ? 2 : 1);      // the materialised-table variant is built for these R and four build waves only
        pl.BW = 4;
        if (pl.S > 1) {
            if (!workspace) return VLUT_ERR_NULL;
            if (workspace_bytes < (size_t)pl.S * (size_t)M * (size_t)N * sizeof(int32_t)) return VLUT_ERR_SMALL_BUFFER;
        }
    }
    const bool al = lut_or_null && (N % 8 == 0) && (((uintptr_t)lut_or_null) % 16 == 0);
    const int mode = lut_or_null ? kFromGlobal : kFast;
    const Derived d = derive(pl, M, K, N);
    LookupParams p;
    std::memset(&p, 0, sizeof(p));
    p.packed = packed; p.a_q = a_q; p.a_scale = a_scale; p.lut = lut_or_null;
    p.y = y; p.acc = acc_or_null; p.ws = (int32_t*)workspace; p.w_scale = w_scale; p.w_rows = w_rows;
    p.M = (int)M; p.K = (int)K; p.N = (int)N; p.G = d.G; p.KCn = d.KCn; p.RGtotal = d.RGtotal; p.ldy = (int)ldy;
    p.Jlog = pl.Jlog; p.S = pl.S; p.tiles_m = d.tiles_m; p.tiles_n = d.tiles_n; p.RGW = d.RGW;
    p.stages_total = d.stages_total; p.stages_per_split = d.stages_per_split;
    p.total_tiles = d.total; p.per_xcd = d.per_xcd;
    p.aligned8 = al ? 1 : 0;
    p.Ka = (int)K;
    rc = d.need32 ? launch_lookup_r<true>(pl.R, pl.BW, mode, p, s) : launch_lookup_r<false>(pl.R, pl.BW, mode, p, s);
    if (rc != VLUT_OK) return rc;
    if (pl.S > 1)
        return launch_splitk_reduce((const int32_t*)workspace, pl.S, M, N, w_scale, w_rows, a_scale, y, ldy, acc_or_null, s);
    return VLUT_OK;
}

int vlut_mpgemm(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale,
                const int16_t* lut_or_null, int64_t M, int64_t K, int64_t N, float* y, int64_t ldy,
                int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    return mpgemm_impl(packed, w_scale, nullptr, a_q, a_scale, lut_or_null, M, K, N, y, ldy, acc_or_null, workspace,
                       workspace_bytes, stream);
}

int vlut_mpgemm_lean(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, const int16_t* lut_or_null, int64_t M, int64_t K,
                     int64_t N, float* y, int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    return mpgemm_impl(packed, w_scale, nullptr, a_q, a_scale, lut_or_null, M, K, N, y, ldy, acc_or_null, workspace, workspace_bytes, stream, true);
}

size_t vlut_static_scratch_bytes(void) { return (size_t)VLUT_STATIC_SCRATCH_BYTES; }

int vlut_mpgemm_static(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K,
                       int64_t N, float* y, int64_t ldy, int32_t* acc_or_null, void* stream) {
    int rc = check_mpgemm_args(packed, a_q, a_scale, M, K, N, y, ldy, acc_or_null);
    if (rc != VLUT_OK) return rc;
    const size_t need = vlut_workspace_bytes(M, K, N);
    if (need > (size_t)VLUT_STATIC_SCRATCH_BYTES) return VLUT_ERR_UNSUPPORTED;   // partial sums beyond the built-in scratch
    void* ptr = nullptr;
    if (need > 0) {
        rc = static_scratch_ptr(&ptr);
        if (rc != VLUT_OK) return rc;
    }
    // Every partial-sum slot the second kernel reads is written by the first kernel of the same call, so nothing of
    // an earlier call's contents has to be cleared.
    return mpgemm_impl(packed, w_scale, nullptr, a_q, a_scale, nullptr, M, K, N, y, ldy, acc_or_null, ptr,
                       need > 0 ? (size_t)VLUT_STATIC_SCRATCH_BYTES : 0, stream);
}

int vlut_mpgemm_rows(const uint8_t* packed, const float* w_scale_rows, const int8_t* a_q, const float* a_scale,
                     const int16_t* lut_or_null, int64_t M, int64_t K, int64_t N, float* y, int64_t ldy,
                     int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    if (!w_scale_rows) return VLUT_ERR_NULL;
    return mpgemm_impl(packed, 1.0f, w_scale_rows, a_q, a_scale, lut_or_null, M, K, N, y, ldy, acc_or_null, workspace,
                       workspace_bytes, stream);
}

size_t vlut_workspace_bytes_f32(int64_t M, int64_t K, int64_t N) {
    if (!shape_ok(M, K, N)) return 0;
    return f32_layout(M, K, N).total;
}

int vlut_query_plan_f32(int64_t M, int64_t K, int64_t N, int* out5) {
    if (!out5) return VLUT_ERR_NULL;
    if (!shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    const F32Layout L = f32_layout(M, K, N);
    out5[4] = L.kind == kF32TwoLaunches && !L.decode ? 0 : 1;
    if (L.kind == kF32Fused) {
        const Derived d = derive(L.plan, M, K, N);
        out5[0] = 1 << L.plan.Jlog; out5[1] = L.plan.R; out5[2] = L.plan.S; out5[3] = d.total;
        return VLUT_OK;
    }
    if (L.kind == kF32Narrow) {                // reported as vlut_query_plan reports the few-token kernel
        const NarrowPlan np = narrow_plan(M, K, N);
        out5[0] = 0; out5[1] = np.rows; out5[2] = 1; out5[3] = np.gridx * np.pairs;
        return VLUT_OK;
    }
    if (L.decode) {
        const int rows = 16 * decode_row_tiles(M);
        out5[0] = 0; out5[1] = rows; out5[2] = 1; out5[3] = (int)((M + rows - 1) / rows);
        return VLUT_OK;
    }
    return vlut_query_plan(M, K, N, out5);
}

int vlut_mpgemm_f32(const uint8_t* packed, float w_scale, const float* w_scale_rows_or_null, const float* x, int64_t ldx,
                    int64_t M, int64_t K, int64_t N, float* y, int64_t ldy, int32_t* acc_or_null,
                    float* a_scale_out_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    if (!shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (!packed || !x) return VLUT_ERR_NULL;
    if (!y && !acc_or_null) return VLUT_ERR_NULL;
    if (y && (ldy < M || ldy > INT32_MAX)) return VLUT_ERR_SHAPE;
    if (ldx < K) return VLUT_ERR_SHAPE;
    if (((uintptr_t)packed) % 16 != 0) return VLUT_ERR_UNSUPPORTED;
    const F32Layout L = f32_layout(M, K, N);
    if (L.kind == kF32TwoLaunches && L.plan.R == 0) return VLUT_ERR_UNSUPPORTED;   // override does not fit the shape
    if (L.total > 0) {
        if (!workspace) return VLUT_ERR_NULL;
        if (workspace_bytes < L.total) return VLUT_ERR_SMALL_BUFFER;
        if (((uintptr_t)workspace) % 16 != 0) return VLUT_ERR_UNSUPPORTED;
    }
    hipStream_t s = (hipStream_t)stream;
    const int x_vec = ((((uintptr_t)x) % 16 == 0) && (ldx % 4 == 0)) ? 1 : 0;
    const float* w_rows = w_scale_rows_or_null;
    const float w_one = w_rows ? 1.0f : w_scale;
    char* ws = (char*)workspace;

    if (L.decode) {
        DecodeParams q;
        std::memset(&q, 0, sizeof(q));
        q.packed = packed; q.x = x; q.w_rows = w_rows; q.y = y; q.acc = acc_or_null; q.a_scale_out = a_scale_out_or_null;
        q.ldx = ldx; q.w_scale = w_one; q.M = (int)M; q.N = (int)N; q.K = (int)K; q.KCn = (int)((K / 4 + 15) / 16);
        q.RGtotal = (int)((M + 3) / 4); q.ldy = (int)ldy; q.macros = (q.KCn + 3) / 4;
        switch (decode_token_slots(N)) {
        case 1: return launch_decode<1>(q, s);
        case 2: return launch_decode<2>(q, s);
        case 4: return launch_decode<4>(q, s);
        case 8: return launch_decode<8>(q, s);
        default: return launch_decode<16>(q, s);
        }
    }
    if (L.kind == kF32Narrow) {
        const NarrowPlan np = narrow_plan(M, K, N);
        NarrowParams q;
        std::memset(&q, 0, sizeof(q));
        q.packed = packed; q.w_rows = w_rows; q.y = y; q.acc = acc_or_null; q.w_scale = w_one;
        q.M = (int)M; q.K = (int)K; q.N = (int)N; q.G = (int)(K / 4);
        q.KCn = (int)((K / 4 + 15) / 16); q.RGtotal = (int)((M + 3) / 4); q.ldy = (int)ldy; q.chunks = np.chunks;
        q.x = x; q.ldx = ldx; q.x_vec = x_vec; q.a_scale_out = a_scale_out_or_null;
        return launch_narrow<true>(np, q, s);
    }
    if (L.kind == kF32TwoLaunches) {
        float* scales = a_scale_out_or_null ? a_scale_out_or_null : (float*)(ws + L.off_scale);
        int8_t* a_q = (int8_t*)(ws + L.off_aq);
        int rc = quantize_impl(x, N, K, ldx, a_q, scales, stream);
        if (rc != VLUT_OK) return rc;
        return mpgemm_impl(packed, w_one, w_rows, a_q, scales, nullptr, M, K, N, y, ldy, acc_or_null, ws + L.off_ws,
                           L.total - L.off_ws, stream);
    }
    const Plan pl = L.plan;
    const Derived d = derive(pl, M, K, N);
    float* scales = a_scale_out_or_null;
    if (pl.S > 1 && !scales) scales = (float*)(ws + L.off_scale);
    LookupParams p;
    std::memset(&p, 0, sizeof(p));
    p.packed = packed; p.x = x; p.ldx = ldx; p.x_vec = x_vec; p.a_scale_out = scales; p.Ka = (int)K;
    p.y = y; p.acc = acc_or_null; p.ws = (int32_t*)(ws + L.off_ws); p.w_scale = w_one; p.w_rows = w_rows;
    p.M = (int)M; p.K = (int)K; p.N = (int)N; p.G = d.G; p.KCn = d.KCn; p.RGtotal = d.RGtotal; p.ldy = (int)ldy;
    p.Jlog = pl.Jlog; p.S = pl.S; p.tiles_m = d.tiles_m; p.tiles_n = d.tiles_n; p.RGW = d.RGW;
    p.stages_total = d.stages_total; p.stages_per_split = d.stages_per_split;
    p.total_tiles = d.total; p.per_xcd = d.per_xcd;
    int rc = d.need32 ? launch_lookup_r<true>(pl.R, pl.BW, kFusedQuant, p, s)
                      : launch_lookup_r<false>(pl.R, pl.BW, kFusedQuant, p, s);
    if (rc != VLUT_OK) return rc;
    if (pl.S > 1) {
        rc = launch_splitk_reduce((const int32_t*)(ws + L.off_ws), pl.S, M, N, w_one, w_rows, (const float*)scales, y, ldy,
                                  acc_or_null, s);
        if (rc != VLUT_OK) return rc;
    }
    return VLUT_OK;
}

// ---- 1.60-bit packing (g = 5)
size_t vlut_packed_weight_bytes_g5(int64_t M, int64_t K) {
    if (!shape5_ok(M, K, 1)) return 0;
    return (size_t)((M + 3) / 4) * (size_t)((K / 5 + 15) / 16) * 64;
}

size_t vlut_packed_offset_g5(int64_t M, int64_t K, int64_t m, int64_t kg) {
    if (!shape5_ok(M, K, 1) || m < 0 || m >= M || kg < 0 || kg >= K / 5) return (size_t)-1;
    size_t KCn = (size_t)((K / 5 + 15) / 16);
    return (((size_t)(m / 4) * KCn + (size_t)(kg / 16)) * 64) + (size_t)(m % 4) * 16 + (size_t)(kg % 16);
}

int vlut_pack_weights_g5(const int8_t* w_ternary, int64_t M, int64_t K, uint8_t* packed, size_t packed_bytes,
                         void* stream) {
    if (!shape5_ok(M, K, 1)) return VLUT_ERR_SHAPE;
    if (!w_ternary || !packed) return VLUT_ERR_NULL;
    size_t need = vlut_packed_weight_bytes_g5(M, K);
    if (packed_bytes < need) return VLUT_ERR_SMALL_BUFFER;
    return pack_parts(w_ternary, M, K, K, packed, stream);
}

size_t vlut_workspace_bytes_g5(int64_t M, int64_t K, int64_t N) {
    if (!shape5_ok(M, K, N)) return 0;
    return find_route(VLUT_FORM_G5, M, K, N).demanded;
}

size_t vlut_workspace_used_g5(int64_t M, int64_t K, int64_t N) {
    return shape5_ok(M, K, N) ? find_route(VLUT_FORM_G5, M, K, N).used() : 0;
}

int vlut_set_plan_g5(int R, int split_k) {
    if (R != 0) {
        bool ok = false;
        for (int v : kSupportedR5) ok = ok || v == R;
        if (!ok) return VLUT_ERR_UNSUPPORTED;
    }
    if (split_k < 0 || split_k > 16) return VLUT_ERR_UNSUPPORTED;
    t_forced5 = {R, split_k};
    forget_routes();
    return VLUT_OK;
}

int vlut_query_plan_g5(int64_t M, int64_t K, int64_t N, int* out3) {
    if (!out3) return VLUT_ERR_NULL;
    if (!shape5_ok(M, K, N)) return VLUT_ERR_SHAPE;
    Plan5 pl = choose_plan5(M, K, N);
    if (!plan5_valid(pl, M, K, N)) return VLUT_ERR_UNSUPPORTED;   // the override does not fit this shape
    Derived5 d = derive5(pl, M, K, N);
    out3[0] = pl.R; out3[1] = pl.S; out3[2] = d.total;
    return VLUT_OK;
}

static int mpgemm_g5_impl(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K, int64_t N, float* y,
                          int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream, bool lean) {
    if (!shape5_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (!packed || !a_q || !a_scale) return VLUT_ERR_NULL;
    if (!y && !acc_or_null) return VLUT_ERR_NULL;
    if (y && (ldy < M || ldy > INT32_MAX)) return VLUT_ERR_SHAPE;
    if (((uintptr_t)a_q) % 8 != 0) return VLUT_ERR_UNSUPPORTED;       // 5 rows x 8 tokens are read 8 bytes at a time
    const Route& r = find_route(VLUT_FORM_G5, M, K, N);
    if (r.status != VLUT_OK) return r.status;
    // the matrix-core path reads both operands 16 bytes at a time, so it wants the alignment and K % 4 == 0 (two activation
    // rows of a chunk are 16 bytes) that this call does not demand
    const bool matrix = r.kernel != kRouteTables && (uintptr_t)packed % 16 == 0 && (uintptr_t)a_q % 16 == 0;
    const int rc_ws = check_workspace(r, workspace, workspace_bytes, lean && matrix);
    if (rc_ws != VLUT_OK) return rc_ws;
    if (matrix) return launch_matrix_route(r, packed, w_scale, nullptr, a_q, a_scale, K, y, ldy, acc_or_null, (hipStream_t)stream);
    const Plan5 pl = r.plan5;
    const Derived5 d = derive5(pl, M, K, N);
    Lookup5Params p;
    std::memset(&p, 0, sizeof(p));
    p.packed = packed; p.a_q = a_q; p.a_scale = a_scale; p.y = y; p.acc = acc_or_null; p.ws = (int32_t*)workspace;
    p.w_scale = w_scale;
    p.M = (int)M; p.K = (int)K; p.N = (int)N; p.G = d.G; p.KCn = d.KCn; p.RGtotal = d.RGtotal; p.ldy = (int)ldy;
    p.S = pl.S; p.tiles_m = d.tiles_m; p.tiles_n = d.tiles_n; p.RGW = d.RGW;
    p.dstages_total = d.dstages_total; p.dstages_per_split = d.dstages_per_split;
    p.total_tiles = d.total; p.per_xcd = d.per_xcd;
    p.Ka = (int)K;
    hipStream_t s = (hipStream_t)stream;
    int grid = d.per_xcd * 8;
    int rc = d.need32 ? launch_lookup5_r<true>(pl.R, p, grid, s) : launch_lookup5_r<false>(pl.R, p, grid, s);
    if (rc != VLUT_OK) return rc;
    if (pl.S > 1)
        return launch_splitk_reduce((const int32_t*)workspace, pl.S, M, N, w_scale, nullptr, a_scale, y, ldy, acc_or_null, s);
    return VLUT_OK;
}

int vlut_mpgemm_g5(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K,
                   int64_t N, float* y, int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes,
                   void* stream) {
    return mpgemm_g5_impl(packed, w_scale, a_q, a_scale, M, K, N, y, ldy, acc_or_null, workspace, workspace_bytes, stream, false);
}

int vlut_mpgemm_g5_lean(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K, int64_t N, float* y,
                        int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    return mpgemm_g5_impl(packed, w_scale, a_q, a_scale, M, K, N, y, ldy, acc_or_null, workspace, workspace_bytes, stream, true);
}

// ---- mixed 1.60-bit / 2-bit packing (Sec. 3.3 "Flexible sub-2-bit weight packing")
int64_t vlut_mixed_k5(int64_t K) {
    if (K < 4 || (K % 4) != 0) return -1;
    return (K / 20) * 20;
}

size_t vlut_packed_weight_bytes_mixed(int64_t M, int64_t K) {
    if (!shape_ok(M, K, 1)) return 0;
    const int64_t K5 = vlut_mixed_k5(K), K4 = K - K5;
    return (K5 > 0 ? vlut_packed_weight_bytes_g5(M, K5) : 0) + (K4 > 0 ? vlut_packed_weight_bytes(M, K4) : 0);
}

int vlut_pack_weights_mixed(const int8_t* w_ternary, int64_t M, int64_t K, uint8_t* packed, size_t packed_bytes,
                            void* stream) {
    if (!shape_ok(M, K, 1)) return VLUT_ERR_SHAPE;
    if (!w_ternary || !packed) return VLUT_ERR_NULL;
    if (packed_bytes < vlut_packed_weight_bytes_mixed(M, K)) return VLUT_ERR_SMALL_BUFFER;
    return pack_parts(w_ternary, M, K, vlut_mixed_k5(K), packed, stream);
}


size_t vlut_workspace_bytes_mixed(int64_t M, int64_t K, int64_t N) {
    return shape_ok(M, K, N) ? find_route(VLUT_FORM_MIXED, M, K, N).demanded : 0;
}

size_t vlut_workspace_used_mixed(int64_t M, int64_t K, int64_t N) {
    return shape_ok(M, K, N) ? find_route(VLUT_FORM_MIXED, M, K, N).used() : 0;
}

static int mpgemm_mixed_impl(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K, int64_t N, float* y,
                             int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream, bool lean) {
    int rc = check_mpgemm_args(packed, a_q, a_scale, M, K, N, y, ldy, acc_or_null);
    if (rc != VLUT_OK) return rc;
    if (((uintptr_t)a_q) % 16 != 0) return VLUT_ERR_UNSUPPORTED;
    const int64_t K5 = vlut_mixed_k5(K), K4 = K - K5;
    const Route& r = find_route(VLUT_FORM_MIXED, M, K, N);
    if (r.status != VLUT_OK) return r.status;
    const bool matrix = r.kernel != kRouteTables && (uintptr_t)packed % 16 == 0;
    rc = check_workspace(r, workspace, workspace_bytes, lean && matrix);
    if (rc != VLUT_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (matrix) return launch_matrix_route(r, packed, w_scale, nullptr, a_q, a_scale, K5, y, ldy, acc_or_null, s);
    const Plan5 pl5 = r.plan5;
    const Plan pl4 = r.plan;
    if (K5 > 0) {
        const Derived5 d = derive5(pl5, M, K5, N);
        Lookup5Params p;
        std::memset(&p, 0, sizeof(p));
        p.packed = packed; p.a_q = a_q; p.a_scale = a_scale; p.ws = (int32_t*)workspace; p.w_scale = w_scale;
        p.M = (int)M; p.K = (int)K5; p.N = (int)N; p.G = d.G; p.KCn = d.KCn; p.RGtotal = d.RGtotal; p.ldy = (int)ldy;
        p.S = pl5.S; p.tiles_m = d.tiles_m; p.tiles_n = d.tiles_n; p.RGW = d.RGW;
        p.dstages_total = d.dstages_total; p.dstages_per_split = d.dstages_per_split;
        p.total_tiles = d.total; p.per_xcd = d.per_xcd;
        p.Ka = (int)K; p.partial = 1;
        const int grid = d.per_xcd * 8;
        rc = d.need32 ? launch_lookup5_r<true>(pl5.R, p, grid, s) : launch_lookup5_r<false>(pl5.R, p, grid, s);
        if (rc != VLUT_OK) return rc;
    }
    if (K4 > 0) {
        const Derived d = derive(pl4, M, K4, N);
        LookupParams p;
        std::memset(&p, 0, sizeof(p));
        p.packed = packed + (K5 > 0 ? vlut_packed_weight_bytes_g5(M, K5) : 0);
        p.a_q = a_q + (size_t)K5 * 8;                      // activation rows K5 .. K-1 of every token chunk
        p.a_scale = a_scale; p.ws = (int32_t*)workspace; p.w_scale = w_scale;
        p.M = (int)M; p.K = (int)K4; p.N = (int)N; p.G = d.G; p.KCn = d.KCn; p.RGtotal = d.RGtotal; p.ldy = (int)ldy;
        p.Jlog = pl4.Jlog; p.S = pl4.S; p.tiles_m = d.tiles_m; p.tiles_n = d.tiles_n; p.RGW = d.RGW;
        p.stages_total = d.stages_total; p.stages_per_split = d.stages_per_split;
        p.total_tiles = d.total; p.per_xcd = d.per_xcd;
        p.Ka = (int)K; p.partial = 1; p.slot0 = pl5.S;
        rc = d.need32 ? launch_lookup_r<true>(pl4.R, pl4.BW, kFast, p, s) : launch_lookup_r<false>(pl4.R, pl4.BW, kFast, p, s);
        if (rc != VLUT_OK) return rc;
    }
    return launch_splitk_reduce((const int32_t*)workspace, pl5.S + pl4.S, M, N, w_scale, nullptr, a_scale, y, ldy,
                                acc_or_null, s);
}

int vlut_mpgemm_mixed(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K,
                      int64_t N, float* y, int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes,
                      void* stream) {
    return mpgemm_mixed_impl(packed, w_scale, a_q, a_scale, M, K, N, y, ldy, acc_or_null, workspace, workspace_bytes, stream, false);
}

int vlut_mpgemm_mixed_lean(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale, int64_t M, int64_t K, int64_t N, float* y,
                           int64_t ldy, int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    return mpgemm_mixed_impl(packed, w_scale, a_q, a_scale, M, K, N, y, ldy, acc_or_null, workspace, workspace_bytes, stream, true);
}

static int codes_kernel(int64_t M, int64_t K, int64_t N) {
    const Route& r = find_route(VLUT_FORM_CODES, M, K, N);
    if (r.narrow) return VLUT_KERNEL_FEW_TOKENS;
    if (r.status != VLUT_OK) return r.status;
    return r.kernel == kRouteTables ? VLUT_KERNEL_LOOKUP : VLUT_KERNEL_MATRIX;
}

// (the queries answer from the routes that the calls take)
int vlut_query_kernel(int form, int64_t M, int64_t K, int64_t N) {
    if (form != VLUT_FORM_CODES && form != VLUT_FORM_F32 && form != VLUT_FORM_MIXED && form != VLUT_FORM_G5) return VLUT_ERR_UNSUPPORTED;
    if (form == VLUT_FORM_G5 ? !shape5_ok(M, K, N) : !shape_ok(M, K, N)) return VLUT_ERR_SHAPE;
    if (form == VLUT_FORM_CODES) return codes_kernel(M, K, N);
    if (form == VLUT_FORM_F32) {
        const F32Layout L = f32_layout(M, K, N);
        if (L.decode) return VLUT_KERNEL_MATRIX_FEW_TOKENS;
        if (L.kind == kF32Narrow) return VLUT_KERNEL_FEW_TOKENS;
        return L.kind == kF32Fused ? VLUT_KERNEL_LOOKUP : codes_kernel(M, K, N);
    }
    const Route& r = find_route(form, M, K, N);
    if (r.status != VLUT_OK) return r.status;
    return r.kernel == kRouteTables ? VLUT_KERNEL_LOOKUP : VLUT_KERNEL_MATRIX;
}

int vlut_query_matrix_plan(int form, int64_t M, int64_t K, int64_t N, int* out4) {
    if (!out4) return VLUT_ERR_NULL;
    const int kernel = vlut_query_kernel(form, M, K, N);
    if (kernel < 0) return kernel;
    if (kernel == VLUT_KERNEL_LOOKUP) return VLUT_ERR_UNSUPPORTED;
    if (kernel == VLUT_KERNEL_MATRIX_FEW_TOKENS) {
        const int mt = decode_row_tiles(M);
        out4[0] = 16 * mt; out4[1] = decode_token_slots(N); out4[2] = kDecodeWaves / mt;
        out4[3] = (int)((M + out4[0] - 1) / out4[0]);
        return VLUT_OK;
    }
    if (form == VLUT_FORM_F32 && f32_layout(M, K, N).kind != kF32TwoLaunches) return VLUT_ERR_UNSUPPORTED;
    const Route& r = find_route(form == VLUT_FORM_F32 ? VLUT_FORM_CODES : form, M, K, N);
    if (r.kernel == kRouteTables) return VLUT_ERR_UNSUPPORTED;       // few tokens: the table kernel's
    if (r.kernel == kRouteCodes) {
        out4[0] = 16 * r.codes.mt; out4[1] = 8 * r.codes.ch; out4[2] = kDecodeWaves / r.codes.mt;
    } else {
        const GemmTile t = gemm_tile(r.tile);
        out4[0] = t.rows(); out4[1] = t.tokens(); out4[2] = t.wk;
    }
    const int64_t tiles = ((M + out4[0] - 1) / out4[0]) * ((N + out4[1] - 1) / out4[1]);
    out4[3] = (int)std::min<int64_t>(tiles, INT32_MAX);
    return VLUT_OK;
}

size_t vlut_mfma_workspace_bytes(int64_t M, int64_t K, int64_t N) {
    if (!shape_ok(M, K, N)) return 0;
    const MfmaPlan mp = mfma_plan(M, K, N);
    return mp.S > 1 ? (size_t)mp.S * (size_t)M * (size_t)N * sizeof(int32_t) : 0;
}

int vlut_mpgemm_mfma(const uint8_t* packed, float w_scale, const int8_t* a_q, const float* a_scale,
                     const int16_t* lut_or_null, int64_t M, int64_t K, int64_t N, float* y, int64_t ldy,
                     int32_t* acc_or_null, void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_mpgemm_args(packed, a_q, a_scale, M, K, N, y, ldy, acc_or_null);
    if (rc != VLUT_OK) return rc;
    if (lut_or_null) return VLUT_ERR_UNSUPPORTED;
    if (((uintptr_t)a_q) % 16 != 0 || ((uintptr_t)packed) % 16 != 0) return VLUT_ERR_UNSUPPORTED;
    const MfmaPlan mp = mfma_plan(M, K, N);
    const size_t need = mp.S > 1 ? (size_t)mp.S * (size_t)M * (size_t)N * sizeof(int32_t) : 0;
    if (need > 0) {
        if (!workspace) return VLUT_ERR_NULL;
        if (workspace_bytes < need) return VLUT_ERR_SMALL_BUFFER;
        if (((uintptr_t)workspace) % 16 != 0) return VLUT_ERR_UNSUPPORTED;
    }
    hipStream_t s = (hipStream_t)stream;
    MfmaParams p;
    std::memset(&p, 0, sizeof(p));
    p.packed = packed; p.a_q = a_q; p.a_scale = a_scale; p.y = y; p.acc = acc_or_null; p.ws = (int32_t*)workspace;
    p.w_scale = w_scale; p.M = (int)M; p.K = (int)K; p.N = (int)N;
    p.KCn = (int)((K / 4 + 15) / 16); p.RGtotal = (int)((M + 3) / 4); p.ldy = (int)ldy; p.chunks = (int)((N + 7) / 8);
    p.S = mp.S; p.steps_per_split = mp.steps_per_split; p.tiles_m = mp.tiles_m; p.tiles_n = mp.tiles_n;
    if (mp.S > 1) p.out_vec = (M % 4 == 0) ? 1 : 0;
    else p.out_vec = (!y || (((uintptr_t)y % 16 == 0) && (ldy % 4 == 0))) ? 1 : 0;
    const dim3 grid((unsigned)mp.grid);
    switch (mp.BN) {
    case 128: hipLaunchKernelGGL(mfma_kernel<128>, grid, dim3(256), 0, s, p); break;
    case 64: hipLaunchKernelGGL(mfma_kernel<64>, grid, dim3(256), 0, s, p); break;
    case 32: hipLaunchKernelGGL(mfma_kernel<32>, grid, dim3(256), 0, s, p); break;
    default: hipLaunchKernelGGL(mfma_kernel<16>, grid, dim3(256), 0, s, p); break;
    }
    if (hipGetLastError() != hipSuccess) return VLUT_ERR_DEVICE;
    if (mp.S > 1)
        return launch_splitk_reduce((const int32_t*)workspace, mp.S, M, N, w_scale, nullptr, a_scale, y, ldy, acc_or_null, s);
    return VLUT_OK;
}

}  // extern "C"
