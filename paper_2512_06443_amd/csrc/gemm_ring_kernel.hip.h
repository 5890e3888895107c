// The tiled product from four weights per byte with both operands loaded straight to LDS, two macro steps ahead.
// Part of the single translation unit vlut.hip (included there, in this order).
#pragma once

namespace {

// ---------------------------------------------------------------------------------------------
// Workgroup, tile, planes, transposing reads and the end are those of gemm_kernel; what differs is how the operands travel.  There a load
// goes through registers into LDS one macro step before its use, and with two waves per SIMD the K loop waits: 128 x 128 (two K groups)
// takes 1762 cycles per pass for 1024 of the matrix cores, without loads or without LDS traffic 1400 to 1600.  Here
//   - three slots of LDS per K group hold a macro step each; a wave loads its share of a step (its chunks of activations, its own rows of
//     weights) into the slot that the step three back has left, so that two steps are on their way or there;
//   - the matrix instructions' activation operands are read AR operands ahead, across the barrier that ends a step;
//   - raw weights (private to the wave) are read once per step, 16 bytes per lane, into the register set that is not in use.
// The loop is unrolled over slots and register sets, so that every LDS address is a register and a constant (addresses worked out per
// step cost 9 %: 1470 -> 1610 cycles).  Cycles per pass, gemm_kernel /
// this one: 256 x 128 2800 / 2450 to 2490 (one K group 1950 / 1480 to 1500), 128 x 128 1762 / 1400 to 1430, 128 x 64 in four K groups 2240 / 1760 to 1850.  us
// per launch back to back on one card, gemm_kernel storing dword by dword / this one: 14336 x 4096 x 512 32.4 / 28.7, 13824 x 2560 x 1024 42.0 / 34.1,
// 2560 x 6912 x 1024 27.2 / 23.2, 2560 x 2560 x 1024 14.1 / 12.5, 4096 x 14336 x 512 36.5 / 31.4 (other cards are up to a tenth slower: the first
// 29 to 32).  What is left of a pass beyond the matrix cores is LDS reads and the power limit (1.8 to 2.1
// GHz where every unit works).  v_mfma_i32_16x16x64_i8 draws less (14.5 ns for the work of 16.5) but takes twice the
// issue slots beside 3.3 unpacking instructions: 2 to 3 % faster than this loop at 256 x 128, 7 % slower at 128 x 128: not taken.
//
// The loads are single instructions written out (no result register; the LDS address in M0): the compiler, when it issues them itself,
// waits for all of them before every LDS read that follows.  Waits are counted by hand: each stage is exactly kLoads of them per wave, also past the
// end of K, where the last step is loaded again, so that vmcnt(kLoads) before the barrier of step t stands for "the loads of step t + 1 are
// done": behind them only those of step t + 2 have been issued.  Nothing else in the loop touches memory.  The scales are loaded ahead
// of the first stage and stored to LDS behind the loop, when every load has been waited for.
//
// What keeps the reads inside the tensors: a stage's descriptors start at its step and end with the tensor (BufferSpan), so that rows and chunks
// past the last one, and the rest of the last row group's and the last chunk's step, are zeros.  Inside the tensor a step that K ends in
// reads on into the next row group or chunk, and a K group whose share of the last pass lies past K multiplies the last step once more:
// both meet weights that keep has set to zero.
// ---------------------------------------------------------------------------------------------
#if defined(__HIP_DEVICE_COMPILE__)
// 16 bytes per lane from offset `at` on to LDS, lane after lane from `to` on
__device__ __forceinline__ void load_to_lds(buffer_rsrc r, unsigned at, unsigned to) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(to), "v"(at), "s"(r) : "memory", "m0");
}
template <int N>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
#else
inline __device__ void load_to_lds(buffer_rsrc, unsigned, unsigned) {}
template <int N>
inline __device__ void wait_loads() {}
#endif

constexpr int kRingSlots = 3;
template <int RT, int CT, int WM>
constexpr int ring_step_bytes() { return 2 * CT * GemmShape<4>::kP2 + RT * WM * 1024; }      // of a K group: activations, then the waves' weights
template <int RT, int CT, int WM, int WK>
constexpr int ring_lds_bytes() {
    const int steps = kRingSlots * WK * ring_step_bytes<RT, CT, WM>(), sums = WM * RT * CT * 4 * (WK - 1) * 1024;
    return (steps > sums ? steps : sums) + 32 * (CT + RT * WM) * 4;
}

template <int RT, int CT, int WM, int WK>
__global__ void __launch_bounds__(64 * WM * WK, 2) gemm_ring_kernel(const GemmParams p) {
    using S = GemmShape<4>;
    constexpr int BN = 32 * CT, BM = 32 * RT * WM, kThreads_ = 64 * WM * WK;
    constexpr int kChunk = S::kUnits * 16;                 // bytes of a chunk of eight tokens per step
    constexpr int kActLoads = 4 * CT / WM;                 // chunks per wave, one load each
    constexpr int kLoads = kActLoads + RT;
    constexpr int kStep = ring_step_bytes<RT, CT, WM>();
    constexpr int kScales = ring_lds_bytes<RT, CT, WM, WK>() - (BN + BM) * 4;
    constexpr int NG = 4 * CT;                             // activation operands of a step: q = 0..3, CT each
    constexpr int AR = CT == 4 ? 8 : 4;                    // of them in registers ahead of use
    constexpr int kBarrier = NG - AR;                      // operand ahead of which the step's barrier stands
    constexpr int kReady = kBarrier - (CT > 2 ? 2 : 1);    // and the wait for the next step's loads
    static_assert((4 * CT) % WM == 0 && NG % AR == 0 && kReady >= 0 && kReady < 3 * CT && 32 * CT + 32 * RT * WM <= 2 * kThreads_, "");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wk = wave / WM;
    const int i = lane & 31, kb = lane >> 5;
    const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);      // as in gemm_kernel
    if (tile >= p.tiles) return;
    const int mt = tile / p.tiles_n, nt = tile - mt * p.tiles_n;
    const int passes = (p.macros + WK - 1) / WK;

    // ---- scales: one or two values per thread
    auto load_scale = [&](int j) { return j < BN ? p.a_scale[min(nt * BN + j, p.N - 1)] : (p.w_rows ? p.w_rows[min(mt * BM + j - BN, p.M - 1)] : p.w_scale); };
    const float scale0 = load_scale(min(tid, BN + BM - 1)), scale1 = load_scale(min(tid + kThreads_, BN + BM - 1));

    // ---- loads.  Descriptors reach from the tile's first byte of a step to the end of the tensor; offsets inside the tile are constant.
    const int rg0 = mt * (BM / 4), chunk0 = nt * (BN / 8);
    const uint8_t* wbase = p.packed + (size_t)rg0 * p.KCn * 64;
    const int8_t* abase = p.a_q + (size_t)chunk0 * p.Ka * 8;
    const int64_t wleft = (int64_t)(p.RGtotal - rg0) * p.KCn * 64, aleft = (int64_t)(p.chunks - chunk0) * p.Ka * 8;
    // weights: load d brings row groups 8 d .. 8 d + 7 of the wave, both tile columns.  Four lanes take the 64 bytes of a group and column, their
    // rows turned by `turn`, so that the 16 lanes that read 16 row groups' same row (or 8 groups' two rows) find them in 16 different slices.
    auto turn = [](int rgl, int d) { return ((rgl >> 2) & 1) | (d << 1); };
    unsigned wat[RT], aat[kActLoads];
#pragma unroll
    for (int d = 0; d < RT; ++d) {
        const int rgl = (lane >> 2) & 7, col = lane >> 5;
        wat[d] = (unsigned)(((wm * RT + d) * 8 + rgl) * p.KCn + col) * 64u + (unsigned)(((lane & 3) ^ turn(rgl, d)) * 16);
    }
#pragma unroll
    for (int u = 0; u < kActLoads; ++u) aat[u] = (unsigned)(u * WM + wm) * (unsigned)p.Ka * 8u + (unsigned)(lane * 16);
    const unsigned group = (unsigned)(wk * kRingSlots * kStep);
    const unsigned weights = group + 2 * CT * S::kP2 + (unsigned)(wm * RT * 1024);
    const BufferSpan act_from(abase, aleft), weights_from(wbase, wleft);
    struct Step { buffer_rsrc act, weights; };
    auto step_at = [&](int t) {                            // pass t of this K group; past K the last step again (unread or, in the last pass, against zeros)
        const unsigned macro = (unsigned)min(wk + t * WK, p.macros - 1);
        return Step{act_from.at(macro * (unsigned)kChunk), weights_from.at(macro * 128u)};
    };
    auto load = [&](const Step& from, int slot, int op) {
        if (op < kActLoads) {
            const int c = op * WM + wm;
            load_to_lds(from.act, aat[op], group + (unsigned)(slot * kStep + (c >> 1) * S::kP2 + (c & 1) * S::kP1));
        } else {
            load_to_lds(from.weights, wat[op - kActLoads], weights + (unsigned)(slot * kStep + (op - kActLoads) * 1024));
        }
    };
#pragma unroll
    for (int s = 0; s < kRingSlots; ++s) {
        const Step from = step_at(s);
#pragma unroll
        for (int op = 0; op < kLoads; ++op) load(from, s, op);
    }

    // ---- operands
    i32x16 acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = i32x16{};
    i32x4 a[AR], b[2][RT], w[2][RT];                       // w: raw weights of this step and the next
    unsigned keep;                                         // 0 in lanes whose tile column lies past the end of K
    auto keep_of = [&](int t) { return 2 * (wk + t * WK) + kb < p.KCn ? 0xffffffffu : 0u; };
    const int r8 = (lane & 15) >> 1;
    const unsigned rd = group + (unsigned)(((lane >> 4) & 1) * S::kP2 + (lane & 1) * S::kP1 + kb * S::kCol * 8 + (r8 & 3) * 32 + (r8 >> 2) * 8);
    auto read_act = [&](unsigned slot, int q, int ct) {
        const unsigned at = rd + slot * kStep + (unsigned)(ct * 2 * S::kP2 + q * 128);
        const i32x2 lo = lds_read_tr8(at), hi = lds_read_tr8(at + 16);
        return i32x4{lo.x, lo.y, hi.x, hi.y};
    };
    unsigned rdw[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int row = gemm_row<RT, kStoreTogether>(i, rt), rg = row >> 2, d = rg >> 3, rgl = rg & 7;
        rdw[rt] = weights + (unsigned)(d * 1024 + (kb * 8 + rgl) * 64 + (((row & 3) ^ turn(rgl, d)) * 16));
    }
    auto read_weights = [&](int set, unsigned slot) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) w[set][rt] = *(const lds_i32x4*)(rdw[rt] + slot * kStep);
    };
    constexpr int kOps = Unpack<4>::kOps, NS = RT * kOps;
    const UnpackConst uc(4);
    Unpack<4> un;
    auto unpack_step = [&](int set, int q, int st) {       // of the weight operands of matrix instructions q
        const int rt = st / kOps, j = st % kOps;
        unsigned none;
        if (j == 0) un.w = ((unsigned)w[set][rt][q] & keep) | (kZeroIdx4 & ~keep);
        un.op(j, uc, b[q & 1][rt], none);
    };
    wait_loads<(kRingSlots - 1) * kLoads>();
    keep = keep_of(0);
    read_weights(0, 0);
#pragma unroll
    for (int st = 0; st < NS; ++st) unpack_step(0, 0, st);
    wg_barrier_lds();
#pragma unroll
    for (int s = 0; s < AR; ++s) a[s] = read_act(0, s / CT, s % CT);

    // ---- a macro step: behind every matrix instruction a few unpacking steps of the next operands, behind the last one of an activation
    //      operand the read of the one AR further on
    auto macro_step = [&](int set, int slot, int t) {
        const int next_slot = slot + 1 == kRingSlots ? 0 : slot + 1;
        const Step from = step_at(t + kRingSlots);
#pragma unroll
        for (int s = 0; s < NG; ++s) {
            const int q = s / CT, ct = s % CT;
            if (s == kReady) wait_loads<kLoads>();
            if (s == kBarrier) wg_barrier_lds();           // (the last operands of this slot are in registers: lgkmcnt(0))
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int g = ct * RT + rt;
                __builtin_amdgcn_sched_barrier(0);
                acc[rt][ct] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[s % AR], b[q & 1][rt], acc[rt][ct], 0, 0, 0);
                if (rt == RT - 1) {
                    const int n = s + AR;
                    a[s % AR] = n < NG ? read_act(slot, n / CT, n % CT) : read_act(next_slot, (n - NG) / CT, (n - NG) % CT);
                }
#pragma unroll
                for (int st = g * NS / (CT * RT); st < (g + 1) * NS / (CT * RT); ++st) unpack_step(q == 3 ? set ^ 1 : set, q == 3 ? 0 : q + 1, st);
            }
            if (s == kReady) read_weights(set ^ 1, next_slot);
            if (s == 3 * CT - 1) keep = keep_of(t + 1);
            if (s >= kBarrier) {
#pragma unroll
                for (int op = (s - kBarrier) * kLoads / AR; op < (s - kBarrier + 1) * kLoads / AR; ++op) load(from, slot, op);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < passes; t += 6) {                  // two register sets, three slots
        macro_step(0, 0, t);
        if (t + 1 < passes) macro_step(1, 1, t + 1);
        if (t + 2 < passes) macro_step(0, 2, t + 2);
        if (t + 3 < passes) macro_step(1, 0, t + 3);
        if (t + 4 < passes) macro_step(0, 1, t + 4);
        if (t + 5 < passes) macro_step(1, 2, t + 5);
    }
    wait_loads<0>();
    *(lds_i32*)(unsigned)(kScales + min(tid, BN + BM - 1) * 4) = __builtin_bit_cast(int, scale0);
    if (tid + kThreads_ < BN + BM) *(lds_i32*)(unsigned)(kScales + (tid + kThreads_) * 4) = __builtin_bit_cast(int, scale1);
    wg_barrier_lds();
    gemm_store<RT, CT, WM, WK, kStoreTogether>(p, acc, lane, wm, wk, mt, nt, kScales);
}

// The tiles that this kernel serves: those that are 64 rows per wave, 128 x 128, and 128 x 64 in two K groups.
constexpr bool gemm_ring_built(int gw, int rt, int ct, int wm, int wk) { return gw == 4 && (rt == 2 || (ct > 1 && wm == 4 && wk == 2)); }

}  // namespace
