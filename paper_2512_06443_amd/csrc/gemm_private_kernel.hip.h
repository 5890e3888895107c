// The tiled product from four weights per byte where every wave has a tile's rows and tokens to itself and its own part of K.
// Part of the single translation unit vlut.hip (included there, in this order).
#pragma once

namespace {

// ---------------------------------------------------------------------------------------------
// Workgroup = WK waves of one tile of 32 * RT rows x 32 * CT tokens, one wave per SIMD with all of its registers; wave wk takes macro steps wk, wk + WK,
// .. of K for the whole tile and the INT32 sums meet in LDS at the end.  Operands travel as in gemm_ring_kernel, but the slots of LDS belong to a wave:
// the K loop has no barrier and every packed byte of a tile is unpacked by one wave.  The registers allow tiles of any number of row tiles up
// to six, and that is what it is for: 160 rows x 64 tokens make 256 tiles of 2560 x 1024, where 128 x 128 make 160.
// Rates: 1650 to 1750 cycles per pass at RT = 4 (gemm_ring_kernel with two waves per SIMD, 128 x 64 in four K groups: 1760 to 1850), 1975 to 2100 at 5,
// for 1024 and 1280 of the matrix cores; unpacking is 6.5 instructions per matrix instruction, and two unpackings side by side are no faster.
// us, graph replays, 128 x 128 or 128 x 64 / this one: 2560 x 6912 x 1024 25.2 / 22.2 (RT = 5), 2560 x 2560 x 1024 12.9 / 12.1 (5), 4096 x 14336 x 512 32.1 / 30.7
// (4); where the others fill the chip as well they are the better ones: 14336 x 4096 x 512 29.7 / 39.2 (5).  In a stream behind the quantiser the gain is
// smaller: a layer's four linears at 1024 tokens 128.4 -> 125.3, 4096 x 14336 x 512 43.2 -> 42.9.
// ---------------------------------------------------------------------------------------------
template <int RT, int CT, int WK>
struct PrivateShape {
    static constexpr int kAct = 2 * CT * GemmShape<4>::kP2, kWeights = RT * 1024;      // bytes of a macro step
    static constexpr int kActSlots = 3, kWeightSlots = 2;
    static constexpr int kGroup = kActSlots * kAct + kWeightSlots * kWeights;           // LDS of a wave
    static constexpr int kSums = RT * CT * 4 * (WK - 1) * 1024;
    static constexpr int kScales = WK * kGroup > kSums ? WK * kGroup : kSums;
    static constexpr int kLds = kScales + 32 * (CT + RT) * 4;
};

template <int RT, int CT, int WK>
__global__ void __launch_bounds__(64 * WK, 1) gemm_private_kernel(const GemmParams p) {
    using S = GemmShape<4>;
    using P = PrivateShape<RT, CT, WK>;
    constexpr int BN = 32 * CT, BM = 32 * RT, kThreads_ = 64 * WK;
    constexpr int kChunk = S::kUnits * 16;                 // bytes of a chunk of eight tokens per step
    constexpr int kActLoads = 4 * CT;                      // chunks, one load each
    constexpr int kLoads = kActLoads + RT;
    constexpr int NG = 4 * CT;                             // activation operands of a step: q = 0..3, CT each
    constexpr int AR = 2;                                  // of them in registers ahead of use
    constexpr int kReady = NG - AR - 1;                    // operand behind which the next step's loads are waited for
    constexpr int kIssue = 3;                              // the loads of the step after that stand behind the first operands
    static_assert(kReady < 3 * CT && kIssue <= kReady && BN + BM <= 2 * kThreads_, "");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wk = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 31, kb = lane >> 5;
    const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);      // as in gemm_kernel
    if (tile >= p.tiles) return;
    const int mt = tile / p.tiles_n, nt = tile - mt * p.tiles_n;
    const int passes = (p.macros + WK - 1) / WK;

    // ---- scales: one or two values per thread
    auto load_scale = [&](int j) { return j < BN ? p.a_scale[min(nt * BN + j, p.N - 1)] : (p.w_rows ? p.w_rows[min(mt * BM + j - BN, p.M - 1)] : p.w_scale); };
    const float scale0 = load_scale(min(tid, BN + BM - 1)), scale1 = load_scale(min(tid + kThreads_, BN + BM - 1));

    // ---- loads, as in gemm_ring_kernel; weights lie in LDS as they are read: 32 rows of a tile column, 16 bytes each, then the other column
    const int rg0 = mt * (BM / 4), chunk0 = nt * (BN / 8);
    const uint8_t* wbase = p.packed + (size_t)rg0 * p.KCn * 64;
    const int8_t* abase = p.a_q + (size_t)chunk0 * p.Ka * 8;
    const int64_t wleft = (int64_t)(p.RGtotal - rg0) * p.KCn * 64, aleft = (int64_t)(p.chunks - chunk0) * p.Ka * 8;
    unsigned wat[RT], aat[kActLoads];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) wat[rt] = (unsigned)((rt * 8 + (i >> 2)) * p.KCn + kb) * 64u + (unsigned)((i & 3) * 16);
#pragma unroll
    for (int c = 0; c < kActLoads; ++c) aat[c] = (unsigned)c * (unsigned)p.Ka * 8u + (unsigned)(lane * 16);
    const unsigned group = (unsigned)(wk * P::kGroup), weights = group + P::kActSlots * P::kAct;
    const BufferSpan act_from(abase, aleft), weights_from(wbase, wleft);
    struct Step { buffer_rsrc act, weights; };
    auto step_at = [&](int t) {                            // pass t of this wave; past K the last step again (unread or, in the last pass, against zeros)
        const unsigned macro = (unsigned)min(wk + t * WK, p.macros - 1);
        return Step{act_from.at(macro * (unsigned)kChunk), weights_from.at(macro * 128u)};
    };
    auto load = [&](const Step& from, int slot, int set, int op) {      // weights first: they come from further away
        if (op < RT) load_to_lds(from.weights, wat[op], weights + (unsigned)(set * P::kWeights + op * 1024));
        else {
            const int c = op - RT;
            load_to_lds(from.act, aat[c], group + (unsigned)(slot * P::kAct + (c >> 1) * S::kP2 + (c & 1) * S::kP1));
        }
    };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const Step from = step_at(s);
#pragma unroll
        for (int op = 0; op < kLoads; ++op) load(from, s, s, op);
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
        const unsigned at = rd + slot * P::kAct + (unsigned)(ct * 2 * S::kP2 + q * 128);
        const i32x2 lo = lds_read_tr8(at), hi = lds_read_tr8(at + 16);
        return i32x4{lo.x, lo.y, hi.x, hi.y};
    };
    const unsigned rdw = weights + (unsigned)(lane * 16);
    auto read_weights = [&](int set) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) w[set][rt] = *(const lds_i32x4*)(rdw + (unsigned)(set * P::kWeights + rt * 1024));
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
    wait_loads<kLoads>();
    keep = keep_of(0);
    read_weights(0);
#pragma unroll
    for (int st = 0; st < NS; ++st) unpack_step(0, 0, st);
#pragma unroll
    for (int s = 0; s < AR; ++s) a[s] = read_act(0, s / CT, s % CT);

    // ---- a macro step: behind every matrix instruction a few unpacking steps of the next operands, behind the last one of an activation
    //      operand the read of the one AR further on.  The slots that the loads of step t + 2 fill were last read by step t - 1 (activations)
    //      and ahead of step t (weights), whose matrix instructions and unpacking have waited for these reads.
    auto macro_step = [&](int set, int slot, int t) {
        const int next_slot = slot + 1 == P::kActSlots ? 0 : slot + 1, free_slot = slot == 0 ? P::kActSlots - 1 : slot - 1;
        const Step from = step_at(t + 2);
#pragma unroll
        for (int s = 0; s < NG; ++s) {
            const int q = s / CT, ct = s % CT;
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
                if (s < kIssue) {
#pragma unroll
                    for (int op = (s * RT + rt) * kLoads / (kIssue * RT); op < (s * RT + rt + 1) * kLoads / (kIssue * RT); ++op) load(from, free_slot, set, op);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (s == kReady) {
                wait_loads<kLoads>();
                read_weights(set ^ 1);
            }
            if (s == 3 * CT - 1) keep = keep_of(t + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int t = 0; t < passes; t += 6) {                  // two sets of weights, three slots of activations
        macro_step(0, 0, t);
        if (t + 1 < passes) macro_step(1, 1, t + 1);
        if (t + 2 < passes) macro_step(0, 2, t + 2);
        if (t + 3 < passes) macro_step(1, 0, t + 3);
        if (t + 4 < passes) macro_step(0, 1, t + 4);
        if (t + 5 < passes) macro_step(1, 2, t + 5);
    }
    wait_loads<0>();                                       // (scales lie behind every slot, the sums of gemm_store where they are)
    *(lds_i32*)(unsigned)(P::kScales + min(tid, BN + BM - 1) * 4) = __builtin_bit_cast(int, scale0);
    if (tid + kThreads_ < BN + BM) *(lds_i32*)(unsigned)(P::kScales + (tid + kThreads_) * 4) = __builtin_bit_cast(int, scale1);
    wg_barrier_lds();
    gemm_store<RT, CT, 1, WK, kStorePairs>(p, acc, lane, 0, wk, mt, nt, P::kScales);
}

// The tiles of kGemmTilesLong that this kernel serves.
constexpr bool gemm_private_built(int gw, int wm, int wk) { return gw == 4 && wm == 1 && wk == 4; }

}  // namespace
