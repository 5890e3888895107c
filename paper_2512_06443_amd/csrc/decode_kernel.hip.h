// A few tokens on the INT8 matrix cores: up to sixteen from fp32 activations in one launch (quantisation, unpacking, product), and
// from INT8 codes.
// Part of the single translation unit vlut.hip (included there, in this order).
#pragma once

namespace {

// ---------------------------------------------------------------------------------------------
// A workgroup (16 waves) owns 16 * MT output rows and all of K for all tokens.  It quantises the tokens itself (every
// workgroup repeats that: N * K floats from L2, while its weights are on their way from HBM), so that a linear is one
// launch and touches no workspace (the call still wants one of vlut_workspace_bytes_f32); the waves then split the row tiles and K, and their INT32 sums meet in LDS.
//
// v_mfma_i32_16x16x64_i8: tokens x rows.  Weights as in gemm_kernel (lane = row and tile column, 16 packed bytes per
// load, planes instead of the natural order of K); a macro step is four tile columns = 256 values of K.  The codes are
// laid out in LDS as the operands: unit (16 values of K) x token slot x 16 bytes, plane order inside, T slots (a power of
// two; lanes of absent tokens read a live slot, their results are not stored).  A wave quantises one macro step of one
// token per pass, its lanes in the order of K; the four lanes of a 16-value unit transpose their bytes by data parallel
// primitives, which is the plane order, and store one dword each.  Slots are rotated by the unit, so that the 16 units of
// a pass lie in distinct banks and the 16 tokens of an operand read do too.
//
// Bound by latency: launch, the rows of x, one trip to HBM for the weights, 13 instructions per four packed bytes.
// ---------------------------------------------------------------------------------------------
struct DecodeParams {
    const uint8_t* packed;
    const float* x;
    const float* w_rows;
    float* y;
    int32_t* acc;
    float* a_scale_out;
    int64_t ldx;
    float w_scale;
    int M, N, K, KCn, RGtotal, ldy, macros;
    const int8_t* a_q;            // decode_codes_kernel: INT8 codes and their scales instead of x
    const float* a_scale;
    const uint8_t* packed4;       // mixed packing: the 2-bit blob of the last K - Kmain < 20 values of K, else null
    int Kmain, KCn4;              // values of K in `packed`
    int chunks, tiles_n, tiles, per_xcd, pitch;
    unsigned magic_n;             // 2^32 / tiles_n rounded up (tiles_n > 1)
};

constexpr int kDecodeWaves = 16;
constexpr int kDecodeKeep = 12;                // float4 of x per lane kept between the two passes; the rest is read twice
constexpr int decode_lds_bytes(int T, int macros) { return macros * 256 * T + kDecodeWaves * 1024 + 128; }

// One lane's packed bytes: row m of the workgroup's rows from m0 on, tile column 4 macro + kb (rows past the last one read zeros, their sums
// are not stored; columns past the last one are clamped and replaced by zeros when they are unpacked).  A workgroup's rows span less than
// 2^31 bytes.
struct DecodeWeights {
    buffer_rsrc from;
    unsigned at, end;
    __device__ __forceinline__ DecodeWeights(const DecodeParams& p, int m0, int m, int kb)
        : from(make_buffer(p.packed + (size_t)(m0 >> 2) * p.KCn * 64, (int64_t)(p.RGtotal - (m0 >> 2)) * p.KCn * 64)) {
        const unsigned row = (unsigned)((m >> 2) * p.KCn) * 64u + (unsigned)((m & 3) * 16);
        at = row + (unsigned)(kb * 64);
        end = row + (unsigned)(p.KCn - 1) * 64u;
    }
    __device__ __forceinline__ i32x4 load(int macro) const { return buffer_load128(from, min(at + (unsigned)macro * 256u, end)); }
};

// Four packed bytes as the four planes of -w; the all-zero pattern where keep is 0.
__device__ __forceinline__ i32x4 unpack_planes4(unsigned w, unsigned keep, const UnpackConst& uc) {
    Unpack<4> un;
    i32x4 b;
    unsigned none;
    un.w = (w & keep) | (kZeroIdx4 & ~keep);
#pragma unroll
    for (int st = 0; st < Unpack<4>::kOps; ++st) un.op(st, uc, b, none);
    return b;
}

// The outputs tid, tid + 1024, .. of the workgroup's 16 * MT rows (from m0) x TOK tokens (from n0).  Their scales are requested ahead of
// the weights: at the end they would cost a trip to memory of their own.
template <int TOK, int MT>
struct DecodeOut {
    static constexpr int kThreads = 64 * kDecodeWaves, kRounds = (16 * MT * TOK + kThreads - 1) / kThreads;
    int first, m0, n0;
    float ws[kRounds], as[kRounds];
    __device__ __forceinline__ DecodeOut(const DecodeParams& p, int tid, int m0_, int n0_) : first(tid), m0(m0_), n0(n0_) {
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int o = tid + kThreads * r, n = n0 + o / (16 * MT), m = m0 + o % (16 * MT);
            ws[r] = p.w_scale;
            as[r] = 0.0f;
            if (n < p.N && m < p.M) {
                if (p.w_rows) ws[r] = p.w_rows[m];
                if (p.a_scale) as[r] = p.a_scale[n];
            }
        }
    }
    // adds the parts of K (sums of -w, 16 tokens x 16 rows per wave), scales, stores; scale(n, as) is the scale of the tile's token n
    template <class Scale>
    __device__ __forceinline__ void store(const DecodeParams& p, unsigned sums, Scale scale) const {
        constexpr int KP = kDecodeWaves / MT;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int o = first + kThreads * r, nl = o / (16 * MT), ml = o % (16 * MT);
            const int n = n0 + nl, m = m0 + ml;
            if (nl >= TOK || n >= p.N) break;
            const unsigned src = sums + (unsigned)((ml >> 4) * 1024 + ((nl >> 2) * 16 + (ml & 15)) * 16 + (nl & 3) * 4);
            int v = 0;
#pragma unroll
            for (int k = 0; k < KP; ++k) v -= *(const lds_i32*)(src + (unsigned)(k * MT * 1024));
            if (m < p.M) {
                if (p.y) p.y[(size_t)n * p.ldy + m] = (float)v * (ws[r] * scale(nl, as[r]));
                if (p.acc) p.acc[(size_t)m * p.N + n] = v;
            }
        }
    }
};

// f(0), f(1), .. for the first `steps` (uniform) of the kDecodeKeep steps.  Nested, so that few steps are few branches, and with something
// in each that the compiler cannot run ahead of its branch: it turned twelve short steps into twelve selections (one token: +0.2 us).
template <int I, class F>
__device__ __forceinline__ void first_steps(int steps, F f) {
    if constexpr (I < kDecodeKeep) {
        if (I < steps) {
#if defined(__HIP_DEVICE_COMPILE__)
            asm volatile("");
#endif
            f(I);
            first_steps<I + 1>(steps, f);
        }
    }
}

template <int T, int MT>
__global__ void __launch_bounds__(64 * kDecodeWaves) decode_kernel(const DecodeParams p) {
    constexpr int KP = kDecodeWaves / MT;      // parts of K
    constexpr int WPT = kDecodeWaves / T;      // waves that quantise one token
    constexpr int kShift = T == 16 ? 0 : (T == 8 ? 1 : (T == 4 ? 2 : (T == 2 ? 3 : 4)));
    constexpr int PF = 4;                      // macro steps of weights in flight
    typedef __attribute__((address_space(3))) float lds_f32;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const unsigned sums = (unsigned)p.macros * (256u * T);
    const unsigned red = sums + kDecodeWaves * 1024;                     // [16] absmax of a wave, then [16] scales of a token

    // ---- request the rows of x first, then the first weights (loads return in order, and x is needed first)
    const int tok = wave / WPT, sub = wave % WPT;
    const bool live = tok < p.N;
    const buffer_rsrc row = make_buffer(p.x + (size_t)(live ? tok : 0) * p.ldx, (int64_t)p.K * 4);
    const unsigned at = (unsigned)(sub * 1024 + lane * 16);              // the wave's macro steps are sub + WPT * it
    const int steps = live ? max(p.macros - sub + WPT - 1, 0) / WPT : 0;
    auto load4 = [&](int it) { return __builtin_bit_cast(f32x4, buffer_load128(row, at + (unsigned)it * (WPT * 1024u))); };
    f32x4 xv[kDecodeKeep];
    first_steps<0>(steps, [&](int it) { xv[it] = load4(it); });
    const int rt = wave % MT, part = wave / MT;
    const int i = lane & 15, kb = lane >> 4;
    const DecodeWeights weights(p, blockIdx.x * 16 * MT, rt * 16 + i, kb);
    auto load_w = [&](int macro) { return weights.load(macro); };
    const DecodeOut<T, MT> out(p, tid, blockIdx.x * 16 * MT, 0);
    i32x4 w[PF];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PF; ++j) w[j] = load_w(part + KP * j);
    __builtin_amdgcn_sched_barrier(0);

    // ---- quantise: absmax over the row, then codes (the decisions of quant_codes4, IEEE divisions).  Maxima that let a NaN through take two
    //      values per instruction; a wave that meets one reads its values again.  18 instructions per four values instead of 32: with
    //      16 tokens a wave quantises a whole row and the vector units are what it waits for.  The four linears of a 2560-wide layer, us in a
    //      stream: 16 tokens 29.0 -> 26.3; one token, where it is the branches around loads that go, 17.0 -> 16.3.
    float amax = 0.0f;
    bool odd = false;                                                    // (uniform)
    auto rest = [&](int first, auto take) {                              // values that no register holds, four steps at a time
        for (int it = first; it < steps; it += 4) {
            f32x4 tv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) tv[c] = load4(it + c);           // (zeros past the end of the row)
#pragma unroll
            for (int c = 0; c < 4; ++c) take(it + c, tv[c]);
        }
    };
    if (live) {
        auto absmax4 = [&](int, const f32x4 v) { amax = nan_max(nan_max(nan_max(nan_max(amax, fabsf(v.x)), fabsf(v.y)), fabsf(v.z)), fabsf(v.w)); };
        first_steps<0>(steps, [&](int it) { absmax4(it, xv[it]); });
        rest(kDecodeKeep, absmax4);
        odd = __builtin_amdgcn_ballot_w64(amax != amax) != 0;
        if (odd) {
            amax = 0.0f;
            rest(0, [&](int, const f32x4 v) { amax = fmaxf(fmaxf(amax, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w))); });
        }
        amax = wave_max_f32(amax);
    }
    if (WPT > 1) {
        if (lane == 0) *(lds_f32*)(red + wave * 4) = amax;
        wg_barrier_lds();
#pragma unroll
        for (int s = 0; s < WPT; ++s) amax = fmaxf(amax, *(const lds_f32*)(red + (tok * WPT + s) * 4));
    }
    if (live) {
        const float inv = (amax > 0.0f) ? 127.0f / amax : 0.0f;
        if (sub == 0 && lane == 0) {
            const float sc = amax / 127.0f;
            *(lds_f32*)(red + 64 + tok * 4) = sc;
            if (p.a_scale_out && blockIdx.x == 0) p.a_scale_out[tok] = sc;
        }
        const int u = lane >> 2;
        const unsigned dst = (unsigned)(((u * T) + ((tok + (u >> kShift)) & (T - 1))) * 16 + (lane & 3) * 4) + (unsigned)sub * (256u * T);
        auto put = [&](int it, unsigned codes) { *(lds_i32*)(dst + (unsigned)it * (WPT * 256u * T)) = (int)quad_transpose_codes(codes, lane); };
        if (!odd && __builtin_amdgcn_readfirstlane((int)quant_in_range(amax))) {
            first_steps<0>(steps, [&](int it) { put(it, quant_codes4<false>(xv[it], inv)); });
            rest(kDecodeKeep, [&](int it, const f32x4 v) { if (it < steps) put(it, quant_codes4<false>(v, inv)); });
        } else {
            rest(0, [&](int it, const f32x4 v) { if (it < steps) put(it, quant_codes4<true>(v, inv)); });
        }
    }
    wg_barrier_lds();

    // ---- multiply: macro steps part, part + KP, ... of row tile rt
    unsigned rd[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) rd[q] = (unsigned)(((kb * 4 + q) * T + ((i + ((kb * 4 + q) >> kShift)) & (T - 1))) * 16);
    const UnpackConst uc(4);
    i32x4 acc = {0, 0, 0, 0};
    for (int m0 = part; m0 < p.macros; m0 += KP * PF) {
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int macro = m0 + KP * j;
            if (macro < p.macros) {
                const unsigned keep = 4 * macro + kb < p.KCn ? 0xffffffffu : 0u;
                i32x4 a[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) a[q] = *(const lds_i32x4*)(rd[q] + (unsigned)macro * (256u * T));
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[q], unpack_planes4((unsigned)w[j][q], keep, uc), acc, 0, 0, 0);
                }
                w[j] = load_w(macro + KP * PF);
            }
        }
    }
    // ---- lane: output row i, tokens 4 kb .. 4 kb + 3
    *(lds_i32x4*)(sums + (unsigned)(wave * 1024 + lane * 16)) = acc;
    wg_barrier_lds();
    out.store(p, sums, [&](int n, float) { return *(const lds_f32*)(red + 64 + n * 4); });
}

// ---------------------------------------------------------------------------------------------
// The same product from INT8 codes, 8 * CH tokens per workgroup, four or five weights per byte: it copies their codes over all of K to LDS
// as they lie in memory, one 16-byte unit (two k of eight tokens) per lane, and reads its operands with the transposing reads of
// gemm_kernel.  Tile columns (64 or 80 k) are pitched 128 bytes beyond their size and chunks 16 bytes beyond a multiple of 256, so that
// the 32 rows of half a read lie in distinct banks (five weights: nearly).  What lies behind the last k in LDS meets zero
// weights, what lies in an absent chunk makes sums that are not stored.
// All of the codes at once, one barrier, all of the weights: a launch is little more than two trips to memory, where gemm_kernel waits
// for one with every macro step.
// ---------------------------------------------------------------------------------------------
constexpr int codes_column(int gw) { return 16 * gw * 8 + 128; }
constexpr int decode_codes_pitch(int gw, int64_t K) { return (int)((K + 64 * gw - 1) / (64 * gw)) * 4 * codes_column(gw) + 16; }
constexpr int decode_codes_lds_bytes(int gw, int ch, int64_t K) { return ch * decode_codes_pitch(gw, K) + kDecodeWaves * 1024; }
// K that the LDS of a workgroup holds: 14592 values for one chunk, 7168 for two (five weights per byte: 14592 and 7360)
constexpr bool decode_codes_fits(int gw, int ch, int64_t K) { return K <= 14592 && decode_codes_lds_bytes(gw, ch, K) <= 160 * 1024; }

template <int GW, int CH, int MT>
__global__ void __launch_bounds__(64 * kDecodeWaves) decode_codes_kernel(const DecodeParams p) {
    constexpr int KP = kDecodeWaves / MT;      // parts of K
    constexpr int PF = 4;                      // macro steps of weights in flight
    constexpr int NU = 4;                      // units per thread and pass
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kColumn = codes_column(GW);
    constexpr unsigned kZero = GW == 4 ? kZeroIdx4 : 0x79797979u;      // four bytes of the all-zero pattern
    const unsigned pitch = (unsigned)p.pitch;
    const unsigned sums = CH * pitch;
    // tiles as in gemm_kernel: the token tiles of a row tile next to each other, a contiguous range of the list for each XCD
    const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (tile >= p.tiles) return;
    const int mt = p.tiles_n == 1 ? tile : (int)__umulhi((unsigned)tile, p.magic_n), nt = tile - mt * p.tiles_n;
    const int m0 = mt * 16 * MT;

    // ---- request the codes first (they are copied while the weights are on their way), then the epilogue's scales, then weights
    const int units = p.K >> 1;                            // of a chunk (K % 4 == 0); chunks lie one behind the other
    const int total = CH == 2 && 2 * nt + 1 < p.chunks ? 2 * units : units;
    const int8_t* codes = p.a_q + (size_t)nt * CH * p.K * 8;
    i32x4 v[NU];
    auto load_units = [&](int u0) {
#pragma unroll
        for (int j = 0; j < NU; ++j)
            if (u0 + 64 * kDecodeWaves * j + 64 * wave < total)        // (uniform)
                v[j] = *(const i32x4*)(codes + (size_t)min(u0 + 64 * kDecodeWaves * j + tid, total - 1) * 16);
    };
    auto store_units = [&](int u0) {
#pragma unroll
        for (int j = 0; j < NU; ++j) {
            const int u = u0 + 64 * kDecodeWaves * j + tid;
            if (u < total) {
                const bool second = CH == 2 && u >= units;
                const unsigned at = (unsigned)(second ? u - units : u);
                *(lds_i32x4*)((second ? pitch : 0u) + at * 16u + (GW == 4 ? at >> 5 : at * 52429u >> 21) * 128u) = v[j];     // at / 32 or / 40, the column
            }
        }
    };
    load_units(0);
    const int rt = wave % MT, part = wave / MT;
    const int i = lane & 15, kb = lane >> 4;
    const DecodeWeights weights(p, m0, rt * 16 + i, kb);
    const DecodeOut<8 * CH, MT> out(p, tid, m0, nt * 8 * CH);
    unsigned w4 = kZeroIdx4;
    if (GW == 5 && p.packed4) {
        const int m = m0 + rt * 16 + i;
        w4 = *(const unsigned*)(p.packed4 + (size_t)min(m >> 2, p.RGtotal - 1) * p.KCn4 * 64 + (m & 3) * 16);
    }
    i32x4 w[PF];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PF; ++j) w[j] = weights.load(part + KP * j);
    __builtin_amdgcn_sched_barrier(0);
    store_units(0);
    for (int u0 = 64 * kDecodeWaves * NU; u0 < total; u0 += 64 * kDecodeWaves * NU) {
        load_units(u0);
        store_units(u0);
    }
    wg_barrier_lds();

    // ---- multiply: macro steps part, part + KP, ... of row tile rt.  Of a group of 16 lanes two point at each of eight rows (k in the
    //      order of the planes), one per chunk, and lane i receives the eight values of token i
    const int r8 = i >> 1;
    const unsigned second = CH == 2 && (lane & 1) ? pitch : 0u;
    const unsigned rd = (unsigned)(kb * kColumn + (r8 & 3) * GW * 8 + (r8 >> 2) * 8) + second;
    const unsigned rd_b = (unsigned)(kb * kColumn + (r8 & 3) * GW * 8 + (r8 >> 2) * 4 * GW * 8 + 32) + second;     // (five weights) plane 4 of two dwords
    const UnpackConst uc(GW);
    i32x4 acc = {0, 0, 0, 0};
    for (int s0 = part; s0 < p.macros; s0 += KP * PF) {
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int macro = s0 + KP * j;
            if (macro < p.macros) {
                const unsigned keep = 4 * macro + kb < p.KCn ? 0xffffffffu : 0u;
                const unsigned at = (unsigned)macro * (4u * kColumn);
                i32x4 a[GW];
#pragma unroll
                for (int q = 0; q < GW; ++q) {
                    const unsigned from = q < 4 ? rd + at + q * 4 * GW * 8 : rd_b + at;
                    const i32x2 lo = lds_read_tr8(from), hi = lds_read_tr8(from + (q < 4 ? 16 : 2 * 4 * GW * 8));
                    a[q] = i32x4{lo.x, lo.y, hi.x, hi.y};
                }
                unsigned left[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    Unpack<GW> un;
                    i32x4 b;
                    un.w = ((unsigned)w[j][q] & keep) | (kZero & ~keep);
#pragma unroll
                    for (int st = 0; st < Unpack<GW>::kOps; ++st) un.op(st, uc, b, left[q]);
                    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[q], b, acc, 0, 0, 0);
                }
                if constexpr (GW == 5)
                    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[4], i32x4{(int)left[0], (int)left[1], (int)left[2], (int)left[3]}, acc, 0, 0, 0);
                w[j] = weights.load(macro + KP * PF);
            }
        }
    }
    if constexpr (GW == 5) {
        if (p.packed4 && part == 0) {                      // (mixed packing) its dword of a row holds up to 16 values, planes of four weights per byte
            const unsigned u0 = (unsigned)p.Kmain >> 1;    // their first unit; they lie in one tile column (Kmain is a multiple of 20)
            const unsigned at = second + u0 * 16u + (u0 * 52429u >> 21) * 128u + (unsigned)((r8 & 3) * 32 + (r8 >> 2) * 8);
            const i32x2 lo = lds_read_tr8(at), hi = lds_read_tr8(at + 16);
            acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(i32x4{lo.x, lo.y, hi.x, hi.y}, unpack_planes4(w4, kb == 0 ? 0xffffffffu : 0u, UnpackConst(4)), acc, 0, 0, 0);
        }
    }
    *(lds_i32x4*)(sums + (unsigned)(wave * 1024 + lane * 16)) = acc;     // output row i, tokens 4 kb .. 4 kb + 3
    wg_barrier_lds();
    out.store(p, sums, [](int, float scale) { return scale; });
}

}  // namespace
