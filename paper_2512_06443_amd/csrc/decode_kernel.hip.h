// Up to sixteen tokens from fp32 activations in one launch: quantisation, unpacking and the INT8 matrix cores.
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
// Bound by latency: launch, the rows of x, one trip to HBM for the weights, 24 instructions per four packed bytes.
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
    int M, N, K, KCn, RGtotal, ldy, macros, x_vec;
};

constexpr int kDecodeWaves = 16;
constexpr int kDecodeKeep = 12;                // float4 of x per lane kept between the two passes; the rest is read twice
constexpr int decode_lds_bytes(int T, int macros) { return macros * 256 * T + kDecodeWaves * 1024 + 128; }

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
    const float* row = p.x + (size_t)(live ? tok : 0) * p.ldx;
    const int nquad = p.K >> 2;
    auto load4 = [&](int macro) -> f32x4 {
        const int qi = macro * 64 + lane;
        if (qi >= nquad) return f32x4{0.f, 0.f, 0.f, 0.f};
        const float* src = row + 4 * (size_t)qi;
        if (p.x_vec) return *(const f32x4*)src;
        return f32x4{src[0], src[1], src[2], src[3]};
    };
    f32x4 xv[kDecodeKeep];
    if (live) {
#pragma unroll
        for (int it = 0; it < kDecodeKeep; ++it)
            if (sub + WPT * it < p.macros) xv[it] = load4(sub + WPT * it);
    }
    const int rt = wave % MT, part = wave / MT;
    const int i = lane & 15, kb = lane >> 4;
    const int m_row = (blockIdx.x * MT + rt) * 16 + i;
    const uint8_t* wrow = p.packed + (size_t)min(m_row >> 2, p.RGtotal - 1) * p.KCn * 64 + (m_row & 3) * 16;
    auto load_w = [&](int macro) { return *(const i32x4*)(wrow + (size_t)min(4 * macro + kb, p.KCn - 1) * 64); };
    i32x4 w[PF];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < PF; ++j) w[j] = load_w(part + KP * j);
    __builtin_amdgcn_sched_barrier(0);

    // ---- quantise: absmax over the row, then codes (the decisions of quant_codes4, IEEE divisions)
    auto absmax4 = [](float m, const f32x4 v) { return fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w))); };
    float amax = 0.0f;
    if (live) {
#pragma unroll
        for (int it = 0; it < kDecodeKeep; ++it)
            if (sub + WPT * it < p.macros) amax = absmax4(amax, xv[it]);
        for (int m0 = sub + WPT * kDecodeKeep; m0 < p.macros; m0 += WPT * 4) {
            f32x4 tv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) tv[c] = m0 + WPT * c < p.macros ? load4(m0 + WPT * c) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c) amax = absmax4(amax, tv[c]);
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
        const unsigned dst = (unsigned)(((u * T) + ((tok + (u >> kShift)) & (T - 1))) * 16 + (lane & 3) * 4);
        auto emit = [&](int macro, const f32x4 v) {
            *(lds_i32*)(dst + (unsigned)macro * (256u * T)) = (int)quad_transpose_codes(quant_codes4(v, inv), lane);
        };
#pragma unroll
        for (int it = 0; it < kDecodeKeep; ++it)
            if (sub + WPT * it < p.macros) emit(sub + WPT * it, xv[it]);
        for (int m0 = sub + WPT * kDecodeKeep; m0 < p.macros; m0 += WPT * 4) {
            f32x4 tv[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) tv[c] = m0 + WPT * c < p.macros ? load4(m0 + WPT * c) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (m0 + WPT * c < p.macros) emit(m0 + WPT * c, tv[c]);
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
                    Unpack<4> un;
                    i32x4 b;
                    unsigned none;
                    un.w = ((unsigned)w[j][q] & keep) | (kZeroIdx4 & ~keep);
#pragma unroll
                    for (int st = 0; st < Unpack<4>::kOps; ++st) un.op(st, uc, b, none);
                    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[q], b, acc, 0, 0, 0);
                }
                w[j] = load_w(macro + KP * PF);
            }
        }
    }
    // ---- lane: output row i, tokens 4 kb .. 4 kb + 3
    *(lds_i32x4*)(sums + (unsigned)(wave * 1024 + lane * 16)) = acc;
    wg_barrier_lds();
    for (int o = tid; o < 16 * MT * p.N; o += 64 * kDecodeWaves) {
        const int n = o / (16 * MT), ml = o % (16 * MT);
        const unsigned src = sums + (unsigned)((ml >> 4) * 1024 + ((n >> 2) * 16 + (ml & 15)) * 16 + (n & 3) * 4);
        int v = 0;
#pragma unroll
        for (int k = 0; k < KP; ++k) v -= *(const lds_i32*)(src + (unsigned)(k * MT * 1024));
        const int m = blockIdx.x * 16 * MT + ml;
        if (m < p.M) {
            const float ws = p.w_rows ? p.w_rows[m] : p.w_scale;
            if (p.y) p.y[(size_t)n * p.ldy + m] = (float)v * (ws * *(const lds_f32*)(red + 64 + n * 4));
            if (p.acc) p.acc[(size_t)m * p.N + n] = v;
        }
    }
}

}  // namespace
