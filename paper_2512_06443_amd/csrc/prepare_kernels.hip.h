// Kernels that prepare operands: offline weight packing (Sec. 3.3), activation quantisation + transposition (Sec. 3.4,
// Sec. 3.3), the table materialised in device memory (Alg. 1 Precompute / Eq. 1).
// Part of the single translation unit vlut.hip (included there, in this order).
#pragma once

namespace {

// ---------------------------------------------------------------------------------------------
// Offline packing (Sec. 3.3), padding bytes included.  A thread makes one dword of the blob: four groups of one row.
// Threads in the order of the blob (4 dwords of a row, 4 rows, then the next tile column), so a wave stores 256
// contiguous bytes and reads 4 * 64 * GW / 4 contiguous bytes of each of four rows.  A group is one signed dot product of
// its bytes with the powers of three, plus the value of the all-zero pattern.
// Bound by memory: 14336 x 4096 (58.7 MB in, 14.7 MB out) 14.2 us, 5.2 TB/s; 30.3 us with one thread per byte and byte loads.
// ---------------------------------------------------------------------------------------------
// Nonzero if a byte of w is outside {-1, 0, +1}: its bits 1..7 differ, or it is -2.
__device__ __forceinline__ unsigned not_ternary(unsigned w) {
    return ((w ^ (w << 1)) & 0xfcfcfcfcu) | ((w >> 1) & ~w & 0x01010101u);
}
__device__ __forceinline__ int dot4_i8(unsigned a, int b, int c) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_sdot4((int)a, b, c, false);
#else
    (void)a; (void)b;
    return c;
#endif
}

// (weights and blob may start at any byte: global memory takes unaligned dwords)
typedef unsigned unaligned_u32 __attribute__((aligned(1)));
typedef int unaligned_i32x4 __attribute__((ext_vector_type(4), aligned(1)));

template <int GW>   // GW = weights per byte: 4 (2.00 bits per weight) or 5 (1.60)
__global__ void __launch_bounds__(256) pack_kernel(const int8_t* __restrict__ w, int M, int64_t ldw, int G, int KCn, int RGtotal,
                                                   unaligned_u32* __restrict__ packed, volatile int* error) {
    const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    const size_t tile = i >> 4;
    if (tile >= (size_t)RGtotal * KCn) return;
    const int rg = (int)(tile / KCn), kc = (int)(tile - (size_t)rg * KCn);
    const int m = rg * 4 + (int)((i >> 2) & 3);
    const int kg = kc * 16 + (int)(i & 3) * 4;             // first of the thread's four groups
    constexpr unsigned kZero = GW == 4 ? 40u : 121u;       // the all-zero pattern: every digit 1
    constexpr int kPow = GW == 4 ? 0x0103091b : 0x03091b51;   // 27, 9, 3, 1 or 81, 27, 9, 3: first weight in the low byte
    unsigned out = kZero * 0x01010101u;
    if (m < M && kg < G) {
        const int8_t* src = w + (size_t)m * (size_t)ldw + (size_t)kg * GW;
        const int groups = min(4, G - kg);
        unsigned d[GW] = {};                               // the 4 * GW weights, zeros past the last group
        if (groups == 4) {
            const unaligned_i32x4 v = *(const unaligned_i32x4*)src;
            d[0] = (unsigned)v.x; d[1] = (unsigned)v.y; d[2] = (unsigned)v.z; d[3] = (unsigned)v.w;
            if constexpr (GW == 5) d[4] = *(const unaligned_u32*)(src + 16);
        } else {
#pragma unroll
            for (int j = 0; j < 4 * GW; ++j)
                if (j < groups * GW) d[j >> 2] |= (unsigned)(unsigned char)src[j] << (8 * (j & 3));
        }
        unsigned bad = 0;
#pragma unroll
        for (int j = 0; j < GW; ++j) bad |= not_ternary(d[j]);
        if (bad) *error = 1;                               // (host memory; every writer writes the same value)
        out = 0;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            int v;
            if constexpr (GW == 4) {
                v = dot4_i8(d[g], kPow, (int)kZero);
            } else {                                       // bytes 5 g .. 5 g + 4 of the twenty
                const unsigned first = g == 0 ? d[0] : __builtin_amdgcn_alignbyte(d[g + 1], d[g], (unsigned)g);
                v = dot4_i8(first, kPow, (int)kZero + (int)(signed char)(d[g + 1] >> (8 * g)));
            }
            out |= (unsigned)(v & 0xff) << (8 * g);
        }
    }
    packed[i] = out;
}

// ---------------------------------------------------------------------------------------------
// Activation quantisation + transposition (Sec. 3.4 first paragraph, Sec. 3.3).
// For many tokens: one workgroup handles four consecutive tokens (half a chunk) or all eight of a chunk over all K, and a
// row stays in registers between the absmax and the rounding (four tokens: up to 14336 values, eight: up to 3072).  Four tokens
// are for about a thousand tokens and more, so that 1024 tokens are one workgroup per compute unit (N = 1024: 8.4 us at K = 6912,
// 15.9 us at K = 14336; one token per workgroup: 8.9 and 17.0 us).  Eight are for several thousand tokens of short rows, where the stores
// bound it: a wave then writes whole lines of the chunk instead of every second dword of them (N = 4096: 5.6 / 8.8 / 11.2 us at K = 1028 /
// 2048 / 2560; four tokens: 7.1 / 10.2 / 12.1).  A wave reads 64 / TOK consecutive float4 of each of its tokens (lane = token + TOK * quad).  The four codes
// a lane makes (4 consecutive k of one token) are transposed inside its quad of lanes, so that every lane leaves with
// one dword of the chunk's [K][8] block (4 tokens of one k); the two halves of a chunk are blocks 8 apart (same XCD under
// round-robin dispatch), so their half lines meet in one L2.
//   TOK tokens per workgroup: 4 or 8
//   NV  float4 values per thread kept in registers between the absmax pass and the rounding pass
//       (0: x is read twice, for large K)
//   VEC true when rows can be read as float4 (x and ldx 16-byte aligned)
// ---------------------------------------------------------------------------------------------
constexpr int kQuantThreads = 1024;
typedef float f32x4 __attribute__((ext_vector_type(4)));

// The larger value, NaN where either is one.  (fmaxf drops NaNs, for which the compiler first rewrites every operand.)
__device__ __forceinline__ float nan_max(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_elementwise_maximum(a, b);
#else
    (void)b;
    return a;
#endif
}

// Absmax quantiser of one token row, decided in fp32: inv = 127 / amax (IEEE division, 0 for an all-zero row),
// code = clamp(rint(x * inv), -127, 127) with ties to even.
// Four values at once, code of v[c] in byte c.  Adding 1.5 * 2^23 to the product (rounded to fp32 first: there is no
// contraction here) rounds it to an integer with ties to even and leaves that integer, two's complement, in the low byte of
// the sum.  The clamp comes before the rounding, which gives the same code; it only matters where 127 / amax overflows
// (rows below 4e-37) or x has an infinity or a NaN: -inf and NaN become -127, +inf 127.  CLAMP false: the caller has ruled these out
// (the product of |x| <= amax and 127 / amax is at most 127 * (1 + 2^-23), which rounds to 127).
template <bool CLAMP = true>
__device__ __forceinline__ unsigned quant_codes4(const f32x4 v, float inv) {
    unsigned u[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float t = v[c] * inv;
        u[c] = __builtin_bit_cast(unsigned, (CLAMP ? __builtin_amdgcn_fmed3f(t, -127.0f, 127.0f) : t) + 12582912.0f);
    }
    return __builtin_amdgcn_perm(u[1], u[0], 0x0c0c0400u) | __builtin_amdgcn_perm(u[3], u[2], 0x04000c0cu);
}
// Rows that need no clamp, from the greatest magnitude of their values without NaN.
__device__ __forceinline__ bool quant_in_range(float amax) { return (amax >= 4e-37f && amax < INFINITY) || amax == 0.0f; }

// The lane holds the codes of k = 4q .. 4q+3 of token `tok` (byte c = k offset c); the four lanes of a quad hold
// four consecutive tokens of the same q.  Returns, for the lane with tok % 4 == c, the codes of those four tokens
// at k = 4q + c (byte e = token 4*(tok/4) + e).  Two exchanges: bytes with the neighbour, halves with the other pair.
__device__ __forceinline__ unsigned quad_transpose_codes(unsigned d, int tok) {
    const unsigned pair = (tok & 1) ? 0x03070105u : 0x06020400u, half = (tok & 2) ? 0x03020706u : 0x05040100u;
    const unsigned e = __builtin_amdgcn_perm((unsigned)lane_xor16<1>((int)d), d, pair);
    return __builtin_amdgcn_perm((unsigned)lane_xor16<2>((int)e), e, half);
}

template <int TOK, int NV, bool VEC>
__global__ void __launch_bounds__(kQuantThreads) quantize_kernel(const float* __restrict__ x, int N, int K, int64_t ldx,
                                                                 int8_t* __restrict__ a_q, float* __restrict__ a_scale, int chunks) {
    constexpr int QW = 64 / TOK;               // quads of each token that a wave handles per pass
    constexpr int QP = kQuantThreads / TOK;    // and the workgroup
    __shared__ __attribute__((aligned(16))) float red[TOK][kQuantThreads / 64];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x;
    const int chunk = TOK == 8 ? b : (b >> 4) * 8 + (b & 7), half = TOK == 8 ? 0 : (b >> 3) & 1;
    if (chunk >= chunks) return;
    const int t = lane & (TOK - 1);            // token of the four or eight
    const int kq = wave * QW + lane / TOK;     // this thread handles k = 4*(kq + QP*i) .. +3
    const int n = chunk * 8 + half * 4 + t;
    const bool live = n < N;
    const float* row = x + (size_t)(live ? n : 0) * ldx;
    const int nquad = K >> 2;                  // K % 4 == 0
    constexpr int NB = NV > 0 ? NV : 8;        // loads in flight per thread and pass
    auto load_pass = [&](int q0, f32x4 (&v)[NB]) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int qi = q0 + kq + QP * i;
            const float* src = row + 4 * (size_t)qi;
            if (!live || qi >= nquad) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            else if (VEC) v[i] = *(const f32x4*)src;
            else v[i] = f32x4{src[0], src[1], src[2], src[3]};
        }
    };
    f32x4 xv[NB];
    float amax = 0.0f;
    for (int q0 = 0; q0 < (NV > 0 ? 1 : nquad); q0 += QP * NB) {
        load_pass(q0, xv);
#pragma unroll
        for (int i = 0; i < NB; ++i)
            amax = fmaxf(fmaxf(amax, fmaxf(fabsf(xv[i].x), fabsf(xv[i].y))), fmaxf(fabsf(xv[i].z), fabsf(xv[i].w)));
    }
    for (int off = 32; off >= TOK; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));   // lanes of the same token
    if (lane < TOK) red[lane][wave] = amax;
    __syncthreads();
    float v = 0.0f;
#pragma unroll
    for (int w4 = 0; w4 < kQuantThreads / 256; ++w4) {
        const f32x4 r = *(const f32x4*)&red[t][4 * w4];
        v = fmaxf(fmaxf(v, fmaxf(r.x, r.y)), fmaxf(r.z, r.w));
    }
    // IEEE-correct fp32 divisions (the default for HIP); no reciprocal approximation.
    const float inv = (v > 0.0f) ? 127.0f / v : 0.0f;
    if (tid < TOK && live) a_scale[n] = v / 127.0f;
    unsigned* dst = (unsigned*)(a_q + (size_t)chunk * K * 8) + (TOK == 8 ? t >> 2 : half);
    for (int q0 = 0; q0 < (NV > 0 ? 1 : nquad); q0 += QP * NB) {
        if (NV == 0) load_pass(q0, xv);
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int qi = q0 + kq + QP * i;   // uniform in a quad of lanes; tokens past N: x = 0 -> code 0
            const unsigned e = quad_transpose_codes(quant_codes4(xv[i], inv), t);
            if (qi < nquad) dst[(size_t)(4 * qi + (t & 3)) * 2] = e;
        }
    }
}

// The same quantiser with one workgroup per token: every CU reads one row once.  A token owns one byte in every 8 of its
// chunk's [K][8] block, so the codes leave as single bytes (distinct bytes written by different workgroups: no race), and
// the address unit takes a byte store line by line: the four codes of a lane (32 bytes apart in the block) first go
// through the wave's 256 bytes of LDS, so that consecutive lanes store consecutive k and an instruction touches 4 lines
// instead of 16.  N = 64: 5.2 -> 3.2 us at K = 6912; N = 512, K = 14336: 20.8 -> 8.4 us.  Tokens past N (padding of the last
// chunk) are written as zeros.  Blocks are numbered so that the 8 tokens of a chunk sit 8 blocks apart (same XCD under
// round-robin dispatch, so their partial lines meet in one L2); this is a matter of speed only.
//   THREADS  by the length of the rows: a wave without a value to load costs its launch and its part of the barriers all the
//            same.  N = 4096: 3.6 us at K = 64 with one wave, 5.8 us at K = 1024 with four (512 threads: 6.5 and 7.8)
//   NV  float4 values per thread kept in registers between the two passes (0: x is read twice)
constexpr int kTokThreads = 512;               // longer rows.  256: 0.7 to 2 us slower from K = 6912 on; 1024: 0.9 us slower at K = 2560, N = 1024

template <int THREADS, int NV, bool VEC>
__global__ void __launch_bounds__(THREADS) quantize_token_kernel(const float* __restrict__ x, int N, int K, int64_t ldx,
                                                                     int8_t* __restrict__ a_q,
                                                                     float* __restrict__ a_scale, int chunks) {
    __shared__ float red[THREADS / 64];
    __shared__ unsigned codes[THREADS / 64][64];
    const int tid = threadIdx.x;
    const int b = blockIdx.x;
    const int chunk = (b >> 6) * 8 + (b & 7);
    const int t = (b >> 3) & 7;
    if (chunk >= chunks) return;
    const int n = chunk * 8 + t;
    const bool live = n < N;
    const float* row = x + (size_t)(live ? n : 0) * ldx;
    const int nquad = K >> 2;
    auto load4 = [&](int qi) -> f32x4 {
        const float* src = row + 4 * (size_t)qi;
        if (VEC) return *(const f32x4*)src;
        return f32x4{src[0], src[1], src[2], src[3]};
    };
    auto absmax4 = [](float m, const f32x4 v) {
        return fmaxf(fmaxf(m, fmaxf(fabsf(v.x), fabsf(v.y))), fmaxf(fabsf(v.z), fabsf(v.w)));
    };
    constexpr int NB = NV > 0 ? NV : 8;            // loads in flight per thread and pass
    f32x4 xv[NB];
    float amax = 0.0f;
    if (live) {
        for (int q0 = 0; q0 < (NV > 0 ? 1 : nquad); q0 += THREADS * NB) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int qi = q0 + tid + THREADS * i;
                xv[i] = qi < nquad ? load4(qi) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < NB; ++i) amax = absmax4(amax, xv[i]);
        }
    }
    amax = wave_max_f32(amax);
    if ((tid & 63) == 0) red[tid >> 6] = amax;
    __syncthreads();
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) v = fmaxf(v, red[w]);
    const float inv = (v > 0.0f) ? 127.0f / v : 0.0f;      // IEEE divisions
    if (tid == 0 && live) a_scale[n] = v / 127.0f;
    int8_t* dst = a_q + (size_t)chunk * K * 8 + t;
    unsigned* const mine = codes[tid >> 6];
    auto store4 = [&](int qi, unsigned d) {                // qi of the lane; every lane of the wave takes part
        mine[tid & 63] = d;
        __builtin_amdgcn_wave_barrier();
        const int k0 = 4 * (qi - (tid & 63)) + (tid & 63);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = k0 + 64 * j;
            if (k < K) dst[(size_t)k * 8] = ((const int8_t*)mine)[64 * j + (tid & 63)];
        }
        __builtin_amdgcn_wave_barrier();
    };
    for (int q0 = 0; q0 < (NV > 0 ? 1 : nquad); q0 += THREADS * NB) {
        if (NV == 0 && live) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int qi = q0 + tid + THREADS * i;
                xv[i] = qi < nquad ? load4(qi) : f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int qi = q0 + tid + THREADS * i;
            if (qi - (tid & 63) < nquad) store4(qi, live ? quant_codes4(xv[i], inv) : 0u);      // (uniform per wave)
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Whole table in global memory (Alg. 1 Precompute / Eq. 1), topological order of Sec. 4:
// every row is one add/sub away from an earlier one.  One thread per (group, token).
// ---------------------------------------------------------------------------------------------
//   TOKEN_OUTER false: lut[kg][i][n], tokens contiguous (Sec. 3.3, the layout of the method)
//               true:  lut[n][kg][i], one table per token (the scalar-LUT arrangement; layout ablation of Sec. 5.6)
template <bool TOKEN_OUTER>
__global__ void __launch_bounds__(256) build_lut_kernel(const int8_t* __restrict__ a_q, int G, int N,
                                                        int16_t* __restrict__ lut) {
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i >= (size_t)G * N) return;
    int n = (int)(i % N);
    int kg = (int)(i / N);
    const int8_t* a = a_q + ((size_t)(n >> 3) * (4 * G) + 4 * kg) * 8 + (n & 7);   // [N/8][K][8]
    int a0 = a[0], a1 = a[8], a2 = a[16], a3 = a[24];
    int16_t* t = TOKEN_OUTER ? lut + ((size_t)n * G + kg) * kRows : lut + ((size_t)kg * kRows) * N + n;
    const size_t row_stride = TOKEN_OUTER ? 1 : (size_t)N;
    int v0 = -a0 - a1 - a2 - a3;                       // row 0, then walk the digits
    for (int d0 = 0; d0 < 3; ++d0) {
        int v1 = v0;
        for (int d1 = 0; d1 < 3; ++d1) {
            int v2 = v1;
            for (int d2 = 0; d2 < 3; ++d2) {
                int v3 = v2;
                for (int d3 = 0; d3 < 3; ++d3) {
                    t[(size_t)(27 * d0 + 9 * d1 + 3 * d2 + d3) * row_stride] = (int16_t)v3;
                    v3 += a3;
                }
                v2 += a2;
            }
            v1 += a1;
        }
        v0 += a0;
    }
}

}  // namespace
