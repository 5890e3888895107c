// The mpGeMM as a contraction on the INT8 matrix cores: the packed bytes are taken apart in registers, next to the
// matrix instruction that uses them.  Serves the 2-bit, the 1.60-bit and the mixed packing.
// Part of the single translation unit vlut.hip (included there, in this order).
#pragma once

namespace {

typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;

// ---------------------------------------------------------------------------------------------
// Workgroup = WM x WK waves; tile = 32*RT*WM output rows x 32*CT tokens.  The WK groups of WM waves take every WK-th
// macro step of K (two packed tile columns: 128 values of K at four weights per byte, 160 at five) and their INT32
// sums meet in LDS at the end, so that a tile keeps eight waves busy without partial sums in device memory.
//
// Weights.  v_mfma_i32_32x32x32_i8 wants, per lane, 16 values of K of one row: a lane loads the 16 packed bytes of
// its row and tile column (one 16-byte load per macro step, whole 128-byte lines per four rows) and unpacks four bytes
// at a time into "planes": plane j holds digit j of the four bytes.  That is a fixed permutation of K inside the 16
// (20) values of a dword, which the activations follow, so no byte is ever moved to its natural place.  Four bytes
// cost 13 VALU instructions (see Unpack).
//
// Activations.  The token-chunked layout [N/8][K][8] goes through LDS as it is, 16 bytes (two k of eight tokens) per
// lane, and ds_read_b64_tr_b8 transposes it on the way to the registers: 16 lanes point at 8 rows (k) x 16 tokens, lane
// i receives the eight values of token i.  Which k a row pointer names is free, so the plane order costs nothing.
// Chunks of eight tokens are pitched so that the 16 eight-byte rows of a read lie in distinct banks.
//
// What bounds it (rates of this chip, measured): power.  13.5 ns per v_mfma_i32_32x32x32_i8 and SIMD on zeros (2.38 GHz), 16.8 on codes and
// ternary weights (1.95 GHz, 4.0 POP/s), 18.5 with four byte permutes beside each (1.88 GHz, 3.6 POP/s); LDS serves transposing reads at
// 183 and writes at 71 bytes per clock.  With CT = 4 a wave spends 3.3 unpacking instructions per matrix instruction, hence the wide
// token tile.  The larger tiles with four weights per byte are gemm_ring_kernel's and gemm_private_kernel's.
// ---------------------------------------------------------------------------------------------
struct GemmParams {
    const uint8_t* packed;
    const uint8_t* packed4;   // mixed packing: the 2-bit blob of the last K - K5 < 20 values of K, else null
    const int8_t* a_q;
    const float* a_scale;
    const float* w_rows;
    float* y;
    int32_t* acc;
    float w_scale;
    int M, N, Ka;             // Ka: activation rows per token chunk
    int Kmain;                // values of K in `packed`
    int KCn, KCn4, RGtotal, ldy, chunks;
    int macros;               // macro steps of `packed`
    int tiles_n, tiles, per_xcd;
    int stream_out;           // y is too large for the caches: store past them
};

template <int GW>
struct GemmShape {
    static constexpr int kCol = 16 * GW;                   // values of K per packed tile column
    static constexpr int kUnits = kCol;                    // 16-byte units of a chunk per macro step: 2 kCol * 8 / 16
    static constexpr int kP1 = kUnits * 16 + 16;           // second chunk of a pair: half an eight-row bank window further
    static constexpr int kP2 = (2 * kUnits * 16 + 16 - 128 + 255) / 256 * 256 + 128;   // pairs alternate between the halves of the banks
};

// Four packed bytes -> GW planes of four INT8 values -w (negated: see below), in kOps single instructions so that the caller
// can place matrix instructions between them.  A byte is two base-3 numbers of two digits, 9 H + L (five weights: 27 H + 3 L + d),
// and v_perm_b32 looks four such numbers up in the eight bytes of a register pair at once.  Of the nine values 0..8 the
// ninth has no byte: its selector is made 13 or more, which the instruction answers with 0xff, the -1 of the largest digit where
// planes hold -w.  H comes from one rounding of a 16-bit float: with 0x64 above it a byte b is the number 1024 + b, and
// (1024 + b) * m + c with m just below -1/9 rounds to 1024 + 15 - H, whose low byte is taken.  Checked for every byte by the tests.
// Four weights: 13 instructions per four bytes (24 with a multiplication and a mask per digit).
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f16x2 as_f16x2(unsigned v) { return __builtin_bit_cast(f16x2, v); }

// What the instructions take from vector registers (one scalar operand each is all they may have), opaque so that the
// compiler keeps it there.
struct UnpackConst {
    unsigned high, mul, table_a, table_b;
    __device__ __forceinline__ explicit UnpackConst(int gw) {
        high = gw == 4 ? 0x64646464u : 0x67676767u;
        mul = gw == 4 ? 0xaf19af19u : 0xb556b556u;
        table_a = 0x01010100u;                             // first digit of 7 - i in byte i
        table_b = 0x0100ff01u;                             // second digit
#if defined(__HIP_DEVICE_COMPILE__)
        asm("" : "+v"(high), "+v"(mul), "+v"(table_a), "+v"(table_b));
#endif
    }
};

template <int GW>
struct Unpack {
    static constexpr int kOps = GW == 4 ? 13 : 19;
    unsigned w, e, o, hi, lo;
    // instruction st; planes into out[0..3], the fifth into out4
    __device__ __forceinline__ void op(int st, const UnpackConst& c, i32x4& out, unsigned& out4) {
        const auto fma = [](unsigned x, unsigned m, unsigned a) {
            return __builtin_bit_cast(unsigned, __builtin_elementwise_fma(as_f16x2(x), as_f16x2(m), as_f16x2(a)));
        };
        const auto plane_a = [&](unsigned index) { return (int)__builtin_amdgcn_perm(c.table_a, 0x0000ffffu, index); };
        const auto plane_b = [&](unsigned index) { return (int)__builtin_amdgcn_perm(c.table_b, 0x00ff0100u, index); };
        if (GW == 4) {
            switch (st) {
            case 0: e = __builtin_amdgcn_perm(w, c.high, 0x00060004u); break;     // 1024 + bytes 0 and 2
            case 1: o = __builtin_amdgcn_perm(w, c.high, 0x00070005u); break;     // bytes 1 and 3
            case 2: e = fma(e, c.mul, 0x64816481u); break;                        // 1024 + 15 - H
            case 3: o = fma(o, c.mul, 0x64816481u); break;
            case 4: hi = __builtin_amdgcn_perm(o, e, 0x06020400u); break;         // 15 - H
            case 5: lo = (hi << 3) + hi; break;
            case 6: lo = lo + w - 0x87878787u; break;                             // 9 * (15 - H) + b - 135 = L
            case 7: hi ^= 0x08080808u; break;                                     // 7 - H, 15 for H = 8
            case 8: out[0] = plane_a(hi); break;
            case 9: out[1] = plane_b(hi); break;
            case 10: lo ^= 0x07070707u; break;                                    // 7 - L, 15 for L = 8
            case 11: out[2] = plane_a(lo); break;
            case 12: out[3] = plane_b(lo); break;
            }
        } else {
            switch (st) {
            case 0: e = __builtin_amdgcn_perm(w, c.high, 0x00060004u); break;     // 1792 + b
            case 1: o = __builtin_amdgcn_perm(w, c.high, 0x00070005u); break;
            case 2: e = fma(e, c.mul, 0x66d566d5u); break;                        // 1024 + 127 - b / 3
            case 3: o = fma(o, c.mul, 0x66d566d5u); break;
            case 4: lo = __builtin_amdgcn_perm(o, e, 0x06020400u); break;         // 127 - b / 3
            case 5: e = fma(e, 0x2f1d2f1du, 0x631f631fu); break;                  // 1024 + 15 - b / 27
            case 6: o = fma(o, 0x2f1d2f1du, 0x631f631fu); break;
            case 7: hi = __builtin_amdgcn_perm(o, e, 0x06020400u); break;         // 15 - H
            case 8: e = (lo << 1) + lo; break;
            case 9: e = e + w - 0x7e7e7e7du; break;                               // b - 3 * (b / 3)
            case 10: o = (hi << 3) + hi; break;
            case 11: lo = o - lo; break;                                          // 9 * (15 - H) - (127 - (9 H + L)) = 8 + L
            case 12: out4 = __builtin_amdgcn_perm(0u, 0x00ff0001u, e); break;
            case 13: hi ^= 0x08080808u; break;
            case 14: out[0] = plane_a(hi); break;
            case 15: out[1] = plane_b(hi); break;
            case 16: lo ^= 0x0f0f0f0fu; break;                                    // 7 - L, 31 for L = 8
            case 17: out[2] = plane_a(lo); break;
            case 18: out[3] = plane_b(lo); break;
            }
        }
    }
};

__device__ __forceinline__ i32x2 lds_read_tr8(unsigned addr) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)addr);
#else
    (void)addr;
    return i32x2{0, 0};
#endif
}

// How the outputs leave.  A compute unit takes some 16 cycles for a store whether a lane gives one dword or four: dword by dword the
// 256 x 128 tile took 3.6 us of 32, and 6.2 with one K group; together 1.6 and 2.0.
//   kStoreTogether   the rows of lanes i and i + 16 and of the two row tiles are neighbours (gemm_row); one lane swap leaves every lane
//                    with 2 RT consecutive outputs of one token.  For weights that come from LDS: loads from memory want four neighbouring
//                    lanes in the four rows of a packed tile (otherwise the K loop is 4 to 14 % longer).
//   kStorePairs      rows in their order; neighbouring lanes exchange one of two tokens and have two consecutive outputs each.
//                    256 x 128 2.7 us, 64 x 128 1.15 -> 0.87.
//   kStoreDwords     for tiles of up to 64 tokens, where pairs gain 0.1 us of stores and lose as much to longer code (3203 x 3116 x 77, 64 x 32
//                    tiles: 5.97 us, pairs 6.04).
enum { kStoreDwords, kStorePairs, kStoreTogether };
template <int RT, int STORE>
__device__ __forceinline__ int gemm_row(int i, int rt) {      // output row, of the 32 * RT of a wave, of lane i in row tile rt
    return STORE == kStoreTogether ? 2 * RT * (i & 15) + 2 * rt + (i >> 4) : 32 * rt + i;
}
// Lanes 2 j and 2 j + 1 with (a0, b0), (a1, b1) -> (a0, a1), (b0, b1)
__device__ __forceinline__ void swap_neighbours(float& a, float& b, int lane) {
#if defined(__HIP_DEVICE_COMPILE__)
    const auto other = [](float v) { return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false)); };
    const float oa = other(a), ob = other(b);
    const float x = lane & 1 ? ob : a, y = lane & 1 ? b : oa;
    a = x;
    b = y;
    asm volatile("" : "+v"(a), "+v"(b));                   // (by all lanes, whoever stores)
#else
    (void)a; (void)b; (void)lane;
#endif
}
// Of a pair of registers: rows of 16 lanes (a0 a1 a2 a3), (b0 b1 b2 b3) -> (a0 b0 a2 b2), (a1 b1 a3 b3).  Two pairs per call.  Written out:
// from the builtin the compiler made code that took the first result for both (a test with two tokens found it).  The
// instruction wants two wait states behind the vector instruction that wrote its operands.
__device__ __forceinline__ void swap_rows16(float& a, float& b, float& c, float& d) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
#else
    (void)a; (void)b; (void)c; (void)d;
#endif
}
// One, two or four consecutive floats.  y and its rows may start at any float, and global memory takes vectors aligned to a dword: the
// store says so (by a type that is named here: one that a template deduces has lost its alignment).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x2_any __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
template <class V>
__device__ __forceinline__ void store_floats(float* dst, V v, bool past_the_caches) {
    constexpr int kWidth = sizeof(V) / 4;
    if constexpr (kWidth == 4) {
        if (past_the_caches) __builtin_nontemporal_store(v, (f32x4_any*)dst);
        else *(f32x4_any*)dst = v;
    } else if constexpr (kWidth == 2) {
        if (past_the_caches) __builtin_nontemporal_store(v, (f32x2_any*)dst);
        else *(f32x2_any*)dst = v;
    } else {
        if (past_the_caches) __builtin_nontemporal_store(v, dst);
        else *dst = v;
    }
}

// The end of a tiled product: the K groups' sums meet in LDS (overwritten from its start; the caller has passed a barrier since its last
// use), scales, stores.  A lane holds, of each 32 x 32 product, one output row (gemm_row) and the tokens 8 g + 4 kb + 0..3 in registers
// 4 g .. 4 g + 3: "quad" g.  The quads are dealt out over the WK groups, those of the RT row tiles together; a group adds the other
// groups' sums to its own.  scales: LDS address of the tile's token scales, its row scales behind them.
template <int RT, int CT, int WM, int WK, int STORE>
__device__ __forceinline__ void gemm_store(const GemmParams& p, const i32x16 (&acc)[RT][CT], int lane, int wm, int wk, int mt, int nt, unsigned scales) {
    constexpr int BN = 32 * CT, BM = 32 * RT * WM;
    constexpr int Q = RT * CT * 4;
    constexpr int kOwn = (Q + WK - 1) / WK;                // quads per group
    static_assert(kOwn % RT == 0, "the row tiles of a quad belong to one group");
    const int i = lane & 31, kb = lane >> 5;
    auto quad = [&](int qd) {
        const i32x16& v = acc[qd % RT][qd / RT / 4];
        const int g = qd / RT & 3;
        return i32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    };
    if (WK > 1) {
#pragma unroll
        for (int qd = 0; qd < Q; ++qd) {
            const int owner = qd / kOwn;
            if (owner != wk) {
                const int slot = wk - (wk > owner ? 1 : 0);
                *(lds_i32x4*)(unsigned)((((wm * Q + qd) * (WK - 1)) + slot) * 1024 + lane * 16) = quad(qd);
            }
        }
        wg_barrier_lds();
    }
    const int m_wave = mt * BM + wm * 32 * RT;
    float ws[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) ws[rt] = __builtin_bit_cast(float, *(const lds_i32*)(scales + (unsigned)((BN + wm * 32 * RT + gemm_row<RT, STORE>(i, rt)) * 4)));
    // (tokens of a store: 4 kb + a bit of the lane, then a number that all lanes share)
    constexpr bool kTogether = STORE == kStoreTogether;
    const int n_lane = nt * BN + 4 * kb + (kTogether ? (lane >> 4) & 1 : STORE == kStorePairs ? lane & 1 : 0);
    const int m_lane = m_wave + (kTogether ? 2 * RT * (i & 15) : STORE == kStorePairs ? i & ~1 : i);
    float* const y_lane = p.y + (size_t)n_lane * p.ldy + m_lane;
    auto store_quads = [&](auto inside) {                  // inside: only y is wanted and no output lies past M or N
        constexpr bool kInside = decltype(inside)::value;
#pragma unroll
        for (int q0 = 0; q0 < Q; q0 += RT) {
            if (q0 / kOwn != wk) continue;
            const int nq = 32 * (q0 / RT / 4) + 8 * (q0 / RT & 3), n = nt * BN + nq + 4 * kb;
            const i32x4 sc = *(const lds_i32x4*)(scales + (unsigned)((nq + 4 * kb) * 4));
            float out[RT][4];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                i32x4 v = -quad(q0 + rt);                  // (planes hold -w)
#pragma unroll
                for (int s = 0; s < WK - 1; ++s) v -= *(const lds_i32x4*)(unsigned)((((wm * Q + q0 + rt) * (WK - 1)) + s) * 1024 + lane * 16);
                if (!kInside && p.acc) {
                    const int m = m_wave + gemm_row<RT, STORE>(i, rt);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (m < p.M && n + e < p.N) p.acc[(size_t)m * p.N + n + e] = v[e];
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) out[rt][e] = (float)v[e] * (ws[rt] * __builtin_bit_cast(float, (int)sc[e]));
            }
            if (!kInside && !p.y) continue;
            auto put = [&](int m, int n, auto v) {         // from m_lane and n_lane on
                constexpr int kWidth = sizeof(v) / 4;
                if (!kInside && n_lane + nq + n >= p.N) return;
                float* const dst = y_lane + (size_t)(nq + n) * p.ldy + m;
                if (kInside || m_lane + m + kWidth <= p.M) {
                    store_floats(dst, v, p.stream_out);
                } else if constexpr (kWidth > 1) {
#pragma unroll
                    for (int j = 0; j + 1 < kWidth; ++j)
                        if (m_lane + m + j < p.M) dst[j] = v[j];
                }
            };
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                if constexpr (kTogether) swap_rows16(out[rt][0], out[rt][1], out[rt][2], out[rt][3]);
                if constexpr (STORE == kStorePairs) swap_neighbours(out[rt][0], out[rt][1], lane), swap_neighbours(out[rt][2], out[rt][3], lane);
            }
            if constexpr (STORE == kStoreDwords) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) put(32 * rt, e, out[rt][e]);
            } else {
#pragma unroll
                for (int h = 0; h < 4; h += 2) {
                    if constexpr (kTogether && RT == 2) {
                        put(0, h, f32x4{out[0][h], out[0][h + 1], out[1][h], out[1][h + 1]});
                    } else {
#pragma unroll
                        for (int rt = 0; rt < RT; ++rt) put(32 * rt, h, f32x2{out[rt][h], out[rt][h + 1]});
                    }
                }
            }
        }
    };
    if (STORE != kStoreDwords && p.y && !p.acc && m_wave + 32 * RT <= p.M && (nt + 1) * BN <= p.N) store_quads(std::true_type{});
    else store_quads(std::false_type{});
}

// LDS bytes of one workgroup: the double-buffered activation tiles of the WK groups, later the sums they exchange;
// behind them the scales of the tile's tokens and rows.
template <int GW, int RT, int CT, int WM, int WK>
constexpr int gemm_lds_bytes() {
    const int stage = WK * 2 * CT * 2 * GemmShape<GW>::kP2, sums = WM * RT * CT * 4 * (WK - 1) * 1024;
    return (stage > sums ? stage : sums) + 32 * (CT + RT * WM) * 4;
}

template <int GW, int RT, int CT, int WM, int WK>
__global__ void __launch_bounds__(64 * WM * WK, 2) gemm_kernel(const GemmParams p) {
    using S = GemmShape<GW>;
    constexpr int NQ = GW;                                 // matrix instructions per macro step and 32 x 32 tile
    constexpr int BN = 32 * CT;
    constexpr int kBuf = CT * 2 * S::kP2;                  // one activation tile
    constexpr int kGroupThreads = 64 * WM;
    constexpr int kUnitsTile = BN / 8 * S::kUnits;
    constexpr int kPer = (kUnitsTile + kGroupThreads - 1) / kGroupThreads;
    constexpr int BM = 32 * RT * WM;
    constexpr unsigned kZero = GW == 4 ? kZeroIdx4 : 0x79797979u;      // four bytes of the all-zero pattern
    constexpr int kScales = gemm_lds_bytes<GW, RT, CT, WM, WK>() - (BN + BM) * 4;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wk = wave / WM;
    const int i = lane & 31, kb = lane >> 5;

    // tiles in a list with the token tiles of a row tile next to each other; each XCD takes a contiguous range of it, so
    // that the workgroups that unpack the same weights share an L2
    const int tile = (blockIdx.x & 7) * p.per_xcd + (blockIdx.x >> 3);
    if (tile >= p.tiles) return;
    const int mt = tile / p.tiles_n, nt = tile - mt * p.tiles_n;
    const int m_wave = (mt * WM + wm) * 32 * RT;
    const int chunk0 = nt * (BN / 8);

    // Loads: 32-bit offsets from the uniform bases of the tile (a tile spans less than 2^31 bytes of either operand).
    // ---- weights: this lane's row of each row tile (rows past the padded matrix read data that is never stored; tile
    //      columns past the end of K are clamped and replaced by the all-zero pattern when they are unpacked)
    const int rg0 = mt * (BM / 4);
    const uint8_t* wbase = p.packed + (size_t)rg0 * p.KCn * 64;
    unsigned woff[RT], wend[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int r = wm * 32 * RT + gemm_row<RT, kStorePairs>(i, rt);
        const unsigned row = (unsigned)min(r >> 2, p.RGtotal - 1 - rg0) * (unsigned)p.KCn * 64u + (unsigned)((r & 3) * 16);
        woff[rt] = row + (unsigned)(kb * 64);
        wend[rt] = row + (unsigned)(p.KCn - 1) * 64u;
    }
    auto load_weights = [&](int macro, i32x4 (&w)[RT]) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) w[rt] = *(const i32x4*)(wbase + min(woff[rt] + (unsigned)macro * 128u, wend[rt]));
    };
    auto keep_mask = [&](int macro) { return 2 * macro + kb < p.KCn ? 0xffffffffu : 0u; };
    // ---- activations: thread of the group -> 16-byte units of the tile; chunks past the last and rows past K are
    //      clamped (such tokens are not stored, such rows meet zero weights)
    const int gt = tid - wk * kGroupThreads;
    const int8_t* abase = p.a_q + (size_t)chunk0 * p.Ka * 8;
    unsigned aoff[kPer], aend[kPer], adst[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int idx = min(gt + u * kGroupThreads, kUnitsTile - 1);
        const int c = idx / S::kUnits, unit = idx - c * S::kUnits;
        const unsigned row = (unsigned)min(c, p.chunks - 1 - chunk0) * (unsigned)p.Ka * 8u;
        aoff[u] = row + (unsigned)unit * 16u;
        aend[u] = row + (unsigned)(p.Kmain / 2 - 1) * 16u;
        adst[u] = (unsigned)((wk * 2) * kBuf + (c >> 1) * S::kP2 + (c & 1) * S::kP1 + unit * 16);
    }
    auto load_act = [&](int macro, int u) { return *(const i32x4*)(abase + min(aoff[u] + (unsigned)macro * (S::kUnits * 16u), aend[u])); };
    auto store_act = [&](int buf, int u, const i32x4 v) {
        if (kUnitsTile % kGroupThreads == 0 || u + 1 < kPer || gt + u * kGroupThreads < kUnitsTile) *(lds_i32x4*)(adst[u] + buf * kBuf) = v;
    };
    // ---- transposing reads: lane of a group of 16 -> row r of the eight, chunk half; the four groups are tokens 0-15
    //      and 16-31 of K block 0, then of K block 1
    const int r8 = (lane & 15) >> 1;
    const unsigned rd = (unsigned)((wk * 2) * kBuf + ((lane >> 4) & 1) * S::kP2 + (lane & 1) * S::kP1 + kb * S::kCol * 8 + (r8 & 3) * GW * 8);
    const unsigned rd_a = rd + (r8 >> 2) * 8;              // planes j and j + 1 of one dword
    const unsigned rd_b = rd + (r8 >> 2) * 5 * 4 * 8;      // (five weights per byte) plane 4 of two neighbouring dwords

    i32x16 acc[RT][CT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[rt][ct] = i32x16{};

    // half (0 or 1) of the activation operand ct of matrix instructions q
    auto read_half = [&](int buf, int q, int ct, int half) {
        const unsigned at = (unsigned)(buf * kBuf + ct * 2 * S::kP2);
        if (GW == 4 || q < 4) return lds_read_tr8(rd_a + at + (4 * GW * q + 2 * half) * 8);      // planes 0..3 of dword q
        return lds_read_tr8(rd_b + at + (half * 2 * 4 * GW + 4) * 8);                             // plane 4 of the four dwords
    };
    unsigned left[RT][4];                                  // plane 4 of the dwords of the current macro step

    // ---- the K loop: macro steps wk, wk + WK, ... of this group (the groups run the same number of passes; a step past
    //      the end has zero weights).  Loads run two steps ahead of their use.
    const int passes = (p.macros + WK - 1) / WK;
    i32x4 w0[RT], w1[RT], a0[kPer];
    load_weights(wk, w0);
#pragma unroll
    for (int u = 0; u < kPer; ++u) a0[u] = load_act(wk, u);
    // (mixed packing) the last < 20 values of K: at most four packed bytes per row, 16 activation rows per chunk
    i32x4 at4 = {0, 0, 0, 0};
    unsigned w4[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) w4[rt] = kZeroIdx4;
    if (GW == 5 && p.packed4) {
        if (tid < BN) {
            const int row2 = min((p.Kmain >> 1) + (tid & 7), (p.Ka >> 1) - 1);
            at4 = *(const i32x4*)(p.a_q + (size_t)min(chunk0 + (tid >> 3), p.chunks - 1) * p.Ka * 8 + (size_t)row2 * 16);
        }
        if (wk == 0 && kb == 0) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const int row = m_wave + gemm_row<RT, kStorePairs>(i, rt);
                w4[rt] = *(const unsigned*)(p.packed4 + (size_t)min(row >> 2, p.RGtotal - 1) * p.KCn4 * 64 + (row & 3) * 16);
            }
        }
    }
    for (int j = tid; j < BN + BM; j += 64 * WM * WK)
        *(lds_i32*)(unsigned)(kScales + j * 4) = __builtin_bit_cast(
            int, j < BN ? p.a_scale[min(nt * BN + j, p.N - 1)] : (p.w_rows ? p.w_rows[min(mt * BM + j - BN, p.M - 1)] : p.w_scale));
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        store_act(0, u, a0[u]);
        a0[u] = load_act(wk + WK, u);
    }
    load_weights(wk + WK, w1);                             // (requested after them, as in the loop: loads return in order)
    i32x4 a[CT], b[RT];
    Unpack<GW> un[RT];
    constexpr int kOps = Unpack<GW>::kOps;
    const UnpackConst uc(GW);
    // step st of making the weight operands of matrix instructions q from the raw dwords w
    auto unpack_step = [&](const i32x4 (&w)[RT], unsigned keep, int q, int st, i32x4 (&o)[RT]) {
        const int rt = st / kOps, j = st % kOps;
        if (q >= 4) {
            if (j == 0) o[rt] = i32x4{(int)left[rt][0], (int)left[rt][1], (int)left[rt][2], (int)left[rt][3]};
            return;
        }
        if (j == 0) un[rt].w = ((unsigned)w[rt][q] & keep) | (kZero & ~keep);
        un[rt].op(j, uc, o[rt], left[rt][q]);
    };
#pragma unroll
    for (int st = 0; st < RT * kOps; ++st) unpack_step(w0, keep_mask(wk), 0, st, b);
    wg_barrier_lds();
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const i32x2 lo = read_half(0, 0, ct, 0), hi = read_half(0, 0, ct, 1);
        a[ct] = i32x4{lo.x, lo.y, hi.x, hi.y};
    }
    // One macro step.  The operands of matrix instructions q + 1 are read and unpacked between the matrix instructions q, a
    // few vector instructions behind each of them: the matrix core works 32 cycles on one, the vector unit is free for
    // 28 of them.  (The order is pinned: left to itself the compiler gathers the vector instructions in blocks.)  The
    // one barrier stands before the last group: by then every wave holds the last operands of this tile, so the other
    // buffer (filled during this step) may be read and this one overwritten.
    auto macro_step = [&](int buf, int macro, i32x4 (&w)[RT], const i32x4 (&w_next)[RT]) {
        const unsigned keep = keep_mask(macro), keep_next = keep_mask(macro + WK);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const bool last = q + 1 == NQ;
            if (last) {
                wg_barrier_lds();
                load_weights(macro + 2 * WK, w);
            }
            i32x4 an[CT], bn[RT];
            constexpr int G = CT * RT, NS = RT * kOps, NR = 2 * CT;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                __builtin_amdgcn_sched_barrier(0);
                acc[g % RT][g / RT] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[g / RT], b[g % RT], acc[g % RT][g / RT], 0, 0, 0);
                // (the writes spread over two groups: in one burst they hold up the reads behind them)
#pragma unroll
                for (int u = (q * G + g) * kPer / (2 * G); q < 2 && u < (q * G + g + 1) * kPer / (2 * G); ++u) {
                    store_act(buf ^ 1, u, a0[u]);
                    a0[u] = load_act(macro + 2 * WK, u);
                }
#pragma unroll
                for (int r = g * NR / G; r < (g + 1) * NR / G; ++r) {
                    const i32x2 v = read_half(last ? buf ^ 1 : buf, last ? 0 : q + 1, r >> 1, r & 1);
                    an[r >> 1][2 * (r & 1)] = v.x;
                    an[r >> 1][2 * (r & 1) + 1] = v.y;
                }
#pragma unroll
                for (int st = g * NS / G; st < (g + 1) * NS / G; ++st) {
                    if (last) unpack_step(w_next, keep_next, 0, st, bn);
                    else unpack_step(w, keep, q + 1, st, bn);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) a[ct] = an[ct];
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) b[rt] = bn[rt];
        }
    };
    for (int t = 0; t < passes; t += 2) {
        macro_step(0, wk + t * WK, w0, w1);
        if (t + 1 < passes) macro_step(1, wk + (t + 1) * WK, w1, w0);
    }
    wg_barrier_lds();
    if (GW == 5 && p.packed4) {                            // its planes are those of four weights per byte
        if (tid < BN) *(lds_i32x4*)(unsigned)((tid >> 4) * S::kP2 + ((tid >> 3) & 1) * S::kP1 + (tid & 7) * 16) = at4;
        wg_barrier_lds();
        if (wk == 0) {
            const UnpackConst uc4(4);
            const unsigned rd4 = (unsigned)(((lane >> 4) & 1) * S::kP2 + (lane & 1) * S::kP1 + (r8 & 3) * 4 * 8 + (r8 >> 2) * 8);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                Unpack<4> u;
                unsigned none;
                u.w = w4[rt];
#pragma unroll
                for (int st = 0; st < Unpack<4>::kOps; ++st) u.op(st, uc4, b[rt], none);
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const i32x2 lo = lds_read_tr8(rd4 + ct * 2 * S::kP2), hi = lds_read_tr8(rd4 + ct * 2 * S::kP2 + 16);
                a[ct] = i32x4{lo.x, lo.y, hi.x, hi.y};
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[rt][ct] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[ct], b[rt], acc[rt][ct], 0, 0, 0);
            }
        }
        wg_barrier_lds();
    }

    gemm_store<RT, CT, WM, WK, (CT > 2 ? kStorePairs : kStoreDwords)>(p, acc, lane, wm, wk, mt, nt, kScales);
}

// The tile shapes that are built and what a launch costs with them, in us, fitted (rms 2 to 4 %) to launches back to back of 4100 and 1700
// shapes of 200 to 14336 rows, K = 256 to 14336 and 16 to 1024 tokens: base + n / per_unit * fixed + M * N / 10^6 * store + passes of the K
// loop * (lat + n * pass), n workgroups per compute unit.  First value four, second five weights per byte; `pass` is one macro step of every
// K group.  The tile of the least cost is within 0.4 % of the fastest on average (2 % of the shapes beyond 5 %, worst 19 %).  It ranks tiles;
// as a time it is less good than the fit: against graph replays, whose launches are shorter, of 185 other shapes 7 % too long on average (rms
// 11 %), 8 % too short above 5 * 10^9 weights times tokens (4096 x 14336 x 512: 29.8 for 36.0), and its terms are a fit's, not a model's
// (256 rows without parts of K: all of the launch in `base`, none of the store in `fixed`).  Fitted before tiles were loaded straight to LDS
// and stored wide, which makes the larger ones 7 to 19 % faster: of 450 shapes timed with that the tile of the least cost is still within 0.4 % of
// the fastest on average (3 % of them beyond 5 %), and constants fitted to the new times rank no better.
// With one K group two workgroups of four waves share a compute unit, and one stores while the other multiplies: 13824 x 2560 x 1024
// 45.7 -> 42.0 us; 128 rows x 64 tokens: 4096 x 14336 x 512 40.1 -> 36.0 us (both of gemm_kernel, which runs neither now).
// Five weights per byte take more registers than four: 64 x 64 133 per lane, so that one workgroup has a unit to itself (per_unit), 256 x 128
// all 256 and three in scratch (at most 2 % of a launch: 13620 x 260 x 281 11.4 -> 11.5 us against the unpacking before, which did
// without; 8 % faster than with that on average of 31 shapes).
struct GemmTile {
    int rt, ct, wm, wk;
    int per_unit[2];               // workgroups that share a compute unit (what a workgroup costs besides its K loop overlaps)
    double base[2], fixed[2], store[2], lat[2], pass[2];
    constexpr int rows() const { return 32 * rt * wm; }
    constexpr int tokens() const { return 32 * ct; }
};
constexpr GemmTile kGemmTiles[] = {
    {2, 4, 4, 2, {1, 1}, {3.70, 4.94}, {4.43, 3.47}, {0.681, 0.760}, {0.000, 0.000}, {1.123, 1.406}},
    {2, 4, 4, 1, {1, 1}, {9.15, 0.00}, {0.00, 0.00}, {0.710, 0.000}, {0.200, 0.000}, {0.489, 0.000}},      // (five weights: spills)
    {1, 4, 4, 2, {1, 1}, {2.95, 3.14}, {2.54, 2.54}, {0.753, 0.834}, {0.000, 0.000}, {0.693, 0.890}},
    {1, 4, 2, 4, {1, 1}, {2.19, 0.00}, {3.28, 0.00}, {0.785, 0.000}, {0.000, 0.000}, {0.881, 0.000}},      // few shapes (one in 10^4): long K; (five weights: more LDS than there is)
    {2, 2, 2, 4, {1, 1}, {2.21, 0.00}, {2.85, 0.00}, {0.721, 0.000}, {0.000, 0.000}, {0.829, 0.000}},
    {1, 2, 2, 4, {2, 1}, {3.01, 2.04}, {1.06, 2.13}, {1.036, 0.921}, {0.000, 0.000}, {0.546, 0.731}},
    {1, 1, 2, 4, {2, 2}, {3.24, 2.78}, {0.26, 0.89}, {1.300, 1.345}, {0.045, 0.070}, {0.350, 0.486}},
    {1, 1, 1, 8, {2, 1}, {2.93, 2.05}, {0.93, 1.81}, {2.161, 1.575}, {0.032, 0.000}, {0.452, 0.658}},
};
constexpr int kGemmTileCount = (int)(sizeof(kGemmTiles) / sizeof(kGemmTiles[0]));

// More tiles for four weights per byte, considered from ten macro steps on.  Fitted on the scale of the others to graph replays of 150
// shapes of 400 to 14336 rows, K = 256 to 14336 and 48 to 1024 tokens.  Of the 47 with fewer steps the tile of the least cost among kGemmTiles is 7 % behind
// the fastest of all on average (43 % of them beyond 5 %, worst 28 %: 7117 x 328 x 569 10.5 / 8.7 us); with 128 x 64 in two groups among them it
// would be 2 % (15 %, worst 23 %: 12800 x 256 x 528 9.5 / 11.7 us, where it would displace 256 x 128).  The line is where its constants rank without
// such losses; one fitted for short K does not exist yet.  In us:
//   128 x 64 in two K groups: 78 KB of LDS and 90 registers, so that two workgroups share a unit; 6912 x 2560 x 256 9.6 -> 9.3, 4870 x 1892 x 821 16.5 -> 13.8
//   128 x 64 in four groups of one wave (gemm_private_kernel), long K: 4096 x 14336 x 512 32.1 -> 30.7, 4864 x 7552 x 225 17.4 -> 17.3
//   160 x 64 so (gemm_private_kernel), where it fills the units as the others don't: 2560 x 6912 x 1024 25.2 -> 22.2
constexpr GemmTile kGemmTilesLong[] = {
    {1, 2, 4, 2, {2, 1}, {3.32, 0.00}, {0.33, 0.00}, {1.020, 0.000}, {0.121, 0.000}, {0.385, 0.000}},
    {4, 2, 1, 4, {1, 1}, {2.27, 0.00}, {3.49, 0.00}, {0.638, 0.000}, {0.000, 0.000}, {0.838, 0.000}},
    {5, 2, 1, 4, {1, 1}, {2.46, 0.00}, {3.88, 0.00}, {0.740, 0.000}, {0.000, 0.000}, {1.002, 0.000}},
};
constexpr int kGemmTilesLongCount = (int)(sizeof(kGemmTilesLong) / sizeof(kGemmTilesLong[0])), kGemmTilesLongMacros = 10;
constexpr GemmTile gemm_tile(int tile) { return tile < kGemmTileCount ? kGemmTiles[tile] : kGemmTilesLong[tile - kGemmTileCount]; }
constexpr bool gemm_tile_built(int gw, int tile) { return gw == 4 || gemm_tile(tile).pass[1] > 0.0; }
// 128 x 64 in four groups of two waves (64 rows each) is left out where these three are considered: of the 103 shapes with ten macro steps or
// more the tile of the least cost is then within 0.6 % of the fastest on average (with it 0.7 %, without the three 2.9 %).
constexpr bool gemm_tile_considered(int gw, int tile, int64_t macros) {
    const bool more = gw == 4 && macros >= kGemmTilesLongMacros;
    const GemmTile t = gemm_tile(tile);
    return gemm_tile_built(gw, tile) && (tile < kGemmTileCount ? !(more && t.rt == 2 && t.ct == 2) : more);
}

}  // namespace
