// The tiled mixed INT8/INT4 GEMM (Section 4.1, Eq. 4) on 128 x 128 tiles with the low
// group on the fp8 matrix cores.  Tiles, stages, loads, LDS image and output write are
// those of resq_gemm.hip.h; what differs:
//
// The low group.  Under the chip's power limit the int8 instruction alone, on nibble
// operands, sustains 3.7 to 3.9 POPS over milliseconds and the fp8 one 4.3 to 4.6 (4.1 to 4.8 and 4.9, its
// full rate, on shorter runs): a 4-bit operand lights up a quarter of an fp8 multiplier's bits.  And 4-bit codes are exact in it:
// the e4m3 numbers below 2^-5 are the multiples of 2^-9, so the byte 0..15 IS the number
// u * 2^-9, u = code + 8 the offset code.  An even activation column and an odd weight column
// are stored offset already (one AND); the others, in two's complement in the upper nibble,
// take a shift (one 64-bit shift for two registers) and one three-input operation for mask
// and sign flip.  Products of offset codes are whole multiples of 2^-18, at most 225 of them,
// so sums over up to 65536 columns (kF8MaxLoWidth) are exact in the fp32 accumulator, and
//   A_lo = sum (a + 8)(w + 8) - 8 (sum a) - 8 (sum w) - 64 columns.
// sum w is stored with the weights, the odd columns' half of sum a in lo_sum; the even
// columns' half is added up here from the widened fragments, four codes to a register and
// four stages' worth in bytes, each wavefront for 32 of its 64 tokens.
//
// Products.  32x32x64 (and 32x32x32 int8 for the high group, whose tiles must have the same
// layout): eight per stage instead of 32, which leaves the issue slots to the widening (a
// product occupies them for about 13 clocks whatever its size).  Stage order
// (b0 a0)(b0 a1)(b1 a1)(b1 a0) of the first 32 bytes, then of the second; one fragment is
// widened behind each product, in place, half a stage ahead of its use, and read from LDS
// three products before that.  No read is in flight where a stage ends, because the compiler,
// which does not know about them, may move registers there.  Buffer numbers are constants in
// the steady loop (four stages a turn): a read needs no address arithmetic.  A lane reads row
// l % 32, piece 2 h + l / 32: 16 lanes meet 16 bank groups (the 16x16x64 reads did not: half
// of their LDS cycles were conflicts).
//
// Measured (int8 kernel / this one, the two in turn): 8192 x 8192 -> 29568 at r = 0 1461 / 1399 us, r = K/8 1558 /
// 1507; 4096 x 14336 -> 4096 182 / 175; 1100 x 14336 -> 8192 125.5 / 117.5.  At r = 0 the matrix pipes are busy
// 79 % of 2.39 M clocks (71 % of 2.66 M), and the clock falls from 1.82 to 1.71 GHz: the power limit again; LDS
// bank conflicts 5.7 M (129 M).  What the rest goes to, timing-only builds at r = 0: global->LDS loads 21 %,
// widening 9 %, LDS reads 8 %.
#pragma once
#include "resq_gemm.hip.h"

namespace resq {

typedef int v8i __attribute__((ext_vector_type(8)));

// sums of products of offset codes, 225 per column at most, stay below 2^24: exact in fp32
constexpr int64_t kF8MaxLoWidth = 1 << 16;
constexpr float kF8Unit = 262144.0f;  // 2^18: an fp8 number u * 2^-9 stands for the offset code u
constexpr int kMetaSe = kMetaWsumLo;  // int32 [128]: per token, the sum of its offset codes in even columns

__device__ __forceinline__ void mfma_32x32x64_f8(v16f& acc, const v8i& b, const v8i& a) {
    asm volatile("v_mfma_f32_32x32x64_f8f6f4 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
__device__ __forceinline__ void mfma_32x32x32_i8(v16i& acc, const v4i& b, const v4i& a) {
    asm volatile("v_mfma_i32_32x32x32_i8 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}
__device__ __forceinline__ void pin(v8i& x) { asm volatile("" : "+v"(x)); }
template <int N>
__device__ __forceinline__ void lds_wait(v4i& f) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(f) : "n"(N));
}

// both registers at once (the compiler takes three-operand shifts of one register each)
__device__ __forceinline__ v2i shift_right_4(v2i x) {
    v2i y;
    asm("v_lshrrev_b64 %0, 4, %1" : "=v"(y) : "v"(x));
    return y;
}

// A fragment's 32 codes as fp8 numbers, u * 2^-9 for the offset code u = code + 8 in 0..15, the even
// columns' registers first in a pair.  lo_mask = 0x0F0F0F0F, flip = 0x08080808 (in registers).
template <bool WEIGHTS>
__device__ __forceinline__ void widen_f8(v8i& w, const v4i& r, int lo_mask, int flip) {
    constexpr int E = WEIGHTS ? 1 : 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        const v2i x = shift_right_4((v2i){r[2 * p], r[2 * p + 1]});
        w[4 * p + E] = r[2 * p] & lo_mask;
        w[4 * p + 2 + E] = r[2 * p + 1] & lo_mask;
        w[4 * p + 1 - E] = __builtin_amdgcn_bitop3_b32((uint32_t)x[0], lo_mask, flip, 0x6A);  // (x & mask) ^ flip
        w[4 * p + 3 - E] = __builtin_amdgcn_bitop3_b32((uint32_t)x[1], lo_mask, flip, 0x6A);
    }
    pin(w);
}

// a stage's fragments as read: [32-row half][32-byte half of the 64-byte rows]
struct RawF8 {
    v4i a[2][2];
    v4i b[2][2];
};

template <bool DBG>
__global__ __launch_bounds__(kGemmThreads, 2) void gemm_mixed_f8_kernel(const GemmArgs a) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kMetaOff + kMetaBytes];

    const int t = threadIdx.x;
    const int lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1;  // 0..1: 64-token half of the tile
    const int wn = wave & 1;   // 0..1: 64-channel half of the tile
    int tile_m, tile_n;
    tile_of_block(a, tile_m, tile_n);
    const int64_t m0 = (int64_t)tile_m * kBM;
    const int64_t n0 = (int64_t)tile_n * kBN;
    if (n0 >= a.L.N) return;  // a tile of padding channels only
    const int S_hi = a.stages_hi, S_lo = a.stages_lo, S = S_hi + S_lo;  // both even, S_lo at least 24 (the host's rule)
    const uint16_t* sw_hi = reinterpret_cast<const uint16_t*>(a.packed + a.L.scale_off);
    const uint16_t* sw_lo = sw_hi + a.L.n_pad;
    const int32_t* wsum_hi = reinterpret_cast<const int32_t*>(a.packed + a.L.scale_off + 8 * a.L.n_pad);
    const int32_t* wsum_lo = wsum_hi + a.L.n_pad;
    const bool asym = a.c_hi != nullptr || a.c_lo != nullptr;

    // ---- epilogue constants -> LDS (the oldest loads of their waves) ------------
    if (wave == 0) {
        if (lane < 32) {
            load_to_lds_16B((lane < 16 ? sw_hi : sw_lo) + n0 + (lane & 15) * 8, lds + kMetaOff + kMetaSwHi);
            if (asym) load_to_lds_16B(wsum_hi + n0 + lane * 4, lds + kMetaOff + kMetaWsumHi);
        }
    } else if (wave == 1) {
        if (lane < 32) load_to_lds_16B(wsum_lo + n0 + lane * 4, lds + kMetaOff + kMetaEven);
    } else {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int64_t m = m0 + h * 64 + lane;
            m = m < a.M ? m : a.M - 1;
            if (wave == 2) {
                if (S_hi > 0) load_to_lds_4B(a.s_hi + m, lds + kMetaOff + kMetaSHi + h * 256);
                load_to_lds_4B(a.s_lo + m, lds + kMetaOff + kMetaSLo + h * 256);
            } else {
                load_to_lds_4B(a.lo_sum + m, lds + kMetaOff + kMetaLoSum + h * 256);
                if (asym && S_hi > 0) load_to_lds_4B(a.c_hi + m, lds + kMetaOff + kMetaCHi + h * 256);
                if (asym) load_to_lds_4B(a.c_lo + m, lds + kMetaOff + kMetaCLo + h * 256);
            }
        }
    }

    // ---- global -> LDS copy: wave w copies A blocks 2w, 2w+1 and B blocks 2w, 2w+1 of each stage ----
    uint32_t a_voff_hi[2], a_voff_lo[2], b_voff[2];
    {
        const int r = lane >> 2, kc = (lane & 3) ^ (lane >> 4);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int64_t row = (wave * 2 + h) * 16 + r;
            row = m0 + row < a.M ? row : a.M - 1 - m0;
            a_voff_hi[h] = (uint32_t)(row * a.ld_hi + kc * 16);
            a_voff_lo[h] = (uint32_t)(row * a.ld_lo + kc * 16);
        }
        b_voff[0] = r * kRowBytes + kc * 16;
        b_voff[1] = b_voff[0] + (uint32_t)a.L.group_bytes;
    }
    // the low rows are addressed by the global stage index too: their resource starts S_hi stages early
    const __amdgpu_buffer_rsrc_t rs_a_hi = make_rsrc(a.q_hi + m0 * a.ld_hi);
    const __amdgpu_buffer_rsrc_t rs_a_lo = make_rsrc(a.q_lo + m0 * a.ld_lo - (int64_t)S_hi * kRowBytes);
    const __amdgpu_buffer_rsrc_t rs_b = make_rsrc(a.packed + (n0 / 16 + wave * 2) * a.L.group_bytes);
    auto issue_load = [&](auto k, int sg, int buf) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value;
        uint8_t* dst = lds + buf * kStageBytes;
        if constexpr (K < 2) {
            const bool lo = sg >= S_hi;
            buffer_load_to_lds_16B(lo ? rs_a_lo : rs_a_hi, lo ? a_voff_lo[K] : a_voff_hi[K], (uint32_t)sg * kRowBytes,
                                   dst + (wave * 2 + K) * kBlockBytes);
        } else {
            buffer_load_to_lds_16B(rs_b, b_voff[K - 2], (uint32_t)sg * kBlockBytes,
                                   dst + kStageABytes + (wave * 2 + K - 2) * kBlockBytes);
        }
    };
    auto issue_load_lo = [&](auto k, int sg, int buf) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value;
        uint8_t* dst = lds + buf * kStageBytes;
        if constexpr (K < 2)
            buffer_load_to_lds_16B(rs_a_lo, a_voff_lo[K], (uint32_t)sg * kRowBytes, dst + (wave * 2 + K) * kBlockBytes);
        else
            buffer_load_to_lds_16B(rs_b, b_voff[K - 2], (uint32_t)sg * kBlockBytes,
                                   dst + kStageABytes + (wave * 2 + K - 2) * kBlockBytes);
    };

    // ---- accumulators: [32 j channels][token half i]; lane l holds token l % 32 and, in element
    // 4 q + v, channel 8 q + 4 (l / 32) + v.  Token half i of this wavefront is half i ^ wn of the
    // wave tile, so that i = 0 is the half whose offset codes it adds up. ----
    v16i acc_hi[2][2];
    v16f acc_lo[2][2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                acc_hi[j][i][v] = 0;
                acc_lo[j][i][v] = 0.0f;
            }
    auto park_hi = [&]() __attribute__((always_inline)) {
        asm volatile("" : "+a"(acc_hi[0][0]), "+a"(acc_hi[0][1]), "+a"(acc_hi[1][0]), "+a"(acc_hi[1][1]));
    };
    auto park_lo = [&]() __attribute__((always_inline)) {
        asm volatile("" : "+a"(acc_lo[0][0]), "+a"(acc_lo[0][1]), "+a"(acc_lo[1][0]), "+a"(acc_lo[1][1]));
    };

    // ---- LDS -> register reads: fragment (rows, h): lane l supplies row l % 32, 16-byte piece 2 h + l / 32 ----
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
    uint32_t a_off[2][2], b_off[2];
    {
        const int r = lane & 15;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kc = 2 * h + (lane >> 5);
            const uint32_t off = lds0 + ((lane >> 4) & 1) * kBlockBytes + (4 * r + (kc ^ (r >> 2))) * 16;
#pragma unroll
            for (int i = 0; i < 2; ++i) a_off[i][h] = off + wm * (4 * kBlockBytes) + (i ^ wn) * (2 * kBlockBytes);
            b_off[h] = off + kStageABytes + wn * (4 * kBlockBytes);
        }
    }
    // fragment K of a stage in the order in which they are widened: (b0, a0, a1, b1) of h = 0, then of h = 1
    auto read_to = [&](auto k, v4i& dst, uint32_t shift) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value, H = K >> 2, Q = K & 3;
        if constexpr (Q == 0) lds_read16<0>(dst, b_off[H] + shift);
        else if constexpr (Q == 3) lds_read16<2 * kBlockBytes>(dst, b_off[H] + shift);
        else lds_read16<0>(dst, a_off[Q - 1][H] + shift);
    };
    // the same with the buffer in the instruction's offset
    auto read_from = [&](auto k, v4i& dst, auto buf_) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value, H = K >> 2, Q = K & 3, B = decltype(buf_)::value * kStageBytes;
        if constexpr (Q == 0) lds_read16<B>(dst, b_off[H]);
        else if constexpr (Q == 3) lds_read16<B + 2 * kBlockBytes>(dst, b_off[H]);
        else lds_read16<B>(dst, a_off[Q - 1][H]);
    };
    auto frag_of = [&](auto k, RawF8& f) __attribute__((always_inline)) -> v4i& {
        constexpr int K = decltype(k)::value, H = K >> 2, Q = K & 3;
        if constexpr (Q == 0) return f.b[0][H];
        else if constexpr (Q == 3) return f.b[1][H];
        else return f.a[Q - 1][H];
    };

    const int tl = wm * 64 + (lane & 31);         // + 32 (i ^ wn)
    const int cl = wn * 64 + (lane >> 5) * 4;     // + 32 j + 8 q + v
    auto fold = [&](auto has_hi, auto is_asym, auto is_glu) __attribute__((always_inline)) {
        constexpr bool HI_ON = decltype(has_hi)::value, ASYM = decltype(is_asym)::value, GLU = decltype(is_glu)::value;
        const uint8_t* meta = lds + kMetaOff;
        float st_hi[2], st_lo[2], ct_hi[2], ct_lo[2], ca[2];
        int row[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            st_hi[i] = st_lo[i] = ct_hi[i] = ct_lo[i] = ca[i] = 0.f;
            row[i] = tl + 32 * (i ^ wn);
            if constexpr (HI_ON) st_hi[i] = *reinterpret_cast<const float*>(meta + kMetaSHi + row[i] * 4);
            if constexpr (ASYM && HI_ON) ct_hi[i] = *reinterpret_cast<const float*>(meta + kMetaCHi + row[i] * 4);
            if constexpr (ASYM) ct_lo[i] = *reinterpret_cast<const float*>(meta + kMetaCLo + row[i] * 4);
            st_lo[i] = *reinterpret_cast<const float*>(meta + kMetaSLo + row[i] * 4);
            ca[i] = (float)(8 * (*reinterpret_cast<const int*>(meta + kMetaLoSum + row[i] * 4) +
                                 *reinterpret_cast<const int*>(meta + kMetaSe + row[i] * 4)) + 32 * (int)a.L.kl_pad);
        }
        int32_t* dbg_row_hi[2] = {nullptr, nullptr};
        int32_t* dbg_row_lo[2] = {nullptr, nullptr};
        bool dbg_ok[2] = {false, false};
        int dbg_cols = 0;
        if constexpr (DBG) {
            dbg_cols = (int)(a.L.N - n0 - cl);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int64_t m = m0 + row[i];
                dbg_ok[i] = m < a.M;
                dbg_row_hi[i] = a.dbg_hi + m * a.L.N + n0 + cl;
                dbg_row_lo[i] = a.dbg_lo + m * a.L.N + n0 + cl;
            }
        }
#pragma unroll
        for (int jq = 0; jq < 8; ++jq) {
            const int j = jq >> 2, q = jq & 3, cc = 32 * j + 8 * q, c = cl + cc;
            float sn_hi[4] = {0.f, 0.f, 0.f, 0.f}, sn_lo[4] = {0.f, 0.f, 0.f, 0.f};
            float zw_hi[4] = {0.f, 0.f, 0.f, 0.f}, zw_lo[4] = {0.f, 0.f, 0.f, 0.f};  // wsum[n] * sw[n]
            float ev[4] = {0.f, 0.f, 0.f, 0.f};
            if constexpr (HI_ON) {
                const v4h h = *reinterpret_cast<const v4h*>(meta + kMetaSwHi + c * 2);
#pragma unroll
                for (int v = 0; v < 4; ++v) sn_hi[v] = (float)h[v];
                if constexpr (ASYM) {
                    const v4i ws = *reinterpret_cast<const v4i*>(meta + kMetaWsumHi + c * 4);
#pragma unroll
                    for (int v = 0; v < 4; ++v) zw_hi[v] = (float)ws[v] * sn_hi[v];
                }
            }
            {
                const v4h h = *reinterpret_cast<const v4h*>(meta + kMetaSwLo + c * 2);
                const v4i ws = *reinterpret_cast<const v4i*>(meta + kMetaEven + c * 4);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    sn_lo[v] = (float)h[v];
                    ev[v] = (float)(8 * ws[v]);
                    if constexpr (ASYM) zw_lo[v] = (float)ws[v] * sn_lo[v];
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float val[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    val[v] = 0.f;
                    if constexpr (HI_ON) {
                        const int ih = from_acc(acc_hi[j][i][4 * q + v]);
                        val[v] = (float)ih * (st_hi[i] * sn_hi[v]);
                        if constexpr (ASYM) val[v] += ct_hi[i] * zw_hi[v];
                        if constexpr (DBG) {
                            if (a.dbg_hi && dbg_ok[i] && cc + v < dbg_cols) dbg_row_hi[i][cc + v] = ih;
                        }
                    }
                    // whole numbers below 2^24 throughout: exact
                    const float fl = __builtin_fmaf(__int_as_float(from_acc(__float_as_int(acc_lo[j][i][4 * q + v]))), kF8Unit, -(ev[v] + ca[i]));
                    val[v] += fl * (st_lo[i] * sn_lo[v]);
                    if constexpr (ASYM) val[v] += ct_lo[i] * zw_lo[v];
                    if constexpr (DBG) {
                        if (a.dbg_lo && dbg_ok[i] && cc + v < dbg_cols) dbg_row_lo[i][cc + v] = (int)fl;
                    }
                }
                if constexpr (GLU)
                    *reinterpret_cast<uint32_t*>(lds + row[i] * kOutRowBytes + c) =
                        pack_bf16(silu_f32(val[0]) * val[1], silu_f32(val[2]) * val[3]);
                else
                    *reinterpret_cast<uint2*>(lds + row[i] * kOutRowBytes + c * 2) =
                        make_uint2(pack_bf16(val[0], val[1]), pack_bf16(val[2], val[3]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- main loop ---------------------------------------------------------------
    {
        RawF8 p0, p1;                 // high stages: the one being multiplied and the next
        v4i raw[8];                   // low stages: fragments on their way, in widening order
        v8i wa[2][2], wb[2][2];       // low stages: widened, [half][h]
        uint32_t sum = 0, bytes = 0;  // offset codes of the even columns, token half 0: total, and four partial sums in bytes
        int lo_mask = 0x0F0F0F0F, flip = 0x08080808;
        asm volatile("" : "+s"(lo_mask), "+v"(flip));
        const int first = S_hi & 2;
        const int ahead = S < kPrefetch ? S : kPrefetch;
        for (int i = 0; i < ahead; ++i)
            static_for<kLoadsPerStage>([&](auto k) __attribute__((always_inline)) { issue_load(k, i, (i + first) & (kNumBuf - 1)); });
        wait_stage_and_barrier(ahead - 1);  // stage 0 (and the epilogue constants) have landed everywhere
        static_for<8>([&](auto k) __attribute__((always_inline)) { read_to(k, frag_of(k, p0), (uint32_t)first * kStageBytes); });

        using YES = std::true_type;
        using NO = std::false_type;

        auto widen_k = [&](auto k, const v4i& r) __attribute__((always_inline)) {
            constexpr int K = decltype(k)::value, H = K >> 2, Q = K & 3;
            if constexpr (Q == 0) widen_f8<true>(wb[0][H], r, lo_mask, flip);
            else if constexpr (Q == 3) widen_f8<true>(wb[1][H], r, lo_mask, flip);
            else widen_f8<false>(wa[Q - 1][H], r, lo_mask, flip);
            if constexpr (Q == 1) {
                bytes += (uint32_t)wa[0][H][0] + (uint32_t)wa[0][H][2];
                bytes += (uint32_t)wa[0][H][4] + (uint32_t)wa[0][H][6];
            }
        };

        // stage sg lives in buffer (sg + first) % 4, so that the first low stage has buffer 0
        int buf = first;
        auto stage_lo = [&](auto steady, auto buf_, int sg) __attribute__((always_inline)) {
            constexpr bool STEADY = decltype(steady)::value;
            // steady stages know their buffer at compile time, the last ones have it in buf
            const int b0 = STEADY ? (int)decltype(buf_)::value : buf;
            const int nbuf = b0 == kNumBuf - 1 ? 0 : b0 + 1, prv = b0 == 0 ? kNumBuf - 1 : b0 - 1;
            constexpr int BUF = decltype(buf_)::value, NBUF = (BUF + 1) % kNumBuf;
            auto read = [&](auto k, bool next) __attribute__((always_inline)) {
                v4i& dst = raw[decltype(k)::value];
                if constexpr (STEADY) {
                    if constexpr (decltype(k)::value >= 6) read_from(k, dst, IC<BUF>{});
                    else read_from(k, dst, IC<NBUF>{});
                } else {
                    read_to(k, dst, (uint32_t)(next ? nbuf : b0) * kStageBytes);
                }
            };
            const bool issue = STEADY || sg + kPrefetch < S;
            park_hi();
            static_for<8>([&](auto g_) __attribute__((always_inline)) {
                constexpr int G = decltype(g_)::value, H = G >> 2, Q = G & 3, J = Q >> 1, I = (Q == 1 || Q == 2) ? 1 : 0;
                __builtin_amdgcn_sched_barrier(0);
                mfma_32x32x64_f8(acc_lo[J][I], wb[J][H], wa[I][H]);
                if constexpr (G == 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (STEADY) {
                        wait_loads_and_barrier<(kPrefetch - 2) * kLoadsPerStage>();
                    } else {
                        const int rem = S - 2 - sg;
                        wait_stage_and_barrier(rem > kPrefetch - 2 ? kPrefetch - 2 : rem);
                    }
                }
                if constexpr (G == 0) {
                    read(IC<6>{}, false);
                    read(IC<7>{}, false);
                } else if constexpr (G < 7) {
                    read(IC<G - 1>{}, true);
                }
                if constexpr (G >= 2 && G < 6) { if (issue) issue_load_lo(IC<G - 2>{}, sg + kPrefetch, prv); }
                __builtin_amdgcn_sched_barrier(0);
                // widened here: this stage's h = 1 up to G = 3, then the next stage's h = 0
                constexpr int K = (G + 4) & 7;
                if constexpr (G >= 2 && G < 7) lds_wait<3>(raw[K]);
                if constexpr (G == 7) lds_wait<2>(raw[K]);
                widen_k(IC<K>{}, raw[K]);
            });
            // nothing is in flight from here to the next stage, where the compiler may move registers
            lds_wait<0>(raw[4]);
            lds_wait<0>(raw[5]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!STEADY) buf = nbuf;
        };
        auto stage_hi = [&](auto steady, RawF8& cur, RawF8& nx, int sg) __attribute__((always_inline)) {
            constexpr bool STEADY = decltype(steady)::value;
            const int nbuf = buf == kNumBuf - 1 ? 0 : buf + 1;
            const int prv = buf == 0 ? kNumBuf - 1 : buf - 1;
            const uint32_t shift = nbuf * kStageBytes;
            const bool issue = STEADY || sg + kPrefetch < S;
            park_lo();
            __builtin_amdgcn_sched_barrier(0);
            static_for<8>([&](auto k) __attribute__((always_inline)) { lds_wait<0>(frag_of(k, cur)); });
            static_for<8>([&](auto g_) __attribute__((always_inline)) {
                constexpr int G = decltype(g_)::value, H = G >> 2, Q = G & 3, J = Q >> 1, I = (Q == 1 || Q == 2) ? 1 : 0;
                __builtin_amdgcn_sched_barrier(0);
                mfma_32x32x32_i8(acc_hi[J][I], cur.b[J][H], cur.a[I][H]);
                if constexpr (G == 1) {
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (STEADY) {
                        wait_loads_and_barrier<(kPrefetch - 2) * kLoadsPerStage>();
                    } else {
                        const int rem = S - 2 - sg;
                        wait_stage_and_barrier(rem > kPrefetch - 2 ? kPrefetch - 2 : rem);
                    }
                }
                if constexpr (G >= 2 && G < 6) {
                    read_to(IC<2 * G - 4>{}, frag_of(IC<2 * G - 4>{}, nx), shift);
                    read_to(IC<2 * G - 3>{}, frag_of(IC<2 * G - 3>{}, nx), shift);
                }
                if constexpr (G >= 6) {
                    if (issue) {
                        issue_load(IC<2 * G - 12>{}, sg + kPrefetch, prv);
                        issue_load(IC<2 * G - 11>{}, sg + kPrefetch, prv);
                    }
                }
            });
            __builtin_amdgcn_sched_barrier(0);
            buf = nbuf;
        };
        int sg = 0;
        for (; sg < S_hi && sg + 1 + kPrefetch < S; sg += 2) {
            stage_hi(YES{}, p0, p1, sg);
            stage_hi(YES{}, p1, p0, sg + 1);
        }
        for (; sg < S_hi; sg += 2) {
            stage_hi(NO{}, p0, p1, sg);
            stage_hi(NO{}, p1, p0, sg + 1);
        }
        static_for<8>([&](auto k) __attribute__((always_inline)) { lds_wait<0>(frag_of(k, p0)); });
        // p0 holds the first low stage, as read
        static_for<4>([&](auto k) __attribute__((always_inline)) { widen_k(k, frag_of(k, p0)); });
        raw[4] = frag_of(IC<4>{}, p0);
        raw[5] = frag_of(IC<5>{}, p0);
        sum = __builtin_amdgcn_sad_u8(bytes, 0u, sum);
        bytes = 0;
        asm volatile("s_nop 4" ::: "memory");  // wait states between the widening and the first product
        auto pair = [&](auto steady, auto buf_) __attribute__((always_inline)) {
            stage_lo(steady, buf_, sg);
            stage_lo(steady, IC<decltype(buf_)::value + 1>{}, sg + 1);
            sum = __builtin_amdgcn_sad_u8(bytes, 0u, sum);  // two stages: 16 codes of 0..15 in each byte
            bytes = 0;
            sg += 2;
        };
        // the buffers are in the instructions, so that a read costs no address: four stages a turn
        while (sg + 3 + kPrefetch < S) {
            pair(YES{}, IC<0>{});
            pair(YES{}, IC<2>{});
        }
        buf = 0;
        while (sg < S) pair(NO{}, IC<0>{});
        // the last stage widened what lies behind it: its h = 0 does not count
        bytes = (uint32_t)wa[0][0][0] + (uint32_t)wa[0][0][2] + (uint32_t)wa[0][0][4] + (uint32_t)wa[0][0][6];
        sum -= __builtin_amdgcn_sad_u8(bytes, 0u, 0u);
        sum += __shfl_xor(sum, 32);
        if (lane < 32) *reinterpret_cast<uint32_t*>(lds + kMetaOff + kMetaSe + (wm * 64 + wn * 32 + lane) * 4) = sum;
        wait_loads_and_barrier<0>();
        __syncthreads();  // every wave is done reading the stage buffers, and the sums are there
        wait_for_products();
        if (a.swiglu) {  // symmetric codes only (checked on the host)
            if (S_hi > 0) fold(YES{}, NO{}, YES{});
            else fold(NO{}, NO{}, YES{});
        } else if (asym) {
            if (S_hi > 0) fold(YES{}, YES{}, NO{});
            else fold(NO{}, YES{}, NO{});
        } else {
            if (S_hi > 0) fold(YES{}, NO{}, NO{});
            else fold(NO{}, NO{}, NO{});
        }
    }
    __syncthreads();
    store_tile(a, lds, wave, lane, m0, n0);
}

}  // namespace resq
