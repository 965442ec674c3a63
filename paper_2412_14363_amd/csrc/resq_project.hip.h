// Rows of bf16 data expressed in an fp32 basis (Section 4.2 and 4.3: X U, W U):
//   out[i][j] = sum_t a[i][t] u[t][j],   a bf16, u fp32, out bf16 or fp32.
//
// The fp32 matrix instruction (157 TFLOP/s) bounds this product at 0.87 ms for a
// 4096^3 fold; it took 1.19 ms there (115 TFLOP/s).  The bf16 matrix cores are
// sixteen times as fast, and u can go through them without losing a bit: an fp32
// number is the exact sum of three bf16 numbers (8 + 8 + 8 significant bits, each
// the truncated rest of the one before), every product with a bf16 a is exact in
// fp32, and the accumulator is fp32 as before.  Three products instead of one, at
// sixteen times the rate: 0.46 ms for the same fold (900 TFLOP/s of bf16 products).
// Error against 64 bits with fp32 output (2-norm, before / now): 1.2e-6 / 7.0e-7 at
// K = 4096, 4.0e-7 / 2.4e-7 at 512, 2.0e-7 / 1.2e-7 at 128: the sum has fewer roundings
// (one per 16 products of the instruction instead of one per 2).
//
// Workgroup: 4 wavefronts, 128 x 128 outputs, 64 x 64 each as 2 x 2 tiles of
// v_mfma_f32_32x32x16_bf16; the reduction in chunks of 32 through two LDS buffers,
// the next chunk travelling through registers while this one is multiplied, one
// barrier per chunk; two workgroups share a compute unit, so that one splits and
// stores while the other multiplies.  The B operand wants eight consecutive t of
// one column per lane: a thread reads them as eight rows of u (lanes along j, 256
// contiguous bytes a wavefront), splits them and writes three 16-byte units, so
// the transposition costs nothing.  LDS units of 16 bytes, column-major over the
// pieces: reads and writes run along consecutive rows or columns.
//
// Inputs are finite, as everywhere in this library; an infinity in u or a makes the
// outputs that it enters NaN (the rests of the split are inf - inf and 0).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "resq_gemm.hip.h"

namespace resq {

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kProjThreads = 256;
constexpr int kProjTile = 128;
constexpr int kProjChunk = 32;                           // reduction steps per LDS buffer
constexpr int kProjPieces = kProjChunk / 8;              // 16-byte units along the reduction
constexpr int kProjPieceA = kProjTile * 16 + 32;         // bytes; padded: a wavefront writes 4 pieces of 16 rows at once
constexpr int kProjPieceB = kProjTile * 16;
constexpr int kProjBytesA = kProjPieces * kProjPieceA;
constexpr int kProjSplitB = kProjPieces * kProjPieceB;   // one of the three parts of u
constexpr int kProjBytes = kProjBytesA + 3 * kProjSplitB;

struct ProjectArgs {
    const uint16_t* a;
    const float* u;
    void* out;
    int64_t lda, ldu, ldo;
    int64_t I, J, T;
};

template <bool OUT_BF16>
__global__ __launch_bounds__(kProjThreads, 2) void project_split_kernel(const ProjectArgs g) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kProjBytes];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wi = wave >> 1, wj = wave & 1;
    const int64_t i0 = (int64_t)blockIdx.y * kProjTile, j0 = (int64_t)blockIdx.x * kProjTile;

    // a: thread (rows t / 4 and t / 4 + 64, piece t % 4); u: thread (column t % 128, pieces w and w + 2 for
    // wavefronts 2 w, 2 w + 1).  Rows past I and columns past J repeat the last one (their outputs are not stored).
    const int ar = t >> 2, ap = t & 3;
    const int bj = t & 127, bp = wave >> 1;
    uint32_t a_row[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t i = i0 + ar + 64 * h;
        a_row[h] = (uint32_t)((i < g.I ? i : g.I - 1) - i0);
    }
    const uint32_t u_col = (uint32_t)((j0 + bj < g.J ? j0 + bj : g.J - 1) - j0);
    const uint16_t* a_base = g.a + i0 * g.lda + ap * 8;
    uint4 ra[2];
    float rb[2][8];
    // the chunk of steps tc .. tc + 31, all of them there
    auto fetch = [&](int64_t tc) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            ra[h] = *reinterpret_cast<const uint4*>(a_base + a_row[h] * g.lda + tc);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float* row = g.u + (tc + (bp + 2 * h) * 8) * g.ldu + j0;   // wave-uniform
#pragma unroll
            for (int e = 0; e < 8; ++e) rb[h][e] = row[e * g.ldu + u_col];
        }
    };
    // the last chunk of a ragged reduction axis: what lies behind it in a row of a is not ours
    auto fetch_tail = [&](int64_t tc) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t tt = tc + ap * 8;
            const uint16_t* src = a_base + a_row[h] * g.lda + tc;
            uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tt + e < g.T) w[e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
            ra[h] = make_uint4(w[0], w[1], w[2], w[3]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t tt = tc + (bp + 2 * h) * 8;
            const float* row = g.u + tt * g.ldu + j0;
#pragma unroll
            for (int e = 0; e < 8; ++e) rb[h][e] = tt + e < g.T ? row[e * g.ldu + u_col] : 0.0f;
        }
    };
    auto fetch_any = [&](int64_t tc) __attribute__((always_inline)) {
        if (tc + kProjChunk <= g.T) fetch(tc);
        else fetch_tail(tc);
    };
    auto stash = [&](int buf) __attribute__((always_inline)) {
        uint8_t* base = lds + buf * kProjBytes;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            *reinterpret_cast<uint4*>(base + ap * kProjPieceA + (ar + 64 * h) * 16) = ra[h];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t part[3][4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                uint32_t x[2], y[2], z[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const float v = rb[h][e + k];
                    x[k] = __float_as_uint(v);
                    const float r1 = v - __uint_as_float(x[k] & 0xFFFF0000u);   // exact
                    y[k] = __float_as_uint(r1);
                    z[k] = __float_as_uint(r1 - __uint_as_float(y[k] & 0xFFFF0000u));  // exact, at most 8 bits left
                }
                // upper halves of two numbers into one register
                part[0][e >> 1] = __builtin_amdgcn_perm(x[1], x[0], 0x07060302);
                part[1][e >> 1] = __builtin_amdgcn_perm(y[1], y[0], 0x07060302);
                part[2][e >> 1] = __builtin_amdgcn_perm(z[1], z[0], 0x07060302);
            }
#pragma unroll
            for (int s = 0; s < 3; ++s)
                *reinterpret_cast<uint4*>(base + kProjBytesA + s * kProjSplitB + (bp + 2 * h) * kProjPieceB + bj * 16) =
                    make_uint4(part[s][0], part[s][1], part[s][2], part[s][3]);
        }
    };

    v16f acc[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[p][q][v] = 0.0f;

    const int ol = lane & 31, oh = lane >> 5;
    fetch_any(0);
    stash(0);
    __syncthreads();
    int buf = 0;
    for (int64_t tc = 0; tc < g.T; tc += kProjChunk) {
        const bool more = tc + kProjChunk < g.T;
        if (more) fetch_any(tc + kProjChunk);
        const uint8_t* base = lds + buf * kProjBytes;
#pragma unroll
        for (int s = 0; s < kProjChunk / 16; ++s) {
            const int piece = 2 * s + oh;
            v8bf fa[2];
#pragma unroll
            for (int p = 0; p < 2; ++p)
                fa[p] = *reinterpret_cast<const v8bf*>(base + piece * kProjPieceA + (wi * 64 + p * 32 + ol) * 16);
            // the smallest parts first
#pragma unroll
            for (int part = 2; part >= 0; --part)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const v8bf fb = *reinterpret_cast<const v8bf*>(base + kProjBytesA + part * kProjSplitB +
                                                                   piece * kProjPieceB + (wj * 64 + q * 32 + ol) * 16);
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[p], fb, acc[p][q], 0, 0, 0);
                }
        }
        if (more) stash(buf ^ 1);  // last read in the previous iteration, before its barrier
        __syncthreads();
        buf ^= 1;
    }

    // acc[p][q][v]: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32 of matrix tile (p, q)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t j = j0 + wj * 64 + q * 32 + ol;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int64_t i = i0 + wi * 64 + p * 32 + 8 * (v >> 2) + 4 * oh + (v & 3);
                if (i < g.I && j < g.J) {
                    if constexpr (OUT_BF16) static_cast<uint16_t*>(g.out)[i * g.ldo + j] = (uint16_t)pack_bf16(acc[p][q][v], 0.0f);
                    else static_cast<float*>(g.out)[i * g.ldo + j] = acc[p][q][v];
                }
            }
        }
    }
}

}  // namespace resq
