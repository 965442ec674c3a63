// Rows of bf16 data expressed in an fp32 basis (Section 4.2 and 4.3: X U, W U):
//   out[i][j] = sum_t a[i][t] u[t][j],   a bf16, u fp32, out bf16 or fp32, more than 16 steps t (fewer: the fp32 kernel).
//
// The fp32 matrix instruction (157 TFLOP/s) bounds this product at 0.87 ms for a
// 4096^3 fold; it took 1.19 ms there (115 TFLOP/s).  The bf16 matrix cores are
// sixteen times as fast, and u can go through them without losing a bit: an fp32
// number is the exact sum of three bf16 numbers (8 + 8 + 8 significant bits, each
// the truncated rest of the one before), every product with a bf16 a is exact in
// fp32, and the accumulator is fp32 as before.  Three products instead of one, at
// sixteen times the rate: 0.40 ms for the same fold (1030 TFLOP/s of bf16 products, matrix
// pipes busy 52 % of the clocks at 1.7 GHz: the power limit; 0.41 to 0.46 behind other work).
// Error against 64 bits with fp32 output (2-norm, before / now): 1.2e-6 / 7.0e-7 at
// K = 4096, 4.0e-7 / 2.4e-7 at 512, 2.0e-7 / 1.2e-7 at 128: the sum has fewer roundings
// (one per 16 products of the instruction instead of one per 2).
//
// Workgroup: 4 wavefronts, 128 x 128 outputs, 64 x 64 each as 2 x 2 tiles of
// v_mfma_f32_32x32x16_bf16; the reduction in chunks of 32 through two LDS buffers, one
// barrier per chunk, two workgroups to a compute unit.  A chunk's fragments are read
// at once; behind each product five vector instructions of the next chunk's split run
// (with the split after the products instead: 1000 x 1003 x 904 46 / 36 us, 256 x 512 x 512
// 25 / 21, 4096^3 at the power limit either way).  The B operand wants eight consecutive
// t of one column per lane: a thread reads them as eight rows of u (lanes along j, 256
// contiguous bytes a wavefront), splits them and writes three 16-byte units, so
// the transposition costs nothing.  LDS units of 16 bytes, column-major over the
// pieces: reads and writes run along consecutive rows or columns.
//
// The split is exact for |u| >= 2^-110; below that the part of u under 2^-133, the smallest
// bf16 subnormal, is dropped.  An infinity or NaN in a or u makes sums that it enters NaN, also
// where the plain sum is an infinity (infinity x 0 and infinity - infinity among the parts): sums
// that come out NaN are taken again in fp32, term by term.  (Looking for them costs 0.1 to 0.25 us a call:
// 128 x 128 x 128 8.15 / 8.39, 256 x 512 x 512 16.8 / 16.9.)
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
    __shared__ int redo;   // a sum of this workgroup is not finite
    const int t = threadIdx.x, lane = t & 63;
    if (t == 0) redo = 0;
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
    // a chunk on its way from memory to LDS
    struct Chunk {
        uint4 a[2];
        float u[2][8];
    };
    // the chunk of steps tc .. tc + 31, all of them there
    auto fetch = [&](Chunk& c, int64_t tc) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            c.a[h] = *reinterpret_cast<const uint4*>(a_base + a_row[h] * g.lda + tc);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float* row = g.u + (tc + (bp + 2 * h) * 8) * g.ldu + j0;   // wave-uniform
#pragma unroll
            for (int e = 0; e < 8; ++e) c.u[h][e] = row[e * g.ldu + u_col];
        }
    };
    // the last chunk of a ragged reduction axis: what lies behind it in a row of a is not ours
    auto fetch_tail = [&](Chunk& c, int64_t tc) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t tt = tc + ap * 8;
            const uint16_t* src = a_base + a_row[h] * g.lda + tc;
            uint32_t w[4] = {0, 0, 0, 0};
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tt + e < g.T) w[e >> 1] |= (uint32_t)src[e] << (16 * (e & 1));
            c.a[h] = make_uint4(w[0], w[1], w[2], w[3]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t tt = tc + (bp + 2 * h) * 8;
            const float* row = g.u + tt * g.ldu + j0;
#pragma unroll
            for (int e = 0; e < 8; ++e) c.u[h][e] = tt + e < g.T ? row[e * g.ldu + u_col] : 0.0f;
        }
    };
    auto fetch_any = [&](Chunk& c, int64_t tc) __attribute__((always_inline)) {
        if (tc + kProjChunk <= g.T) fetch(c, tc);
        else if (tc < g.T) fetch_tail(c, tc);
    };
    auto stash = [&](const Chunk& c, int buf) __attribute__((always_inline)) {
        uint8_t* base = lds + buf * kProjBytes;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            *reinterpret_cast<uint4*>(base + ap * kProjPieceA + (ar + 64 * h) * 16) = c.a[h];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t part[3][4];
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
                uint32_t x[2], y[2], z[2];
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    const float v = c.u[h][e + k];
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
    constexpr int kSteps = kProjChunk / 16;
    struct Frags {
        v8bf a[kSteps][2], b[kSteps][3][2];
    };
    auto read_frags = [&](Frags& f, int buf) __attribute__((always_inline)) {
        const uint8_t* base = lds + buf * kProjBytes;
#pragma unroll
        for (int s = 0; s < kSteps; ++s) {
            const int piece = 2 * s + oh;
#pragma unroll
            for (int p = 0; p < 2; ++p)
                f.a[s][p] = *reinterpret_cast<const v8bf*>(base + piece * kProjPieceA + (wi * 64 + p * 32 + ol) * 16);
#pragma unroll
            for (int part = 2; part >= 0; --part)
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    f.b[s][part][q] = *reinterpret_cast<const v8bf*>(base + kProjBytesA + part * kProjSplitB +
                                                                     piece * kProjPieceB + (wj * 64 + q * 32 + ol) * 16);
        }
    };
    // the smallest parts first
    auto multiply = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < kSteps; ++s)
#pragma unroll
            for (int part = 2; part >= 0; --part)
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
                        acc[p][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[s][p], f.b[s][part][q], acc[p][q], 0, 0, 0);
    };

    // Chunk i is multiplied out of buffer i % 2 while chunk i + 1, in registers since the step before, is
    // split and written into the other one, a few instructions behind each product, and chunk
    // i + 2 is on its way from memory.
    Chunk c0, c1;
    fetch_any(c0, 0);
    stash(c0, 0);
    fetch_any(c0, kProjChunk);
    __syncthreads();
    auto step = [&](Chunk& here, Chunk& next, int64_t tc, int buf) __attribute__((always_inline)) {
        fetch(next, tc + 2 * kProjChunk);
        Frags f;
        read_frags(f, buf);
        __builtin_amdgcn_sched_barrier(0);
        multiply(f);
        stash(here, buf ^ 1);
#pragma unroll
        for (int k = 0; k < 24; ++k) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // a product
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);   // vector instructions
            if (k % 3 == 2) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // an LDS write
        }
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
    };
    int64_t tc = 0;
    for (; tc + 4 * kProjChunk <= g.T; tc += 2 * kProjChunk) {
        step(c0, c1, tc, 0);
        step(c1, c0, tc + kProjChunk, 1);
    }
    for (int buf = 0; tc < g.T; tc += kProjChunk, buf ^= 1) {   // up to four chunks are left, the last one perhaps ragged
        fetch_any(c1, tc + 2 * kProjChunk);
        Frags f;
        read_frags(f, buf);
        multiply(f);
        if (tc + kProjChunk < g.T) {
            stash(c0, buf ^ 1);
            __syncthreads();
        }
        c0 = c1;
    }

    // any sum that is not finite (0 x it is NaN) sends the whole workgroup to the second way out
    float probe[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};   // eight short chains instead of a long one
#pragma unroll
    for (int e = 0; e < 64; ++e) probe[e & 7] = fmaf(acc[e >> 5][(e >> 4) & 1][e & 15], 0.0f, probe[e & 7]);
    const float sum = ((probe[0] + probe[1]) + (probe[2] + probe[3])) + ((probe[4] + probe[5]) + (probe[6] + probe[7]));
    if (sum != sum) redo = 1;
    __syncthreads();

    // acc[p][q][v]: row 8 (v / 4) + 4 (lane / 32) + v % 4, column lane % 32 of matrix tile (p, q)
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(redo) == 0, 1)) {
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
        return;
    }
    // number e = 32 p + 16 q + v of the lane's 64 sums at 256 e: one column of LDS per thread
    float* sums = reinterpret_cast<float*>(lds) + t;
    static_assert(64 * kProjThreads * sizeof(float) <= sizeof(lds), "a place for every sum");
#pragma unroll
    for (int e = 0; e < 64; ++e) sums[e * kProjThreads] = acc[e >> 5][(e >> 4) & 1][e & 15];
    for (int store = 0; store < 2; ++store) {
#pragma unroll 1
        for (int e = 0; e < 64; ++e) {
            const int64_t i = i0 + wi * 64 + (e >> 5) * 32 + 8 * ((e >> 2) & 3) + 4 * oh + (e & 3);
            const int64_t j = j0 + wj * 64 + ((e >> 4) & 1) * 32 + ol;
            if (i >= g.I || j >= g.J) continue;
            float s = sums[e * kProjThreads];
            if (store) {
                if constexpr (OUT_BF16) static_cast<uint16_t*>(g.out)[i * g.ldo + j] = (uint16_t)pack_bf16(s, 0.0f);
                else static_cast<float*>(g.out)[i * g.ldo + j] = s;
            } else if (s != s) {
                const uint16_t* row = g.a + i * g.lda;
                s = 0.0f;
                for (int64_t k = 0; k < g.T && s == s; ++k) s = fmaf(__uint_as_float((uint32_t)row[k] << 16), g.u[k * g.ldu + j], s);
                sums[e * kProjThreads] = s;
            }
        }
        __syncthreads();   // out may lie on a (one column of tiles): all is read before anything is written
    }
}

}  // namespace resq
