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
typedef float v4f __attribute__((ext_vector_type(4)));

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

// eight consecutive t of one column of u, split into their three parts, one unit of LDS each
__device__ __forceinline__ void stash_split(uint8_t* unit, const float (&u)[8]) {
    uint32_t part[3][4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        uint32_t x[2], y[2], z[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float v = u[e + k];
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
        *reinterpret_cast<uint4*>(unit + s * kProjSplitB) = make_uint4(part[s][0], part[s][1], part[s][2], part[s][3]);
}

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
            stash_split(base + kProjBytesA + (bp + 2 * h) * kProjPieceB + bj * 16, c.u[h]);
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

// ---- 256 x 128 outputs ----------------------------------------------------------------------------
//
// The same product where there are enough such tiles to fill the chip.  In the kernel above LDS is as busy as
// the matrix pipes: a wavefront reads 16 KiB (one operand, three parts of the other) for 64 x 64 outputs of a chunk, and
// every 128 rows split u again.  Here a wavefront owns 128 x 64 outputs (128 accumulation registers), which takes 20 KiB
// for twice the products, and u is split once for 256 rows.  The instruction is v_mfma_f32_16x16x32_bf16, which alone
// sustains 1980 TFLOP/s under the power limit where the 32x32x16 one sustains 1755 (random operands, milliseconds).  One
// chunk is in registers on its way: it is split behind the products of the smallest parts and written, and the chunk after it is
// asked for behind those of the middle ones.  4096 x 4096 x 4096 390 -> 313 us (1317 TFLOP/s of bf16 products), error against 64
// bits with fp32 output 7.02e-7 -> 7.01e-7, at K = 256 1.65e-7 -> 1.60e-7 (one rounding per 32 products instead of 16).
constexpr int kProjWideRows = 256;
constexpr int kProjWidePieceA = kProjWideRows * 16;
constexpr int kProjWideBytesA = kProjPieces * kProjWidePieceA;
constexpr int kProjWideBytes = kProjWideBytesA + 3 * kProjSplitB;
static_assert(2 * 2 * kProjWideBytes <= 160 * 1024, "LDS of two resident workgroups");

// acc += b a on the bf16 matrix cores, in place in accumulation registers
__device__ __forceinline__ void mfma_16x16x32_bf16(v4f& acc, const v8bf& b, const v8bf& a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

template <bool OUT_BF16>
__global__ __launch_bounds__(kProjThreads, 2) void project_split_wide_kernel(const ProjectArgs g) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[2 * kProjWideBytes];
    const int t = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wi = wave >> 1, wj = wave & 1;
    const int64_t i0 = (int64_t)blockIdx.y * kProjWideRows, j0 = (int64_t)blockIdx.x * kProjTile;

    // a: thread (rows t / 4 + 64 h, piece t % 4); u as above
    const int ar = t >> 2, ap = t & 3;
    const int bj = t & 127, bp = wave >> 1;
    uint32_t a_off[4];   // bytes from the tile's first row (the launch sees to it that they fit)
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int64_t i = i0 + ar + 64 * h;
        a_off[h] = (uint32_t)(((i < g.I ? i : g.I - 1) - i0) * g.lda + ap * 8) * 2;
    }
    const uint32_t u_off = (uint32_t)((j0 + bj < g.J ? j0 + bj : g.J - 1) - j0) * 4;
    const uint8_t* a_base = reinterpret_cast<const uint8_t*>(g.a + i0 * g.lda);
    uint4 ca[4];     // the chunk on its way from memory to LDS
    float cu[2][8];
    // Buffer loads: a base in scalar registers, a per-lane offset that never changes and a scalar one (given pointers, the
    // compiler adds up 64-bit addresses per load and lane, and spills some: 4096 x 4096 x 4096 325 us, so 313).
    auto fetch = [&](int64_t tc) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t ra = make_rsrc(a_base + 2 * tc);
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(ra, (int)a_off[h], 0, 0);
            ca[h] = make_uint4(v[0], v[1], v[2], v[3]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const __amdgpu_buffer_rsrc_t ru = make_rsrc(g.u + (tc + (bp + 2 * h) * 8) * g.ldu + j0);   // wave-uniform
#pragma unroll
            for (int e = 0; e < 8; ++e)
                cu[h][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(ru, (int)u_off, e * (int)g.ldu * 4, 0));
        }
    };
    // The first two and the last four chunks; the last one may end inside (on a whole piece): zeros for a, the last row of u
    // again.  All from the thread's number anew: kept for here, the addresses would be spilled around the loop.
    auto fetch_any = [&](int64_t tc) __attribute__((always_inline)) {
        int n = t;
        asm volatile("" : "+v"(n));
        const int64_t at = tc + (n & 3) * 8;
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const int64_t i = i0 + (n >> 2) + 64 * h;
            ca[h] = make_uint4(0u, 0u, 0u, 0u);
            if (at < g.T) ca[h] = *reinterpret_cast<const uint4*>(g.a + (i < g.I ? i : g.I - 1) * g.lda + at);
        }
        const int64_t j = j0 + (n & 127);
        const float* col = g.u + (j < g.J ? j : g.J - 1);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int64_t row = tc + (bp + 2 * h) * 8 + e;
                cu[h][e] = col[(row < g.T ? row : g.T - 1) * g.ldu];
            }
    };
    // (n: the thread's number, here and below)
    auto stash = [&](int buf, int n) __attribute__((always_inline)) {
        uint8_t* base = lds + buf * kProjWideBytes;
        const int row = n >> 2, piece = n & 3;
#pragma unroll
        for (int h = 0; h < 4; ++h)
            *reinterpret_cast<uint4*>(base + piece * kProjWidePieceA + ((row ^ (4 * piece)) + 64 * h) * 16) = ca[h];   // rows of four pieces side by side
#pragma unroll
        for (int h = 0; h < 2; ++h) stash_split(base + kProjWideBytesA + (bp + 2 * h) * kProjPieceB + (n & 127) * 16, cu[h]);
    };

    // acc[q][p]: columns 16 q .., rows 16 p .. of the wavefront's 128 x 64
    v4f acc[4][8];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < 8; ++p) acc[q][p] = (v4f){0.0f, 0.0f, 0.0f, 0.0f};
    // row (column) of a fragment: lane % 16, piece along the reduction: lane / 16
    static_assert(kProjChunk == 32, "an instruction takes a whole chunk");
    v8bf fa[8], fb[2][4];
    auto read_a = [&](int buf, int n) __attribute__((always_inline)) {
        const int ol = n & 15, oh = (n & 63) >> 4;
        const uint8_t* base = lds + buf * kProjWideBytes + oh * kProjWidePieceA + (wi * 128 + (ol ^ (4 * oh))) * 16;
#pragma unroll
        for (int p = 0; p < 8; ++p) fa[p] = *reinterpret_cast<const v8bf*>(base + p * 256);
    };
    auto read_b = [&](int part, int set, int buf, int n) __attribute__((always_inline)) {
        const int ol = n & 15, oh = (n & 63) >> 4;
        const uint8_t* base = lds + buf * kProjWideBytes + kProjWideBytesA + part * kProjSplitB + oh * kProjPieceB + (wj * 64 + ol) * 16;
#pragma unroll
        for (int q = 0; q < 4; ++q) fb[set][q] = *reinterpret_cast<const v8bf*>(base + q * 256);
    };
    // Product K of a part: tile (q, p) = (K / 8, K % 8), u as first operand, so that a lane ends with four consecutive
    // columns of a row.  As in resq_gemm.hip.h the instruction is assembly with its tile in place in accumulation
    // registers: given the builtin, the compiler renames the tiles and spills (8192 x 4096 x 4096 1244 us, this 612).
    auto product = [&](auto k, int set) __attribute__((always_inline)) {
        constexpr int K = decltype(k)::value;
        mfma_16x16x32_bf16(acc[K >> 3][K & 7], fb[set][K >> 3], fa[K & 7]);
    };
    auto multiply = [&](int set) __attribute__((always_inline)) {
        static_for<32>([&](auto k) __attribute__((always_inline)) { product(k, set); });
    };
    // columns e, e + 1 of unit h of the chunk in registers into their three parts
    uint32_t part[3][4];
    auto split2 = [&](auto h_, auto e_) __attribute__((always_inline)) {
        constexpr int H = decltype(h_)::value, E = decltype(e_)::value;
        uint32_t x[2], y[2], z[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float v = cu[H][E + k];
            x[k] = __float_as_uint(v);
            const float r1 = v - __uint_as_float(x[k] & 0xFFFF0000u);   // exact
            y[k] = __float_as_uint(r1);
            z[k] = __float_as_uint(r1 - __uint_as_float(y[k] & 0xFFFF0000u));  // exact, at most 8 bits left
        }
        part[0][E >> 1] = __builtin_amdgcn_perm(x[1], x[0], 0x07060302);
        part[1][E >> 1] = __builtin_amdgcn_perm(y[1], y[0], 0x07060302);
        part[2][E >> 1] = __builtin_amdgcn_perm(z[1], z[0], 0x07060302);
    };

    // Chunk i is multiplied out of buffer i % 2, the smallest parts of u first, while chunk i + 1 is split and written
    // into the other one and chunk i + 2 sets out.
    fetch_any(0);
    stash(0, t);
    fetch_any(kProjChunk);
    __syncthreads();
    auto step = [&](int64_t tc, int buf) __attribute__((always_inline)) {
        read_a(buf, t);
        read_b(2, 0, buf, t);
        __builtin_amdgcn_sched_barrier(0);
        uint8_t* const to = lds + (buf ^ 1) * kProjWideBytes;
        static_for<32>([&](auto k_) __attribute__((always_inline)) {
            constexpr int K = decltype(k_)::value;
            product(k_, 0);
            if constexpr (K < 24 && K % 3 == 1) split2(IC<K / 12>{}, IC<2 * (K / 3 % 4)>{});   // behind every third
            if constexpr (K == 11 || K == 23) {
                constexpr int H = K / 12;
#pragma unroll
                for (int s = 0; s < 3; ++s)
                    *reinterpret_cast<uint4*>(to + kProjWideBytesA + s * kProjSplitB + (bp + 2 * H) * kProjPieceB + bj * 16) =
                        make_uint4(part[s][0], part[s][1], part[s][2], part[s][3]);
            }
            if constexpr (K % 6 == 3 && K < 24) {
                constexpr int H = K / 6;
                *reinterpret_cast<uint4*>(to + ap * kProjWidePieceA + ((ar ^ (4 * ap)) + 64 * H) * 16) = ca[H];
            }
            if constexpr (K == 25) read_b(1, 1, buf, t);
            __builtin_amdgcn_sched_barrier(0);
        });
        static_for<32>([&](auto k_) __attribute__((always_inline)) {
            constexpr int K = decltype(k_)::value;
            product(k_, 1);
            if constexpr (K == 1) read_b(0, 0, buf, t);
            if constexpr (K == 3) fetch(tc + 2 * kProjChunk);
            if constexpr (K == 1 || K == 3) __builtin_amdgcn_sched_barrier(0);
        });
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
    };
    int64_t tc = 0;
    for (; tc + 4 * kProjChunk <= g.T; tc += 2 * kProjChunk) {
        step(tc, 0);
        step(tc + kProjChunk, 1);
    }
    for (int buf = 0; tc < g.T; tc += kProjChunk, buf ^= 1) {   // up to four chunks are left, the last one perhaps ragged
        int n = t;   // as in fetch_any
        asm volatile("" : "+v"(n));
        read_a(buf, n);
        read_b(2, 0, buf, n);
        read_b(1, 1, buf, n);
        multiply(0);
        read_b(0, 0, buf, n);
        multiply(1);
        multiply(0);
        if (tc + kProjChunk < g.T) {
            stash(buf ^ 1, n);
            fetch_any(tc + 2 * kProjChunk);
            __syncthreads();
        }
    }

    wait_for_products();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int p = 0; p < 8; ++p) asm volatile("" : "+a"(acc[q][p]));   // read behind the wait, not in front of it
    // any sum that is not finite (0 x it is NaN) sends the whole workgroup to the second way out
    float probe[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};   // eight short chains instead of a long one
#pragma unroll
    for (int e = 0; e < 128; ++e) probe[e & 7] = fmaf(acc[e >> 5][(e >> 2) & 7][e & 3], 0.0f, probe[e & 7]);
    const float sum = ((probe[0] + probe[1]) + (probe[2] + probe[3])) + ((probe[4] + probe[5]) + (probe[6] + probe[7]));
    int* redo = reinterpret_cast<int*>(lds);   // a sum of this workgroup is not finite
    __syncthreads();
    if (t == 0) *redo = 0;
    __syncthreads();
    if (sum != sum) *redo = 1;
    __syncthreads();
    const bool again = __builtin_amdgcn_readfirstlane(*redo) != 0;

    // acc[q][p][v]: column 4 (lane / 16) + v, row lane % 16 of matrix tile (q, p)
    int n = t;   // as in fetch_any
    asm volatile("" : "+v"(n));
    auto place = [&](int q, int p, int64_t& i, int64_t& j) __attribute__((always_inline)) {
        i = i0 + wi * 128 + p * 16 + (n & 15);
        j = j0 + wj * 64 + q * 16 + 4 * ((n & 63) >> 4);
    };
    // J is a multiple of eight, so four columns are there or none; rows start at any address, see Piece16
    auto store4 = [&](int64_t i, int64_t j, const v4f& c) __attribute__((always_inline)) {
        if constexpr (OUT_BF16) {
            uint16_t* dst = static_cast<uint16_t*>(g.out) + i * g.ldo + j;
            *reinterpret_cast<Piece8*>(dst) = Piece8{pack_bf16(c[0], c[1]), pack_bf16(c[2], c[3])};
        } else {
            float* dst = static_cast<float*>(g.out) + i * g.ldo + j;
            *reinterpret_cast<Piece16*>(dst) = Piece16{__float_as_uint(c[0]), __float_as_uint(c[1]), __float_as_uint(c[2]), __float_as_uint(c[3])};
        }
    };
#pragma unroll
    for (int p = 0; p < 8; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            int64_t i, j;
            place(q, p, i, j);
            if (i < g.I && j < g.J) store4(i, j, acc[q][p]);
        }
    if (__builtin_expect(!again, 1)) return;
    // out does not lie on a or u (the launch sees to it): a lane reads its own outputs again and takes the NaN sums anew
#pragma unroll 1
    for (int e = 0; e < 128; ++e) {
        int64_t i, j;
        place(e >> 5, (e >> 2) & 7, i, j);
        j += e & 3;
        if (i >= g.I || j >= g.J) continue;
        float s = OUT_BF16 ? __uint_as_float((uint32_t)static_cast<const uint16_t*>(g.out)[i * g.ldo + j] << 16)
                           : static_cast<const float*>(g.out)[i * g.ldo + j];
        if (s == s) continue;
        const uint16_t* row = g.a + i * g.lda;
        s = 0.0f;
        for (int64_t k = 0; k < g.T && s == s; k += 8) {   // whole pieces; a NaN stays one
            const uint4 piece = *reinterpret_cast<const uint4*>(row + k);
            const uint32_t w[4] = {piece.x, piece.y, piece.z, piece.w};
            float c[8];
#pragma unroll
            for (int n = 0; n < 8; ++n) c[n] = g.u[(k + n) * g.ldu + j];
#pragma unroll
            for (int n = 0; n < 8; ++n)
                s = fmaf(__uint_as_float(n & 1 ? w[n >> 1] & 0xFFFF0000u : w[n >> 1] << 16), c[n], s);
        }
        if constexpr (OUT_BF16) static_cast<uint16_t*>(g.out)[i * g.ldo + j] = (uint16_t)pack_bf16(s, 0.0f);
        else static_cast<float*>(g.out)[i * g.ldo + j] = s;
    }
}

}  // namespace resq
