// Symmetric eigendecomposition for the PCA step of the basis construction
// (Section 4.2: P = eigenvectors of the activations' covariance matrix; the r
// of largest eigenvalue span the high-precision subspace): cyclic Jacobi in
// fp64 with the round-robin ("tournament") ordering, n / 2 disjoint rotations
// per round, n - 1 rounds per sweep.
//
// A round applies J = product of its plane rotations as A <- J^T A J, V <- V J,
// in one pass over the matrix: the workgroup of pair (p, q) owns rows p and q.
// J^T A mixes exactly those two rows, element by element; (J^T A) J then mixes,
// inside each row, the elements of every pair of the round, so the two rotated
// rows sit in LDS (16 n bytes) while all n / 2 column rotations are applied to
// them, and go back in place.  The eigenvectors are kept transposed, so that
// their update Vt <- J^T Vt is the same two-row operation.  Every access to
// memory is a contiguous row.  Offline step, bound by HBM: 4 n^2 fp64 words move
// per round (matrix and vectors, read and written once).  Rotations of elements
// already negligible are skipped, and once a whole sweep has skipped all of them
// the remaining kernels return at once.
//
// Matrices of at most 128 columns (head-size bases) take eig_small_kernel, which
// runs the whole iteration in one launch on LDS.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace resq {

constexpr int kEigThreads = 256;
constexpr int kEigMaxOrder = 8192;  // two fp64 rows in LDS: 128 KiB

struct EigPlan {
    int n;            // matrix order, even
    double* a;        // the matrix, [n][n], symmetric between rounds
    double* vt;       // eigenvectors as rows, [n][n]
    int* pq;          // [n / 2][2]: the round's pairs, p < q
    double* cs;       // [n / 2][2]: cosine and sine of each pair's rotation
    int* nrot;        // [kEigMaxSweeps]: rotations that each sweep still had to make
};

constexpr int kEigMaxSweeps = 64;
// an off-diagonal element below this fraction of sqrt(a_pp a_qq) is left alone: fp32
// outputs cannot tell, and a sweep that finds nothing larger ends the iteration
constexpr double kEigSkip = 1.0 / (1ull << 40);

// a sweep after one that rotated nothing has nothing to do (the host enqueues a fixed
// number of sweeps, so that the call never waits for the device)
__device__ __forceinline__ bool eig_converged(const EigPlan& e, int sweep) {
    return sweep > 0 && e.nrot[sweep - 1] == 0;
}

// pair k of round s: (n - 1, s) for k = 0, else ((s + k) mod (n - 1), (s - k) mod (n - 1))
__device__ __forceinline__ void eig_pair(int n, int s, int k, int& p, int& q) {
    const int m = n - 1;
    int a = s + k, b = s - k;   // 0 <= s < m, 0 <= k < n / 2
    a = k == 0 ? m : (a >= m ? a - m : a);
    b = b < 0 ? b + m : b;
    p = a < b ? a : b;
    q = a < b ? b : a;
}

__global__ void eig_init_kernel(const float* __restrict__ c, int64_t ldc, EigPlan e) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nn = (int64_t)e.n * e.n;
    if (idx < kEigMaxSweeps) e.nrot[idx] = 0;   // the grid has at least that many threads
    if (idx >= nn) return;
    const int i = (int)(idx / e.n), j = (int)(idx % e.n);
    // the symmetric part, so that rounding differences between c[i][j] and c[j][i] do not matter
    e.a[idx] = 0.5 * ((double)c[(int64_t)i * ldc + j] + (double)c[(int64_t)j * ldc + i]);
    e.vt[idx] = i == j ? 1.0 : 0.0;
}

// rotation that annihilates a[p][q] (the smaller of the two angles)
__global__ void eig_rotations_kernel(EigPlan e, int sweep, int round) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= e.n / 2 || eig_converged(e, sweep)) return;
    int p, q;
    eig_pair(e.n, round, k, p, q);
    const double* a = e.a;
    const double app = a[(int64_t)p * e.n + p], aqq = a[(int64_t)q * e.n + q], apq = a[(int64_t)p * e.n + q];
    double c = 1.0, s = 0.0;
    if (fabs(apq) > kEigSkip * sqrt(fabs(app * aqq))) {
        atomicAdd(&e.nrot[sweep], 1);
        const double tau = (aqq - app) / (2.0 * apq);
        const double t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
        c = 1.0 / sqrt(1.0 + t * t);
        s = t * c;
    }
    e.pq[2 * k] = p;
    e.pq[2 * k + 1] = q;
    e.cs[2 * k] = c;
    e.cs[2 * k + 1] = s;
}

// ---- orders up to 128: the whole iteration in one launch ------------------------------------
//
// Two launches per round (a rotation kernel of one workgroup, a row kernel) cost
// more than the rounds themselves at head sizes: 12 sweeps of a 128 x 128 matrix
// are 3048 launches, 10.5 ms.  Here a workgroup keeps the matrix in LDS (fp64,
// one copy of each off-diagonal pair) and walks all rounds by itself.
//
// Slots.  What made a first version of this kernel slow (5200 clocks a round) was
// finding the elements: the pairs change every round.  So the DATA moves instead:
// pair k owns slots (k, 0) and (k, 1) for good, and after a round the element in a
// slot moves one place along the tournament's circle (slot (0, 0) stays).  A round
// reads and writes the same addresses every time, from one buffer into the other;
// after n - 1 rounds, a sweep, everything is back where it was.  The four elements of
// the 2 x 2 block of two pairs lie in four planes: no bank is met twice.
//
// The vectors do not fit beside the matrix, but column j of Vt is rotated
// independently of every other column: each of the ceil(n / 8) workgroups repeats
// the iteration on the matrix (same arithmetic, same decisions) and carries 8
// columns of Vt, so that the workgroups never talk to each other.  The vectors'
// rotation of round r runs on wavefronts 1..15 while wavefront 0 computes the
// angles of round r + 1, a chain of fp64 roots and quotients.  (Wavefront 0 rotating
// only the blocks that the next angles need, and the others all the rest behind one
// barrier a round instead of two, measured the same: 1.04 ms at n = 128.)
//
// Measured, 12 sweeps allowed, two launches a round / this kernel: n = 128 9.9 to 10.5 / 1.70 ms on a
// covariance with a spectrum that decays by e^-6, 6.9 / 1.06 on that of Gaussian rows, which
// converges in fewer sweeps (3000 clocks a round); Gaussian n = 64 4.9 / 0.39, n = 32 1.69 / 0.15.
constexpr int kEigSmallMax = 128;
constexpr int kEigSmallThreads = 1024;
constexpr int kEigSmallCols = 8;  // columns of Vt per workgroup

// blocks (k, l), k < l: lanes of `units` rows of n / 2 (see below)
__host__ __device__ inline int eig_small_units(int half) { return (half + 1) >> 1; }
// doubles of one of the two buffers: the four planes, the diagonal blocks (three numbers each)
__host__ __device__ inline int eig_small_buf(int half) { return 4 * eig_small_units(half) * half + 3 * half + (half & 1); }  // even: what lies behind is 16-byte aligned
// bytes of LDS: both buffers, both buffers of the Vt slice [n][8], cosines and sines of two rounds, two flags
__host__ __device__ inline int eig_small_lds_bytes(int n) {
    return (2 * eig_small_buf(n / 2) + 2 * n * kEigSmallCols + 2 * n) * (int)sizeof(double) + 2 * (int)sizeof(int);
}

__global__ __launch_bounds__(kEigSmallThreads) void eig_small_kernel(const float* __restrict__ c, int64_t ldc, int n,
                                                                     int sweeps, float* __restrict__ eigvals,
                                                                     float* __restrict__ p, int64_t ldp) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    const int half = n >> 1, units = eig_small_units(half), plane = units * half, bufsz = eig_small_buf(half);
    const int diag = 4 * plane;                        // a00[half], a11[half], a01[half] of the pairs
    double* vt = lds + 2 * bufsz;                      // [2][n][8]: columns j0 .. j0 + 7 of Vt, rows by slot 2 k + x
    double2* cs = reinterpret_cast<double2*>(vt + 2 * n * kEigSmallCols);  // [2][half]
    int* flag = reinterpret_cast<int*>(cs + n);        // [2]: does the round rotate anything
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int j0 = blockIdx.x * kEigSmallCols;

    // the index whose row and column start (and end every sweep) in slot (k, x): eig_pair's round 0
    auto index_of = [&](int k, int x) { return k == 0 ? (x == 0 ? n - 1 : 0) : (x == 0 ? k : n - 1 - k); };
    // where the element in slot (k, x) goes after a round
    auto move = [&](int& k, int& x) {
        if (half == 1 || (k == 0 && x == 0)) return;
        if (x == 0) {
            if (k == 1) { k = 0; x = 1; }
            else --k;
        } else {
            if (k < half - 1) ++k;
            else x = 0;
        }
    };
    // Block (k, l), k < l: row k of the units, lane l, for the lower half of the pairs; the rows'
    // free lanes below k hold, turned round, the blocks of pair half - 1 - k, so that all lanes work.
    auto block_at = [&](int k, int l) { return k < units ? k * half + l : (half - 1 - k) * half + half - 1 - l; };
    // offset in a buffer of the element between two slots
    auto at = [&](int k, int x, int l, int y) {
        if (k == l) return diag + (x != y ? 2 * half : x * half) + k;
        if (k > l) {
            int s = k; k = l; l = s;
            s = x; x = y; y = s;
        }
        return (2 * x + y) * plane + block_at(k, l);
    };

    for (int idx = t; idx < n * n; idx += kEigSmallThreads) {
        const int s0 = idx / n, s1 = idx % n;
        if (s0 > s1) continue;
        const int i = index_of(s0 >> 1, s0 & 1), j = index_of(s1 >> 1, s1 & 1);
        lds[at(s0 >> 1, s0 & 1, s1 >> 1, s1 & 1)] =
            0.5 * ((double)c[(int64_t)i * ldc + j] + (double)c[(int64_t)j * ldc + i]);
    }
    for (int idx = t; idx < n * kEigSmallCols; idx += kEigSmallThreads) {
        const int s0 = idx / kEigSmallCols;
        vt[idx] = index_of(s0 >> 1, s0 & 1) == j0 + idx % kEigSmallCols ? 1.0 : 0.0;
    }

    // this thread's blocks (two rows of units at most), their places and where their four elements go
    bool on[2];
    int bk[2], bl[2], rd[2], wr[2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int u = wave + h * (kEigSmallThreads / 64);
        const bool upper = lane > u;
        // not the diagonal, and not the lower lanes of the middle row of an odd number of pairs
        on[h] = u < units && lane < half && lane != u && (upper || 2 * u != half - 1);
        bk[h] = on[h] ? (upper ? u : half - 1 - u) : 0;
        bl[h] = on[h] ? (upper ? lane : half - 1 - lane) : 0;
        rd[h] = on[h] ? u * half + lane : 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int k = bk[h], x = e >> 1, l = bl[h], y = e & 1;
            move(k, x);
            move(l, y);
            wr[h][e] = on[h] ? at(k, x, l, y) : 0;
        }
    }
    // wavefront 0: the diagonal block of pair `lane`
    int wd[3];
    {
        int k0 = lane < half ? lane : 0, x0 = 0, k1 = k0, x1 = 1;
        move(k0, x0);
        move(k1, x1);
        wd[0] = at(k0, x0, k0, x0);
        wd[1] = at(k1, x1, k1, x1);
        wd[2] = at(k0, x0, k1, x1);
    }
    // the others: two rows of one column of Vt
    const int vk = (t - 64) / kEigSmallCols, vc = t & (kEigSmallCols - 1);
    const bool v_on = t >= 64 && vk < half;
    int vw[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        int k = v_on ? vk : 0, y = x;
        move(k, y);
        vw[x] = (2 * k + y) * kEigSmallCols + vc;
    }
    __syncthreads();

    // Vt <- J^T Vt for the round whose rotations are rot, from buffer b of the slice into the other
    auto rotate_vectors = [&](const double2* rot, int b) __attribute__((always_inline)) {
        if (!v_on) return;
        const double* src = vt + b * n * kEigSmallCols + 2 * vk * kEigSmallCols + vc;
        double* dst = vt + (b ^ 1) * n * kEigSmallCols;
        const double2 r = rot[vk];
        const double x = src[0], y = src[kEigSmallCols];
        dst[vw[0]] = r.x * x - r.y * y;
        dst[vw[1]] = r.y * x + r.x * y;
    };

    int buf = 0, rounds = 0;  // the vectors are one round behind the matrix
    for (int sweep = 0; sweep < sweeps; ++sweep) {
        int rotated = 0;
        for (int round = 0; round < n - 1; ++round) {
            const double* cur = lds + buf * bufsz;
            double* nxt = lds + (buf ^ 1) * bufsz;
            double2* rot = cs + buf * half;
            double a00 = 0.0, a11 = 0.0, a01 = 0.0;
            double2 r = make_double2(1.0, 0.0);
            if (wave == 0) {
                bool turn = false;
                if (lane < half) {
                    a00 = cur[diag + lane];
                    a11 = cur[diag + half + lane];
                    a01 = cur[diag + 2 * half + lane];
                    // As eig_rotations_kernel has it, |a01| > 2^-40 sqrt(|a00 a11|) and tan of the smaller angle =
                    // sign(tau) / (|tau| + sqrt(1 + tau^2)), tau = (a11 - a00) / (2 a01), in a form with fewer
                    // roots and quotients in a row.  (The hardware's approximate ones are not enough: the
                    // signs of some vectors then come out otherwise.)
                    turn = a01 * a01 > kEigSkip * kEigSkip * fabs(a00 * a11);
                    if (turn) {
                        const double d = a11 - a00, b = 2.0 * a01;
                        double tn = fabs(b) / (fabs(d) + sqrt(d * d + b * b));
                        if (d != 0.0 && (d < 0.0) != (b < 0.0)) tn = -tn;
                        r.x = rsqrt(1.0 + tn * tn);
                        r.y = tn * r.x;
                    }
                    rot[lane] = r;
                }
                const bool any = __ballot(turn) != 0;
                if (lane == 0) flag[buf] = any ? 1 : 0;
            } else if (rounds > 0) {
                rotate_vectors(cs + (buf ^ 1) * half, buf ^ 1);
            }
            __syncthreads();
            rotated |= flag[buf];
            double2 x0[2], x1[2], ra[2], rb[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (!on[h]) continue;
                ra[h] = rot[bk[h]];
                rb[h] = rot[bl[h]];
                x0[h] = make_double2(cur[rd[h]], cur[plane + rd[h]]);
                x1[h] = make_double2(cur[2 * plane + rd[h]], cur[3 * plane + rd[h]]);
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (!on[h]) continue;
                const double y00 = ra[h].x * x0[h].x - ra[h].y * x1[h].x, y10 = ra[h].y * x0[h].x + ra[h].x * x1[h].x;
                const double y01 = ra[h].x * x0[h].y - ra[h].y * x1[h].y, y11 = ra[h].y * x0[h].y + ra[h].x * x1[h].y;
                nxt[wr[h][0]] = rb[h].x * y00 - rb[h].y * y01;
                nxt[wr[h][1]] = rb[h].y * y00 + rb[h].x * y01;
                nxt[wr[h][2]] = rb[h].x * y10 - rb[h].y * y11;
                nxt[wr[h][3]] = rb[h].y * y10 + rb[h].x * y11;
            }
            if (wave == 0 && lane < half) {
                const double r00 = r.x * a00 - r.y * a01, r01 = r.x * a01 - r.y * a11;
                const double r10 = r.y * a00 + r.x * a01, r11 = r.y * a01 + r.x * a11;
                nxt[wd[0]] = r.x * r00 - r.y * r01;
                nxt[wd[1]] = r.y * r10 + r.x * r11;
                nxt[wd[2]] = r.y * r00 + r.x * r01;
            }
            __syncthreads();
            buf ^= 1;
            ++rounds;
        }
        if (!rotated) break;  // as every later sweep would find: the same for all threads
    }
    rotate_vectors(cs + (buf ^ 1) * half, buf ^ 1);
    // positions in decreasing order (ties by index), as eig_finish_kernel has them; rank by slot
    const double* a = lds + buf * bufsz + diag;
    vt += buf * n * kEigSmallCols;
    int* rank = reinterpret_cast<int*>(cs + buf * half);   // not the rotations that are still read
    if (t < n) {
        const double li = a[(t & 1) * half + (t >> 1)];
        const int i = index_of(t >> 1, t & 1);
        int r = 0;
        for (int s = 0; s < n; ++s) {
            const double lj = a[(s & 1) * half + (s >> 1)];
            r += (lj > li || (lj == li && index_of(s >> 1, s & 1) < i)) ? 1 : 0;
        }
        rank[t] = r;
        if (blockIdx.x == 0) eigvals[r] = (float)li;
    }
    __syncthreads();
    for (int idx = t; idx < n * kEigSmallCols; idx += kEigSmallThreads) {
        const int col = idx / n, s = idx % n;
        if (j0 + col < n) p[(int64_t)(j0 + col) * ldp + rank[s]] = (float)vt[s * kEigSmallCols + col];
    }
}

// one round for pair blockIdx.x: rows p, q of A <- J^T A J, rows p, q of Vt <- J^T Vt
__global__ __launch_bounds__(kEigThreads) void eig_round_kernel(EigPlan e, int sweep) {
    extern __shared__ __attribute__((aligned(16))) double rows[];  // [2][n]
    if (eig_converged(e, sweep)) return;
    const int n = e.n, t = threadIdx.x, k = blockIdx.x;
    const int p = e.pq[2 * k], q = e.pq[2 * k + 1];
    const double c = e.cs[2 * k], s = e.cs[2 * k + 1];
    double* ap = e.a + (int64_t)p * n;
    double* aq = e.a + (int64_t)q * n;
    double* rp = rows;
    double* rq = rows + n;
    for (int j = t; j < n; j += kEigThreads) {
        const double x = ap[j], y = aq[j];
        rp[j] = c * x - s * y;
        rq[j] = s * x + c * y;
    }
    {
        double* vp = e.vt + (int64_t)p * n;
        double* vq = e.vt + (int64_t)q * n;
        for (int j = t; j < n; j += kEigThreads) {
            const double x = vp[j], y = vq[j];
            vp[j] = c * x - s * y;
            vq[j] = s * x + c * y;
        }
    }
    __syncthreads();
    // the column rotations of every pair of the round, on both rows (the pairs are disjoint)
    for (int kk = t; kk < n / 2; kk += kEigThreads) {
        const int p2 = e.pq[2 * kk], q2 = e.pq[2 * kk + 1];
        const double c2 = e.cs[2 * kk], s2 = e.cs[2 * kk + 1];
        const double x0 = rp[p2], y0 = rp[q2], x1 = rq[p2], y1 = rq[q2];
        rp[p2] = c2 * x0 - s2 * y0;
        rp[q2] = s2 * x0 + c2 * y0;
        rq[p2] = c2 * x1 - s2 * y1;
        rq[q2] = s2 * x1 + c2 * y1;
    }
    __syncthreads();
    for (int j = t; j < n; j += kEigThreads) {
        ap[j] = rp[j];
        aq[j] = rq[j];
    }
}

// eigenvalue i = a[i][i]; its position in decreasing order (ties by index); column
// rank[i] of P = row i of Vt
__global__ __launch_bounds__(kEigThreads) void eig_finish_kernel(EigPlan e, float* __restrict__ eigvals,
                                                                 float* __restrict__ p, int64_t ldp) {
    const int i = blockIdx.x;
    const int n = e.n;
    const double* a = e.a;
    const double li = a[(int64_t)i * n + i];
    __shared__ int count[kEigThreads];
    int c = 0;
    for (int j = threadIdx.x; j < n; j += kEigThreads) {
        const double lj = a[(int64_t)j * n + j];
        c += (lj > li || (lj == li && j < i)) ? 1 : 0;
    }
    count[threadIdx.x] = c;
    __syncthreads();
    for (int w = kEigThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) count[threadIdx.x] += count[threadIdx.x + w];
        __syncthreads();
    }
    const int rank = count[0];
    if (threadIdx.x == 0) eigvals[rank] = (float)li;
    for (int j = threadIdx.x; j < n; j += kEigThreads) p[(int64_t)j * ldp + rank] = (float)e.vt[(int64_t)i * n + j];
}

}  // namespace resq
