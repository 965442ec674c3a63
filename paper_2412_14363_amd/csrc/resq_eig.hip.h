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
// are 3048 launches, 10.5 ms.  Here a workgroup keeps the matrix in LDS (fp64, one
// copy of each off-diagonal pair: 132 KB at n = 128) and walks all rounds by
// itself: a round is 2 x 2 blocks (pair k, pair kk) that no two threads share, so
// it needs two barriers (2.75 ms in all).  The vectors do not fit beside it, but column j of Vt is
// rotated independently of every other column: each of the ceil(n / 16) workgroups
// repeats the iteration on the matrix (same arithmetic, same decisions) and carries
// 16 columns of Vt, so that the workgroups never talk to each other.  The vectors'
// rotation of round r runs on wavefronts 1..15 while wavefront 0 computes the
// angles of round r + 1, a chain of fp64 roots and quotients that is the longest
// part of a round.
constexpr int kEigSmallMax = 128;
constexpr int kEigSmallThreads = 1024;
constexpr int kEigSmallCols = 16;  // columns of Vt per workgroup

// Bytes of LDS: matrix [n][n + 3], Vt slice [n][16], cosines and sines of two rounds, two flags.
// The pitch is odd, so that neither a run along a row nor one along a column meets a bank twice,
// and not n + 1, with which all elements of a round's pairs (p + q is the same for all) would.
__host__ __device__ inline int eig_small_lds_bytes(int n) {
    return (n * (n + 3) + n * kEigSmallCols + 2 * n) * (int)sizeof(double) + 2 * (int)sizeof(int);
}

__global__ __launch_bounds__(kEigSmallThreads) void eig_small_kernel(const float* __restrict__ c, int64_t ldc, int n,
                                                                     int sweeps, float* __restrict__ eigvals,
                                                                     float* __restrict__ p, int64_t ldp) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    const int pitch = n + 3, half = n >> 1;
    double* a = lds;                                   // element (i, j), i <= j, at i * pitch + j
    double* vt = a + n * pitch;                        // [n][16]: columns j0 .. j0 + 15 of Vt
    double2* cs = reinterpret_cast<double2*>(vt + n * kEigSmallCols);  // [2][half]
    int* flag = reinterpret_cast<int*>(cs + n);        // [2]: does the round rotate anything
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int j0 = blockIdx.x * kEigSmallCols;

    for (int idx = t; idx < n * n; idx += kEigSmallThreads) {
        const int i = idx / n, j = idx % n;
        if (i <= j) a[i * pitch + j] = 0.5 * ((double)c[(int64_t)i * ldc + j] + (double)c[(int64_t)j * ldc + i]);
    }
    for (int idx = t; idx < n * kEigSmallCols; idx += kEigSmallThreads)
        vt[idx] = idx / kEigSmallCols == j0 + idx % kEigSmallCols ? 1.0 : 0.0;
    __syncthreads();

    auto at = [&](int i, int j) __attribute__((always_inline)) -> double& {
        return a[i < j ? i * pitch + j : j * pitch + i];
    };
    // Vt <- J^T Vt for the round whose rotations are rot, on `threads` threads from `first` on
    auto rotate_vectors = [&](const double2* rot, int round, int first, int threads) __attribute__((always_inline)) {
        for (int idx = t - first; idx < half * kEigSmallCols; idx += threads) {
            const int k = idx / kEigSmallCols, col = idx % kEigSmallCols;
            const double2 r = rot[k];
            if (r.y == 0.0) continue;
            int pp, qq;
            eig_pair(n, round, k, pp, qq);
            double* vp = vt + pp * kEigSmallCols + col;
            double* vq = vt + qq * kEigSmallCols + col;
            const double x = *vp, y = *vq;
            *vp = r.x * x - r.y * y;
            *vq = r.y * x + r.x * y;
        }
    };

    int buf = 0, pending = 0, pending_round = 0;  // the vectors are one round behind the matrix
    for (int sweep = 0; sweep < sweeps; ++sweep) {
        int rotated = 0;
        for (int round = 0; round < n - 1; ++round) {
            double2* rot = cs + buf * half;
            if (wave == 0) {
                bool turn = false;
                if (lane < half) {
                    int pp, qq;
                    eig_pair(n, round, lane, pp, qq);
                    const double app = a[pp * pitch + pp], aqq = a[qq * pitch + qq], apq = a[pp * pitch + qq];
                    double2 r = make_double2(1.0, 0.0);
                    turn = fabs(apq) > kEigSkip * sqrt(fabs(app * aqq));
                    if (turn) {
                        // As eig_rotations_kernel has it.  (Approximate quotients and roots shorten this chain to a
                        // third, and the signs of some vectors then come out otherwise.)
                        const double tau = (aqq - app) / (2.0 * apq);
                        const double tn = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
                        r.x = 1.0 / sqrt(1.0 + tn * tn);
                        r.y = tn * r.x;
                    }
                    rot[lane] = r;
                }
                const bool any = __ballot(turn) != 0;
                if (lane == 0) flag[buf] = any ? 1 : 0;
            } else if (pending) {
                rotate_vectors(cs + (buf ^ 1) * half, pending_round, 64, kEigSmallThreads - 64);
            }
            __syncthreads();
            const int any = flag[buf];
            if (any) {
                // Blocks (k, kk), k < kk.  Unit k of half / 2 (rounded up) takes kk > k of pair k on its upper
                // lanes and, turned round, kk >= k' of pair k' = half - 1 - k on its lower ones, so that all
                // lanes work and each half runs along one pair of rows.  A wavefront loads the blocks of two
                // units before it writes the first.  The diagonal blocks (lane k of unit k, and those of the
                // lower pairs, which no unit meets) are wavefront 0's afterwards.
                const int mate = half - 1 - lane;
                const bool live = lane < half;
                const double2 r_up = rot[live ? lane : 0], r_dn = rot[live ? mate : 0];
                int up_p, up_q, dn_p, dn_q;
                eig_pair(n, round, live ? lane : 0, up_p, up_q);
                eig_pair(n, round, live ? mate : 0, dn_p, dn_q);
                const int units = (half + 1) >> 1;
                for (int u0 = wave; u0 < units; u0 += 2 * (kEigSmallThreads / 64)) {
                    double x[2][4];
                    double* e[2][4];
                    double2 ra[2], rb[2];
                    bool on[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int k = u0 + h * (kEigSmallThreads / 64);
                        const bool upper = lane > k;
                        const int kr = upper ? k : half - 1 - k;
                        // off the diagonal, and not the lower half of the middle unit of an odd number of pairs
                        on[h] = k < units && live && lane != k && (upper || 2 * k != half - 1);
                        ra[h] = rot[on[h] ? kr : 0];
                        rb[h].x = upper ? r_up.x : r_dn.x;
                        rb[h].y = upper ? r_up.y : r_dn.y;
                        on[h] = on[h] && (ra[h].y != 0.0 || rb[h].y != 0.0);
                        int p1, q1;
                        eig_pair(n, round, kr < 0 ? 0 : kr, p1, q1);
                        const int p2 = upper ? up_p : dn_p, q2 = upper ? up_q : dn_q;
                        e[h][0] = &at(p1, p2);
                        e[h][1] = &at(p1, q2);
                        e[h][2] = &at(q1, p2);
                        e[h][3] = &at(q1, q2);
                        if (on[h]) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) x[h][v] = *e[h][v];
                        }
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (!on[h]) continue;
                        const double y00 = ra[h].x * x[h][0] - ra[h].y * x[h][2], y10 = ra[h].y * x[h][0] + ra[h].x * x[h][2];
                        const double y01 = ra[h].x * x[h][1] - ra[h].y * x[h][3], y11 = ra[h].y * x[h][1] + ra[h].x * x[h][3];
                        *e[h][0] = rb[h].x * y00 - rb[h].y * y01;
                        *e[h][1] = rb[h].y * y00 + rb[h].x * y01;
                        *e[h][2] = rb[h].x * y10 - rb[h].y * y11;
                        *e[h][3] = rb[h].y * y10 + rb[h].x * y11;
                    }
                }
                if (wave == 0 && live && r_up.y != 0.0) {
                    const double2 r = r_up;
                    double& xpp = a[up_p * pitch + up_p];
                    double& xqq = a[up_q * pitch + up_q];
                    double& xpq = a[up_p * pitch + up_q];
                    const double app = xpp, aqq = xqq, apq = xpq;
                    const double rpp = r.x * app - r.y * apq, rpq = r.x * apq - r.y * aqq;
                    const double rqp = r.y * app + r.x * apq, rqq = r.y * apq + r.x * aqq;
                    xpp = r.x * rpp - r.y * rpq;
                    xpq = r.y * rpp + r.x * rpq;
                    xqq = r.y * rqp + r.x * rqq;
                }
                __syncthreads();
            }
            rotated |= any;
            pending = any;
            pending_round = round;
            buf ^= 1;
        }
        if (!rotated) break;  // as every later sweep would find: the same for all threads
    }
    if (pending) rotate_vectors(cs + (buf ^ 1) * half, pending_round, 0, kEigSmallThreads);
    __syncthreads();
    // positions in decreasing order (ties by index), as eig_finish_kernel has them
    int* rank = reinterpret_cast<int*>(cs);
    if (t < n) {
        const double li = a[t * pitch + t];
        int r = 0;
        for (int j = 0; j < n; ++j) {
            const double lj = a[j * pitch + j];
            r += (lj > li || (lj == li && j < t)) ? 1 : 0;
        }
        rank[t] = r;
        if (blockIdx.x == 0) eigvals[r] = (float)li;
    }
    __syncthreads();
    for (int idx = t; idx < n * kEigSmallCols; idx += kEigSmallThreads) {
        const int col = idx / n, i = idx % n;
        if (j0 + col < n) p[(int64_t)(j0 + col) * ldp + rank[i]] = (float)vt[i * kEigSmallCols + col];
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
