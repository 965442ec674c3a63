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

#include <type_traits>

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
// independently of every other column: each of the n / kEigSmallCols workgroups repeats
// the iteration on the matrix (same arithmetic, same decisions) and carries two
// columns of Vt, so that the workgroups never talk to each other.  (Eight columns are a tenth of the traffic of a workgroup's LDS,
// which bounds a round of the large orders: n = 128 1267 us with eight, 1234 with four, 1208 with two.)
//
// One barrier a round.  Wavefront 0 is a round ahead: it turns the blocks that the diagonal blocks of the NEXT round
// come from, and computes that round's angles, a chain of two fp64 roots, while the others turn the matrix
// by this round's and, two of them, the vectors.  (With the angles of a round between two barriers, 900 of 2870
// clocks were theirs alone.)  What bounds a round of n = 128 now is LDS, 8 elements and 4 numbers of rotations a block, about
// 1650 of 2050 clocks; of n = 64 and less the chain of wavefront 0.  Measured and not taken: two neighbouring rows of blocks to a wavefront, half of their elements handed
// on from lane to lane (6 % a round, and what wavefront 0 needs of them is written to LDS after all), the rotations handed from lane to lane instead of read again (29 % slower:
// vector instructions), n known to the compiler (14 % slower at 128: it joins reads of two planes into one
// instruction, on the same banks), a thread's blocks loaded together (4 % slower).
//
// Measured, 12 sweeps allowed, two launches a round / two barriers a round / this kernel: n = 128 9.9 to 10.5 / 1.79 / 1.20 to 1.32 ms on
// covariances with a spectrum that decays by e^-6 (11 or 12 sweeps of 127 rounds, 0.86 us a round), - / 1.50 / 1.10 on that of
// Gaussian rows (10 sweeps); n = 100 - / 1.11 / 0.89 (with eight columns of the vectors to a workgroup 0.93), n = 64 4.9 / 0.58 /
// 0.35, n = 34 - / 0.22 / 0.15, n = 32 1.69 / 0.19 / 0.145.
constexpr int kEigSmallMax = 128;
constexpr int kEigSmallThreads = 1024;
constexpr int kEigSmallCols = 2;  // columns of Vt per workgroup
static_assert(kEigSmallCols == 2, "every workgroup has whole columns only, n being even");

// As eig_rotations_kernel has it, |a01| > 2^-40 sqrt(|a00 a11|) and tan of the smaller angle =
// sign(tau) / (|tau| + sqrt(1 + tau^2)), tau = (a11 - a00) / (2 a01), in a form with two roots and no quotient in
// the chain, which is the longest of a round: with h the root of (a11 - a00)^2 + (2 a01)^2, the square of the cosine is (1 + |a11 - a00| / h) / 2
// and the sine |a01| / (h cos).  A root, a quotient and a root, us (the columns of Vt two in both): n = 128 1208 / 1206, 100 922 / 904,
// 64 371 / 351, 32 157 / 142, 8 30.9 / 28.4.  (The hardware's approximate roots are not enough: the
// signs of some vectors then come out otherwise.)  Squares below 1e-280 are no turn: roots of what has lost digits there
// would not give an orthogonal one.  (Two comparisons, not one with the larger bound, which would drop
// a NaN: with one on the diagonal the first comparison fails, the pair is not turned and no vector becomes NaN.)
__device__ __forceinline__ bool eig_turns(double a00, double a11, double a01) {
    return a01 * a01 > kEigSkip * kEigSkip * fabs(a00 * a11) && a01 * a01 > 1e-280;
}
__device__ __forceinline__ double2 eig_rotation(double a00, double a11, double a01) {
    const double d = a11 - a00, q = 2.0 * a01;
    const double rh = rsqrt(fma(d, d, q * q));              // 1 / hypotenuse
    const double x = fma(0.5 * fabs(d), rh, 0.5);           // the square of the cosine
    const double rc = rsqrt(x);
    const double s = 0.5 * fabs(q) * rh * rc;
    return make_double2(x * rc, d != 0.0 && (d < 0.0) != (q < 0.0) ? -s : s);
}

// Order 2: one block, the iteration below in one thread's registers.  (eig_small_kernel, whose length is mostly that of its code
// there, takes 4.65 us, this 4.05; with two barriers a round it took 4.0.)  Index 1 in slot 0, index 0 in slot 1, as there.
__global__ __launch_bounds__(64) void eig_pair_kernel(const float* __restrict__ c, int64_t ldc, int sweeps,
                                                      float* __restrict__ eigvals, float* __restrict__ p, int64_t ldp) {
    if (threadIdx.x > 0) return;
    double a00 = c[ldc + 1], a11 = c[0], a01 = 0.5 * ((double)c[1] + (double)c[ldc]);
    double v0[2] = {0.0, 1.0}, v1[2] = {1.0, 0.0};   // rows of Vt
    for (int sweep = 0; sweep < sweeps && eig_turns(a00, a11, a01); ++sweep) {
        const double2 r = eig_rotation(a00, a11, a01);
        const double x0 = r.x * a00 - r.y * a01, x1 = r.x * a01 - r.y * a11;
        const double y0 = r.y * a00 + r.x * a01, y1 = r.y * a01 + r.x * a11;
        a00 = r.x * x0 - r.y * x1;
        a01 = r.y * x0 + r.x * x1;
        a11 = r.y * y0 + r.x * y1;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const double x = v0[j], y = v1[j];
            v0[j] = r.x * x - r.y * y;
            v1[j] = r.y * x + r.x * y;
        }
    }
    const int at0 = a11 >= a00 ? 1 : 0, at1 = 1 - at0;   // decreasing, ties by index
    eigvals[at0] = (float)a00;
    eigvals[at1] = (float)a11;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        p[j * ldp + at0] = (float)v0[j];
        p[j * ldp + at1] = (float)v1[j];
    }
}

// blocks (k, l), k < l: lanes of `units` rows of n / 2 (see below)
__host__ __device__ inline int eig_small_units(int half) { return (half + 1) >> 1; }
// doubles of one of the two buffers: the four planes, the diagonal blocks (three numbers each)
// and a place that nothing reads; even, so that what lies behind is 16-byte aligned
__host__ __device__ inline int eig_small_buf(int half) { return 4 * eig_small_units(half) * half + 3 * half + (half & 1) + 2; }
// bytes of LDS: both buffers, both buffers of the Vt slice [n][kEigSmallCols], cosines and sines of two rounds, two flags
__host__ __device__ inline int eig_small_lds_bytes(int n) {
    return (2 * eig_small_buf(n / 2) + 2 * n * kEigSmallCols + 2 * n) * (int)sizeof(double) + 2 * (int)sizeof(int);
}

__global__ __launch_bounds__(kEigSmallThreads) void eig_small_kernel(const float* __restrict__ c, int64_t ldc, int n,
                                                                     int sweeps, float* __restrict__ eigvals,
                                                                     float* __restrict__ p, int64_t ldp) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    const int half = n >> 1, units = eig_small_units(half), plane = units * half, bufsz = eig_small_buf(half);
    const int diag = 4 * plane;                        // a00[half], a11[half], a01[half] of the pairs
    double* vt = lds + 2 * bufsz;                      // [2][n][kEigSmallCols]: columns of Vt from j0 on, rows by slot: half x + k
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
        vt[idx] = index_of(s0 % half, s0 / half) == j0 + idx % kEigSmallCols ? 1.0 : 0.0;
    }

    // wavefronts 1 .. 15: this thread's blocks (two rows of units, a third one on the first two), their places and
    // where their four elements go (what goes to a diagonal block is wavefront 0's to write)
    constexpr int kWaves = kEigSmallThreads / 64;
    const int unused = bufsz - 1;
    bool on[3], row_on[3];   // row_on: for the whole wavefront
    int bk[3], bl[3], rd[3], wr[3][4];
#pragma unroll
    for (int h = 0; h < 3; ++h) {
        const int u = wave - 1 + h * (kWaves - 1);
        const bool upper = lane > u;
        // not the diagonal, and not the lower lanes of the middle row of an odd number of pairs
        row_on[h] = wave > 0 && u < units;
        on[h] = row_on[h] && lane < half && lane != u && (upper || 2 * u != half - 1);
        bk[h] = on[h] ? (upper ? u : half - 1 - u) : 0;
        bl[h] = on[h] ? (upper ? lane : half - 1 - lane) : 0;
        rd[h] = row_on[h] && lane < half ? u * half + lane : 0;   // lanes without a block compute for nobody
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int k = bk[h], x = e >> 1, l = bl[h], y = e & 1;
            move(k, x);
            move(l, y);
            wr[h][e] = on[h] && k != l ? at(k, x, l, y) : unused;
        }
    }
    // Wavefront 0, lane k, in the same registers: the slots that the elements in slots (k, 0) and (k, 1) come from, bk[0], rd[0]
    // and bl[0], rd[1], the block that they share, wr[0], and where the off-diagonal element of lane k's own diagonal block goes, wr[1][0].
    const bool lk_on = lane < half;
    if (wave == 0) {
        auto from = [&](int& k, int& x) {
            if (half == 1 || (k == 0 && x == 0)) return;
            if (x == 0) {
                if (k < half - 1) ++k;
                else x = 1;
            } else {
                if (k == 0) { k = 1; x = 0; }
                else --k;
            }
        };
        const int own = lk_on ? lane : 0;
        int k0 = own, x0 = 0, k1 = own, x1 = 1;
        from(k0, x0);
        from(k1, x1);
        bk[0] = k0;
        rd[0] = x0;
        bl[0] = k1;
        rd[1] = x1;
#pragma unroll
        for (int e = 0; e < 4; ++e) wr[0][e] = at(k0, e >> 1, k1, e & 1);
        k0 = k1 = own;
        x0 = 0;
        x1 = 1;
        move(k0, x0);
        move(k1, x1);
        wr[1][0] = lk_on && half > 1 ? at(k0, x0, k1, x1) : unused;
    }
    // wavefronts 8 and 9, the first n threads: two rows of one column of Vt
    const int vk = (t - kEigSmallThreads / 2) / kEigSmallCols, vc = t & (kEigSmallCols - 1);
    const bool v_on = wave >= kWaves / 2 && vk < half;
    int vw[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        int k = v_on ? vk : 0, y = x;
        move(k, y);
        vw[x] = (half * y + k) * kEigSmallCols + vc;
    }
    __syncthreads();

    // the rotation of the pair whose diagonal block is (a00, a01; a01, a11), for the round that reads buffer b
    auto angle = [&](double a00, double a11, double a01, int b) __attribute__((always_inline)) {
        double2 r = make_double2(1.0, 0.0);
        const bool turn = lk_on && eig_turns(a00, a11, a01);
        if (turn) r = eig_rotation(a00, a11, a01);
        if (lk_on) cs[b * half + lane] = r;
        const bool any = __ballot(turn) != 0;
        if (lane == 0) flag[b] = any ? 1 : 0;
    };
    if (wave == 0) angle(lds[diag + lk_on * lane], lds[diag + half + lk_on * lane], lds[diag + 2 * half + lk_on * lane], 0);
    __syncthreads();
    // One round, from buffer B, known to the compiler (every access cost an index sum before), into the other.
    auto one_round = [&](auto buf_) __attribute__((always_inline)) {
        constexpr int B = decltype(buf_)::value;
        const double* cur = lds + B * bufsz;
        double* nxt = lds + (B ^ 1) * bufsz;
        const double2* rot = cs + B * half;
        if (wave == 0) {
            // the diagonal blocks of the next round, and its angles
            const int lk0 = bk[0], lk1 = bl[0];
            const bool lx0 = rd[0] != 0, lx1 = rd[1] != 0;
            const double2 r0 = rot[lk0], r1 = rot[lk1];
            const double p00 = cur[diag + lk0], p11 = cur[diag + half + lk0], p01 = cur[diag + 2 * half + lk0];
            const double q00 = cur[diag + lk1], q11 = cur[diag + half + lk1], q01 = cur[diag + 2 * half + lk1];
            const double e00 = cur[wr[0][0]], e01 = cur[wr[0][1]], e10 = cur[wr[0][2]], e11 = cur[wr[0][3]];
            // row x of the rotation: new = f old_0 + g old_1
            const double f0 = lx0 ? r0.y : r0.x, g0 = lx0 ? r0.x : -r0.y;
            const double f1 = lx1 ? r1.y : r1.x, g1 = lx1 ? r1.x : -r1.y;
            const double a00 = f0 * (f0 * p00 + g0 * p01) + g0 * (f0 * p01 + g0 * p11);
            const double a11 = f1 * (f1 * q00 + g1 * q01) + g1 * (f1 * q01 + g1 * q11);
            double a01;
            if (half == 1) a01 = f1 * (f0 * p00 + g0 * p01) + g1 * (f0 * p01 + g0 * p11);
            else a01 = f1 * (f0 * e00 + g0 * e10) + g1 * (f0 * e01 + g0 * e11);
            if (lk_on) {
                nxt[diag + lane] = a00;
                nxt[diag + half + lane] = a11;
                nxt[diag + 2 * half + lane] = a01;
            }
            angle(a00, a11, a01, B ^ 1);
            const int own = lk_on ? lane : 0;
            const double2 r = rot[own];
            const double o00 = cur[diag + own], o11 = cur[diag + half + own], o01 = cur[diag + 2 * half + own];
            nxt[wr[1][0]] = r.y * (r.x * o00 - r.y * o01) + r.x * (r.x * o01 - r.y * o11);
        } else {
#pragma unroll
            for (int h = 0; h < 3; ++h) {
                if (!row_on[h]) continue;
                const double* at = cur + rd[h];
                const double2 ra = rot[bk[h]], rb = rot[bl[h]];
                const double2 x0 = make_double2(at[0], at[plane]), x1 = make_double2(at[2 * plane], at[3 * plane]);
                const double y00 = ra.x * x0.x - ra.y * x1.x, y10 = ra.y * x0.x + ra.x * x1.x;
                const double y01 = ra.x * x0.y - ra.y * x1.y, y11 = ra.y * x0.y + ra.x * x1.y;
                nxt[wr[h][0]] = rb.x * y00 - rb.y * y01;
                nxt[wr[h][1]] = rb.y * y00 + rb.x * y01;
                nxt[wr[h][2]] = rb.x * y10 - rb.y * y11;
                nxt[wr[h][3]] = rb.y * y10 + rb.x * y11;
            }
            if (v_on) {   // Vt <- J^T Vt
                const double* src = vt + B * n * kEigSmallCols + vk * kEigSmallCols + vc;
                double* dst = vt + (B ^ 1) * n * kEigSmallCols;
                const double2 r = rot[vk];
                const double x = src[0], y = src[half * kEigSmallCols];
                dst[vw[0]] = r.x * x - r.y * y;
                dst[vw[1]] = r.y * x + r.x * y;
            }
        }
    };
    int buf = 0, rotated = 0, round = 0;
    for (int sweep = 0;;) {
        // true when the iteration is over
        auto step = [&](auto buf_) __attribute__((always_inline)) {
            constexpr int B = decltype(buf_)::value;
            rotated |= __builtin_amdgcn_readfirstlane(flag[B]);
            one_round(buf_);
            __syncthreads();
            buf = B ^ 1;
            if (++round < n - 1) return false;
            const bool over = !rotated || ++sweep == sweeps;  // a sweep that turned nothing: as every later one would
            round = rotated = 0;
            return over;
        };
        if (step(std::integral_constant<int, 0>{})) break;
        if (step(std::integral_constant<int, 1>{})) break;
    }
    // positions in decreasing order (ties by index), as eig_finish_kernel has them; rank by slot
    const double* a = lds + buf * bufsz + diag;
    vt += buf * n * kEigSmallCols;
    int* rank = reinterpret_cast<int*>(cs + buf * half);   // no rotation is read any more
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
        p[(int64_t)(j0 + col) * ldp + rank[s]] = (float)vt[((s & 1) * half + (s >> 1)) * kEigSmallCols + col];
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
