"""GPU parity of the offline basis construction (Section 4.2) against its oracle, through the C ABI.

Floating point: the Gram matrix and the projections accumulate exact bf16/fp32 products in
fp32, so they are compared with the fp64 oracle at a tolerance derived from the length of the
sum; eigenvalues are unique and compared directly; eigenvectors are unique only up to sign
and, inside clusters, up to a rotation, so what is compared is the projector onto the top-r
subspace (unique when the r-th gap is open) and the rest is checked for validity (orthonormal,
small residual).
"""
import numpy as np
import pytest
import torch

from oracle import resq_basis_oracle as bo
from paper_2412_14363_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rq():
    from paper_2412_14363_amd import binding
    binding.lib()
    return binding


def calib(seed, T, K, outliers=6):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(T, K, generator=g)
    cols = torch.randperm(K, generator=g)[:outliers]
    x[:, cols] *= 20.0
    return x.to(torch.bfloat16)


@pytest.mark.parametrize("T,K", [(300, 128), (1000, 256), (77, 8), (4096, 520), (5000, 64), (16, 1024)])
def test_gram_accumulate(rq, T, K):
    x = calib(T + K, T, K)
    ref = bo.gram(x.double().numpy())
    c = rq.resq_gram_accumulate(x.cuda())
    torch.cuda.synchronize()
    got = c.double().cpu().numpy()
    # fp32 accumulation of T exact products: error <= T * 2^-24 * sum |x_i x_j|, far below this
    bound = 4 * T * 2.0 ** -24 * (np.abs(x.double().numpy()).T @ np.abs(x.double().numpy())) + 1e-30
    assert np.all(np.abs(got - ref) <= bound)
    # accumulates: a second call with other tokens adds
    x2 = calib(T + K + 1, 130, K)
    rq.resq_gram_accumulate(x2.cuda(), c)
    torch.cuda.synchronize()
    ref2 = ref + bo.gram(x2.double().numpy())
    assert np.allclose(c.double().cpu().numpy(), ref2, rtol=1e-4, atol=1e-4 * np.abs(ref2).max())


def test_gram_strided_rows_and_untouched_padding(rq):
    T, K = 200, 72
    buf = torch.randn(T, K + 24).to(torch.bfloat16)
    cbuf = torch.full((K, K + 8), 7.0, dtype=torch.float32, device="cuda")
    cbuf[:, :K] = 0
    rq.resq_gram_accumulate(buf.cuda()[:, :K], cbuf[:, :K])
    torch.cuda.synchronize()
    assert torch.all(cbuf[:, K:] == 7.0)
    assert np.allclose(cbuf[:, :K].double().cpu().numpy(), bo.gram(buf[:, :K].double().numpy()), rtol=1e-4, atol=1e-3)


@pytest.mark.parametrize("rows,K,J,a_dtype,out_dtype", [
    (300, 128, 128, torch.bfloat16, torch.bfloat16), (130, 256, 64, torch.float32, torch.float32),
    (7, 72, 8, torch.bfloat16, torch.float32), (257, 1000, 264, torch.float32, torch.bfloat16),
    (1, 16, 16, torch.float32, torch.float32),
])
def test_project_rows(rq, rows, K, J, a_dtype, out_dtype):
    g = torch.Generator().manual_seed(rows + K + J)
    a = torch.randn(rows, K, generator=g).to(a_dtype)
    u = torch.randn(K, J, generator=g) / K ** 0.5
    ref = bo.project(a.double().numpy(), u.double().numpy())
    out = rq.resq_project_rows(a.cuda(), u.cuda(), out_dtype=out_dtype)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    mag = np.abs(a.double().numpy()) @ np.abs(u.double().numpy())
    if out_dtype == torch.bfloat16:
        # fp32 result rounded once more to bf16
        assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 4 * K * 2.0 ** -24 * mag)
    else:
        assert np.all(np.abs(got - ref) <= 4 * K * 2.0 ** -24 * mag + 1e-30)


# bf16 rows go through the bf16 matrix cores with u in three exact parts: edges of the 128 x 128
# tiles and of the 32 steps of a chunk; rows of at most 16 steps through the fp32 ones
@pytest.mark.parametrize("rows,K,J", [(1, 1, 8), (129, 16, 136), (130, 15, 8), (40, 17, 264), (128, 32, 128), (129, 33, 136), (127, 31, 120), (40, 64, 1000), (300, 515, 16)])
def test_project_rows_split(rq, rows, K, J):
    g = torch.Generator().manual_seed(rows + K + J)
    ld = (K + 7) // 8 * 8 + 8
    a = torch.full((rows, ld), float("nan"), dtype=torch.bfloat16)   # what lies behind a row is not read
    a[:, :K] = torch.randn(rows, K, generator=g).bfloat16()
    # parts of very different size, exact zeros and bf16 numbers among them
    u = torch.randn(K, J, generator=g) * torch.exp2(torch.randint(-40, 10, (K, J), generator=g).float())
    u[::3] = u[::3].bfloat16().float()
    u[1::5] = 0.0
    buf = torch.full((rows, J + 3), 7.0, device="cuda")
    rq.resq_project_rows(a.cuda()[:, :K], u.cuda(), out=buf[:, :J])
    torch.cuda.synchronize()
    ad, ud = a[:, :K].double().numpy(), u.double().numpy()
    assert torch.all(buf[:, J:] == 7.0)
    # products are exact; 3 K additions in fp32
    assert np.all(np.abs(buf[:, :J].double().cpu().numpy() - ad @ ud) <= 3 * K * 2.0 ** -24 * (np.abs(ad) @ np.abs(ud)) + 1e-30)


# 256 x 128 tiles (kernel 2): ragged rows and columns, a reduction axis of less than a chunk, of whole chunks, with one to
# three pieces of a last one, through the loop and without it; beside them what the smaller tiles (1) keep: one tile less, a
# ragged piece, rounds that would be emptier
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,K,J,kernel", [
    (16380, 24, 1032, 2), (16129, 32, 1032, 1), (16129, 32, 1024, 2), (16385, 40, 1000, 2), (130817, 56, 128, 2), (130816, 56, 128, 1),
    (16300, 64, 1032, 1), (16300, 64, 1016, 2), (16300, 96, 1016, 2), (16300, 128, 1024, 2), (16300, 160, 1032, 1), (16300, 160, 1024, 2),
    (16300, 168, 1032, 2), (16300, 232, 1032, 2), (16300, 161, 1032, 1)])
def test_project_rows_wide_tiles(rq, rows, K, J, kernel, out_dtype):
    g = torch.Generator(device="cuda").manual_seed(rows + K + J)
    ld = (K + 7) // 8 * 8 + 8
    a = torch.full((rows, ld), float("nan"), dtype=torch.bfloat16, device="cuda")   # what lies behind a row is not read
    a[:, :K] = torch.randn(rows, K, generator=g, device="cuda").bfloat16()
    u = torch.randn(K, J, generator=g, device="cuda") * torch.exp2(torch.randint(-40, 10, (K, J), generator=g, device="cuda").float())
    u[::3] = u[::3].bfloat16().float()
    buf = torch.full((rows, J + 3), 7.0, device="cuda", dtype=out_dtype)
    assert rq.resq_project_rows_plan(a[:, :K], u, buf[:, :J]) == kernel
    rq.resq_project_rows(a[:, :K], u, out=buf[:, :J])
    ad, ud = a[:, :K].double(), u.double()
    ref, mag = ad @ ud, ad.abs() @ ud.abs()
    assert torch.all(buf[:, J:] == 7.0)
    # products are exact; 3 K additions in fp32, one rounding of the output
    tol = 3 * K * 2.0 ** -24 * mag + (2.0 ** -8 * ref.abs() if out_dtype == torch.bfloat16 else 0) + 1e-30
    assert torch.all((buf[:, :J].double() - ref).abs() <= tol)


def test_project_rows_wide_tiles_infinities_and_in_place(rq):
    rows, K, J, inf, nan = 131072, 72, 128, float("inf"), float("nan")
    g = torch.Generator(device="cuda").manual_seed(9)
    a = torch.randn(rows, 128, generator=g, device="cuda").bfloat16()
    u = torch.randn(K, J, generator=g, device="cuda")
    u[:, ::2] = u[:, ::2].bfloat16().float()   # two of the three parts are zero
    a[0, 3], a[300, K - 1], a[5000, 2], a[5000, 9], a[131071, 1] = inf, -inf, inf, -inf, nan
    u[K - 6, 4], u[K - 1, 7] = inf, nan
    ref = a[:, :K].double() @ u.double()
    for out_dtype in (torch.float32, torch.bfloat16):
        got = torch.empty((rows, J), dtype=out_dtype, device="cuda")
        assert rq.resq_project_rows_plan(a[:, :K], u, got) == 2
        rq.resq_project_rows(a[:, :K], u, out=got)
        assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got.isinf(), ref.isinf())
        assert torch.equal(got[ref.isinf()].double(), ref[ref.isinf()])
        fin = ref.isfinite()
        assert torch.allclose(got[fin].double(), ref[fin], rtol=2.0 ** -8, atol=1e-4)
    want = rq.resq_project_rows(a[:, :K], u, out_dtype=torch.bfloat16)
    buf = a.clone()
    assert rq.resq_project_rows_plan(buf[:, :K], u, buf) == 1
    rq.resq_project_rows(buf[:, :K], u, out=buf)   # the smaller tiles, another order of the sum
    assert torch.equal(buf.isnan(), want.isnan())
    assert torch.allclose(buf[want.isfinite()].double(), want[want.isfinite()].double(), rtol=2.0 ** -7, atol=1e-4)


# Operands that are column blocks, out in the columns beside a's: the bits of contiguous copies, from the same kernel
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("rows,K,J", [(131072, 72, 128), (131000, 136, 120), (66000, 264, 256)])
def test_project_rows_wide_tiles_on_column_blocks(rq, rows, K, J, out_dtype):
    g = torch.Generator(device="cuda").manual_seed(rows + K)
    per = 2 if out_dtype == torch.float32 else 1   # bf16 columns that an output takes
    buf = torch.randn(rows, K + 16 + J * per + 8, generator=g, device="cuda").bfloat16()
    u_buf = torch.randn(K, J + 24, generator=g, device="cuda")
    a, u = buf[:, 8:8 + K], u_buf[:, 16:16 + J]
    out = buf.view(out_dtype)[:, (K + 16) // per:(K + 16) // per + J]
    assert rq.resq_project_rows_plan(a, u, out) == 2
    a_copy, u_copy = a.contiguous(), u.contiguous()
    want = torch.empty((rows, J), dtype=out_dtype, device="cuda")
    assert rq.resq_project_rows_plan(a_copy, u_copy, want) == 2
    rq.resq_project_rows(a_copy, u_copy, out=want)
    before = buf.clone()
    rq.resq_project_rows(a, u, out=out)
    assert torch.equal(out, want)
    out.copy_(before.view(out_dtype)[:, (K + 16) // per:(K + 16) // per + J])
    assert torch.equal(buf.view(torch.int16), before.view(torch.int16))   # nothing beside out


# Infinities and NaN in either operand: what a plain sum gives, not the NaN that infinity x 0 among the three
# parts of u would leave (bf16 numbers have two zero parts).
@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("K", [70, 16])
def test_project_rows_split_infinities(rq, out_dtype, K):
    rows, J = 131, 136
    g = torch.Generator().manual_seed(5)
    a = torch.randn(rows, K, generator=g).bfloat16()
    u = torch.randn(K, J, generator=g)
    u[:, ::2] = u[:, ::2].bfloat16().float()
    inf, nan = float("inf"), float("nan")
    a[0, 3], a[5, K - 10], a[130, K - 1], a[7, 2], a[7, 9], a[9, 1], a[11, 5] = inf, -inf, inf, inf, -inf, nan, 0.0
    u[K - 6, 4], u[5, 7], u[2, 135], u[3, 8] = inf, -inf, inf, 0.0
    ld = (K + 7) // 8 * 8
    ad = torch.zeros(rows, ld, dtype=torch.bfloat16)
    ad[:, :K] = a
    got = rq.resq_project_rows(ad.cuda()[:, :K], u.cuda(), out_dtype=out_dtype).cpu().double().numpy()
    with np.errstate(invalid="ignore"):
        ref = a.double().numpy() @ u.double().numpy()
    assert np.isinf(ref).sum() > 500 and np.isnan(ref).sum() > 100
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    mag = np.abs(np.nan_to_num(a.double().numpy(), posinf=0, neginf=0)) @ np.abs(np.nan_to_num(u.double().numpy(), posinf=0, neginf=0))
    tol = 3 * K * 2.0 ** -24 * mag + (2.0 ** -8 * np.abs(np.where(fin, ref, 0)) if out_dtype == torch.bfloat16 else 0)
    assert np.all(np.abs(got[fin] - ref[fin]) <= tol[fin])
    if out_dtype == torch.bfloat16 and K >= 64:   # out on a: one column of tiles, so that rows stay a workgroup's own
        buf = ad.cuda()
        rq.resq_project_rows(buf[:, :K], u[:, :64].contiguous().cuda(), out=buf[:, :64])
        assert np.array_equal(buf[:, :64].cpu().double().numpy(), got[:, :64], equal_nan=True)


# Entries of u so small that their third part falls under the smallest bf16 subnormal, 2^-133
def test_project_rows_split_tiny_basis(rq):
    rows, K, J = 40, 96, 64
    g = torch.Generator().manual_seed(6)
    a = (torch.randn(rows, K, generator=g) * 2.0 ** 60).bfloat16()
    u = torch.randn(K, J, generator=g) * torch.exp2(torch.randint(-130, -105, (K, J), generator=g).float())
    got = rq.resq_project_rows(a.cuda(), u.cuda(), out_dtype=torch.float32).cpu().double().numpy()
    ad, ud = a.double().numpy(), u.double().numpy()
    tol = 3 * K * 2.0 ** -24 * (np.abs(ad) @ np.abs(ud)) + 2.0 ** -133 * np.abs(ad).sum(1, keepdims=True)
    assert np.all(np.abs(got - ad @ ud) <= tol)


def test_project_rows_on_column_blocks(rq):
    # U_h = P_h R_h written into the first r columns of U: sub-blocks in and out
    K, r = 64, 16
    p = wl.random_orthogonal(K, 3).contiguous().cuda()
    r_h = wl.random_orthogonal(r, 4).contiguous().cuda()
    u = torch.zeros(K, K, device="cuda")
    rq.resq_project_rows(p[:, :r], r_h, out=u[:, :r])
    torch.cuda.synchronize()
    assert torch.all(u[:, r:] == 0)
    assert np.allclose(u[:, :r].double().cpu().numpy(),
                       p[:, :r].double().cpu().numpy() @ r_h.double().cpu().numpy(), atol=1e-6)


@pytest.mark.parametrize("K,r", [(8, 2), (64, 8), (128, 16), (256, 32),
                                 (1024, 128),      # a hidden-size basis of a small model
                                 (4608, 576)])     # two rows of this order need more than 64 KiB of LDS
def test_sym_eig_against_oracle(rq, K, r):
    # planted spectrum with an open gap after the r-th eigenvalue
    sig = np.concatenate([np.linspace(30.0, 20.0, r), np.linspace(4.0, 0.5, K - r)])
    q = wl.random_orthogonal(K, K).double().numpy()
    c = (q * sig ** 2) @ q.T
    c32 = torch.tensor(c, dtype=torch.float32)
    lam_ref, p_ref = bo.pca_basis(c32.double().numpy())
    lam, p = rq.resq_sym_eig(c32.cuda(), sweeps=10 if K <= 256 else 14)
    torch.cuda.synchronize()
    lam, p = lam.double().cpu().numpy(), p.double().cpu().numpy()
    scale = lam_ref[0]
    assert np.all(np.diff(lam) <= 0)
    assert np.allclose(lam, lam_ref, atol=1e-6 * scale)          # fp32 outputs of an fp64 iteration
    assert np.allclose(p.T @ p, np.eye(K), atol=1e-5)             # orthonormal columns
    # eigenpairs of the input; the fp32 rounding of the K entries of a vector adds up in c @ p
    assert np.abs(c32.double().numpy() @ p - p * lam).max() <= (1e-5 if K <= 256 else 4e-5) * scale
    # the high-precision subspace is the oracle's
    assert np.allclose(p[:, :r] @ p[:, :r].T, p_ref[:, :r] @ p_ref[:, :r].T, atol=1e-4)


# order 2, a kernel of its own: nothing to turn, equal values, either order, either sign, an element far below the others
@pytest.mark.parametrize("c", [[[3., 0.], [0., 1.]], [[1., 0.], [0., 3.]], [[2., 0.], [0., 2.]], [[2., 1.], [1., 2.]], [[2., -1.], [-1., 2.]],
                               [[0., 0.], [0., 0.]], [[0., 5.], [5., 0.]], [[-4., 1.], [1., -7.]], [[1e-20, 1e-21], [1e-21, 3e-20]],
                               [[1e30, 1e18], [1e18, 1.]], [[1., 1e-8], [1e-8, 1.]], [[1., 1e-5], [2e-5, 1e-9]]])
@pytest.mark.parametrize("sweeps", [1, 12])
def test_sym_eig_order_two(rq, c, sweeps):
    buf = torch.full((2, 5), 7.0, device="cuda")
    buf[:, :2] = torch.tensor(c)
    lam, p = (t.double().cpu().numpy() for t in rq.resq_sym_eig(buf[:, :2], sweeps=sweeps))
    m = buf[:, :2].double().cpu().numpy()
    m = 0.5 * (m + m.T)
    scale = np.abs(m).max()
    # fp32 outputs of an fp64 iteration, which one rotation ends
    assert lam[0] >= lam[1] and np.all(np.abs(lam - np.linalg.eigvalsh(m)[::-1]) <= 2.0 ** -23 * scale)
    assert np.allclose(p.T @ p, np.eye(2), atol=2.0 ** -22)
    assert np.all(np.abs(m @ p - p * lam) <= 2.0 ** -21 * scale)


# orders that take the single-launch kernel (at most 128): the smallest, odd and even numbers of
# pairs, the largest, and the first order beyond it
@pytest.mark.parametrize("K", [2, 4, 6, 18, 30, 32, 62, 98, 122, 126, 128, 130])
def test_sym_eig_small_orders(rq, K):
    g = torch.Generator().manual_seed(K)
    x = torch.randn(2 * K + 3, K, generator=g, dtype=torch.float64) * torch.exp(-3.0 * torch.arange(K) / K)
    c = torch.zeros(K, K + 8)
    c[:, :K] = (x.T @ x).float()
    buf = torch.full((K, K + 3), 7.0, device="cuda")
    lam, p = torch.empty(K, device="cuda"), buf[:, :K]
    rq.resq_sym_eig_static(c.cuda()[:, :K], lam, p)
    torch.cuda.synchronize()
    c64 = c[:, :K].double().numpy()
    lam_ref = np.linalg.eigvalsh(c64)[::-1]
    lam, p = lam.double().cpu().numpy(), p.double().cpu().numpy()
    assert torch.all(buf[:, K:] == 7.0)
    # fp32 outputs of an fp64 iteration: half an fp32 step of the largest value, of each entry of a vector
    assert np.abs(lam - lam_ref).max() <= 1e-7 * lam_ref[0]
    assert np.allclose(p.T @ p, np.eye(K), atol=1e-6)
    assert np.abs(c64 @ p - p * lam).max() <= 1e-6 * lam_ref[0]


# zero eigenvalues (fewer rows than columns), and entries at both ends of fp32: squares and products far out of its range
@pytest.mark.parametrize("K", [4, 34, 128])
@pytest.mark.parametrize("scale", [2.0 ** -110, 1.0, 2.0 ** 110])
def test_sym_eig_small_orders_rank_and_scale(rq, K, scale):
    g = torch.Generator().manual_seed(K)
    x = torch.randn(K // 2 + 1, K, generator=g, dtype=torch.float64)
    c = (x.T @ x * scale).float()
    lam, p = (t.double().cpu().numpy() for t in rq.resq_sym_eig(c.cuda()))
    c64 = c.double().numpy()
    lam_ref = np.linalg.eigvalsh(c64 / scale)[::-1] * scale
    assert np.abs(lam - lam_ref).max() <= 1e-7 * lam_ref[0]      # the bounds of the test above
    assert np.allclose(p.T @ p, np.eye(K), atol=1e-6)
    assert np.abs(c64 @ p - p * lam).max() <= 1e-6 * lam_ref[0]


# A NaN on the diagonal turns no pair: at order 2 the other value and both vectors come out; in larger matrices it
# reaches every value (but no angle), so all share the first place, and what is written of the vectors is finite.
@pytest.mark.parametrize("K,at", [(2, 0), (2, 1), (4, 0), (34, 33), (128, 64)])
def test_sym_eig_nan_on_the_diagonal(rq, K, at):
    g = torch.Generator().manual_seed(K + at)
    x = torch.randn(2 * K + 3, K, generator=g, dtype=torch.float64)
    c = (x.T @ x).float()
    c[at, at] = float("nan")
    lam, p = torch.full((K,), 7.0, device="cuda"), torch.full((K, K), 7.0, device="cuda")
    rq.resq_sym_eig_static(c.cuda(), lam, p)
    lam, p = lam.cpu(), p.cpu()
    assert int(lam.isnan().sum()) == 1 and not p.isnan().any()
    if K == 2:
        assert torch.equal(lam[~lam.isnan()], c[1 - at, 1 - at].reshape(1))
        assert torch.equal(p.abs().sum(0), torch.ones(2)) and torch.equal(p.abs().sum(1), torch.ones(2))


# Outputs on the memory of c, at orders on both sides of the single-launch kernel's limit.  Its workgroups do not
# wait for each other, so such calls go through the workspace, which they leave written.
@pytest.mark.parametrize("K", [2, 8, 10, 64, 126, 128, 130])
def test_sym_eig_in_place(rq, K):
    g = torch.Generator().manual_seed(K)
    x = torch.randn(2 * K + 3, K, generator=g, dtype=torch.float64) * torch.exp(-3.0 * torch.arange(K) / K)
    c0 = (x.T @ x).float()
    c64 = c0.double().numpy()
    lam_ref = np.linalg.eigvalsh(c64)[::-1]
    L, st = rq.lib(), torch.cuda.current_stream().cuda_stream
    nbytes = L.resq_sym_eig_workspace_bytes(K)

    def call(c, lam, p, through_workspace):
        work = torch.full((nbytes,), 0xA5, dtype=torch.uint8, device="cuda")
        rc = L.resq_sym_eig(c.data_ptr(), c.stride(0), K, 12, lam.data_ptr(), p.data_ptr(), p.stride(0), work.data_ptr(), nbytes, st)
        assert rc == 0, rq.STATUS_NAMES.get(rc, rc)
        torch.cuda.synchronize()
        assert bool((work != 0xA5).any()) == through_workspace
        ld, pd = lam.double().cpu().numpy(), p.double().cpu().numpy()
        assert np.abs(ld - lam_ref).max() <= 1e-7 * lam_ref[0]
        assert np.allclose(pd.T @ pd, np.eye(K), atol=1e-6)
        assert np.abs(c64 @ pd - pd * ld).max() <= 1e-6 * lam_ref[0]

    def buffers(rows, cols):
        return torch.full((rows, cols), 7.0, device="cuda")

    c, lam = buffers(K, K), torch.empty(K, device="cuda")
    c.copy_(c0)
    call(c, lam, c, True)                                          # p on c
    wide = buffers(K, K + 6)
    wide[:, :K].copy_(c0)
    call(wide[:, :K], lam, wide[:, 1:K + 1], True)                 # ... shifted by a column
    both = buffers(2 * K, K + 2)
    both[:K, :K].copy_(c0)
    call(both[:K, :K], lam, both[K - 1:2 * K - 1, :K], True)       # ... p begins in c's last row
    c.copy_(c0)
    call(c, c.view(-1)[:K], buffers(K, K), True)                   # eigenvalues on c
    pair = buffers(K, 2 * K)
    pair[:, K:].copy_(c0)
    call(pair[:, K:], lam, pair[:, :K], K > 128)                   # column blocks of one matrix: separate
    assert torch.equal(pair[:, K:].cpu(), c0)
    if K <= 512:
        c.copy_(c0)
        rq.resq_sym_eig_static(c, lam, c)
        torch.cuda.synchronize()
        pd = c.double().cpu().numpy()
        assert np.abs(c64 @ pd - pd * lam.double().cpu().numpy()).max() <= 1e-6 * lam_ref[0]


def test_sym_eig_small_orders_without_rotations(rq):
    # nothing to rotate, singular and indefinite input
    lam, p = rq.resq_sym_eig(torch.zeros(64, 64, device="cuda"))
    assert torch.all(lam == 0) and torch.equal(p, torch.eye(64, device="cuda"))
    one = torch.ones(16, 16)
    one[0, 0] = -3.0
    lam, p = rq.resq_sym_eig(one.cuda())
    torch.cuda.synchronize()
    ref = np.linalg.eigvalsh(one.double().numpy())[::-1]
    assert np.allclose(lam.double().cpu().numpy(), ref, atol=2e-6)
    pd = p.double().cpu().numpy()
    assert np.allclose(pd @ np.diag(ref) @ pd.T, one.numpy(), atol=1e-5)


def test_sym_eig_repeated_eigenvalues_and_diagonal_input(rq):
    # a matrix that is already diagonal with a repeated value: sorted, vectors a permutation
    d = np.array([3.0, 1.0, 3.0, 2.0, 0.0, 5.0, 1.0, 4.0])
    lam, p = rq.resq_sym_eig(torch.tensor(np.diag(d), dtype=torch.float32).cuda(), sweeps=3)
    torch.cuda.synchronize()
    assert np.array_equal(lam.cpu().numpy(), np.sort(d)[::-1].astype(np.float32))
    pp = p.double().cpu().numpy()
    assert np.allclose(pp.T @ pp, np.eye(8), atol=1e-12) and np.allclose(np.abs(pp).sum(0), 1.0)


def test_basis_end_to_end_raises_layer_snr(rq):
    # the whole offline path on the GPU (Gram matrix, PCA, U = P blockdiag(R), X U, W U), then
    # the layer on the projected operands: the output SNR against the unprojected fp64 product
    # must equal what the oracle's basis gives, and beat quantizing the raw operands
    from oracle import resq_oracle as oracle
    oracle.build()
    K, N, T, r = 128, 96, 512, 16
    x = calib(5, T, K)
    g = torch.Generator().manual_seed(6)
    w = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16)
    r_h, r_l = wl.random_orthogonal(r, 1).contiguous(), wl.random_orthogonal(K - r, 2).contiguous()
    xd, wd = x.cuda(), w.cuda()
    c = rq.resq_gram_accumulate(xd)
    lam, p = rq.resq_sym_eig(c, sweeps=10)
    u = torch.empty(K, K, device="cuda")
    rq.resq_project_rows(p[:, :r], r_h.cuda(), out=u[:, :r])
    rq.resq_project_rows(p[:, r:], r_l.cuda(), out=u[:, r:])
    xr = rq.resq_project_rows(xd, u)
    wr = rq.resq_project_rows(wd, u)
    y = rq.resq_gemm_mixed(rq.resq_quantize_act(xr, r), rq.resq_pack_weights(wr, r), N)
    torch.cuda.synchronize()
    un = u.double().cpu().numpy()
    assert np.allclose(un.T @ un, np.eye(K), atol=1e-5)
    ref = x.double().numpy() @ w.double().numpy().T
    snr_gpu = oracle.snr_db(ref, y.float().cpu().numpy())
    # the oracle's own path
    _, p_o = bo.pca_basis(bo.gram(x.double().numpy()))
    u_o = bo.compose_basis(p_o, r_h.double().numpy(), r_l.double().numpy())
    xo = bo.f64_to_bf16_bits(bo.project(x.double().numpy(), u_o))
    wo = bo.f64_to_bf16_bits(bo.project(w.double().numpy(), u_o))
    snr_cpu = oracle.snr_db(ref, oracle.linear(xo, wo, r).y)
    snr_raw = oracle.snr_db(ref, oracle.linear(wl.bf16_bits(x), wl.bf16_bits(w), r).y)
    # eigenvector signs differ, so codes differ: the SNRs agree statistically, not bitwise
    assert abs(snr_gpu - snr_cpu) < 1.0, (snr_gpu, snr_cpu)
    assert snr_gpu > snr_raw + 6.0, (snr_gpu, snr_raw)
    # the span of the high group is the oracle's
    ph = p[:, :r].double().cpu().numpy()
    assert np.allclose(ph @ ph.T, p_o[:, :r] @ p_o[:, :r].T, atol=1e-3)
