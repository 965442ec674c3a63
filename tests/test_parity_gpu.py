"""GPU parity: every step of the HIP path against the CPU oracle, through the
C ABI, on the same seeded inputs.  Integer codes, scales and int32
accumulators must match bit for bit; bf16 outputs within 1e-2 relative."""
import numpy as np
import pytest
import torch

from paper_2412_14363_amd import workloads as wl
from parity_util import REL_TOL, y_within_tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rq():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU; there is no CPU fallback")
    from paper_2412_14363_amd import binding
    binding.lib()
    return binding


def check_act_codes(oracle, rq, x: torch.Tensor, r: int):
    M, K = x.shape
    act = rq.resq_quantize_act(x.cuda(), r)
    torch.cuda.synchronize()
    q_hi, q_lo, s_hi, s_lo = oracle.quantize_act(wl.bf16_bits(x), r)
    if r > 0:
        want = np.zeros((M, act.ld_hi), np.int8)
        want[:, :r] = q_hi
        assert np.array_equal(act.q_hi.cpu().numpy(), want), "INT8 codes differ"
        assert np.array_equal(act.s_hi.cpu().numpy().view(np.uint32), s_hi.view(np.uint32))
    if K - r > 0:
        want = oracle.pack_nibbles(q_lo, act.ld_lo)
        assert np.array_equal(act.q_lo.cpu().numpy(), want), "INT4 codes differ"
        assert np.array_equal(act.s_lo.cpu().numpy().view(np.uint32), s_lo.view(np.uint32))
        assert np.array_equal(act.lo_sum.cpu().numpy(), oracle.odd_code_sums(q_lo)), "lo_sum differs"
    return act


def compare_act_codes(oracle, act, x_bits: np.ndarray, r: int):
    """Codes, scales and lo_sum in `act` against the oracle's quantizer on x_bits."""
    M, K = x_bits.shape
    q_hi, q_lo, s_hi, s_lo = oracle.quantize_act(x_bits, r)
    if r > 0:
        want = np.zeros((M, act.ld_hi), np.int8)
        want[:, :r] = q_hi
        assert np.array_equal(act.q_hi.cpu().numpy(), want), "INT8 codes differ"
        assert np.array_equal(act.s_hi.cpu().numpy().view(np.uint32), s_hi.view(np.uint32))
    if K - r > 0:
        want = oracle.pack_nibbles(q_lo, act.ld_lo)
        assert np.array_equal(act.q_lo.cpu().numpy(), want), "INT4 codes differ"
        assert np.array_equal(act.s_lo.cpu().numpy().view(np.uint32), s_lo.view(np.uint32))
        assert np.array_equal(act.lo_sum.cpu().numpy(), oracle.odd_code_sums(q_lo)), "lo_sum differs"


def check_weights(oracle, rq, w: torch.Tensor, r: int):
    N, K = w.shape
    packed = rq.resq_pack_weights(w.cuda(), r)
    got = [t.cpu().numpy() for t in rq.resq_unpack_weights(packed, N, K, r)]
    want = oracle.quantize_weights(wl.bf16_bits(w), r)
    if r > 0:
        assert np.array_equal(got[0], want[0]), "INT8 weight codes differ"
        assert np.array_equal(got[2].view(np.uint16), want[2]), "high weight scales differ"
    if K - r > 0:
        assert np.array_equal(got[1], want[1]), "INT4 weight codes differ"
        assert np.array_equal(got[3].view(np.uint16), want[3]), "low weight scales differ"
    return packed, want


def check_layer(oracle, rq, x: torch.Tensor, w: torch.Tensor, r: int, ldy_extra: int = 0):
    M, K = x.shape
    N = w.shape[0]
    act = check_act_codes(oracle, rq, x, r)
    packed, wq = check_weights(oracle, rq, w, r)
    ref = oracle.linear(wl.bf16_bits(x), None, r, weights=wq)
    dbg_hi = torch.full((M, N), -12345, dtype=torch.int32, device="cuda")
    dbg_lo = torch.full((M, N), -12345, dtype=torch.int32, device="cuda")
    ybuf = torch.zeros((M, N + ldy_extra), dtype=torch.bfloat16, device="cuda")
    y = rq.resq_gemm_mixed(act, packed, N, y=ybuf[:, :N], dbg_acc_hi=dbg_hi, dbg_acc_lo=dbg_lo)
    torch.cuda.synchronize()
    if r > 0:
        assert np.array_equal(dbg_hi.cpu().numpy().astype(np.int64), ref.acc_hi), "A_hi differs"
    if K - r > 0:
        assert np.array_equal(dbg_lo.cpu().numpy().astype(np.int64), ref.acc_lo), "A_lo differs"
    rel = y_within_tolerance(y, ref.y)
    assert rel <= REL_TOL, f"bf16 output off by {rel}"
    # the same call without the accumulator dump runs the kernel variant that ships
    y2 = rq.resq_gemm_mixed(act, packed, N, y=torch.zeros_like(ybuf)[:, :N])
    torch.cuda.synchronize()
    rel2 = y_within_tolerance(y2, ref.y)
    assert rel2 <= REL_TOL, f"bf16 output (no dump) off by {rel2}"
    assert torch.equal(y2, y), "output differs with and without the accumulator dump"
    if ldy_extra:
        assert not ybuf[:, N:].any(), "wrote past N"
    # without the debug outputs the result must be the same
    y2 = rq.resq_gemm_mixed(act, packed, N)
    torch.cuda.synchronize()
    assert torch.equal(y2, y.contiguous())
    return rel


# ---- activations -----------------------------------------------------------

def test_quantize_act_tiny_config(oracle, rq):
    check_act_codes(oracle, rq, wl.make_activations(wl.TINY), wl.TINY.r)


@pytest.mark.parametrize("M,K,r", [(3, 2048, 256), (5, 4096, 512), (2, 8192, 1024),
                                   (2, 14336, 1792), (7, 4096, 0), (7, 4096, 4096),
                                   (4, 264, 8), (4, 16384, 2048)])
def test_quantize_act_vector_path(oracle, rq, M, K, r):
    s = wl.LayerShape("qa", M=M, K=K, N=1, r=r, act="student_t3", seed=M + K)
    check_act_codes(oracle, rq, wl.make_activations(s), r)


@pytest.mark.parametrize("M,K,r", [(3, 250, 30), (2, 1000, 2), (5, 77, 77), (4, 90, 0),
                                   (1, 2, 0), (3, 33, 1), (2, 20000, 4000)])
def test_quantize_act_generic_path(oracle, rq, M, K, r):
    s = wl.LayerShape("qg", M=M, K=K, N=1, r=r, outliers="first4" if K > 8 else "none", seed=K)
    check_act_codes(oracle, rq, wl.make_activations(s), r)


# Rows without whole 16-byte pieces: short last units of both groups, groups of exactly one unit and of one unit and a
# bit, units at the edges of what a thread holds (256, 512, 1024, 2048 and 4096 of them), 256 and 1024 threads
@pytest.mark.parametrize("M,K,r", [
    # units that begin and end in a group of 8 columns and a bit, in rows that take this kernel
    (257, 700, 8), (257, 657, 9), (257, 1001, 993), (257, 1003, 993), (257, 651, 651), (257, 650, 0), (12289, 458, 10), (32769, 330, 18),
    (3, 2042, 250), (257, 35, 17), (257, 16, 8), (257, 18, 8), (300, 25, 9), (260, 57, 57), (3, 1100, 0), (3, 1101, 1101), (3, 2048, 12),
    (3, 2051, 11), (257, 1024, 12), (256, 1022, 12), (256, 2050, 258), (257, 2050, 258), (256, 3072, 12), (256, 3074, 12),
    (300, 4090, 8), (300, 4098, 1022), (513, 8190, 14), (513, 8193, 1023), (2, 8190, 14), (2, 8193, 1023), (2, 16382, 4),
    (600, 16382, 2046), (600, 16386, 2046), (512, 12290, 1538), (513, 12290, 1538), (2, 16386, 2046), (3, 32766, 4094), (3, 32770, 4094)])
@pytest.mark.parametrize("asym", [False, True])
def test_quantize_act_rows_at_any_address(oracle, rq, M, K, r, asym):
    s = wl.LayerShape("qr", M=M, K=K, N=1, r=r, act="student_t3", seed=K + r)
    x = wl.make_activations(s)
    for offset, ld in ((0, K), (1, K + 1), (3, K + 5), (6, (K + 7) // 8 * 8)):
        buf = torch.full((offset + M * ld + 8,), float("inf"), dtype=torch.bfloat16, device="cuda")  # beside the rows
        rows = torch.as_strided(buf, (M, K), (ld, 1), offset)
        rows.copy_(x)
        act = (rq.resq_quantize_act_asym if asym else rq.resq_quantize_act)(rows, r)
        torch.cuda.synchronize()
        (compare_asym_codes if asym else compare_act_codes)(oracle, act, wl.bf16_bits(x), r)


def test_quantize_act_rows_at_any_address_not_finite(rq):
    """Infinities and NaN in rows without whole pieces: what the element-wise definition gives (a NaN does not count
    for the maximum; quotients that are NaN clip to the lowest code)."""
    K, r = 2050, 258
    x = torch.randn(260, K, generator=torch.Generator().manual_seed(5)).bfloat16()
    x[0, 3], x[0, 400], x[1, K - 1], x[2, 0], x[2, K - 2], x[3, r] = (float(v) for v in ("nan", "nan", "inf", "-inf", "nan", "-inf"))
    act = rq.resq_quantize_act(x.cuda(), r)
    v = x.float()
    for g, (lo, hi, qmax) in enumerate(((0, r, 127), (r, K, 7))):
        amax = torch.nan_to_num(v[:, lo:hi].abs(), nan=0.0, posinf=float("inf")).amax(1, keepdim=True)
        scale = amax / qmax
        want = torch.nan_to_num(torch.round(v[:, lo:hi] / scale), nan=-qmax).clamp(-qmax, qmax).int()
        assert torch.equal((act.s_hi if g == 0 else act.s_lo).cpu(), scale[:, 0])
        if g == 0:
            assert torch.equal(act.q_hi.cpu()[:, :r].int(), want)
        else:
            byte = act.q_lo.cpu()[:, :(K - r) // 2].int()
            got = torch.stack([(byte & 15) - 8, ((byte >> 4) ^ 8) - 8], 2).reshape(len(x), K - r)
            assert torch.equal(got, want)
            assert torch.equal(act.lo_sum.cpu().long(), want[:, 1::2].sum(1))


# both sides of each line between 256 and 1024 threads to a row, and rows that end inside a wavefront
@pytest.mark.parametrize("M,K,r", [(256, 4104, 520), (257, 4104, 520), (2, 4096, 512), (3, 8192, 1024), (2, 8200, 1032),
                                   (512, 8200, 1032), (513, 8200, 1032), (256, 8200, 1032), (257, 16384, 2048), (1, 16384, 0), (2, 12296, 12296),
                                   # beyond 16384 columns, the last that 1024 threads hold and the first that they do not
                                   (3, 16392, 2056), (1030, 17000, 128), (2, 32768, 4096), (2, 32776, 4096), (2, 20000, 0),
                                   # ... and rows without whole 16-byte pieces
                                   (256, 2050, 258), (257, 2050, 258), (3, 2046, 0), (512, 4100, 516), (513, 4100, 516),
                                   (1024, 8198, 1026), (1025, 8198, 1026), (1, 28674, 3584)])
def test_quantize_act_threads_per_row(oracle, rq, M, K, r):
    x = wl.random_small_case(M + K, M, K, 16, r, act="student_t3")[0]
    check_act_codes(oracle, rq, x, r)
    act = rq.resq_quantize_act_asym(x.cuda(), r)
    torch.cuda.synchronize()
    compare_asym_codes(oracle, act, wl.bf16_bits(x), r)


@pytest.mark.parametrize("M,K,r", [(256, 4608, 256), (257, 4608, 256), (2, 8448, 256), (512, 8704, 512), (513, 8704, 512),
                                   (3, 16896, 256), (5, 28672, 3584), (1025, 16896, 512),
                                   # ... and the transform's own lines: 10240 low columns, 2048 high ones, 16384 low ones
                                   (512, 11776, 1536), (512, 12032, 1536), (257, 10240, 2304), (513, 10240, 2304), (256, 10240, 2048),
                                   (257, 10240, 2048), (1024, 18432, 2048), (1024, 18688, 2048), (257, 18688, 2048), (256, 18688, 2048)])
@pytest.mark.parametrize("asym", [False, True])
def test_hadamard256_quantize_threads_per_row(oracle, rq, M, K, r, asym):
    # codes bit-exact on the kernel's own rotated row; the row itself is the transform's test elsewhere
    x = wl.random_small_case(M + K, M, K, 16, r, act="student_t3")[0]
    x_rot = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
    fn = rq.resq_hadamard_quantize_act_asym if asym else rq.resq_hadamard_quantize_act
    act = fn(x.cuda(), r, 256, x_rot=x_rot)
    torch.cuda.synchronize()
    x_rot[:, :r] = x[:, :r].cuda()
    want = rq.resq_online_hadamard(x.cuda(), r, K, 256)
    torch.cuda.synchronize()
    # the two take their sums in another order: neighbouring bf16 numbers at most
    assert (x_rot.float() - want.float()).abs().max() <= 2.0 ** -7 * want.float().abs().max()
    (compare_asym_codes if asym else compare_act_codes)(oracle, act, wl.bf16_bits(x_rot.cpu()), r)


def test_quantize_act_strided_rows_zero_rows_and_ties(oracle, rq):
    # rows taken from a wider buffer (ldx > K), an all-zero token, an all-zero group,
    # and exact ties (values on half-integers of a power-of-two scale)
    g = torch.Generator().manual_seed(5)
    big = torch.randn(6, 640, generator=g).to(torch.bfloat16)
    x = big[:, 64:576]                       # K = 512, ldx = 640, 16-byte aligned start
    x[1] = 0
    x[2, :64] = 0
    x[3, 64:] = 0
    x[4, :64] = torch.tensor([127.0] + [0.5 * k for k in range(63)]).to(torch.bfloat16)
    x[4, 64:] = torch.tensor([7.0] + [0.5 * (k % 14) for k in range(447)]).to(torch.bfloat16)
    xc = x.contiguous()
    M, K, r = 6, 512, 64
    dev = big.cuda()
    act = rq.resq_quantize_act(dev[:, 64:576], r)
    torch.cuda.synchronize()
    q_hi, q_lo, s_hi, s_lo = oracle.quantize_act(wl.bf16_bits(xc), r)
    assert np.array_equal(act.q_hi.cpu().numpy()[:, :r], q_hi)
    assert np.array_equal(act.q_lo.cpu().numpy()[:, :(K - r) // 2], oracle.pack_nibbles(q_lo))
    assert np.array_equal(act.s_hi.cpu().numpy(), s_hi) and np.array_equal(act.s_lo.cpu().numpy(), s_lo)
    assert s_hi[1] == 1 and s_lo[1] == 1 and s_hi[2] == 1 and s_lo[3] == 1


@pytest.mark.parametrize("K,r", [(512, 64), (4096, 512), (250, 30), (128, 16)])
def test_quantize_act_rows_with_tiny_scales(oracle, rq, K, r):
    # rows whose absmax is so small that the reciprocal of the scale overflows (scale below
    # 2^-128): the kernels multiply by that reciprocal and must fall back to the division of
    # the definition for every element of such a row
    g = torch.Generator().manual_seed(K)
    x = torch.randn(6, K, generator=g)
    x[1] *= 2.0 ** -125
    x[2] *= 2.0 ** -121          # scales around 2^-126: reciprocal finite, quotients fine
    x[3] = 0
    x[3, 5] = 2.0 ** -126
    x[3, K - 3] = -(2.0 ** -126)
    x[4, :r] *= 2.0 ** -124      # only the high group tiny
    x[5, r:] *= 2.0 ** -124      # only the low group tiny
    x = x.to(torch.bfloat16)
    check_act_codes(oracle, rq, x, r)
    act = rq.resq_quantize_act_asym(x.cuda(), r)
    torch.cuda.synchronize()
    compare_asym_codes(oracle, act, wl.bf16_bits(x), r)


# ---- weights ---------------------------------------------------------------

@pytest.mark.parametrize("N,K,r", [(256, 256, 32), (300, 520, 72), (17, 90, 30), (64, 512, 0),
                                   (64, 512, 512), (513, 4096, 512)])
def test_pack_weights_roundtrip(oracle, rq, N, K, r):
    s = wl.LayerShape("w", M=1, K=K, N=N, r=r, seed=N)
    w = wl.make_weights(s)
    w[0] = 0                                 # an all-zero output channel
    check_weights(oracle, rq, w, r)


# Both packing kernels (rows of whole 16-byte pieces and any others): units at the edges of what a thread holds, weights at and
# beside ties, rows whose scale is cut off at either end of fp16 (codes are clipped there), zero rows, infinities
@pytest.mark.parametrize("N,K,r", [(40, 4096, 512), (17, 4104, 520), (16, 8192, 0), (20, 256, 256), (33, 8, 8), (18, 4098, 514), (20, 2050, 0), (17, 66, 66)])
def test_pack_weights_values_at_the_edges(oracle, rq, N, K, r):
    g = torch.Generator().manual_seed(N + K)
    w = torch.randn(N, K, generator=g) * 0.02
    w[0] = torch.randint(-14, 15, (K,), generator=g).float() * 0.5     # halves: ties of the low group at scale 1
    w[0, K - 1] = 7.0
    w[1] *= 1e-9
    w[2] *= 1e9
    w[3] = 0.0
    w[4, 0], w[4, K - 1] = float("inf"), float("-inf")
    w[5] = torch.randint(-254, 255, (K,), generator=g).float() * 0.5
    w[5, 0] = 127.0
    w = w.bfloat16()
    check_weights(oracle, rq, w, r)
    wide = torch.zeros(N, K + 8, dtype=torch.bfloat16, device="cuda")   # strided rows, from an odd address
    for off in (0, 3):
        wide[:, off:off + K] = w.cuda()
        assert torch.equal(rq.resq_pack_weights(wide[:, off:off + K], r), rq.resq_pack_weights(w.cuda(), r))


# ---- the layer -------------------------------------------------------------

def test_layer_tiny_config(oracle, rq):
    s = wl.TINY
    check_layer(oracle, rq, wl.make_activations(s), wl.make_weights(s), s.r)


@pytest.mark.parametrize("M,K,N,r", [
    (16, 256, 256, 0), (16, 256, 256, 256),      # uniform INT4, uniform INT8
    (130, 640, 300, 128),                        # ragged M and N, several tiles
    (257, 1000, 515, 104),                       # K, r off the stage size; N % 4 != 0
    (64, 4096, 512, 512),                        # Llama-8B K with d/8
    (200, 90, 40, 30),                           # everything smaller than one stage
    (1, 512, 256, 64), (4, 512, 256, 64),        # decode-sized M
    (300, 2048, 768, 256),
    (260, 640, 300, 128), (385, 90, 40, 30), (290, 4096, 512, 512), (258, 256, 256, 0), (258, 256, 256, 256),
])
def test_layer_shapes(oracle, rq, M, K, N, r):
    # 64 < M <= 1024 takes the tiled kernel or the weight-streaming kernel in slices of 64
    # tokens, whichever the dispatch estimates to be faster (few channels: the latter)
    x, w = wl.random_small_case(M * 7 + K, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", [
    (1, 8192, 4096, 1024), (4, 8192, 4096, 1024), (16, 8192, 4100, 1024),   # Llama-70B K, d/8
    (16, 1000, 515, 104),                        # K, r off the block size; N % 4 != 0
    (3, 256, 256, 0), (16, 256, 256, 256),       # uniform INT4, uniform INT8
    (7, 14336, 272, 1792),                       # longest K of the workloads
    (14, 640, 300, 128), (15, 1024, 8720, 128), (9, 1024, 8720, 128),
])
def test_layer_decode_shapes(oracle, rq, M, K, N, r):
    # M <= 16 takes the weight-streaming kernel
    x, w = wl.random_small_case(M * 11 + K, M, K, N, r, outliers="first4")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", [
    (17, 8192, 528, 1024), (32, 4096, 272, 512),         # two token groups
    (33, 1000, 515, 104), (64, 14336, 144, 1792),        # four; K, r off the block size; longest K
    (65, 2048, 400, 256), (100, 4096, 130, 512), (128, 8192, 272, 1024),   # eight
    (128, 3200, 256, 448),                               # high blocks end inside a chunk of eight
    (200, 8192, 4100, 1024), (256, 1000, 515, 104), (129, 14336, 272, 1792),   # two to four slices
    (90, 256, 256, 0), (128, 256, 64, 256),              # uniform INT4, uniform INT8
    (40, 90, 40, 30),                                    # everything smaller than one chunk
])
def test_layer_batched_decode_shapes(oracle, rq, M, K, N, r):
    # 16 < M <= 64 takes the weight-streaming kernel with the activation codes chunked through LDS;
    # the larger M here take it in slices of 64 tokens (few tiles) or the tiled kernel
    x, w = wl.random_small_case(M * 13 + K, M, K, N, r, outliers="first4")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", [
    (16, 28672, 272, 3584),      # Llama-70B down_proj's K: 16 token rows do not fit LDS; eight runs per group
    (9, 30000, 100, 3000),       # ragged everything
    (16, 16384, 8208, 2048),     # two runs per group
    (16, 16384, 16400, 2048),    # one run per group
])
def test_layer_decode_long_rows(oracle, rq, M, K, N, r):
    # M <= 16 with rows too long for LDS: the chunked weight-streaming kernel with one token group
    x, w = wl.random_small_case(M * 3 + N, M, K, N, r, outliers="first4")
    check_layer(oracle, rq, x, w, r)


# more than 1024 tokens: always a tiled kernel; on these small ragged layers the one with 64 x 128
# tiles, and at most 256 of them: eight wavefronts per tile in two rings
TILED_SHAPES = [
    (1030, 640, 300, 128), (1100, 1000, 515, 104), (1025, 90, 40, 30),
    (1153, 256, 256, 0), (1153, 256, 256, 256), (1200, 2048, 768, 256),
    # 32 x 8 = 256 tiles: the tile order in 8 x 8 patches per XCD needs a multiple of 512, so this is
    # the order that deals contiguous runs of tiles to the eight XCDs (e.g. a grouped-query
    # key/value projection); ragged M too
    (2048, 256, 1024, 32), (1925, 256, 1024, 32),
    # up to 1024 tokens on layers wide enough that the tiles beat the sliced streaming kernel
    (300, 256, 4100, 32), (130, 520, 8200, 64), (200, 640, 6000, 640),
    (1030, 128, 300, 128), (1030, 256, 300, 128), (1030, 640, 300, 128),   # 1, 2, 3 pairs of stages (the second ring gets none; the
                                                                           # high pair and the low pair; one pair less than the first)
    (1100, 896, 300, 128),                                                 # one high pair, three low pairs
]
# 257 to 512 such tiles: four wavefronts per tile, two workgroups per compute unit
TILED64_ONE_RING_SHAPES = [
    (65, 256, 28672, 0), (513, 90, 4100, 30), (1153, 256, 2100, 32), (1300, 640, 2300, 128),
    (1100, 384, 3000, 384), (1500, 520, 2000, 0),
    (1024, 128, 4096, 128),  # 16 x 32 = 512 tiles: the 8 x 8 patches
]
# more than 512 tiles of 64 x 128: the kernel with 128 x 128 tiles
TILED128_SHAPES = [
    (2100, 256, 2200, 32), (4100, 256, 1100, 0), (4100, 256, 1100, 256), (1100, 1000, 4200, 104),
    (1925, 256, 4096, 32),   # 16 x 32 = 512 tiles, ragged M: the 8 x 8 patches
    (4200, 90, 1040, 30),
]


@pytest.mark.parametrize("M,K,N,r", TILED_SHAPES)
def test_layer_tiled_kernel_small_layers(oracle, rq, M, K, N, r):
    assert rq.resq_gemm_mixed_plan(M, N, K, r) == (3, 0, 2)
    x, w = wl.random_small_case(M * 17 + K, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", TILED64_ONE_RING_SHAPES)
def test_layer_tiled_kernel_narrow_tiles_one_ring(oracle, rq, M, K, N, r):
    assert rq.resq_gemm_mixed_plan(M, N, K, r) == (3, 0, 1)
    x, w = wl.random_small_case(M * 17 + K + 2, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", TILED128_SHAPES)
def test_layer_tiled_kernel_wide_tiles(oracle, rq, M, K, N, r):
    assert rq.resq_gemm_mixed_plan(M, N, K, r) == (2, 0, 0)
    x, w = wl.random_small_case(M * 17 + K + 1, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


# 128 x 128 tiles in more than one round and 24 low stages or more: the low group on the fp8 matrix
# cores.  Ragged tiles; 2 and 4 high stages (the first buffer) and none; 24, 26 and 28 low stages (what
# the four-stage turns of the loop leave over); groups that fill their padded width, and groups that end inside it:
# each padding column adds 64 to the sums of offset codes, which the epilogue takes out again (2, 72 and 254 of them)
TILED_F8_SHAPES = [(1925, 3200, 4500, 128), (1921, 3584, 4400, 256), (1930, 3072, 4300, 0), (4200, 3450, 2050, 122),
                   (1921, 3202, 4400, 128), (1930, 3712, 4300, 130), (1925, 3000, 4500, 0)]
F8_STAGES = [(2, 24), (4, 26), (0, 24), (2, 26), (2, 26), (4, 28), (0, 24)]   # high, low


def is_f8(rq, M, K, N, r):
    return rq.resq_gemm_mixed_plan(M, N, K, r) == (2, 0, 0) and rq.resq_gemm_mixed_low_fp8(M, N, K, r)


@pytest.mark.parametrize("M,K,N,r", TILED_F8_SHAPES)
def test_layer_tiled_kernel_fp8_low_group(oracle, rq, M, K, N, r):
    assert is_f8(rq, M, K, N, r)
    assert (-(-r // 128) * 2, -(-(K - r) // 256) * 2) == F8_STAGES[TILED_F8_SHAPES.index((M, K, N, r))]
    x, w = wl.random_small_case(M * 17 + K + 3, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


def test_layer_tiled_kernel_fp8_low_group_asym_and_saturated(oracle, rq):
    M, K, N, r = TILED_F8_SHAPES[0]
    x, w = wl.random_small_case(5, M, K, N, r, act="student_t3")
    check_layer_asym(oracle, rq, (x.float() + 1.5).to(torch.bfloat16), w, r)
    # every low code at +7 or -7, the same in all columns of a row
    x[:, r:] = torch.where(torch.arange(M) % 2 == 0, 1.0, -1.0)[:, None].to(torch.bfloat16)
    w[:, r:] = torch.where(torch.arange(N) % 3 == 0, 0.5, -0.5)[:, None].to(torch.bfloat16)
    check_layer(oracle, rq, x, w, r)


@pytest.mark.parametrize("M,K,N,r", TILED_F8_SHAPES[4:])
def test_layer_tiled_kernel_fp8_low_group_asym_padding(oracle, rq, M, K, N, r):
    assert is_f8(rq, M, K, N, r)
    x, w = wl.random_small_case(M + K, M, K, N, r, act="student_t3")
    check_layer_asym(oracle, rq, (x.float() + 1.5).to(torch.bfloat16), w, r, ldy_extra=3)


# The largest sums of offset codes there are, up to 225 x 65536 < 2^24, odd and even ones: codes of 7 and here and
# there 6, so that a sum that lost its lowest bits in the fp32 accumulator would show.  One more pair of columns goes
# to the int8 kernel.
@pytest.mark.parametrize("low,f8", [(65536, True), (65534, True), (32770, True), (65538, False)])
def test_layer_tiled_kernel_fp8_low_group_largest_sums(rq, low, f8):
    M, N = 2930, 2900
    assert rq.resq_gemm_mixed_plan(M, N, low, 0) == (2, 0, 0) and rq.resq_gemm_mixed_low_fp8(M, N, low, 0) == f8
    g = torch.Generator(device="cuda").manual_seed(low)

    def codes(rows):
        c = 7 - (torch.rand(rows, low, generator=g, device="cuda") < 0.05).to(torch.bfloat16)
        c[:, 0] = 7.0   # scale 1
        return c

    x, w = codes(M), codes(N)
    dbg = torch.zeros((M, N), dtype=torch.int32, device="cuda")
    act = rq.resq_quantize_act(x, 0)
    y = rq.resq_gemm_mixed(act, rq.resq_pack_weights(w, 0), N, dbg_acc_lo=dbg)
    y2 = rq.resq_gemm_mixed(act, rq.resq_pack_weights(w, 0), N)
    torch.cuda.synchronize()
    want = x.double() @ w.double().t().contiguous()     # whole numbers, exact in fp64
    offset = want + 8 * x.double().sum(1, keepdim=True) + 8 * w.double().sum(1) + 64 * low
    assert 0.95 * 225 * low < offset.max() <= 225 * low and bool((offset % 2 == 1).any())
    assert torch.equal(dbg.double(), want)
    assert torch.equal(y, want.float().to(torch.bfloat16)) and torch.equal(y2, y)   # both scales are 1


# Grids whose number of tiles, padding tiles included, leaves 2, 4 and 6 over eight: bands of eight token tiles, of the layer's
# own tiles.  Whole bands and a last one of 1 to 7, one channel tile and many, padding tiles left out and none there
@pytest.mark.parametrize("M,K,N,r,kernel,tiles", [
    (385, 512, 2562, 64, 3, 154), (321, 512, 3300, 64, 3, 156), (385, 512, 3300, 64, 3, 182),
    (1025, 512, 2050, 64, 3, 306), (577, 512, 3300, 64, 3, 260), (700, 512, 3300, 64, 3, 286),
    (1537, 512, 3300, 64, 2, 338), (1700, 512, 2562, 64, 2, 308), (1793, 512, 2300, 64, 2, 270),
    (1025, 512, 256, 64, 3, 34), (1100, 512, 100, 64, 3, 36), (1153, 512, 300, 64, 3, 76), (1537, 512, 2562, 0, 2, 286), (7550, 256, 1065, 32, 2, 590),
    # a column of padding tiles in a multiple of eight: left out as well
    (512, 512, 3200, 64, 3, 208), (1537, 512, 3967, 64, 2, 416), (2500, 512, 3200, 64, 2, 520), (5100, 256, 129, 32, 3, 160),
])
def test_layer_tile_order(oracle, rq, M, K, N, r, kernel, tiles):
    assert rq.resq_gemm_mixed_plan(M, N, K, r)[0] == kernel
    assert -(-M // (64 if kernel == 3 else 128)) * -(-N // 256) * 2 == tiles
    x, w = wl.random_small_case(M + N, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r,kernel", [
    (3, 512, 21, 64, 0), (16, 512, 130, 64, 0), (40, 512, 150, 64, 1), (1025, 512, 2049, 64, 3), (700, 512, 3300, 64, 3),
    (1100, 512, 8190, 64, 2), (300, 512, 4094, 0, 3), (8200, 3072, 998, 0, 2)])
def test_layer_output_rows_at_any_address(rq, M, K, N, r, kernel):
    """Outputs whose rows start at any 2-byte aligned address, rows of any length: the values of a call on rows of
    whole 16-byte pieces (which other tests hold against the oracle), and not a byte beside them."""
    assert rq.resq_gemm_mixed_plan(M, N, K, r)[0] == kernel
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    packed = rq.resq_pack_weights((torch.randn(N, K, generator=g, device="cuda") * 0.02).bfloat16(), r)
    act = rq.resq_quantize_act(x, r)
    calls = [(rq.resq_gemm_mixed, N)] + ([(rq.resq_gemm_mixed_swiglu, N // 2)] if N % 2 == 0 else [])
    for call, width in calls:
        want = call(act, packed, N, y=torch.zeros((M, (width + 15) // 8 * 8), dtype=torch.bfloat16, device="cuda")[:, :width])
        for offset, ld in ((1, width), (0, width + 1), (5, width + 3), (2, width + 4)):
            buf = torch.full((offset + M * ld + 16,), 77.0, dtype=torch.bfloat16, device="cuda")
            expect = buf.clone()
            torch.as_strided(expect, (M, width), (ld, 1), offset).copy_(want)
            call(act, packed, N, y=torch.as_strided(buf, (M, width), (ld, 1), offset))
            assert torch.equal(buf, expect), (call.__name__, offset, ld)


@pytest.mark.parametrize("M,K,N,r", [
    (385, 2048, 400, 256), (512, 4096, 272, 512), (1000, 1000, 515, 104), (1024, 3200, 256, 448),
    (700, 256, 256, 0), (640, 256, 64, 256), (1024, 14336, 144, 1792),
])
def test_layer_sliced_streaming_up_to_1024_tokens(oracle, rq, M, K, N, r):
    # few channels, up to 16 slices of 64 tokens through the weight-streaming kernel
    x, w = wl.random_small_case(M * 19 + K, M, K, N, r, outliers="first4")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", [
    (1, 8192, 4096, 1024), (4, 8192, 4096, 1024), (16, 8192, 4112, 1024),   # one run per group
    (1, 4096, 512, 512), (3, 4096, 272, 512), (16, 14336, 272, 1792),       # split reduction axis
    (2, 256, 256, 0), (5, 256, 64, 256), (7, 1000, 515, 104), (16, 1000, 40, 104),
    (9, 2048, 1024, 256),
    # 4, 8 and 16 units a thread: the last width of each and the first of the next, 1 to 8 rows at a time, with and without split
    (1, 16384, 64, 2048), (1, 16392, 64, 2056), (1, 32768, 48, 4096), (1, 32776, 48, 4096), (2, 8192, 64, 0), (2, 8200, 16400, 1032),
    (3, 4096, 16400, 512), (4, 4104, 100, 512), (4, 8192, 100, 8192), (4, 8200, 100, 1032), (8, 2048, 16400, 256), (7, 2056, 64, 256),
    (8, 4096, 64, 512), (8, 4104, 64, 512), (9, 512, 64, 64), (16, 2048, 64, 256), (1, 8, 16, 0), (4, 16, 300, 8),
])
def test_quantize_gemm_mixed_one_call(oracle, rq, M, K, N, r):
    # the quantizer inside the weight-streaming kernel: bit-identical to the two calls, and
    # against the oracle like every other layer test
    x, w = wl.random_small_case(M * 23 + K, M, K, N, r, outliers="first4")
    xd = x.cuda()
    packed = rq.resq_pack_weights(w.cuda(), r)
    ybuf = torch.zeros((M, N + 8), dtype=torch.bfloat16, device="cuda")
    y = rq.resq_quantize_gemm_mixed(xd, packed, N, r, y=ybuf[:, :N])
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(xd, r), packed, N)
    torch.cuda.synchronize()
    assert torch.equal(y, two)
    assert not ybuf[:, N:].any(), "wrote past N"
    ref = oracle.linear(wl.bf16_bits(x), wl.bf16_bits(w), r)
    assert y_within_tolerance(y, ref.y) <= REL_TOL
    # strided rows of x
    xs = torch.zeros((M, K + 24), dtype=torch.bfloat16, device="cuda")
    xs[:, :K] = xd
    y2 = rq.resq_quantize_gemm_mixed(xs[:, :K], packed, N, r)
    torch.cuda.synchronize()
    assert torch.equal(y2, two)


def _random_one_call_shapes(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        M = int(rng.integers(1, 17))
        K = int(rng.choice([64, 136, 520, 1000, 2048, 4096, 8192]))
        r = int(rng.choice([0, K // 8, K // 4, K])) // 8 * 8
        N = int(rng.choice([16, 40, 272, 515, 1024, 4100]))
        out.append((M, K, N, r))
    return out


@pytest.mark.parametrize("M,K,N,r", _random_one_call_shapes(16, 4321))
def test_quantize_gemm_mixed_one_call_random_shapes(oracle, rq, M, K, N, r):
    x, w = wl.random_small_case(M * 29 + K + N, M, K, N, r, act="student_t3")
    packed = rq.resq_pack_weights(w.cuda(), r)
    y = rq.resq_quantize_gemm_mixed(x.cuda(), packed, N, r)
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(x.cuda(), r), packed, N)
    torch.cuda.synchronize()
    assert torch.equal(y, two)
    ref = oracle.linear(wl.bf16_bits(x), wl.bf16_bits(w), r)
    assert y_within_tolerance(y, ref.y) <= REL_TOL


def test_quantize_gemm_mixed_one_call_full_size(oracle, rq):
    s = wl.decode_shape(4)
    x, w = wl.make_activations(s), wl.make_weights(s)
    packed = rq.resq_pack_weights(w.cuda(), s.r)
    y = rq.resq_quantize_gemm_mixed(x.cuda(), packed, s.N, s.r)
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(x.cuda(), s.r), packed, s.N)
    torch.cuda.synchronize()
    assert torch.equal(y, two)
    ref = oracle.linear(wl.bf16_bits(x), wl.bf16_bits(w), s.r)
    assert y_within_tolerance(y, ref.y) <= REL_TOL


def _stream_plan_shapes():
    from test_boundary_cpu import STREAM_PLAN_SHAPES
    return [shape for shape, _ in STREAM_PLAN_SHAPES]


@pytest.mark.parametrize("M,K,N,r", _stream_plan_shapes())
def test_layer_every_token_group_and_run_count(oracle, rq, M, K, N, r):
    # one shape per (token groups, runs) pair of the chunked kernel (the CPU test pins which)
    assert rq.resq_gemm_mixed_plan(M, N, K, r)[0] == 1
    x, w = wl.random_small_case(M * 37 + K + N, M, K, N, r, outliers="first4")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


def _second_set_shapes():
    from test_boundary_cpu import SECOND_SET_SHAPES
    return [shape for shape, _ in SECOND_SET_SHAPES]


@pytest.mark.parametrize("M,K,N,r", _second_set_shapes())
@pytest.mark.parametrize("asym", [False, True])
def test_layer_second_set_of_a_workgroup(oracle, rq, M, K, N, r, asym):
    # the chunked kernel's loop over sets: weights carried over the epilogue, constants and codes fetched anew
    x, w = wl.random_small_case(M * 41 + K + N, M, K, N, r, outliers="first4")
    (check_layer_asym if asym else check_layer)(oracle, rq, x, w, r, ldy_extra=3)


def test_layer_batched_decode_full_size(oracle, rq):
    # the decode workload's layer with 64 tokens in flight; every accumulator and output
    s = wl.decode_shape(64)
    check_layer(oracle, rq, wl.make_activations(s), wl.make_weights(s), s.r)


@pytest.mark.parametrize("M", [16, 9, 1])
def test_layer_decode_full_size(oracle, rq, M):
    # the decode workload at full size (Llama-3-70B up_proj; 16 tokens: the chunked kernel, 9 and 1: the plain one); the
    # oracle checks all codes and every accumulator and output
    s = wl.decode_shape(M)
    check_layer(oracle, rq, wl.make_activations(s), wl.make_weights(s), s.r)


def _random_layer_shapes(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    for _ in range(n):
        M = int(rng.choice([1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 100, 128, 129, 200, 255, 256, 257, 300]))
        K = int(rng.choice([64, 90, 256, 520, 1000, 2048, 3200, 4096, 8192]))
        K += int(rng.integers(0, 3)) * 2 if K not in (2048, 4096, 8192) else 0
        N = int(rng.choice([16, 40, 130, 256, 272, 515, 1024, 2100]))
        r = int(rng.choice([0, K // 8, K // 4, K])) // 2 * 2
        if (K - r) % 2:
            r += 1
        out.append((M, K, N, min(r, K)))
    return out


@pytest.mark.parametrize("M,K,N,r", _random_layer_shapes(40, 2024))
def test_layer_random_shapes_across_dispatch_boundaries(oracle, rq, M, K, N, r):
    # seeded draw over the sizes at which resq_gemm_mixed changes kernel (16/17, 64/65, 256/257
    # tokens; few or many channel groups; reduction axes short, ragged and long)
    x, w = wl.random_small_case(M * 31 + K * 7 + N, M, K, N, r, act="student_t3")
    check_layer(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


def test_layer_saturated_codes(oracle, rq):
    # every code at +-qmax: the largest accumulators the shapes allow
    M, K, N, r = 32, 2048, 256, 256
    x = torch.ones(M, K)
    x[::2, ::3] = -1
    w = torch.ones(N, K) * 0.5
    w[:, ::5] = -0.5
    check_layer(oracle, rq, x.to(torch.bfloat16), w.to(torch.bfloat16), r)


QWEN_SNR = {}   # r -> (SNR of the HIP path, SNR of the oracle) on the sampled rows, filled by the test below


@pytest.mark.parametrize("which", ["oproj_prefill", "gate_up_prefill", "qwen_r0", "qwen_r1024", "qwen_r2048",
                                   "oproj_m512", "oproj_m1024"])
def test_layer_prefill_full_size_sampled(oracle, rq, which):
    # the benchmark's prefill configurations at full size, in the launch configuration the
    # benchmark times; the oracle checks all activation codes, all packed weights, and a
    # seeded sample of token rows of the accumulators and outputs.  For the Qwen-72B shape
    # (r = 0, K/8, K/4: the rank sweep) the output SNR on those rows is taken too.
    s = {"oproj_prefill": wl.OPROJ_PREFILL, "gate_up_prefill": wl.MLP_GATE_UP,
         "qwen_r0": wl.qwen_mlp_shape(0), "qwen_r1024": wl.qwen_mlp_shape(1024),
         "qwen_r2048": wl.qwen_mlp_shape(2048),
         # prefill chunks: 64 x 128 tiles, one per compute unit and two per compute unit
         "oproj_m512": wl.chunk_shape("o_proj", 512), "oproj_m1024": wl.chunk_shape("o_proj", 1024)}[which]
    nrows = 48 if which.startswith("oproj") else 24
    x, w = wl.make_activations(s), wl.make_weights(s)
    act = check_act_codes(oracle, rq, x, s.r)
    packed, wq = check_weights(oracle, rq, w, s.r)
    dbg_hi = torch.empty((s.M, s.N), dtype=torch.int32, device="cuda")
    dbg_lo = torch.empty((s.M, s.N), dtype=torch.int32, device="cuda")
    y = rq.resq_gemm_mixed(act, packed, s.N, dbg_acc_hi=dbg_hi, dbg_acc_lo=dbg_lo)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(0).choice(s.M, nrows, replace=False))
    rt = torch.from_numpy(rows).cuda()
    ref = oracle.linear(wl.bf16_bits(x[rows]), None, s.r, weights=wq)
    if s.r > 0:
        assert np.array_equal(dbg_hi[rt].cpu().numpy().astype(np.int64), ref.acc_hi)
    assert np.array_equal(dbg_lo[rt].cpu().numpy().astype(np.int64), ref.acc_lo)
    assert y_within_tolerance(y[rt], ref.y) <= REL_TOL
    del dbg_hi, dbg_lo
    y2 = rq.resq_gemm_mixed(act, packed, s.N)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    if which.startswith("qwen"):
        exact = x[rows].double().numpy() @ w.double().numpy().T      # the unquantized layer, fp64
        snr_gpu = oracle.snr_db(exact, y[rt].float().cpu().numpy())
        snr_cpu = oracle.snr_db(exact, ref.y)
        assert abs(snr_gpu - snr_cpu) < 0.05, (s.r, snr_gpu, snr_cpu)
        QWEN_SNR[s.r] = (snr_gpu, snr_cpu)


def test_qwen_snr_grows_with_rank_at_full_size():
    # Section 5.4's rank ablation on the synthetic Qwen-72B-shaped layer, at full size: more
    # columns in 8 bits, higher output SNR (needs the three sampled cases above to have run)
    if sorted(QWEN_SNR) != [0, 1024, 2048]:
        pytest.skip("the three Qwen-72B cases of test_layer_prefill_full_size_sampled did not all run")
    assert QWEN_SNR[0][0] < QWEN_SNR[1024][0] < QWEN_SNR[2048][0], QWEN_SNR
    print("SNR dB per r (HIP path, oracle):", QWEN_SNR)


# ---- Hadamard --------------------------------------------------------------

def check_hadamard(oracle, rq, x, c0, c1, block, inplace=False):
    b = block or rq.resq_hadamard_block(c1 - c0)
    xd = x.cuda()
    yd = rq.resq_online_hadamard(xd, c0, c1, block, out=xd if inplace else None)
    torch.cuda.synchronize()
    got = wl.bf16_bits(yd.cpu())
    want = oracle.hadamard(wl.bf16_bits(x), c0, c1, b)
    # fp32 butterflies against the fp64 definition: the same bf16 value, or its neighbour
    g64, w64 = wl.bits_to_f64(got), wl.bits_to_f64(want)
    assert np.array_equal(got[:, :c0], want[:, :c0]) and np.array_equal(got[:, c1:], want[:, c1:])
    scale = np.abs(w64).max()
    assert np.all(np.abs(g64 - w64) <= np.maximum(np.abs(w64), 2.0 ** -8 * scale) * 2.0 ** -7)
    assert np.mean(got == want) > 0.99
    return yd


@pytest.mark.parametrize("M,K,c0,c1,block", [
    (5, 512, 0, 512, 0), (3, 1024, 256, 1024, 256), (3, 1024, 256, 1024, 16),
    (2, 2048, 0, 2048, 0), (2, 8192, 0, 8192, 0), (4, 1792 + 12544, 1792, 1792 + 12544, 0),
    (3, 520, 8, 520, 8), (3, 64, 0, 64, 1), (2, 4096, 0, 4096, 1024), (2, 48, 8, 40, 0),
])
def test_hadamard(oracle, rq, M, K, c0, c1, block):
    g = torch.Generator().manual_seed(K + c0)
    x = torch.randn(M, K, generator=g).to(torch.bfloat16)
    check_hadamard(oracle, rq, x, c0, c1, block)
    check_hadamard(oracle, rq, x, c0, c1, block, inplace=True)


def test_down_proj_path_hadamard_then_quantize(oracle, rq):
    # the down_proj input: Hadamard on the low group, then the quantizer.  The
    # quantizer is checked bit-exactly on the GPU's own transformed activations.
    s = wl.LayerShape("down_small", M=24, K=1792 + 12544, N=256, r=1792, act="student_t3",
                      hadamard=True, seed=3)
    x, w = wl.make_activations(s), wl.make_weights(s)
    xt = check_hadamard(oracle, rq, x, s.r, s.K, 0)
    check_layer(oracle, rq, xt.cpu(), w, s.r)


@pytest.mark.parametrize("M,K,N,r", [(24, 1792 + 12544, 256, 1792), (130, 2048, 300, 512), (4096, 1792 + 12544, 4096, 1792)])
def test_down_proj_chain_end_to_end(oracle, rq, M, K, N, r):
    # the whole down_proj step against the oracle's own chain (its fp64 transform rounded to
    # bf16, its quantizer, its GEMMs): nothing of the HIP path enters the oracle.  The fp32
    # butterflies differ from the fp64 ones in the last bf16 bit of < 1 % of the elements, which
    # moves a few codes by one step, so integers are not compared here, only the output, on a
    # sample of rows at the full size (the last case is the benchmark's down_proj workload).
    s = wl.LayerShape("down_chain", M=M, K=K, N=N, r=r, act="student_t3", hadamard=True, seed=M + N)
    x, w = wl.make_activations(s), wl.make_weights(s)
    b = rq.resq_hadamard_block(K - r)
    act = rq.resq_hadamard_quantize_act(x.cuda(), r, 0)
    packed = rq.resq_pack_weights(w.cuda(), r)
    y = rq.resq_gemm_mixed(act, packed, N)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(1).choice(M, min(M, 24), replace=False))
    xr = oracle.hadamard(wl.bf16_bits(x[rows]), r, K, b)
    ref = oracle.linear(xr, wl.bf16_bits(w), r)
    assert y_within_tolerance(y[torch.from_numpy(rows).cuda()], ref.y) <= REL_TOL


def test_down_proj_full_size_sampled_integers(oracle, rq):
    # the benchmark's down_proj workload (M = 4096, K = 14336, N = 4096, r = 1792) in the launch
    # configuration the benchmark times, integers included: the fused transform + quantizer
    # hands out its rotated rows, which are checked against the oracle's transform like the
    # stand-alone kernel's; codes, scales and sums of a sample of token rows bit-exact against
    # the oracle's quantizer on those rotated rows; all packed weights; both accumulators and
    # the outputs of the sampled rows against the oracle's GEMMs on the oracle's codes
    s = wl.MLP_DOWN
    x, w = wl.make_activations(s), wl.make_weights(s)
    xd = x.cuda()
    x_rot = torch.zeros_like(xd)
    act = rq.resq_hadamard_quantize_act(xd, s.r, 0, x_rot=x_rot)
    packed, wq = check_weights(oracle, rq, w, s.r)
    dbg_hi = torch.empty((s.M, s.N), dtype=torch.int32, device="cuda")
    dbg_lo = torch.empty((s.M, s.N), dtype=torch.int32, device="cuda")
    y = rq.resq_gemm_mixed(act, packed, s.N, dbg_acc_hi=dbg_hi, dbg_acc_lo=dbg_lo)
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(2).choice(s.M, 24, replace=False))
    rt = torch.from_numpy(rows).cuda()
    b = rq.resq_hadamard_block(s.K - s.r)
    got = wl.bf16_bits(x_rot[rt].cpu())
    want = oracle.hadamard(wl.bf16_bits(x[rows]), s.r, s.K, b)
    g64, w64 = wl.bits_to_f64(got[:, s.r:]), wl.bits_to_f64(want[:, s.r:])
    scale = np.abs(w64).max()
    assert np.all(np.abs(g64 - w64) <= np.maximum(np.abs(w64), 2.0 ** -8 * scale) * 2.0 ** -7)
    assert np.mean(got[:, s.r:] == want[:, s.r:]) > 0.99
    rotated = wl.bf16_bits(x[rows]).copy()
    rotated[:, s.r:] = got[:, s.r:]
    q_hi, q_lo, s_hi, s_lo = oracle.quantize_act(rotated, s.r)
    assert np.array_equal(act.q_hi[rt].cpu().numpy()[:, :s.r], q_hi), "INT8 codes differ"
    assert np.array_equal(act.q_lo[rt].cpu().numpy(), oracle.pack_nibbles(q_lo, act.ld_lo)), "INT4 codes differ"
    assert np.array_equal(act.s_hi[rt].cpu().numpy().view(np.uint32), s_hi.view(np.uint32))
    assert np.array_equal(act.s_lo[rt].cpu().numpy().view(np.uint32), s_lo.view(np.uint32))
    assert np.array_equal(act.lo_sum[rt].cpu().numpy(), oracle.odd_code_sums(q_lo)), "lo_sum differs"
    ref = oracle.linear(rotated, None, s.r, weights=wq)
    assert np.array_equal(dbg_hi[rt].cpu().numpy().astype(np.int64), ref.acc_hi), "A_hi differs"
    assert np.array_equal(dbg_lo[rt].cpu().numpy().astype(np.int64), ref.acc_lo), "A_lo differs"
    assert y_within_tolerance(y[rt], ref.y) <= REL_TOL
    del dbg_hi, dbg_lo
    y2 = rq.resq_gemm_mixed(act, packed, s.N)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)


@pytest.mark.parametrize("M,K,r,block", [
    (5, 1792 + 12544, 1792, 0),      # the down_proj input: 49 blocks of 256
    (3, 2048, 512, 512), (4, 1024, 256, 64), (3, 4096, 0, 512), (2, 528, 16, 16),
    (130, 4096, 512, 256), (3, 1024, 512, 8),
    (3, 3584 + 25088, 3584, 256),    # Llama-70B down_proj input: 98 blocks, two high units per thread
    (4, 1024, 256, 256), (3, 1280, 0, 256), (2, 512 + 4096, 512, 256), (2, 2048 + 4352, 2048, 256),
    (9, 256, 0, 256), (2, 4096 + 26624, 4096, 256),
])
def test_hadamard_quantize_fused(oracle, rq, M, K, r, block):
    # one kernel: rotate the low group, round to bf16, quantize.  (1) the rotated
    # values against the oracle's transform (fp32 sums vs the fp64 definition);
    # (2) codes, scales and lo_sum bit-exact against the oracle's quantizer fed the
    # kernel's own rotated row; (3) everything identical to the separate kernels:
    # for blocks of 256 the fused kernel takes its sums on the matrix cores, in
    # another order than the stand-alone transform, so there the rotated rows agree
    # to the neighbouring bf16 value and the stand-alone quantizer is given the
    # fused kernel's rotated row.
    s = wl.LayerShape("hq", M=M, K=K, N=1, r=r, act="student_t3", seed=K + r + M)
    x = wl.make_activations(s)
    xd = x.cuda()
    b = block or rq.resq_hadamard_block(K - r)
    x_rot = torch.zeros_like(xd)
    act = rq.resq_hadamard_quantize_act(xd, r, block, x_rot=x_rot)
    torch.cuda.synchronize()
    got = wl.bf16_bits(x_rot.cpu())
    want = oracle.hadamard(wl.bf16_bits(x), r, K, b)
    assert not got[:, :r].any(), "columns of the high group must not be written"
    g64, w64 = wl.bits_to_f64(got[:, r:]), wl.bits_to_f64(want[:, r:])
    scale = np.abs(w64).max()
    assert np.all(np.abs(g64 - w64) <= np.maximum(np.abs(w64), 2.0 ** -8 * scale) * 2.0 ** -7)
    assert np.mean(got[:, r:] == want[:, r:]) > 0.99
    rotated = wl.bf16_bits(x).copy()
    rotated[:, r:] = got[:, r:]
    compare_act_codes(oracle, act, rotated, r)
    y = rq.resq_online_hadamard(xd, r, K, block)
    torch.cuda.synchronize()
    if b == 256:
        y64 = wl.bits_to_f64(wl.bf16_bits(y.cpu())[:, r:])
        assert np.all(np.abs(g64 - y64) <= np.maximum(np.abs(y64), 2.0 ** -8 * scale) * 2.0 ** -7)
        assert np.mean(g64 == y64) > 0.99
        y = xd.clone()
        y[:, r:] = x_rot[:, r:]
    else:
        assert torch.equal(y[:, r:], x_rot[:, r:])
    act2 = rq.resq_quantize_act(y, r)
    torch.cuda.synchronize()
    for name in ("q_hi", "q_lo", "s_hi", "s_lo", "lo_sum"):
        if name in ("q_hi", "s_hi") and r == 0:
            continue
        assert torch.equal(getattr(act, name), getattr(act2, name)), name
    # and without the inspection output
    act3 = rq.resq_hadamard_quantize_act(xd, r, block)
    torch.cuda.synchronize()
    assert torch.equal(act3.q_lo, act.q_lo) and torch.equal(act3.s_lo, act.s_lo)
    if r > 0:
        assert torch.equal(act3.q_hi, act.q_hi) and torch.equal(act3.s_hi, act.s_hi)


def _random_h256_shapes(n, seed):
    rng = np.random.default_rng(seed)
    return [(int(rng.integers(1, 12)), 256 * int(rng.integers(0, 17)), 256 * int(rng.integers(1, 105)))
            for _ in range(n)]


@pytest.mark.parametrize("M,r,lo", _random_h256_shapes(12, 2468))
def test_hadamard256_quantize_random_shapes(oracle, rq, M, r, lo):
    # every instantiation of the matrix-core kernel: high widths 0 .. 4096, 1 .. 104 low blocks
    K = r + lo
    s = wl.LayerShape("h256", M=M, K=K, N=1, r=r, act="student_t3", seed=K + M)
    x = wl.make_activations(s)
    x_rot = torch.zeros((M, K), dtype=torch.bfloat16, device="cuda")
    act = rq.resq_hadamard_quantize_act(x.cuda(), r, 256, x_rot=x_rot)
    torch.cuda.synchronize()
    got = wl.bf16_bits(x_rot.cpu())
    want = oracle.hadamard(wl.bf16_bits(x), r, K, 256)
    g64, w64 = wl.bits_to_f64(got[:, r:]), wl.bits_to_f64(want[:, r:])
    scale = np.abs(w64).max()
    assert np.all(np.abs(g64 - w64) <= np.maximum(np.abs(w64), 2.0 ** -8 * scale) * 2.0 ** -7)
    assert np.mean(got[:, r:] == want[:, r:]) > 0.99
    rotated = wl.bf16_bits(x).copy()
    rotated[:, r:] = got[:, r:]
    compare_act_codes(oracle, act, rotated, r)


def test_hadamard_quantize_fused_strided_rows(oracle, rq):
    # the matrix-core path on rows that are slices of wider buffers, input and inspection output
    M, K, r = 7, 256 + 1280, 256
    s = wl.LayerShape("hqs", M=M, K=K, N=1, r=r, act="student_t3", seed=5)
    x = wl.make_activations(s)
    xbuf = torch.zeros((M, K + 40), dtype=torch.bfloat16, device="cuda")
    xbuf[:, :K] = x.cuda()
    rbuf = torch.full((M, K + 16), 3.0, dtype=torch.bfloat16, device="cuda")
    act = rq.resq_hadamard_quantize_act(xbuf[:, :K], r, 256, x_rot=rbuf[:, :K])
    ref = rq.resq_hadamard_quantize_act(x.cuda(), r, 256)
    torch.cuda.synchronize()
    assert torch.all(rbuf[:, K:] == 3.0) and torch.all(rbuf[:, :r] == 3.0), "wrote outside the low columns"
    for name in ("q_hi", "q_lo", "s_hi", "s_lo", "lo_sum"):
        assert torch.equal(getattr(act, name), getattr(ref, name)), name
    rotated = wl.bf16_bits(x).copy()
    rotated[:, r:] = wl.bf16_bits(rbuf[:, r:K].cpu())
    compare_act_codes(oracle, act, rotated, r)


# ---- asymmetric activations (the other branch of Eq. 1, the setting of Section 5.1) ----

def stored_to_codes(act, r, K):
    """GPU storage (code - 2^(N-1)) back to the oracle's unsigned codes."""
    q_hi = (act.q_hi.cpu().numpy()[:, :r].astype(np.int32) + 128).astype(np.uint8)
    from parity_util import unpack_nibbles
    q_lo = (unpack_nibbles(act.q_lo.cpu().numpy(), K - r).astype(np.int32) + 8).astype(np.uint8)
    return q_hi, q_lo


def compare_asym_codes(oracle, act, x_bits, r):
    M, K = x_bits.shape
    q_hi, q_lo, s_hi, s_lo, z_hi, z_lo = oracle.quantize_act_asym(x_bits, r)
    g_hi, g_lo = stored_to_codes(act, r, K)
    if r > 0:
        assert np.array_equal(g_hi, q_hi), "INT8 codes differ"
        assert not act.q_hi.cpu().numpy()[:, r:].any(), "padding of the high codes must be the stored code 0"
        assert np.array_equal(act.s_hi.cpu().numpy().view(np.uint32), s_hi.view(np.uint32))
        want_c = (z_hi + np.float32(128) * s_hi).astype(np.float32)
        assert np.array_equal(act.c_hi.cpu().numpy().view(np.uint32), want_c.view(np.uint32))
    if K - r > 0:
        assert np.array_equal(g_lo, q_lo), "INT4 codes differ"
        stored = q_lo.astype(np.int8) - 8
        assert np.array_equal(act.q_lo.cpu().numpy(), oracle.pack_nibbles(stored, act.ld_lo)), "packing differs"
        assert np.array_equal(act.s_lo.cpu().numpy().view(np.uint32), s_lo.view(np.uint32))
        want_c = (z_lo + np.float32(8) * s_lo).astype(np.float32)
        assert np.array_equal(act.c_lo.cpu().numpy().view(np.uint32), want_c.view(np.uint32))
        assert np.array_equal(act.lo_sum.cpu().numpy(), oracle.odd_code_sums(stored)), "lo_sum differs"


def check_layer_asym(oracle, rq, x, w, r, ldy_extra=0):
    M, K = x.shape
    N = w.shape[0]
    act = rq.resq_quantize_act_asym(x.cuda(), r)
    torch.cuda.synchronize()
    compare_asym_codes(oracle, act, wl.bf16_bits(x), r)
    packed, wq = check_weights(oracle, rq, w, r)
    ref = oracle.linear_asym(wl.bf16_bits(x), None, r, weights=wq)
    dbg_hi = torch.full((M, N), -12345, dtype=torch.int32, device="cuda")
    dbg_lo = torch.full((M, N), -12345, dtype=torch.int32, device="cuda")
    ybuf = torch.zeros((M, N + ldy_extra), dtype=torch.bfloat16, device="cuda")
    y = rq.resq_gemm_mixed_asym(act, packed, N, y=ybuf[:, :N], dbg_acc_hi=dbg_hi, dbg_acc_lo=dbg_lo)
    torch.cuda.synchronize()
    # the kernel's integer sums run over the stored codes: A_stored = A_unsigned - 2^(N-1) wsum
    if r > 0:
        want = ref.acc_hi - 128 * ref.wsum_hi[None, :]
        assert np.array_equal(dbg_hi.cpu().numpy().astype(np.int64), want), "A_hi differs"
    if K - r > 0:
        want = ref.acc_lo - 8 * ref.wsum_lo[None, :]
        assert np.array_equal(dbg_lo.cpu().numpy().astype(np.int64), want), "A_lo differs"
    rel = y_within_tolerance(y, ref.y)
    assert rel <= REL_TOL, f"bf16 output off by {rel}"
    # the same call without the accumulator dump runs the kernel variant that ships (the
    # compiler may contract its multiply-adds differently: same tolerance, not bit equality)
    y2 = rq.resq_gemm_mixed_asym(act, packed, N, y=torch.zeros_like(ybuf)[:, :N])
    torch.cuda.synchronize()
    rel2 = y_within_tolerance(y2, ref.y)
    assert rel2 <= REL_TOL, f"bf16 output (no dump) off by {rel2}"
    assert (y2.float() - y.float()).abs().max() <= 2.0 ** -7 * y.float().abs().max()
    if ldy_extra:
        assert not ybuf[:, N:].any(), "wrote past N"


@pytest.mark.parametrize("M,K,r", [(3, 2048, 256), (5, 4096, 512), (7, 4096, 0), (7, 4096, 4096),
                                   (2, 14336, 1792), (4, 264, 8),               # vector path
                                   (3, 250, 30), (5, 77, 77), (4, 90, 0), (3, 34, 2)])   # generic path
def test_quantize_act_asym(oracle, rq, M, K, r):
    s = wl.LayerShape("qa", M=M, K=K, N=1, r=r, act="student_t3", seed=M + K + 1)
    x = wl.make_activations(s)
    x[0] = x[0].abs()                        # a one-sided row
    x[1, K // 2:] = 3.0                      # a constant stretch
    act = rq.resq_quantize_act_asym(x.cuda(), r)
    torch.cuda.synchronize()
    compare_asym_codes(oracle, act, wl.bf16_bits(x), r)


def test_quantize_act_asym_constant_rows_and_ties(oracle, rq):
    x = torch.zeros(4, 512, dtype=torch.bfloat16)
    x[1] = 2.5                               # constant row: s = 1, codes 0
    x[2, :256] = torch.arange(256, dtype=torch.float32).to(torch.bfloat16) * 0.5   # ties on a power-of-two grid
    x[2, 255] = 127.5
    x[3, 256:] = torch.linspace(-3, 4.5, 256).to(torch.bfloat16)
    for r in (0, 256, 512):
        act = rq.resq_quantize_act_asym(x.cuda(), r)
        torch.cuda.synchronize()
        compare_asym_codes(oracle, act, wl.bf16_bits(x), r)


@pytest.mark.parametrize("M,K,N,r", [
    (130, 640, 300, 128), (257, 1000, 515, 104), (64, 4096, 512, 512), (200, 90, 40, 30),
    (48, 512, 256, 0), (48, 512, 256, 512),
    (1, 512, 256, 64), (16, 1000, 515, 104), (7, 2048, 272, 256), (3, 256, 256, 0),   # activation codes resident in LDS
    (24, 2048, 272, 256), (100, 4096, 130, 512), (128, 1000, 515, 104),               # chunked codes, one or several slices
])
def test_layer_asym(oracle, rq, M, K, N, r):
    x, w = wl.random_small_case(M * 5 + K, M, K, N, r, act="student_t3")
    x = (x.float() + 1.5).to(torch.bfloat16)          # off-centre activations: a real zero-point
    check_layer_asym(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", TILED_SHAPES[:4] + TILED_SHAPES[8:10] + TILED_SHAPES[11:] + TILED64_ONE_RING_SHAPES[1:5] +
                         TILED128_SHAPES[:4] + [(900, 1000, 272, 104)])
def test_layer_asym_tiled_kernels_and_many_slices(oracle, rq, M, K, N, r):
    x, w = wl.random_small_case(M * 5 + K + 1, M, K, N, r, act="student_t3")
    x = (x.float() + 1.5).to(torch.bfloat16)
    check_layer_asym(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,r,block", [
    (6, 2048, 512, 256), (4, 1792 + 12544, 1792, 0), (3, 1280, 0, 256), (3, 3584 + 25088, 3584, 256),
    (5, 2048, 512, 64), (3, 1024, 0, 512),
])
def test_hadamard_then_asym_quantize_fused(oracle, rq, M, K, r, block):
    # rotation fused in front of the asymmetric quantizer: codes, scales and offsets bit-exact
    # against the oracle's quantizer fed the kernel's own rotated row, which agrees with the
    # stand-alone transform (exactly, or to the neighbouring bf16 for blocks of 256: the
    # matrix-core path), and identical to the stand-alone quantizer on that row
    s = wl.LayerShape("hqa", M=M, K=K, N=1, r=r, act="student_t3", seed=11 + K)
    x = (wl.make_activations(s).float().abs()).to(torch.bfloat16)
    xd = x.cuda()
    b = block or rq.resq_hadamard_block(K - r)
    x_rot = torch.zeros_like(xd)
    fused = rq.resq_hadamard_quantize_act_asym(xd, r, block, x_rot=x_rot)
    y = rq.resq_online_hadamard(xd, r, K, block)
    torch.cuda.synchronize()
    assert not x_rot[:, :r].any()
    if b == 256:
        g64 = wl.bits_to_f64(wl.bf16_bits(x_rot.cpu())[:, r:])
        y64 = wl.bits_to_f64(wl.bf16_bits(y.cpu())[:, r:])
        scale = np.abs(y64).max()
        assert np.all(np.abs(g64 - y64) <= np.maximum(np.abs(y64), 2.0 ** -8 * scale) * 2.0 ** -7)
        assert np.mean(g64 == y64) > 0.99
    else:
        assert torch.equal(y[:, r:], x_rot[:, r:])
    rotated = xd.clone()
    rotated[:, r:] = x_rot[:, r:]
    compare_asym_codes(oracle, fused, wl.bf16_bits(rotated.cpu()), r)
    two = rq.resq_quantize_act_asym(rotated, r)
    plain = rq.resq_quantize_act_asym(xd, r, hadamard_block=block or -1)   # the entry without the inspection output
    torch.cuda.synchronize()
    for name in ("q_hi", "q_lo", "s_hi", "s_lo", "c_hi", "c_lo", "lo_sum"):
        if name in ("q_hi", "s_hi", "c_hi") and r == 0:
            continue
        assert torch.equal(getattr(fused, name), getattr(two, name)), name
        assert torch.equal(getattr(fused, name), getattr(plain, name)), name


# ---- short rows: per-head quantization of a K/V cache entry (Section 4.3) ----------

@pytest.mark.parametrize("rows,d_head,r", [(8 * 37, 128, 16), (8 * 37 + 3, 128, 16), (50, 64, 8),
                                           (21, 512, 64), (33, 128, 0), (33, 128, 128), (5, 8, 8)])
def test_kv_cache_head_quantization(oracle, rq, rows, d_head, r):
    # [tokens x heads, d_head] rows, each a group pair of its own: symmetric and asymmetric
    # (the paper quantizes the cache per head, asymmetrically), one wavefront per row
    s = wl.LayerShape("kv", M=rows, K=d_head, N=1, r=r, act="student_t3", seed=rows + d_head)
    x = wl.make_activations(s)
    x[0] = 0
    check_act_codes(oracle, rq, x, r)
    act = rq.resq_quantize_act_asym(x.cuda(), r)
    torch.cuda.synchronize()
    compare_asym_codes(oracle, act, wl.bf16_bits(x), r)


@pytest.mark.parametrize("rows,d_head,r,pad", [(8 * 37, 128, 16, 0), (8 * 37 + 3, 128, 16, 8), (50, 64, 8, 0),
                                               (21, 512, 64, 4), (33, 128, 0, 0), (33, 128, 128, 0), (5, 8, 8, 0),
                                               (4099, 256, 32, 0), (7, 16, 8, 0)])
def test_kv_cache_compact_rows(oracle, rq, rows, d_head, r, pad):
    # the compact cache format (Section 5.1, Appendix C): every byte of every row against the
    # oracle's layout of the oracle's own codes, scales and zero-points; rows wider than needed
    # keep their padding; the reader against the oracle's reconstruction in fp64
    s = wl.LayerShape("kvc", M=rows, K=d_head, N=1, r=r, act="student_t3", seed=rows + d_head + r)
    x = wl.make_activations(s)
    x[0] = 0                                   # a constant head: scale 1, codes 0
    if rows > 2:
        x[2] = x[2].abs()                      # a one-sided head: a real zero-point
    need = rq.resq_kv_cache_row_bytes(d_head, r)
    assert need == oracle.kv_cache_row_bytes(d_head, r)
    buf = torch.full((rows, need + pad), 0xEE, dtype=torch.uint8, device="cuda")
    xbuf = torch.zeros((rows, d_head + 8), dtype=torch.bfloat16, device="cuda")
    xbuf[:, :d_head] = x.cuda()
    cache = rq.resq_quantize_kv_cache(xbuf[:, :d_head], r, cache=buf)
    torch.cuda.synchronize()
    q_hi, q_lo, s_hi, s_lo, z_hi, z_lo = oracle.quantize_act_asym(wl.bf16_bits(x), r)
    want = oracle.pack_kv_cache(q_hi, q_lo, s_hi, z_hi, s_lo, z_lo)
    got = cache.cpu().numpy()
    assert np.array_equal(got[:, :need], want), "cache rows differ"
    assert np.all(got[:, need:] == 0xEE), "wrote past the row"
    # the reader: fp32 multiply-add rounded to bf16 against the fp64 reconstruction
    back = rq.resq_dequantize_kv_cache(cache, d_head, r)
    torch.cuda.synchronize()
    ref = oracle.dequantize_kv_cache(want, d_head, r)
    b64 = wl.bits_to_f64(wl.bf16_bits(back.cpu()))
    assert np.all(np.abs(b64 - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-30)
    # and what comes back is within half a quantization step (plus the bf16 rounding of the
    # reconstructed value, which is at most half a step away from the input) of what went in
    x64 = wl.bits_to_f64(wl.bf16_bits(x))
    step = np.concatenate([np.repeat(s_hi[:, None], r, 1), np.repeat(s_lo[:, None], d_head - r, 1)], axis=1).astype(np.float64)
    assert np.all(np.abs(b64 - x64) <= 0.5 * step * (1 + 2.0 ** -7) + 2.0 ** -8 * np.abs(x64))


def test_kv_cache_no_rows(rq):
    c = rq.resq_quantize_kv_cache(torch.empty((0, 128), dtype=torch.bfloat16, device="cuda"), 16)
    assert c.shape == (0, 88)


def test_online_head_projection_as_uniform_int8_layer(oracle, rq):
    # the 8-bit online projection of queries and keys (U_C, d_head x d_head, Section 4.3):
    # rows = tokens x heads, K = N = d_head, every column in the high group
    g = torch.Generator().manual_seed(4)
    rows, d = 32 * 40, 128
    x = torch.randn(rows, d, generator=g).to(torch.bfloat16)
    u = torch.linalg.qr(torch.randn(d, d, generator=g))[0].contiguous().to(torch.bfloat16)   # an orthogonal U_C
    check_layer(oracle, rq, x, u, d)


@pytest.mark.parametrize("rows,d,ldx_extra,ldy_extra", [
    (32 * 40, 128, 0, 0), (32 * 40 + 5, 128, 0, 0), (1, 128, 0, 0), (31, 128, 8, 4), (33, 128, 16, 3),
    (700, 64, 0, 0), (45, 64, 8, 1), (4096 * 5 + 17, 128, 0, 0),      # the last: more tiles than wavefronts in flight
])
def test_project_heads_fused(oracle, rq, rows, d, ldx_extra, ldy_extra):
    # the same projection as one kernel: row quantizer, INT8 product and dequantization,
    # against the oracle's layer with every column high, and against the two-kernel path
    g = torch.Generator().manual_seed(rows + d)
    xbuf = torch.randn(rows, d + ldx_extra, generator=g).to(torch.bfloat16)
    xbuf[rows // 2] = 0                                              # an all-zero head: scale 1, output 0
    x = xbuf[:, :d]
    u = torch.linalg.qr(torch.randn(d, d, generator=g))[0].contiguous().to(torch.bfloat16)
    packed = rq.resq_pack_weights(u.cuda(), d)
    ybuf = torch.zeros((rows, d + ldy_extra), dtype=torch.bfloat16, device="cuda")
    y = rq.resq_project_heads(xbuf.cuda()[:, :d], packed, y=ybuf[:, :d])
    torch.cuda.synchronize()
    ref = oracle.linear(wl.bf16_bits(x.contiguous()), wl.bf16_bits(u), d)
    rel = y_within_tolerance(y, ref.y)
    assert rel <= REL_TOL, f"projected heads off by {rel}"
    assert not ybuf[:, d:].any(), "wrote past d_head"
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(x.contiguous().cuda(), d), packed, d)
    assert torch.equal(y, two)


# Rows whose codes come from refined quotients, and beside them in one wavefront rows whose scale is at or past either end of
# what these take: the codes, and with them the outputs, of the row quantizer and the layer
@pytest.mark.parametrize("d", [64, 128])
def test_project_heads_scales_and_ties(rq, d):
    g = torch.Generator().manual_seed(d)
    rows = 6000
    x = torch.randint(-254, 255, (rows, d), generator=g).float() * 0.5     # every quotient of a scale of 1 a half or whole number
    x[:, 0] = 127.0
    x[2000:4000] = torch.randn(2000, d, generator=g)
    x *= torch.exp2(torch.randint(-20, 20, (rows, 1), generator=g).float())
    for k, e in enumerate((-133, -126, -97, -96, -91, -90, -89, -84, -83, 92, 93, 94, 99, 100, 101, 119)):
        x[4000 + k * 16] = torch.randn(d, generator=g).clamp(-1, 1) * 2.0 ** e
        x[4300 + k * 16:4316 + k * 16] = torch.randn(16, d, generator=g).clamp(-1, 1) * 2.0 ** e
    x[5000] = 0.0
    x = x.bfloat16().cuda()
    packed = rq.resq_pack_weights((torch.randn(d, d, generator=g) / d ** 0.5).bfloat16().cuda(), d)
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(x, d), packed, d)
    assert torch.equal(rq.resq_project_heads(x, packed), two)
    x[100, 3], x[117, 5] = float("inf"), float("nan")
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(x, d), packed, d)
    got = rq.resq_project_heads(x, packed)
    fine = torch.ones(rows, dtype=torch.bool)
    fine[100] = fine[117] = False
    assert torch.equal(got[fine], two[fine])


# Rows with a NaN at each place of a lane's piece, and the neighbours in the wavefront of these and of rows with an infinity
# (whose own outputs, codes of finite values times an infinite scale, are nobody's): what the row quantizer and the layer give
@pytest.mark.parametrize("d", [64, 128])
def test_project_heads_not_finite(rq, d):
    g = torch.Generator().manual_seed(d + 1)
    x = torch.randn(40 * d, d, generator=g).clamp(-3, 3)
    for k in range(d):
        x[40 * k, (k + 8) % d] = 3.5   # the maximum is in another unit than the NaN, which takes its own unit out of it
        x[40 * k, k] = float("nan")
        x[40 * k + 21, k] = (-1.0) ** k * float("inf")
    x[7, :d // 2], x[23] = float("nan"), float("inf")
    x = x.bfloat16().cuda()
    packed = rq.resq_pack_weights((torch.randn(d, d, generator=g) / d ** 0.5).bfloat16().cuda(), d)
    two = rq.resq_gemm_mixed(rq.resq_quantize_act(x, d), packed, d)
    got = rq.resq_project_heads(x, packed)
    scaled = ~x.isinf().any(1)
    assert torch.equal(got[scaled], two[scaled]) and two[scaled].isfinite().all()


def test_project_heads_no_rows(rq):
    packed = rq.resq_pack_weights(torch.eye(128, dtype=torch.bfloat16, device="cuda"), 128)
    y = rq.resq_project_heads(torch.empty((0, 128), dtype=torch.bfloat16, device="cuda"), packed)
    assert y.shape == (0, 128)


# ---- gate/up as one layer with the gated activation in the epilogue ----------------

@pytest.mark.parametrize("M,K,F,r", [
    (130, 640, 150, 128), (64, 512, 256, 64), (300, 1024, 384, 0), (40, 256, 130, 256),
    (1, 512, 128, 64), (16, 1000, 257, 104), (5, 256, 64, 0),                             # activation codes resident in LDS
    (20, 1000, 257, 104), (128, 2048, 136, 256), (900, 1000, 136, 104),                   # chunked codes, one or several slices
    (1030, 640, 150, 128), (1100, 1000, 257, 104), (1153, 256, 128, 0), (1153, 256, 128, 256),   # above 1024 tokens: tiled kernel, 64 x 128 tiles
    (300, 256, 2050, 32), (130, 520, 4100, 64),                                           # ... and below, on wide layers
    (1153, 256, 1050, 32), (1300, 640, 1150, 128),                                        # ... 257 to 512 such tiles: one ring
    (2100, 256, 1100, 32), (4100, 256, 550, 0), (4100, 256, 550, 256), (1100, 1000, 2100, 104),  # 128 x 128 tiles
    (1925, 3200, 2250, 128), (1921, 3202, 2200, 128),                                     # ... with the low group in fp8, without and with padding
])
def test_layer_swiglu(oracle, rq, M, K, F, r):
    x, w = wl.random_small_case(M + K + F, M, K, 2 * F, r, act="student_t3")
    w = (w.float() * 8).to(torch.bfloat16)     # outputs of order one, so that silu is exercised off its linear part
    act = rq.resq_quantize_act(x.cuda(), r)
    packed = rq.resq_pack_weights(w.cuda(), r)
    ref = oracle.swiglu(oracle.linear(wl.bf16_bits(x), wl.bf16_bits(w), r).y)
    ybuf = torch.zeros((M, F + 8), dtype=torch.bfloat16, device="cuda")
    y = rq.resq_gemm_mixed_swiglu(act, packed, 2 * F, y=ybuf[:, :F])
    torch.cuda.synchronize()
    rel = y_within_tolerance(y, ref)
    assert rel <= REL_TOL, f"gated output off by {rel}"
    assert not ybuf[:, F:].any(), "wrote past F"
    # and it is the two-step computation on the plain layer's fp32 result, up to bf16 rounding in between
    z = rq.resq_gemm_mixed(act, packed, 2 * F).float()
    two_step = torch.nn.functional.silu(z[:, 0::2]) * z[:, 1::2]
    assert (y.float() - two_step).abs().max() <= 0.03 * two_step.abs().max()


# ---- SNR per rank: the accuracy-side figure of the rank ablation (Section 5.4) -----

def test_snr_per_rank_matches_oracle(oracle, rq):
    # Qwen2.5-72B MLP proportions at 1/16 scale, r in {0, K/8, K/4}: the output SNR of the
    # HIP path equals the oracle's (same codes, bf16 rounding aside) and grows with r
    import numpy as np
    shape = wl.LayerShape("snr", M=96, K=512, N=1848, r=0, act="student_t3", outliers="one_percent_hi", seed=5)
    x, w = wl.make_activations(shape), wl.make_weights(shape)
    xb, wb = wl.bf16_bits(x), wl.bf16_bits(w)
    ref = wl.bits_to_f64(xb) @ wl.bits_to_f64(wb).T
    got = []
    for r in (0, 64, 128):
        act = rq.resq_quantize_act(x.cuda(), r)
        y = rq.resq_gemm_mixed(act, rq.resq_pack_weights(w.cuda(), r), shape.N)
        torch.cuda.synchronize()
        snr_gpu = oracle.snr_db(ref, y.float().cpu().numpy())
        snr_cpu = oracle.snr_db(ref, oracle.linear(xb, wb, r).y)
        assert abs(snr_gpu - snr_cpu) < 0.05, (r, snr_gpu, snr_cpu)
        got.append(snr_gpu)
    assert got[0] < got[1] < got[2], got


# ---- the variants over the same dispatch boundaries --------------------------------

@pytest.mark.parametrize("M,K,N,r", _random_layer_shapes(16, 77))
def test_layer_asym_random_shapes(oracle, rq, M, K, N, r):
    x, w = wl.random_small_case(M * 3 + K + N, M, K, N, r, act="student_t3")
    x = (x.float() + 1.5).to(torch.bfloat16)
    check_layer_asym(oracle, rq, x, w, r, ldy_extra=8 if N % 4 == 0 else 3)


@pytest.mark.parametrize("M,K,N,r", _random_layer_shapes(16, 99))
def test_layer_swiglu_random_shapes(oracle, rq, M, K, N, r):
    F = max(N // 2, 1)
    x, w = wl.random_small_case(M + K + F, M, K, 2 * F, r, act="student_t3")
    w = (w.float() * 8).to(torch.bfloat16)
    act = rq.resq_quantize_act(x.cuda(), r)
    packed = rq.resq_pack_weights(w.cuda(), r)
    ref = oracle.swiglu(oracle.linear(wl.bf16_bits(x), wl.bf16_bits(w), r).y)
    ybuf = torch.zeros((M, F + 8), dtype=torch.bfloat16, device="cuda")
    y = rq.resq_gemm_mixed_swiglu(act, packed, 2 * F, y=ybuf[:, :F])
    torch.cuda.synchronize()
    assert y_within_tolerance(y, ref) <= REL_TOL
    assert not ybuf[:, F:].any(), "wrote past F"
