"""Parity of single operations (RMSNorm, the three GEMM epilogues) against the CPU oracle, through
the C ABI, at shapes that span several tiles and ragged tails in M, N and K."""
import numpy as np
import pytest

from oracle import decoder as O
from tests import _util as U

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.mark.parametrize("fp32", [False, True], ids=["bf16", "fp32dbg"])
@pytest.mark.parametrize("T,H", [(1, 256), (7, 256), (130, 4096), (3, 8192), (5, 688)])
def test_rmsnorm(torch, fp32, T, H):
    from paper_2412_17246_amd import op_rmsnorm
    rng = np.random.default_rng([7, T, H])
    x, xr = U.f64_to_device(rng.standard_normal((T, H)) * 3.0, fp32)
    g, gr = U.f64_to_device(1.0 + 0.1 * rng.standard_normal(H), False)
    y = torch.empty_like(x)
    op_rmsnorm(x, g, y, 1e-5, fp32_debug=fp32)
    want = O.rmsnorm(xr, gr, 1e-5)
    err = U.rel_err(U.from_device(y), want)
    assert err <= (U.FP32_TOL if fp32 else U.BF16_TOL), err
    U.assert_rms(U.from_device(y), want, U.RMS_FP32 if fp32 else U.RMS_BF16_OP)


def test_rmsnorm_constant_vector(torch):
    from paper_2412_17246_amd import op_rmsnorm
    x = torch.full((2, 256), 3.0, dtype=torch.bfloat16, device="cuda")
    g = torch.ones(256, dtype=torch.bfloat16, device="cuda")
    y = torch.empty_like(x)
    op_rmsnorm(x, g, y, 1e-5)
    want = 3.0 / np.sqrt(9.0 + 1e-5)
    assert np.max(np.abs(U.from_device(y) - want)) <= 2 ** -8


GEMM_SHAPES = [
    # M, N, K: single tile, ragged M, ragged N (not a multiple of 32), K tail (688 = 10*64 + 48)
    (64, 128, 64), (1, 768, 256), (65, 768, 256), (200, 688, 256), (333, 256, 688), (130, 1376, 2048),
    (257, 4096, 512), (31, 48, 72),
    # 65 .. 2048 rows, K a multiple of 64: ragged M, N tails, one and many K tiles
    (300, 768, 256), (700, 688, 1024), (513, 520, 64), (1030, 1024, 2048), (257, 132, 128),
    # large-tile kernel, more than 256 tiles with a small last round (272 / 544 tiles): with a workspace the last tiles are
    # split over K
    (4300, 4092, 1024),
    # decode-sized problems (M <= 64, K a multiple of 64): the split-K kernel when a workspace is given
    (64, 4096, 4096), (33, 688, 1024), (7, 260, 640), (48, 1024, 14336),
    # few rows and long K: several ranges of K, ragged last tile
    (128, 1024, 4096), (97, 688, 1024), (100, 256, 4096), (250, 512, 2048),
    # a few hundred rows, fewer tiles than CUs
    (200, 4096, 2048), (600, 1376, 4096),
    # one row of tiles, a power-of-two row pitch and 32 k-tiles per workgroup: tiles start their walk over K at different
    # places (and two rows of tiles, which start by XCD)
    (40, 7168, 4096), (150, 7168, 4096),
]


@pytest.mark.parametrize("fp32", [False, True], ids=["bf16", "fp32dbg"])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm(torch, fp32, mode, M, N, K):
    from paper_2412_17246_amd import op_gemm
    rng = np.random.default_rng([11, mode, M, N, K])
    a, ar = U.f64_to_device(rng.standard_normal((M, K)), fp32)
    rows = 2 * N if mode == 2 else N
    w, wr = U.f64_to_device(rng.standard_normal((rows, K)) * (2.0 / np.sqrt(K)), False)
    r, rr = U.f64_to_device(rng.standard_normal((M, N)), fp32)
    c = torch.zeros_like(r)
    from paper_2412_17246_amd import op_gemm_workspace_bytes
    nws = op_gemm_workspace_bytes(mode, M, N, K, fp32_debug=fp32)
    ws = torch.empty(max(nws, 16), dtype=torch.uint8, device="cuda")
    op_gemm(mode, a, w, r if mode == 1 else None, c, M, N, K, fp32_debug=fp32, workspace=ws if nws else None)
    if nws and not fp32:
        # the same problem without a workspace takes the kernel that needs none; both must pass
        c2 = torch.zeros_like(r)
        op_gemm(mode, a, w, r if mode == 1 else None, c2, M, N, K)
    else:
        c2 = None
    if mode == 0:
        want = O.linear(ar, wr)
    elif mode == 1:
        want = rr + O.linear(ar, wr)
    else:
        want = O.swiglu(ar, wr[:N], wr[N:])
    got = U.from_device(c)
    err = U.rel_err(got, want)
    assert err <= (U.FP32_TOL if fp32 else U.BF16_TOL), err
    U.assert_rms(got, want, U.RMS_FP32 if fp32 else U.RMS_BF16_OP)
    if not fp32:
        # bf16 output rounding alone bounds the error far below the gate; a wrong tile would not
        assert U.mixed_err(got, want, 8e-3) <= 1.0
    if c2 is not None:
        assert U.rel_err(U.from_device(c2), want) <= U.BF16_TOL


@pytest.mark.parametrize("case", range(10))
def test_gemm_random_problems(torch, case):
    """Seeded random problems: any N (odd ones take the element-wise store path), K any multiple of 8, row counts on
    both sides of every kernel boundary; all three modes, both builds."""
    import random
    rnd = random.Random(case)
    M = rnd.choice([1, 2, 63, 64, 65, 255, 256, 257, rnd.randint(1, 900)])
    N = rnd.choice([rnd.randint(1, 1500), 4 * rnd.randint(1, 400), 8 * rnd.randint(1, 300), 256 * rnd.randint(1, 6)])
    K = 8 * rnd.choice([rnd.randint(1, 300), 8 * rnd.randint(1, 64)])
    for mode in (0, 1, 2):
        for fp32 in (False, True):
            test_gemm(torch, fp32, mode, M, N, K)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K,whole,ranges", [
    (2049, 4, 64, True, 1), (2177, 252, 128, True, 1), (2049, 264, 192, True, 1), (2305, 520, 448, True, 1),
    (2049, 260, 512, False, 2), (2111, 512, 640, False, 2), (2600, 1004, 1088, False, 2),
    (2305, 6660, 512, True, 2), (2305, 6656, 576, True, 2)])
def test_gemm_large_tile_edges(torch, mode, M, N, K, whole, ranges):
    """The large-tile kernel around its 16-row blocks and 256-wide tiles, rows of 8k and 8k + 4 features, one k-tile
    to many, all tiles whole, all split over K, and whole ones with a split last round."""
    from paper_2412_17246_amd import op_gemm_plan
    from paper_2412_17246_amd.binding import BZ_GEMM_LARGE
    p = op_gemm_plan(mode, M, N, K)
    assert p.kernel == BZ_GEMM_LARGE and (p.whole_tiles > 0) == whole and min(p.ranges, 2) == ranges
    test_gemm(torch, False, mode, M, N, K)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(65, 36, 64), (96, 4100, 192), (129, 2064, 1024), (225, 5120, 640), (257, 4092, 4096),
                                   (321, 3004, 320), (552, 7172, 2048), (2048, 520, 448), (65, 4, 64), (272, 252, 128),
                                   (511, 260, 192), (513, 1004, 448), (769, 520, 640)])
def test_gemm_mid_sized_edges(torch, mode, M, N, K):
    """The mid-sized kernel's tiles: one row past a tile, rows of 8k and 8k + 4 features, one k-tile, fewer than the
    ring holds, many; one range of K and several; one row of tiles (walks that start inside K among them) and more."""
    from paper_2412_17246_amd import op_gemm_plan
    from paper_2412_17246_amd.binding import BZ_GEMM_MID
    assert op_gemm_plan(mode, M, N, K).kernel == BZ_GEMM_MID
    test_gemm(torch, False, mode, M, N, K)


@pytest.mark.parametrize("mode,N,K,narrow", [(0, 8204, 4104, False), (1, 4100, 8256, False), (2, 5000, 4160, False), (1, 33000, 1024, True),
                                            (2, 16648, 1032, True), (2, 11004, 1536, True)])
def test_gemm_long_streams_of_few_and_many_rows(torch, mode, N, K, narrow):
    """Decode-sized products of 64 MiB of weights and more: up to 32 rows the activations take half of the stage, with more tiles
    than CUs it has fewer stages, and tiles narrow down to fill the chip; with and without a K tail.  A row's bits do not depend
    on the other rows."""
    from paper_2412_17246_amd import op_gemm, op_gemm_plan, op_gemm_workspace_bytes
    from paper_2412_17246_amd.binding import BZ_GEMM_DECODE
    rng = np.random.default_rng([12, mode, N, K])
    a, ar = U.f64_to_device(rng.standard_normal((64, K)), False)
    w, wr = U.f64_to_device(rng.standard_normal((2 * N if mode == 2 else N, K)) * (2.0 / np.sqrt(K)), False)
    r, rr = U.f64_to_device(rng.standard_normal((64, N)), False)
    assert w.numel() * 2 >= 64 << 20
    want = O.linear(ar, wr) if mode == 0 else rr + O.linear(ar, wr) if mode == 1 else O.swiglu(ar, wr[:N], wr[N:])
    whole = None
    for M in (64, 33, 32, 31, 5):
        p = op_gemm_plan(mode, M, N, K)
        assert p.kernel == BZ_GEMM_DECODE and (p.tile_cols < 96) == narrow
        ws = torch.empty(op_gemm_workspace_bytes(mode, M, N, K), dtype=torch.uint8, device="cuda")
        c = torch.zeros_like(r[:M])
        op_gemm(mode, a[:M], w, r[:M] if mode == 1 else None, c, M, N, K, workspace=ws)
        got = U.from_device(c)
        assert U.rel_err(got, want[:M]) <= U.BF16_TOL
        U.assert_rms(got, want[:M], U.RMS_BF16_OP)
        whole = c if whole is None else whole
        assert torch.equal(c.view(torch.int16), whole[:M].view(torch.int16)), M


@pytest.mark.parametrize("mode,M,N,K,cols,ranges", [(0, 5, 17100, 264, 40, 1), (1, 33, 17100, 320, 40, 1), (2, 64, 8708, 192, 40, 1),
                                                   (0, 31, 8708, 1536, 40, 1), (2, 33, 5004, 520, 40, 1), (1, 64, 1020, 2048, 32, 8)])
def test_gemm_short_streams_in_narrow_tiles(torch, mode, M, N, K, cols, ranges):
    """Short streams whose tiles narrow down to 40 and 32 of 64 rows, in several rounds of workgroups and in one, K cut and not."""
    from paper_2412_17246_amd import op_gemm_plan
    p = op_gemm_plan(mode, M, N, K)
    assert (p.tile_cols, p.ranges) == (cols, ranges)
    test_gemm(torch, False, mode, M, N, K)


@pytest.mark.parametrize("mode,M,N,K", [(0, 300, 8300, 1984), (0, 300, 8300, 2048), (1, 300, 8300, 2112), (2, 420, 8300, 2496),
                                        (0, 700, 4100, 2112)])
def test_gemm_mid_sized_walks(torch, mode, M, N, K):
    """Two rows of tiles over one range of 31 k-tiles (every walk from its start), and of 32, 33 and 39 (an XCD's start of its
    own, the walk wrapping around); four rows of tiles (in step again)."""
    from paper_2412_17246_amd import op_gemm_plan
    from paper_2412_17246_amd.binding import BZ_GEMM_MID
    p = op_gemm_plan(mode, M, N, K)
    assert p.kernel == BZ_GEMM_MID and p.tiles_m > 1 and p.ranges == 1
    test_gemm(torch, False, mode, M, N, K)


@pytest.mark.parametrize("mode,M,N,K,cols,ranges", [(0, 210, 2048, 16384, 64, 4), (2, 150, 4096, 4096, 64, 1), (2, 170, 2048, 16384, 128, 4),
                                                   (2, 300, 1536, 16384, 128, 5), (0, 330, 1536, 16384, None, 8)])
def test_gemm_mid_sized_walks_in_step(torch, mode, M, N, K, cols, ranges):
    """Two rows of tiles at distances at which all XCDs start at the same place: tiles 2^11 and 2^8 times the starts apart, or 2 MiB;
    eight ranges."""
    from paper_2412_17246_amd import op_gemm_plan
    from paper_2412_17246_amd.binding import BZ_GEMM_MID
    p = op_gemm_plan(mode, M, N, K)
    assert (p.kernel, p.ranges) == (BZ_GEMM_MID, ranges) and p.tiles_m in (2, 3)
    if cols:
        apart, start = (cols // 2 if mode == 2 else cols) * K * 2, K // 64 // ranges * 128 // 8
        assert p.tile_cols == cols and apart in (start << 11, start << 8, 2 << 20)
    test_gemm(torch, False, mode, M, N, K)


# Every tile of the mid-sized kernel, plain and gated, with one row of tiles where a problem of this size has that, and more:
# K of one k-tile, and of twice what the tile's ring holds and more.  (rows, weight rows of the tile; mode, M, N, K)
MID_TILES = [
    (96, 128, 0, 132, 4180, 1856), (96, 128, 0, 264, 7688, 64), (96, 128, 1, 67, 8300, 1920),
    (96, 128, 2, 129, 6684, 640), (96, 128, 2, 133, 6228, 64), (128, 64, 0, 148, 1900, 640),
    (128, 64, 1, 129, 4, 64), (128, 64, 0, 75, 3596, 640), (128, 64, 0, 65, 4, 64), (128, 64, 2, 131, 4, 640),
    (128, 64, 2, 129, 4, 64), (128, 64, 2, 65, 4, 640), (128, 64, 2, 65, 4, 64), (128, 96, 1, 135, 9016, 640),
    (128, 96, 0, 129, 8296, 64), (128, 96, 0, 68, 5728, 2112), (128, 96, 2, 137, 4176, 640),
    (128, 96, 2, 129, 4204, 64), (128, 96, 2, 71, 8364, 640), (128, 96, 2, 67, 8324, 64),
    (160, 128, 1, 391, 7932, 512), (160, 128, 1, 386, 7740, 64), (160, 128, 2, 221, 6224, 512),
    (160, 128, 2, 194, 6252, 64), (160, 192, 1, 593, 8424, 384), (160, 192, 0, 779, 6212, 64),
    (160, 192, 2, 258, 8900, 384), (160, 192, 2, 258, 8540, 64), (160, 256, 0, 910, 9428, 384),
    (160, 256, 1, 905, 9236, 64), (160, 256, 2, 476, 8284, 384), (160, 256, 2, 449, 8292, 64),
    (192, 96, 1, 786, 3100, 512), (192, 96, 1, 385, 6236, 64), (192, 96, 0, 132, 8412, 2368),
    (192, 96, 2, 1082, 1184, 512), (192, 96, 2, 1048, 1156, 64), (192, 96, 2, 131, 8488, 512),
    (192, 96, 2, 129, 8324, 64), (192, 128, 1, 484, 8452, 512), (192, 128, 1, 962, 4124, 64),
    (192, 128, 2, 978, 2052, 512), (192, 128, 2, 641, 3164, 64), (192, 192, 0, 1059, 6212, 384),
    (192, 192, 1, 1057, 6176, 64), (192, 192, 2, 335, 9060, 384), (192, 192, 2, 326, 8268, 64),
    (224, 192, 1, 770, 9244, 384), (224, 192, 1, 770, 9408, 64), (224, 192, 2, 397, 8252, 384),
    (224, 192, 2, 397, 8308, 64), (256, 96, 1, 1009, 5160, 384), (256, 96, 0, 388, 10344, 64),
    (256, 96, 2, 395, 5436, 384), (256, 96, 2, 387, 5644, 64), (256, 96, 2, 196, 8316, 384),
    (256, 96, 2, 199, 8236, 64), (256, 128, 0, 963, 6188, 384), (256, 128, 0, 646, 9264, 64),
    (256, 128, 2, 401, 7740, 384), (256, 128, 2, 970, 3076, 64),
]


@pytest.mark.parametrize("rows,cols,mode,M,N,K", MID_TILES)
def test_gemm_every_mid_sized_tile(torch, rows, cols, mode, M, N, K):
    from paper_2412_17246_amd import op_gemm_plan
    from paper_2412_17246_amd.binding import BZ_GEMM_MID
    p = op_gemm_plan(mode, M, N, K)
    assert (p.kernel, p.tile_rows, p.tile_cols) == (BZ_GEMM_MID, rows, cols)
    test_gemm(torch, False, mode, M, N, K)


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", [(1, 256, 688), (64, 36, 8), (17, 68, 72), (5, 2048, 1016), (33, 9216, 4104),
                                   (64, 36, 200), (17, 68, 328), (9, 132, 248), (1, 4, 440)])
def test_gemm_decode_sized_k_tails(torch, mode, M, N, K):
    """The decode kernel where K is no multiple of its 64-wide tiles: a tail of one to seven 8-element pieces, alone, in a
    range of its own and behind others; small matrices and (last) the 128-row tiles of the long streams."""
    test_gemm(torch, False, mode, M, N, K)


def test_gemm_residual_in_place_and_identity(torch):
    from paper_2412_17246_amd import op_gemm
    M, N = 150, 256
    rng = np.random.default_rng(5)
    a, ar = U.f64_to_device(rng.standard_normal((M, N)), False)
    eye = torch.eye(N, dtype=torch.bfloat16, device="cuda")
    x, xr = U.f64_to_device(rng.standard_normal((M, N)), False)
    op_gemm(1, a, eye, x, x, M, N, N)           # x <- x + a, residual aliased with the output
    got = U.from_device(x)
    want = U.f64(__import__("workloads").bf16_bits_from_f32((xr + ar).astype(np.float32)))
    assert np.array_equal(got, want)            # one rounding of an exact sum


@pytest.mark.parametrize("M,N,K", [(100, 512, 1024), (600, 1376, 4096), (4300, 4096, 1024)])
def test_gemm_residual_in_place_with_split_schedules(torch, M, N, K):
    # the residual aliased with the output, in the schedules that go through partial sums or partial tiles
    from paper_2412_17246_amd import op_gemm, op_gemm_workspace_bytes
    rng = np.random.default_rng([17, M, N, K])
    a, ar = U.f64_to_device(rng.standard_normal((M, K)), False)
    w, wr = U.f64_to_device(rng.standard_normal((N, K)) * (2.0 / np.sqrt(K)), False)
    x, xr = U.f64_to_device(rng.standard_normal((M, N)), False)
    nws = op_gemm_workspace_bytes(1, M, N, K)
    assert nws > 0
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    op_gemm(1, a, w, x, x, M, N, K, workspace=ws)
    assert U.rel_err(U.from_device(x), xr + O.linear(ar, wr)) <= U.BF16_TOL


def test_gemm_is_deterministic(torch):
    from paper_2412_17246_amd import op_gemm
    M, N, K = 300, 768, 688
    rng = np.random.default_rng(9)
    a, _ = U.f64_to_device(rng.standard_normal((M, K)), False)
    w, _ = U.f64_to_device(rng.standard_normal((N, K)) * 0.05, False)
    c1 = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    c2 = torch.empty_like(c1)
    op_gemm(0, a, w, None, c1, M, N, K)
    op_gemm(0, a, w, None, c2, M, N, K)
    torch.cuda.synchronize()
    assert torch.equal(c1.view(torch.int16), c2.view(torch.int16))
    # split last round: partial tiles are added in a fixed order
    from paper_2412_17246_amd import op_gemm_workspace_bytes
    M, N, K = 4352, 4096, 512
    nws = op_gemm_workspace_bytes(0, M, N, K)
    assert nws > 0
    a, _ = U.f64_to_device(rng.standard_normal((M, K)), False)
    w, _ = U.f64_to_device(rng.standard_normal((N, K)) * 0.05, False)
    ws = torch.empty(nws, dtype=torch.uint8, device="cuda")
    c1 = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    c2 = torch.empty_like(c1)
    op_gemm(0, a, w, None, c1, M, N, K, workspace=ws)
    ws.fill_(0xFF)                               # stale scratch contents must not matter
    op_gemm(0, a, w, None, c2, M, N, K, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(c1.view(torch.int16), c2.view(torch.int16))
