"""GPU parity: q8_quantize_matrix, q8_gemv, q8_gemm_narrow against the CPU oracle (Section 3)."""
import numpy as np
import pytest
import torch

from parity import assert_close, assert_same, np_

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import paper_1804_05038_amd as q
    return q


@pytest.fixture(scope="module")
def ctx(q):
    return q.Context()


def _w(rng, rows, cols, std=0.05):
    return (rng.standard_normal((rows, cols)) * std).astype(np.float32)


@pytest.mark.parametrize("rows,cols", [(768, 256), (3072, 512), (1024, 2048), (33, 620), (7, 5), (1, 16), (2500, 1000)])
def test_quantize_matrix_bit_exact(q, ctx, oracle, rows, cols):
    rng = np.random.default_rng(rows * 7 + cols)
    W = _w(rng, rows, cols)
    W[rng.integers(rows), rng.integers(cols)] = 0.0
    m = q.q8_quantize_matrix(ctx, W)
    Wq, s = oracle.quantize_matrix(W)
    assert m.ld == Wq.shape[1] and m.scale == float(s)
    assert_same(m.data, Wq, "Wq")


def test_quantize_matrix_zero_and_halfway(q, ctx, oracle):
    m = q.q8_quantize_matrix(ctx, np.zeros((4, 20), np.float32))
    assert m.scale == 1.0 and not np_(m.data).any()
    W = np.array([[127, -63.5, 0.5, 1.5, 2.5, 0], [-127, 63.5, -0.5, -1.5, -2.5, 3.5]], np.float32)
    m = q.q8_quantize_matrix(ctx, W)
    assert np_(m.data)[:, :6].tolist() == [[127, -64, 0, 2, 2, 0], [-127, 64, 0, -2, -2, 4]]


GEMV_SHAPES = [(768, 256), (3072, 512), (3072, 1024), (1024, 2048), (1000, 620), (5, 16), (37, 3000),
               (100, 8200), (131, 48), (50000, 512)]


@pytest.mark.parametrize("rows,cols", GEMV_SHAPES)
@pytest.mark.parametrize("use_bias", [False, True])
def test_gemv(q, ctx, oracle, rows, cols, use_bias):
    rng = np.random.default_rng(rows + cols)
    W = _w(rng, rows, cols)
    b = (rng.standard_normal(rows) * 0.01).astype(np.float32) if use_bias else None
    x = rng.standard_normal(cols).astype(np.float32)
    L = oracle.QLinear(W, b)
    M = q.q8_quantize_matrix(ctx, W)
    y, taps = q.q8_gemv(ctx, M, ctx.f32(x), ctx.f32(b), taps=True)
    y_ref, xq, xs, acc = L.gemv(x, taps=True)
    assert_same(taps["xq"][0], xq, "xq")
    assert float(taps["xscale"][0]) == float(xs)
    assert_same(taps["acc"][0], acc, "acc")
    assert_same(y, y_ref, "y (one multiply and one add per element: identical bits expected)")
    # taps off gives the same result
    assert_same(q.q8_gemv(ctx, M, ctx.f32(x), ctx.f32(b)), y_ref, "y, no taps")


def test_gemv_degenerate_inputs(q, ctx, oracle):
    rng = np.random.default_rng(0)
    W = _w(rng, 64, 128)
    L, M = oracle.QLinear(W), q.q8_quantize_matrix(ctx, W)
    for x in (np.zeros(128, np.float32), np.full(128, 1e-35, np.float32),
              np.eye(128, dtype=np.float32)[5] * -3, np.full(128, 7.0, np.float32)):
        y, taps = q.q8_gemv(ctx, M, ctx.f32(x), taps=True)
        y_ref, xq, xs, acc = L.gemv(x, taps=True)
        assert_same(taps["xq"][0], xq); assert float(taps["xscale"][0]) == float(xs)
        assert_same(taps["acc"][0], acc); assert_same(y, y_ref)
    # extreme accumulators: all +127 against all -127 over 2048 columns
    Wq = torch.full((16, 2048), 127, dtype=torch.int8, device=ctx.device)
    M2 = q.Mat(Wq, 2048, 1.0)
    y, taps = q.q8_gemv(ctx, M2, ctx.f32(np.full(2048, -1.0, np.float32)), taps=True)
    assert (np_(taps["acc"]) == -33032192).all()


@pytest.mark.parametrize("rows,cols", [(3072, 512), (1024, 2048), (1000, 620), (50, 16), (50000, 512)])
@pytest.mark.parametrize("n", [2, 5, 8])
def test_gemm_narrow_streaming(q, ctx, oracle, rows, cols, n):
    rng = np.random.default_rng(rows + cols + n)
    W = _w(rng, rows, cols)
    b = (rng.standard_normal(rows) * 0.01).astype(np.float32)
    X = rng.standard_normal((n, cols)).astype(np.float32) * rng.uniform(0.1, 10, (n, 1)).astype(np.float32)
    if n > 2:
        X[1] = 0
    L, M = oracle.QLinear(W, b), q.q8_quantize_matrix(ctx, W)
    Y, taps = q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(b), taps=True)
    Y_ref, xq, xs, acc = L.gemm_narrow(X, taps=True)
    assert_same(taps["xq"], xq, "xq"); assert_same(taps["xscale"], xs, "xscale")
    assert_same(taps["acc"], acc, "acc"); assert_same(Y, Y_ref, "Y")
    # column identity: the narrow product is n matrix-vector products
    y0 = q.q8_gemv(ctx, M, ctx.f32(X[0]), ctx.f32(b))
    assert_same(y0, np_(Y)[0], "column 0 vs gemv")


@pytest.mark.parametrize("rows,cols", [(50000, 512), (9001, 1024), (8300, 1012), (40003, 252), (17000, 500)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 8])
def test_gemm_narrow_one_pass_over_a_large_matrix(q, ctx, oracle, rows, cols, n):
    """One product without taps over a matrix of more than 8 MB with rows of 256, 512 or 1024 bytes runs on the
    kernel without a loop (8 KB of consecutive rows per wave, totals over 16, 32 or 64 lanes per row): identical
    to the oracle and to the looping kernel (which the taps select)."""
    rng = np.random.default_rng(rows + cols + n)
    W = _w(rng, rows, cols)
    b = (rng.standard_normal(rows) * 0.01).astype(np.float32)
    X = rng.standard_normal((n, cols)).astype(np.float32) * rng.uniform(0.1, 10, (n, 1)).astype(np.float32)
    L, M = oracle.QLinear(W, b), q.q8_quantize_matrix(ctx, W)
    assert M.data.shape[0] * M.data.shape[1] >= 8 << 20 and M.data.shape[1] in (256, 512, 1024)
    Y_ref = L.gemm_narrow(X)
    assert_same(q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(b)), Y_ref, "Y, with bias")
    Y_taps, _ = q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(b), taps=True)
    assert_same(Y_taps, Y_ref, "Y from the looping kernel")
    assert_same(q.q8_gemm_narrow(ctx, M, ctx.f32(X)), oracle.QLinear(W).gemm_narrow(X), "Y, no bias")
    if n in (1, 5, 8):
        # the variant with one weight scale per row takes the same kernel
        R, rs = q.q8_quantize_matrix_rows(ctx, W)
        assert_same(q.q8_gemm_narrow_rows(ctx, R, rs, ctx.f32(X), ctx.f32(b)), oracle.QLinearRows(W, b).gemm_narrow(X), "Y, row scales")


@pytest.mark.parametrize("rows,cols,n", [(3072, 512, 50), (1024, 2048, 30), (1000, 620, 13), (100, 48, 9),
                                         (3072, 512, 60), (77, 1000, 70), (3072, 1024, 320), (130, 272, 129),
                                         (9000, 512, 130), (50000, 512, 40), (8200, 144, 257)])
def test_gemm_narrow_matrix_cores(q, ctx, oracle, rows, cols, n):
    rng = np.random.default_rng(rows + cols + n)
    W = _w(rng, rows, cols)
    b = (rng.standard_normal(rows) * 0.01).astype(np.float32)
    X = rng.standard_normal((n, cols)).astype(np.float32) * rng.uniform(0.1, 10, (n, 1)).astype(np.float32)
    X[3] = 0
    L, M = oracle.QLinear(W, b), q.q8_quantize_matrix(ctx, W)
    Y, taps = q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(b), taps=True)
    Y_ref, xq, xs, acc = L.gemm_narrow(X, taps=True)
    assert_same(taps["xq"], xq, "xq"); assert_same(taps["xscale"], xs, "xscale")
    assert_same(taps["acc"], acc, "acc"); assert_same(Y, Y_ref, "Y")
    assert_same(q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(b)), Y_ref, "Y, no taps")
    assert_same(q.q8_gemm_narrow(ctx, M, ctx.f32(X)), oracle.QLinear(W, None).gemm_narrow(X), "Y, no taps, no bias")


def test_argument_errors_are_reported_not_launched(q, ctx):
    W = q.q8_quantize_matrix(ctx, np.ones((4, 16), np.float32))
    x = ctx.f32(np.ones(20, np.float32))
    with pytest.raises(q.Q8Error) as e:
        q.q8_gemv(ctx, W, x[1:17])            # misaligned vector
    assert e.value.code == 3
    bad = q.Mat(W.data, 16, 1.0); bad.c.ld = 8
    with pytest.raises(q.Q8Error) as e:
        q.q8_gemv(ctx, bad, x[:16])
    assert e.value.code == 2
    with pytest.raises(q.Q8Error) as e:
        q.q8_gemm_narrow(ctx, W, ctx.f32(np.ones((2000, 16), np.float32)))
    assert e.value.code == 2


# ---- the variant with one weight scale per row -------------------------------------------

def _rows_case(rng, rows, cols):
    # rows of very different size, one zero row, one tiny row: per-row scales differ by orders of magnitude
    W = _w(rng, rows, cols) * np.logspace(-3, 0, rows, dtype=np.float32)[:, None]
    W[rows // 2] = 0.0
    if rows > 4:
        W[3] = 1e-36
    return W


@pytest.mark.parametrize("rows,cols", [(768, 256), (3072, 1024), (33, 620), (7, 5), (2500, 1000), (50000, 512)])
def test_quantize_matrix_rows_bit_exact(q, ctx, oracle, rows, cols):
    rng = np.random.default_rng(rows * 3 + cols)
    W = _rows_case(rng, rows, cols)
    M, rs = q.q8_quantize_matrix_rows(ctx, W)
    R = oracle.QLinearRows(W)
    assert_same(rs, R.row_scale, "row scales")
    assert_same(M.data, R.Wq, "Wq")


@pytest.mark.parametrize("rows,cols", [(3072, 512), (1024, 2048), (1000, 620), (50, 16), (37, 3001), (50000, 512)])
@pytest.mark.parametrize("n", [1, 5, 8])
def test_gemm_narrow_rows_streaming(q, ctx, oracle, rows, cols, n):
    if cols % 4 and n > 1:
        pytest.skip("several vectors need a leading dimension that is a multiple of 4")
    rng = np.random.default_rng(rows + cols + n + 1)
    W = _rows_case(rng, rows, cols)
    b = (rng.standard_normal(rows) * 0.01).astype(np.float32)
    X = rng.standard_normal((n, cols)).astype(np.float32) * rng.uniform(0.1, 10, (n, 1)).astype(np.float32)
    R = oracle.QLinearRows(W, b)
    M, rs = q.q8_quantize_matrix_rows(ctx, W)
    Y, taps = q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X), ctx.f32(b), taps=True)
    Y_ref, xq, xs, acc = R.gemm_narrow(X, taps=True)
    assert_same(taps["xq"], xq, "xq"); assert_same(taps["xscale"], xs, "xscale")
    assert_same(taps["acc"], acc, "acc"); assert_same(Y, Y_ref, "Y")
    assert_same(q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X)), oracle.QLinearRows(W).gemm_narrow(X), "Y, no taps, no bias")


@pytest.mark.parametrize("rows,cols,n", [(3072, 512, 50), (1024, 2048, 30), (1000, 620, 13), (3072, 1024, 320),
                                         (130, 272, 129), (9000, 512, 130)])
def test_gemm_narrow_rows_matrix_cores(q, ctx, oracle, rows, cols, n):
    rng = np.random.default_rng(rows + cols + n + 2)
    W = _rows_case(rng, rows, cols)
    b = (rng.standard_normal(rows) * 0.01).astype(np.float32)
    X = rng.standard_normal((n, cols)).astype(np.float32) * rng.uniform(0.1, 10, (n, 1)).astype(np.float32)
    X[3] = 0
    R = oracle.QLinearRows(W, b)
    M, rs = q.q8_quantize_matrix_rows(ctx, W)
    Y, taps = q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X), ctx.f32(b), taps=True)
    Y_ref, xq, xs, acc = R.gemm_narrow(X, taps=True)
    assert_same(taps["acc"], acc, "acc"); assert_same(Y, Y_ref, "Y")
    assert_same(q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X), ctx.f32(b)), Y_ref, "Y, no taps")
    assert_same(q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X)), oracle.QLinearRows(W).gemm_narrow(X), "Y, no taps, no bias")


def test_rows_variant_argument_errors(q, ctx):
    M, rs = q.q8_quantize_matrix_rows(ctx, np.ones((4, 16), np.float32))
    with pytest.raises(q.Q8Error) as e:
        q.q8_gemm_narrow_rows(ctx, M, None, ctx.f32(np.ones((1, 16), np.float32)))
    assert e.value.code == 1


# rows, columns, vectors, tile-packed, the kernel that the product takes with results at a pitch of `rows` floats (checked against the
# library's rule on the host)
LARGE_PANELS = [
    # 128 x 128 tiles: rows and vectors at the remainders of a tile, k steps and stages at theirs, row by row and packed; rows of 513-1024
    # bytes on both sides of 800 and 700 blocks and of 192 vectors
    (2945, 1040, 769, False, "tiles of 128"), (33000, 1100, 64, False, "tiles of 128"), (3000, 1088, 895, True, "tiles of 128"),
    (2433, 2112, 897, True, "tiles of 128"), (12804, 576, 512, False, "tiles of 128"), (13068, 1024, 500, True, "tiles of 128"),
    (12800, 576, 512, True, "once 128 x 64"), (22272, 576, 256, True, "once 128 x 64"), (22404, 576, 256, False, "tiles of 128"),
    (30000, 576, 160, True, "once 128 x 64"), (30000, 576, 193, True, "tiles of 128"),
    # 64 x 64 tiles, and the line to the streamed form
    (130, 2112, 33, True, "tiles of 64"), (33001, 1088, 64, True, "tiles of 64"), (65, 2112, 65, True, "tiles of 64"),
    (1472, 1088, 960, True, "tiles of 64"), (1400, 1088, 960, True, "stream"),
    # staged, and the line to the streamed form
    (17, 2500, 9, False, "staged"), (65, 2064, 65, False, "staged"), (1000, 2064, 513, False, "staged"), (130, 4096, 33, False, "staged"),
    (1400, 1040, 960, False, "staged"), (1300, 1040, 960, False, "stream"),
    # rows of at most 512 bytes
    (2049, 16, 1024, False, "resident"), (1537, 512, 1023, True, "resident"), (33, 500, 9, False, "resident"), (64, 512, 64, True, "resident"),
    # rows of 513-1024 bytes, 128 rows x 32 and x 64 vectors at once, and the line between them
    (4096, 576, 256, False, "once 128 x 32"), (4100, 576, 256, True, "once 128 x 64"), (2324, 576, 1023, False, "once 128 x 64"),
    (3072, 576, 897, True, "once 128 x 64"), (3000, 1000, 900, False, "once 128 x 64"), (1553, 1024, 1024, False, "once 128 x 64 trade"),
    (1537, 528, 1023, False, "once 128 x 64"), (33658, 640, 65, True, "once 128 x 64"), (33000, 640, 64, False, "once 128 x 64 trade"),
    # rows of 1025-2048 bytes, 64 x 64 at once and streamed, and the lines between them
    (641, 1104, 960, False, "once 64 x 64"), (640, 1104, 960, False, "stream"), (1024, 1088, 1024, True, "once 64 x 64"),
    (1025, 2048, 1024, True, "stream"), (2415, 1860, 903, False, "stream"), (64, 1088, 64, True, "stream"), (1024, 2048, 513, True, "stream"),
    (65, 1088, 65, True, "stream"), (127, 1152, 9, True, "stream"), (8200, 1088, 33, True, "stream"), (17, 1100, 9, False, "stream"),
    (65, 1040, 65, False, "stream"), (1000, 2000, 513, False, "stream"), (8201, 1088, 33, False, "stream"),
    # row by row in rows of whole 128 bytes: K-resident, at the edges of its blocks and on both sides of one round of them, and 128 x 64 with the trade
    (1, 640, 9, False, "resident 1024"), (65, 896, 65, False, "resident 1024"), (127, 1024, 64, False, "resident 1024"),
    (300, 640, 1024, False, "resident 1024"), (8192, 640, 128, False, "resident 1024"), (20000, 640, 20, False, "once 128 x 32"),
    (2324, 640, 1023, False, "once 128 x 64 trade"), (3073, 768, 353, False, "once 128 x 64 trade"), (8200, 1024, 260, False, "once 128 x 64 trade"),
    (20001, 896, 100, False, "once 128 x 64 trade"),
]


@pytest.mark.parametrize("rows,cols,n,tiled,route", LARGE_PANELS)
@pytest.mark.parametrize("by_row", [False, True])
def test_large_panels(q, oracle, rows, cols, n, tiled, route, by_row):
    """Every kernel of the plain panel products at the edges of its tiles, stages and k steps and on both sides of the rule's
    lines, packed and row by row, one scale and one per row, results at an odd pitch: exact integer sums, one product of
    scales, one addition, so identical bits."""
    rng = np.random.default_rng(rows + n)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=rows, max_ld=4096))
    W, b, X = _w(rng, rows, cols), (rng.standard_normal(rows) * 0.01).astype(np.float32), rng.standard_normal((n, cols)).astype(np.float32)
    M, rs = q.q8_quantize_matrix_rows(ctx, W) if by_row else (q.q8_quantize_matrix(ctx, W), None)
    if tiled:
        M = q.q8_pack_tiles(ctx, M)
    pick = sorted({0, 1, 127, 128, n // 2, n - 2, n - 1} & set(range(n)))
    codes = np_(M.data)[:, :cols].astype(np.int64)
    for pitch, bias in ((rows, None), (rows + 3, b)):
        Y = ctx.empty(n, pitch)[:, :rows]
        if by_row: q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X), ctx.f32(bias), Y=Y)
        else: q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(bias), Y=Y)
        got = np_(Y)
        for j in pick:
            xq, xs = oracle.quantize(X[j])
            acc = (codes @ xq[:cols].astype(np.int64)).astype(np.float32)
            scale = (np_(rs) if by_row else np.float32(M.scale)) * np.float32(xs)
            y = acc * scale
            assert_same(got[j], y if bias is None else y + bias, "vector %d" % j)


WHOLE_PANELS = [
    # rows of 513-1024 bytes: 128 rows x 32 and x 64 vectors, at the remainders of both, of the k parts and of a matrix-core step
    (1, 516, 9, False, "once 128 x 32"), (129, 1024, 31, True, "once 128 x 32"), (127, 1000, 33, False, "once 128 x 32"),
    (128, 576, 64, True, "once 128 x 32"), (3072, 1024, 320, True, "once 128 x 32"), (3073, 720, 353, False, "once 128 x 64"),
    (4096, 1024, 1000, True, "once 128 x 64"), (300, 528, 1024, False, "once 128 x 32"), (33000, 1024, 50, True, "once 128 x 64"),
    # rows of 1025-2048 bytes: 64 rows x 64 vectors at once
    (1024, 2048, 1024, True, "once 64 x 64"), (1000, 1100, 1009, False, "once 64 x 64"), (2999, 2000, 300, False, "once 64 x 64"),
    (2880, 1600, 255, True, "once 64 x 64"),
    # the same streamed: one share of the vectors and several, a last group of one vector, an odd number of groups
    (1, 1028, 9, False, "stream"), (65, 2048, 33, True, "stream"), (64, 1536, 64, True, "stream"), (3071, 2000, 61, False, "stream"),
    (1500, 2048, 700, True, "stream"), (8200, 2048, 97, True, "stream"), (2000, 1500, 641, False, "stream"),
]


@pytest.mark.parametrize("rows,cols,n,tiled,route", WHOLE_PANELS)
@pytest.mark.parametrize("by_row", [False, True])
def test_panels_requested_whole(q, oracle, rows, cols, n, tiled, route, by_row):
    """The products whose blocks request all they need at once, and the ones that keep their weights for a stream of vectors,
    at the edges of their tiles, parts and groups, with one scale and one per row, results at an odd pitch: the same integer
    sums, product of scales and addition as everywhere, so the same bits."""
    rng = np.random.default_rng(rows + n + cols)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=rows, max_ld=2112))
    W, b, X = _w(rng, rows, cols), (rng.standard_normal(rows) * 0.01).astype(np.float32), rng.standard_normal((n, cols)).astype(np.float32)
    M, rs = q.q8_quantize_matrix_rows(ctx, W) if by_row else (q.q8_quantize_matrix(ctx, W), None)
    if tiled:
        M = q.q8_pack_tiles(ctx, M)
    codes = np_(M.data)[:, :cols].astype(np.int64)
    for pitch, bias in ((rows, b), (rows + 3, None)):
        Y = ctx.empty(n, pitch)
        Y.fill_(7.0)
        if by_row: q.q8_gemm_narrow_rows(ctx, M, rs, ctx.f32(X), ctx.f32(bias), Y=Y[:, :rows])
        else: q.q8_gemm_narrow(ctx, M, ctx.f32(X), ctx.f32(bias), Y=Y[:, :rows])
        got = np_(Y)
        assert (got[:, rows:] == 7.0).all()
        for j in sorted({0, 1, 31, 32, 63, 64, n // 2, n - 2, n - 1} & set(range(n))):
            xq, xs = oracle.quantize(X[j])
            acc = (codes @ xq[:cols].astype(np.int64)).astype(np.float32)
            y = acc * ((np_(rs) if by_row else np.float32(M.scale)) * np.float32(xs))
            assert_same(got[j, :rows], y if bias is None else y + bias, "vector %d" % j)


# rows, columns, vectors, tile-packed, tiles of 16 rows per block (checked against the library's rule on the host): rows and vectors at the
# remainders of a block, parts of the k range of no, one and several matrix-core steps
QUANT_PANELS = [
    (1, 16, 9, False, 1), (4, 4, 10, False, 1), (257, 320, 16, True, 1), (1024, 516, 30, False, 1), (640, 1024, 17, True, 1), (1000, 2048, 64, True, 1),
    (1031, 512, 100, True, 2), (3072, 1000, 31, False, 2), (2000, 1100, 40, False, 2),
    (3072, 512, 200, True, 4), (65, 256, 1024, False, 2), (1000, 620, 333, False, 4), (1030, 2048, 240, True, 4), (8200, 1536, 16, True, 4),
]


@pytest.mark.parametrize("rows,cols,n,tiled,tiles", QUANT_PANELS)
@pytest.mark.parametrize("by_row", [False, True])
def test_panels_whose_blocks_quantize(q, oracle, rows, cols, n, tiled, tiles, by_row):
    """Few vectors are quantized by the blocks that multiply them, with one scale and one per row, results at an odd pitch: the
    same codes, integer sums and roundings as everywhere, so the same bits; also for vectors of zeros, of next to nothing and with an infinity."""
    rng = np.random.default_rng(rows + n + cols)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=rows, max_ld=2112))
    W, b, X = _w(rng, rows, cols), (rng.standard_normal(rows) * 0.01).astype(np.float32), rng.standard_normal((n, cols)).astype(np.float32)
    X[1], X[3] = 0.0, np.float32(2.0 ** -101)
    M, rs = q.q8_quantize_matrix_rows(ctx, W) if by_row else (q.q8_quantize_matrix(ctx, W), None)
    if tiled:
        M = q.q8_pack_tiles(ctx, M)
    codes = np_(M.data)[:, :cols].astype(np.int64)
    call = lambda Xd, bias, Y: q.q8_gemm_narrow_rows(ctx, M, rs, Xd, bias, Y=Y) if by_row else q.q8_gemm_narrow(ctx, M, Xd, bias, Y=Y)
    for pitch, bias in ((rows, b), (rows + 3, None)):
        Y = ctx.empty(n, pitch)
        Y.fill_(7.0)
        call(ctx.f32(X), ctx.f32(bias), Y[:, :rows])
        got = np_(Y)
        assert (got[:, rows:] == 7.0).all()
        for j in sorted({0, 1, 3, 15, 16, n // 2, n - 2, n - 1} & set(range(n))):
            xq, xs = oracle.quantize(X[j])
            acc = (codes @ xq[:cols].astype(np.int64)).astype(np.float32)
            y = acc * ((np_(rs) if by_row else np.float32(M.scale)) * np.float32(xs))
            assert_same(got[j, :rows], y if bias is None else y + bias, "vector %d" % j)
    X[2, cols // 2] = np.inf
    one, two = ctx.empty(n, rows), _beside(ctx, X, rows)
    call(ctx.f32(X), None, one)
    call(two[1], None, two[0])
    np.testing.assert_array_equal(np_(one), np_(two[0].contiguous()))
    assert np.isfinite(np_(one)[np.arange(n) != 2]).all()


def _beside(ctx, X, rows):
    """Results and vectors side by side in one buffer: vectors that lie among their results are quantized in a launch of their own."""
    at = (rows + 3) // 4 * 4
    buf = ctx.empty(X.shape[0], at + (X.shape[1] + 3) // 4 * 4)
    buf[:, at:at + X.shape[1]] = ctx.f32(X)
    return buf[:, :rows], buf[:, at:at + X.shape[1]]


# few results from codes that are there: the k range in eight parts (tiles of 16 rows per block, checked against the rule on the host)
PART_PANELS = [(1, 516, 9, False, 1), (129, 1024, 31, True, 1), (65, 2048, 33, True, 1), (1000, 1008, 100, False, 2), (1024, 2048, 70, True, 2),
               (3071, 2000, 61, False, 4), (1030, 1024, 240, True, 4)]


@pytest.mark.parametrize("rows,cols,n,tiled,route", [s for s in LARGE_PANELS + WHOLE_PANELS if s[0] * s[2] <= 1 << 20] + PART_PANELS)
def test_panels_of_vectors_that_lie_among_their_results(q, rows, cols, n, tiled, route):
    """Quantization and product in two launches, at the sizes that one launch takes otherwise: the kernels that the products of already
    quantized vectors use.  The same bits."""
    rng = np.random.default_rng(rows + n + cols)
    ctx = q.Context(workspace_bytes=q.q8_workspace_bytes(max_n=n, max_l=8, max_rows=rows, max_ld=4112))
    M = q.q8_quantize_matrix(ctx, _w(rng, rows, cols))
    if tiled:
        M = q.q8_pack_tiles(ctx, M)
    X, b = rng.standard_normal((n, cols)).astype(np.float32), ctx.f32((rng.standard_normal(rows) * 0.01).astype(np.float32))
    Y, Xd = _beside(ctx, X, rows)
    q.q8_gemm_narrow(ctx, M, Xd, b, Y=Y)
    assert_same(q.q8_gemm_narrow(ctx, M, ctx.f32(X), b), np_(Y.contiguous()), "results")
