"""q4nx_gemm_ex through the C ABI: the matrix product with a caller workspace,
where the launch plan splits K for shapes with few output tiles.

  * SPLIT_SHAPES take a plan that splits K into two, three or four segments
    (checked against the planner), with ragged M and N, K not a multiple of 64,
    float32 and bf16 outputs;
  * parity with the float64 oracle: the projection tolerance and the tight
    bound against the product of the bf16 weights;
  * the three weight formats give the same bits for the same bf16 weights
    (same plan, same partial products, same order of the final sum);
  * the workspace starts filled with NaN, so a partial that is read before it
    is written would show; repeated calls are bitwise identical;
  * without a workspace the result equals q4nx_gemm bit for bit;
  * Q4NX products with a large M dequantize W to bf16 in the workspace first
    (each weight once) and give the fused kernel's bits.
"""
import numpy as np
import pytest

import oracle
from gemm_launches import FORMATS, launches
from workloads import gen_weights, gen_mx_weights, gen_activations

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q4():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2602_06063_amd as mod
    return mod


def _say(*a):
    print("[case]", *a, flush=True)


def dev_u8(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def dev_bf16(bits):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).cuda().view(torch.bfloat16)


def host_f32(t):
    torch.cuda.synchronize()
    return t.float().cpu().numpy() if t.dtype == torch.bfloat16 else t.cpu().numpy()


def work_for(q4, M, N, K, fmt=None):
    """A NaN-filled workspace big enough for every weight format."""
    fmts = [fmt] if fmt is not None else [q4.Q4NX_WEIGHTS_Q4NX, q4.Q4NX_WEIGHTS_MXFP4, q4.Q4NX_WEIGHTS_BF16]
    nbytes = max(q4.q4nx_gemm_workspace_size(f, M, N, K) for f in fmts)
    assert nbytes > 0, "this shape is meant to use a workspace"
    return torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda")


def work_if_any(q4, M, N, K, fmt):
    """The workspace the planner asks for (NaN-filled), or None when its plan
    takes none."""
    nbytes = q4.q4nx_gemm_workspace_size(fmt, M, N, K)
    return torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda") if nbytes else None


# (M, N, K, rows checked by the oracle: None = all).  The last six: ragged
# tiles at the edges of a split, and outputs that the sum of the segments takes
# one by one (N not a multiple of 4).
SPLIT_SHAPES = [(2048, 2560, 10240, 64), (2048, 2560, 10208, 64), (4096, 5376, 21504, 48), (700, 3333, 6912, 48),
                (394, 5145, 5472, 48), (1540, 2447, 4928, 48), (1291, 2987, 4832, 48), (827, 5455, 7296, 48),
                (859, 5399, 7264, 48)]
# A long K that one launch takes, with the workspace at hand.
LONG_K_SHAPES = [(512, 512, 16384, None), (512, 512, 16352, None), (300, 520, 20000, None), (260, 257, 12000, None),
                 (1, 256, 20480, None)]


def _rows(M, n):
    if n is None:
        return None
    rng = np.random.default_rng(M)
    return np.unique(np.concatenate([np.arange(8), M - 8 + np.arange(8), rng.integers(0, M, n)]))


@pytest.mark.parametrize("M,N,K,nrows", SPLIT_SHAPES + LONG_K_SHAPES)
@pytest.mark.parametrize("bf16_out", [False, True])
def test_gemm_ex_split_parity(q4, M, N, K, nrows, bf16_out):
    assert ("split" in launches(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, work=True)) == ((M, N, K, nrows) in SPLIT_SHAPES)
    _say("gemm_ex split", M, N, K, "bf16" if bf16_out else "f32")
    codes, s, o = gen_weights(N, K, seed=M + K)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    X = gen_activations((M, K), seed=N + K)
    Y = torch.empty((M, N), dtype=torch.bfloat16 if bf16_out else torch.float32, device="cuda")
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, dev_bf16(X), blob, Y, work=work_for(q4, M, N, K))
    Yh = host_f32(Y)
    rows = _rows(M, nrows)
    if rows is not None:
        X, Yh = X[rows], Yh[rows]
    w32 = oracle.dequant_f32(codes, s, o)
    ok, worst = oracle.check_close(Yh, oracle.gemm_f64(X, w32), oracle.abs_bound(X, w32), bf16_out=bf16_out)
    assert ok, worst
    w16 = oracle.bf16_to_f32(oracle.f32_to_bf16(w32))
    ref16 = oracle.gemm_f64(X, w16)
    tight = np.abs(Yh.astype(np.float64) - ref16) <= (
        1e-5 * oracle.abs_bound(X, w16) + 1e-6 + (2.0 ** -8 * np.abs(ref16) if bf16_out else 0))
    assert tight.all()


@pytest.mark.parametrize("M,N,K,split", [(300, 520, 20000, False), (260, 257, 12000, False), (2048, 2560, 10208, True),
                                         (700, 3333, 6912, True), (394, 5145, 5472, True)])
def test_gemm_ex_formats_agree_bitwise(q4, M, N, K, split):
    """Q4NX and MXFP4-variant blobs against the bf16 weights they dequantize
    to, through split plans or with the workspace unused: identical bits."""
    for f in FORMATS:
        assert ("split" in launches(f, M, N, K, work=True)) == split
    _say("gemm_ex formats", M, N, K)
    X = dev_bf16(gen_activations((M, K), seed=M))
    work = work_for(q4, M, N, K)
    W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    Y1 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    Y2 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    codes, s, o = gen_weights(N, K, seed=K)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Y1, work=work)
    q4.q4nx_dequant(blob, N, K, W)
    work.fill_(float("nan"))
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_BF16, M, N, K, X, W, Y2, work=work)
    torch.cuda.synchronize()
    assert torch.equal(Y1.view(torch.int32), Y2.view(torch.int32))
    mcodes, msc = gen_mx_weights(N, K, seed=K, mode="edge")
    mblob = dev_u8(q4.q4nx_mx_pack(mcodes, msc))
    work.fill_(float("nan"))
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_MXFP4, M, N, K, X, mblob, Y1, work=work)
    q4.q4nx_mx_dequant(mblob, N, K, W)
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_BF16, M, N, K, X, W, Y2, work=work)
    torch.cuda.synchronize()
    assert torch.equal(Y1.view(torch.int32), Y2.view(torch.int32))
    w32 = oracle.mx_dequant_f32(mcodes, msc)
    Xh = gen_activations((M, K), seed=M)
    ok, worst = oracle.check_close(host_f32(Y1), oracle.gemm_f64(Xh, w32), oracle.abs_bound(Xh, w32))
    assert ok, worst


def test_gemm_ex_repeatable_and_unsplit_without_workspace(q4):
    M, N, K = 700, 3333, 6944
    assert "split" in launches(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, work=True)
    assert "split" not in launches(q4.Q4NX_WEIGHTS_Q4NX, M, N, K)
    _say("gemm_ex repeat / no workspace", M, N, K)
    codes, s, o = gen_weights(N, K, seed=9)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    X = dev_bf16(gen_activations((M, K), seed=9))
    work = work_for(q4, M, N, K)
    Ys = [torch.empty((M, N), dtype=torch.float32, device="cuda") for _ in range(4)]
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Ys[0], work=work)
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Ys[1], work=work)
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Ys[2])      # no workspace: nothing split
    q4.q4nx_gemm(M, N, K, X, blob, Ys[3])
    torch.cuda.synchronize()
    assert torch.equal(Ys[0].view(torch.int32), Ys[1].view(torch.int32))
    assert torch.equal(Ys[2].view(torch.int32), Ys[3].view(torch.int32))
    # split and unsplit differ only by the order of the float32 sums
    d = (Ys[0] - Ys[3]).abs().max().item()
    assert d <= 1e-4 * Ys[3].abs().max().item()


@pytest.mark.parametrize("M,N,K,split", [(4096, 1024, 4096, False), (4096, 5376, 21504, True),
                                         (2048, 20480, 2560, False)])
def test_gemm_ex_dequantize_then_multiply(q4, M, N, K, split):
    """Shapes whose Q4NX workspace holds bf16 W (M = 4096, and the 4B gate/up
    product at M = 2048): the result equals the fused product of the same plan
    bit for bit (q4nx_gemm when nothing is split,
    the bf16-weight product of the dequantized W when K is split), and meets
    the oracle on sampled rows."""
    _say("gemm_ex two-phase", M, N, K)
    nbytes = q4.q4nx_gemm_workspace_size(q4.Q4NX_WEIGHTS_Q4NX, M, N, K)
    assert nbytes >= N * K * 2
    codes, s, o = gen_weights(N, K, seed=N)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    Xh = gen_activations((M, K), seed=K)
    X = dev_bf16(Xh)
    work = torch.full((nbytes // 4,), float("nan"), dtype=torch.float32, device="cuda")
    Y1 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    Y2 = torch.empty((M, N), dtype=torch.float32, device="cuda")
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Y1, work=work)
    if split:
        W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
        q4.q4nx_dequant(blob, N, K, W)
        q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_BF16, M, N, K, X, W, Y2, work=work_for(q4, M, N, K, q4.Q4NX_WEIGHTS_BF16))
    else:
        q4.q4nx_gemm(M, N, K, X, blob, Y2)
    torch.cuda.synchronize()
    assert torch.equal(Y1.view(torch.int32), Y2.view(torch.int32))
    rows = _rows(M, 24)
    w32 = oracle.dequant_f32(codes, s, o)
    ok, worst = oracle.check_close(host_f32(Y1)[rows], oracle.gemm_f64(Xh[rows], w32), oracle.abs_bound(Xh[rows], w32))
    assert ok, worst


# Shapes whose tiles do not fill whole rounds of the 256 CUs: a round and a few
# tiles (4352 x 4096), two rounds and a part (4352 x 8448), the Gemma3-4B o
# shape (80 tiles), few tiles over a long K with M and N ragged (2000 x 1100 x
# 6912: the few-rows kernel), a K tail with a ragged M (1999 x 2500 x 2016), and
# M and N ragged with N a multiple of 32 or not (2040 x 4000 and 3999).  The
# first two dequantize once.
PLANNED_SHAPES = [(4352, 4096, 2560, 32), (4352, 8448, 2560, 32), (2048, 2560, 2048, 48), (2000, 1100, 6912, 48),
                  (1999, 2500, 2016, 48), (2040, 4000, 2560, 48), (2040, 3999, 2560, 48)]


@pytest.mark.parametrize("M,N,K,nrows", PLANNED_SHAPES)
@pytest.mark.parametrize("bf16_out", [False, True])
def test_gemm_ex_planned_parity(q4, M, N, K, nrows, bf16_out):
    """The planned launches against the oracle on sampled rows, against the
    bf16-weight product within the tight bound, and against the launch without
    a workspace (no split) within the order of float32 sums."""
    _say("gemm_ex planned", M, N, K, "bf16" if bf16_out else "f32")
    codes, s, o = gen_weights(N, K, seed=M + 3 * K)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    Xh = gen_activations((M, K), seed=N + 5)
    X = dev_bf16(Xh)
    odt = torch.bfloat16 if bf16_out else torch.float32
    Y = torch.empty((M, N), dtype=odt, device="cuda")
    Y0 = torch.empty((M, N), dtype=odt, device="cuda")
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Y, work=work_if_any(q4, M, N, K, q4.Q4NX_WEIGHTS_Q4NX))
    q4.q4nx_gemm(M, N, K, X, blob, Y0)
    Yh, Y0h = host_f32(Y), host_f32(Y0)
    assert np.isfinite(Yh).all()
    rows = _rows(M, nrows)
    w32 = oracle.dequant_f32(codes, s, o)
    ok, worst = oracle.check_close(Yh[rows], oracle.gemm_f64(Xh[rows], w32), oracle.abs_bound(Xh[rows], w32),
                                   bf16_out=bf16_out)
    assert ok, worst
    w16 = oracle.bf16_to_f32(oracle.f32_to_bf16(w32))
    ref16 = oracle.gemm_f64(Xh[rows], w16)
    tight = np.abs(Yh[rows].astype(np.float64) - ref16) <= (
        1e-5 * oracle.abs_bound(Xh[rows], w16) + 1e-6 + (2.0 ** -8 * np.abs(ref16) if bf16_out else 0))
    assert tight.all()
    # Every element, split or not, against the unsplit launch: the same
    # products summed in another order (float32), or equal after bf16 rounding.
    scale = np.abs(Y0h).max()
    assert np.abs(Yh - Y0h).max() <= (1e-4 if not bf16_out else 2.0 ** -7) * scale


@pytest.mark.parametrize("M,N,K", [(2048, 4096, 2560), (2048, 2560, 2048), (2048, 20480, 2560), (2048, 2560, 10240)])
def test_gemm_ex_gemma3_4b_products(q4, M, N, K):
    """The four stacked Gemma3-4B prefill products at M = 2048 (q/k/v, o,
    gate/up, down) through the plans the benchmark runs, against the oracle on
    sampled rows."""
    _say("gemm_ex 4B", M, N, K)
    codes, s, o = gen_weights(N, K, seed=N + K)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    Xh = gen_activations((M, K), seed=K + 1)
    Y = torch.empty((M, N), dtype=torch.float32, device="cuda")
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, dev_bf16(Xh), blob, Y,
                    work=work_if_any(q4, M, N, K, q4.Q4NX_WEIGHTS_Q4NX))
    rows = _rows(M, 24)
    w32 = oracle.dequant_f32(codes, s, o)
    ok, worst = oracle.check_close(host_f32(Y)[rows], oracle.gemm_f64(Xh[rows], w32), oracle.abs_bound(Xh[rows], w32))
    assert ok, worst


def test_gemm_ex_split_repeats_with_workspace_cleared(q4):
    """Ten calls of a split-K plan in a row, the workspace refilled with NaN
    before each: a partial read before its writer finished, or one left over
    from the previous call, would show as a NaN or a changed bit."""
    M, N, K = 700, 3333, 6912
    assert "split" in launches(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, work=True)
    _say("gemm_ex split repeats", M, N, K)
    codes, s, o = gen_weights(N, K, seed=77)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    X = dev_bf16(gen_activations((M, K), seed=78))
    work = work_for(q4, M, N, K, q4.Q4NX_WEIGHTS_Q4NX)
    ref = torch.empty((M, N), dtype=torch.float32, device="cuda")
    q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, ref, work=work)
    Y = torch.empty_like(ref)
    for _ in range(10):
        work.fill_(float("nan"))
        Y.fill_(float("nan"))
        q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, Y, work=work)
        torch.cuda.synchronize()
        assert torch.equal(Y.view(torch.int32), ref.view(torch.int32))
    # And ten back to back without clearing (the partials of the previous
    # call in place).
    outs = [torch.empty_like(ref) for _ in range(10)]
    for y in outs:
        q4.q4nx_gemm_ex(q4.Q4NX_WEIGHTS_Q4NX, M, N, K, X, blob, y, work=work)
    torch.cuda.synchronize()
    assert all(torch.equal(y.view(torch.int32), ref.view(torch.int32)) for y in outs)


# The kernel that splits K over a workgroup's waves (q4nx_gemm's choice for few
# rows on a 256-CU device): ragged N (not a multiple of a strip) and mostly a
# ragged M, K that ends inside a 128-column unit, K of one group, one unit, and
# many units.
FEW_ROWS = [(16, 100, 1184), (1, 6001, 1184), (34, 3001, 1184), (47, 6001, 1184), (145, 2501, 1184),
            (67, 8001, 1184), (193, 4001, 1184), (145, 6001, 1184), (163, 6001, 1184), (193, 6001, 1184),
            (3, 40, 32), (17, 33, 128), (77, 2560, 10272),
            # the tiles of 80 x 64, 128 x 64 and those of 80 and 96 columns, K ending inside a unit
            (65, 12001, 672), (110, 15001, 1184), (49, 18001, 672), (65, 18001, 672), (49, 24001, 672), (65, 24001, 672),
            (163, 10001, 672)]
# One shape per tile (test_gemm_launches.py checks that they reach it), with several ragged tiles in
# either direction and K ending inside a unit.
FEW_ROWS_TILES = [(18, 35, 320, "16x16"), (20, 2101, 416, "16x32"), (68, 847, 288, "32x32"), (101, 2203, 288, "48x32"),
                  (105, 3551, 288, "32x64"), (66, 7535, 544, "48x64"), (421, 2199, 416, "64x64"),
                  (130, 7597, 480, "80x64"), (247, 4177, 608, "96x64"), (435, 4089, 1312, "128x64"),
                  (97, 8427, 736, "64x80"), (133, 9891, 736, "80x80"), (217, 5523, 864, "64x96"),
                  (258, 5719, 352, "80x96"), (175, 8353, 736, "96x96")]


@pytest.mark.parametrize("M,N,K", FEW_ROWS + [shape[:3] for shape in FEW_ROWS_TILES])
def test_gemm_few_rows(q4, M, N, K):
    """Float32 and bf16 outputs against the float64 product of the bf16
    weights (within 1e-5 of sum |x w|: float32 sums of exact products, over
    sampled rows), nothing written past M x N, and the same bits from the
    packed matrix, the MXFP4 variant and the bf16 weights they dequantize to."""
    _say("gemm few rows", M, N, K)
    codes, s, o = gen_weights(N, K, seed=M + N)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    Xh = gen_activations((M, K), seed=K + M)
    X = dev_bf16(Xh)
    W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    Y = [torch.full((M * N + 64,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
    q4.q4nx_gemm(M, N, K, X, blob, Y[0])
    q4.q4nx_dequant(blob, N, K, W)
    q4.q4nx_gemm_bf16(M, N, K, X, W, Y[1])
    Yb = torch.full((M * N + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    q4.q4nx_gemm(M, N, K, X, blob, Yb)
    torch.cuda.synchronize()
    assert torch.equal(Y[0].view(torch.int32), Y[1].view(torch.int32))
    assert torch.equal(Yb[:M * N].view(torch.int16), Y[0][:M * N].bfloat16().view(torch.int16))
    assert torch.isnan(Y[0][M * N:]).all() and torch.isnan(Yb[M * N:]).all()
    rows = np.unique(np.concatenate([np.arange(min(M, 4)), M - 1 - np.arange(min(M, 20))]))
    w16 = oracle.bf16_to_f32(oracle.f32_to_bf16(oracle.dequant_f32(codes, s, o)))
    err = np.abs(host_f32(Y[0])[:M * N].reshape(M, N)[rows].astype(np.float64) - oracle.gemm_f64(Xh[rows], w16))
    assert (err <= 1e-5 * oracle.abs_bound(Xh[rows], w16) + 1e-6).all()
    mcodes, msc = gen_mx_weights(N, K, seed=K, mode="edge")
    mblob = dev_u8(q4.q4nx_mx_pack(mcodes, msc))
    q4.q4nx_mx_gemm(M, N, K, X, mblob, Y[0])
    q4.q4nx_mx_dequant(mblob, N, K, W)
    q4.q4nx_gemm_bf16(M, N, K, X, W, Y[1])
    torch.cuda.synchronize()
    assert torch.equal(Y[0].view(torch.int32), Y[1].view(torch.int32))


# The hand-scheduled kernel and the general one, one launch or two over a split
# of the rows or the columns: ragged M and N throughout, K of one, two, three
# and five steps.
TILE_SHAPES = [(80, 5000, 64), (80, 20001, 64), (140, 20001, 64), (200, 20001, 64), (60, 43001, 64),
               (260, 30001, 64), (400, 20001, 128), (140, 43001, 64), (260, 43001, 192), (580, 20001, 320),
               (520, 30001, 64), (580, 30001, 64), (400, 43001, 192), (1999, 20001, 192)]


# K of at most 448, a multiple of 64: the general kernel's 128 and 256 row tiles (test_gemm_launches.py
# checks that they reach it), of one, two, four and seven steps.
SHORT_K = [(272, 9909, 64, "128x128"), (504, 12417, 128, "256x128"), (741, 7685, 256, "256x128"),
           (1835, 1257, 448, "128x128")]
# Each tile of the hand-scheduled kernel with each weight operand (the packed and the other operands may
# take another tile at a shape), over an odd and an even number of steps that takes every register set
# around at least twice; and the general kernel's tiles with a K tail, of several steps.
TILE_STEPS = [(33, 8213, 576), (33, 11403, 640), (33, 33813, 320), (33, 33351, 384), (67, 16387, 576), (66, 16457, 640),
              (129, 16571, 576), (130, 16899, 640), (129, 33057, 320), (131, 32775, 384), (257, 21929, 320),
              (258, 22457, 384), (194, 16599, 576), (193, 16701, 640), (257, 33027, 320), (257, 34171, 384),
              (387, 24609, 320), (386, 24615, 384), (323, 24947, 320), (323, 24613, 384), (193, 32825, 320),
              (195, 33139, 384)]
K_TAILS = [(66, 11059, 288, "general 128x64"), (33, 28325, 288, "general 128x128"),
           (134, 16407, 352, "general 256x128"), (260, 17547, 288, "gemm256 256x256"),
           (84, 36249, 352, "general 128x128 + general 128x64")]


@pytest.mark.parametrize("M,N,K", TILE_SHAPES + TILE_STEPS + [shape[:3] for shape in SHORT_K + K_TAILS])
def test_gemm_tiles(q4, M, N, K):
    """Sampled rows against the float64 product of the bf16 weights within the
    tight bound, every element (packed, MXFP4 and bf16 weights, float32 and
    bf16 outputs) against the same bits, nothing written past M x N."""
    _say("gemm tiles", M, N, K)
    codes, s, o = gen_weights(N, K, seed=M + N)
    blob = dev_u8(q4.q4nx_pack(codes, s, o))
    Xh = gen_activations((M, K), seed=K + M)
    X = dev_bf16(Xh)
    W = torch.empty((N, K), dtype=torch.bfloat16, device="cuda")
    Y = [torch.full((M * N + 64,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(2)]
    Yb = torch.full((M * N + 64,), float("nan"), dtype=torch.bfloat16, device="cuda")
    q4.q4nx_gemm(M, N, K, X, blob, Y[0])
    q4.q4nx_dequant(blob, N, K, W)
    q4.q4nx_gemm_bf16(M, N, K, X, W, Y[1])
    q4.q4nx_gemm(M, N, K, X, blob, Yb)
    torch.cuda.synchronize()
    assert torch.equal(Y[0].view(torch.int32), Y[1].view(torch.int32))
    assert torch.equal(Yb[:M * N].view(torch.int16), Y[0][:M * N].bfloat16().view(torch.int16))
    assert torch.isnan(Y[0][M * N:]).all() and torch.isnan(Yb[M * N:]).all()
    rng = np.random.default_rng(M)
    rows = np.unique(np.concatenate([np.arange(4), M - 1 - np.arange(8), rng.integers(0, M, 8)]))
    w16 = oracle.bf16_to_f32(oracle.f32_to_bf16(oracle.dequant_f32(codes, s, o)))
    got = Y[0][:M * N].view(M, N)[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    assert (np.abs(got - oracle.gemm_f64(Xh[rows], w16)) <= 1e-5 * oracle.abs_bound(Xh[rows], w16) + 1e-6).all()
    mcodes, msc = gen_mx_weights(N, K, seed=K, mode="edge")
    mblob = dev_u8(q4.q4nx_mx_pack(mcodes, msc))
    q4.q4nx_mx_gemm(M, N, K, X, mblob, Y[0])
    q4.q4nx_mx_dequant(mblob, N, K, W)
    q4.q4nx_gemm_bf16(M, N, K, X, W, Y[1])
    torch.cuda.synchronize()
    assert torch.equal(Y[0].view(torch.int32), Y[1].view(torch.int32))
