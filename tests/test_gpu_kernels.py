"""Parity of each HIP kernel with the matching step of the oracle (GPU only).
Sizes span several tiles and a ragged tail; tolerances are the per-dtype bars
(relative L2 1e-4 fp32, 2e-2 bf16)."""
import numpy as np
import pytest
import torch

from oracle import layer as L
from paper_2204_12013_amd import synth
from util import TOL, assert_close, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def B():
    from paper_2204_12013_amd import binding
    return binding


def _mk(rng, shape, dtype, scale=1.0, shift=0.0):
    a = synth.round_to_storage(rng.standard_normal(shape).astype(np.float32) * np.float32(scale) + np.float32(shift), dtype)
    return a


def _dev(B, a, dtype):
    return B.to_device(a, dtype, DEV)


def _empty(shape, dtype):
    return torch.empty(*shape, dtype=torch.bfloat16 if dtype == 1 else torch.float32, device=DEV)


IMPLS = [(0, 1), (1, 1), (1, 0)]          # (dtype, impl)
GEMM_SHAPES = [(32, 64, 64), (200, 136, 72), (333, 520, 264), (512, 768, 256)]
# shapes for the MFMA kernel alone: every tile configuration (128x128, 256x128,
# 256x256 output tiles), ragged edges in all three dimensions, K tails
MFMA_SHAPES = [(8, 8, 8), (136, 264, 72), (520, 392, 200), (1024, 1024, 512), (4096, 2048, 192),
               (4096, 4096, 128), (4104, 4040, 72), (2048, 1600, 320)]


@pytest.mark.parametrize("dtype,impl", IMPLS)
@pytest.mark.parametrize("T,N,K", GEMM_SHAPES)
def test_linear_forward_variants(B, dtype, impl, T, N, K):
    rng = np.random.default_rng(T + N + K)
    X, W = _mk(rng, (T, K), dtype), _mk(rng, (K, N), dtype, 0.05)
    b, R = _mk(rng, (N,), dtype, 0.1), _mk(rng, (T, N), dtype)
    ref = X.astype(np.float64) @ W.astype(np.float64) + b
    Y = _empty((T, N), dtype)
    B.bk_linear_fwd(_dev(B, X, dtype), _dev(B, W, dtype), _dev(B, b, dtype), Y, impl=impl)
    assert_close(B.to_host(Y), ref, TOL[dtype], "kernels B.to_host(Y)")
    B.bk_linear_fwd(_dev(B, X, dtype), _dev(B, W, dtype), _dev(B, b, dtype), Y, res=_dev(B, R, dtype), impl=impl)
    assert_close(B.to_host(Y), ref + R, TOL[dtype], "kernels B.to_host(Y)")
    G = _empty((T, N), dtype)
    B.bk_linear_fwd(_dev(B, X, dtype), _dev(B, W, dtype), _dev(B, b, dtype), Y, gelu_out=G, impl=impl)
    assert_close(B.to_host(Y), L.gelu_grad(ref), TOL[dtype], "kernels B.to_host(Y)")  # the derivative the backward multiplies by
    assert_close(B.to_host(G), L.gelu(ref), TOL[dtype], "kernels B.to_host(G)")


@pytest.mark.parametrize("T,N,K", MFMA_SHAPES)
def test_linear_forward_mfma(B, T, N, K):
    test_linear_forward_variants(B, 1, 2, T, N, K)


@pytest.mark.parametrize("T,N,K", MFMA_SHAPES)
def test_linear_backward_mfma(B, T, N, K):
    test_linear_backward_variants(B, 1, 2, T, N, K)


@pytest.mark.parametrize("T,N,K", [(520, 392, 448), (1024, 1152, 1024)])
def test_mfma_tiles_and_pipeline_depths_agree_bitwise(B, T, N, K):
    """Every output tile shape and every depth of the LDS slice ring walks K in the same order with the
    same matrix instruction, so the results must be identical to the last bit: the tile choice can
    then never break the bitwise FRC == successor and failover == failure-free invariants."""
    rng = np.random.default_rng(T + N)
    X, W, b = _mk(rng, (T, K), 1), _mk(rng, (K, N), 1, 0.05), _mk(rng, (N,), 1, 0.1)
    dY, R = _mk(rng, (T, N), 1), _mk(rng, (T, N), 1)
    Xd, Wd, bd, dYd, Rd = (_dev(B, a, 1) for a in (X, W, b, dY, R))
    ref = None
    try:
        for tile in (22, 11, 24, 42, 44, 43):
            for depth in (2, 3, 4):
                B.bk_gemm_tile(tile)
                B.bk_gemm_stages(depth)
                Y, G, dX = _empty((T, N), 1), _empty((T, N), 1), _empty((T, K), 1)
                dW = torch.zeros(K, N, dtype=torch.float32, device=DEV)
                B.bk_linear_fwd(Xd, Wd, bd, Y, gelu_out=G, impl=2)
                Y2, Y3 = _empty((T, N), 1), _empty((T, N), 1)
                B.bk_linear_fwd(Xd, Wd, bd, Y2, res=Rd, impl=2)
                B.bk_linear_fwd(Xd, Wd, bd, Y3, impl=2)          # bias only: the form that has the 256 x 192 tile
                B.bk_linear_bwd_input(dYd, Wd, dX, mul=Xd, impl=2)
                B.bk_linear_bwd_weight(Xd, dYd, dW, impl=2)
                torch.cuda.synchronize()
                got = (Y, G, Y2, Y3, dX, dW)
                if ref is None:
                    ref = got
                    assert_close(B.to_host(Y2), X.astype(np.float64) @ W.astype(np.float64) + b + R, TOL[1], "kernels B.to_host(Y2)")
                else:
                    for a, r in zip(got, ref):
                        assert torch.equal(a, r), (tile, depth)
    finally:
        B.bk_gemm_tile(0)
        B.bk_gemm_stages(0)


def test_a_forced_ring_depth_holds_for_products_that_would_split_K(B):
    T, K, N = 512, 4096, 1024
    gen = torch.Generator(device=DEV)
    gen.manual_seed(1)
    X, W, b = (torch.randn(*s, generator=gen, device=DEV).bfloat16() for s in ((T, K), (K, N), (N,)))
    tiled, auto, forced = (_empty((T, N), 1) for _ in range(3))
    B.bk_linear_fwd(X, W, b, tiled, impl=2)
    B.bk_linear_fwd(X, W, b, auto)
    B.bk_gemm_stages(3)
    try:
        B.bk_linear_fwd(X, W, b, forced)
    finally:
        B.bk_gemm_stages(0)
    assert torch.equal(forced, tiled) and not torch.equal(auto, tiled)


@pytest.mark.parametrize("shapes", [
    # (T, K, N) per problem: ragged edges, different contraction lengths, one to four problems
    [(512, 136, 264), (192, 128, 128)],
    [(448, 1024, 392), (448, 64, 72), (320, 520, 8), (1024, 256, 256)],
    [(4096, 1024, 1024), (4096, 1024, 3072)],
    [(256, 200, 96)],
    [(100, 64, 64), (256, 64, 64)],            # a contraction length that ends inside a 64-deep slice
    [(130, 6400, 1600), (130, 1600, 6400), (130, 1600, 1600), (130, 1600, 4800)],   # short products: two workgroups to a CU
])
def test_grouped_weight_gradients_equal_the_single_launches_bitwise(B, shapes):
    rng = np.random.default_rng(len(shapes) * 7 + shapes[0][0])
    Xs, dYs, inits = [], [], []
    for T, K, N in shapes:
        Xs.append(_dev(B, _mk(rng, (T, K), 1), 1))
        dYs.append(_dev(B, _mk(rng, (T, N), 1), 1))
        inits.append(torch.from_numpy(rng.normal(0, 1, (K, N)).astype(np.float32)).to(DEV))
    single = [w.clone() for w in inits]
    for X, dY, dW in zip(Xs, dYs, single):
        B.bk_linear_bwd_weight(X, dY, dW)
    try:
        for tile in (0, 22, 44, 24, 42):             # the last two are launched singly
            B.bk_gemm_tile(tile)
            grouped = [w.clone() for w in inits]
            B.bk_linear_bwd_weight_group(Xs, dYs, grouped)
            torch.cuda.synchronize()
            for a, b in zip(grouped, single):
                assert torch.equal(a, b), tile
    finally:
        B.bk_gemm_tile(0)
    T, K, N = shapes[0]
    want = inits[0].cpu().numpy().astype(np.float64) + B.to_host(Xs[0]).T @ B.to_host(dYs[0])
    assert_close(single[0].cpu().numpy(), want, 1e-5, "kernels single[0].cpu().numpy()")


@pytest.mark.parametrize("depth", [2, 3])
@pytest.mark.parametrize("shapes", [[(64, 136, 264), (64, 128, 128)], [(65, 520, 72), (1, 64, 64), (200, 256, 1032)],
                                    [(1000, 640, 2560), (1000, 2560, 640), (1000, 640, 640), (1000, 640, 1920)]])
def test_grouped_weight_gradients_with_either_ring_of_the_128_tile(B, shapes, depth):
    """One slice and fewer than the ring holds, a contraction that ends inside a slice, more tiles than fit the chip at two
    a CU; bitwise the single launches."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(depth)
    Xs = [torch.randn(T, K, generator=gen, device=DEV).bfloat16() for T, K, N in shapes]
    dYs = [torch.randn(T, N, generator=gen, device=DEV).bfloat16() for T, K, N in shapes]
    single = [torch.randn(K, N, generator=gen, device=DEV) for T, K, N in shapes]
    grouped = [w.clone() for w in single]
    for X, dY, dW in zip(Xs, dYs, single):
        B.bk_linear_bwd_weight(X, dY, dW)
    try:
        B.bk_gemm_tile(22)
        B.bk_gemm_stages(depth)
        B.bk_linear_bwd_weight_group(Xs, dYs, grouped)
    finally:
        B.bk_gemm_tile(0)
        B.bk_gemm_stages(0)
    assert all(torch.equal(a, b) for a, b in zip(grouped, single))


@pytest.mark.parametrize("dtype", [0, 1])
def test_grouped_weight_gradients_into_the_same_matrix_are_added_in_order(B, dtype):
    """Two problems that add to one matrix (and a third that adds to rows of it) are the single launches one after the other."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(dtype)
    act = torch.bfloat16 if dtype == 1 else torch.float32
    T, K, N = 96, 128, 72
    Xs, dYs = ([torch.randn(T, n, generator=gen, device=DEV).to(act) for n in ns] for ns in ((K, K, 64), (N, N, N)))
    init = torch.randn(K, N, generator=gen, device=DEV)
    single, grouped = init.clone(), init.clone()
    for X, dY, dW in zip(Xs, dYs, (single, single, single[32:96])):
        B.bk_linear_bwd_weight(X, dY, dW)
    B.bk_linear_bwd_weight_group(Xs, dYs, [grouped, grouped, grouped[32:96]])
    assert torch.equal(single, grouped)


def test_mfma_kernel_refuses_what_it_does_not_cover(B):
    X, W, b = _empty((12, 16), 1), _empty((16, 24), 1), _empty((24,), 1)
    with pytest.raises(B.BambooError) as e:
        B.bk_linear_fwd(X, W, b, _empty((12, 24), 1), impl=2)        # 12 rows: not a multiple of 8
    assert e.value.status == B.E_STATE
    Xf, Wf, bf = _empty((16, 16), 0), _empty((16, 24), 0), _empty((24,), 0)
    with pytest.raises(B.BambooError) as e:
        B.bk_linear_fwd(Xf, Wf, bf, _empty((16, 24), 0), impl=2)     # fp32 has no MFMA kernel here
    assert e.value.status == B.E_STATE


@pytest.mark.parametrize("T,K,N", [
    # few output tiles: the kernels whose wavefronts split K, at the edges of their 32 / 64 tiles and of K's slices
    (1, 8, 8), (7, 56, 1032), (31, 1024, 264), (33, 520, 40), (129, 4096, 72), (333, 1096, 1024), (999, 1024, 1032),
    # many: the tiled kernels (every shape is forced below)
    (2077, 200, 1032), (2049, 56, 1160), (1999, 1032, 1544)])
def test_any_row_count_and_contraction_tail(B, T, K, N):
    """Token counts that divide by nothing and contraction lengths that end inside a 64-deep slice (the missing part
    is loaded as zeros), in every form; the row behind the output stays untouched.  Bound: the
    results round once to bf16 (2^-9 relative per element, so relative L2 below it), the weight gradient sums
    T products in fp32 (T 2^-24 relative to the sum of magnitudes at most; 1e-5 leaves an order of magnitude)."""
    rng = np.random.default_rng(T * 31 + K + N)
    X, W = _mk(rng, (T, K), 1), _mk(rng, (K, N), 1, 0.05)
    b, dY, Mu = _mk(rng, (N,), 1, 0.1), _mk(rng, (T, N), 1), _mk(rng, (T, K), 1)
    Xd, Wd, bd, dYd, Md = (_dev(B, a, 1) for a in (X, W, b, dY, Mu))
    h = X.astype(np.float64) @ W.astype(np.float64) + b
    dx = dY.astype(np.float64) @ W.astype(np.float64).T
    dw = X.astype(np.float64).T @ dY.astype(np.float64)
    dYs = [dYd, _dev(B, _mk(rng, (T, N), 1), 1)]
    try:
        for tile in (0, 11, 22, 24, 42, 44):
            B.bk_gemm_tile(tile)
            B.bk_gemm_stages(2 if tile else 0)           # with a forced depth no product goes to the kernels that split K
            Y, G, dX = (torch.full((T + 1, n), 7.0, device=DEV).to(torch.bfloat16) for n in (N, N, K))
            B.bk_linear_fwd(Xd, Wd, bd, Y[:T])
            assert rel_l2(B.to_host(Y[:T]), h) < 2.0 ** -8 and bool((Y[T] == 7).all())
            B.bk_linear_fwd(Xd, Wd, bd, Y[:T], gelu_out=G[:T])
            # evaluated at the fp32 pre-activation: what a rounding of the exact values to bf16 costs, and fp32 errors
            # (1e-5 of h at most), twice where they move a value over a rounding boundary
            for got, want in ((G, L.gelu(h)), (Y, L.gelu_grad(h))):
                rounded = synth.round_to_storage(want.astype(np.float32), 1).astype(np.float64)
                assert rel_l2(B.to_host(got[:T]), want) < rel_l2(rounded, want) + 2e-5 and bool((got[T] == 7).all())
            B.bk_linear_bwd_input(dYd, Wd, dX[:T], mul=Md)
            assert rel_l2(B.to_host(dX[:T]), dx * Mu) < 2.0 ** -8 and bool((dX[T] == 7).all())
            single, grouped = ([torch.zeros(K, N, device=DEV) for _ in dYs] for _ in range(2))
            for g, dW in zip(dYs, single):
                B.bk_linear_bwd_weight(Xd, g, dW)
            assert rel_l2(single[0].cpu().numpy(), dw) < 1e-5
            B.bk_gemm_stages(0)                          # a forced depth takes the group apart
            B.bk_linear_bwd_weight_group([Xd, Xd], dYs, grouped)
            for a, b in zip(grouped, single):
                assert torch.equal(a, b), tile
    finally:
        B.bk_gemm_tile(0)
        B.bk_gemm_stages(0)


def test_operands_whose_rows_are_millions_long(B):
    """A tile's loads count their offsets from its first row, and 256 rows of 4.26 M elements span more than the 2 GiB
    that such a load reaches; with rows of 17.2 M 64 of them do, and only the 32-row tiles are left.  The last row must
    count like the first, in both forms with contiguous rows.  Sums of powers of two: exact up to the rounding to bf16."""
    for rows, cols, unit, tiles in ((256, 65 * 65536, 2.0 ** -10, (0, 44, 43)), (64, 262 * 65536, 2.0 ** -12, (0,))):
        A = torch.zeros(rows, cols, dtype=torch.bfloat16, device=DEV)
        A[0] = A[rows - 1] = 1
        u = torch.full((8 * cols,), unit, dtype=torch.bfloat16, device=DEV)
        bias = torch.zeros(8, dtype=torch.bfloat16, device=DEV)
        for tile in tiles:
            Y, dX = _empty((rows, 8), 1), _empty((8, rows), 1)
            B.bk_gemm_tile(tile)
            try:
                B.bk_linear_fwd(A, u.view(cols, 8), bias, Y, impl=2 if tile else 0)      # Y = A W
                B.bk_linear_bwd_input(u.view(8, cols), A, dX, impl=2 if tile else 0)     # dX = dY A^T
            finally:
                B.bk_gemm_tile(0)
            for got in (Y, dX.t()):
                assert torch.allclose(got[[0, -1]].float(), torch.tensor(cols * unit, device=DEV), rtol=2.0 ** -8), (rows, tile)
                assert bool((got[1:-1] == 0).all()), (rows, tile)
        if rows == 64:
            with pytest.raises(B.BambooError) as e:
                B.bk_linear_fwd(A, u.view(cols, 8), bias, Y, impl=2)       # the smallest tile without a split of K has 64 rows
            assert e.value.status == B.E_STATE
        del A, u
        torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,impl", IMPLS)
@pytest.mark.parametrize("T,N,K", GEMM_SHAPES)
def test_linear_backward_variants(B, dtype, impl, T, N, K):
    rng = np.random.default_rng(T * 3 + N + K)
    X, W, dY = _mk(rng, (T, K), dtype), _mk(rng, (K, N), dtype, 0.05), _mk(rng, (T, N), dtype)
    R, Hh = _mk(rng, (T, K), dtype), _mk(rng, (T, K), dtype)
    ref = dY.astype(np.float64) @ W.astype(np.float64).T
    dX = _empty((T, K), dtype)
    B.bk_linear_bwd_input(_dev(B, dY, dtype), _dev(B, W, dtype), dX, impl=impl)
    assert_close(B.to_host(dX), ref, TOL[dtype], "kernels B.to_host(dX)")
    B.bk_linear_bwd_input(_dev(B, dY, dtype), _dev(B, W, dtype), dX, res=_dev(B, R, dtype), impl=impl)
    assert_close(B.to_host(dX), ref + R, TOL[dtype], "kernels B.to_host(dX)")
    B.bk_linear_bwd_input(_dev(B, dY, dtype), _dev(B, W, dtype), dX, mul=_dev(B, Hh, dtype), impl=impl)
    assert_close(B.to_host(dX), ref * Hh.astype(np.float64), TOL[dtype], "kernels B.to_host(dX)")
    # weight gradient accumulates into fp32
    dW0 = rng.standard_normal((K, N)).astype(np.float32)
    dW = torch.from_numpy(dW0.copy()).to(DEV)
    db0 = rng.standard_normal(N).astype(np.float32)
    db = torch.from_numpy(db0.copy()).to(DEV)
    B.bk_linear_bwd_weight(_dev(B, X, dtype), _dev(B, dY, dtype), dW, impl=impl)
    B.bk_linear_bwd_weight(_dev(B, X, dtype), _dev(B, dY, dtype), dW, db=db, impl=impl)
    want = 2 * (X.astype(np.float64).T @ dY.astype(np.float64))
    assert_close(dW.cpu().numpy().astype(np.float64) - dW0, want, TOL[dtype], "kernels dW.cpu().numpy().astype(np.float64) - dW0")
    # the bias gradient of the same linear layer
    assert_close(db.cpu().numpy().astype(np.float64) - db0, dY.astype(np.float64).sum(0), 1e-4, "kernels db.cpu().numpy().astype(np.float64) - db0")


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("T,N", [(32, 64), (333, 200), (4096, 1024)])
def test_colsum(B, dtype, T, N):
    rng = np.random.default_rng(T + N)
    A = _mk(rng, (T, N), dtype)
    out0 = rng.standard_normal(N).astype(np.float32)
    out = torch.from_numpy(out0.copy()).to(DEV)
    B.bk_colsum_acc(_dev(B, A, dtype), out)
    assert_close(out.cpu().numpy() - out0, A.astype(np.float64).sum(0), 1e-4, "kernels out.cpu().numpy() - out0")


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("T,H", [(32, 64), (77, 200), (515, 1024), (130, 1600), (70, 12288), (37, 5000)])
def test_layernorm_forward_backward(B, dtype, T, H):
    rng = np.random.default_rng(T + H)
    r = _mk(rng, (T, H), dtype, 2.0, 0.5)
    g, b = _mk(rng, (H,), dtype, 0.1, 1.0), _mk(rng, (H,), dtype, 0.1)
    dout, add = _mk(rng, (T, H), dtype), _mk(rng, (T, H), dtype)
    y_ref, cache = L.layernorm_fwd(r.astype(np.float64), g.astype(np.float64), b.astype(np.float64), 1e-5)
    y, stats = _empty((T, H), dtype), torch.empty(T, 2, dtype=torch.float32, device=DEV)
    B.bk_layernorm_fwd(_dev(B, r, dtype), _dev(B, g, dtype), _dev(B, b, dtype), y, stats)
    assert_close(B.to_host(y), y_ref, TOL[dtype], "kernels B.to_host(y)")
    st = stats.cpu().numpy()
    assert_close(st[:, 0], r.astype(np.float64).mean(-1), 1e-5, "kernels st[:, 0]")
    assert_close(st[:, 1], cache[1][:, 0], 1e-5, "kernels st[:, 1]")
    dr_ref, dg_ref, db_ref = L.layernorm_bwd(dout.astype(np.float64), g.astype(np.float64), cache)
    dr = _empty((T, H), dtype)
    dg = torch.zeros(H, dtype=torch.float32, device=DEV)
    db = torch.zeros(H, dtype=torch.float32, device=DEV)
    B.bk_layernorm_bwd(_dev(B, dout, dtype), _dev(B, r, dtype), stats, _dev(B, g, dtype), dr, dg, db)
    assert_close(B.to_host(dr), dr_ref, TOL[dtype], "kernels B.to_host(dr)")
    assert_close(dg.cpu().numpy(), dg_ref, 1e-4, "kernels layernorm gain gradient")
    assert_close(db.cpu().numpy(), db_ref, 1e-4, "kernels layernorm shift gradient")
    B.bk_layernorm_bwd(_dev(B, dout, dtype), _dev(B, r, dtype), stats, _dev(B, g, dtype), dr, dg, db,
                       add=_dev(B, add, dtype))
    assert_close(B.to_host(dr), dr_ref + add, TOL[dtype], "kernels B.to_host(dr)")
    assert_close(dg.cpu().numpy(), 2 * dg_ref, 1e-4, "kernels dg.cpu().numpy()")


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("T,H", [(1, 8), (7, 512), (8, 520), (9, 1024), (17, 1032), (25, 2048), (2049, 72), (3, 2056), (9, 4104),
                                 (5, 8192), (257, 8200), (5, 12288), (3, 12296), (2, 16392)])
def test_layernorm_at_the_edges_of_its_kernels(B, dtype, T, H):
    """Rows a wavefront holds in one, two and four vectors a lane, rows a workgroup holds in one to four a thread, and
    longer ones; fewer rows than wavefronts, one more than a pass takes, one more than the partial rows."""
    test_layernorm_forward_backward(B, dtype, T, H)


@pytest.mark.parametrize("residual", [0, 1])
@pytest.mark.parametrize("dtype,T,H", [(0, 9, 64), (0, 700, 512), (0, 300, 1024), (0, 301, 1032), (0, 2100, 2056), (0, 5, 4104),
                                       (0, 20, 6144), (0, 7, 6152), (1, 9, 72), (1, 700, 1024), (1, 2100, 1600), (1, 301, 2048),
                                       (1, 301, 2056), (1, 2100, 4104), (1, 300, 8200), (1, 2057, 12288), (1, 7, 12296)])
def test_layernorm_backward_with_the_bias_gradient(B, dtype, T, H, residual):
    """The sums a stage asks for beside gain and shift: of dr as it is stored.  Every kernel, few rows, several a workgroup
    (one or two passes of its wavefronts) and a short last workgroup.  dr is the same as without them but for an fp32
    rounding (half an ulp, 2^-24, on either side); sums of T fp32 terms are off by at most T 2^-24 of the sum of magnitudes."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(T + H)
    act = torch.bfloat16 if dtype else torch.float32
    r, d, add = (torch.randn(T, H, generator=gen, device=DEV).to(act) for _ in range(3))
    gamma, beta = (torch.randn(H, generator=gen, device=DEV).to(act) for _ in range(2))
    add = add if residual else None
    y, stats = torch.empty_like(r), torch.empty(T, 2, device=DEV)
    B.bk_layernorm_fwd(r, gamma, beta, y, stats)
    plain, dr = torch.empty_like(r), torch.empty_like(r)
    g0, b0, g1, b1 = (torch.zeros(H, device=DEV) for _ in range(4))
    c1 = torch.full((H,), 3.0, device=DEV)
    B.bk_layernorm_bwd(d, r, stats, gamma, plain, g0, b0, add=add)
    B.bk_layernorm_bwd_bias(d, r, stats, gamma, dr, g1, b1, c1, add=add)
    assert (dr.double() - plain.double()).norm() <= 2.0 ** -23 * plain.double().norm()
    assert torch.equal(g0, g1) and torch.equal(b0, b1)
    want = 3.0 + dr.double().sum(0)
    assert bool(((c1.double() - want).abs() <= T * 2.0 ** -24 * (3.0 + dr.double().abs().sum(0))).all())


def _fma(a, b, c):
    """One rounding, as the device's fma (fp64 holds the product of two fp32 values exactly)."""
    return (a.double() * b.double() + c.double()).float()


def _wavefront_sum(step, H, V, T):
    """A wavefront's sum over a row: lane l takes vectors l, l + 64, .. in order, then pairs 32, 16, .. 1 lanes apart.
    step(s, e): s with element e [T, lanes] of a lane's vector added; e indexes the columns, at least one lane's."""
    s = torch.zeros(T, 64, device=DEV)
    cols = torch.arange(H, device=DEV).view(H // V, V)
    for k in range(0, H // V, 64):
        c = cols[k:k + 64]
        for i in range(V):
            s[:, :len(c)] = step(s[:, :len(c)], c[:, i])
    for o in (32, 16, 8, 4, 2, 1):
        s = s[:, :o] + s[:, o:]
    return s[:, 0]


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("T,H", [(3, 1032), (9, 2056), (300, 2056), (17, 4104), (3, 8192), (2, 12288), (2, 16384)])
def test_layernorm_sums_a_row_in_the_order_of_a_wavefront(B, dtype, T, H):
    """Whatever kernel takes a row (a wavefront, or a workgroup for several): mean, rstd and dr to the bit as single
    operations in that order give them, since everything behind a LayerNorm is rounded to bf16."""
    rng = np.random.default_rng(H + T)
    V = 8 if dtype else 4
    mk = lambda s: B.to_device(synth.round_to_storage(s, dtype), dtype)
    r, d = mk(rng.normal(0.3, 1, (T, H))), mk(rng.normal(0, 1, (T, H)))
    gamma, beta = mk(rng.normal(1, 0.1, H)), mk(rng.normal(0, 0.1, H))
    y, stats, dr = torch.empty_like(r), torch.empty(T, 2, device=DEV), torch.empty_like(r)
    dg, db = torch.zeros(H, device=DEV), torch.zeros(H, device=DEV)
    B.bk_layernorm_fwd(r, gamma, beta, y, stats)
    B.bk_layernorm_bwd(d, r, stats, gamma, dr, dg, db)
    x, df, g = r.float(), d.float(), gamma.float()
    n = torch.tensor(float(H), device=DEV)
    mean = _wavefront_sum(lambda s, c: s + x[:, c], H, V, T) / n
    assert torch.equal(stats[:, 0], mean)
    m, rs = stats[:, :1], stats[:, 1:]
    var = _wavefront_sum(lambda s, c: _fma(x[:, c] - m, x[:, c] - m, s), H, V, T) / n
    assert (stats[:, 1].double() * (var.double() + 1e-5).sqrt() - 1).abs().max() < 2.0 ** -22      # rsqrt: an ulp or so
    dh, xh = df * g, (x - m) * rs
    m1 = _wavefront_sum(lambda s, c: _fma(df[:, c], g[c], s), H, V, T) / n
    m2 = _wavefront_sum(lambda s, c: _fma(dh[:, c], xh[:, c], s), H, V, T) / n
    want = _fma(-xh, m2[:, None], _fma(df, g, -m1[:, None])) * rs
    assert torch.equal(dr, want.to(dr.dtype))


def test_mfma_attention_refuses_sequences_beyond_its_32_bit_tile_offsets(B):
    # the MFMA kernels address a (batch, head) slice of qkv with 32-bit byte offsets: a sequence whose rows span
    # 4 GiB or more is refused when the kernels are forced, nothing is launched
    heads, d = 96, 128
    seq = (1 << 32) // (3 * heads * d * 2) + 1
    qkv = torch.empty((seq, 3 * heads * d), dtype=torch.bfloat16, device=DEV)
    ctx = torch.empty((seq, heads * d), dtype=torch.bfloat16, device=DEV)
    lse = torch.empty(heads * seq, dtype=torch.float32, device=DEV)
    with pytest.raises(B.BambooError) as e:
        B.bk_attention_fwd(qkv, ctx, lse, 1, seq, heads, 1, impl=2)
    assert e.value.status == B.E_STATE
    del qkv, ctx, lse
    torch.cuda.empty_cache()


ATTN_CASES = [(2, 16, 2, 32), (1, 100, 3, 64), (2, 200, 2, 128), (3, 77, 2, 40), (1, 512, 2, 64), (1, 300, 1, 128),
              (1, 1, 1, 64), (1, 129, 2, 64), (1, 8, 1, 128)]


@pytest.mark.parametrize("dtype,impl", IMPLS + [(1, 2)])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("batch,seq,heads,d", ATTN_CASES)
def test_attention_forward_backward(B, dtype, impl, causal, batch, seq, heads, d):
    rng = np.random.default_rng(seq + d + causal)
    H, T = heads * d, batch * seq
    qkv = _mk(rng, (T, 3 * H), dtype)
    dctx = _mk(rng, (T, H), dtype)
    if impl == 2 and d not in (64, 128):
        # the MFMA kernels cover head sizes 64 and 128 only: forcing them elsewhere is refused, not undefined
        # (the automatic choice, impl 0, falls back to the vector-ALU kernels and is checked below like any other)
        out = _empty((T, H), dtype)
        lse = torch.empty(batch * heads * seq, dtype=torch.float32, device=DEV)
        with pytest.raises(B.BambooError) as e:
            B.bk_attention_fwd(_dev(B, qkv, dtype), out, lse, batch, seq, heads, causal, impl=2)
        assert e.value.status == B.E_STATE
        with pytest.raises(B.BambooError) as e:
            B.bk_attention_bwd(_dev(B, qkv, dtype), out, lse, _dev(B, dctx, dtype), _empty((T, 3 * H), dtype), batch, seq,
                               heads, causal, impl=2)
        assert e.value.status == B.E_STATE
        return
    q64 = qkv.astype(np.float64)
    ctx_ref, probs = L.attention_fwd(q64, batch, seq, heads, bool(causal))
    ctx = _empty((T, H), dtype)
    lse = torch.empty(batch * heads * seq, dtype=torch.float32, device=DEV)
    dq = _dev(B, qkv, dtype)
    B.bk_attention_fwd(dq, ctx, lse, batch, seq, heads, causal, impl=impl)
    assert_close(B.to_host(ctx), ctx_ref, TOL[dtype], "kernels B.to_host(ctx)")
    # log-sum-exp against its definition
    lse_ref = np.zeros((batch, heads, seq))
    for b in range(batch):
        for h in range(heads):
            q = q64[b * seq:(b + 1) * seq, h * d:(h + 1) * d]
            k = q64[b * seq:(b + 1) * seq, H + h * d:H + (h + 1) * d]
            s = q @ k.T / np.sqrt(d)
            if causal:
                s = np.where(np.tril(np.ones((seq, seq), bool)), s, -np.inf)
            m = s.max(-1)
            lse_ref[b, h] = m + np.log(np.exp(s - m[:, None]).sum(-1))
    assert np.abs(lse.cpu().numpy().reshape(batch, heads, seq) - lse_ref).max() <= (1e-4 if dtype == 0 else 2e-2)
    dqkv_ref = L.attention_bwd(dctx.astype(np.float64), q64, probs, batch, seq, heads)
    dqkv = _empty((T, 3 * H), dtype)
    B.bk_attention_bwd(dq, ctx, lse, _dev(B, dctx, dtype), dqkv, batch, seq, heads, causal, impl=impl)
    got = B.to_host(dqkv)
    # a one-token sequence has dq = dk = 0 by cancellation (dP = delta): the three slices share the scale of
    # the terms they sum, that of the whole gradient
    floor = float(np.sqrt(np.mean(dqkv_ref ** 2))) if seq == 1 else 0.0
    for name, sl in (("dq", slice(0, H)), ("dk", slice(H, 2 * H)), ("dv", slice(2 * H, 3 * H))):
        assert_close(got[:, sl], dqkv_ref[:, sl], TOL[dtype], "kernels got[:, sl] %s" % (name,), floor=floor)


@pytest.mark.parametrize("dtype,impl,seq,d", [(0, 0, 1, 32), (0, 0, 40, 64), (1, 0, 77, 40), (1, 1, 33, 64), (1, 0, 200, 64),
                                             (1, 0, 3000, 64)])
def test_attention_backward_returns_delta(B, dtype, impl, seq, d):
    """The rows' sums of ctx * dctx come back from every path: the vector-ALU kernels, the matrix-core passes in one launch
    and in two.  Bound: 128 products at most in fp32."""
    act = torch.bfloat16 if dtype == 1 else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seq + d)
    heads, batch = 2, 2
    H, T = heads * d, batch * seq
    qkv, dctx = (torch.randn(T, n, generator=gen, device=DEV).to(act) for n in (3 * H, H))
    ctx, dqkv, lse = _empty((T, H), dtype), _empty((T, 3 * H), dtype), torch.empty(batch * heads * seq, device=DEV)
    B.bk_attention_fwd(qkv, ctx, lse, batch, seq, heads, 0, impl=impl)
    delta = B.bk_attention_bwd(qkv, ctx, lse, dctx, dqkv, batch, seq, heads, 0, impl=impl)
    want = (ctx.double() * dctx.double()).view(batch, seq, heads, d).sum(-1).permute(0, 2, 1).reshape(-1)
    size = (ctx.double() * dctx.double()).abs().view(batch, seq, heads, d).sum(-1).permute(0, 2, 1).reshape(-1)
    assert ((delta.double() - want).abs() <= 128 * 2.0 ** -24 * size).all()


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("seq,heads,d", [(1024, 1, 64), (1025, 1, 64), (1023, 2, 128)])
def test_attention_at_the_longest_sequence_of_the_one_launch_backward(B, causal, seq, heads, d):
    test_attention_forward_backward(B, 1, 2, causal, 1, seq, heads, d)


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("batch,seq,heads,d", [(1, 1, 3, 64), (2, 64, 2, 64), (1, 65, 2, 128), (2, 128, 2, 128), (1, 129, 2, 64),
                                               (1, 192, 2, 128), (1, 193, 3, 64), (2, 257, 2, 128), (1, 129, 128, 128),
                                               (1, 129, 129, 128)])
def test_attention_at_the_ends_of_its_tile_ring(B, causal, batch, seq, heads, d):
    """One to five tiles of 64 rows through a ring of two, a last tile of one row, and at head size 128 both sides of the
    256 workgroups from which on some CUs hold two."""
    test_attention_forward_backward(B, 1, 2, causal, batch, seq, heads, d)


@pytest.mark.parametrize("causal,batch,seq,heads,d", [(1, 9, 641, 3, 64), (1, 9, 704, 3, 64), (0, 3, 1025, 5, 128),
                                                      (0, 21, 300, 9, 128), (1, 9, 200, 9, 128), (1, 9, 192, 9, 128),
                                                      (1, 13, 260, 5, 128)])
def test_attention_forward_through_registers_and_straight_to_lds_is_the_same(B, causal, batch, seq, heads, d):
    """A whole batch (more keys and values than a chiplet's L2 holds, or more workgroups than CUs: tiles through registers)
    against its samples one by one (straight to LDS); odd and even numbers of tiles, a last tile of one row."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seq + d)
    H, T = heads * d, batch * seq
    qkv = torch.randn(T, 3 * H, generator=gen, device=DEV).bfloat16()
    ctx, lse = _empty((T, H), 1), torch.empty(batch * heads * seq, device=DEV)
    B.bk_attention_fwd(qkv, ctx, lse, batch, seq, heads, causal, impl=2)
    one, lse_one = _empty((seq, H), 1), torch.empty(heads * seq, device=DEV)
    for b in range(batch):
        rows = slice(b * seq, (b + 1) * seq)
        B.bk_attention_fwd(qkv[rows], one, lse_one, 1, seq, heads, causal, impl=2)
        assert torch.equal(one, ctx[rows]) and torch.equal(lse_one, lse[b * heads * seq:(b + 1) * heads * seq]), b


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("batch,seq,heads,d", [(8, 129, 16, 64), (8, 129, 17, 64), (3, 200, 27, 128),
                                                (12, 129, 17, 64), (6, 300, 43, 64), (5, 200, 27, 128)])
def test_attention_backward_in_one_launch_and_in_two_is_the_same(B, causal, batch, seq, heads, d):
    """A whole batch against its samples one by one (one launch): two launches for the third case without a mask, for
    the fourth to sixth (408, 774 and 270 workgroups a pass) with and without."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seq + heads)
    H, T = heads * d, batch * seq
    qkv = torch.randn(T, 3 * H, generator=gen, device=DEV).bfloat16()
    dctx = torch.randn(T, H, generator=gen, device=DEV).bfloat16()
    ctx, dqkv = _empty((T, H), 1), _empty((T, 3 * H), 1)
    lse = torch.empty(batch * heads * seq, device=DEV)
    B.bk_attention_fwd(qkv, ctx, lse, batch, seq, heads, causal, impl=2)
    B.bk_attention_bwd(qkv, ctx, lse, dctx, dqkv, batch, seq, heads, causal, impl=2)
    one = _empty((seq, 3 * H), 1)
    for b in range(batch):
        rows = slice(b * seq, (b + 1) * seq)
        B.bk_attention_bwd(qkv[rows], ctx[rows], lse[b * heads * seq:(b + 1) * heads * seq], dctx[rows], one, 1, seq,
                           heads, causal, impl=2)
        assert torch.equal(one, dqkv[rows]), b


@pytest.mark.parametrize("T,K,N", [(1, 1, 1), (31, 33, 65), (32, 64, 256), (100, 72, 200), (513, 130, 2049),
                                   # on the vector ALU: the forward, the input gradient, the forward with 16-byte loads
                                   (2100, 67, 1601), (2112, 1026, 1281), (2880, 512, 2944)])
def test_fp32_matrix_core_gemm(B, T, K, N):
    """The fp32 kernel at tile and step edges, unaligned lengths (no 16-byte loads) and on both sides of its split of K
    over wavefronts.  Bound: a sum of n products in fp32 is off by at most n 2^-24 of the sum of magnitudes, far less in
    relative L2; 1e-6 + n 2^-24 covers it."""
    rng = np.random.default_rng(T + K + N)
    X, W = rng.standard_normal((T, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    b, R = rng.standard_normal(N).astype(np.float32), rng.standard_normal((T, N)).astype(np.float32)
    dY, Mu = rng.standard_normal((T, N)).astype(np.float32), rng.standard_normal((T, K)).astype(np.float32)
    Xd, Wd, bd, Rd, dYd, Md = (torch.from_numpy(a).to(DEV) for a in (X, W, b, R, dY, Mu))
    f = lambda a: a.astype(np.float64)
    tol = lambda n: 1e-6 + n * 2.0 ** -24
    Y, G, dX, dW = (torch.empty(*s, device=DEV) for s in ((T, N), (T, N), (T, K), (K, N)))
    h = f(X) @ f(W) + b
    B.bk_linear_fwd(Xd, Wd, bd, Y, res=Rd)
    assert rel_l2(B.to_host(Y), h + R) < tol(K)
    B.bk_linear_fwd(Xd, Wd, bd, Y, gelu_out=G)
    # 1 + erf cancels for negative h: GELU and its derivative are off by an fp32 ulp of h resp. of 1, whatever their value
    for got, want, size in ((G, L.gelu(h), h), (Y, L.gelu_grad(h), np.maximum(np.abs(h), 1.0))):
        assert np.linalg.norm(B.to_host(got) - want) < tol(K) * np.linalg.norm(size)
    B.bk_linear_bwd_input(dYd, Wd, dX, mul=Md)
    assert rel_l2(B.to_host(dX), (f(dY) @ f(W).T) * Mu) < tol(N)
    dW.fill_(1.0)
    B.bk_linear_bwd_weight(Xd, dYd, dW)
    assert rel_l2(dW.cpu().numpy(), 1.0 + f(X).T @ f(dY)) < tol(T)
