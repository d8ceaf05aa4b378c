"""The MFMA projection y = x w against fp64 numpy, ragged shapes included."""
import numpy as np
import pytest

from helpers import PRODUCT_RTOL, relative_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,fin,fout", [(1, 1, 1), (127, 15, 16), (129, 17, 65), (1000, 602, 256),
                                        (513, 500, 64), (300, 64, 192), (2049, 33, 130)])
def test_linear(n, fin, fout):
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import assert_close, dev, empty
    print(f"linear: {n}x{fin}x{fout}", flush=True)
    rng = np.random.default_rng(n + fin + fout)
    x = rng.standard_normal((n, fin)).astype(np.float32)
    w = (rng.standard_normal((fin, fout)) / np.sqrt(fin)).astype(np.float32)
    y = empty((n, fout))
    pk.gnn_linear_fwd(dev(x), dev(w), y)
    torch.cuda.synchronize()
    assert_close("y", y.cpu().numpy(), x.astype(np.float64) @ w.astype(np.float64))


def _assert_within_rounding(name, got, a, b, parts=1):
    """|got - a b| <= (6 ceil(K / 16) + parts + 2) 2^-23 |a| |b| elementwise: each of the six partial products of 16 k is
    added with a loss of at most one unit in the last place of a sum that |a| |b| bounds, so is each part of a
    split product, and what the bf16 parts leave out is at most 2^-24 of it.  That worst case grows with K, the error with
    its root, so a lost partial product shows in the 2-norm."""
    a, b = a.astype(np.float64), b.astype(np.float64)
    ref = a @ b
    bound = (6 * -(-a.shape[1] // 16) + parts + 2) * 2.0 ** -23 * (np.abs(a) @ np.abs(b))
    worst = (np.abs(got - ref) / np.maximum(bound, 1e-300)).max()
    norm = relative_error(got, ref)
    print(f"{name}: worst error {worst:.3f} of the bound, 2-norm {norm:.1e}", flush=True)
    assert worst <= 1.0 and norm <= PRODUCT_RTOL


@pytest.mark.parametrize("n,fin,fout", [(31, 15, 4), (64, 16, 32), (65, 17, 36), (129, 31, 64), (33000, 33, 68),
                                        (66000, 48, 132), (66000, 600, 96), (33001, 130, 20), (33000, 5, 68),
                                        (66000, 8, 132), (40000, 16, 16), (33000, 17, 28), (300, 30, 260), (900, 32, 32),
                                        (66000, 48, 256), (66000, 256, 36), (300, 130, 140)])
def test_products_of_every_layout_and_tile(n, fin, fout):
    """A GCN layer on a graph of loops alone is its three products: x w, x^T g and g w^T."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    print(f"products: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fin + fout)
    x, w, gout = (rng.standard_normal(s).astype(np.float32) for s in ((n, fin), (fin, fout), (n, fout)))
    g = pk.Graph(dev(np.arange(n + 1, dtype=np.int32)), dev(np.arange(n, dtype=np.int32)))
    one, zs, out, gx, gw = dev(np.ones(n, np.float32)), empty((n, fout)), empty((n, fout)), empty((n, fin)), empty((fin, fout))
    ws = torch.empty(max(pk.gnn_gcn_workspace_bytes(g, fin, fout), 16), dtype=torch.uint8, device="cuda")
    pk.gnn_gcn_fwd(g, fin, fout, dev(x), dev(w), one, one, zs, out)
    pk.gnn_gcn_bwd(g, fin, fout, dev(x), dev(w), one, one, dev(gout), gx, gw, ws)
    torch.cuda.synchronize()
    _assert_within_rounding("x w", zs.cpu().numpy(), x, w)
    _assert_within_rounding("g w^T", gx.cpu().numpy(), gout, w.T)
    # the product over the vertices is split into up to 512 parts of at least 128
    _assert_within_rounding("x^T g", gw.cpu().numpy(), np.ascontiguousarray(x.T), gout, max(1, min(n // 128, 512)))


@pytest.mark.parametrize("n,fin,fout", [(1, 33, 1), (8192, 97, 32), (8192, 96, 33), (8193, 113, 32), (8192, 97, 64), (8224, 97, 64),
                                        (16384, 34, 64), (16384, 47, 61), (16416, 34, 64), (33, 640, 8), (4064, 200, 128)])
def test_products_of_few_tiles(n, fin, fout):
    """Tiles of 32 rows with the slabs of 16 k dealt out to 4 or 8 wavefronts: one and two tiles to a CU and the first product
    beyond, runs of slabs that are uneven or empty, a last slab of 1 to 15; x w and g w^T."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    print(f"few tiles: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fin)
    x, w, gout = (rng.standard_normal(s).astype(np.float32) for s in ((n, fin), (fin, fout), (n, fin)))
    y = torch.full((n + 1, fout), 7.0, device="cuda")
    pk.gnn_linear_fwd(dev(x), dev(w), y[:n])
    torch.cuda.synchronize()
    assert (y[n] == 7).all()        # nothing past the last row
    _assert_within_rounding("x w", y[:n].cpu().numpy(), x, w, 8)
    # gx = gout v^T of a layer fout -> fin
    g = pk.Graph(dev(np.arange(n + 1, dtype=np.int32)), dev(np.arange(n, dtype=np.int32)))
    v = np.ascontiguousarray(w.T)
    gx, gw = empty((n, fout)), empty((fout, fin))
    ws = torch.empty(max(pk.gnn_gcn_workspace_bytes(g, fout, fin), 16), dtype=torch.uint8, device="cuda")
    if fin % 4 == 0:
        pk.gnn_gcn_bwd(g, fout, fin, dev(np.zeros((n, fout), np.float32)), dev(v), dev(np.ones(n, np.float32)),
                       dev(np.ones(n, np.float32)), dev(gout), gx, gw, ws)
        torch.cuda.synchronize()
        _assert_within_rounding("g w^T", gx.cpu().numpy(), gout, w, 8)


@pytest.mark.parametrize("n,fin,fout", [(8104, 64, 60), (8104, 114, 60), (3000, 128, 64), (3000, 512, 32)])
def test_products_of_few_tiles_lose_to_neither_side(n, fin, fout):
    """The matrix core cuts off towards minus infinity.  What the even and the odd slabs lose, an even number of them here, cancels:
    the mean error of N entries is that of N independent ones, 0.01 of their rms or less at N > 9 10^4, and at most five times that."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, empty
    print(f"few tiles, mean error: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fin)
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((n, fin), (fin, fout)))
    y = empty((n, fout))
    pk.gnn_linear_fwd(dev(x), dev(w), y)
    err = y.cpu().numpy().astype(np.float64) - x.astype(np.float64) @ w.astype(np.float64)
    print(f"  mean {err.mean():.2e} rms {np.sqrt((err ** 2).mean()):.2e}", flush=True)
    assert abs(err.mean()) <= 0.05 * np.sqrt((err ** 2).mean())


def test_as_many_rows_as_vertices_can_have():
    """2^31 - 100 rows: their 128-row tiles have 2^32 threads, more than one launch may."""
    import paper_2110_09524_amd as pk
    import torch
    n = 2 ** 31 - 100
    print(f"linear: {n} rows", flush=True)
    x = torch.empty((n, 1), device="cuda")
    for r in range(0, n, 2 ** 27):
        x[r:r + 2 ** 27, 0] = torch.randn(min(2 ** 27, n - r), device="cuda")
    w = torch.tensor([[1.0, -0.3, 1e-3, 7.7]], device="cuda")
    y = torch.full((n, 4), float("nan"), device="cuda")
    pk.gnn_linear_fwd(x, w, y)
    for r in range(0, n, 2 ** 27):
        assert torch.equal(y[r:r + 2 ** 27], x[r:r + 2 ** 27] * w)


@pytest.mark.parametrize("fin", [1, 2])
@pytest.mark.parametrize("n,fout", [(70, 24), (300, 64), (40000, 132)])
def test_one_and_two_terms_are_rounded_like_fp32(n, fin, fout):
    """Products of so few terms are the chain of fused multiply-adds, bit for bit: x w alone, with the attention halves in
    its epilogue, and x^T g of two rows."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty, run_gat
    from test_gpu_edgeconv import fma_chain
    from test_gpu_gat import synth
    print(f"terms: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fin)
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((n, fin), (fin, fout)))
    y = empty((n, fout))
    pk.gnn_linear_fwd(dev(x), dev(w), y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), fma_chain(x, w))
    c = synth(rng, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), fin, fout // 4, 4)
    assert np.array_equal(run_gat(c)["z"].reshape(n, -1), fma_chain(c["x"], c["w"]))
    g = pk.Graph(dev(np.arange(fin + 1, dtype=np.int32)), dev(np.arange(fin, dtype=np.int32)))
    one, gw = dev(np.ones(fin, np.float32)), empty((n, fout))
    ws = torch.empty(max(pk.gnn_gcn_workspace_bytes(g, n, fout), 16), dtype=torch.uint8, device="cuda")
    pk.gnn_gcn_bwd(g, n, fout, dev(np.ascontiguousarray(x.T)), dev(np.zeros((n, fout), np.float32)), one, one, dev(w), None,
                   gw, ws)
    torch.cuda.synchronize()
    assert np.array_equal(gw.cpu().numpy(), fma_chain(x, w))


@pytest.mark.parametrize("n,fin,fout", [(1, 1, 1), (70, 2, 3), (300, 1, 33), (40000, 2, 131), (66000, 2, 127), (66001, 1, 130)])
def test_one_and_two_terms_of_any_width(n, fin, fout):
    """Widths that no vector of four columns divides, on every tile of the chain."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    from test_gpu_edgeconv import fma_chain
    print(f"terms: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fout)
    x, w = (rng.standard_normal(s).astype(np.float32) for s in ((n, fin), (fin, fout)))
    y = empty((n, fout))
    pk.gnn_linear_fwd(dev(x), dev(w), y)
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().numpy(), fma_chain(x, w))


@pytest.mark.parametrize("n,fin,fout", [(90, 8, 16), (100, 40, 20), (200, 33, 60), (300, 70, 132), (33000, 48, 68),
                                        (66000, 96, 132)])
def test_equal_rows_have_equal_products(n, fin, fout):
    """Rows repeated at even and odd places, in x w and in g w^T."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    print(f"equal rows: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fin)
    again = rng.integers(0, 37, size=n)
    x, gout = (np.ascontiguousarray(rng.standard_normal((37, s)).astype(np.float32)[again]) for s in (fin, fout))
    w = rng.standard_normal((fin, fout)).astype(np.float32)
    g = pk.Graph(dev(np.arange(n + 1, dtype=np.int32)), dev(np.arange(n, dtype=np.int32)))
    one, zs, out, gx, gw = dev(np.ones(n, np.float32)), empty((n, fout)), empty((n, fout)), empty((n, fin)), empty((fin, fout))
    ws = torch.empty(max(pk.gnn_gcn_workspace_bytes(g, fin, fout), 16), dtype=torch.uint8, device="cuda")
    pk.gnn_gcn_fwd(g, fin, fout, dev(x), dev(w), one, one, zs, out)
    pk.gnn_gcn_bwd(g, fin, fout, dev(x), dev(w), one, one, dev(gout), gx, gw, ws)
    torch.cuda.synchronize()
    first = np.unique(again, return_index=True)[1]
    for got in (zs.cpu().numpy(), gx.cpu().numpy()):
        assert np.array_equal(got, got[first][np.unique(again, return_inverse=True)[1]])


@pytest.mark.parametrize("n,fin,fout", [(100, 40, 20), (200, 33, 60), (300, 70, 130)])
def test_values_at_the_end_of_the_range(n, fin, fout):
    """Infinities, NaN, the largest floats and tiny ones come out as fp32 arithmetic gives them."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    rng = np.random.default_rng(fin)
    x = rng.standard_normal((n, fin)).astype(np.float32)
    w = rng.standard_normal((fin, fout)).astype(np.float32)
    w[1] = np.abs(w[1]) + 0.5
    x[3, 1], x[40, 1], x[41, 2], x[42, 1] = np.inf, -np.inf, np.nan, np.finfo(np.float32).max
    x[43] = 0
    x[43, 1] = np.finfo(np.float32).max      # its bf16 rounding is an infinity, the product may be finite
    w[1, 0] = 0.5
    x[44] *= np.float32(2.0 ** -100)
    y = empty((n, fout))
    pk.gnn_linear_fwd(dev(x), dev(w), y)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    with np.errstate(all="ignore"):
        ref = (x.astype(np.float64) @ w.astype(np.float64)).astype(np.float32)
    assert (got[3] == np.inf).all() and (got[40] == -np.inf).all() and np.isnan(got[41]).all()
    assert got[43, 0] == np.float32(np.finfo(np.float32).max / 2)
    assert np.array_equal(np.isfinite(got[42:44]), np.isfinite(ref[42:44]))
    rest = np.setdiff1d(np.arange(n), (3, 40, 41, 42, 43))
    _assert_within_rounding("the other rows", got[rest], x[rest], w)


@pytest.mark.parametrize("n,fin,fout", [(100, 40, 20), (200, 33, 60), (300, 70, 132), (33000, 48, 68), (66000, 96, 132),
                                        (100, 10, 8), (200, 16, 60), (33000, 29, 68), (900, 32, 132)])
def test_results_beside_infinities_and_nan(n, fin, fout):
    """What is not finite takes the fp32 matrix instruction; every other element keeps the bits it has without that."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    print(f"beside infinities: {n} x {fin} x {fout}", flush=True)
    rng = np.random.default_rng(n + fin)
    x, w, gout = (rng.standard_normal(s).astype(np.float32) for s in ((n, fin), (fin, fout), (n, fout)))
    g = pk.Graph(dev(np.arange(n + 1, dtype=np.int32)), dev(np.arange(n, dtype=np.int32)))
    one = dev(np.ones(n, np.float32))
    ws = torch.empty(max(pk.gnn_gcn_workspace_bytes(g, fin, fout), 16), dtype=torch.uint8, device="cuda")

    def products(x, w, gout):
        zs, out, gx, gw = empty((n, fout)), empty((n, fout)), empty((n, fin)), empty((fin, fout))
        pk.gnn_gcn_fwd(g, fin, fout, dev(x), dev(w), one, one, zs, out)
        pk.gnn_gcn_bwd(g, fin, fout, dev(x), dev(w), one, one, dev(gout), gx, gw, ws)
        torch.cuda.synchronize()
        return [t.cpu().numpy() for t in (zs, gx, gw)]

    zs, gx, gw = products(x, w, gout)
    x2, w2, g2 = x.copy(), w.copy(), gout.copy()
    x2[[3, 50], [1, 9]] = np.inf, np.nan     # rows 3, 50 of x w; columns 1, 9 of x, rows of x^T g
    w2[5, 7] = -np.inf                       # column 7 of x w, column 5 of g w^T
    g2[[11, 40], [2, 4]] = np.nan, np.inf    # rows 11, 40 of g w^T, columns 2, 4 of x^T g
    zs2, gx2, gw2 = products(x2, w2, g2)
    for got, ref, rows, cols in ((zs2, zs, (3, 50), (7,)), (gx2, gx, (11, 40), (5,)), (gw2, gw, (1, 9), (2, 4))):
        same = np.ones(ref.shape, dtype=bool)
        same[list(rows)], same[:, list(cols)] = False, False
        assert np.array_equal(got[same], ref[same])
        assert not np.isfinite(got[~same]).any()


@pytest.mark.parametrize("sx,sw", [(-115, 0), (0, -122), (60, -126), (-126, 70), (60, -140), (85, 20), (100, -60)])
@pytest.mark.parametrize("n,fin,fout", [(100, 40, 20), (300, 70, 130)])
def test_products_of_very_small_and_large_operands(n, fin, fout, sx, sw):
    """Operands near and below the smallest normal float keep their whole significand; sums above 2^96 take the
    fp32 matrix instruction.  The results are normal floats, so the bound is the one of ordinary values."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty
    print(f"scaled products: {n} x {fin} x {fout}, 2^{sx} and 2^{sw}", flush=True)
    rng = np.random.default_rng(fin)
    x = (rng.uniform(0.5, 2, (n, fin)) * 2.0 ** sx).astype(np.float32)
    w = (rng.uniform(0.5, 2, (fin, fout)) * 2.0 ** sw).astype(np.float32)
    y = empty((n, fout))
    pk.gnn_linear_fwd(dev(x), dev(w), y)
    torch.cuda.synchronize()
    _assert_within_rounding("y", y.cpu().numpy(), x, w)
