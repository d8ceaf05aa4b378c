"""MoNet layer with the projection of the degree pair fused into the gather kernels (gnn_monet_fwd/bwd):
HIP path against the fp64 oracle chain projection -> GMM layer -> projection's backward, and against the
two-call form of the library, which it must reproduce bit for bit wherever the summation order is the same."""
import numpy as np
import pytest

from helpers import sparse_graph_with_hubs, random_graph, tiny_graph
from oracle import gmm as om

pytestmark = pytest.mark.gpu


def synth(rng, indptr, indices, fin, fout, K, r):
    n = len(indptr) - 1
    return dict(n=n, fin=fin, fout=fout, k=K, r=r, indptr=indptr, indices=indices,
                x=rng.standard_normal((n, fin)).astype(np.float32),
                w_fc=(rng.standard_normal((fin, K * fout)) * 0.3).astype(np.float32),
                c=(1.0 / np.sqrt(np.maximum(np.diff(indptr), 1))).astype(np.float32),
                proj_w=rng.standard_normal((r, 2)).astype(np.float32),
                proj_b=(0.2 * rng.standard_normal(r)).astype(np.float32),
                mu=(rng.standard_normal((K, r)) * 0.3).astype(np.float32),
                inv_sigma=(0.5 + rng.random((K, r))).astype(np.float32),
                gout=rng.standard_normal((n, fout)).astype(np.float32))


def run(c, fused=True, want_gx=True):
    import torch
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, empty, workspace
    n, fin, fout, K, r, E = c["n"], c["fin"], c["fout"], c["k"], c["r"], len(c["indices"])
    g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
    x, w_fc, mu, isg, cc = dev(c["x"]), dev(c["w_fc"]), dev(c["mu"]), dev(c["inv_sigma"]), dev(c["c"])
    P, pb, gout = dev(c["proj_w"]), dev(c["proj_b"]), dev(c["gout"])
    hk, out = empty((n, K * fout)), empty((n, fout))
    gx = empty((n, fin)) if want_gx else None
    gw, gmu, gis, gP, gpb = empty((fin, K * fout)), empty((K, r)), empty((K, r)), empty((r, 2)), empty((r,))
    ws = workspace(max(pk.gnn_monet_workspace_bytes(g, fin, fout, K), pk.gnn_pseudo_proj_workspace_bytes(g)))
    ws.fill_(0xFF)
    if fused:
        pk.gnn_monet_fwd(g, fin, fout, K, r, x, w_fc, cc, P, pb, mu, isg, hk, out)
        pk.gnn_monet_bwd(g, fin, fout, K, r, x, w_fc, cc, P, pb, mu, isg, hk, gout, gx, gw, gmu, gis, gP, gpb, ws)
    else:
        pseudo, gps = empty((max(E, 1), r)), empty((max(E, 1), r))
        pk.gnn_pseudo_proj_fwd(g, r, cc, P, pb, pseudo)
        pk.gnn_gmmp_fwd(g, fin, fout, K, r, x, w_fc, pseudo, mu, isg, hk, out)
        pk.gnn_gmmp_bwd(g, fin, fout, K, r, x, w_fc, pseudo, mu, isg, hk, gout, gx, gw, gmu, gis, gps, ws)
        pk.gnn_pseudo_proj_bwd(g, r, cc, pseudo, gps, gP, gpb, ws)
    torch.cuda.synchronize()
    res = dict(hk=hk, out=out, gw_fc=gw, gmu=gmu, ginv_sigma=gis, gproj_w=gP, gproj_b=gpb)
    if want_gx:
        res["gx"] = gx
    g.close()
    return {k: v.cpu().numpy() for k, v in res.items()}


def oracle(c):
    ip, ix = c["indptr"], c["indices"]
    ps = om.pseudo_projection_forward(ip, ix, c["c"], c["proj_w"], c["proj_b"])
    args = (ip, ix, c["x"], c["w_fc"], ps, c["mu"], c["inv_sigma"])
    fwd = om.gmm_pseudo_forward(*args)
    bwd = om.gmm_pseudo_backward(*args, c["gout"], fwd)
    gP, gpb = om.pseudo_projection_backward(ip, ix, c["c"], c["proj_w"], c["proj_b"], bwd["gpseudo"])
    return fwd, bwd, gP, gpb


def check(c, **kw):
    from gpu_harness import assert_close
    fwd, bwd, gP, gpb = oracle(c)
    res = run(c, **kw)
    assert_close("hk", res["hk"], fwd["Hk"].reshape(c["n"], -1))
    assert_close("out", res["out"], fwd["out"])
    assert_close("gw_fc", res["gw_fc"], bwd["gw_fc"], reduce_scale=True)
    assert_close("gmu", res["gmu"], bwd["gmu"])
    assert_close("ginv_sigma", res["ginv_sigma"], bwd["ginv_sigma"])
    assert_close("gproj_w", res["gproj_w"], gP)
    assert_close("gproj_b", res["gproj_b"], gpb)
    if "gx" in res:
        assert_close("gx", res["gx"], bwd["gx"])
    return res


@pytest.mark.parametrize("fin,fout,K,r", [(16, 16, 2, 1), (16, 16, 3, 3), (9, 8, 4, 2), (5, 4, 1, 4), (12, 16, 4, 4),
                                          (7, 64, 1, 2), (6, 12, 3, 1)])
def test_shapes(fin, fout, K, r):
    print(f"monet: {fin}->{fout} K={K} r={r}", flush=True)
    rng = np.random.default_rng(100 + fin + fout + 10 * K + r)
    indptr, indices = random_graph(rng, 400, 5000, self_loops=True, duplicates=True)
    check(synth(rng, indptr, indices, fin, fout, K, r))


@pytest.mark.parametrize("K", [1, 2, 3, 4])
@pytest.mark.parametrize("r", [1, 2, 3, 4])
def test_every_number_of_kernels_and_dimensions(K, r):
    """The backward walk is compiled for each; groups of 8 and of 16 lanes, whole and partial, sources without out-edges,
    of as many as a chunk and one more, and hub sources whose row a workgroup shares."""
    print(f"monet: K={K} r={r}", flush=True)
    rng = np.random.default_rng(16 * K + r)
    n = 700
    edges = [(3, v) for v in range(n)] * 2 + [(u, int(v)) for u in range(10, n) for v in rng.integers(0, n, (0, 1, 8, 9, 16, 17)[u % 6])]
    indptr, indices = tiny_graph(n, edges)
    for fout in (4, 8 if K > 2 else 16, 64 // K // 4 * 4):
        check(synth(rng, indptr, indices, 5, fout, K, r))


@pytest.mark.parametrize("n", [32 * 256, 32 * 256 + 1, 16 * 512, 16 * 512 + 1])
def test_parameter_sums_at_the_edges_of_their_ranges(n):
    """32 or 16 rows per workgroup, 256 workgroups per range of partial sums: one range, two, one row in the last."""
    print(f"monet: {n} vertices", flush=True)
    rng = np.random.default_rng(n)
    indptr, indices = random_graph(rng, n, 2 * n, self_loops=True, duplicates=True)
    check(synth(rng, indptr, indices, 4, 4, 2, 1))
    check(synth(rng, indptr, indices, 4, 16, 3, 3))


@pytest.mark.parametrize("n,fin,fout,K", [(200, 5, 16, 2), (300, 33, 12, 3), (2300, 5, 4, 1), (2300, 33, 12, 3), (2300, 601, 32, 2)])
def test_parameter_sums_beside_the_parts_of_the_weight_gradient(n, fin, fout, K):
    """No parts; two, a sum to a thread; 17, a sum to eight threads, one block of sums or several; a sum to a thread again."""
    print(f"monet: {n} vertices {fin}->{fout} K={K}", flush=True)
    rng = np.random.default_rng(n + fin)
    indptr, indices = random_graph(rng, n, 2 * n, self_loops=True, duplicates=True)
    c = synth(rng, indptr, indices, fin, fout, K, 2)
    c["w_fc"] *= np.float32(fin ** -0.5)      # hk of the size of x
    check(c)


def test_the_papers_settings_on_a_power_law_graph_and_the_two_call_form():
    """k = 3, r = 3 and k = 2, r = 1 with 16 hidden features (Sec. 7.2, 7.3) on a graph with hub rows.  The
    fused kernels evaluate the same expressions in the same order as projection + general layer, so
    everything but the projection's own gradient (summed in another order there) is bit-equal."""
    from gpu_harness import assert_close
    from workloads import graphs
    print("monet: paper settings", flush=True)
    indptr, indices = graphs.chung_lu(5000, 100_000, 2.1, 99)
    rng = np.random.default_rng(5)
    for K, r in ((3, 3), (2, 1)):
        c = synth(rng, indptr, indices, 32, 16, K, r)
        a = check(c)
        b = run(c, fused=False)
        for k in ("hk", "out", "gx", "gw_fc", "gmu", "ginv_sigma"):
            assert np.array_equal(a[k], b[k]), k
        assert_close("gproj_w", a["gproj_w"], b["gproj_w"].astype(np.float64))
        assert_close("gproj_b", a["gproj_b"], b["gproj_b"].astype(np.float64))


def test_hub_empty_rows_no_edges_optional_gx_and_limits():
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, empty
    print("monet: hub / empty / optional / limits", flush=True)
    rng = np.random.default_rng(6)
    n = 500
    edges = [(u, 0) for u in range(n)] + [(0, v) for v in range(1, n, 2)]
    edges += [(int(rng.integers(0, n)), int(v)) for v in range(20, n) for _ in range(int(v) % 3)]
    indptr, indices = tiny_graph(n, edges)
    assert (np.diff(indptr) == 0).any()
    c = synth(rng, indptr, indices, 12, 16, 3, 2)
    res = check(c)
    assert (res["out"][np.diff(indptr) == 0] == 0).all()
    check(c, want_gx=False)
    res = check(synth(rng, np.zeros(34, dtype=np.int32), np.zeros(0, dtype=np.int32), 6, 16, 2, 2))
    assert not res["gproj_w"].any() and not res["gmu"].any()
    g = pk.Graph(dev(indptr), dev(indices))
    a = empty((4, 4))
    with pytest.raises(pk.GnnError) as e:                 # 3 x 32 projected floats: the two-call form's range
        pk.gnn_monet_fwd(g, 4, 32, 3, 2, a, a, a, a, a, a, a, a, a)
    assert e.value.status == 4 and "64" in str(e.value)
    with pytest.raises(pk.GnnError) as e:
        pk.gnn_monet_bwd(g, 4, 16, 2, 1, a, a, a, a, a, a, a, a, a, None, a, a, a, a, a, None)
    assert e.value.status == 3                           # no workspace
    assert pk.gnn_monet_workspace_bytes(g, 4, 16, 2) > 0
    g.close()


@pytest.mark.parametrize("fout,K,r,block_cols", [(16, 2, 1, 256), (16, 2, 1, 700), (32, 2, 2, 256), (4, 1, 1, 256), (64, 1, 3, 256),
                                                 (16, 4, 4, 500), (20, 3, 2, 256), (12, 3, 1, 1400), (8, 2, 1, 100)])
def test_all_column_blocks_in_one_launch(fout, K, r, block_cols):
    """The forward launch that keeps its sums in LDS: segments of no, few and many edges, rows cut into parts (one of 40 000
    edges into 128), rows without edges.  Its sums are grouped by block, so they are compared with the oracle and with the other kernels; what is not finite stays in the rows that gather it.  With coordinates per edge the
    same bits; a row out of the order of the blocks leaves it to the other kernels."""
    import paper_2110_09524_amd as pk
    from gpu_harness import assert_close
    print(f"monet: one launch, {fout} x {K}, r={r}, block_cols={block_cols}", flush=True)
    rng = np.random.default_rng(block_cols + fout)
    n = 1500
    deg = rng.integers(0, 40, n)
    deg[[5, 30, 700, 1499]] = 40000, 12, 3000, 300
    indptr = np.concatenate(([0], np.cumsum(deg))).astype(np.int32)
    indices = rng.integers(0, n, indptr[-1]).astype(np.int32)
    indices[indptr[20]:indptr[21]] = 77                     # a row that gathers one vertex only
    for v in range(n):
        row = indices[indptr[v]:indptr[v + 1]]
        row[row == 9] = 10                                   # vertex 9 is gathered by row 30 alone
        row.sort()
    indices[indptr[30]] = 9
    indices[indptr[30]:indptr[31]].sort()
    c = synth(rng, indptr, indices, 16, fout, K, r)
    pk.gnn_config_set("block_cols", block_cols)
    pk.gnn_config_set("resident_sums", 2)       # this launch on any graph with column blocks
    try:
        one, apart = run(c), run(c, fused=False)
        bad = dict(c, x=c["x"].copy())
        bad["x"][9] = np.inf
        beside = run(bad)
        turned = dict(c, indices=indices.copy())
        turned["indices"][indptr[5]:indptr[6]] = indices[indptr[5]:indptr[6]][::-1]
        disorder = run(turned)["out"]
        pk.gnn_config_set("resident_sums", 0)
        other, turned = run(c), run(turned)["out"]
    finally:
        pk.gnn_config_set("resident_sums", 1)
        pk.gnn_config_set("block_cols", 12288)
    ps = om.pseudo_projection_forward(indptr, indices, c["c"], c["proj_w"], c["proj_b"])
    ref = om.gmm_pseudo_forward(indptr, indices, c["x"], c["w_fc"], ps, c["mu"], c["inv_sigma"])["out"]
    # 40 000 terms of either sign round by the row's scale
    assert_close("out", one["out"], ref, row_scale=True)
    assert_close("out of the other kernel", other["out"], ref, row_scale=True)
    assert not np.array_equal(one["out"], other["out"])      # another kernel it was
    assert np.array_equal(apart["out"], one["out"]) and np.array_equal(disorder, turned)
    rest = np.arange(n) != 30
    assert np.array_equal(beside["out"][rest], one["out"][rest]) and not np.isfinite(beside["out"][30]).any()
    assert (one["out"][deg == 0] == 0).all()


@pytest.mark.parametrize("fout,K,r", [(16, 2, 1), (12, 3, 2), (16, 4, 3)])
def test_rows_of_tables_that_32_bits_do_not_reach(fout, K, r):
    """Row offsets of 64 bits, which tables of more than 2 GB take, give the same bits, with coordinates per edge as well."""
    import paper_2110_09524_amd as pk
    print(f"monet: wide offsets, {fout} x {K}, r={r}", flush=True)
    rng = np.random.default_rng(fout + K)
    n = 900
    edges = [(u, int(v)) for u in range(n) for v in rng.integers(0, n, (0, 1, 3, 4, 8, 9, 17, 40)[u % 8])] + [(7, v) for v in range(n)]
    indptr, indices = tiny_graph(n, edges)
    c = synth(rng, indptr, indices, 12, fout, K, r)
    narrow = [run(c, fused=fused) for fused in (True, False)]
    pk.gnn_config_set("wide_offsets", 1)
    try:
        wide = [run(c, fused=fused) for fused in (True, False)]
    finally:
        pk.gnn_config_set("wide_offsets", 0)
    for a, b in zip(narrow, wide):
        for name in a:
            assert np.array_equal(a[name], b[name]), name


@pytest.mark.parametrize("n,fout,K,r", [(98_305, 8, 2, 1), (41_000, 16, 4, 4)])
def test_few_rows_in_flight(n, fout, K, r):
    """Rows of 6 MB that are gathered evenly are asked for two at a time, longer ones of 10 MB one at a time, in the latter with four kernels of
    four coordinates by their addresses.  Rows of 0, 1, 2, 7, 8, 9 edges and more; the same bits with offsets of 64 bits and with
    coordinates per edge."""
    import paper_2110_09524_amd as pk
    from gpu_harness import assert_close
    print(f"monet: few rows in flight n={n} {fout} x {K}, r={r}", flush=True)
    rng = np.random.default_rng(n)
    deg = np.array([0, 1, 2, 7, 8, 9, 15, 33, 40, 55])[np.arange(n) % 10]
    indptr = np.concatenate(([0], np.cumsum(deg))).astype(np.int32)
    indices = rng.integers(0, n, indptr[-1]).astype(np.int32)
    c = synth(rng, indptr, indices, 6, fout, K, r)
    ps = om.pseudo_projection_forward(indptr, indices, c["c"], c["proj_w"], c["proj_b"])
    ref = om.gmm_pseudo_forward(indptr, indices, c["x"], c["w_fc"], ps, c["mu"], c["inv_sigma"])["out"]
    pk.gnn_config_set("blocked_min_edges", 16)
    try:
        out = run(c)["out"]
        assert_close("out", out, ref)
        assert np.array_equal(run(c, fused=False)["out"], out)
        pk.gnn_config_set("wide_offsets", 1)
        assert np.array_equal(run(c)["out"], out)
    finally:
        pk.gnn_config_set("wide_offsets", 0)
        pk.gnn_config_set("blocked_min_edges", 0)


@pytest.mark.parametrize("n,fout,K", [(95_000, 64, 1), (173_000, 32, 2)])
@pytest.mark.parametrize("hubs", [False, True])
def test_more_rows_than_the_workgroups_hold(n, fout, K, hubs):
    """The forward launch over all column blocks takes its rows in several batches: 256 workgroups hold up to 366 rows of 64 columns
    each, or 673 of 32, beside a block's scalars; rows whole and in parts.  The same bits with coordinates per edge."""
    import paper_2110_09524_amd as pk
    from gpu_harness import assert_close
    print(f"monet: rows in batches n={n} {fout} x {K} hubs={hubs}", flush=True)
    rng = np.random.default_rng(n + fout)
    indptr, indices = sparse_graph_with_hubs(rng, n, hubs)
    c = synth(rng, indptr, indices, 6, fout, K, 1)
    res = {}
    try:
        for resident in (2, 0):
            pk.gnn_config_set("resident_sums", resident)
            res[resident] = run(c)["out"], run(c, fused=False)["out"]
    finally:
        pk.gnn_config_set("resident_sums", 1)
    assert np.array_equal(*res[2]) and np.array_equal(*res[0])
    assert hubs is False or not np.array_equal(res[2][0], res[0][0])     # rows of several blocks: another kernel it was
    assert_close("out", res[2][0], res[0][0], row_scale=hubs)
