"""GAT layer: HIP path (through the C ABI) against the fp64 oracle, element by element."""
import numpy as np
import pytest

from oracle import gat as og
from helpers import PRODUCT_RTOL, graph_with_unheard_vertices, random_graph, relative_error, sparse_graph_with_hubs, tiny_graph
from workloads import make

pytestmark = pytest.mark.gpu


def oracle_all(c, backward=True):
    fwd = og.gat_forward(c["indptr"], c["indices"], c["x"], c["w"], c["a_l"], c["a_r"], c["slope"])
    bwd = None
    if backward:
        bwd = og.gat_backward(c["indptr"], c["indices"], c["x"], c["w"], c["a_l"], c["a_r"],
                              c["slope"], c["gout"], fwd)
    return fwd, bwd


def compare(c, res, fwd, bwd):
    from gpu_harness import assert_close, gat_kink_masks
    n, H, F = c["n"], c["heads"], c["f"]
    amb_vh, amb_vertex = gat_kink_masks(c["indptr"], fwd)
    keep_vh = ~amb_vh
    keep_hf = np.repeat(keep_vh, F, axis=1)
    Ht = fwd["Ht"].reshape(n, H * F)
    assert_close("z", res["z"], Ht)
    assert_close("el", res["el"], np.einsum("nhf,hf->nh", fwd["Ht"], c["a_l"].astype(np.float64)))
    assert_close("er", res["er"], np.einsum("nhf,hf->nh", fwd["Ht"], c["a_r"].astype(np.float64)))
    assert_close("m", res["m"], fwd["mx"])
    assert_close("d", res["d"], fwd["den"])
    assert_close("out", res["out"], fwd["out"])
    if "t" in res:
        # stashed destination-side sums: t = sum alpha_e g_e Ht[u], sg = sum alpha_e g_e,
        # g_e = LeakyReLU'(M0_e), written out from the oracle's materialised tensors
        from oracle.segments import segment_sum
        ag = fwd["M2"] * np.where(fwd["M0"] > 0, 1.0, c["slope"])
        sg_ref = segment_sum(c["indptr"], ag)
        t_ref = segment_sum(c["indptr"], ag[:, :, None] * fwd["Ht"][fwd["src"]]).reshape(n, H * F)
        assert_close("sg", np.where(keep_vh, res["sg"], sg_ref), sg_ref)
        assert_close("t", np.where(keep_hf, res["t"], t_ref), t_ref)
    if bwd is not None:
        assert_close("gx", np.where(amb_vertex[:, None], bwd["gx"], res["gx"]), bwd["gx"])
        assert_close("gw", res["gw"], bwd["gw"], reduce_scale=True)
        assert_close("ga_l", res["ga_l"], bwd["ga_l"], reduce_scale=True)
        assert_close("ga_r", res["ga_r"], bwd["ga_r"], reduce_scale=True)


def synth(rng, indptr, indices, fin, H, F, slope=0.2):
    n = len(indptr) - 1
    return dict(n=n, nnz=len(indices), fin=fin, heads=H, f=F, slope=slope, indptr=indptr,
                indices=indices,
                x=rng.standard_normal((n, fin)).astype(np.float32),
                # Glorot-scaled like the workloads: scores stay O(1)
                w=(rng.standard_normal((fin, H * F)) * np.sqrt(2.0 / (fin + H * F))).astype(np.float32),
                a_l=(rng.standard_normal((H, F)) * np.sqrt(2.0 / (F + 1))).astype(np.float32),
                a_r=(rng.standard_normal((H, F)) * np.sqrt(2.0 / (F + 1))).astype(np.float32),
                gout=rng.standard_normal((n, H * F)).astype(np.float32))


def test_c1_forward():
    from gpu_harness import run_gat
    print("gat: gat_c1 forward", flush=True)
    c = make("gat_c1")
    fwd, _ = oracle_all(c, backward=False)
    compare(c, run_gat(c, backward=False), fwd, None)


@pytest.mark.parametrize("name", ["gat_c1", "gat_c2", "gat_c4_mid"])
def test_workload_forward_backward(name):
    from gpu_harness import run_gat
    print("gat:", name, "fwd+bwd", flush=True)
    c = make(name)
    fwd, bwd = oracle_all(c)
    compare(c, run_gat(c), fwd, bwd)
    # without the stash the backward call recomputes the destination-side sums
    compare(c, run_gat(c, stash=False), fwd, bwd)


@pytest.mark.parametrize("fin,H,F", [(7, 1, 4), (33, 3, 8), (5, 2, 12), (19, 5, 4), (64, 2, 64),
                                     (12, 2, 64), (20, 3, 64), (31, 1, 128), (32, 4, 32), (40, 8, 64), (24, 3, 256), (130, 1, 16)])
def test_shapes_heads_and_widths(fin, H, F):
    from gpu_harness import run_gat
    print(f"gat: shape fin={fin} H={H} F={F}", flush=True)
    rng = np.random.default_rng(fin * 1000 + H * 10 + F)
    indptr, indices = random_graph(rng, 257, 3000, self_loops=True, duplicates=True)
    c = synth(rng, indptr, indices, fin, H, F)
    fwd, bwd = oracle_all(c)
    compare(c, run_gat(c), fwd, bwd)


@pytest.mark.parametrize("n", [31, 33, 161, 400])
def test_column_slices(n):
    """Four heads of 64 columns, a head to two XCDs: whole and partial workgroups of 16 rows, numbers of them that do not
    divide by the XCDs of a slice, shared rows, rows around one chunk of 16 edges and without any; each way to keep or
    recompute the forward pass."""
    from gpu_harness import run_gat
    print(f"gat: slices n={n}", flush=True)
    rng = np.random.default_rng(n)
    edges = [(int(u), 1) for u in rng.integers(0, n, 300)] + [(2, int(u)) for u in rng.integers(3, n, 300)]
    edges += [(int(u), v) for v in range(2, n) for u in rng.integers(0, n, (0, 1, 15, 16, 17, 33)[v % 6])]
    indptr, indices = tiny_graph(n, edges)
    c = synth(rng, indptr, indices, 11, 4, 64)
    fwd, bwd = oracle_all(c)
    for stash, alpha in ((True, False), (False, False), (True, True)):
        res = run_gat(c, stash=stash, alpha_stash=alpha)
        res.pop("alpha_t", None)
        compare(c, res, fwd, bwd)


@pytest.mark.parametrize("hot", [False, True])
@pytest.mark.parametrize("n", [32768, 32769])
def test_past_the_slices(n, hot):
    """33.6 MB of gathered rows, from which four heads of 64 columns are sliced where the gathers are skewed only; hot: eight
    sources have a twentieth of the edges, so that the forward side is sliced and the source side is not."""
    import paper_2110_09524_amd as pk
    from gpu_harness import run_gat
    print(f"gat: past the slices n={n} hot={hot}", flush=True)
    rng = np.random.default_rng(n)
    deg = np.arange(n) % 5
    indptr = np.concatenate(([0], np.cumsum(deg))).astype(np.int32)
    src = rng.integers(0, n, indptr[-1]).astype(np.int32)
    if hot:
        few = rng.random(src.size) < 0.05
        src[few] %= 8
    c = synth(rng, indptr, src, 11, 4, 64)
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("blocked_min_edges", 16)
    try:
        res = run_gat(c)
    finally:
        pk.gnn_config_set("blocked_min_edges", 0)
    compare(c, res, fwd, bwd)


def test_past_the_slices_of_neighbours():
    """As many rows, of sixteen edges from the neighbourhood each: sliced."""
    import paper_2110_09524_amd as pk
    from gpu_harness import run_gat
    n, deg = 32769, 16
    print("gat: past the slices, neighbours", flush=True)
    rng = np.random.default_rng(n)
    src = (np.repeat(np.arange(n), deg) + rng.integers(-1000, 1000, n * deg)) % n
    c = synth(rng, (np.arange(n + 1) * deg).astype(np.int32), src.astype(np.int32), 11, 4, 64)
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("blocked_min_edges", 16)
    try:
        res = run_gat(c)
    finally:
        pk.gnn_config_set("blocked_min_edges", 0)
    compare(c, res, fwd, bwd)


@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("n,heads,f", [(20490, 4, 32), (40970, 1, 44), (40970, 8, 8)])
def test_one_row_in_flight(n, heads, f, near):
    """10.5 MB of rows (lines of 128 bytes) gathered evenly from all over the graph, just enough for one row in flight per
    lane; near: from the neighbourhood, several in flight.  Rows are empty, shorter and longer than a chunk."""
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import run_gat
    print(f"gat: one row in flight n={n} {heads}x{f} near={near}", flush=True)
    rng = np.random.default_rng(n + heads)
    deg = np.array([0, 1, 3, 5, 16, 17, 32, 33, 64, 71])[np.arange(n) % 10]
    indptr = np.concatenate(([0], np.cumsum(deg))).astype(np.int32)
    if near:
        src = (np.repeat(np.arange(n), deg) + rng.integers(-100, 100, indptr[-1])) % n
    else:
        src = rng.integers(0, n, indptr[-1])
    c = synth(rng, indptr, src.astype(np.int32), 11, heads, f)
    # Some of the 10^7 scores lie on the LeakyReLU kink.  Masks cannot take them out of gw, which sums over all edges,
    # so these edges are taken out; the scores of the others stay.
    keep = (np.abs(oracle_all(c, backward=False)[0]["M0"]) >= 1e-5).all(axis=1)
    c.update(indptr=np.concatenate(([0], np.cumsum(keep)))[indptr].astype(np.int32), indices=c["indices"][keep], nnz=int(keep.sum()))
    g = pk.Graph(torch.from_numpy(c["indptr"]).cuda(), torch.from_numpy(c["indices"]).cuda())
    assert [pk.gnn_gat_rows_in_flight(g, heads, f, side) for side in (0, 1)] == ([4, 4] if near else [1, 1])
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("blocked_min_edges", 16)
    try:
        for alpha in (False, True):
            res = run_gat(c, alpha_stash=alpha)
            res.pop("alpha_t", None)
            compare(c, res, fwd, bwd)
    finally:
        pk.gnn_config_set("blocked_min_edges", 0)


def test_empty_rows_isolated_vertices_and_hub():
    from gpu_harness import run_gat
    print("gat: empty rows + hub", flush=True)
    rng = np.random.default_rng(5)
    n = 700
    # vertex 0 is a hub receiving from everyone (several chunks and a ragged tail),
    # vertices 1..9 have no in-edges, vertex 10 sends to nobody, the rest is sparse
    edges = [(u, 0) for u in range(n) if u != 10]
    edges += [(int(rng.integers(0, n)), int(v)) for v in range(11, n) for _ in range(int(v) % 4)]
    edges = [(u if u != 10 else 11, v) for (u, v) in edges]
    indptr, indices = tiny_graph(n, edges)
    c = synth(rng, indptr, indices, 20, 4, 16)
    fwd, bwd = oracle_all(c)
    res = run_gat(c)
    compare(c, res, fwd, bwd)
    assert (res["out"][1:10] == 0).all() and (res["m"][1:10] == 0).all() and (res["d"][1:10] == 1).all()


def test_single_vertex_self_loop_and_skipped_input_gradient():
    from gpu_harness import run_gat
    print("gat: single vertex", flush=True)
    rng = np.random.default_rng(6)
    c = synth(rng, np.array([0, 1], dtype=np.int32), np.array([0], dtype=np.int32), 3, 2, 4)
    fwd, bwd = oracle_all(c)
    res = run_gat(c, want_gx=False)
    res["gx"] = bwd["gx"]
    compare(c, res, fwd, bwd)


def test_graph_without_edges():
    from gpu_harness import run_gat
    print("gat: no edges", flush=True)
    rng = np.random.default_rng(61)
    n = 37
    c = synth(rng, np.zeros(n + 1, dtype=np.int32), np.zeros(0, dtype=np.int32), 5, 2, 8)
    fwd, bwd = oracle_all(c)
    res = run_gat(c)
    compare(c, res, fwd, bwd)
    assert (res["out"] == 0).all() and (res["m"] == 0).all() and (res["d"] == 1).all()
    for k in ("gx", "gw", "ga_l", "ga_r"):
        assert (res[k] == 0).all(), k


def test_results_are_bit_reproducible():
    from gpu_harness import run_gat
    print("gat: reproducibility", flush=True)
    c = make("gat_c2")
    a, b = run_gat(c), run_gat(c)
    for k in a:
        assert np.array_equal(a[k], b[k]), k


def test_bad_arguments_raise():
    import paper_2110_09524_amd as pk
    import torch
    from gpu_harness import dev, empty, workspace
    print("gat: error paths", flush=True)
    c = make("gat_c1")
    g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
    n = c["n"]
    x, w = dev(c["x"]), dev(c["w"])
    bufs = [empty((n, 16)) for _ in range(2)] + [empty((n, 1)) for _ in range(4)]
    z, out, el, er, m, d = bufs
    a6 = empty((1, 6))
    with pytest.raises(pk.GnnError) as e:        # f = 6 is not a multiple of 4
        pk.gnn_gat_fwd(g, 64, 1, 6, 0.2, x, w, a6, a6, z, el, er, m, d, out)
    assert e.value.status == 4
    a = dev(c["a_l"])
    with pytest.raises(pk.GnnError) as e:        # t without sg
        pk.gnn_gat_fwd(g, 64, 1, 16, 0.2, x, w, a, a, z, el, er, m, d, out, empty((n, 16)), None)
    assert e.value.status == 1
    pk.gnn_gat_fwd(g, 64, 1, 16, 0.2, x, w, a, a, z, el, er, m, d, out)
    need = pk.gnn_gat_workspace_bytes(g, 64, 1, 16)
    assert need > 0
    with pytest.raises(pk.GnnError) as e:        # workspace too small
        pk.gnn_gat_bwd(g, 64, 1, 16, 0.2, x, w, a, a, z, el, er, m, d, out, None, None,
                       dev(c["gout"]), None, empty((64, 16)), empty((1, 16)), empty((1, 16)),
                       workspace(need - 256))
    assert e.value.status == 3
    torch.cuda.synchronize()


@pytest.mark.parametrize("block_cols,H,F", [(256, 4, 64), (1024, 4, 64), (500, 1, 256), (300, 8, 16),
                                            (200, 2, 256), (128, 8, 128),
                                            # 512-byte rows: four slices of 128 bytes; narrower rows
                                            # take the single-launch kernels on such graphs, too
                                            (256, 1, 128), (300, 4, 32), (256, 2, 64), (500, 1, 64),
                                            # one head of at most 64 columns: a single slice of the
                                            # persistent kernels (merge = 2), rows shorter than the slice
                                            (300, 1, 44), (256, 1, 4), (200, 1, 60)])
@pytest.mark.parametrize("merge", [0, 1, 2])
def test_column_blocked_path(block_cols, H, F, merge):
    """The multi-launch, column-blocked kernels (used when the gathered matrix exceeds
    the L2 caches) on a graph small enough for the oracle, with small blocks forced: one launch
    per block (0), launches that walk several sparse blocks per row (1), and all blocks in one
    persistent launch that keeps the running sums in LDS (2; rows cut into 256-byte slices, the
    other shapes fall back to the launches)."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: blocked path block_cols={block_cols} H={H} F={F} merge={merge}", flush=True)
    if (H, F) == (4, 64):
        c = make("gat_c4_mid")
    else:
        rng = np.random.default_rng(block_cols + H + F)
        indptr, indices = random_graph(rng, 1500, 30000, self_loops=False, duplicates=True)
        c = synth(rng, indptr, indices, 24, H, F)
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("block_cols", block_cols)
    pk.gnn_config_set("merge_blocks", int(merge == 1))
    pk.gnn_config_set("resident_sums", int(merge == 2))
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        nb = g.blocked(0)[0]
        assert nb == -(-c["n"] // block_cols)
        launches = len(g.launch_groups(0, 2)) - 1
        print(f"  {nb} blocks in {launches} launches", flush=True)
        assert launches == nb if merge != 1 else 1 <= launches <= nb
        res = run_gat(c, graph=g)
        res_recompute = run_gat(c, graph=g, stash=False)   # blocked recompute of the dst side
    finally:
        pk.gnn_config_set("block_cols", 12288)
        pk.gnn_config_set("merge_blocks", 1)
        pk.gnn_config_set("resident_sums", 1)
    compare(c, res, fwd, bwd)
    compare(c, res_recompute, fwd, bwd)
    # same inputs through the single-launch kernels: both paths must agree with the oracle
    pk.gnn_config_set("force_simple_kernels", 1)
    try:
        res2 = run_gat(c, graph=g)
    finally:
        pk.gnn_config_set("force_simple_kernels", 0)
    compare(c, res2, fwd, bwd)
    assert np.array_equal(res["m"], res2["m"])      # the row maximum is exact on both paths


@pytest.mark.parametrize("H,F,block_cols", [(4, 64, 256), (1, 256, 500), (2, 256, 200), (1, 128, 256), (2, 64, 300)])
def test_resident_sums_repeat_the_launch_per_block_results_bit_for_bit(H, F, block_cols):
    """The persistent kernel adds a row's chunks in the order of the launch-per-block kernels, whoever
    draws the row and however the workgroups pace each other (also with the bounded wait cut to zero
    polls): every output equals the unmerged launches' bit for bit."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: resident sums H={H} F={F} block_cols={block_cols}", flush=True)
    rng = np.random.default_rng(7 * block_cols + H + F)
    n = 1800
    indptr, indices = random_graph(rng, n, 40000, self_loops=False, duplicates=True)
    c = synth(rng, indptr, indices, 16, H, F)
    pk.gnn_config_set("block_cols", block_cols)
    pk.gnn_config_set("merge_blocks", 0)
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        runs = {}
        for key, resident, spin in (("launches", 0, 4096), ("resident", 1, 4096), ("unpaced", 1, 0)):
            pk.gnn_config_set("resident_sums", resident)
            pk.gnn_config_set("resident_spin", spin)
            runs[key] = (run_gat(c, graph=g), run_gat(c, graph=g, stash=False))
    finally:
        pk.gnn_config_set("block_cols", 12288)
        pk.gnn_config_set("merge_blocks", 1)
        pk.gnn_config_set("resident_sums", 1)
        pk.gnn_config_set("resident_spin", 4096)
    g.close()
    for key in ("resident", "unpaced"):
        for a, b in zip(runs["launches"], runs[key]):
            for name in a:
                if isinstance(a[name], np.ndarray):
                    assert np.array_equal(a[name], b[name]), f"{key}: {name} differs from the launch-per-block result"


@pytest.mark.parametrize("H,F", [(4, 64), (8, 32), (1, 512), (2, 128), (1, 256)])
def test_blocked_path_with_the_score_table_in_lds(H, F):
    """A column block whose rows are long (>= 128 edges per row on average) is walked by the
    persistent variant that keeps the block's el table in LDS and draws rows from a counter;
    sparser blocks of the same graph take the plain variant.  Both against the oracle, and
    the two variants bit for bit against each other (they add the same terms in the same order)."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: blocked path, LDS score table H={H} F={F}", flush=True)
    rng = np.random.default_rng(1000 + H * F)
    n, block_cols = 700, 512
    edges = []
    for v in range(n):
        if v == 5:
            continue                                   # a row without in-edges
        k0 = n if v == 0 else 150 + int(rng.integers(0, 60))   # vertex 0: every source, the rest: a long row
        srcs = np.arange(n) if v == 0 else np.concatenate(
            [rng.choice(block_cols, size=k0, replace=False),
             block_cols + rng.choice(n - block_cols, size=20, replace=False)])
        edges += [(int(u), v) for u in srcs]
    indptr, indices = tiny_graph(n, edges)
    c = synth(rng, indptr, indices, 16, H, F)
    in_block0 = int((indices < block_cols).sum())
    assert in_block0 >= 128 * n and len(indices) - in_block0 < 128 * n   # one block of each kind
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("block_cols", block_cols)
    pk.gnn_config_set("resident_sums", 0)       # the launch-per-block kernels are the ones with the table
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        assert g.blocked(0)[0] == 2
        pk.gnn_prof_reset()
        pk.gnn_prof_enable(True)
        res = run_gat(c, graph=g)
        pk.gnn_prof_enable(False)
        assert "gat_blk_queue_reset" in pk.gnn_prof_report()       # the persistent variant was set up
        res_nostash = run_gat(c, graph=g, stash=False)
        pk.gnn_config_set("lds_scalar_table", 0)
        try:
            ref = run_gat(c, graph=g)
        finally:
            pk.gnn_config_set("lds_scalar_table", 1)
        g.close()
    finally:
        pk.gnn_config_set("block_cols", 12288)
        pk.gnn_config_set("resident_sums", 1)
    compare(c, res, fwd, bwd)
    compare(c, res_nostash, fwd, bwd)
    for k in res:
        assert np.array_equal(res[k], ref[k]), f"{k}: LDS-table and plain variants differ"


@pytest.mark.parametrize("blocked", [False, True, "launch per block"])
def test_large_score_range_is_stable(blocked):
    """Scores spanning hundreds of units: without the max subtraction exp() would overflow,
    with it most weights underflow to exactly 0 and the rest must still match (Sec. 7.2, the
    numerically stable softmax of App. A.1).  Forward values are held to the usual bar.  A raw
    score of magnitude |s| carries |s| 2^-24 of fp32 rounding, which exp() turns into the same
    relative error of every weight; at |s| ~ 150 that is ~1e-5 per edge, ten times the usual
    1e-6, so the gradients (sums of differences of such weights) get ten times the usual bar."""
    import paper_2110_09524_amd as pk
    from gpu_harness import ATOL, RTOL, assert_close, dev, gat_kink_masks, run_gat
    print(f"gat: large score range, blocked={blocked}", flush=True)
    rng = np.random.default_rng(77)
    indptr, indices = random_graph(rng, 600, 9000, self_loops=True, duplicates=False)
    c = synth(rng, indptr, indices, 12, 4, 32)
    c["a_l"] = (c["a_l"] * 60).astype(np.float32)
    c["a_r"] = (c["a_r"] * 60).astype(np.float32)
    fwd, bwd = oracle_all(c)
    spread = float(np.abs(fwd["M1"]).max())
    assert spread > 100.0                                       # the case is what it claims to be
    pk.gnn_config_set("block_cols", 128 if blocked else 12288)
    pk.gnn_config_set("resident_sums", int(blocked != "launch per block"))
    try:
        res = run_gat(c)
    finally:
        pk.gnn_config_set("block_cols", 12288)
        pk.gnn_config_set("resident_sums", 1)
    grads = {k: res.pop(k) for k in ("gx", "gw", "ga_l", "ga_r")}
    compare(c, res, fwd, None)
    assert np.isfinite(res["out"]).all() and (res["d"] >= 1.0 - 1e-6).all()
    _, amb_vertex = gat_kink_masks(c["indptr"], fwd)
    assert_close("gx", np.where(amb_vertex[:, None], bwd["gx"], grads["gx"]), bwd["gx"], rtol=10 * RTOL,
                 atol=10 * ATOL, row_scale=True)
    for k in ("gw", "ga_l", "ga_r"):
        assert_close(k, grads[k], bwd[k], rtol=10 * RTOL, atol=10 * ATOL, reduce_scale=True)


@pytest.mark.parametrize("fin,H,F", [(8, 64, 16), (8, 1, 1024), (1024, 2, 8), (4, 64, 4)])
def test_largest_supported_shapes(fin, H, F):
    """heads*f = 1024 (the widest row the kernels take), 64 heads, a wide input."""
    from gpu_harness import run_gat
    print(f"gat: largest shapes fin={fin} H={H} F={F}", flush=True)
    rng = np.random.default_rng(fin + 7 * H + 13 * F)
    indptr, indices = random_graph(rng, 200, 1500, self_loops=True, duplicates=True)
    c = synth(rng, indptr, indices, fin, H, F)
    fwd, bwd = oracle_all(c)
    compare(c, run_gat(c), fwd, bwd)


def test_many_vertices_few_edges_on_the_blocked_path():
    """More vertices than one column block holds, almost all (row, block) segments empty,
    rows without any edge in the first block, whole rows without edges."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print("gat: 70000 vertices, sparse", flush=True)
    rng = np.random.default_rng(4242)
    n = 70_000
    src = rng.integers(0, n, size=150_000)
    dst = rng.integers(0, n // 2, size=150_000)            # the upper half has no in-edges
    order = np.lexsort((src, dst))
    src, dst = src[order], dst[order]
    indptr = np.zeros(n + 1, dtype=np.int32)
    np.add.at(indptr, dst + 1, 1)
    indptr = np.cumsum(indptr).astype(np.int32)
    indices = src.astype(np.int32)
    c = synth(rng, indptr, indices, 6, 4, 32)
    fwd, bwd = oracle_all(c)
    g = pk.Graph(dev(indptr), dev(indices))
    assert g.blocked(0)[0] == -(-n // 12288)
    res = run_gat(c, graph=g)
    compare(c, res, fwd, bwd)
    assert (res["out"][n // 2:] == 0).all()
    compare(c, run_gat(c, graph=g, stash=False), fwd, bwd)
    g.close()


@pytest.mark.parametrize("stash", [True, False])
@pytest.mark.parametrize("name", ["gat_c2", "gat_c4_mid"])
def test_fusion_with_stashing_arm(name, stash):
    """The per-edge softmax values stored after the forward pass (CSC order, signed by the raw
    score) equal the oracle's materialised M2, and the backward pass that reads them back gives
    the oracle's gradients."""
    from gpu_harness import assert_close, run_gat
    print(f"gat: fusion with stashing {name} vertex-stash={stash}", flush=True)
    c = make(name)
    fwd, bwd = oracle_all(c)
    res = run_gat(c, stash=stash, alpha_stash=True)
    # CSC order: edges by (source, CSR position)
    order = np.lexsort((np.arange(c["nnz"]), c["indices"]))
    ref = (fwd["M2"] * np.where(fwd["M0"] > 0, 1.0, -1.0))[order]
    got = res.pop("alpha_t")[:c["nnz"]]
    near_kink = np.abs(fwd["M0"][order]) < 1e-5
    assert_close("alpha_t", np.where(near_kink, ref, got), ref)
    compare(c, res, fwd, bwd)


def test_fusion_with_stashing_arm_on_a_column_blocked_graph_and_bad_arguments():
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, empty, run_gat
    rng = np.random.default_rng(321)
    indptr, indices = random_graph(rng, 1500, 30000, self_loops=False, duplicates=True)
    c = synth(rng, indptr, indices, 24, 4, 64)
    fwd, bwd = oracle_all(c)
    from gpu_harness import assert_close
    n, nnz, H = c["n"], c["nnz"], c["heads"]
    pk.gnn_config_set("block_cols", 256)
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        assert pk.gnn_gat_stash_layout(g, 4, 64) == 1    # the stash is laid out for the column-blocked kernel
        res = run_gat(c, graph=g, alpha_stash=True)      # forward and stashed backward both column-blocked
    finally:
        pk.gnn_config_set("block_cols", 12288)
    # layout 1: [h][q], q = position in the source side's blocked list = the CSC entries (source,
    # CSR position) stable-sorted by (block of the destination, source)
    csc = np.lexsort((np.arange(nnz), c["indices"]))
    dst = np.repeat(np.arange(n), np.diff(c["indptr"]))
    key = (dst[csc] // 256).astype(np.int64) * n + c["indices"][csc]
    order = csc[np.argsort(key, kind="stable")]
    ref = (fwd["M2"] * np.where(fwd["M0"] > 0, 1.0, -1.0))[order].T
    got = res.pop("alpha_t").reshape(-1)[:H * nnz].reshape(H, nnz)
    near_kink = np.abs(fwd["M0"][order]).T < 1e-5
    assert_close("alpha_b", np.where(near_kink, ref, got), ref)
    compare(c, res, fwd, bwd)
    a = empty((4, 4))
    with pytest.raises(pk.GnnError) as e:
        pk.gnn_gat_bwd_stashed(g, 24, 4, 64, 0.2, a, a, a, a, a, a, a, a, a, a, None, None, None, a, None, a, a, a,
                               None)
    assert e.value.status == 1
    g.close()


def test_sparse_graph_spanning_blocks_takes_the_single_launch_kernels():
    """Default rule: column blocking is used from 16 edges per (row, block) on average."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    rng = np.random.default_rng(77)
    n = 1500
    indptr, indices = random_graph(rng, n, 30000, self_loops=False, duplicates=True)   # 20 edges per row
    c = synth(rng, indptr, indices, 16, 4, 64)

    def kernels_used(min_edges, block_cols):
        pk.gnn_config_set("blocked_min_edges", min_edges)
        pk.gnn_config_set("block_cols", block_cols)
        try:
            g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
            pk.gnn_prof_reset()
            pk.gnn_prof_enable(True)
            run_gat(c, graph=g)
            names = set(pk.gnn_prof_report())
            pk.gnn_prof_enable(False)
            g.close()
        finally:
            pk.gnn_config_set("block_cols", 12288)
            pk.gnn_config_set("blocked_min_edges", 0)
        return names
    assert "gat_head_major" not in kernels_used(16, 256)      # 6 blocks: 3.3 edges per (row, block)
    assert "gat_head_major" not in kernels_used(16, 1024)     # 2 blocks: 10 per (row, block)
    assert "gat_head_major" in kernels_used(8, 1024)          # the same graph with the bar at 8


@pytest.mark.parametrize("resident", [1, 0])
@pytest.mark.parametrize("H,F", [(4, 64), (2, 64), (2, 128), (1, 512), (8, 64), (1, 128)])
def test_fp16_gather_storage(H, F, resident):
    """gather_precision = 1: the column-blocked kernels (the persistent launch, or a launch per block with
    resident = 0) gather from an fp16 copy of z / gout and sum in fp32.  Every gathered element carries a relative rounding error of up to 2^-11; in the backward
    pass these errors enter dot products over f columns, so the worst entry of a gradient may be off by
    several 1e-3 of the tensor's rms.  The results are compared with the oracle at 1.5e-2 of the rms
    (worst entry) and 2e-3 (rms of the error), not at the 1e-4 contract; the fp32 path on the same
    inputs must be at least as close."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: fp16 gather storage H={H} F={F} resident={resident}", flush=True)
    rng = np.random.default_rng(4000 + H * F)
    indptr, indices = random_graph(rng, 1200, 30000, self_loops=True, duplicates=True)
    c = synth(rng, indptr, indices, 20, H, F)
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("block_cols", 256)
    pk.gnn_config_set("resident_sums", resident)
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        ref32 = run_gat(c, graph=g)
        pk.gnn_config_set("gather_precision", 1)
        try:
            res16 = run_gat(c, graph=g)
        finally:
            pk.gnn_config_set("gather_precision", 0)
        g.close()
    finally:
        pk.gnn_config_set("block_cols", 12288)
        pk.gnn_config_set("resident_sums", 1)
    compare(c, ref32, fwd, bwd)                       # the default path keeps the contract

    def rel(a, b):
        b = np.asarray(b, dtype=np.float64).reshape(np.shape(a))
        scale = max(np.sqrt(np.mean(b * b)), 1e-30)
        return float(np.abs(a - b).max() / scale), float(np.sqrt(np.mean((a - b) ** 2)) / scale)
    for key, ref in (("out", fwd["out"]), ("gx", bwd["gx"]), ("gw", bwd["gw"]), ("ga_l", bwd["ga_l"]),
                     ("ga_r", bwd["ga_r"])):
        (w16, r16), (w32, _) = rel(res16[key], ref), rel(ref32[key], ref)
        print(f"  {key}: fp16 worst {w16:.1e} rms {r16:.1e}; fp32 worst {w32:.1e}", flush=True)
        assert w16 < 1.5e-2 and r16 < 2e-3, f"{key}: fp16 gather error worst {w16:.2e} rms {r16:.2e}"
        assert w32 <= w16 + 1e-7 or w16 < 1e-6, f"{key}: fp32 {w32:.2e} vs fp16 {w16:.2e}"
    assert np.array_equal(res16["m"], ref32["m"]) and np.array_equal(res16["el"], ref32["el"])   # scores are fp32
    # the copy was used, by the forward pass and by the source-side backward
    assert not np.array_equal(res16["out"], ref32["out"])
    assert not np.array_equal(res16["gx"], ref32["gx"])


@pytest.mark.parametrize("H,F,n,block_cols,table", [(4, 64, 9000, 256, True), (4, 64, 9000, 5000, True),
                                                    (1, 128, 18000, 12288, True), (1, 128, 18000, 13000, False)])
def test_fp16_gather_of_two_float4_a_lane(H, F, n, block_cols, table):
    """Graphs without long rows: a lane takes 16 bytes of an fp16 row, and the forward pass reads the block's scores from LDS
    (a block of more than 12288 vertices: from memory).  Segments of no, few and more than 16 edges.  What differs from fp32
    is the rounding of the gathered rows, so the sums are compared with those of the rounded rows at the fp32 tolerance."""
    import paper_2110_09524_amd as pk
    from gpu_harness import assert_close, dev, empty, gat_kink_masks, run_gat, workspace
    from oracle.segments import segment_sum
    print(f"gat: fp16 rows in pairs H={H} F={F} n={n} block_cols={block_cols}", flush=True)
    rng = np.random.default_rng(n + block_cols)
    indptr, indices = random_graph(rng, n, 32 * n, self_loops=False, duplicates=True)
    c = synth(rng, indptr, indices, 16, H, F)
    pk.gnn_config_set("block_cols", block_cols)
    try:
        g = pk.Graph(dev(indptr), dev(indices))
        pk.gnn_config_set("gather_precision", 1)
        names = [pk.gnn_gat_blocked_kernel_name(g, H, F, mode) for mode in (0, 2, 3)]
        infer, train = run_gat(c, backward=False, graph=g, stash=False), run_gat(c, backward=False, graph=g)
        ws = workspace(pk.gnn_gat_workspace_bytes(g, 16, H, F))
        pk.gnn_config_set("gather_precision", 0)
        # the backward pass after a forward pass in fp32: only the rounding of gout is left
        x, w, a_l, a_r = (dev(c[k]) for k in ("x", "w", "a_l", "a_r"))
        z, out, t, sg = empty((n, H * F)), empty((n, H * F)), empty((n, H * F)), empty((n, H))
        el, er, m, d = (empty((n, H)) for _ in range(4))
        gx, gw, ga_l, ga_r = empty((n, 16)), empty((16, H * F)), empty((H, F)), empty((H, F))
        pk.gnn_gat_fwd(g, 16, H, F, c["slope"], x, w, a_l, a_r, z, el, er, m, d, out, t, sg, ws)
        pk.gnn_config_set("gather_precision", 1)
        pk.gnn_gat_bwd(g, 16, H, F, c["slope"], x, w, a_l, a_r, z, el, er, m, d, out, t, sg, dev(c["gout"]), gx, gw, ga_l,
                       ga_r, ws)
        gx = gx.cpu().numpy()
        g.close()
    finally:
        pk.gnn_config_set("gather_precision", 0)
        pk.gnn_config_set("block_cols", 12288)
    assert names[0].startswith(f"k_gat_res<16, 0, 2, {'true' if table else 'false'},"), names
    assert names[1].startswith("k_gat_res<16, 2, 2, false,") and names[2].startswith("k_gat_res<16, 3, 2, false,"), names
    c["gout"] = c["gout"].astype(np.float16).astype(np.float32)
    fwd, bwd = oracle_all(c)
    amb_vh, amb_vertex = gat_kink_masks(indptr, fwd)
    rows = train["z"].astype(np.float16).astype(np.float64).reshape(n, H, F)[fwd["src"]]
    ref = segment_sum(indptr, fwd["M2"][:, :, None] * rows).reshape(n, H * F)
    assert_close("out, with stash", train["out"], ref)
    assert_close("out", infer["out"], ref)
    ag = fwd["M2"] * np.where(fwd["M0"] > 0, 1.0, c["slope"])
    ref = segment_sum(indptr, ag[:, :, None] * rows).reshape(n, H * F)
    assert_close("t", np.where(np.repeat(~amb_vh, F, axis=1), train["t"], ref), ref)
    assert_close("gx", np.where(amb_vertex[:, None], bwd["gx"], gx), bwd["gx"])


def test_fp16_gather_storage_leaves_uncovered_shapes_in_fp32():
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    rng = np.random.default_rng(4100)
    indptr, indices = random_graph(rng, 900, 20000, self_loops=True, duplicates=True)
    c = synth(rng, indptr, indices, 12, 4, 32)          # 64-column slices would span two heads
    pk.gnn_config_set("block_cols", 256)
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        a = run_gat(c, graph=g)
        pk.gnn_config_set("gather_precision", 1)
        try:
            b = run_gat(c, graph=g)
        finally:
            pk.gnn_config_set("gather_precision", 0)
        g.close()
    finally:
        pk.gnn_config_set("block_cols", 12288)
    for k in a:
        assert np.array_equal(a[k], b[k]), k
    with pytest.raises(pk.GnnError):
        pk.gnn_config_set("gather_precision", 2)


@pytest.mark.parametrize("resident", [1, 0])
@pytest.mark.parametrize("H,F", [(4, 64), (1, 128)])
def test_column_blocked_path_with_64_bit_row_offsets(H, F, resident):
    """Gathered matrices of 4 GB and more are addressed with 64-bit offsets; the configuration key
    "wide_offsets" takes that path on a graph small enough for the oracle."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: blocked path, 64-bit row offsets H={H} F={F}", flush=True)
    rng = np.random.default_rng(77 + H)
    indptr, indices = random_graph(rng, 1500, 30000, self_loops=False, duplicates=True)
    c = synth(rng, indptr, indices, 24, H, F)
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("block_cols", 300)
    pk.gnn_config_set("wide_offsets", 1)
    pk.gnn_config_set("resident_sums", resident)
    try:
        g = pk.Graph(dev(c["indptr"]), dev(c["indices"]))
        res = run_gat(c, graph=g)
        g.close()
    finally:
        pk.gnn_config_set("block_cols", 12288)
        pk.gnn_config_set("wide_offsets", 0)
        pk.gnn_config_set("resident_sums", 1)
    compare(c, res, fwd, bwd)



def hub_graph(rng, n, pairs):
    """A random graph with duplicates, one vertex with an edge from and one with an edge to every other, and some without any."""
    indptr, indices = random_graph(rng, n, pairs, self_loops=False, duplicates=True)
    rows = [indices[indptr[v]:indptr[v + 1]] for v in range(n)]
    for v in range(n):
        rows[v] = np.append(rows[v], 11) if v % 50 else rows[v][:0]
    rows[7] = np.arange(n, dtype=np.int32)
    counts = np.array([len(r) for r in rows])
    return np.concatenate(([0], np.cumsum(counts))).astype(np.int32), np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("H,F,block_cols", [(2, 32, 256), (4, 16, 300), (8, 8, 1000), (4, 32, 300), (8, 16, 256), (16, 8, 1000),
                                            (8, 32, 300), (16, 32, 256)])
@pytest.mark.parametrize("hub", [False, True])
def test_heads_that_share_a_slice(H, F, block_cols, hub):
    """Two, four or eight heads in a 64-column slice of the persistent kernels: with stashed and recomputed sums of the
    destination side, stored softmax values and 64-bit row offsets; rows whole and in parts."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: shared slices H={H} F={F} block_cols={block_cols} hub={hub}", flush=True)
    rng = np.random.default_rng(block_cols + H + F)
    n = 1500
    indptr, indices = hub_graph(rng, n, 20000) if hub else random_graph(rng, n, 30000, self_loops=False, duplicates=True)
    c = synth(rng, indptr, indices, 24, H, F)
    fwd, bwd = oracle_all(c)
    pk.gnn_config_set("block_cols", block_cols)
    pk.gnn_config_set("resident_sums", 2)
    try:
        g = pk.Graph(dev(indptr), dev(indices))
        for mode in (0, 2, 3):
            name = pk.gnn_gat_blocked_kernel_name(g, H, F, mode)
            assert name == f"k_gat_res<16, {mode}, 1, false, true, false, true, {64 // F}, {'true' if hub else 'false'}>", name
        res, recompute = run_gat(c, graph=g), run_gat(c, graph=g, stash=False)
        stored = run_gat(c, graph=g, alpha_stash=True)
        stored.pop("alpha_t")
        pk.gnn_config_set("wide_offsets", 1)
        wide = run_gat(c, graph=g)
        g.close()
    finally:
        pk.gnn_config_set("wide_offsets", 0)
        pk.gnn_config_set("resident_sums", 1)
        pk.gnn_config_set("block_cols", 12288)
    compare(c, res, fwd, bwd)
    compare(c, recompute, fwd, bwd)
    compare(c, stored, fwd, bwd)
    for key in res:
        assert np.array_equal(res[key], wide[key]), key


@pytest.mark.parametrize("H,F,block_cols", [(1, 64, 256), (1, 44, 300), (1, 128, 1000), (2, 64, 300), (4, 64, 256)])
def test_long_rows_in_parts(H, F, block_cols):
    """Rows that the persistent kernels cut into parts, against the oracle, and from fp16 rows against the launches per block,
    which take a row in one piece."""
    import paper_2110_09524_amd as pk
    from gpu_harness import assert_close, dev, run_gat
    print(f"gat: long rows in parts H={H} F={F} block_cols={block_cols}", flush=True)
    rng = np.random.default_rng(block_cols + H + F)
    n = 1700
    indptr, indices = hub_graph(rng, n, 20000)
    c = synth(rng, indptr, indices, 24, H, F)
    fwd, bwd = oracle_all(c)
    half = {}
    pk.gnn_config_set("block_cols", block_cols)
    try:
        g = pk.Graph(dev(indptr), dev(indices))
        for mode in (0, 1, 2, 3):
            name = pk.gnn_gat_blocked_kernel_name(g, H, F, mode)
            assert name.startswith(f"k_gat_res<16, {mode}, ") and name.endswith(", 1, true>"), name
        res, recompute, infer = run_gat(c, graph=g), run_gat(c, graph=g, stash=False), run_gat(c, backward=False, graph=g, stash=False)
        if F % 64 == 0 and H * F > 64:
            pk.gnn_config_set("gather_precision", 1)
            for resident in (0, 1):
                pk.gnn_config_set("resident_sums", resident)
                half[resident] = (run_gat(c, backward=False, graph=g, stash=False), run_gat(c, graph=g))
        g.close()
    finally:
        pk.gnn_config_set("gather_precision", 0)
        pk.gnn_config_set("resident_sums", 1)
        pk.gnn_config_set("block_cols", 12288)
    compare(c, res, fwd, bwd)
    compare(c, recompute, fwd, bwd)
    compare(c, infer, fwd, None)
    if half:
        assert_close("out, forward only", half[1][0]["out"], half[0][0]["out"])
        for key in ("out", "t", "sg", "m", "d", "gx"):
            assert_close(key, half[1][1][key], half[0][1][key])


@pytest.mark.parametrize("n,fin,H,F", [
    (130, 7, 1, 8),        # no parts of gw
    (300, 33, 2, 16),      # both sums short: 5 and 2 parts
    (1100, 20, 1, 4),      # long sums of the attention gradients, few parts of gw
    (2500, 20, 3, 8),      # both long, ends inside a workgroup
    (2500, 520, 4, 16),    # gw a sum to a thread, the other eight threads to a sum
    (2500, 513, 4, 64),    # few tiles of gw, so fewer parts
])
def test_parameter_gradients_summed_in_one_launch(n, fin, H, F):
    from gpu_harness import run_gat
    rng = np.random.default_rng(n + fin)
    indptr, indices = random_graph(rng, n, 4 * n)
    c = synth(rng, indptr, indices, fin, H, F)
    fwd, bwd = oracle_all(c)
    compare(c, run_gat(c), fwd, bwd)


@pytest.mark.parametrize("H,F,block_cols", [(8, 8, 300), (4, 16, 256), (2, 32, 300), (8, 16, 256), (4, 32, 300), (1, 44, 256), (1, 64, 300),
                                            (1, 128, 256), (4, 64, 300), (2, 256, 256), (4, 256, 300)])
@pytest.mark.parametrize("resident", [2, 0])
def test_what_is_not_finite_stays_with_its_neighbours(H, F, block_cols, resident):
    """Non-finite rows of z (forward) and gout (backward) at the first vertex of every column block, which one row gathers in one
    block and none in the others: every other row keeps its bits.  fp32 and fp16 rows, 32-bit and 64-bit offsets."""
    import paper_2110_09524_amd as pk
    from gpu_harness import dev, run_gat
    print(f"gat: not finite H={H} F={F} block_cols={block_cols} resident={resident}", flush=True)
    rng = np.random.default_rng(block_cols + H + F)
    n = 1500
    indptr, indices = graph_with_unheard_vertices(rng, n, 30000, block_cols)
    c = synth(rng, indptr, indices, 24, H, F)
    first = np.arange(0, n, block_cols)
    bad_x, bad_g = dict(c, x=c["x"].copy()), dict(c, gout=c["gout"].copy())
    bad_x["x"][first[::2]], bad_x["x"][first[1::2]] = np.inf, np.nan
    bad_g["gout"][first[::2]], bad_g["gout"][first[1::2]] = np.nan, -np.inf
    out_rows, gx_rows = np.ones(n, bool), np.ones(n, bool)
    out_rows[[5, *first]] = False
    gx_rows[[3, *first]] = False
    pk.gnn_config_set("block_cols", block_cols)
    pk.gnn_config_set("resident_sums", resident)
    try:
        g = pk.Graph(dev(indptr), dev(indices))
        for half, wide in ((0, 0), (0, 1), (1, 0)):
            pk.gnn_config_set("gather_precision", half)
            pk.gnn_config_set("wide_offsets", wide)
            for kw in (dict(stash=True), dict(stash=False), dict(alpha_stash=True)):
                ok, x, go = (run_gat(d, graph=g, **kw) for d in (c, bad_x, bad_g))
                for key in ("out", "t", "sg", "m", "d"):
                    if key in ok:
                        assert np.array_equal(x[key][out_rows], ok[key][out_rows]), (half, wide, kw, key)
                assert not np.isfinite(x["out"][5]).any()
                assert np.array_equal(go["gx"][gx_rows], ok["gx"][gx_rows]), (half, wide, kw)
                assert not np.isfinite(go["gx"][3]).any()
        g.close()
    finally:
        pk.gnn_config_set("gather_precision", 0)
        pk.gnn_config_set("wide_offsets", 0)
        pk.gnn_config_set("resident_sums", 1)
        pk.gnn_config_set("block_cols", 12288)


FEW, HALVES, SPLIT = {"gemm_f32_mfma_attn"}, {"gemm_f32_mfma", "gat_attn_halves"}, {"gemm_f32_mfma_splitk", "gemm_sum_partials", "gat_attn_halves"}


@pytest.mark.parametrize("n,fin,H,F,route", [
    (70, 255, 1, 128, FEW), (70, 256, 1, 128, HALVES), (33, 602, 1, 72, HALVES), (129, 1792, 1, 128, HALVES), (31, 1793, 1, 128, SPLIT),
    (90, 1792, 8, 8, FEW), (90, 1793, 8, 8, SPLIT), (100, 20_001, 8, 8, SPLIT), (40, 3000, 2, 64, SPLIT),
    (7168, 1793, 1, 16, SPLIT), (7169, 1793, 1, 16, FEW), (8193, 1024, 1, 16, FEW), (8193, 1025, 1, 16, SPLIT),
    (3600, 4096, 2, 64, FEW), (3600, 4097, 2, 64, SPLIT)])
def test_routes_of_the_projection(n, fin, H, F, route):
    """Slabs dealt out to wavefronts, with the halves in the epilogue or (one head past 64 columns) in a launch of their own, or K split
    over workgroups: long sums of few rows go the last way.  Errors of the product as on every tile and layout."""
    import paper_2110_09524_amd as pk
    from gpu_harness import run_gat
    print(f"gat: projection {n} x {fin} x {H} x {F}", flush=True)
    rng = np.random.default_rng(n + fin)
    indptr, indices = random_graph(rng, n, 2 * n)
    c = synth(rng, indptr, indices, fin, H, F)
    pk.gnn_prof_reset()
    pk.gnn_prof_enable(True)
    try:
        res = run_gat(c, backward=False)
    finally:
        pk.gnn_prof_enable(False)
    names = {s for s in pk.gnn_prof_report() if s.startswith("gemm") or s == "gat_attn_halves"}
    assert names == route
    assert relative_error(res["z"], c["x"].astype(np.float64) @ c["w"].astype(np.float64)) <= PRODUCT_RTOL
    compare(c, res, *oracle_all(c, backward=False))


@pytest.mark.parametrize("H,F,n,half", [(4, 64, 33_500, 0), (4, 64, 31_000, 1), (16, 8, 41_000, 0)])
@pytest.mark.parametrize("hubs", [False, True])
def test_more_rows_than_the_workgroups_hold(H, F, n, half, hubs):
    """The persistent kernels take their rows in several batches: 256 workgroups, of which each has H F / 64 slices to serve, hold at most
    512 (row, slice) pairs (with scores in LDS 336, with heads that share a slice 314, with two sums 256 or 192).  Rows whole, as the
    launches per block give them bit for bit, and in parts; shared slices as the single-launch kernels give them."""
    import paper_2110_09524_amd as pk
    from gpu_harness import assert_close, dev, run_gat
    print(f"gat: rows in batches H={H} F={F} n={n} half={half} hubs={hubs}", flush=True)
    rng = np.random.default_rng(n + H)
    indptr, indices = sparse_graph_with_hubs(rng, n, hubs)
    c = synth(rng, indptr, indices, 16, H, F)
    res, infer = {}, {}
    pk.gnn_config_set("gather_precision", half)
    pk.gnn_config_set("merge_blocks", 0)        # each block by itself, like the persistent kernels
    try:
        g = pk.Graph(dev(indptr), dev(indices))
        for resident in (2, 0):
            pk.gnn_config_set("resident_sums", resident)
            if resident:
                names = [pk.gnn_gat_blocked_kernel_name(g, H, F, mode) for mode in (0, 2, 3)]
            res[resident], infer[resident] = run_gat(c, graph=g), run_gat(c, backward=False, graph=g, stash=False)
        g.close()
    finally:
        pk.gnn_config_set("merge_blocks", 1)
        pk.gnn_config_set("gather_precision", 0)
        pk.gnn_config_set("resident_sums", 1)
    assert all(name.startswith("k_gat_res<") and name.endswith(f"{str(hubs).lower()}>") for name in names), names
    for key in res[0]:
        if not hubs and F == 64 and not (half and key.startswith("g")):     # del of fp16 rows: other lanes add up other columns
            assert np.array_equal(res[2][key], res[0][key]), key
        else:   # vertex 11 sums over a third of the rows
            assert_close(key, res[2][key], res[0][key], reduce_scale=key in ("gw", "ga_l", "ga_r"), row_scale=hubs and key == "gx")
    assert_close("out, forward only", infer[2]["out"], infer[0]["out"])
    assert_close("out", infer[2]["out"], res[2]["out"])
