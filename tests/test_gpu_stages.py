"""Stage-by-stage parity of the HIP path (called through the C ABI) with the CPU oracle."""
import numpy as np
import pytest

from oracle import compgraph, gcn, sampling, solve
from synth import csr_from_undirected_edges, make_workload
from tests.gpu_common import make_context, say, to_u64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx_tiny():
    w = make_workload("c1")
    ctx = make_context(w)
    yield ctx, w
    ctx.close()


# ---------------------------------------------------------------- sampler: bit-exact
@pytest.mark.parametrize("n,ns,seed,tag", [
    (12, 4096, 1, 0),            # enumeration
    (2, 4, 1, 0), (3, 100, 7, 1), (24, 5000, 3, 9),
    (30, 2000, 5, 3), (64, 1000, 11, 4), (65, 1000, 12, 5), (130, 3001, 2 ** 40 + 17, 2 ** 31 + 5),
    (255, 777, 1, 1), (256, 778, 1, 1), (257, 4, 1, 1),
    (1000, 20000, 22668002, 7965), (5000, 3000, 9, 10), (40000, 600, 13, 77),
    (4096, 500, 21, 3), (4099, 700, 23, 4), (6241, 9000, 25, 5),   # the one-pass kernel (4,096 players and more)
    # a wave per pair below that: the most columns of each instance and one more, a workgroup that is not full
    (511, 600, 2, 1), (512, 602, 3, 1), (513, 604, 4, 1), (1024, 700, 5, 1), (1025, 702, 6, 1), (2048, 900, 7, 1), (2049, 902, 8, 1),
    (4095, 2002, 9, 1), (26, 6, 10, 1),
    (4095, 2002, 6609, 7), (4095, 2002, 6632, 7),   # several keys equal a threshold: the lowest columns go first
    (27, 524288, 10, 1), (27, 524290, 11, 1),   # as many workgroups as one direction of the grid takes, and one more
])
def test_sampler_bit_exact(ctx_tiny, n, ns, seed, tag):
    ctx, _ = ctx_tiny
    say(f"sampler n={n} n_samples={ns} seed={seed} tag={tag}")
    Z, w, sz = ctx.sample(n, ns, seed, tag)
    Zo, wo, szo = sampling.sample(n, ns, seed, tag)
    assert np.array_equal(to_u64(Z), Zo)
    assert np.array_equal(w.cpu().numpy().view(np.uint32), wo.view(np.uint32))
    assert np.array_equal(sz.cpu().numpy(), szo)


@pytest.mark.parametrize("window", [-1, 3])
def test_sampler_four_pass_route_gives_the_same_masks(ctx_tiny, window):
    from paper_2506_22668_amd import Tuning
    ctx, _ = ctx_tiny
    say(f"sampler forced fallback window={window}")
    ctx.set_tuning(Tuning(sampler_window=window))
    try:
        for n, ns in [(300, 2000), (5000, 600)]:
            Z, w, sz = ctx.sample(n, ns, 31, 8)
            Zo, wo, szo = sampling.sample(n, ns, 31, 8)
            assert np.array_equal(to_u64(Z), Zo)
            assert np.array_equal(sz.cpu().numpy(), szo)
    finally:
        ctx.set_tuning(None)


@pytest.mark.parametrize("n,ns", [(30, 25000), (200, 3000), (12, 1000), (9, 510), (1010, 20000), (333, 70000)])
def test_sampler_with_saturated_size_classes_bit_exact(ctx_tiny, n, ns):
    """ds_options.saturate: size classes allotted at least C(n, s) pairs are enumerated (subsets in lexicographic
    order, kernel weights); masks, weights and sizes against the oracle run with the same option."""
    from paper_2506_22668_amd import Options, DistShapError
    ctx, _ = ctx_tiny
    say(f"sampler saturate n={n} n_samples={ns}")
    Z, w, sz = ctx.sample(n, ns, 11, 5, Options(saturate=1))
    Zo, wo, szo = sampling.sample(n, ns, 11, 5, saturate=True)
    assert sampling.allocation(n, ns, saturate=True)["enum_upto"] >= 1
    assert np.array_equal(to_u64(Z), Zo)
    assert np.array_equal(w.cpu().numpy().view(np.uint32), wo.view(np.uint32))
    assert np.array_equal(sz.cpu().numpy(), szo)
    with pytest.raises(DistShapError):
        ctx.sample(n, ns, 11, 5, Options(saturate=1, weighting=1))


def test_sampler_pair_ranges_equal_the_full_run(ctx_tiny):
    ctx, _ = ctx_tiny
    n, ns, seed, tag = 333, 5000, 99, 3
    say("sampler ranges")
    Z, w, sz = ctx.sample(n, ns, seed, tag)
    for r0, r1 in [(0, 1), (0, 100), (100, 1777), (1777, 2500), (5, 5)]:
        Zp, wp, szp = ctx.sample_range(n, ns, seed, tag, r0, r1)
        assert torch.equal(Zp, Z[2 * r0:2 * r1])
        assert torch.equal(wp, w[2 * r0:2 * r1])
        assert torch.equal(szp, sz[2 * r0:2 * r1])


def test_sampler_takes_more_pairs_than_one_direction_of_a_grid(ctx_tiny):
    """2^26 pairs at four pairs to 256 threads are 2^32 threads."""
    ctx, _ = ctx_tiny
    n, ns, seed, tag = 28, 2 ** 27 + 6, 17, 3
    say(f"sampler n={n} n_samples={ns}")
    Z, w, sz = ctx.sample(n, ns, seed, tag)
    K = Z.shape[0] // 2
    assert K == 2 ** 26 + 3
    assert bool(((Z[0::2] ^ Z[1::2]) == 2 ** n - 1).all()) and bool((sz[0::2] + sz[1::2] == n).all())
    for lo, hi in [(0, 300), (K // 2 - 150, K // 2 + 150), (K - 300, K)]:
        Zr, wr, szr = ctx.sample_range(n, ns, seed, tag, lo, hi)
        assert torch.equal(Z[2 * lo:2 * hi], Zr) and torch.equal(w[2 * lo:2 * hi], wr) and torch.equal(sz[2 * lo:2 * hi], szr)


def test_sampler_rejects_bad_arguments(ctx_tiny):
    from paper_2506_22668_amd import DistShapError, DS_EINVAL
    ctx, _ = ctx_tiny
    say("sampler errors")
    with pytest.raises(DistShapError) as e:
        ctx.sample(100, 3, 1, 1)
    assert e.value.code == DS_EINVAL
    with pytest.raises(DistShapError) as e:
        ctx.sample(1, 10, 1, 1)
    assert e.value.code == DS_EINVAL
    with pytest.raises(DistShapError) as e:
        ctx.sample_range(100, 50, 1, 1, 3, 26)
    assert e.value.code == DS_EINVAL


# ---------------------------------------------------------------- extraction: exact
def _check_extraction(ctx, w, target, hops, directed):
    from paper_2506_22668_amd import Options
    cgo = compgraph.extract(w.row_ptr, w.col, target, hops, undirected=not directed)
    cg = ctx.extract(target, Options(hops=hops, directed=int(directed)))
    info = ctx.cgraph_info(cg)
    assert info.num_players == cgo["num_players"]
    assert info.num_nodes == cgo["num_nodes"]
    assert list(info.ball[:hops + 1]) == cgo["ball"]
    gid, hop = ctx.cgraph_nodes(cg)
    assert np.array_equal(gid.cpu().numpy(), cgo["node_gid"])
    assert np.array_equal(hop.cpu().numpy(), cgo["hop"])
    es, ed = ctx.cgraph_edges(cg)
    assert np.array_equal(es.cpu().numpy(), cgo["edge_src"])
    assert np.array_equal(ed.cpu().numpy(), cgo["edge_dst"])
    return cg, cgo


@pytest.mark.parametrize("key,hops,directed", [
    ("c1", 2, False), ("c1", 1, False), ("c1", 3, False), ("c1", 2, True),
    ("c2_small", 3, False), ("c2_small", 2, True), ("c2_small", 4, False),
    ("c3_small", 3, False), ("c4_small", 3, False), ("c4_small", 1, True),
])
def test_extraction_matches_oracle(key, hops, directed):
    w = make_workload(key)
    say(f"extract {key} hops={hops} directed={directed}")
    ctx = make_context(w)
    for target in w.targets[:2]:
        cg, _ = _check_extraction(ctx, w, target, hops, directed)
        ctx.cgraph_free(cg)
    ctx.close()


def test_extraction_isolated_and_pendant_targets():
    # node 3 is isolated (no players); node 2 hangs off node 1 (one player at 1 hop)
    rp, ci = csr_from_undirected_edges(5, [0, 1], [1, 2])
    from synth.workloads import Workload
    rng = np.random.default_rng(0)
    w = Workload("iso", 5, rp, ci, rng.standard_normal((5, 4), dtype=np.float32), (4, 3, 2),
                 [rng.standard_normal((4, 3)).astype(np.float32), rng.standard_normal((3, 2)).astype(np.float32)],
                 [3], 16, 1, "gram_chol")
    say("extract isolated")
    ctx = make_context(w)
    cg, cgo = _check_extraction(ctx, w, 3, 2, False)
    assert cgo["num_players"] == 0
    ctx.cgraph_free(cg)
    cg, cgo = _check_extraction(ctx, w, 2, 1, False)
    assert cgo["num_players"] == 1
    ctx.cgraph_free(cg)
    ctx.close()


# The one-workgroup extraction takes graphs of at most 65,536 nodes (a thread to 64 of them) whose hops have at most 1,024 rows and
# 16,384 entries; beyond that the general kernels follow. Sizes at both sides of each limit, single words, ragged last words,
# more than one round of its prefix sums.
@pytest.mark.parametrize("num_nodes,first,second,hops", [
    (2, 1, 0, 1), (64, 20, 2, 2), (65, 21, 2, 2), (700, 40, 15, 7), (4097, 1023, 2, 3), (4097, 1024, 2, 3), (4097, 1025, 2, 3),
    (40_000, 30, 540, 2), (40_000, 30, 550, 2), (65_536, 300, 50, 3), (65_537, 300, 50, 2),
])
@pytest.mark.parametrize("directed", [False, True])
def test_extraction_in_one_workgroup_and_past_its_limits(num_nodes, first, second, hops, directed):
    from synth.workloads import Workload
    say(f"extract {num_nodes} {first} {second} hops={hops} directed={directed}")
    rng = np.random.default_rng(num_nodes + first)
    ids = rng.permutation(num_nodes)
    kids = np.arange(1, 1 + first)
    leaves = np.arange(1 + first, min(1 + first * (1 + second), num_nodes))
    parent = np.concatenate([np.zeros(first, np.int64), 1 + (leaves - 1 - first) // max(second, 1)])
    child = np.concatenate([kids, leaves])
    more = rng.integers(0, num_nodes, (num_nodes // 8, 2))        # within the leaves and the rest of the graph
    more = more[(more.min(axis=1) > first) & (more[:, 0] != more[:, 1])]
    key = np.unique(np.minimum(np.r_[parent, more[:, 0]], np.r_[child, more[:, 1]]) * num_nodes +
                    np.maximum(np.r_[parent, more[:, 0]], np.r_[child, more[:, 1]]))
    rp, ci = csr_from_undirected_edges(num_nodes, ids[key // num_nodes], ids[key % num_nodes])
    w = Workload("ball", num_nodes, rp, ci, rng.standard_normal((num_nodes, 4), dtype=np.float32), (4, 3, 2),
                 [rng.standard_normal((4, 3)).astype(np.float32), rng.standard_normal((3, 2)).astype(np.float32)],
                 [int(ids[0])], 16, 1, "gram_chol")
    ctx = make_context(w)
    for target in (int(ids[0]), int(ids[-1])):
        cg, _ = _check_extraction(ctx, w, target, hops, directed)
        ctx.cgraph_free(cg)
    ctx.close()


# ... and where it hands over: before hop 1 (the target's entries at and one past the limit), before a middle hop because of the rows
# or of the entries so far, several hops to go, more members than a workgroup numbers, last words and blocks that are not whole
@pytest.mark.parametrize("num_nodes,first,second,hops", [
    (20_001, 16_384, 0, 1), (20_001, 16_385, 0, 1), (5000, 1500, 2, 5), (33_000, 40, 700, 4), (9000, 1024, 5, 2), (65_473, 1100, 40, 7),
])
@pytest.mark.parametrize("directed", [False, True])
def test_extraction_handed_over_by_the_one_workgroup(num_nodes, first, second, hops, directed):
    test_extraction_in_one_workgroup_and_past_its_limits(num_nodes, first, second, hops, directed)


def test_extraction_handed_over_is_no_slower_than_the_general_kernels():
    """1,200 rows in hop 2: past what one workgroup takes. The same graph with more than 65,536 nodes goes to the general
    kernels at once, which took 25 us less than the workgroup that gave up and they after it."""
    import time
    from paper_2506_22668_amd import Context, Options
    from synth import csr_from_undirected_edges
    kids, leaves = np.arange(1, 31), np.arange(31, 1231)
    more = np.arange(1231, 2431)
    src, dst = np.r_[np.zeros(30, np.int64), 1 + (leaves - 31) % 30, leaves], np.r_[kids, leaves, more]
    rng = np.random.default_rng(0)
    times = {}
    for N in (3000, 66_000):
        ctx = Context("cuda:0")
        rp, ci = csr_from_undirected_edges(N, src, dst)
        ctx.set_graph(rp, ci)
        ctx.set_features(rng.standard_normal((N, 4), dtype=np.float32))
        ctx.set_gcn([rng.standard_normal((4, 4)).astype(np.float32) for _ in range(3)])
        t = []
        for i in range(60):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            cg = ctx.extract(0, Options(hops=3))
            t.append(time.perf_counter() - t0)
            assert ctx.cgraph_info(cg).num_players == 2430
            ctx.cgraph_free(cg)
        times[N] = 1e6 * sorted(t[10:])[25]
        ctx.close()
    say(f"extract past one workgroup {times[3000]:.0f} us, general {times[66_000]:.0f} us")
    assert times[3000] <= 0.95 * times[66_000]


def test_malformed_graphs_are_rejected():
    from paper_2506_22668_amd import Context, DistShapError, DS_EINVAL, Options
    say("graph validation")
    ctx = Context("cuda:0")
    bad = [
        (np.array([0, 2, 1, 3]), np.array([1, 2, 0])),          # row_ptr not monotone
        (np.array([0, 2, 3, 3]), np.array([2, 1, 0])),          # row not ascending
        (np.array([0, 2, 3, 3]), np.array([1, 1, 0])),          # duplicate
        (np.array([0, 1, 2, 3]), np.array([1, 7, 0])),          # id out of range
        (np.array([1, 1, 2, 3]), np.array([1, 2, 0])),          # row_ptr[0] != 0
    ]
    for rp, ci in bad:
        with pytest.raises(DistShapError) as e:
            ctx.set_graph(rp, ci)
        assert e.value.code == DS_EINVAL
    # asymmetric CSR: fine for directed players, an error for undirected ones
    ctx.set_graph(np.array([0, 1, 1]), np.array([1]))
    ctx.set_features(np.zeros((2, 3), dtype=np.float32))
    ctx.set_gcn([np.zeros((3, 2), dtype=np.float32)])
    with pytest.raises(DistShapError) as e:
        ctx.extract(0, Options(hops=1))
    assert e.value.code == DS_EINVAL
    cg = ctx.extract(0, Options(hops=1, directed=1))
    assert ctx.cgraph_info(cg).num_players == 1
    ctx.cgraph_free(cg)
    with pytest.raises(DistShapError):
        ctx.extract(5, Options(hops=1))
    ctx.close()


# ---------------------------------------------------------------- shared first transform (MFMA)
@pytest.mark.parametrize("key,dtype,tol", [("c1", 0, 2e-6), ("c2_small", 0, 2e-6), ("c3_small", 0, 2e-6),
                                           ("c2", 0, 5e-6), ("c5_small", 1, 2e-2)])
def test_first_transform_matches_matmul(key, dtype, tol):
    w = make_workload(key)
    say(f"first transform {key} dtype={dtype}")
    ctx = make_context(w, transform_dtype=dtype)
    cg = ctx.extract(w.targets[0])
    gid, _ = ctx.cgraph_nodes(cg)
    P = ctx.cgraph_first_transform(cg).cpu().numpy().astype(np.float64)
    ref = w.features[gid.cpu().numpy()].astype(np.float64) @ w.weights[0].astype(np.float64)
    scale = np.abs(ref).max()
    assert np.abs(P - ref).max() <= tol * scale
    ctx.cgraph_free(cg)
    ctx.close()


# widths on both sides of the kernel's steps of 32 columns (two in flight) and of its tiles; rows that do not fill a tile. A sum of d0
# products in fp32 is within d0 * 2^-24 of its terms' magnitudes
@pytest.mark.parametrize("nodes,d0,d1", [(2, 1, 1), (31, 8, 33), (33, 31, 32), (64, 32, 31), (65, 33, 64), (90, 63, 65),
                                         (40, 64, 5), (40, 65, 97), (33, 97, 3), (129, 128, 33), (70, 130, 40)])
def test_first_transform_odd_widths(nodes, d0, d1, transform_dtype=0):
    from synth import csr_from_undirected_edges
    from paper_2506_22668_amd import Context, Options
    rng = np.random.default_rng(nodes + d0)
    rp, ci = csr_from_undirected_edges(nodes, [0] * (nodes - 1), list(range(1, nodes)))
    X = rng.standard_normal((nodes, d0), dtype=np.float32)
    W1 = rng.standard_normal((d0, d1), dtype=np.float32)
    say(f"first transform {nodes} x {d0} x {d1}")
    ctx = Context("cuda:0")
    ctx.set_graph(rp, ci)
    ctx.set_features(X)
    ctx.set_gcn([W1], transform_dtype=transform_dtype)
    cg = ctx.extract(0, Options(hops=1))
    P = ctx.cgraph_first_transform(cg).cpu().numpy().astype(np.float64)
    bound = d0 * 2.0 ** -24 * (np.abs(X).astype(np.float64) @ np.abs(W1).astype(np.float64)) + 1e-30
    assert (np.abs(P - X.astype(np.float64) @ W1.astype(np.float64)) <= bound).all()
    ctx.cgraph_free(cg)
    ctx.close()


# ... which the bfloat16 configuration does not round: the product is formed once per target and feeds every coalition
@pytest.mark.parametrize("nodes,d0,d1", [(31, 8, 33), (65, 33, 64), (40, 65, 97), (70, 130, 40)])
def test_first_transform_odd_widths_bf16(nodes, d0, d1):
    test_first_transform_odd_widths(nodes, d0, d1, transform_dtype=1)


# ---------------------------------------------------------------- masked inference
def _eval_case(w, hops, directed, score, biases, rows, rng, tol=1e-5, layers=None):
    from paper_2506_22668_amd import Options
    weights = w.weights if layers is None else w.weights[:layers]
    if layers is not None:
        w = type(w)(**{**w.__dict__, "weights": weights, "dims": w.dims[:layers + 1]})
    ctx = make_context(w, biases=biases)
    target = w.targets[0]
    cg = ctx.extract(target, Options(hops=hops, directed=int(directed)))
    cgo = compgraph.extract(w.row_ptr, w.col, target, hops, undirected=not directed)
    n = cgo["num_players"]
    f = gcn.ValueFunction(cgo, w.features, weights, biases, "logit" if score else "prob")
    bits = np.zeros((rows, n), dtype=bool)
    bits[1] = True
    for i in range(2, rows):
        bits[i] = rng.random(n) < rng.random() ** 2
    bits[rows - 1] = ~bits[rows - 2]
    Z = torch.from_numpy(sampling.pack_rows(bits).view(np.int64)).cuda()
    ref = f.batch(bits)
    scale = max(1.0, np.abs(ref).max())
    # every inference kernel on the same rows: the size-based choice, then each kernel forced (one workgroup per
    # coalition; one coalition per lane with the masks on chip; the mask-streaming kernel + layers on its output;
    # layer by layer over blocks of 64 coalitions from the transposed mask matrix)
    from paper_2506_22668_amd import Tuning
    for path in (0, 1, 2, 3, 4):
        ctx.set_tuning(Tuning(eval_path=path))
        y, pc = ctx.eval(cg, Z, score)
        assert pc == f.pred_class
        err = np.abs(y.cpu().numpy().astype(np.float64) - ref).max()
        assert err <= tol * scale, f"path {path}: max |y - oracle| = {err}"
    # rows as complementary pairs (only the even rows are read): masks 2r+1 = complement of 2r
    if rows % 2 == 0 and n > 0:
        pbits = bits.copy()
        pbits[1::2] = ~pbits[0::2]
        Zp = torch.from_numpy(sampling.pack_rows(pbits).view(np.int64)).cuda()
        refp = f.batch(pbits)
        for path in (0, 3, 4):
            ctx.set_tuning(Tuning(eval_path=path))
            y, pc = ctx.eval(cg, Zp, score, pairs=True)
            err = np.abs(y.cpu().numpy().astype(np.float64) - refp).max()
            assert err <= tol * max(1.0, np.abs(refp).max()), f"pairs, path {path}: max |y - oracle| = {err}"
    ctx.cgraph_free(cg)
    ctx.close()


@pytest.mark.parametrize("key,hops,directed,score,with_bias,layers", [
    ("c1", 2, False, 0, False, None), ("c1", 2, False, 1, True, None), ("c1", 3, False, 0, False, None),
    ("c1", 1, False, 0, False, None), ("c1", 2, True, 0, True, None), ("c1", 2, False, 0, False, 1),
    ("c2_small", 3, False, 0, False, None), ("c2_small", 3, False, 1, True, None),
    ("c2_small", 4, False, 0, False, None), ("c2_small", 2, False, 0, False, 2),
    ("c2_small", 3, True, 0, False, None),
    ("c3_small", 3, False, 0, False, None), ("c4_small", 3, False, 1, False, None),
])
def test_masked_inference_matches_oracle(key, hops, directed, score, with_bias, layers):
    w = make_workload(key)
    say(f"eval {key} hops={hops} directed={directed} score={score} bias={with_bias} layers={layers}")
    rng = np.random.default_rng(5)
    biases = None
    if with_bias:
        L = layers or w.num_layers
        biases = [0.1 * rng.standard_normal(w.dims[l + 1]).astype(np.float32) for l in range(L)]
    # 96 rows go through the one-workgroup-per-coalition kernel; 320 rows through the
    # one-coalition-per-lane kernel when the graph has at most 2048 players
    _eval_case(w, hops, directed, score, biases, 96, rng, layers=layers)
    _eval_case(w, hops, directed, score, biases, 320, rng, layers=layers)


# widths around the 32- and 64-feature tiles and 4-feature pieces of the kernels, odd ones among them; rows of every
# length class of the masks-on-chip kernel (a hub of 300 entries, which the waves share, 130, 70, 33, 17 and single
# entries), and a directed graph, whose first-layer rows are read through other players than their own entries
@pytest.mark.parametrize("dims,directed", [((6, 1, 3), False), ((6, 33, 5, 4), False), ((6, 64, 36, 3), False), ((6, 65, 63, 3), False),
                                           ((6, 131, 17, 2), False), ((6, 66, 5, 4), True)])
def test_masked_inference_widths_and_row_lengths(dims, directed):
    from synth import csr_from_undirected_edges
    from synth.workloads import Workload, glorot_uniform
    rng = np.random.default_rng(41)
    src, dst, at = [], [], 7
    for i, kids in enumerate((300, 130, 70, 33, 17, 1)):
        src += [0] + [1 + i] * kids
        dst += [1 + i] + list(range(at, at + kids))
        at += kids
    src += [1, 1, 2, 8, 9]                       # and a few edges within the shells
    dst += [2, 3, 4, 400, 410]
    rp, ci = csr_from_undirected_edges(at, src, dst)
    w = Workload("row_lengths", at, rp, ci, rng.standard_normal((at, dims[0]), dtype=np.float32), dims,
                 [glorot_uniform(rng, dims[i], dims[i + 1]) for i in range(len(dims) - 1)], [0], 0, 0, "gram_chol")
    biases = [0.1 * rng.standard_normal(d).astype(np.float32) for d in dims[1:]]
    say(f"masked inference dims={dims} directed={directed}")
    _eval_case(w, len(dims) - 1, directed, 1, biases, 322, rng)


# layer by layer a wave takes a row for four coalitions of a block of 64: row counts that end at every place in a group and
# at a whole block, pairs included, over a row of more than 64 entries
@pytest.mark.parametrize("rows,pairs", [(257, False), (258, True), (259, False), (260, True), (320, False), (384, True)])
def test_layer_by_layer_inference_at_the_ends_of_groups(rows, pairs):
    from paper_2506_22668_amd import Options, Tuning
    w = make_workload("c4b_small")
    rng = np.random.default_rng(rows)
    ctx = make_context(w)
    cg = ctx.extract(w.targets[0], Options(hops=3))
    cgo = compgraph.extract(w.row_ptr, w.col, w.targets[0], 3)
    bits = rng.random((rows, cgo["num_players"])) < rng.random((rows, 1))
    if pairs:
        bits[1::2] = ~bits[0::2]
    Z = torch.from_numpy(sampling.pack_rows(bits).view(np.int64)).cuda()
    say(f"layer by layer rows={rows} pairs={pairs}")
    ctx.set_tuning(Tuning(eval_path=4))
    y, pc = ctx.eval(cg, Z, 1, pairs=pairs)
    f = gcn.ValueFunction(cgo, w.features, w.weights, None, "logit")
    ref = f.batch(bits)
    # float32 sums of at most a few hundred terms, three layers: some 1e-6 of the largest logit
    assert pc == f.pred_class and np.abs(y.cpu().numpy() - ref).max() <= 1e-5 * max(1.0, np.abs(ref).max())
    ctx.cgraph_free(cg)
    ctx.close()


# the later layers' transform with the weights in registers (widths that are multiples of four, at most 64, from 16 rows on):
# whole and partial 32-feature tiles on either side, and the first widths outside
@pytest.mark.parametrize("dims", [(32, 64, 64, 5), (32, 4, 64, 5), (32, 64, 4, 5), (32, 36, 28, 5), (32, 60, 32, 5), (32, 32, 36, 5),
                                  (32, 68, 64, 5), (32, 64, 68, 5), (32, 62, 64, 5)])
@pytest.mark.parametrize("dtype", [0, 1])
def test_layer_by_layer_transform_widths(dims, dtype):
    from paper_2506_22668_amd import Options, Tuning
    from synth.workloads import glorot_uniform
    w = make_workload("c4b_small")
    rng = np.random.default_rng(sum(dims))
    w = type(w)(**{**w.__dict__, "weights": [glorot_uniform(rng, dims[i], dims[i + 1]) for i in range(3)], "dims": dims})
    biases = [0.1 * rng.standard_normal(d).astype(np.float32) for d in dims[1:]]
    ctx = make_context(w, biases=biases, transform_dtype=dtype)
    cg = ctx.extract(w.targets[0], Options(hops=3))
    cgo = compgraph.extract(w.row_ptr, w.col, w.targets[0], 3)
    assert cgo["ball"][1] >= 16
    bits = rng.random((300, cgo["num_players"])) < rng.random((300, 1))
    Z = torch.from_numpy(sampling.pack_rows(bits).view(np.int64)).cuda()
    say(f"layer by layer dims={dims} dtype={dtype}")
    ctx.set_tuning(Tuning(eval_path=4))
    y, pc = ctx.eval(cg, Z, 1)
    f = gcn.ValueFunction(cgo, w.features, w.weights, biases, "logit")
    full = f.logits(np.ones(cgo["num_players"], dtype=bool))
    oracle_class, f.pred_class = f.pred_class, pc   # the logits of the class that was reported
    ref = f.batch(bits)
    # float32: sums of at most a few hundred terms; bfloat16 operands: 2^-9 each, two transforms
    tol = (1e-2 if dtype else 1e-5) * max(1.0, np.abs(ref).max())
    assert np.abs(y.cpu().numpy() - ref).max() <= tol
    assert pc == oracle_class or full[oracle_class] - full[pc] <= 2 * tol   # (a tie within the precision)
    ctx.cgraph_free(cg)
    ctx.close()


# graphs past the limits of the smaller ones above: degrees outside of LDS (more than 640 nodes), with the local CSR in LDS
# and without, and more than 4,096 first-layer entries, where the waves of the paired external-input form add up a
# shared row in a single tile; an odd width and one above 64 of each, two layers (as many shared rows as children above
# 256) and three
@pytest.mark.parametrize("kids,dims", [((420, 130, 70, 33, 17, 1), (6, 33, 3)), ((420, 130, 70, 33, 17, 1), (6, 131, 5, 4)),
                                       ((1800, 1500, 1200, 900, 600, 300, 70, 33, 17, 1), (6, 33, 3)),
                                       ((1800, 1500, 1200, 900, 600, 300, 70, 33, 17, 1), (6, 131, 3)),
                                       ((1800, 1500, 1200, 900, 600, 300, 70, 33, 17, 1), (6, 66, 5, 4))])
def test_masked_inference_beyond_the_on_chip_limits(kids, dims):
    from synth import csr_from_undirected_edges
    from synth.workloads import Workload, glorot_uniform
    rng = np.random.default_rng(43)
    m = len(kids)
    src, dst, at = [], [], 1 + m
    for i, c in enumerate(kids):
        src += [0] + [1 + i] * c
        dst += [1 + i] + list(range(at, at + c))
        at += c
    src += [1, 1, 2, m + 3, m + 4]
    dst += [2, 3, 4, m + 500, m + 510]
    rp, ci = csr_from_undirected_edges(at, src, dst)
    w = Workload("limits", at, rp, ci, rng.standard_normal((at, dims[0]), dtype=np.float32), dims,
                 [glorot_uniform(rng, dims[i], dims[i + 1]) for i in range(len(dims) - 1)], [0], 0, 0, "gram_chol")
    lengths, entries = np.diff(rp), int(rp[1 + m])          # (rows 0 .. m are within one hop)
    assert at > 640 and int((lengths[:1 + m] > 256).sum()) == sum(c > 256 for c in kids)
    if sum(kids) > 4096:   # neither the CSR (12 bytes an entry pair, beside the masks) nor a tile per wave fits
        assert entries > 4096 and 8 * len(ci) + 512 * (len(ci) // 128) > 160 * 1024 - 16384
    biases = [0.1 * rng.standard_normal(d).astype(np.float32) for d in dims[1:]]
    say(f"masked inference nodes={at} first-layer entries={entries} dims={dims}")
    _eval_case(w, len(dims) - 1, False, 1, biases, 322, rng)


# masks on chip, degrees in LDS and the local CSR, of more entries than fit beside them, in memory: later layers whose rows end at every
# place in a step of four entries, slices of whole and partial widths
@pytest.mark.parametrize("nodes,edges,dims", [(600, 5000, (6, 33, 17, 3)), (640, 4500, (6, 64, 16, 12)), (630, 4700, (6, 5, 40, 30))])
def test_masked_inference_csr_outside_of_lds(nodes, edges, dims):
    from synth import csr_from_undirected_edges
    from synth.workloads import Workload, glorot_uniform
    rng = np.random.default_rng(edges)
    kids = np.arange(1, 8)
    u, v = rng.integers(1, nodes, edges), rng.integers(8, nodes, edges)
    rp, ci = csr_from_undirected_edges(nodes, np.r_[np.zeros(7, np.int64), u[u != v]], np.r_[kids, v[u != v]])
    n = len(ci) // 2
    assert 4096 < n < 8192 and 512 * ((n + 63) // 64) + 128 * nodes + 8 * len(ci) + 16384 > 160 * 1024
    w = Workload("csr in memory", nodes, rp, ci, rng.standard_normal((nodes, dims[0]), dtype=np.float32), dims,
                 [glorot_uniform(rng, dims[i], dims[i + 1]) for i in range(3)], [0], 0, 0, "gram_chol")
    biases = [0.1 * rng.standard_normal(d).astype(np.float32) for d in dims[1:]]
    say(f"masked inference CSR in memory nodes={nodes} players={n} dims={dims}")
    _eval_case(w, 3, False, 1, biases, 322, rng)


# ... with as many (row, 16 features) items as one look-ahead loop takes (64: four to a wave) and more, degrees in LDS and in memory
@pytest.mark.parametrize("nodes,edges", [(640, 5000), (900, 8200)])
@pytest.mark.parametrize("kids,dims", [(15, (6, 64, 33, 3)), (16, (6, 64, 16, 12)), (15, (6, 49, 100, 5)), (21, (6, 33, 65, 40))])
def test_masked_inference_csr_outside_of_lds_by_items(nodes, edges, kids, dims):
    from synth import csr_from_undirected_edges
    from synth.workloads import Workload, glorot_uniform
    rng = np.random.default_rng(edges + kids)
    near = np.arange(1, kids + 1)
    u, v = rng.integers(1, nodes, edges), rng.integers(kids + 1, nodes, edges)
    rp, ci = csr_from_undirected_edges(nodes, np.r_[np.zeros(kids, np.int64), u[u != v]], np.r_[near, v[u != v]])
    n = len(ci) // 2
    assert 4096 < n < 12_288 and 512 * ((n + 63) // 64) + (128 * nodes if nodes <= 640 else 0) + 8 * len(ci) + 16384 > 160 * 1024
    assert ((kids + 1) * ((dims[1] + 15) // 16) <= 64) == (kids == 15)
    w = Workload("csr in memory", nodes, rp, ci, rng.standard_normal((nodes, dims[0]), dtype=np.float32), dims,
                 [glorot_uniform(rng, dims[i], dims[i + 1]) for i in range(3)], [0], 0, 0, "gram_chol")
    biases = [0.1 * rng.standard_normal(d).astype(np.float32) for d in dims[1:]]
    say(f"masked inference CSR in memory nodes={nodes} players={n} items={(kids + 1) * ((dims[1] + 15) // 16)}")
    _eval_case(w, 3, False, 1, biases, 322, rng)


# a row's own term stays what it is where the row's features are infinite: the slots that fill up the last step of a row
# (steps of 2, 4 and 8 entries) must not multiply it by a zero. One layer, so that no other row reads the target's.
@pytest.mark.parametrize("leaves", [1, 2, 3, 4, 5, 6, 7, 8, 9, 21, 260, 301])
def test_infinite_features_of_the_target_stay_infinite(leaves):
    from paper_2506_22668_amd import Options, Tuning
    from synth import csr_from_undirected_edges
    from synth.workloads import Workload
    rng = np.random.default_rng(leaves)
    rp, ci = csr_from_undirected_edges(leaves + 1, [0] * leaves, list(range(1, leaves + 1)))
    X = rng.standard_normal((leaves + 1, 5), dtype=np.float32)
    X[0, 0] = np.inf
    W1 = rng.uniform(0.5, 1.0, (5, 3)).astype(np.float32) * np.array([-1, 1, -1], dtype=np.float32)
    w = Workload("inf", leaves + 1, rp, ci, X, (5, 3), [W1], [0], 0, 0, "gram_chol")
    ctx = make_context(w)
    cg = ctx.extract(0, Options(hops=1))
    bits = rng.random((258, leaves)) < rng.random((258, 1))
    bits[1::2] = ~bits[0::2]
    Z = torch.from_numpy(sampling.pack_rows(bits).view(np.int64)).cuda()
    for path, pairs in ((0, False), (1, False), (2, False), (3, False), (0, True), (3, True)):
        say(f"infinite features leaves={leaves} path={path} pairs={pairs}")
        ctx.set_tuning(Tuning(eval_path=path))
        y, pc = ctx.eval(cg, Z, 1, pairs=pairs)
        assert pc == 1 and bool((y == np.inf).all())
    ctx.cgraph_free(cg)
    ctx.close()


def test_masked_inference_all_enumerated_rows_tiny(ctx_tiny):
    ctx, w = ctx_tiny
    say("eval c1 all 4096 rows")
    cg = ctx.extract(0)
    Z, wt, sz = ctx.sample(12, 4096, w.seed, 0)
    y, pc = ctx.eval(cg, Z)
    cgo = compgraph.extract(w.row_ptr, w.col, 0, 2)
    f = gcn.ValueFunction(cgo, w.features, w.weights)
    ref = f.batch(sampling.unpack_rows(to_u64(Z), 12))
    assert np.abs(y.cpu().numpy() - ref).max() <= 1e-5
    ctx.cgraph_free(cg)


# ---------------------------------------------------------------- solvers
def _solve_inputs(n, ns, seed):
    rng = np.random.default_rng(seed)
    Z, w, sz = sampling.sample(n, ns, seed, 3)
    bits = sampling.unpack_rows(Z, n)
    a = rng.standard_normal(n) / np.sqrt(n)
    y = (0.2 + bits @ a + 0.1 * np.tanh(bits @ rng.standard_normal(n))).astype(np.float32)
    return Z, w, bits, y


# sizes around the factorisation's block edges too: one block exactly (64), a block and one column (65), whole blocks
# only (128, 192: the last fused step is followed by a full last block), a last block of one column (129)
@pytest.mark.parametrize("n,ns", [(12, 4096), (40, 2000), (63, 3000), (64, 3000), (65, 3000), (128, 4000), (129, 4000),
                                  (192, 4000), (200, 3000), (333, 6000), (1000, 20000),
                                  # back substitution, 256 unknowns per launch: one launch exactly, one column more, two
                                  (256, 4000), (257, 4000), (512, 6000)])
def test_gram_cholesky_matches_oracle_least_squares(ctx_tiny, n, ns):
    from paper_2506_22668_amd import Options, DS_SOLVER_GRAM_CHOL
    ctx, _ = ctx_tiny
    say(f"gram+chol n={n} n_samples={ns}")
    Z, w, bits, y = _solve_inputs(n, ns, 100 + n)
    ref = solve.solve_lstsq(bits, w, y)
    phi, rep, rc = ctx.solve(n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(),
                             torch.from_numpy(y).cuda(), Options(solver=DS_SOLVER_GRAM_CHOL))
    assert rep.solver_used == DS_SOLVER_GRAM_CHOL
    got = phi.cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    assert abs(got.sum() - (float(y[1]) - float(y[0]))) <= 1e-5 * max(1.0, abs(float(y[1]) - float(y[0])))


@pytest.mark.parametrize("n,ns,paired", [(12, 4096, 1), (40, 2000, 0), (40, 2000, 1), (333, 6000, 1),
                                         (1000, 20000, 1), (1000, 20000, 0), (3000, 1000, 1), (3000, 1000, 0),
                                         # >= 4096 players and paired: index lists + the matrix-core product of the dense rows
                                         (4100, 3000, 1), (6000, 14000, 1), (4097, 130, 1), (5000, 2000, 0),
                                         # exactly one 8192-column chunk / one column more; more than 8192 sparse
                                         # rows (several row blocks of tile entries)
                                         (8192, 3000, 1), (8193, 9000, 1), (5000, 40000, 1)])
def test_cgls_matches_oracle(ctx_tiny, n, ns, paired):
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    say(f"cgls n={n} n_samples={ns} paired={paired}")
    Z, w, bits, y = _solve_inputs(n, ns, 200 + n)
    ref, it_ref, _ = solve.solve_cgls(bits, w, y, tol=1e-12)
    phi, rep, rc = ctx.solve(n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(),
                             torch.from_numpy(y).cuda(), Options(solver=DS_SOLVER_CGLS, tol=1e-9, paired=paired))
    got = phi.cpu().numpy().astype(np.float64)
    assert rep.cgls_rel_residual <= 1e-9
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    if n <= 1000:   # well-determined: also the dense least-squares answer
        assert np.abs(got - solve.solve_lstsq(bits, w, y)).max() <= 1e-4 * np.abs(ref).max()


# the two-launch iteration of small games: whole words and one column more, the most players it takes (4,095), as many
# rows as its LDS copy holds (8,192 pairs, or rows) and one pair more (the general loop)
@pytest.mark.parametrize("n,ns,paired", [(3, 6, 1), (64, 128, 1), (65, 130, 0), (1025, 514, 1), (4095, 300, 1), (4095, 131, 0),
                                         (130, 16384, 1), (130, 16386, 1), (70, 8192, 0)])
def test_cgls_small_games_step_by_step(ctx_tiny, n, ns, paired):
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    Z, w, bits, y = _solve_inputs(n, ns, 300 + n)
    args = (n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y).cuda())
    for steps in (1, 6, 17):   # (the scalars come back every 16 steps)
        say(f"cgls n={n} n_samples={ns} paired={paired} steps={steps}")
        ref, it_ref, rel_ref = solve.solve_cgls(bits, w, y, tol=1e-9, max_iter=steps)
        phi, rep, _ = ctx.solve(*args, Options(solver=DS_SOLVER_CGLS, tol=1e-9, max_iter=steps, paired=paired),
                                allow_not_converged=True)
        assert abs(rep.cgls_iterations - it_ref) <= 1 and rep.cgls_iterations <= steps
        if it_ref == steps:
            assert abs(rep.cgls_rel_residual - rel_ref) <= 1e-6 * rel_ref + 1e-12
        # fp32 scores of an fp64 iteration: half an ulp each, and a step's rounding is far below it
        assert np.abs(phi.cpu().numpy() - ref).max() <= 3e-7 * np.abs(ref).max()


# The matrix-core product of the dense rows (all of them here, but the empty coalition): transposed rows of one word, of an odd and of
# an even number, padded to whole cache lines and not; fewer units of work than compute units, one more than a round, row
# groups that two or more workgroups share; a last chunk of one column.
@pytest.mark.parametrize("n,ns", [(4096, 40), (4097, 130), (5121, 2200), (4160, 15000), (9000, 20000), (30000, 3000)])
def test_cgls_dense_products_step_by_step(ctx_tiny, n, ns):
    from paper_2506_22668_amd import Options, Tuning, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    Z, w, bits, y = _solve_inputs(n, ns, 700 + n)
    args = (n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y).cuda())
    ctx.set_tuning(Tuning(cgls_dense_div=65536))
    for steps in (1, 3):
        say(f"cgls dense n={n} n_samples={ns} steps={steps}")
        ref, it_ref, rel_ref = solve.solve_cgls(bits, w, y, tol=1e-9, max_iter=steps)
        phi, rep, _ = ctx.solve(*args, Options(solver=DS_SOLVER_CGLS, tol=1e-9, max_iter=steps, paired=1), allow_not_converged=True)
        assert rep.cgls_iterations == it_ref
        assert abs(rep.cgls_rel_residual - rel_ref) <= 1e-6 * rel_ref + 1e-12
        # fp32 scores: half an ulp; vectors in fixed point at 2^-54 of their largest entry are far below it
        assert np.abs(phi.cpu().numpy() - ref).max() <= 3e-7 * np.abs(ref).max()
    ctx.set_tuning(Tuning())


@pytest.mark.parametrize("dense_div", [32, 1024, 65536])
def test_cgls_dense_row_threshold_leaves_the_solution_alone(ctx_tiny, dense_div):
    """Which pair rows are multiplied as bitmaps on the matrix cores and which as index lists is a tuning choice:
    nearly all dense (65536), the built-in split, nearly all sparse (32). 6,200 players: rows of 97 words, so the last
    1024-column chunk is short and the transposed copy has an odd number of words per row."""
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS
    from paper_2506_22668_amd.binding import Tuning
    ctx, _ = ctx_tiny
    n, ns = 6200, 8250
    say(f"cgls dense_div={dense_div}")
    Z, w, bits, y = _solve_inputs(n, ns, 77)
    ref, _, _ = solve.solve_cgls(bits, w, y, tol=1e-12)
    args = (n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y).cuda(),
            Options(solver=DS_SOLVER_CGLS, tol=1e-9, paired=1))
    base, rep0, _ = ctx.solve(*args)
    try:
        ctx.set_tuning(Tuning(cgls_dense_div=dense_div))
        phi, rep, _ = ctx.solve(*args)
    finally:
        ctx.set_tuning(None)
    assert rep.cgls_rel_residual <= 1e-9
    got = phi.cpu().numpy().astype(np.float64)
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
    assert np.abs(got - base.cpu().numpy()).max() <= 1e-6 * np.abs(ref).max()
    assert abs(rep.cgls_iterations - rep0.cgls_iterations) <= 2


# the sparse rows' tiles by the number of column chunks: one, two, four, 14, 22 and 37. At these numbers of rows a block holds 65,536
# entries (all but the last: 67,000 each in sixteen parts), so that blocks and groups are few
@pytest.mark.parametrize("n,ns", [(8192, 16000), (8193, 16000), (24_600, 16000), (110_000, 12000), (180_000, 8000), (300_007, 6000)])
def test_cgls_tile_groups_by_width(ctx_tiny, n, ns):
    from oracle import cfast
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    say(f"cgls tile groups n={n} n_samples={ns}")
    Z, w, sz = ctx.sample(n, ns, 11, 3)
    y = torch.from_numpy(np.random.default_rng(n).random(Z.shape[0], dtype=np.float32)).cuda()
    phi, rep, rc = ctx.solve(n, Z, w, y, Options(solver=DS_SOLVER_CGLS, paired=1, max_iter=4), allow_not_converged=True)
    assert rep.cgls_iterations == 4
    ref = cfast.cgls(n, to_u64(Z), w.cpu().numpy(), y.cpu().numpy(), tol=0.0, max_iter=4)[0]
    # both in fp64 or exact integers of 2^-47 and better, four steps; the scores come as float32
    assert np.abs(phi.cpu().numpy().astype(np.float64) - ref).max() <= 1e-6 * np.abs(ref).max()


# ... and where the blocks' entries follow from the number of groups, more than 65,536 of them: 62 groups of a block each (four chunks),
# 17 (14 chunks), ten of two blocks (22 chunks); the coarse split of 37 chunks, whose forward product takes a third chunk per
# workgroup instead of a second round
@pytest.mark.parametrize("n,ns,dense_div", [(24_600, 120_000, 32), (110_000, 12000, 32), (180_000, 8000, 32), (300_007, 8000, 64)])
def test_cgls_tile_groups_by_entries(ctx_tiny, n, ns, dense_div):
    from oracle import cfast
    from paper_2506_22668_amd import Options, Tuning, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    say(f"cgls tile groups n={n} n_samples={ns} dense_div={dense_div}")
    Z, w, sz = ctx.sample(n, ns, 11, 3)
    small = sz.view(-1, 2).min(dim=1).values
    assert small[small <= n // dense_div].sum().item() > 65536 * (62 if n == 24_600 else 16)   # (in so many parts)
    y = torch.from_numpy(np.random.default_rng(n).random(Z.shape[0], dtype=np.float32)).cuda()
    try:
        ctx.set_tuning(Tuning(cgls_dense_div=dense_div))
        phi, rep, rc = ctx.solve(n, Z, w, y, Options(solver=DS_SOLVER_CGLS, paired=1, max_iter=4), allow_not_converged=True)
    finally:
        ctx.set_tuning(None)
    assert rep.cgls_iterations == 4
    ref = cfast.cgls(n, to_u64(Z), w.cpu().numpy(), y.cpu().numpy(), tol=0.0, max_iter=4)[0]
    # both in fp64 or exact integers of 2^-47 and better, four steps; the scores come as float32
    assert np.abs(phi.cpu().numpy().astype(np.float64) - ref).max() <= 1e-6 * np.abs(ref).max()


def test_cgls_one_iteration_under_enumeration(ctx_tiny):
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    say("cgls enumeration one step")
    Z, w, bits, y = _solve_inputs(10, 1 << 10, 5)
    phi, rep, rc = ctx.solve(10, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(),
                             torch.from_numpy(y).cuda(), Options(solver=DS_SOLVER_CGLS, tol=1e-6, paired=1))
    assert rep.cgls_iterations == 1


def test_auto_falls_back_where_both_solvers_fill_the_workspace(ctx_tiny):
    """Many rows, none of which tells the last two players apart: the direct solver's buffers leave no room for those of the iterative one.
    A linear game, whose minimum-norm solution splits what the two have together."""
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS
    ctx, _ = ctx_tiny
    n, ns = 4090, 400000
    say(f"auto fallback n={n} n_samples={ns}")
    Z, w, _ = ctx.sample(n, ns, 7, 2)
    last = Z.shape[1] - 1
    two = (Z[:, last] >> ((n - 2) & 63)) & 1
    Z[:, last] = (Z[:, last] & ~(1 << ((n - 1) & 63))) | (two << ((n - 1) & 63))
    a = np.zeros(n, dtype=np.float32)
    who = np.array([0, 5, 77, 1800, n - 2, n - 1])
    a[who] = [3.0, -2.0, 0.5, 1.0, 1.5, 0.5]
    y = torch.zeros(Z.shape[0], dtype=torch.float32, device="cuda")
    for j in who:
        y += ((Z[:, j >> 6] >> (int(j) & 63)) & 1).float() * float(a[j])
    phi, rep, _ = ctx.solve(n, Z, w, y, Options(tol=1e-9))
    assert rep.solver_used == DS_SOLVER_CGLS
    a[n - 2:] = 1.0
    assert np.abs(phi.cpu().numpy() - a).max() <= 1e-5


def test_cgls_reports_non_convergence(ctx_tiny):
    from paper_2506_22668_amd import Options, DS_SOLVER_CGLS, DS_ENOTCONV
    ctx, _ = ctx_tiny
    say("cgls max_iter")
    Z, w, bits, y = _solve_inputs(200, 3000, 6)
    phi, rep, rc = ctx.solve(200, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(),
                             torch.from_numpy(y).cuda(), Options(solver=DS_SOLVER_CGLS, tol=1e-14, max_iter=2, paired=1),
                             allow_not_converged=True)
    assert rc == DS_ENOTCONV and rep.cgls_iterations == 2
    ref2 = solve.solve_cgls(bits, w, y, tol=1e-30, max_iter=2)[0]
    assert np.abs(phi.cpu().numpy() - ref2).max() <= 1e-4 * np.abs(ref2).max()


def test_gram_cholesky_mid_size_crosses_every_factorisation_regime(ctx_tiny):
    """2,700 players: the factorisation starts with super-panels of 256 columns (one wide trailing update each),
    continues with single blocks and ends with the steps whose update factorises the next diagonal block; the
    back substitution takes one launch per block."""
    from paper_2506_22668_amd import Options, DS_SOLVER_GRAM_CHOL
    ctx, _ = ctx_tiny
    n, ns = 2700, 9000
    say(f"gram+chol n={n} n_samples={ns}")
    Z, w, bits, y = _solve_inputs(n, ns, 77)
    ref = solve.solve_lstsq(bits, w, y)
    phi, rep, rc = ctx.solve(n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(),
                             torch.from_numpy(y).cuda(), Options(solver=DS_SOLVER_GRAM_CHOL, paired=1))
    got = phi.cpu().numpy().astype(np.float64)
    err = np.abs(got - ref).max()
    say(f"  err={err:.2e} max|phi|={np.abs(ref).max():.2e}")
    assert err <= 1e-4 * np.abs(ref).max()


# Which rows are sparse is decided 64 rows at a time: rows of more than 64 words (copied in two rounds), a last word of a
# few rows, a single word; and the sizes up to which the sparse rows' tiles ride in the column-wise kernel's launch. Games of
# at most 64 players: one pair of players per thread and one more, more rows than a workgroup's step holds; two groups of threads
# exactly (31), one and waves that are left over (32 to 43), a last workgroup of a single row (37, paired).
@pytest.mark.parametrize("n,ns", [(4161, 17030), (65, 512), (1408, 6000), (1409, 6000), (44, 400),
                                  (45, 400), (64, 80000), (3, 64), (31, 386), (32, 386), (36, 386), (37, 8066), (43, 386),
                                  (70, 1048640)])   # unpaired: one word of rows more than the grid takes in one direction
def test_gram_row_classes(ctx_tiny, n, ns):
    from paper_2506_22668_amd import Options, DS_SOLVER_GRAM_CHOL
    ctx, _ = ctx_tiny
    say(f"gram classes n={n}")
    Z, w, bits, y = _solve_inputs(n, ns, 40 + n)
    y, B, wt = y.astype(np.float64), bits[2:].astype(np.float64), w[2:].astype(np.float64)
    delta = y[1] - y[0]
    G, c = (B * wt[:, None]).T @ B, B.T @ (wt * (y[2:] - y[0] - delta / n * B.sum(1)))
    P = lambda a: a - a.mean(0)
    A = P(P(G).T)
    psi = np.linalg.solve(A + np.trace(A) / n / n, P(c))
    ref = psi - psi.mean() + delta / n
    for paired in (0, 1):
        got = ctx.solve(n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y.astype(np.float32)).cuda(),
                        Options(solver=DS_SOLVER_GRAM_CHOL, paired=paired))[0].cpu().numpy().astype(np.float64)
        # the column-wise sums are fp32 over 2,048 rows, 2^-24 of an entry, times the condition of the system (1e3 here)
        assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()


def test_gram_takes_more_rows_than_one_direction_of_a_grid(ctx_tiny):
    """2^28 rows at sixteen threads to a row are 2^32 threads. A linear game, whose coefficients are the answer."""
    from paper_2506_22668_amd import Options, DS_SOLVER_GRAM_CHOL
    ctx, _ = ctx_tiny
    n, ns = 65, 2 ** 28 + 64
    say(f"gram n={n} n_samples={ns}")
    Z, w, _ = ctx.sample(n, ns, 7, 2)
    a = np.random.default_rng(5).integers(-64, 65, n).astype(np.float32) / 128   # (every sum of them is exact in float32)
    y = torch.zeros(Z.shape[0], dtype=torch.float32, device="cuda")
    for j in range(n):
        for i in range(0, Z.shape[0], 1 << 26):
            y[i:i + (1 << 26)] += ((Z[i:i + (1 << 26), j >> 6] >> (j & 63)) & 1).float() * float(a[j])
    phi = ctx.solve(n, Z, w, y, Options(solver=DS_SOLVER_GRAM_CHOL))[0].cpu().numpy()
    assert np.abs(phi - a).max() <= 1e-6
    del Z, w, y
    torch.cuda.empty_cache()


# The 128 x 128 tiles of the wide update start at row 512: 2,304 leaves a last row of tiles that holds nothing but the
# right-hand side, 2,305 one of a single column, 2,431 a whole last tile less the right-hand side; 2,561 runs two
# super-panels, the second one's columns updated ahead of the rest.
@pytest.mark.parametrize("n", [2304, 2305, 2431, 2561])
def test_gram_cholesky_at_the_edges_of_the_wide_update(ctx_tiny, n):
    from paper_2506_22668_amd import Options, DS_SOLVER_GRAM_CHOL
    ctx, _ = ctx_tiny
    ns = 9000
    say(f"gram+chol wide n={n}")
    Z, w, bits, y = _solve_inputs(n, ns, 500 + n)
    ref = solve.solve_lstsq(bits, w, y)
    args = (n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y).cuda())
    got = [ctx.solve(*args, Options(solver=DS_SOLVER_GRAM_CHOL, paired=1))[0].cpu().numpy() for _ in range(3)]
    # a system of condition 1e3 at most (eigenvalues 5e-3 .. 5.3) solved in fp64: what is left is the rounding of the
    # scores to float32, 6e-8 of the largest
    assert np.abs(got[0].astype(np.float64) - ref).max() <= 1e-6 * np.abs(ref).max()
    for g in got[1:]:   # the two streams of the factorisation meet the same tiles in the same order every time
        assert np.array_equal(g, got[0])


def test_rank_deficient_gram_is_reported_and_auto_falls_back(ctx_tiny):
    from paper_2506_22668_amd import Options, DistShapError, DS_SOLVER_GRAM_CHOL, DS_SOLVER_CGLS, DS_ESINGULAR
    ctx, _ = ctx_tiny
    say("singular gram")
    Z, w, bits, y = _solve_inputs(300, 40, 8)      # 38 weighted rows for 300 players
    args = (300, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y).cuda())
    with pytest.raises(DistShapError) as e:
        ctx.solve(*args, Options(solver=DS_SOLVER_GRAM_CHOL))
    assert e.value.code == DS_ESINGULAR
    phi, rep, rc = ctx.solve(*args, Options(tol=1e-10, paired=1))
    assert rep.solver_used == DS_SOLVER_CGLS
    ref = solve.solve_lstsq(bits, w, y)
    assert np.abs(phi.cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("n,ns", [(150, 1000), (400, 3000)])
def test_gram_with_one_lost_direction_is_reported_and_auto_falls_back(ctx_tiny, n, ns):
    """Nullity one: two players that appear together in every sampled row (column n-1 is made a copy of column
    n-2). Exact arithmetic gives one zero pivot; in fp64 it comes out as round-off of either sign, which only a
    relative test catches. The direct solver must report the singular system, AUTO must return the minimum-norm
    solution (the oracle's projected least-squares solution)."""
    from paper_2506_22668_amd import Options, DistShapError, DS_SOLVER_GRAM_CHOL, DS_SOLVER_CGLS, DS_ESINGULAR
    ctx, _ = ctx_tiny
    say(f"gram nullity 1 n={n}")
    Z, w, bits, y = _solve_inputs(n, ns, 300 + n)
    bits = bits.copy()
    bits[2:, n - 1] = bits[2:, n - 2]
    Z = sampling.pack_rows(bits)
    args = (n, torch.from_numpy(Z.view(np.int64)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(y).cuda())
    with pytest.raises(DistShapError) as e:
        ctx.solve(*args, Options(solver=DS_SOLVER_GRAM_CHOL))
    assert e.value.code == DS_ESINGULAR
    phi, rep, rc = ctx.solve(*args, Options(tol=1e-11))
    assert rep.solver_used == DS_SOLVER_CGLS
    ref = solve.solve_lstsq(bits, w, y)
    got = phi.cpu().numpy().astype(np.float64)
    assert abs(ref[n - 1] - ref[n - 2]) <= 1e-9            # minimum norm splits the pair's share evenly
    assert np.abs(got - ref).max() <= 1e-4 * np.abs(ref).max()
