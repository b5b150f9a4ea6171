"""Layers of small batches that one workgroup takes in one launch (at most 1024 destinations and 2048 slots by the bound that
the targets give, fewer for a batch by itself with direct tables): bit-exact against the oracle at the edges of that rule, with both forms of the tables behind it, and the
same bits as the launches of the general path, which a batch takes when it is grouped with a large one.  Replays of
a captured call, whose seed, iteration and targets are read from the device, and groups of batches with several such layers."""
import pytest
import torch

import workloads
import sage_check as SC
from test_gpu_parity import _dev, _oracle_batch, assert_batch_equal

pytestmark = pytest.mark.gpu


# fanouts (top layer last), splits, sizes of the batches that follow one another in one context
CASES = {
    "one-layer": ([7], 3, [292, 293, 1, 257, 0]),
    "two": ([3, 5], 4, [33, 409, 410, 113, 114, 2, 64]),
    "three": ([4, 3, 2], 8, [42, 43, 227, 228, 1, 63, 65]),
    "wide-fan": ([20, 33], 2, [1, 3, 4, 62, 63]),
    "fan64": ([64, 31], 8, [1, 2, 66, 67]),
    "many-rows": ([3, 2], 4, [679, 680, 681, 1000, 1024, 1025]),
    "fan1": ([1, 1, 1], 1, [256, 257, 512, 513, 1024, 1025, 5]),
    "deep": ([2, 2, 2, 2, 2, 2, 2, 2], 5, [1, 3, 28, 600]),
}


@pytest.mark.parametrize("table_mode", [1, 2], ids=["hashed", "direct"])
@pytest.mark.parametrize("name", list(CASES))
def test_small_layers_bit_exact(name, table_mode):
    from paper_2303_13775_amd import Context
    dev = _dev()
    fan, S, sizes = CASES[name]
    gat = name in ("two", "deep")
    w = workloads.custom(4000, 30000, dims=[4] * (len(fan) + 1), fanouts=fan, batch=max(sizes), n_splits=S,
                         index64=name == "three", name=name)
    ctx = Context(w.indptr.to(dev), w.indices.to(dev), w.pmap.to(dev), S, fan, max(sizes), gat_index=gat, table_mode=table_mode)
    for it, n in enumerate(sizes):
        tg = w.targets(it)[:n]
        ctx.gsplit_sample_split(tg.to(dev), seed=77, it=it)
        ob = _oracle_batch(w, tg, 77, it)
        assert_batch_equal(ctx.fetch_batch(), ob, S, len(fan))
        for l in range(len(fan)):
            SC.assert_shuffle_index_equal(ctx, ob, l, has_rev=gat or l >= 1, has_eid=gat)
    ctx.close()


@pytest.mark.parametrize("table_mode, group, n, fan, taken", [
    (2, 1, 680, 2, True), (2, 1, 681, 2, False), (2, 1, 906, 1, True), (2, 1, 907, 1, False), (2, 1, 204, 10, True), (2, 1, 205, 10, False),
    (1, 1, 1024, 2, True), (1, 1, 205, 10, False), (2, 2, 1024, 2, True)])
def test_batches_by_themselves_with_direct_tables_take_fewer_destinations(table_mode, group, n, fan, taken):
    """1000 destinations x 2 are slower in one workgroup than in the general launches, unless batches share them or the tables
    are hashed."""
    from paper_2303_13775_amd import Context, gsplit_sample_split_multi
    dev = _dev()
    w = workloads.custom(4000, 30000, dims=[4, 4, 4], fanouts=[3, fan], batch=n, n_splits=4, name="route")
    graph = [t.to(dev) for t in (w.indptr, w.indices, w.pmap)]
    ctxs = [Context(*graph, 4, w.fanouts, n, table_mode=table_mode) for _ in range(group)]
    ctxs[0].gsplit_timing_enable(True)
    if group == 1:
        ctxs[0].gsplit_sample_split(w.targets(0).to(dev), 3, 0)
    else:
        gsplit_sample_split_multi(ctxs, [w.targets(b).to(dev) for b in range(group)], 3, list(range(group)))
    assert ("sample_small.l1" in ctxs[0].gsplit_timing_read()) == taken
    for b, c in enumerate(ctxs):
        assert_batch_equal(c.fetch_batch(), _oracle_batch(w, w.targets(b), 3, b), 4, 2)
        c.close()


@pytest.mark.parametrize("n", [40, 300])
@pytest.mark.parametrize("hub", [False, True], ids=["rmat", "star"])
def test_small_layers_give_the_bits_of_the_general_path(n, hub):
    """Edge positions, degrees and a training step; a star graph's hub has more than 256 entries in the reverse index."""
    from paper_2303_13775_amd import Context, SageParams, gsplit_sample_split_multi
    dev = _dev()
    w = workloads.custom(6000, 50000, dims=[8, 12, 12, 4], fanouts=[4, 3, 5], batch=1500, n_splits=4, name="bits")
    indptr, indices = w.indptr, w.indices
    if hub:         # every vertex aggregates from vertex 0 alone, vertex 0 from two others
        indptr = torch.arange(w.indptr.numel(), dtype=torch.int32) + 1
        indptr[0] = 0
        indices = torch.zeros(int(indptr[-1]), dtype=torch.int32)
        indices[0], indices[1] = 5, 9
    graph = [t.to(dev) for t in (indptr, indices, w.pmap)]
    params = SageParams(w.dims, [t.to(dev) for t in w.w_self], [t.to(dev) for t in w.w_neigh], [t.to(dev) for t in w.bias])
    feat, labels = w.feat.to(dev), w.labels.to(dev)
    targets, many = w.targets(0)[:n].to(dev), w.targets(1).to(dev)
    out = []
    for grouped in (False, True):
        ctx, big = [Context(*graph, w.n_splits, w.fanouts, w.batch, keep_edge_ids=True) for _ in range(2)]
        if grouped:
            gsplit_sample_split_multi([ctx, big], [targets, many], 3, [8, 9])
        else:
            ctx.gsplit_sample_split(targets, 3, 8)
        counts = [torch.zeros(m, dtype=torch.int32, device=dev) for m in (graph[0].numel() - 1, graph[1].numel())]
        ctx.gsplit_presample_accumulate(*counts)
        x0 = torch.empty((ctx.gsplit_max_rows(0), w.dims[0]), device=dev)
        ctx.gsplit_gather_features(feat, x0)
        logits = torch.empty((w.batch, w.dims[-1]), device=dev)
        grads = [[torch.empty_like(t, device=dev) for t in p] for p in (w.w_self, w.w_neigh, w.bias)]
        ctx.gsplit_sage_step(params, x0, labels, logits, *grads)
        got = ctx.fetch_batch()
        out.append([logits[:n], *counts] + [t for g in grads for t in g] + [t for f in got["local_front"] for t in f] +
                   [t for lay in got["layers"] for v in lay.values() for t in (v if isinstance(v, list) else [v])] +
                   [torch.tensor(got[k][l]) for k in ("n_mixed", "bucket") for l in range(3)])
        ctx.close()
        big.close()
    for a, b in zip(*out):
        assert torch.equal(a, b)


def test_small_batch_with_a_target_outside_the_graph():
    from paper_2303_13775_amd import Context, GsplitError
    dev = _dev()
    w = workloads.custom(500, 4000, dims=[4, 4, 4], fanouts=[3, 2], batch=50, n_splits=4, name="bad")
    ctx = Context(w.indptr.to(dev), w.indices.to(dev), w.pmap.to(dev), 4, w.fanouts, 50)
    for bad in (500, -1):
        tg = w.targets(0).to(dev).clone()
        tg[7] = bad
        ctx.gsplit_sample_split(tg, 1, 0)
        with pytest.raises(GsplitError):
            ctx.gsplit_batch_sizes()
        ctx.gsplit_sample_split(w.targets(0).to(dev), 1, 0)
        ctx.gsplit_batch_sizes()
    ctx.close()


@pytest.mark.parametrize("table_mode", [1, 2], ids=["hashed", "direct"])
@pytest.mark.parametrize("fan, n", [([15, 10, 5], 33), ([4, 3, 2], 42), ([7], 60)])
def test_replays_of_a_captured_small_batch(fan, n, table_mode):
    """All layers in the launch, or a layer of the general path behind it (whose hashed table the launch clears)."""
    from paper_2303_13775_amd import Context
    dev = _dev()
    w = workloads.custom(4000, 60000, dims=[4] * (len(fan) + 1), fanouts=fan, batch=300, n_splits=4, name="replay")
    ctx, other = [Context(w.indptr.to(dev), w.indices.to(dev), w.pmap.to(dev), 4, fan, 300, table_mode=table_mode) for _ in range(2)]
    targets, seed_iter = torch.zeros(n, dtype=torch.int32, device=dev), torch.zeros(2, dtype=torch.int64, device=dev)

    def set_up(seed, it):
        tg = w.targets(it)[it:it + n]
        targets.copy_(tg.to(dev))
        seed_iter.copy_(torch.tensor([seed, it]))
        return tg

    def check(c, tg, seed, it):
        ob = _oracle_batch(w, tg, seed, it)
        assert_batch_equal(c.fetch_batch(), ob, 4, len(fan))
        for l in range(len(fan)):
            SC.assert_shuffle_index_equal(c, ob, l, has_rev=l >= 1)

    ctx.gsplit_sample_split(w.targets(8).to(dev), 5, 8)     # a batch of the general path, then a small one
    tg = set_up(21, 2)
    ctx.gsplit_sample_split_dev(targets, seed_iter)
    check(ctx, tg, 21, 2)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        ctx.gsplit_sample_split_dev(targets, seed_iter)
    for seed, it in ((21, 2), (22, 2), (1 << 40, 7), (22, 0), (22, 0)):
        tg = set_up(seed, it)
        torch.cuda.synchronize()
        graph.replay()
        other.gsplit_sample_split(tg.to(dev), seed, it)     # eager work between the replays
        check(ctx, tg, seed, it)
        check(other, tg, seed, it)
    ctx.close()
    other.close()


@pytest.mark.parametrize("table_mode", [1, 2], ids=["hashed", "direct"])
@pytest.mark.parametrize("fan, sizes", [([4, 3, 2], [42, 1, 33]), ([3, 4, 3, 2], [33, 20, 0, 5, 31]),
                                        ([2, 2, 2], [5, 33, 0, 1, 17, 113, 64, 30])])
def test_groups_of_small_batches_bit_exact(fan, sizes, table_mode):
    """Several layers of every batch in the launch (up to sixteen over the batches)."""
    from paper_2303_13775_amd import Context, gsplit_sample_split_multi
    dev = _dev()
    w = workloads.custom(4000, 30000, dims=[4] * (len(fan) + 1), fanouts=fan, batch=120, n_splits=5, name="groups")
    graph = [t.to(dev) for t in (w.indptr, w.indices, w.pmap)]
    ctxs = [Context(*graph, 5, fan, 120, gat_index=len(sizes) == 5, table_mode=table_mode) for _ in sizes]
    for rnd in range(2):
        its = [10 * rnd + b for b in range(len(sizes))]
        tgs = [w.targets(it)[:sizes[(b + rnd) % len(sizes)]] for b, it in enumerate(its)]
        gsplit_sample_split_multi(ctxs, [t.to(dev) for t in tgs], 31, its)
        for c, tg, it in zip(ctxs, tgs, its):
            ob = _oracle_batch(w, tg, 31, it)
            assert_batch_equal(c.fetch_batch(), ob, 5, len(fan))
            for l in range(len(fan)):
                SC.assert_shuffle_index_equal(c, ob, l, has_rev=l >= 1 or len(sizes) == 5, has_eid=len(sizes) == 5)
    for c in ctxs:
        c.close()
