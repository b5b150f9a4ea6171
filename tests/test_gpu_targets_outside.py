"""Target ids outside the graph are left out of the batch and reported: the rows of every level are those of the oracle's
batch of the ids inside it, whichever launches separate the targets, and stay within the bounds (which count a vertex once)
when every vertex of a small graph is a target and any number of ids lie outside."""
import numpy as np
import pytest
import torch

import workloads
from oracle import reference as R
from test_gpu_parity import _dev, assert_batch_equal

pytestmark = pytest.mark.gpu


def _levels(ctx, L, S, dev):
    from paper_2303_13775_amd import binding as B
    out = []
    for l in range(L + 1):
        v = ctx.gsplit_batch_level(l)
        off = B._view_i32(v.d_local_off, S + 1, dev).tolist()
        assert off[S] <= ctx.gsplit_max_rows(l)
        cat = B._view_i32(v.d_local_cat, off[S], dev).cpu().numpy()
        out.append([cat[off[s]:off[s + 1]] for s in range(S)])
    return out


# vertices, fanouts (top layer last), targets: one launch for targets and layers, one for the targets, two for the targets
CASES = {"one-launch": (500, [3, 2], 50), "layers-beside": (2000, [4, 3, 9], 300), "targets-alone": (2000, [4, 3], 1000),
         "two-launches": (4000, [3, 2], 1500), "whole-graph": (1023, [2, 2], 1023), "whole-graph-wide": (1023, [2, 9], 1023)}


@pytest.mark.parametrize("share", ["one", "half", "all"])
@pytest.mark.parametrize("table_mode", [1, 2], ids=["hashed", "direct"])
@pytest.mark.parametrize("name", list(CASES))
def test_ids_outside_the_graph_are_left_out(name, table_mode, share):
    from paper_2303_13775_amd import Context, GsplitError
    dev = _dev()
    n, fan, batch = CASES[name]
    w = workloads.custom(n, 12 * n, dims=[4] * (len(fan) + 1), fanouts=fan, batch=batch, n_splits=4, name=name)
    ctx = Context(w.indptr.to(dev), w.indices.to(dev), w.pmap.to(dev), 4, fan, batch, table_mode=table_mode)
    gen = torch.Generator().manual_seed(len(name))
    tg = w.targets(0).clone()
    out = torch.randperm(batch, generator=gen)[:{"one": 1, "half": batch // 2, "all": batch}[share]]
    tg[out] = torch.tensor([n, -1, 2 ** 31 - 1, n + 7, -2 ** 31])[torch.arange(out.numel()) % 5].to(tg.dtype)
    inside = tg[(tg >= 0) & (tg < n)]
    for it in range(2):
        ctx.gsplit_sample_split(tg.to(dev), 77, it)
        with pytest.raises(GsplitError) as e:
            ctx.gsplit_batch_sizes()
        assert e.value.code == -1
        got = _levels(ctx, len(fan), 4, dev)
        if inside.numel() == 0:
            assert all(part.size == 0 for level in got for part in level)
            continue
        ob = R.sp_sample(w.indptr.numpy(), w.indices.numpy(), w.pmap.numpy(), 4, fan, inside.numpy(), 77, it)
        for l in range(len(fan) + 1):
            for s in range(4):
                assert np.array_equal(got[l][s], ob.local_front[l][s]), (l, s)
    good = w.targets(1)
    ctx.gsplit_sample_split(good.to(dev), 77, 5)            # the context stays usable
    assert_batch_equal(ctx.fetch_batch(), R.sp_sample(w.indptr.numpy(), w.indices.numpy(), w.pmap.numpy(), 4, fan, good.numpy(), 77, 5),
                       4, len(fan))
    ctx.close()
