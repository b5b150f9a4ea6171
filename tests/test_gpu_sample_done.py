"""The batches of a grouped sampling call share the event behind them: the host-side sizes stay those of the context's own
last batch when contexts are grouped anew, used alone in between and closed while others still hold the event."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def test_sizes_when_contexts_are_regrouped():
    from paper_2303_13775_amd import Context, gsplit_sample_split_multi
    dev = torch.device("cuda:0")
    w = workloads.custom(5000, 60000, dims=[8, 8, 4], fanouts=[5, 3], batch=60, n_splits=3, name="regroup")
    g = [t.to(dev) for t in (w.indptr, w.indices, w.pmap)]
    make = lambda: Context(*g, w.n_splits, w.fanouts, w.batch)  # noqa: E731
    ctxs, alone = [make() for _ in range(4)], make()
    targets = [w.targets(k).to(dev) for k in range(4)]
    streams = [torch.cuda.Stream() for _ in range(2)]

    def check(ctx, k, it):
        alone.gsplit_sample_split(targets[k], 9, it)
        assert ctx.gsplit_batch_sizes() == alone.gsplit_batch_sizes(), (k, it)

    def group(which, it):
        stream = streams[it % 2]
        with torch.cuda.stream(stream):
            gsplit_sample_split_multi([ctxs[k] for k in which], [targets[k] for k in which], 9, [it] * len(which))
        return [(k, it) for k in which]

    torch.cuda.synchronize()
    last = {}
    for it, which in enumerate([(0, 1, 2, 3), (0, 1, 2, 3), (1,), (2, 3), (0, 1), (3, 0, 2, 1), (2,), (3,), (2, 0)]):
        last.update(group(which, it))
        torch.cuda.synchronize()
        for k, i in last.items():
            check(ctxs[k], k, i)
    group((0, 1, 2, 3), 40)
    ctxs[0].close()
    for k in (1, 2, 3):
        check(ctxs[k], k, 40)
    for c in ctxs[1:] + [alone]:
        c.close()
