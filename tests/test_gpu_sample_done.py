"""The batches of a grouped sampling call share the event behind them: the host-side sizes stay those of the context's own
last batch when contexts are grouped anew, used alone in between and closed while others still hold the event; and a query
waits for the event alone where the call is still queued behind other work on a stream that nothing else orders."""
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


def _sizes(ctx, targets, it):
    ctx.gsplit_sample_split(targets, 9, it)
    return ctx.gsplit_batch_sizes()


def test_sizes_of_calls_that_are_still_queued():
    """No synchronisation between a call and its query: torch's streams do not block one another, and the call stands behind
    some eighty milliseconds of other work when the query is made, so that the sizes are right only if the query waits for
    this call's own event.  Contexts hold events of different calls and streams at the end."""
    from paper_2303_13775_amd import Context, gsplit_sample_split_multi
    dev = torch.device("cuda:0")
    w = workloads.custom(5000, 60000, dims=[8, 8, 4], fanouts=[5, 3], batch=900, n_splits=3, name="queued")
    g = [t.to(dev) for t in (w.indptr, w.indices, w.pmap)]
    ctxs, alone = [Context(*g, w.n_splits, w.fanouts, w.batch) for _ in range(4)], Context(*g, w.n_splits, w.fanouts, w.batch)
    # (odd iterations have few targets and go as one launch, the others do not)
    targets = {(k, it): w.targets(10 * it + k)[:(20 + 5 * k if it % 2 else 700 + 50 * k)].to(dev) for k in range(4) for it in range(8)}
    want = {key: _sizes(alone, t, key[1]) for key, t in targets.items()}
    assert len({str(x) for x in want.values()}) == len(want)
    streams = [torch.cuda.Stream() for _ in range(2)]
    markers = {s: torch.zeros(1, dtype=torch.int32, device=dev) for s in streams}
    torch.cuda.synchronize()

    def call(stream, which, it):
        markers[stream].zero_()
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            torch.cuda._sleep(200_000_000)
            markers[stream].fill_(1)
            if len(which) == 1:
                ctxs[which[0]].gsplit_sample_split(targets[which[0], it], 9, it)
            else:
                gsplit_sample_split_multi([ctxs[k] for k in which], [targets[k, it] for k in which], 9, [it] * len(which))

    def check(which, it, queued=None):
        if queued is not None:      # the call is still queued, and a copy to the host does not wait for its stream
            assert not queued.query() and markers[queued].item() == 0
        for k in which:
            assert ctxs[k].gsplit_batch_sizes() == want[k, it], (k, it)

    a, b = streams
    for it, which in enumerate([(0, 1, 2, 3), (0, 1, 2, 3), (3, 1), (2,)]):
        call(a, which, it)
        check(which, it, a)
    call(a, (0, 1, 2, 3), 4)            # all four wait for one event ...
    b.wait_stream(a)
    call(b, (1,), 5)                    # ... one of them moves to the other stream and to a call of its own
    check((1,), 5, b)
    check((0, 2, 3), 4)
    call(b, (0, 2), 6)                  # two of them as a new group, while the last one holds the event of the old one
    check((0, 2), 6, b)
    check((3,), 4)
    check((1,), 5)
    call(a, (3,), 7)
    check((3,), 7, a)
    torch.cuda.synchronize()
    for c in ctxs + [alone]:
        c.close()
