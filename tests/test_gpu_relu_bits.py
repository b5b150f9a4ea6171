"""Float levels whose forward product leaves a bit per activation for the pull of the gradient above it (more than 16384
destinations above, rows that the tiled forms take): gradients against the oracle at widths around the words of 32 bits, in
narrow and wide tiles, with rows of more entries than a wave holds, and where the product is formed again in plain fp32."""
import pytest
import torch

import workloads
from test_gpu_parity import _dev, _run_fwd_bwd, check_sage
from split_rules import FEW, form

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d0, hidden, huge", [(8, 4, False), (8, 36, False), (6, 64, False), (20, 100, False), (50, 132, False),
                                              (12, 256, False), (12, 260, True), (8, 36, True)])
def test_gradients_gated_by_bits(d0, hidden, huge):
    w = workloads.custom(20000, 120000, dims=[d0, hidden, 5], fanouts=[3, 2], batch=16500, n_splits=3, abc=(0.6, 0.15, 0.15),
                         permute_ids=False, name="bits")
    assert form(20000, 10000, 2 * d0, hidden) != FEW
    if huge:        # operands beyond what the parts of a split product carry
        w.feat = w.feat * 1e34
        for t in (w.w_self, w.w_neigh):
            t[0] = t[0] * 1e-34
    check_sage(_run_fwd_bwd(w, _dev(), seed=5, it=2), w.n_layers, tag=f"bits {d0} {hidden}")


@pytest.mark.parametrize("d0, hidden, huge", [(20, 92, False), (20, 96, False), (6, 100, False), (50, 132, False), (12, 256, False),
                                              (12, 260, True), (8, 96, True)])
def test_gradients_of_a_step_gated_by_bits(d0, hidden, huge):
    """The one-call step, whose forward products leave the bits (rows of at least 96)."""
    w = workloads.custom(20000, 120000, dims=[d0, hidden, 5], fanouts=[3, 2], batch=16500, n_splits=3, abc=(0.6, 0.15, 0.15),
                         permute_ids=False, name="bits")
    assert form(20000, 10000, 2 * d0, hidden) != FEW
    if huge:
        w.feat = w.feat * 1e34
        for t in (w.w_self, w.w_neigh):
            t[0] = t[0] * 1e-34
    check_sage(_run_fwd_bwd(w, _dev(), seed=5, it=2, step=True), w.n_layers, tag=f"bits of a step {d0} {hidden}")


def test_bits_are_a_matter_of_the_step():
    """Forward and backward passes by themselves neither hold nor read any; whatever order they and steps come in, captured
    steps of a context that has none among them, the gradients have the same bits."""
    from paper_2303_13775_amd import Context, SageParams
    dev = _dev()
    w = workloads.custom(200000, 900000, dims=[8, 256, 7], fanouts=[3, 2], batch=60000, n_splits=3, name="order")
    graph = [t.to(dev) for t in (w.indptr, w.indices, w.pmap)]
    params = SageParams(w.dims, [t.to(dev) for t in w.w_self], [t.to(dev) for t in w.w_neigh], [t.to(dev) for t in w.bias])
    feat, labels, targets = w.feat.to(dev), w.labels.to(dev), [w.targets(k).to(dev) for k in range(2)]
    logits, glog = [torch.empty((w.batch, w.dims[-1]), device=dev) for _ in range(2)]
    grads = [[torch.empty_like(t, device=dev) for t in part] for part in (w.w_self, w.w_neigh, w.bias)]
    free = lambda: torch.cuda.mem_get_info()[0]  # noqa: E731

    def batch(ctx, k):
        ctx.gsplit_sample_split(targets[k], 3, k)
        ctx.gsplit_gather_features(feat, x0)

    def step(ctx):
        ctx.gsplit_sage_step(params, x0, labels, logits, *grads)

    def separate(ctx):
        ctx.gsplit_sage_fwd(params, x0, logits)
        ctx.gsplit_softmax_xent(logits, labels, glog)
        ctx.gsplit_sage_bwd(params, glog, *grads)

    def taken():
        torch.cuda.synchronize()
        out = [t.clone() for part in grads for t in part]
        for part in grads:
            for t in part:
                t.fill_(7.0)
        return out

    ctx = Context(*graph, w.n_splits, w.fanouts, w.batch)
    x0 = torch.empty((ctx.gsplit_max_rows(0), w.dims[0]), device=dev)
    want = []
    for k in range(2):
        batch(ctx, k)
        separate(ctx)
        want.append(taken())
    # a step captured before any was made eagerly
    side, captured = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured, stream=side):
        step(ctx)
    for k in (0, 1):
        batch(ctx, k)
        captured.replay()
        assert all(torch.equal(a, b) for a, b in zip(taken(), want[k])), ("captured", k)
    before = free()
    for n, (k, run) in enumerate([(0, step), (1, separate), (1, step), (0, separate), (0, step), (0, step)]):
        batch(ctx, k)
        run(ctx)
        assert all(torch.equal(a, b) for a, b in zip(taken(), want[k])), (n, k)
        if n == 0:
            first = free()
    bits = ctx.gsplit_max_rows(1) * w.dims[1] // 8
    assert before - first >= bits and free() == first
    # a forward pass between a step's batch and a captured step with bits
    captured = torch.cuda.CUDAGraph()
    with torch.cuda.graph(captured, stream=side):
        step(ctx)
    for k in (1, 0):
        batch(ctx, k)
        ctx.gsplit_sage_fwd(params, x0, logits)
        captured.replay()
        assert all(torch.equal(a, b) for a, b in zip(taken(), want[k])), ("captured with bits", k)
    ctx.close()
