"""Which form the top layer of gsplit_sage_step takes (one fused kernel up to 2048 targets of the batch, launches of
their own above), that either gives what the three calls one after the other give (in bf16 bit for bit, up to the order in
which the top layer's weight gradients are summed), and that a captured step holds for batches of more targets than the
one it was captured on."""
import pytest
import torch

import workloads
from test_gpu_parity import TOL_F32

pytestmark = pytest.mark.gpu


class _Step:
    def __init__(self, cap, dims=(16, 32, 40), bf16=False):
        from paper_2303_13775_amd import GSPLIT_BF16, GSPLIT_F32, Context, SageParams
        assert torch.cuda.is_available(), "these tests need the MI355X"
        dev = torch.device("cuda:0")
        self.w = w = workloads.custom(20000, 400000, dims=list(dims), fanouts=[3, 2], batch=cap, n_splits=4, name="top-layer")
        self.ctx = Context(w.indptr.to(dev), w.indices.to(dev), w.pmap.to(dev), w.n_splits, w.fanouts, cap)
        ws = [[t.to(dev) for t in lst] for lst in (w.w_self, w.w_neigh, w.bias)]
        self.w_self, self.w_neigh, self.bias = ws
        self.params = SageParams(w.dims, *ws, dtype=GSPLIT_BF16 if bf16 else GSPLIT_F32)
        self.grads = [[torch.zeros_like(t) for t in lst] for lst in ws]
        self.feat, self.labels = w.feat.to(dev).to(torch.bfloat16 if bf16 else torch.float32), w.labels.to(dev)
        self.x0 = torch.zeros((self.ctx.gsplit_max_rows(0), w.dims[0]), dtype=self.feat.dtype, device=dev)
        self.logits = torch.zeros((cap, w.dims[-1]), device=dev)
        self.glog, self.loss = torch.zeros_like(self.logits), torch.zeros(cap, device=dev)
        self.dev = dev

    def sample(self, n):
        self.ctx.gsplit_sample_split(self.w.targets(3)[:n].to(self.dev).contiguous(), 11, 4)

    def step(self):
        self.ctx.gsplit_gather_features(self.feat, self.x0)
        self.ctx.gsplit_sage_step(self.params, self.x0, self.labels, self.logits, *self.grads, row_loss=self.loss)

    def calls(self):
        self.ctx.gsplit_gather_features(self.feat, self.x0)
        self.ctx.gsplit_sage_fwd(self.params, self.x0, self.logits)
        self.ctx.gsplit_softmax_xent(self.logits, self.labels, self.glog, self.loss)
        self.ctx.gsplit_sage_bwd(self.params, self.glog, *self.grads)

    def results(self, n):
        out = [self.logits[:n].clone(), self.loss[:n].clone()] + [t.clone() for lst in self.grads for t in lst]
        for t in [self.logits, self.loss] + [t for lst in self.grads for t in lst]:
            t.fill_(7.0)
        return out


def _same_bits_below_the_top(a, b):
    """Logits, loss and the gradients of the lower layer bit for bit; the top layer's weight and bias gradients within a
    float32 sum over at most 4096 rows in another order."""
    for i, (x, y) in enumerate(zip(a, b)):      # logits, loss, (bottom, top) x (self, neighbour, bias)
        if i < 2 or i % 2 == 0:
            assert torch.equal(x, y), (i, float((x - y).abs().max()))
        else:
            assert float((x - y).abs().max()) <= 1e-5 * (float(y.abs().max()) + 1e-30), i


def _same(a, b):
    for x, y in zip(a, b):
        assert float((x - y).abs().max()) <= TOL_F32 * (float(y.abs().max()) + 1e-30)


@pytest.mark.parametrize("cap, n", [(2048, 2048), (2049, 2049), (2049, 2048), (4096, 2041), (4096, 9), (4096, 2049), (6000, 512)])
def test_form_follows_the_targets_of_the_batch(cap, n):
    s = _Step(cap)
    s.sample(n)
    s.calls()
    want = s.results(n)
    s.ctx.gsplit_timing_enable(True)
    s.ctx.gsplit_timing_read()
    s.step()
    torch.cuda.synchronize()
    assert any(k.startswith("top_fused") for k in s.ctx.gsplit_timing_read()) == (n <= 2048)
    _same(s.results(n), want)
    s.ctx.close()


# classes around the contractions that are formed as plain sums (below three) and around blocks of 16 and 32; targets that
# leave one, two and three rows to the last workgroup; the narrowest and widest rows
@pytest.mark.parametrize("n", [1, 2, 18, 333])
@pytest.mark.parametrize("D, N", [(4, 1), (8, 2), (12, 3), (36, 16), (100, 17), (68, 33), (256, 47), (384, 64)])
def test_float_step_against_the_three_calls(D, N, n):
    s = _Step(400, (16, D, N))
    s.sample(n)
    s.calls()
    want = s.results(n)
    s.ctx.gsplit_timing_enable(True)
    s.ctx.gsplit_timing_read()
    s.step()
    torch.cuda.synchronize()
    assert any(k.startswith("top_fused") for k in s.ctx.gsplit_timing_read())
    _same(s.results(n), want)
    s.ctx.close()


@pytest.mark.parametrize("heavy", [False, True], ids=["", "heavy-weight"])
@pytest.mark.parametrize("kind", ["flt-max", "inf", "nan"])
@pytest.mark.parametrize("N, n", [(2, 1), (5, 18), (47, 333)])
def test_float_step_with_values_the_parts_cannot_carry(N, n, kind, heavy):
    """Rows of the top layer with FLT_MAX (infinite in bfloat16), an infinity or a NaN, and a weight of FLT_MAX that meets
    zeros in the logits but not in the input gradient: infinities and NaN where the three calls have them, and what is
    finite within a float32 sum.  The bottom layer copies the features; the weights that meet the large value differ by
    more than a rounding of it, so that the loss does not hang on one."""
    D = 24
    s = _Step(400, (D, D, N))
    for t in (s.w_self[0], s.w_neigh[0], s.bias[0]):
        t.zero_()
    s.w_self[0].copy_(torch.eye(D))
    s.w_self[0][9, 9] = 4.0
    s.w_self[0][11, 11] = 0.0
    for t in (s.w_self[1], s.w_neigh[1]):
        t[3] = 0.125 / (torch.arange(N, device=s.dev) + 1)
    if heavy:
        s.w_self[1][11, 0] = 3.4028e38
    s.feat.copy_(torch.rand(s.feat.shape, generator=torch.Generator().manual_seed(1)) + 0.5)
    col, value = {"flt-max": (3, 3.4028e38), "inf": (9, 3.4028e38), "nan": (3, float("nan"))}[kind]
    s.feat[0::7, col] = value
    s.sample(n)
    s.calls()
    want = s.results(n)
    s.step()
    got = s.results(n)
    s.ctx.close()
    assert kind != "inf" or n < 18 or bool(torch.isinf(want[0]).any() or torch.isnan(want[0]).any())
    for i, (x, y) in enumerate(zip(got, want)):
        for f in (torch.isnan, torch.isposinf, torch.isneginf):
            assert torch.equal(f(x), f(y)), (i, f)
        ok = torch.isfinite(y)
        # (per row: the inputs of a weight gradient differ by forty orders of magnitude)
        scale = torch.where(ok, y, torch.zeros_like(y)).abs()
        scale = scale.max(-1, keepdim=True).values if y.dim() > 1 else scale.max()
        assert bool(((x - y).abs() <= TOL_F32 * scale + 1e-30)[ok].all()), i


def test_captured_step_takes_larger_and_smaller_batches():
    s = _Step(4096)
    s.sample(300)
    s.step()                    # sizes the internal buffers
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(device=s.dev)):
        s.step()
    for n in (300, 4096, 17, 2500, 300):
        s.sample(n)
        s.calls()
        torch.cuda.synchronize()
        want = s.results(n)
        graph.replay()
        torch.cuda.synchronize()
        _same(s.results(n), want)
    s.ctx.close()


# widths and classes at the edges of the tiles: one, two and four steps of 16 classes, classes that are no multiple of 8,
# inputs whose pair of rows ends inside a block of 32 columns, more than one round of column blocks, the narrowest and widest
@pytest.mark.parametrize("n", [1, 15, 17, 333])
@pytest.mark.parametrize("D, N", [(8, 1), (8, 5), (24, 16), (72, 47), (136, 33), (256, 47), (264, 17), (384, 64)])
def test_bf16_step_gives_the_bits_of_the_three_calls(D, N, n):
    s = _Step(400, (16, D, N), bf16=True)
    s.sample(n)
    s.calls()
    want = s.results(n)
    s.ctx.gsplit_timing_enable(True)
    s.ctx.gsplit_timing_read()
    s.step()
    torch.cuda.synchronize()
    assert any(k.startswith("top_fused") for k in s.ctx.gsplit_timing_read())
    _same_bits_below_the_top(s.results(n), want)
    s.ctx.close()


def test_captured_bf16_step_takes_larger_and_smaller_batches():
    s = _Step(4096, (16, 72, 47), bf16=True)
    s.sample(300)
    s.step()                    # sizes the internal buffers
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(device=s.dev)):
        s.step()
    for n in (300, 4096, 17, 2500, 300):
        s.sample(n)
        s.calls()
        torch.cuda.synchronize()
        want = s.results(n)
        graph.replay()
        torch.cuda.synchronize()
        _same_bits_below_the_top(s.results(n), want)
    s.ctx.close()
