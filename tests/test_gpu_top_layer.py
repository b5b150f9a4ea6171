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
