"""Layer input assembly and reverse shuffle for rows that are read in pieces of 16, 8 and 4 bytes (widths that are
multiples of 4 or 8, of 2, odd; features that start on a 16-, 8- or 4-byte boundary), with hub rows of more entries than
a wave has lanes, against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from test_gpu_parity import _dev, _run_fwd_bwd, check_sage

pytestmark = pytest.mark.gpu

# (dims, bf16): widths at the edges of the lane groups (8, 16, 32, 64 pieces and one more)
SHAPES = [([34, 66, 130, 5], False), ([65, 33, 17, 5], False), ([2, 1, 7, 3], False), ([32, 36, 68, 5], False),
          ([258, 257, 260, 5], False), ([64, 72, 128, 5], True), ([136, 264, 520, 5], True), ([4, 12, 36, 5], True)]


@pytest.mark.parametrize("dims, bf16", SHAPES, ids=lambda x: "x".join(map(str, x)) if isinstance(x, list) else ("bf16" if x else "f32"))
def test_widths_with_hub_rows(dims, bf16):
    w = workloads.custom(3000, 60000, dims=dims, fanouts=[4, 25, 25], batch=1200, n_splits=3, abc=(0.7, 0.1, 0.1),
                         permute_ids=False, name="pieces")
    r = _run_fwd_bwd(w, _dev(), seed=5, it=2, bf16=bf16)
    entries = [np.bincount(np.concatenate([b.shuffle_src_row[b.blk_src] for b in r["batch"].blocks[l]])).max() for l in (1, 2)]
    assert entries[0] > 256 and entries[1] > 64, entries        # workgroup path; several registers per lane
    check_sage(r, 3, bf16=bf16, tag="pieces")


@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
@pytest.mark.parametrize("fanouts", [[4, 5, 3], [8, 9, 1], [16, 7, 17]], ids=str)
def test_edges_in_flight(fanouts, bf16):
    """Fanouts at the edges of the rounds of 4, 8 and 16 edges, rows of 8, 16 and 64 lanes."""
    w = workloads.custom(3000, 60000, dims=[200, 40, 16, 5], fanouts=fanouts, batch=70, n_splits=3, name="rounds")
    check_sage(_run_fwd_bwd(w, _dev(), seed=5, it=2, bf16=bf16), 3, bf16=bf16, tag="rounds")


@pytest.mark.parametrize("dim", [32, 30])
@pytest.mark.parametrize("skip", [0, 1, 2, 3])
def test_features_off_a_16_byte_boundary(dim, skip):
    """float32 rows that start 4, 8 or 12 bytes behind a 16-byte boundary give the same bits as aligned ones."""
    from paper_2303_13775_amd import Context, SageParams
    dev = _dev()
    w = workloads.custom(3000, 60000, dims=[dim, 24, 7], fanouts=[6, 4], batch=150, n_splits=2, name="unaligned")
    ctx = Context(w.indptr.to(dev), w.indices.to(dev), w.pmap.to(dev), w.n_splits, w.fanouts, w.batch)
    ctx.gsplit_sample_split(w.targets(0).to(dev), 3, 1)
    rows = ctx.gsplit_max_rows(0)
    x0 = torch.zeros((rows, dim), device=dev)
    ctx.gsplit_gather_features(w.feat.to(dev), x0)
    params = SageParams(w.dims, *[[t.to(dev) for t in lst] for lst in (w.w_self, w.w_neigh, w.bias)])
    out = [torch.zeros((w.batch, 7), device=dev) for _ in range(2)]
    ctx.gsplit_sage_fwd(params, x0, out[0])
    moved = torch.zeros(rows * dim + 4, device=dev)[skip:skip + rows * dim].view(rows, dim)
    moved.copy_(x0)
    ctx.gsplit_sage_fwd(params, moved, out[1])
    torch.cuda.synchronize()
    assert float(out[0].abs().max()) > 0 and torch.equal(*out)
    ctx.close()
