"""Float levels whose forward product leaves a bit per activation for the pull of the gradient above it (more than 16384
destinations above, rows that the tiled forms take): gradients against the oracle at widths around the words of 32 bits, in
narrow and wide tiles, with rows of more entries than a wave holds, and where the product is formed again in plain fp32."""
import pytest

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
