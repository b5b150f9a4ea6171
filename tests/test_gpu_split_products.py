"""The fp32 products formed from bfloat16 parts, at the edges of their tiles, chunks and k-tiles, against
float64 on a ring graph (vertex v samples v + 1, so a layer input is [x(v) | x(v + 1)]), held to the bound
of a float32 sum, K u sum|a||b| with u = 2^-24 (plus one u for what the parts drop); and with infinities,
NaN and magnitudes that bfloat16 rounds to infinity, which must come out as float32 gives them; and with
operands near and below the smallest normal float."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

U = 2.0 ** -24
N_VERT = 20000          # capacity of the batches: the level's bound, beyond the bar of the chunked weight gradients


def _context(cap, layers=1, n_vert=N_VERT):
    from paper_2303_13775_amd import Context
    assert torch.cuda.is_available(), "these tests need the MI355X"
    dev = torch.device("cuda:0")
    indptr = torch.arange(n_vert + 1, dtype=torch.int32, device=dev)
    indices = ((torch.arange(n_vert, device=dev) + 1) % n_vert).to(torch.int32)
    pmap = (torch.arange(n_vert, device=dev) % 3).to(torch.uint8)
    return Context(indptr, indices, pmap, 3, [1] * layers, cap), dev


def _case(rows, D, N, cap, feat=None, glog=None, weights=None):
    """Logits and gradients of a one-layer model, and the float64 layer input X and gradient dZ."""
    from paper_2303_13775_amd import SageParams
    ctx, dev = _context(cap)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows * 131 + D * 7 + N)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=dev)  # noqa: E731
    if feat is None:
        feat = rnd(N_VERT, D)
    ws, wn, b = weights(dev) if weights else (rnd(D, N), rnd(D, N), rnd(N))
    glog = rnd(cap, N) if glog is None else glog(dev, cap)
    tg = torch.randperm(N_VERT, generator=gen, device=dev)[:rows].to(torch.int32)
    params = SageParams([D, N], [ws], [wn], [b])
    ctx.gsplit_sample_split(tg, 5, 1)
    x0 = torch.zeros((ctx.gsplit_max_rows(0), D), device=dev)
    ctx.gsplit_gather_features(feat, x0)
    logits = torch.full((cap, N), 7.0, device=dev)
    ctx.gsplit_sage_fwd(params, x0, logits)
    grads = [[torch.zeros_like(t)] for t in (ws, wn, b)]
    ctx.gsplit_sage_bwd(params, glog, *grads)
    ids = torch.cat(ctx.fetch_batch()["local_front"][1]).long()
    f64 = feat.double()
    X = torch.cat([f64[ids], f64[(ids + 1) % N_VERT]], 1)
    W = torch.cat([ws, wn]).double()
    ctx.close()
    return logits, torch.cat([grads[0][0], grads[1][0]]), grads[2][0], X, W, b.double(), glog[:rows].double()


def _within(got, want, scale, k):
    assert bool(((got.double() - want).abs() <= (k + 3) * U * scale + 1e-37).all()), float(
        ((got.double() - want).abs() / scale.clamp_min(1e-30)).max() / U)


# (cap, rows, D, N); the forms that these take are held by test_split_rules.py
PRODUCTS = [(cap, rows, D, N) for cap in (1024, N_VERT) for rows in (1, 31, 64, 65, 97, 777)
            for D, N in ((1, 1), (3, 2), (8, 31), (16, 33), (17, 128), (64, 129), (100, 132), (130, 47))]
# weight gradients in blocks of 128, of whole blocks, with remainders of M and N, rows in pieces and float by float
PRODUCTS += [(N_VERT, rows, D, N) for rows in (1, 95, 97, 777) for D, N in ((130, 132), (129, 200), (192, 256), (129, 131))]
# wide tiles: rows and columns of whole tiles and with remainders, contractions of less than a k-tile, of whole ones and not,
# rows in pieces and float by float
PRODUCTS += [(N_VERT, rows, D, N) for rows, D, N in ((12352, 8, 256), (12353, 34, 200), (6300, 64, 500), (16000, 130, 201),
                                                     (9000, 7, 100), (8257, 17, 128), (16401, 65, 72), (4200, 129, 256))]


@pytest.mark.parametrize("cap, rows, D, N", PRODUCTS)
def test_products_against_float64(cap, rows, D, N):
    logits, gw, gb, X, W, b, dz = _case(rows, D, N, cap)
    _within(logits[:rows], X @ W + b, X.abs() @ W.abs() + b.abs(), 2 * D)
    assert bool((logits[rows:] == 7.0).all())           # rows the batch does not have are not written
    _within(gw, X.T @ dz, X.abs().T @ dz.abs(), rows)
    _within(gb, dz.sum(0), dz.abs().sum(0), rows)


@pytest.mark.parametrize("cap", [1024, N_VERT])
# (the last two with N = 200: weight gradients in blocks of 128; 9000 rows with N = 200: wide tiles)
@pytest.mark.parametrize("rows, D", [(1, 40), (2, 40), (1, 1), (2, 1), (3, 1), (1000, 1), (9000, 1), (1, 130), (2, 130)])
@pytest.mark.parametrize("N", [7, 64, 200])
def test_contractions_of_one_and_two_products(cap, rows, D, N):
    """As float32 forms them: one rounding per product, so K u sum|a||b| with nothing added (logits: 2 D = 2 products,
    no bias; weight gradients: `rows` products)."""
    cap = max(cap, rows)
    for seed in range(4):       # (the dropped terms are that large for some operands only)
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(seed)
        feat = torch.randn(N_VERT, D, generator=gen, device="cuda:0")
        par = [torch.randn(D, N, generator=gen, device="cuda:0") for _ in range(2)]
        logits, gw, gb, X, W, b, dz = _case(rows, D, N, cap, feat=feat, weights=lambda dev: (*par, torch.zeros(N, device=dev)))
        for got, want, scale, k in ((logits[:rows], X @ W, X.abs() @ W.abs(), 2 * D), (gw, X.T @ dz, X.abs().T @ dz.abs(), rows)):
            if k <= 2:
                assert bool(((got.double() - want).abs() <= k * U * scale + 1e-37).all()), k


# the last three: wide tiles (rows in pieces, float by float) and, with 20000 rows of room, blocks of 128
SMALL_OPERANDS = [(97, 24, 40), (300, 23, 100), (1000, 34, 130), (9000, 24, 100), (6300, 24, 500), (9000, 23, 100), (300, 130, 132)]


@pytest.mark.parametrize("cap", [1024, N_VERT])
@pytest.mark.parametrize("rows, D, N", SMALL_OPERANDS)
@pytest.mark.parametrize("small, large", [(1e-34, 1e30), (1e-36, 1e30), (1e-38, 1e31), (1e-42, 1e33)])
def test_small_operands_keep_their_bits(cap, rows, D, N, small, large):
    """Nothing but small values in one operand and large ones in the other, so that the results are of ordinary
    size and the bound of a float32 sum sees every bit of the small operand (down to subnormal floats)."""
    cap = max(cap, rows)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows + D)
    rnd = lambda *s: torch.randn(*s, generator=gen, device=dev)  # noqa: E731
    for x, w, z in ((small, large, large), (large, small, small)):
        feat, zero = rnd(N_VERT, D) * x, torch.zeros(N, device=dev)
        logits, gw, gb, X, W, _, dz = _case(rows, D, N, cap, feat=feat, weights=lambda dev: (rnd(D, N) * w, rnd(D, N) * w, zero),
                                            glog=lambda dev, cap: rnd(cap, N) * z)
        assert float(X.abs().max()) > 0 and float(W.abs().max()) > 0
        _within(logits[:rows], X @ W, X.abs() @ W.abs(), 2 * D)
        _within(gw, X.T @ dz, X.abs().T @ dz.abs(), rows)


# The last four: more tiles than the chip holds workgroups (three per compute unit), so that every one walks several tiles
# of several k-tiles, rows read in 16-byte pieces and one by one, outputs of more and of at most 64 columns.
@pytest.mark.parametrize("rows, dims, n_vert", [(5, (6, 5, 3), N_VERT), (65, (12, 132, 9), N_VERT), (300, (20, 36, 70), N_VERT),
                                                (777, (16, 65, 33), N_VERT), (40000, (64, 132, 72), 1 << 17),
                                                (40000, (33, 130, 70), 1 << 17), (70000, (24, 30, 36), 1 << 18),
                                                (70000, (25, 32, 33), 1 << 18)])
def test_two_layers_against_float64(rows, dims, n_vert):
    """The input-gradient product and its side inputs: hidden pre-activations are kept far from zero."""
    from paper_2303_13775_amd import SageParams
    cap = max(1024, rows)
    ctx, dev = _context(cap, 2, n_vert)
    gen = torch.Generator(device=dev)
    gen.manual_seed(rows)
    uni = lambda *s: torch.rand(*s, generator=gen, device=dev) + 0.5  # noqa: E731
    sign = torch.where(torch.arange(dims[1], device=dev) % 3 > 0, 1.0, -1.0)
    par = [[uni(dims[0], dims[1]) * sign, uni(dims[1], dims[2]) - 1], [uni(dims[0], dims[1]) * sign, uni(dims[1], dims[2]) - 1],
           [torch.zeros(dims[1], device=dev), uni(dims[2])]]
    feat = uni(n_vert, dims[0])
    tg = torch.randperm(n_vert, generator=gen, device=dev)[:rows].to(torch.int32)
    glog = torch.randn(cap, dims[2], generator=gen, device=dev)
    ctx.gsplit_sample_split(tg, 5, 1)
    x0 = torch.zeros((ctx.gsplit_max_rows(0), dims[0]), device=dev)
    ctx.gsplit_gather_features(feat, x0)
    logits = torch.zeros((cap, dims[2]), device=dev)
    params = SageParams(list(dims), *par)
    ctx.gsplit_sage_fwd(params, x0, logits)
    grads = [[torch.zeros_like(t) for t in part] for part in par]
    ctx.gsplit_sage_bwd(params, glog, *grads)
    ids = torch.cat(ctx.fetch_batch()["local_front"][2]).long()
    ctx.close()
    p64 = [[t.double().requires_grad_() for t in part] for part in par]
    f = feat.double()

    def layer(l, h):
        return h @ p64[0][l] + torch.roll(h, -1, 0) @ p64[1][l] + p64[2][l]
    out = layer(1, torch.relu(layer(0, f)))[ids]
    (out * glog[:rows].double()).sum().backward()
    err = lambda a, o: float((a.double() - o).norm() / o.norm().clamp_min(1e-300))  # noqa: E731
    assert err(logits[:rows], out.detach()) < 4e-6
    for l in range(2):
        for k in range(3):
            # (sums over the rows of products of three float32 stages)
            assert err(grads[k][l], p64[k][l].grad) < 4e-6, (l, k)


# the form for few rows, narrow tiles of one block of columns and of several, wide tiles; the last with blocks of 128
VALUES = [(130, 40, 24), (9000, 40, 24), (9000, 100, 24), (9000, 500, 24), (9000, 100, 23), (9000, 500, 130)]


@pytest.mark.parametrize("rows, N, D", VALUES)
def test_values_the_parts_cannot_carry(rows, N, D):
    """Rows with an infinity, a NaN, FLT_MAX (infinite in bfloat16), and small values beside ordinary ones."""
    def weights(dev):
        w = torch.full((D, N), 0.5, device=dev)
        w[:, 1::2] = -0.25
        return w, w.clone(), torch.zeros(N, device=dev)
    dev = torch.device("cuda:0")
    feat = torch.ones(N_VERT, D, device=dev)
    feat[0::7, 3] = float("inf")
    feat[1::7, 5] = float("-inf")
    feat[2::7, 9] = float("nan")
    feat[3::7, 1] = 3.4028e38
    feat[4::7] = 1e-36
    glog = lambda dev, cap: torch.full((cap, N), 2.0 ** -10, device=dev)  # noqa: E731
    for cap in (1024, N_VERT):
        cap = max(cap, rows)
        logits, gw, gb, X, W, b, dz = _case(rows, D, N, cap, feat=feat, glog=glog, weights=weights)
        for got, want in ((logits[:rows], X @ W + b), (gw, X.T @ dz)):
            got, want = got.cpu().numpy(), want.float().cpu().numpy()
            assert np.array_equal(np.isnan(got), np.isnan(want))
            assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isneginf(got), np.isneginf(want))
            ok = np.isfinite(want)
            assert np.allclose(got[ok], want[ok], rtol=2e-6, atol=0)
