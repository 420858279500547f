"""GPU parity at the sizes where the kernels' dispatch changes or their tiles end: stage by stage against the oracle,
with the tolerances of test_gpu_parity (bf16 2e-2, fp32 1e-5 of the reference's maximum, also per expert and bucket)."""
import numpy as np
import pytest
import torch

from paper_2304_03946_amd import workloads as W
from test_dispatch import paths
from test_gpu_parity import api, check_gate, run_stagewise, upload  # noqa: F401  (api: module fixture)

pytestmark = pytest.mark.gpu
F32 = dict(dtype=torch.float32, device="cuda")


def stagewise(api, cfg, seed=3):  # noqa: F811
    inp = W.make_layer_inputs(cfg, seed=seed)
    run_stagewise(api, cfg, inp, *W.placement_from_loads(W.prior_loads(cfg, seed), cfg.V, cfg.max_rep, shuffle_seed=11))


# 128 x 128 weight-gradient tiles (the work lists in load order): several jobs per patch, 70 jobs, and segments of 16 K tiles:
# the first size that is cut and the last that is not, and 32 K tiles from a share of 8 on
@pytest.mark.parametrize("N,d,f,E,V", [(2100, 256, 1024, 12, 17), (1300, 256, 2048, 6, 9), (4200, 512, 1024, 5, 8), (3000, 256, 512, 70, 80),
                                       (1024, 136, 264, 3, 5), (1023, 136, 264, 3, 5), (16500, 136, 264, 3, 5)])
def test_weight_gradient_work_lists(api, N, d, f, E, V):  # noqa: F811
    stagewise(api, W.scaled(W.CONFIGS["gpt_m"], N=N, d=d, f=f, E=E, V=V, max_rep=3))


def exact_step(api, A, d, f, E, V, seed=1):  # noqa: F811
    """One expert FFN, forward and backward, of whole numbers, on skewed buckets (some experts and buckets empty): every sum is exact in
    fp32, so every output is the exact sum rounded once, in whatever order and tiles it was computed."""
    B, layer_mod = api
    rng = np.random.default_rng(seed)
    owner = np.concatenate([np.arange(E), rng.integers(E, size=V - E)])
    rng.shuffle(owner)
    share = rng.random(V) ** 3 * (rng.random(V) < 0.9)
    share[rng.integers(V)] += 0.5
    rows = rng.multinomial(A, share / share.sum())
    i32 = lambda v: torch.from_numpy(np.asarray(v, dtype=np.int32)).cuda()
    voff, own = i32(np.concatenate([[0], np.cumsum(rows)])), i32(owner)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, dyp, w1, w2 = (torch.empty(s, **bf).random_(-1, 2, generator=g) for s in ((A, d), (A, d), (E, d, f), (E, f, d)))
    hpre, h, yp, dxp, dw1, dw2 = (torch.full(s, 7.0, **bf) for s in ((A, f), (A, f), (A, d), (A, d), (E, d, f), (E, f, d)))
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, E, 1, V, B.BF16), dtype=torch.uint8, device="cuda")
    B.flexmoe_expert_ffn_fwd(x, voff, own, w1, None, w2, None, B.RELU, hpre, yp, ws, h=h)
    B.flexmoe_expert_ffn_bwd(dyp, x, hpre, w1, w2, voff, own, B.RELU, dxp, dw1, dw2, ws, h=h)
    of = torch.from_numpy(np.repeat(owner, rows)).cuda()
    same = lambda got, want: torch.equal(got, want.bfloat16())
    for e in range(E):
        t = (of == e).nonzero()[:, 0]
        z = x[t].float() @ w1[e].float()
        assert same(hpre[t], z) and same(h[t], z.clamp(min=0)), e
        dz = ((dyp[t].float() @ w2[e].float().t()) * (z > 0)).bfloat16().float()
        assert same(yp[t], h[t].float() @ w2[e].float()) and same(dxp[t], dz @ w1[e].float().t()), e
        assert same(dw2[e], h[t].float().t() @ dyp[t].float()) and same(dw1[e], x[t].float().t() @ dz), e


# 256 x 256 weight-gradient tiles, whole: the work lists dealt out over 64 bins down to 2, in one pass of the wave and (70 experts) in
# several, cut into segments or not, and in load order where the tile grid is irregular; nine column tiles, in bands, whole and ragged;
# ragged ones in strips, with 300 buckets
@pytest.mark.parametrize("A,d,f,E,V,bins,seg", [
    (210000, 256, 1024, 12, 17, 64, 102), (20600, 512, 1024, 5, 8, 32, 32), (21000, 512, 1024, 70, 80, 32, 32), (10400, 512, 2048, 6, 9, 16, 32),
    (5300, 1024, 2048, 5, 7, 8, 32), (2700, 1024, 4096, 3, 5, 4, 0), (4200, 1024, 4096, 3, 5, 4, 32), (1500, 2048, 4096, 2, 3, 2, 0),
    (11000, 768, 1280, 6, 9, 1, 32), (18400, 256, 2304, 4, 6, 1, 32), (9300, 392, 2200, 4, 6, 1, 32), (21000, 392, 1000, 6, 300, 1, 32)])
def test_large_weight_gradient_tiles(api, A, d, f, E, V, bins, seg):  # noqa: F811
    p = paths(A, d, f, E, V)
    assert not p["small_gradients"] and p["bins2"] == p["bins1"] == bins and p["seg_tiles"] == seg
    exact_step(api, A, d, f, E, V)


# rows products past the few-rows kernels' line, with nine column tiles of 256: register-staged (d no multiple of 128) and persistent ones
@pytest.mark.parametrize("A,d,f,E,V", [(9000, 264, 2304, 4, 6), (9000, 256, 2304, 4, 6)])
def test_bands_of_column_tiles_in_the_rows_products(api, A, d, f, E, V):  # noqa: F811
    assert paths(A, d, f, E, V)["few_rows"] == 0
    exact_step(api, A, d, f, E, V)


# dXp and both weight gradients in one launch up to 512 row tiles x column tiles of dXp and 6144 tiles of weight gradients: the last
# sizes and the first past them, with 32-row and 64-row tiles, ragged ones among them
@pytest.mark.parametrize("A,d,f,E,V,rows,merged", [
    (3647, 1024, 2048, 8, 10, 64, True), (3648, 1024, 2048, 8, 10, 64, False), (300, 512, 1024, 96, 110, 32, True),
    (300, 512, 1024, 97, 110, 32, False), (3000, 264, 776, 30, 40, 64, True), (11605, 192, 768, 12, 15, 64, True), (11606, 192, 768, 12, 15, 0, False)])
def test_lines_of_the_merged_backward_launch(api, A, d, f, E, V, rows, merged):  # noqa: F811
    p = paths(A, d, f, E, V)
    assert p["small_gradients"] and p["few_rows"] == rows and p["merged"] == merged
    for _ in range(3):      # the segment counters are left as they were found
        exact_step(api, A, d, f, E, V)


# rows kernels for few rows per expert or little output: 32-row tiles (at most 4 rows per expert on average; N = 1: two
# experts with a single row, the contraction cut into its most segments) and the first size of 64-row tiles, K with a partial last
# tile (d, f multiples of 8 only), K below one tile, ragged column tiles, 512 buckets; (7500, 136, 1032) is past their line
@pytest.mark.parametrize("N,d,f,E,k,V,act", [
    (1, 1024, 4096, 32, 2, 48, W.ACT_GELU_ERF), (31, 264, 520, 16, 2, 21, W.ACT_GELU_TANH), (33, 264, 520, 16, 2, 21, W.ACT_RELU),
    (7, 48, 8, 4, 1, 6, W.ACT_GELU_ERF), (640, 136, 392, 8, 2, 12, W.ACT_GELU_ERF), (641, 136, 392, 8, 2, 12, W.ACT_GELU_ERF),
    (896, 128, 8192, 2, 2, 3, W.ACT_GELU_ERF), (897, 128, 8192, 2, 2, 3, W.ACT_GELU_ERF), (7500, 136, 1032, 4, 2, 6, W.ACT_GELU_TANH),
    (130, 512, 2048, 8, 2, 9, W.ACT_RELU), (900, 128, 256, 256, 4, 512, W.ACT_GELU_ERF)])
def test_rows_products_with_few_rows_per_expert(api, N, d, f, E, k, V, act):  # noqa: F811
    stagewise(api, W.scaled(W.CONFIGS["gpt_m"], N=N, d=d, f=f, E=E, k=k, V=V, act=act, max_rep=3))


# the last size of these kernels and the first of the 256 x 256 ones: by the outputs (register-staged and persistent), by the row
# tiles per vExpert
@pytest.mark.parametrize("N,d,f,E,k,V,act", [
    (9613, 136, 392, 8, 2, 12, W.ACT_RELU), (9614, 136, 392, 8, 2, 12, W.ACT_GELU_ERF), (3584, 512, 2048, 8, 2, 9, W.ACT_GELU_TANH),
    (3585, 512, 2048, 8, 2, 9, W.ACT_RELU), (17612, 128, 256, 256, 4, 512, W.ACT_GELU_ERF), (17613, 128, 256, 256, 4, 512, W.ACT_GELU_ERF)])
def test_rows_products_at_the_line(api, N, d, f, E, k, V, act):  # noqa: F811
    stagewise(api, W.scaled(W.CONFIGS["gpt_m"], N=N, d=d, f=f, E=E, k=k, V=V, act=act, max_rep=3))


# (the first two: contractions cut into segments in both products, so that the second counts on what the first left, and with
# gathered loads and scattered stores)
@pytest.mark.parametrize("N,d,f,E,V,k", [(3, 1024, 1024, 16, 20, 1), (3, 1024, 1024, 16, 20, 2), (3, 256, 1024, 16, 20, 1), (100, 384, 640, 8, 13, 1), (300, 128, 1024, 64, 96, 2)])
def test_forward_variants_with_few_rows_per_expert(api, N, d, f, E, V, k):  # noqa: F811
    """Gathered loads, the scattered store of the top-1 call and the replayed contraction segments: the staged forward's bits."""
    binding, layer_mod = api
    cfg = W.scaled(W.CONFIGS["gpt_m"], N=N, d=d, f=f, E=E, V=V, k=k, backward=False, max_rep=3)
    inp = W.make_layer_inputs(cfg)
    dev = upload(layer_mod, inp)
    rng = np.random.default_rng(4)
    b1, b2 = (layer_mod.to_device(W.Bf16Tensor.from_f32((rng.standard_normal((E, n)) * 0.3).astype(np.float32))) for n in (f, d))
    rep = W.placement_from_loads(W.prior_loads(cfg), cfg.V, cfg.max_rep, shuffle_seed=11)
    L = layer_mod.MoELayer.for_config(cfg)
    L.yp.fill_(float("nan"))
    L.forward(dev["x"], dev["wg"], dev["w1"], dev["w2"], *rep, b1, b2)
    want = L.y.clone()
    assert not want.isnan().any()
    for fwd in [L.forward, L.forward_fused] + ([L.forward_top1] if k == 1 else []):
        for _ in range(3):      # the segment counters are left as they were found
            L.y.fill_(float("nan"))
            L.yp.fill_(float("nan"))
            fwd(dev["x"], dev["wg"], dev["w1"], dev["w2"], *rep, b1, b2, keep_hpre=False)
            assert torch.equal(L.y, want)


# fp32: tiles of 64 x 64 outputs and 32-wide K tiles (below one tile, whole tiles, ragged in every dimension), experts
# without tokens, one token, more buckets than a wave has lanes, a contraction over many buckets of one expert
@pytest.mark.parametrize("N,d,f,E,k,V,act", [
    (1, 8, 8, 2, 1, 2, W.ACT_RELU), (65, 64, 96, 3, 1, 5, W.ACT_GELU_ERF), (300, 40, 136, 5, 2, 9, W.ACT_GELU_TANH),
    (513, 128, 256, 4, 4, 6, W.ACT_GELU_ERF), (400, 72, 64, 100, 3, 180, W.ACT_GELU_ERF), (128, 256, 512, 1, 1, 3, W.ACT_RELU)])
def test_fp32_layer(api, N, d, f, E, k, V, act):  # noqa: F811
    stagewise(api, W.scaled(W.CONFIGS["tiny"], N=N, d=d, f=f, E=E, k=k, V=V, act=act, max_rep=3, backward=True))


# groups of 1 .. 64 lanes per token and four experts per lane; features below, at and past the pieces held in LDS
@pytest.mark.parametrize("N,d,E,k", [(1, 8, 1, 1), (17, 128, 2, 2), (50, 136, 6, 3), (330, 136, 64, 8), (210, 40, 65, 2), (700, 72, 256, 4), (95, 264, 33, 3)])
def test_fp32_gate(api, N, d, E, k):  # noqa: F811
    binding, layer_mod = api
    rng = np.random.default_rng(N + E)
    x = rng.standard_normal((N, d)).astype(np.float32)
    wg = (rng.standard_normal((d, E)) / np.sqrt(d)).astype(np.float32)
    idx = torch.full((N, k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((N, k), dtype=torch.float32, device="cuda")
    ws = torch.empty(1 << 16, dtype=torch.uint8, device="cuda")
    binding.flexmoe_gate_topk(layer_mod.to_device(x), layer_mod.to_device(wg), k, idx, w, ws)
    check_gate(idx.cpu().numpy(), w.cpu().numpy(), x, wg, k, W.DT_F32)


# bf16 gate.  Both sides of the lines between one chunk in flight per wave and several (256 features, 8192 tokens), between the quarters
# and the streaming kernel and its two widths (32768 and 65536 tokens, up to 64 experts); fewer chunks of features than waves, a partial
# last chunk, padded expert tiles; experts in whole groups of four (W_g transposed by the LDS reads) and not, in every kernel.
# (check_gate wants at most 5 % of the tokens within
# its error bound of a tie; the bound grows as d^1.5, 5e-4 at d = 520, against gaps of about 0.2 between k + 1 neighbouring
# logits: about 1 % per pick at d = 520 but 3 % at d = 1032, so the larger d come with k = 1.)
@pytest.mark.parametrize("N,d,E,k", [(8192, 520, 64, 2), (8193, 520, 64, 2), (16384, 72, 20, 1), (16385, 72, 20, 1), (24577, 248, 20, 1), (24577, 256, 20, 1), (33, 512, 33, 2),
                                     (400, 1032, 100, 1), (400, 520, 128, 2), (1, 8, 48, 8), (165, 504, 64, 3), (500, 776, 256, 1),
                                     (32767, 136, 64, 1), (32768, 136, 64, 1), (65535, 72, 64, 1), (65536, 72, 64, 1), (32768, 72, 30, 1), (65536, 72, 37, 1), (32768, 136, 4, 1),
                                     (8193, 520, 128, 1), (300, 136, 100, 1), (300, 520, 101, 1), (8193, 136, 101, 1), (300, 264, 30, 2), (500, 264, 6, 2), (300, 264, 250, 1)])
def test_bf16_gate(api, N, d, E, k):  # noqa: F811
    binding, layer_mod = api
    rng = np.random.default_rng(N + E)
    x, wg = (W.Bf16Tensor.from_f32(a.astype(np.float32)) for a in (rng.standard_normal((N, d)), rng.standard_normal((d, E)) / np.sqrt(d)))
    idx = torch.full((N, k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((N, k), dtype=torch.float32, device="cuda")
    ws = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    binding.flexmoe_gate_topk(layer_mod.to_device(x), layer_mod.to_device(wg), k, idx, w, ws)
    check_gate(idx.cpu().numpy(), w.cpu().numpy(), W.decode(x), W.decode(wg), k, W.DT_BF16)


# bias and gate gradients: chunks of 128 rows (one row, whole chunks, one row more), column blocks of 512 (bf16) or 256
# (fp32) columns and ragged ones, experts without tokens, more token rows than chunks
@pytest.mark.parametrize("dtype,N,d,f,E,k,V", [
    ("bf16", 1, 8, 8, 2, 1, 2), ("bf16", 128, 512, 520, 1, 1, 1), ("bf16", 129, 520, 512, 1, 1, 1), ("bf16", 2100, 136, 1032, 5, 2, 8),
    ("bf16", 300, 72, 64, 200, 4, 300), ("f32", 129, 256, 264, 1, 1, 1), ("f32", 700, 40, 520, 6, 3, 9)])
def test_bias_and_gate_gradients(api, dtype, N, d, f, E, k, V):  # noqa: F811
    """Against the same sums in float64.  Errors: the result's rounding (2^-8 in bf16) and 2^-22 per term summed in fp32."""
    B, layer_mod = api
    cfg = W.scaled(W.CONFIGS["gpt_m" if dtype == "bf16" else "tiny"], N=N, d=d, f=f, E=E, k=k, V=V, max_rep=3, backward=True)
    inp = W.make_layer_inputs(cfg, seed=5)
    dev = upload(layer_mod, inp)
    L = layer_mod.MoELayer.for_config(cfg)
    L.forward(dev["x"], dev["wg"], dev["w1"], dev["w2"], *W.placement_from_loads(W.prior_loads(cfg), V, 3, shuffle_seed=2))
    dx0 = L.backward(dev["dy"], dev["w1"], dev["w2"])[0].clone()
    A, tdt = N * k, L.dx.dtype
    dhpre = L.ws[:A * f * L.dx.element_size()].view(tdt).view(A, f).double()
    voff = L.vexpert_off.long()
    row_e = torch.repeat_interleave(L.vexpert_owner.long(), voff[1:] - voff[:-1])

    def check(got, ref, size, terms):
        bound = (2.0 ** -8 if tdt == torch.bfloat16 and got.dtype == tdt else 2.0 ** -22) * (ref.abs() + 1e-30) + terms * 2.0 ** -22 * size
        assert bool(((got.double() - ref).abs() <= bound).all()), ((got.double() - ref).abs() / bound).max()

    def expert_sums(rows):
        return torch.zeros(E, rows.shape[1], dtype=torch.float64, device="cuda").index_add_(0, row_e, rows)

    want = [(t, expert_sums(t), expert_sums(t.abs())) for t in (dhpre, L.dyp.double())]
    db1, db2 = torch.full((E, f), 7.0, dtype=tdt, device="cuda"), torch.full((E, d), 7.0, dtype=tdt, device="cuda")
    for one, two in ((db1, None), (None, db2), (db1, db2)):      # either may be left out
        B.flexmoe_expert_bias_grads(L.dyp, L.vexpert_off, L.vexpert_owner, f, E, one, two, L.ws)
        for got, (_, ref, size) in zip((one, two), want):
            if got is not None:
                check(got, ref, size, A)
                got.fill_(7.0)
    dl, dwg = torch.zeros((N, k), dtype=torch.float32, device="cuda"), torch.full((d, E), 7.0, dtype=tdt, device="cuda")
    B.flexmoe_gate_bwd(dev["wg"], L.topk_idx, L.topk_w, dev["dy"], L.yp, L.xp, L.dest, L.src, L.vexpert_off, L.vexpert_owner,
                       dl, L.dx, dwg, L.ws)
    g, yk = L.topk_w.double(), L.yp.double()[L.dest.long()].view(N, k, d)
    dg, size = (dev["dy"].double()[:, None] * yk).sum(2), (dev["dy"].double()[:, None] * yk).abs().sum(2)
    check(dl, g * (dg - (g * dg).sum(1, keepdim=True)), g * (size + (g * size).sum(1, keepdim=True)), d)
    cols = dev["wg"].double().t()[L.topk_idx.long()]
    step = (dl.double()[:, :, None] * cols)
    check(L.dx, dx0.double() + step.sum(1), dx0.double().abs() + step.abs().sum(1), k + 1)
    rows = dl.double().flatten()[L.src.long()][:, None] * L.xp.double()
    check(dwg, expert_sums(rows).t(), expert_sums(rows.abs()).t(), A)


# the same kernels: logits that differ in the order of their fp32 sums alone.  One feature per 64-wide chunk is non-zero; an
# expert's products are one 2^24 and small whole numbers, so that each addition rounds and the order decides ties
@pytest.mark.parametrize("N,d,E,k", [(257, 256, 20, 2), (33, 1024, 32, 1), (300, 448, 64, 3), (257, 1024, 64, 2), (100, 712, 40, 8), (300, 576, 128, 2),
                                     (200, 320, 100, 2), (200, 1024, 200, 2), (8192, 1024, 48, 2), (8193, 1024, 48, 2), (16384, 520, 32, 2),
                                     (16385, 520, 32, 2), (24577, 520, 32, 2), (16385, 2048, 32, 2), (32767, 1032, 64, 2)])
def test_order_of_the_gate_sums(api, N, d, E, k):  # noqa: F811
    """Fewer than 32768 tokens or more than 64 experts: chunks c, c + 4, .. in ascending order, then 0 + (1 + (2 + 3))."""
    binding, layer_mod = api
    rng = np.random.default_rng(N + d + E)
    chunks, patterns = (d + 63) // 64, d % 64 or 64
    small = rng.choice([-1.0, 0.0, 1.0, 1.0, 2.0], size=(chunks, patterns, E)).astype(np.float32)
    big = rng.integers(chunks, size=(patterns, E))
    small[big, np.arange(patterns)[:, None], np.arange(E)] = 2.0 ** 24
    wg, x = np.zeros((chunks, 64, E), dtype=np.float32), np.zeros((N, chunks, 64), dtype=np.float32)
    wg[:, :patterns] = small
    of = rng.integers(patterns, size=N)                  # a token's pattern: its feature within every chunk
    x[np.arange(N), :, of] = 1.0
    wg, x = wg.reshape(-1, E)[:d], x.reshape(N, -1)[:, :d]
    quarter = [np.zeros((patterns, E), dtype=np.float32) for _ in range(4)]
    for c in range(chunks):
        quarter[c % 4] = quarter[c % 4] + small[c]
    logits = quarter[0] + (quarter[1] + (quarter[2] + quarter[3]))
    assert logits.dtype == np.float32 and (logits != small.astype(np.float64).sum(0)).mean() > 0.1, "the order must matter"
    want = np.argsort(-logits, axis=1, kind="stable")[:, :k]
    idx = torch.full((N, k), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((N, k), dtype=torch.float32, device="cuda")
    ws = torch.empty(4 << 20, dtype=torch.uint8, device="cuda")
    up = lambda a: layer_mod.to_device(W.Bf16Tensor.from_f32(np.ascontiguousarray(a)))
    binding.flexmoe_gate_topk(up(x), up(wg), k, idx, w, ws)
    assert np.array_equal(idx.cpu().numpy(), want[of])
    ex = np.exp(np.take_along_axis(logits, want, 1).astype(np.float64) - logits.max(1, keepdims=True))
    np.testing.assert_allclose(w.cpu().numpy(), (ex / ex.sum(1, keepdims=True))[of], rtol=1e-5, atol=1e-7)


# whole numbers and +-2^24 in one column: an addition past 2^24 rounds, so the order decides what is left
@pytest.mark.parametrize("dtype,A,d", [("f32", 1, 8), ("f32", 61, 256), ("f32", 300, 264), ("bf16", 64, 512), ("bf16", 128, 520), ("bf16", 449, 40)])
def test_order_of_the_bias_sums(api, dtype, A, d):  # noqa: F811
    """Chunks of 128 rows: rows r, r + 4, .. in ascending order, the four sums in order; then the chunks in order (four at most here)."""
    B, layer_mod = api
    tdt, code = (torch.float32, B.F32) if dtype == "f32" else (torch.bfloat16, B.BF16)
    rng = np.random.default_rng(A + d)
    rows = rng.integers(-1, 3, size=(A, d)).astype(np.float32)
    for sign in (1.0, -1.0):
        rows[rng.integers(A, size=d), np.arange(d)] = sign * 2.0 ** 24
    chunks = []
    for c0 in range(0, A, 128):
        chains = np.zeros((4, d), dtype=np.float32)
        for r in range(c0, min(c0 + 128, A)):
            chains[(r - c0) % 4] += rows[r]
        chunks.append(((chains[0] + chains[1]) + chains[2]) + chains[3])
    want = np.zeros(d, dtype=np.float32)
    for c in chunks:
        want = want + c
    assert A < 8 or (want != rows.sum(0, dtype=np.float64)).any(), "the order must matter"
    f, i32 = 16, lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    ws = torch.zeros(B.flexmoe_workspace_bytes(A, d, f, 1, 1, 1, code), dtype=torch.uint8, device="cuda")
    got = torch.empty((1, d), dtype=tdt, device="cuda")
    B.flexmoe_expert_bias_grads(torch.from_numpy(rows).cuda().to(tdt), i32([0, A]), i32([0]), f, 1, None, got, ws)
    assert torch.equal(got[0].cpu(), torch.from_numpy(want).to(tdt))


# contractions that are no whole 128-wide rounds evaluate the activation instead of reading it from a table, in the kernels for
# few rows and in the 256 x 256 ones past their line
@pytest.mark.parametrize("act", [W.ACT_GELU_ERF, W.ACT_GELU_TANH, W.ACT_RELU])
@pytest.mark.parametrize("A,d,f", [(3, 136, 264), (200, 40, 264), (15000, 136, 1032)])
def test_activation_of_zero_and_nan(api, act, A, d, f):  # noqa: F811
    B, layer_mod = api
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    bf = dict(dtype=torch.bfloat16, device="cuda")
    w1, w2, x = torch.ones((1, d, f), **bf), torch.ones((1, f, d), **bf), torch.zeros((A, d), **bf)
    hpre, h, yp = torch.empty((A, f), **bf), torch.empty((A, f), **bf), torch.empty((A, d), **bf)
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, 1, 1, 1, B.BF16), dtype=torch.uint8, device="cuda")
    B.flexmoe_expert_ffn_fwd(x, i32([0, A]), i32([0]), w1, None, w2, None, act, hpre, yp, ws, h=h)
    assert not hpre.any() and not h.any() and not yp.any(), "act(0) is 0"
    if act != W.ACT_RELU:
        b1 = torch.zeros((1, f), **bf)
        b1.view(torch.int16)[0, 5] = -64                  # 0xffc0: a NaN with its sign set
        B.flexmoe_expert_ffn_fwd(x, i32([0, A]), i32([0]), w1, b1, w2, None, act, hpre, yp, ws, h=h)
        assert hpre.isnan().sum() == A and torch.equal(h.isnan(), hpre.isnan()) and bool(yp.isnan().all())


def test_offsets_of_a_very_wide_layer(api):  # noqa: F811
    """64 contraction rows of 34 million columns: beyond the 32-bit offsets of the few-rows kernels, although the rows are few."""
    B, layer_mod = api
    A, d, f = 2, 64, 34_089_000
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    bf = dict(dtype=torch.bfloat16, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.empty((A, d), **bf).random_(-1, 2, generator=g)
    w1, w2 = torch.empty((1, d, f), **bf).random_(-2, 3, generator=g), torch.zeros((1, f, d), **bf)
    hpre, yp = torch.empty((A, f), **bf), torch.empty((A, d), **bf)
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, 1, 1, 1, B.BF16), dtype=torch.uint8, device="cuda")
    B.flexmoe_expert_ffn_fwd(x, i32([0, A]), i32([0]), w1, None, w2, None, B.RELU, hpre, yp, ws)
    for c in range(0, f, 1 << 22):
        assert torch.equal(hpre[:, c:c + (1 << 22)].float(), x.float() @ w1[0, :, c:c + (1 << 22)].float()), c
    assert not yp.any()


# dXp, dW2 and dW1 in one launch, dW2 and dW1 in one, and in launches of their own (256 x 256 tiles)
@pytest.mark.parametrize("A,d,f,E", [(512, 64, 256, 2), (256, 128, 256, 2), (40000, 64, 128, 2), (256, 512, 2048, 2), (10000, 512, 2048, 2)])
def test_weight_gradients_over_what_is_read_no_longer(api, A, d, f, E):  # noqa: F811
    """dXp, dW2, dW1 are computed in this order: w1, h and dyp may be overwritten by what comes after their last use."""
    B, layer_mod = api
    bf = dict(dtype=torch.bfloat16, device="cuda")
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(A + d)
    w1, w2, x, dyp = (torch.empty(s, **bf).normal_(0, std, generator=g) for s, std in
                      (((E, d, f), 0.05), ((E, f, d), 0.05), ((A, d), 1.0), ((A, d), 1.0)))
    hpre, h, yp = torch.empty((A, f), **bf), torch.empty((A, f), **bf), torch.empty((A, d), **bf)
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, E, 1, E, B.BF16), dtype=torch.uint8, device="cuda")
    voff, owner = i32([0, A // 3, A]), i32([0, 1])
    B.flexmoe_expert_ffn_fwd(x, voff, owner, w1, None, w2, None, B.GELU_ERF, hpre, yp, ws, h=h)

    def bwd(over=None, with_dw2=False):
        """The products, with dw1 (or dw2) at the start of a copy of the tensor `over`."""
        t = {"w1": w1.clone(), "w2": w2.clone(), "h": h.clone(), "dyp": dyp.clone()}
        dxp, dw1, dw2 = torch.zeros((A, d), **bf), torch.zeros((E, d, f), **bf), torch.zeros((E, f, d), **bf)
        if over is not None and t[over].numel() < w1.numel():      # (a tensor smaller than the gradient: with room behind it)
            room = torch.empty(w1.numel(), **bf)
            room[:t[over].numel()] = t[over].flatten()
            base, t[over] = room, room[:t[over].numel()].view(t[over].shape)
        elif over is not None:
            base = t[over].flatten()
        if over is not None:
            view = base[:w1.numel()]
            dw1, dw2 = (dw1, view.view(E, f, d)) if with_dw2 else (view.view(E, d, f), dw2)
        B.flexmoe_expert_ffn_bwd(t["dyp"], x, hpre, t["w1"], t["w2"], voff, owner, B.GELU_ERF, dxp, dw1, dw2, ws, h=t["h"])
        return dxp, dw1, dw2
    want = bwd()
    assert all(t.any() for t in want)
    for over, with_dw2 in (("w1", False), ("w1", True), ("w2", False), ("w2", True), ("h", False), ("dyp", False)):
        for _ in range(3):
            assert all(torch.equal(a, b) for a, b in zip(bwd(over, with_dw2), want)), (over, with_dw2)


def test_fp32_products_of_more_tiles_than_a_launch_takes(api):  # noqa: F811
    """512 vExperts, each with room for a row tile, times 2^15 column tiles: 2^32 threads in one grid.  Whole numbers: exact sums."""
    B, layer_mod = api
    A, d, f, E, V = 16, 8, 1 << 21, 2, 512
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(2)
    x, dyp = (torch.empty((A, d), **F32).random_(-1, 2, generator=g) for _ in range(2))
    w1, w2 = torch.empty((E, d, f), **F32).random_(-2, 3, generator=g), torch.empty((E, f, d), **F32).random_(-1, 2, generator=g)
    hpre, h = torch.full((A, f), 7.0, **F32), torch.full((A, f), 7.0, **F32)
    yp, dxp, dw1, dw2 = torch.full((A, d), 7.0, **F32), torch.full((A, d), 7.0, **F32), torch.empty_like(w1), torch.empty_like(w2)
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, E, 1, V, B.F32), dtype=torch.uint8, device="cuda")
    voff, owner = i32([0] * 100 + [10] * 300 + [A] * 113), i32([0] * 200 + [1] * 312)      # rows in buckets 99 and 399
    B.flexmoe_expert_ffn_fwd(x, voff, owner, w1, None, w2, None, B.RELU, hpre, yp, ws, h=h)
    B.flexmoe_expert_ffn_bwd(dyp, x, hpre, w1, w2, voff, owner, B.RELU, dxp, dw1, dw2, ws, h=h)
    for e, rows in ((0, slice(0, 10)), (1, slice(10, A))):
        z = x[rows].double() @ w1[e].double()
        assert torch.equal(hpre[rows].double(), z) and torch.equal(h[rows].double(), z.clamp(min=0))
        assert torch.equal(yp[rows].double(), z.clamp(min=0) @ w2[e].double())
        dz = (dyp[rows].double() @ w2[e].double().t()) * (z > 0)
        assert torch.equal(dxp[rows].double(), dz @ w1[e].double().t())
        assert torch.equal(dw1[e].double(), x[rows].double().t() @ dz)
        assert torch.equal(dw2[e].double(), z.clamp(min=0).t() @ dyp[rows].double())


def test_fp32_weight_gradients_of_very_many_tiles(api):  # noqa: F811
    """65538 tiles of 64 columns, in the columns of dW1 and the rows of dW2.  Whole numbers: exact sums."""
    B, layer_mod = api
    A, d, f = 3, 8, 65538 * 64
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(3)
    x, dyp, hpre = (torch.empty(s, **F32).random_(-2, 3, generator=g) for s in ((A, d), (A, d), (A, f)))
    w1, w2 = torch.empty((1, d, f), **F32).random_(-2, 3, generator=g), torch.empty((1, f, d), **F32).random_(-1, 2, generator=g)
    dxp, dw1, dw2 = torch.empty((A, d), **F32), torch.full((1, d, f), 7.0, **F32), torch.full((1, f, d), 7.0, **F32)
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, 1, 1, 1, B.F32), dtype=torch.uint8, device="cuda")
    B.flexmoe_expert_ffn_bwd(dyp, x, hpre, w1, w2, i32([0, A]), i32([0]), B.RELU, dxp, dw1, dw2, ws)
    dz = (dyp.double() @ w2[0].double().t()) * (hpre > 0)
    assert torch.equal(dw2[0].double(), hpre.double().clamp(min=0).t() @ dyp.double()) and torch.equal(dw1[0].double(), x.double().t() @ dz)
    assert torch.equal(dxp.double(), dz @ w1[0].double().t())


# a row among 300 (32 x 64 tiles) and among 25000 (64 x 64 tiles in all four products); whole K tiles, an odd number of them, a ragged one
@pytest.mark.parametrize("d,f", [(256, 1024), (264, 1048), (224, 1000)])
def test_fp32_rows_do_not_depend_on_the_batch(api, d, f):  # noqa: F811
    B, layer_mod = api
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(d)
    most, few = 25000, 300
    x, dyp = (torch.empty((most, d), **F32).normal_(0, 1, generator=g) for _ in range(2))
    w1, w2 = torch.empty((1, d, f), **F32).normal_(0, 0.05, generator=g), torch.empty((1, f, d), **F32).normal_(0, 0.05, generator=g)

    def layer(A, E):
        """Rows 0 .. A - 1 with expert 0; E - 1 experts without rows behind it."""
        c = lambda t: torch.cat([t, torch.zeros((E - 1,) + t.shape[1:], **F32)])
        out = [torch.empty((A, n), **F32) for n in (f, f, d, d)]
        dw1, dw2 = torch.empty((E, d, f), **F32), torch.empty((E, f, d), **F32)
        ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, E, 1, E, B.F32), dtype=torch.uint8, device="cuda")
        voff, owner = i32([0] + [A] * E), i32(list(range(E)))
        hpre, h, yp, dxp = out
        B.flexmoe_expert_ffn_fwd(x[:A], voff, owner, c(w1), None, c(w2), None, B.GELU_ERF, hpre, yp, ws, h=h)
        B.flexmoe_expert_ffn_bwd(dyp[:A], x[:A], hpre, c(w1), c(w2), voff, owner, B.GELU_ERF, dxp, dw1, dw2, ws, h=h)
        return out, (dw1[0], dw2[0])
    (many, _), (small, grads) = layer(most, 1), layer(few, 1)
    for a, b in zip(many, small):
        assert torch.equal(a[:few], b)
    # the weight gradients likewise: 64 x 64 tiles where the rows per expert are few
    assert all(torch.equal(a, b) for a, b in zip(layer(few, 4)[1], grads))


# 64 x 64 tiles (few rows per expert) and 32 x 64 ones; buckets of none to a few rows, so that many meet in a K tile, and rows of several K tiles
@pytest.mark.parametrize("A,E,V,d,f", [(1, 1, 1, 8, 8), (50, 2, 37, 40, 72), (59, 2, 512, 72, 136), (150, 2, 70, 72, 136), (700, 3, 130, 264, 40), (700, 3, 5, 136, 520), (900, 40, 512, 64, 64)])
def test_fp32_weight_gradients_over_short_buckets(api, A, E, V, d, f):  # noqa: F811
    """Whole numbers: exact sums."""
    B, layer_mod = api
    rng = np.random.default_rng(A + V)
    owner = np.concatenate([np.arange(E), rng.integers(E, size=V - E)])
    rng.shuffle(owner)
    rows = np.bincount(rng.integers(V, size=A) // 2 * 2 % V, minlength=V)      # (every other bucket is empty)
    voff = np.concatenate([[0], np.cumsum(rows)])
    i32 = lambda v: torch.from_numpy(np.asarray(v, dtype=np.int32)).cuda()
    g = torch.Generator(device="cuda").manual_seed(A)
    x, dyp, hpre = (torch.empty(s, **F32).random_(-2, 3, generator=g) for s in ((A, d), (A, d), (A, f)))
    w1, w2 = (torch.empty(s, **F32).random_(-2, 3, generator=g) for s in ((E, d, f), (E, f, d)))
    dxp, dw1, dw2 = torch.empty((A, d), **F32), torch.full((E, d, f), 7.0, **F32), torch.full((E, f, d), 7.0, **F32)
    ws = torch.empty(B.flexmoe_workspace_bytes(A, d, f, E, 1, V, B.F32), dtype=torch.uint8, device="cuda")
    B.flexmoe_expert_ffn_bwd(dyp, x, hpre, w1, w2, i32(voff), i32(owner), B.RELU, dxp, dw1, dw2, ws)
    of = torch.from_numpy(np.repeat(owner, rows)).cuda()
    for e in range(E):
        t = of == e
        dz = (dyp[t].double() @ w2[e].double().t()) * (hpre[t] > 0)
        assert torch.equal(dw2[e].double(), hpre[t].double().clamp(min=0).t() @ dyp[t].double())
        assert torch.equal(dw1[e].double(), x[t].double().t() @ dz)
        assert torch.equal(dxp[t].double(), dz @ w1[e].double().t())
