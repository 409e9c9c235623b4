"""Parity of the whole layer (forward + backward through the C ABI) against the CPU oracle."""
import numpy as np
import pytest

from paper_2511_09741_amd import inputs as I
from tests import util as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_c1_fp32_tiny_layer(taw, seed):
    """The smallest stated configuration: fp32, B=1 S=128 H=64, 4 heads x 16, I=176; tensor-scale error <= 1e-4."""
    U.check_layer(taw, I.CONFIGS["C1"], seed=seed)


def test_c1_shapes_with_peaked_attention_and_nontrivial_gains(taw):
    """At sigma_w = 0.02 the scores are nearly flat; sigma_w = 0.5 makes the softmax peaked, and
    gains away from 1 make a dropped gamma visible."""
    U.check_layer(taw, I.CONFIGS["C1"], seed=3, sigma_w=0.5, gamma_jitter=0.3)


@pytest.mark.parametrize("B,S,H,nh,I_", [(2, 37, 48, 3, 40), (1, 1, 32, 2, 24), (3, 65, 64, 4, 100), (1, 200, 30, 3, 50)])
def test_fp32_ragged_shapes(taw, B, S, H, nh, I_):
    """Generic kernels on shapes that are no multiple of any tile or vector width (S=1 included)."""
    cfg = I.LayerConfig("ragged", I.F32, B, S, H, nh, H // nh, I_)
    U.check_layer(taw, cfg, seed=4, sigma_w=0.3, gamma_jitter=0.2)


def test_bf16_storage_on_generic_kernels(taw):
    """bf16 storage with head_dim 16: the generic attention between the MFMA products."""
    cfg = I.LayerConfig("bf16-generic", I.BF16, 2, 48, 64, 4, 16, 88)
    U.check_layer(taw, cfg, seed=5, sigma_w=0.2, gamma_jitter=0.2)


def test_accumulate_flag_adds_into_the_shard(taw):
    import torch
    cfg = I.CONFIGS["C1"]
    w = I.make_weights(cfg, 0)
    x, dy = I.make_activations(cfg, 0)
    L = U.DeviceLayer(taw, cfg, flags=taw.TAW_ACCUMULATE)
    L.set_weights(w)
    xd, dyd = U.to_dev(x, cfg.dtype), U.to_dev(dy, cfg.dtype)
    L.fwd(xd)
    L.G.fill_(7.0)                       # padding and payload start at a known value
    L.bwd(xd, dyd)
    L.bwd(xd, dyd)
    g2 = L.grads()
    L2 = U.DeviceLayer(taw, cfg, flags=0)
    L2.set_weights(w)
    L2.fwd(xd)
    L2.G.fill_(7.0)
    L2.bwd(xd, dyd)
    g1 = L2.grads()
    for k in g1:
        assert U.tensor_scale_err(g2[k] - 7.0, 2 * g1[k]) < 1e-5, k
    # the padding between sub-tensors is never written
    flat = L2.G.cpu().numpy()
    mask = np.ones(flat.size, bool)
    shapes = {"gamma_attn": 64, "w_qkv": 192 * 64, "w_o": 64 * 64, "gamma_mlp": 64, "w_gate_up": 352 * 64, "w_down": 64 * 176}
    for k, n in shapes.items():
        mask[L2.layout[k]:L2.layout[k] + n] = False
    assert np.all(flat[mask] == 7.0)
    torch.cuda.synchronize()


def test_microbatch_accumulation_matches_oracle_sum(taw):
    """Same weights, independent micro-batches, G accumulated across them (config 5's pattern at tiny size)."""
    from oracle import decoder_layer as O
    cfg = I.CONFIGS["C1"]
    w = I.make_weights(cfg, 0, sigma_w=0.2)
    w64 = I.weights_to_f64(w, cfg.dtype)
    L = U.DeviceLayer(taw, cfg, flags=taw.TAW_ACCUMULATE)
    L.set_weights(w)
    Gsum = None
    for mb in range(4):
        x, dy = I.make_activations(cfg, 0, mb=mb)
        xd, dyd = U.to_dev(x, cfg.dtype), U.to_dev(dy, cfg.dtype)
        y = L.fwd(xd)
        dx = L.bwd(xd, dyd)
        yr, cache = O.layer_fwd(w64, I.to_f64(x, cfg.dtype), cfg.n_heads, cfg.rope_theta, cfg.rms_eps)
        dxr, G = O.layer_bwd(w64, cache, I.to_f64(dy, cfg.dtype))
        assert U.tensor_scale_err(U.from_dev(y), yr) < 1e-4 and U.tensor_scale_err(U.from_dev(dx), dxr) < 1e-4
        Gsum = G if Gsum is None else {k: O.grad_accum(Gsum[k], G[k]) for k in G}
    got = L.grads()
    for k in Gsum:
        assert U.tensor_scale_err(got[k], Gsum[k]) < 1e-4, k


@pytest.mark.parametrize("B,S,nh,I_,sigma", [(1, 256, 2, 384, 0.02), (2, 333, 2, 392, 0.05), (1, 1024, 4, 1408, 0.02), (1, 77, 1, 136, 0.1),
                                             (1, 256, 2, 400, 0.02), (16, 48, 2, 384, 0.05)])
def test_bf16_layer_on_mfma_kernels(taw, B, S, nh, I_, sigma):
    """bf16, head_dim 128: the MFMA GEMM and attention kernels carry the layer.  Sizes span several
    tiles and leave ragged tails in tokens, widths and the SwiGLU dimension.  The backward linears run
    pairwise in one grid.  The first, third, fifth and last case (token counts a multiple of 256, an even
    number of heads, S >= 32) rotate unrounded q and k, the others round them first; the last has sequences
    of 48 tokens, whose positions wrap inside a tile."""
    cfg = I.LayerConfig("bf16-mfma", I.BF16, B, S, nh * 128, nh, 128, I_, sigma_w=sigma)
    U.check_layer(taw, cfg, seed=B + S, gamma_jitter=0.1)


def _cuts(taw, T, H, I_):
    """ranges each product's contraction is cut into: the forward products, and the input gradients ("d...") and weight gradients ("G...")"""
    out = {}
    for k, N, K in (("qkv", 3 * H, H), ("o", H, H), ("gate_up", 2 * I_, H), ("down", H, I_)):
        f, b = taw.taw_diag_gemm_plan(0, T, N, K), taw.taw_diag_gemm_plan(1, T, N, K)
        out.update({k: f["splits"], "d" + k: b["splits_dx"], "G" + k: b["splits"]})
    return {k: n for k, n in out.items() if n > 1}


@pytest.mark.parametrize("H,nh,B,S", [(1024, 8, 4, 512), (2048, 16, 2, 384)])
def test_bf16_layer_at_the_widths_of_the_papers_throughput_table(taw, H, nh, B, S):
    """The narrower models of the paper's throughput table (Experiments, Throughput and Memory Usage: H = 1024 and 2048,
    heads of 128, I = 8H/3 rounded up to 256, micro-batches of several sequences): whole layer against the oracle, every
    element, at a reduced sequence length.  Some of their products are cut into ranges summed by the second kernel: weight
    gradients along the tokens, input gradients and the 2048-wide down projection along the widths."""
    cfg = I.LayerConfig(f"table-{H}", I.BF16, B, S, H, nh, 128, (8 * H // 3 + 255) // 256 * 256)
    assert _cuts(taw, B * S, H, cfg.I) == ({"Gdown": 2, "Go": 2, "dqkv": 2, "dgate_up": 4} if H == 1024 else {"down": 2, "dqkv": 2, "dgate_up": 2})
    U.check_layer(taw, cfg, seed=H + S)


def test_bf16_layer_with_the_other_forms_of_the_attention_backward(taw):
    """TAW_ATTN_BWD_FUSED (one kernel, dQ partial sums in private slots inside the workspace) and TAW_ATTN_BWD_RECOMPUTE
    (two kernels, the scores recomputed, nothing extra in the workspace) against the oracle, beside the default (two
    kernels, dS handed over through the workspace); same tolerance, they differ in summation order at most."""
    cfg = I.LayerConfig("bf16-fused-bwd", I.BF16, 2, 1100, 512, 4, 128, 1408, sigma_w=0.05)
    w = I.make_weights(cfg, 7, gamma_jitter=0.1)
    x, dy = I.make_activations(cfg, 7)
    w64 = I.weights_to_f64(w, cfg.dtype)
    from oracle import decoder_layer as O
    yr, cache = O.layer_fwd(w64, I.to_f64(x, cfg.dtype), cfg.n_heads, cfg.rope_theta, cfg.rms_eps)
    dxr, Gr = O.layer_bwd(w64, cache, I.to_f64(dy, cfg.dtype))
    ws = {f: taw.taw_layer_workspace_bytes(taw.desc_from_config(cfg, f)) for f in (0, taw.TAW_ATTN_BWD_FUSED, taw.TAW_ATTN_BWD_RECOMPUTE)}
    assert ws[taw.TAW_ATTN_BWD_RECOMPUTE] < ws[0] and ws[taw.TAW_ATTN_BWD_RECOMPUTE] < ws[taw.TAW_ATTN_BWD_FUSED]
    for flags in (taw.TAW_ATTN_BWD_FUSED, taw.TAW_ATTN_BWD_RECOMPUTE, 0):
        L = U.DeviceLayer(taw, cfg, flags=flags)
        L.set_weights(w)
        xd, dyd = U.to_dev(x, cfg.dtype), U.to_dev(dy, cfg.dtype)
        L.fwd(xd)
        dx = L.bwd(xd, dyd)
        assert U.tensor_scale_err(U.from_dev(dx), dxr) < U.TOL[cfg.dtype]
        G = L.grads()
        for k in Gr:
            assert U.tensor_scale_err(G[k], Gr[k]) < U.TOL[cfg.dtype], (flags, k)


def test_four_chained_layers_with_staged_weights(taw):
    """Config 4's pattern at reduced width (bf16, MFMA kernels): forward through layers 0..3, backward
    3..0, every layer's weights arriving through taw_weight_stage into one of two staging buffers on a
    side stream (ready / consumed events).  The oracle chains the same four layers in fp64; the device
    passes bf16 activations between layers.  Compared: the last output, the gradient of the first
    input and all four gradient shards."""
    import torch
    from oracle import decoder_layer as O
    nl = 4
    cfg = I.LayerConfig("chain", I.BF16, 2, 320, 256, 2, 128, 392, sigma_w=0.05, n_layers=nl)
    ws = [I.make_weights(cfg, 0, layer=l, gamma_jitter=0.1) for l in range(nl)]
    x, dy = I.make_activations(cfg, 0)
    # ---- oracle
    w64 = [I.weights_to_f64(w, cfg.dtype) for w in ws]
    a, caches = I.to_f64(x, cfg.dtype), []
    for l in range(nl):
        a, c = O.layer_fwd(w64[l], a, cfg.n_heads, cfg.rope_theta, cfg.rms_eps)
        caches.append(c)
    y_ref = a
    g, G_ref = I.to_f64(dy, cfg.dtype), [None] * nl
    for l in reversed(range(nl)):
        g, G_ref[l] = O.layer_bwd(w64[l], caches[l], g)
    dx_ref = g
    # ---- device
    desc = taw.desc_from_config(cfg, 0)
    lay = taw.taw_layer_weight_layout(desc)
    P = lay["total_elems"]
    store = [U.to_dev(I.pack_chunk(w, lay, P, cfg.dtype), cfg.dtype) for w in ws]      # the owners' copies
    stage = [torch.empty_like(store[0]) for _ in range(2)]
    ctx = [torch.empty(taw.taw_layer_ctx_bytes(desc), dtype=torch.uint8, device="cuda") for _ in range(nl)]
    wsb = taw.taw_layer_workspace_bytes(desc)
    wsp = torch.empty(wsb, dtype=torch.uint8, device="cuda")
    rope = torch.empty(cfg.S * (cfg.head_dim // 2) * 2, dtype=torch.float32, device="cuda")
    taw.taw_rope_table_init(desc, rope)
    G = [torch.zeros(P, dtype=torch.float32, device="cuda") for _ in range(nl)]
    compute, side = torch.cuda.current_stream(), torch.cuda.Stream()
    ready = [torch.cuda.Event() for _ in range(2)]
    consumed = [torch.cuda.Event() for _ in range(2)]
    order = list(range(nl)) + list(reversed(range(nl)))          # layer whose weights each step needs
    for b in range(2):
        consumed[b].record(compute)
    taw.taw_weight_stage(stage[0], store[order[0]], P * 2, side, consumed[0], ready[0])
    acts = [U.to_dev(x, cfg.dtype)]
    grad = U.to_dev(dy, cfg.dtype)
    for i, l in enumerate(order):
        buf = i & 1
        if i + 1 < len(order):                                    # next step's weights into the other buffer
            taw.taw_weight_stage(stage[buf ^ 1], store[order[i + 1]], P * 2, side, consumed[buf ^ 1], ready[buf ^ 1])
        compute.wait_event(ready[buf])
        if i < nl:
            y = torch.empty_like(acts[0])
            taw.taw_layer_fwd(desc, stage[buf], rope, acts[l], y, ctx[l], wsp, wsb, compute)
            acts.append(y)
        else:
            dx = torch.empty_like(grad)
            taw.taw_layer_bwd(desc, stage[buf], rope, acts[l], grad, ctx[l], dx, G[l], wsp, wsb, compute)
            grad = dx
        consumed[buf].record(compute)
    torch.cuda.synchronize()
    e_y, e_dx = U.tensor_scale_err(U.from_dev(acts[nl]), y_ref), U.tensor_scale_err(U.from_dev(grad), dx_ref)
    print(f"4 chained layers: y={e_y:.2e} dx={e_dx:.2e}", flush=True)
    assert e_y < 2e-2 and e_dx < 2e-2
    for l in range(nl):
        got = {k: v.astype(np.float64) for k, v in I.unpack_shard(G[l].cpu().numpy(), lay, cfg).items()}
        for k in G_ref[l]:
            e = U.tensor_scale_err(got[k], G_ref[l][k])
            assert e < 2e-2, (l, k, e)


def test_bf16_microbatch_accumulation_with_staging(taw):
    """Config 5's pattern at reduced width (bf16, MFMA kernels): one layer, four micro-batches, the
    weight gradients accumulated by the backward's epilogue into the fp32 shard, while the next
    layer's chunk is staged on a side stream."""
    import torch
    from oracle import decoder_layer as O
    cfg = I.LayerConfig("mb4", I.BF16, 1, 384, 256, 2, 128, 520, sigma_w=0.05, n_microbatches=4)
    w = I.make_weights(cfg, 0, gamma_jitter=0.1)
    w64 = I.weights_to_f64(w, cfg.dtype)
    L = U.DeviceLayer(taw, cfg, flags=taw.TAW_ACCUMULATE)
    L.set_weights(w)
    nxt = U.to_dev(I.pack_chunk(I.make_weights(cfg, 0, layer=1), L.layout, L.layout["total_elems"], cfg.dtype), cfg.dtype)
    staged = torch.empty_like(nxt)
    side = torch.cuda.Stream()
    taw.taw_weight_stage(staged, nxt, nxt.numel() * 2, side, None, None)
    Gsum = None
    for mb in range(4):
        x, dy = I.make_activations(cfg, 0, mb=mb)
        xd, dyd = U.to_dev(x, cfg.dtype), U.to_dev(dy, cfg.dtype)
        y = L.fwd(xd)
        dx = L.bwd(xd, dyd)
        yr, cache = O.layer_fwd(w64, I.to_f64(x, cfg.dtype), cfg.n_heads, cfg.rope_theta, cfg.rms_eps)
        dxr, G = O.layer_bwd(w64, cache, I.to_f64(dy, cfg.dtype))
        assert U.tensor_scale_err(U.from_dev(y), yr) < 2e-2 and U.tensor_scale_err(U.from_dev(dx), dxr) < 2e-2
        Gsum = G if Gsum is None else {k: O.grad_accum(Gsum[k], G[k]) for k in G}
    got = L.grads()
    for k in Gsum:
        assert U.tensor_scale_err(got[k], Gsum[k]) < 2e-2, k
    torch.cuda.synchronize()
    assert torch.equal(staged, nxt)


@pytest.mark.parametrize("cfg", [I.CONFIGS["C1"], I.LayerConfig("recompute-bf16", I.BF16, 2, 333, 256, 2, 128, 392, sigma_w=0.05)],
                         ids=["fp32", "bf16"])
def test_recompute_mode_gives_the_same_results(taw, cfg):
    """Activation checkpointing (TAW_RECOMPUTE): the forward keeps only x, the backward rebuilds the
    intermediates in the workspace.  Results against the oracle as in the default mode, and bit-identical
    to the default mode's own results (the same kernels on the same values)."""
    import torch
    w = I.make_weights(cfg, 3, gamma_jitter=0.1)
    x, dy = I.make_activations(cfg, 3)
    xd, dyd = U.to_dev(x, cfg.dtype), U.to_dev(dy, cfg.dtype)
    outs = []
    for flags in (0, taw.TAW_RECOMPUTE):
        L = U.DeviceLayer(taw, cfg, flags=flags)
        L.set_weights(w)
        y = L.fwd(xd)
        L.ws.fill_(0x5A)                    # nothing of the forward may survive in the workspace
        dx = L.bwd(xd, dyd)
        torch.cuda.synchronize()
        outs.append((y, dx, L.G.clone()))
    assert taw.taw_layer_ctx_bytes(taw.desc_from_config(cfg, taw.TAW_RECOMPUTE)) == 0
    for a, b in zip(outs[0], outs[1]):
        assert torch.equal(a, b)
    w64 = I.weights_to_f64(w, cfg.dtype)
    from oracle import decoder_layer as O
    yr, cache = O.layer_fwd(w64, I.to_f64(x, cfg.dtype), cfg.n_heads, cfg.rope_theta, cfg.rms_eps)
    dxr, _ = O.layer_bwd(w64, cache, I.to_f64(dy, cfg.dtype))
    assert U.tensor_scale_err(U.from_dev(outs[1][0]), yr) < U.TOL[cfg.dtype]
    assert U.tensor_scale_err(U.from_dev(outs[1][1]), dxr) < U.TOL[cfg.dtype]


@pytest.mark.parametrize("B,S,nh,I_,cuts", [(1, 50, 8, 2816, {"down": 8, "dqkv": 4, "dgate_up": 4}), (3, 111, 8, 2816, {"dqkv": 8, "dgate_up": 2}),
                                            (1, 1, 4, 1000, {"dgate_up": 8}),
                                            (2, 9, 20, 2560, {"qkv": 4, "o": 8, "gate_up": 4, "down": 8, "dqkv": 8, "do": 4, "dgate_up": 8, "ddown": 4})],
                         ids=["50-tokens", "333-tokens", "1-token", "18-tokens-2560-wide"])
def test_bf16_layer_of_few_tokens(taw, B, S, nh, I_, cuts):
    """Few rows against wide weights: contractions are cut into ranges of at least 256, the last one shorter, and summed by the second
    kernel, the down and output projections with their residual, the qkv projection with its rotation (last case, two sequences).
    The rounding of q and k to bf16 moves a score s by up to 2^-8 |s| and a probability by that share: with scores of standard deviation
    sigma_w^2 H, sigma_w = 0.05 is within the tolerance up to H = 1024 (four of them: 4 %, of a few probabilities), 0.02 at H = 2560 (1.6 %)."""
    H = nh * 128
    assert _cuts(taw, B * S, H, I_) == cuts
    U.check_layer(taw, I.LayerConfig("few-tokens", I.BF16, B, S, H, nh, 128, I_, sigma_w=0.05 if H <= 1024 else 0.02), seed=B + S, gamma_jitter=0.1)


def test_bf16_forward_of_few_tokens_at_the_widest(taw):
    """Seven sequences of 11 tokens, 8192 wide: the qkv projection cut into two ranges on 128 x 256 tiles, rotated by the second kernel."""
    from oracle import decoder_layer as O
    cfg = I.LayerConfig("few-tokens-wide", I.BF16, 7, 11, 8192, 64, 128, 136)
    assert _cuts(taw, 77, 8192, 136)["qkv"] == 2 and taw.taw_diag_gemm_plan(0, 77, 3 * 8192, 8192)["tile_n"] == 256
    w = I.make_weights(cfg, 0)
    x, _ = I.make_activations(cfg, 0)
    L = U.DeviceLayer(taw, cfg)
    L.set_weights(w)
    y = U.from_dev(L.fwd(U.to_dev(x, cfg.dtype)))
    yr, _ = O.layer_fwd(I.weights_to_f64(w, cfg.dtype), I.to_f64(x, cfg.dtype), cfg.n_heads, cfg.rope_theta, cfg.rms_eps)
    assert U.tensor_scale_err(y, yr) < U.TOL[cfg.dtype]


@pytest.mark.parametrize("cfg", [I.CONFIGS["C1"], I.LayerConfig("few", I.BF16, 2, 8, 2560, 20, 128, 6912), I.LayerConfig("some", I.BF16, 1, 1024, 1024, 8, 128, 2816)],
                         ids=["fp32", "16-tokens", "1024-tokens"])
def test_forward_leaves_the_shared_workspace_alone(taw, cfg):
    """Without TAW_RECOMPUTE the forward writes its cache and y, nothing else: a backward of another layer may be using the workspace on
    another stream.  With few tokens its contractions are cut, and the partial products have to fit the cache, not overrun it."""
    import torch
    L = U.DeviceLayer(taw, cfg)
    L.set_weights(I.make_weights(cfg, 0))
    x, _ = I.make_activations(cfg, 0)
    n = L.ctx.numel()
    L.ctx = torch.full((n + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    L.ws.fill_(0x5A)
    L.fwd(U.to_dev(x, cfg.dtype))
    torch.cuda.synchronize()
    assert bool((L.ws == 0x5A).all())
    assert bool((L.ctx[n:] == 0x5A).all())


@pytest.mark.parametrize("B,S,nh,d,I_", [(2, 67, 3, 10, 77), (1, 130, 2, 24, 100), (1, 64, 1, 32, 33), (1, 65, 5, 8, 90), (1, 40, 2, 2, 8), (1, 50, 2, 36, 50)])
def test_fp32_layer_head_dims(taw, B, S, nh, d, I_):
    """Narrow heads (up to 32: rows in registers, loaded in pairs or fours) and one just beyond, on products with odd widths, one key more and
    one less than a wavefront, rotation, SwiGLU and both of its backward's halves inside the products."""
    U.check_layer(taw, I.LayerConfig("narrow", I.F32, B, S, nh * d, nh, d, I_, sigma_w=0.2), seed=d, gamma_jitter=0.1)


@pytest.mark.parametrize("dtype,B,S,nh,d,I_", [(I.BF16, 2, 67, 3, 10, 77), (I.BF16, 1, 130, 3, 20, 100), (I.BF16, 1, 65, 5, 8, 91), (I.BF16, 1, 50, 3, 36, 50),
                                               (I.F32, 1, 1100, 33, 32, 1001), (I.BF16, 1, 1100, 33, 30, 1001)], ids=str)
def test_layer_on_generic_products(taw, dtype, B, S, nh, d, I_):
    """bf16 layers with widths no MFMA product takes (H or I no multiple of 8): rotation, SwiGLU and its backward inside the generic products, on
    16 x 16 tiles; and layers whose products have too many of those (4096) for one grid of the two gradients, with SwiGLU's backward on its own.
    Weights of H^-1/2: scores of standard deviation 1, which the rounding of q and k to bf16 moves by about 2^-8 of themselves, 1 - 2 % at most."""
    U.check_layer(taw, I.LayerConfig("generic", dtype, B, S, nh * d, nh, d, I_, sigma_w=(nh * d) ** -0.5), seed=d, gamma_jitter=0.1)


@pytest.mark.parametrize("B,S", [(52, 100), (160, 33), (41, 128), (260, 20), (64, 48)])
def test_short_sequences_across_large_tiles(taw, B, S):
    """Many short sequences in one call: 256 x 256 tiles whose 32-row slices start anywhere in a sequence and cross into the next (the rotation's
    positions wrap inside a tile, at 20 tokens inside a slice more than once), against one sequence at a time on the small tiles.  The two differ in the order of fp32 sums only, so by a bf16
    rounding here and there: h's and y's, 2^-8 of an element each, and through attention and MLP at most about as much again.  In the last case the
    batch (a multiple of 256 tokens) rotates unrounded sums and one sequence rounds q and k first: scores (standard deviation 2.6) move by up to
    2^-8 of themselves, the attention's half of h by up to 4 %."""
    import torch
    mk = lambda b: I.LayerConfig("short", I.BF16, b, S, 1024, 8, 128, 136, sigma_w=0.05)
    assert taw.taw_diag_gemm_plan(0, B * S, 3 * 1024, 1024)["tile_m"] == 256 and taw.taw_diag_gemm_plan(0, S, 3 * 1024, 1024)["tile_m"] == 64
    w = I.make_weights(mk(B), 1)
    x, _ = I.make_activations(mk(B), 1)
    xd = U.to_dev(x, I.BF16)
    many, one = U.DeviceLayer(taw, mk(B)), U.DeviceLayer(taw, mk(1))
    many.set_weights(w)
    one.set_weights(w)
    y = many.fwd(xd).double().reshape(B, S, -1)
    for b in sorted({0, 1, 2, 256 // S, 512 // S, B // 2, B - 1}):
        ref = one.fwd(xd.reshape(B, S, -1)[b:b + 1].contiguous()).double().reshape(S, -1)
        err = float((y[b] - ref).abs().max() / ref.abs().max())
        assert err < (2.0 ** -6 if B * S % 256 else 2.0 ** -5), (b, err)


@pytest.mark.parametrize("dtype,B,S,nh,d,I_", [(I.F32, 2, 67, 3, 10, 77), (I.BF16, 2, 67, 3, 10, 77), (I.BF16, 2, 48, 4, 16, 88), (I.BF16, 2, 333, 2, 128, 392),
                                               (I.BF16, 8, 64, 2, 128, 392)], ids=["fp32", "bf16-generic", "bf16-narrow-heads", "bf16-ragged", "bf16-512-tokens"])
def test_kernel_level_qkv_projection_is_the_layers(taw, dtype, B, S, nh, d, I_):
    """taw_op_qkv_rope on the normalised input that the layer cached gives the cached q, k and v, bit for bit: the same kernels, the same roundings."""
    import torch
    cfg = I.LayerConfig("qkv", dtype, B, S, nh * d, nh, d, I_, sigma_w=0.2)
    L = U.DeviceLayer(taw, cfg)
    w = I.make_weights(cfg, 0)
    L.set_weights(w)
    x, _ = I.make_activations(cfg, 0)
    L.fwd(U.to_dev(x, dtype))
    H, T, tdt = cfg.H, B * S, torch.bfloat16 if dtype == I.BF16 else torch.float32
    e = 2 if dtype == I.BF16 else 4
    up = lambda n: -(-n // 256) * 256                     # the cache holds xn, then qkv, each from a multiple of 256 bytes
    xn = L.ctx[:T * H * e].view(tdt)
    qkv = L.ctx[up(T * H * e):up(T * H * e) + 3 * T * H * e].view(tdt)
    out = torch.empty_like(qkv)
    lo = L.layout["w_qkv"]
    impl = taw.TAW_IMPL_GENERIC if dtype == I.F32 or H % 8 else taw.TAW_IMPL_AUTO
    taw.taw_op_qkv_rope(dtype, B, S, nh, d, xn, L.chunk[lo:lo + 3 * H * H], out, L.rope, impl)
    torch.cuda.synchronize()
    assert torch.equal(out, qkv)


@pytest.mark.parametrize("B,S,H,d,I_", [(1, 4503, 1024, 128, 2816), (1, 16385, 1024, 128, 2816), (1, 16300, 1152, 128, 1152), (1, 8192, 2048, 128, 2816), (32, 512, 1032, 24, 2816)])
def test_gate_up_projection_with_swiglu_in_its_epilogue(taw, B, S, H, d, I_):
    """Where the gate/up product takes 256 x 256 tiles (and I is a multiple of 128) its epilogue stores silu(gate) up too.  The cached gate and up are the
    product's, and the cached a is the separate pass's on them, bit for bit: tiles over the last row, a last step of the contraction that is not whole (the last case), saturated and tiny sigmoids, infinities and NaN."""
    import torch
    T = B * S
    cfg = I.LayerConfig("swi", I.BF16, B, S, H, H // d, d, I_, sigma_w=0.2)
    L = U.DeviceLayer(taw, cfg)
    info = taw.taw_diag_gemm_plan(False, T, 2 * I_, H)
    assert (info["tile_m"], info["tile_n"], info["splits"]) == (256, 256, 1)
    g = torch.Generator(device="cuda").manual_seed(T)
    w = torch.empty(L.layout["total_elems"], device="cuda").normal_(0, 0.05, generator=g)
    lay = L.layout
    w[lay["gamma_attn"]:lay["gamma_attn"] + H] = 1.0
    w[lay["gamma_mlp"]:lay["gamma_mlp"] + H] = 1.0
    gate = w[lay["w_gate_up"]:lay["w_gate_up"] + I_ * H].view(I_, H)
    gate[3::8] *= 60.0                                    # gates of +-100: exp overflows, sigmoids are denormal numbers or 1
    gate[5], gate[6] = float("inf"), float("nan")
    gate[7, 0] = 3e38
    L.chunk = w.bfloat16()
    x = torch.empty(B, S, H, device="cuda").normal_(generator=g).bfloat16()
    L.fwd(x)
    up = lambda n: -(-n // 256) * 256
    at, off = 0, {}
    for name, n in (("xn", H), ("qkv", 3 * H), ("o", H), ("h", H), ("hn", H), ("gu", 2 * I_), ("a", I_)):      # each from a multiple of 256 bytes
        off[name] = L.ctx[at:at + 2 * T * n].view(torch.bfloat16).view(T, n)
        at += up(2 * T * n)
    gu, a = torch.empty_like(off["gu"]), torch.empty_like(off["a"])
    lo = lay["w_gate_up"]
    taw.taw_op_gemm(I.BF16, taw.TAW_GEMM_NT, T, 2 * I_, H, off["hn"], H, L.chunk[lo:lo + 2 * I_ * H], H, gu, 2 * I_, I.BF16, 0, None, 0, taw.TAW_IMPL_MFMA)
    taw.taw_op_swiglu_fwd(I.BF16, T, I_, off["gu"], a)
    torch.cuda.synchronize()
    assert torch.equal(gu.view(torch.int16), off["gu"].view(torch.int16))
    assert torch.equal(a.isnan(), off["a"].isnan())
    assert torch.equal(torch.nan_to_num(a, 0.0), torch.nan_to_num(off["a"], 0.0))
