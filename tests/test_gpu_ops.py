"""Each kernel on its own against the matching step of the oracle, through the C ABI."""
import numpy as np
import pytest

from oracle import decoder_layer as O
from paper_2511_09741_amd import inputs as I
from tests import util as U

pytestmark = pytest.mark.gpu


def draw(rng, shape, dtype, scale=1.0):
    """random values already representable in the storage dtype: (storage array, fp64 values)"""
    a = (scale * rng.standard_normal(shape)).astype(np.float32)
    st = I.to_storage(a, dtype)
    return st, I.to_f64(st, dtype)


GEMM_SHAPES = [(64, 64, 64), (200, 136, 72), (8, 8, 8), (257, 264, 520), (1, 8, 16), (300, 40, 1000)]


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_generic(taw, dtype, mode, M, N, K):
    _gemm_case(taw, dtype, mode, M, N, K, taw.TAW_IMPL_GENERIC, seed=M + N + K + mode)


def _gemm_case(taw, dtype, mode, M, N, K, impl, seed=0, c_f32=False, accumulate=False, residual=False):
    import torch
    rng = np.random.default_rng(seed)
    a_shape = (K, M) if mode == 2 else (M, K)
    b_shape = (N, K) if mode == 0 else (K, N)
    A, A64 = draw(rng, a_shape, dtype)
    B, B64 = draw(rng, b_shape, dtype)
    opA = A64.T if mode == 2 else A64
    opB = B64.T if mode == 0 else B64
    ref = opA @ opB
    c_dtype = I.F32 if c_f32 else dtype
    Cd = U.empty_dev((M, N), c_dtype)
    if accumulate:
        C0, C064 = draw(rng, (M, N), c_dtype, 3.0)
        Cd.copy_(U.to_dev(C0, c_dtype))
        ref = ref + C064
    Rd = None
    if residual:
        R, R64 = draw(rng, (M, N), c_dtype, 2.0)
        Rd = U.to_dev(R, c_dtype)
        ref = ref + R64
    Ad, Bd = U.to_dev(A, dtype), U.to_dev(B, dtype)
    taw.taw_op_gemm(dtype, mode, M, N, K, Ad, a_shape[1], Bd, b_shape[1], Cd, N, c_dtype, int(accumulate), Rd, N, impl)
    torch.cuda.synchronize()
    tol = 2e-2 if (dtype == I.BF16 and not c_f32) else 1e-4
    err = U.tensor_scale_err(U.from_dev(Cd), ref)
    assert err < tol, err
    return err


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
def test_gemm_generic_epilogues(taw, dtype):
    _gemm_case(taw, dtype, 0, 100, 72, 64, taw.TAW_IMPL_GENERIC, residual=True)
    _gemm_case(taw, dtype, 2, 72, 40, 333, taw.TAW_IMPL_GENERIC, c_f32=True, accumulate=True)
    _gemm_case(taw, dtype, 2, 72, 40, 333, taw.TAW_IMPL_GENERIC, c_f32=True, accumulate=False)


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("T,H", [(5, 64), (130, 4096), (33, 100), (7, 1000), (2, 8192 if True else 0), (64, 1022), (65, 1022)])
def test_rmsnorm_fwd_bwd(taw, dtype, T, H):
    import torch
    if dtype == I.F32 and H > 4096:
        H = 4096
    rng = np.random.default_rng(T * H)
    x, x64 = draw(rng, (T, H), dtype)
    g, g64 = draw(rng, (H,), dtype, 0.3)
    g64 = g64 + 1.0
    g = I.to_storage((g64).astype(np.float32), dtype); g64 = I.to_f64(g, dtype)
    dout, dout64 = draw(rng, (T, H), dtype)
    dres, dres64 = draw(rng, (T, H), dtype)
    eps = 1e-6
    xd, gd = U.to_dev(x, dtype), U.to_dev(g, dtype)
    out = U.empty_dev((T, H), dtype)
    r = torch.empty(T, dtype=torch.float32, device="cuda")
    taw.taw_op_rmsnorm_fwd(dtype, T, H, xd, gd, eps, out, r)
    ref, rref = O.rmsnorm_fwd(x64, g64, eps)
    tol = U.TOL[dtype]
    assert U.tensor_scale_err(U.from_dev(out), ref) < tol
    assert U.tensor_scale_err(U.from_dev(r), rref) < 1e-5
    # backward with the oracle's r (fp32-rounded) so the op is tested on its own
    r32 = torch.from_numpy(rref.astype(np.float32)).cuda()
    dz = U.empty_dev((T, H), dtype)
    dgam = torch.full((H,), 5.0, dtype=torch.float32, device="cuda")
    scratch = torch.empty(taw.taw_op_rmsnorm_bwd_scratch_floats(H), dtype=torch.float32, device="cuda")
    taw.taw_op_rmsnorm_bwd(dtype, T, H, U.to_dev(dout, dtype), xd, r32, gd, U.to_dev(dres, dtype), dz, dgam, 1, scratch)
    dzr, dgr = O.rmsnorm_bwd(dout64, x64, rref, g64)
    assert U.tensor_scale_err(U.from_dev(dz), dzr + dres64) < tol
    assert U.tensor_scale_err(U.from_dev(dgam) - 5.0, dgr) < 1e-4
    taw.taw_op_rmsnorm_bwd(dtype, T, H, U.to_dev(dout, dtype), xd, r32, gd, None, dz, dgam, 0, scratch)
    assert U.tensor_scale_err(U.from_dev(dz), dzr) < tol
    assert U.tensor_scale_err(U.from_dev(dgam), dgr) < 1e-4


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("B,S,nh,d", [(2, 33, 3, 16), (1, 300, 2, 128), (1, 5, 2, 6)])
def test_rope_forward_and_inverse(taw, dtype, B, S, nh, d):
    import torch
    rng = np.random.default_rng(S + d)
    H = nh * d
    z, z64 = draw(rng, (B * S, 3 * H), dtype)
    desc = taw.make_desc(dtype, B, S, H, nh, d, 8, 10000.0)
    table = torch.empty(S * (d // 2) * 2, dtype=torch.float32, device="cuda")
    taw.taw_rope_table_init(desc, table)
    phi = O.rope_angles(S, d, 10000.0)
    tab = U.from_dev(table).reshape(S, d // 2, 2)
    assert np.max(np.abs(tab[..., 0] - np.cos(phi))) < 1e-7 and np.max(np.abs(tab[..., 1] - np.sin(phi))) < 1e-7
    zd = U.to_dev(z, dtype)
    taw.taw_op_rope(dtype, B, S, 2 * H, d, zd, 3 * H, table, 0)
    ref = z64.copy()
    for part in range(2):
        blk = z64[:, part * H:(part + 1) * H].reshape(B, S, nh, d)
        ref[:, part * H:(part + 1) * H] = O.rope_apply(blk, phi).reshape(B * S, H)
    got = U.from_dev(zd)
    assert U.tensor_scale_err(got, ref) < (1e-2 if dtype == I.BF16 else 1e-6)
    assert np.array_equal(got[:, 2 * H:], z64[:, 2 * H:])          # v untouched
    taw.taw_op_rope(dtype, B, S, 2 * H, d, zd, 3 * H, table, 1)
    assert U.tensor_scale_err(U.from_dev(zd), z64) < (2e-2 if dtype == I.BF16 else 1e-6)


def test_rope_table_accuracy_at_long_context(taw):
    """Angles up to 32767 rad: the table must stay at fp32 rounding accuracy (fp64 evaluation)."""
    import torch
    S, d = 32768, 128
    desc = taw.make_desc(I.BF16, 1, S, 4096, 32, d, 11008)
    table = torch.empty(S * (d // 2) * 2, dtype=torch.float32, device="cuda")
    taw.taw_rope_table_init(desc, table)
    rows = np.array([0, 1, 1000, 20000, 32767])
    tab = U.from_dev(table).reshape(S, d // 2, 2)[rows]
    phi = O.rope_angles(S, d, 10000.0)[rows]
    assert np.max(np.abs(tab[..., 0] - np.cos(phi))) < 1e-6 and np.max(np.abs(tab[..., 1] - np.sin(phi))) < 1e-6


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("T,I_", [(7, 176), (129, 1000), (3, 11008), (5, 37)])
def test_swiglu_fwd_bwd(taw, dtype, T, I_):
    rng = np.random.default_rng(T + I_)
    gu, gu64 = draw(rng, (T, 2 * I_), dtype, 2.0)
    da, da64 = draw(rng, (T, I_), dtype)
    a = U.empty_dev((T, I_), dtype)
    dgu = U.empty_dev((T, 2 * I_), dtype)
    gud = U.to_dev(gu, dtype)
    taw.taw_op_swiglu_fwd(dtype, T, I_, gud, a)
    taw.taw_op_swiglu_bwd(dtype, T, I_, U.to_dev(da, dtype), gud, dgu)
    g, u = gu64[:, :I_], gu64[:, I_:]
    tol = 1e-2 if dtype == I.BF16 else 1e-5
    assert U.tensor_scale_err(U.from_dev(a), O.swiglu_fwd(g, u)) < tol
    dg, du = O.swiglu_bwd(da64, g, u)
    assert U.tensor_scale_err(U.from_dev(dgu), np.concatenate([dg, du], axis=1)) < tol


def _attn_case(taw, dtype, B, S, nh, d, impl, seed=0, scale=1.0, bwd_impl=None, rotated=False):
    import torch
    rng = np.random.default_rng(seed)
    H = nh * d
    qkv, qkv64 = draw(rng, (B * S, 3 * H), dtype, scale)
    dO, dO64 = draw(rng, (B * S, H), dtype)
    q, k, v = (qkv64[:, i * H:(i + 1) * H].reshape(B, S, nh, d) for i in range(3))
    oref = O.attention_fwd(q, k, v)
    qkvd = U.to_dev(qkv, dtype)
    o = U.empty_dev((B * S, H), dtype)
    lse = torch.empty(B * nh * S, dtype=torch.float32, device="cuda")
    taw.taw_op_attn_fwd(dtype, B, S, nh, d, qkvd, o, lse, impl)
    tol = U.TOL[dtype]
    e_o = U.tensor_scale_err(U.from_dev(o), oref.reshape(B * S, H))
    # log-sum-exp of the scaled scores: the oracle's own (pinned) row-wise form, every row of every head
    lref = np.empty((B, nh, S))
    for b in range(B):
        for h in range(nh):
            _, lref[b, h] = O.attention_fwd_rows(q[b, :, h], k[b, :, h], v[b, :, h], np.arange(S))
    e_l = float(np.max(np.abs(U.from_dev(lse).reshape(B, nh, S) - lref)))
    # backward from the stored (storage-rounded) forward output of the oracle, so bwd is tested on its own
    o_st = I.to_storage(oref.reshape(B * S, H).astype(np.float32), dtype)
    o64 = I.to_f64(o_st, dtype).reshape(B, S, nh, d)
    dq, dk, dv = O.attention_bwd(q, k, v, o64, dO64.reshape(B, S, nh, d))
    dref = np.concatenate([dq.reshape(B * S, H), dk.reshape(B * S, H), dv.reshape(B * S, H)], axis=1)
    lse_ref32 = torch.from_numpy(lref.astype(np.float32).reshape(-1)).cuda()
    dqkv = U.empty_dev((B * S, 3 * H), dtype)
    scratch = torch.full((taw.taw_op_attn_bwd_scratch_floats(B, S, nh),), float("nan"), dtype=torch.float32, device="cuda")
    table = None
    if rotated:                                        # the gradients of q, k before their rotation
        table = torch.empty(S * d, dtype=torch.float32, device="cuda")
        taw.taw_rope_table_init(taw.make_desc(dtype, B, S, H, nh, d, 8), table)
        phi = O.rope_angles(S, d, 10000.0)
        for i, z in enumerate((dq, dk)):
            dref[:, i * H:(i + 1) * H] = O.rope_apply(z, phi, inverse=True).reshape(B * S, H)
    taw.taw_op_attn_bwd(dtype, B, S, nh, d, qkvd, U.to_dev(o_st, dtype), U.to_dev(dO, dtype), lse_ref32, dqkv, scratch, table, impl if bwd_impl is None else bwd_impl)
    got = U.from_dev(dqkv)
    # at S = 1 the exact dq and dk are identically zero: measure them on the scale of dv
    fl = 1e-3 * float(np.max(np.abs(dref[:, 2 * H:])))
    e_dq = U.tensor_scale_err(got[:, :H], dref[:, :H], floor=fl)
    e_dk = U.tensor_scale_err(got[:, H:2 * H], dref[:, H:2 * H], floor=fl)
    e_dv = U.tensor_scale_err(got[:, 2 * H:], dref[:, 2 * H:])
    print(f"attn dtype={dtype} B={B} S={S} nh={nh} d={d} impl={impl}: o={e_o:.2e} lse={e_l:.2e} dq={e_dq:.2e} dk={e_dk:.2e} dv={e_dv:.2e}", flush=True)
    assert e_o < tol and e_l < (2e-2 if dtype == I.BF16 else 1e-4)
    assert e_dq < tol and e_dk < tol and e_dv < tol


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("B,S,nh,d", [(1, 128, 4, 16), (2, 67, 3, 8), (1, 1, 2, 16), (1, 130, 1, 128), (1, 40, 2, 2), (2, 65, 3, 18), (1, 70, 5, 30), (1, 200, 1, 32)])
def test_attention_generic(taw, dtype, B, S, nh, d):
    _attn_case(taw, dtype, B, S, nh, d, taw.TAW_IMPL_GENERIC, seed=S)


@pytest.mark.parametrize("d", [6, 8, 16, 32, 36])
def test_attention_generic_scores_that_overflow(taw, d):
    """Finite q and k whose scores overflow fp32 to -inf: such a key has weight 0, first in its lane or not, as long as the row has one
    finite score.  Keys 0 - 3, 64 and 70 are anti-parallel to every later query at 1e20 each; the rest of the row is ordinary."""
    import torch
    S, nh = 140, 2
    H = nh * d
    rng = np.random.default_rng(d)
    qkv, _ = draw(rng, (S, 3 * H), I.F32)
    far = [0, 1, 2, 3, 64, 70]
    q, k = qkv[:, :H].reshape(S, nh, d), qkv[:, H:2 * H].reshape(S, nh, d)
    q[:, :, 0] = 1e20
    k[:, :, 0] = 0.0
    k[far, :, 0] = -1e20
    q[far, :, 0] = 0.0                                  # their own scores stay finite
    o = U.empty_dev((S, H), I.F32)
    lse = torch.empty(nh * S, dtype=torch.float32, device="cuda")
    taw.taw_op_attn_fwd(I.F32, 1, S, nh, d, U.to_dev(qkv, I.F32), o, lse, taw.TAW_IMPL_GENERIC)
    got_o, got_lse = U.from_dev(o).reshape(S, nh, d), U.from_dev(lse).reshape(nh, S)
    v = qkv[:, 2 * H:].reshape(S, nh, d).astype(np.float64)
    for h in range(nh):
        for t in range(S):
            s = q[t, h].astype(np.float64) @ k[:t + 1, h].astype(np.float64).T / np.sqrt(d)
            s[s < -np.finfo(np.float32).max] = -np.inf
            if not np.isfinite(s).any():
                continue                                # no key left: 0 / 0
            m = s.max()
            p = np.exp(s - m)
            assert abs(got_lse[h, t] - (m + np.log(p.sum()))) < 1e-4, (h, t)
            assert np.max(np.abs(got_o[t, h] - p @ v[:t + 1, h] / p.sum())) < 1e-4, (h, t)


def test_attention_generic_of_very_many_rows(taw):
    """2^25 rows (batch x heads x positions): one wavefront each is half of the 2^32 work-items a launch takes along x.  A batch of repeated pairs of
    sequences equals the pair, bit for bit."""
    import torch
    B, S, nh, d = 16384, 64, 32, 2
    H = nh * d
    g = torch.Generator(device="cuda").manual_seed(0)
    qkv, dO = (torch.empty(2, S, n, device="cuda").normal_(generator=g) for n in (3 * H, H))

    def both(qkv, dO):
        b = qkv.shape[0]
        o, dqkv = torch.empty_like(dO), torch.empty_like(qkv)
        lse, scratch = (torch.empty(b * nh * S, dtype=torch.float32, device="cuda") for _ in range(2))
        taw.taw_op_attn_fwd(I.F32, b, S, nh, d, qkv, o, lse, taw.TAW_IMPL_GENERIC)
        taw.taw_op_attn_bwd(I.F32, b, S, nh, d, qkv, o, dO, lse, dqkv, scratch, None, taw.TAW_IMPL_GENERIC)
        return o, dqkv

    for a, b in zip(both(qkv, dO), both(qkv.repeat(B // 2, 1, 1), dO.repeat(B // 2, 1, 1))):
        assert torch.equal(a.expand(B // 2, *a.shape), b.view(B // 2, *a.shape))


@pytest.mark.parametrize("src_dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("n", [0, 1, 3, 4, 1027, 13490, 1 << 20])      # 13490: whole workgroups, a partly filled one and a scalar tail
def test_grad_accum(taw, src_dtype, n):
    import torch
    rng = np.random.default_rng(n + 1)
    G0 = rng.standard_normal(n + 8).astype(np.float32)
    g, g64 = draw(rng, (n + 8,), src_dtype)
    Gd = torch.from_numpy(G0.copy()).cuda()
    taw.taw_grad_accum(Gd, U.to_dev(g, src_dtype), src_dtype, n, 0.25)
    got = U.from_dev(Gd)
    ref = O.grad_accum(G0[:n].astype(np.float64), g64[:n], 0.25)
    assert np.max(np.abs(got[:n] - ref), initial=0.0) < 1e-6
    assert np.array_equal(got[n:], G0[n:].astype(np.float64))        # nothing past n_elems is touched


def test_weight_stage_double_buffer(taw):
    """Chunks staged on a side stream, ordered against the compute stream by the two events."""
    import torch
    n = 1 << 22
    shards = [torch.full((n,), float(j + 1), dtype=torch.float32, device="cuda") for j in range(4)]
    bufs = [torch.zeros(n, dtype=torch.float32, device="cuda") for _ in range(2)]
    sums = torch.zeros(4, dtype=torch.float32, device="cuda")
    copy_stream = torch.cuda.Stream()
    compute = torch.cuda.current_stream()
    ready = [torch.cuda.Event() for _ in range(2)]
    consumed = [torch.cuda.Event() for _ in range(2)]
    torch.cuda.synchronize()
    taw.taw_weight_stage(bufs[0], shards[0], n * 4, copy_stream, None, ready[0])
    for j in range(4):
        if j + 1 < 4:
            nb = (j + 1) & 1
            taw.taw_weight_stage(bufs[nb], shards[j + 1], n * 4, copy_stream, consumed[nb] if j >= 1 else None, ready[nb])
        compute.wait_event(ready[j & 1])
        sums[j] = bufs[j & 1].sum() / n          # "the layer" reads its weights
        consumed[j & 1].record(compute)
    torch.cuda.synchronize()
    assert sums.cpu().tolist() == [1.0, 2.0, 3.0, 4.0]
    taw.taw_weight_stage(None, None, 0, copy_stream, None, ready[0])   # bytes == 0 only handles the events
    torch.cuda.synchronize()


# ----------------------------------------------------------------------------- MFMA kernels (bf16)
# 1, 2, 3 and many steps of K (64 deep), the last one whole or not.  NT with bf16 results takes the tile its
# plan names, everything else 256 x 256
MFMA_GEMM_SHAPES = {
    0: [(256, 256, 64), (8, 8, 8), (300, 520, 136), (257, 263, 72), (1000, 264, 4104), (512, 768, 1024), (1, 3, 8),
        (300, 520, 96), (257, 263, 128), (264, 520, 192), (300, 264, 160), (1000, 264, 4096), (5, 3, 32)],
    1: [(256, 256, 64), (8, 8, 8), (300, 520, 136), (257, 264, 72), (1000, 264, 4104), (512, 768, 1024), (1, 8, 8),
        (300, 520, 96), (257, 264, 128), (264, 520, 192), (300, 264, 160), (1000, 264, 4096), (5, 8, 32)],
    2: [(256, 256, 64), (8, 8, 8), (304, 520, 133), (264, 256, 77), (1000, 264, 4100), (512, 768, 1024), (8, 8, 1),
        (304, 520, 96), (264, 256, 128), (264, 520, 192), (304, 264, 160), (1000, 264, 4096), (8, 8, 32)],
}


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_gemm_mfma_shapes(taw, mode):
    """Several tiles, ragged tails in M, N and K, and degenerate sizes; bf16 output."""
    for (M, N, K) in MFMA_GEMM_SHAPES[mode]:
        err = _gemm_case(taw, I.BF16, mode, M, N, K, taw.TAW_IMPL_MFMA, seed=M + N + K)
        print(f"mfma gemm mode={mode} {M}x{N}x{K}: err={err:.2e}", flush=True)


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_gemm_mfma_epilogues(taw, mode):
    for shp in ((520, 264, 200) if mode != 2 else (520, 264, 203), (520, 264, 192), (520, 264, 160)):   # a last step of 8 (TN: 11), 64 and 32
        _gemm_case(taw, I.BF16, mode, *shp, taw.TAW_IMPL_MFMA, residual=True)
        _gemm_case(taw, I.BF16, mode, *shp, taw.TAW_IMPL_MFMA, c_f32=True)
        _gemm_case(taw, I.BF16, mode, *shp, taw.TAW_IMPL_MFMA, c_f32=True, accumulate=True)
        _gemm_case(taw, I.BF16, mode, *shp, taw.TAW_IMPL_MFMA, c_f32=True, accumulate=True, residual=True)


def test_gemm_mfma_fp32_output_is_accurate(taw):
    """With fp32 output the only error left is the accumulation order: far below bf16 rounding."""
    for mode in (0, 1, 2):
        err = _gemm_case(taw, I.BF16, mode, 264, 512, 2048, taw.TAW_IMPL_MFMA, c_f32=True, seed=mode)
        assert err < 2e-6, (mode, err)


# the forms of the MFMA backward: the split dK/dV + dQ pair, fused with private dQ slots, fused with atomics, and the split
# pair whose dK/dV kernel stores dS for the dQ kernel
BWD_FORMS = {"split": 2, "fused": 3, "atomic": 4, "stored": 5}


@pytest.mark.parametrize("form", list(BWD_FORMS))
@pytest.mark.parametrize("B,S,nh", [(1, 64, 1), (1, 256, 2), (2, 333, 2), (1, 1, 1), (1, 1000, 1), (1, 130, 3), (1, 2081, 2), (3, 520, 1), (4, 2304, 16)])
def test_attention_mfma(taw, B, S, nh, form):
    """Tiled online-softmax kernels: several query/key tiles, ragged S, S = 1, more than one head and batch; every
    form of the backward (2081 keys: nine key blocks dealt to several workers per head in the fused form, each adding
    into its slot more than once; 520: a last query block with rows beyond the sequence; 4 x 16 heads x 2304: four workers per head with up to three key blocks each)."""
    _attn_case(taw, I.BF16, B, S, nh, 128, taw.TAW_IMPL_MFMA, seed=S + nh, bwd_impl=BWD_FORMS[form])


@pytest.mark.parametrize("form", list(BWD_FORMS))
def test_attention_mfma_peaked_scores(taw, form):
    """Scores of order 10: the running maximum moves a lot between key tiles."""
    _attn_case(taw, I.BF16, 1, 700, 2, 128, taw.TAW_IMPL_MFMA, seed=9, scale=3.0, bwd_impl=BWD_FORMS[form])


@pytest.mark.parametrize("B", [1, 75])                    # 128-row workgroups of 4 wavefronts; 256-row ones of 8
@pytest.mark.parametrize("quarter", [0, 1, 2, 3])
@pytest.mark.parametrize("rise", [5.0, 7.9, 12.0, 150.0])
def test_attention_mfma_maximum_raised_by_one_quarter(taw, B, quarter, rise):
    """A row's scores of a key tile lie in four lanes, keys 4 q ... 4 q + 3 of every 16 in quarter q.  Here only one quarter's lie above the running maximum:
    by `rise` (log2) more in every tile, so it is raised in none, some or all of them.  Probabilities are rounded to bf16 (2^-9 of each) in
    the sum as in the product, and the result once more: |o - exact| <= 3 * 2^-9 max |v|, and |lse - exact| <= 2^-8."""
    import torch
    S, nh, d = 333, 4, 128
    H = nh * d
    g = torch.Generator(device="cuda").manual_seed(quarter)
    qkv = torch.empty(B, S, 3, nh, d, device="cuda").normal_(0.0, 0.1, generator=g)
    qkv[:, :, 2].normal_(0.0, 1.0, generator=g)
    kv = torch.arange(S, device="cuda")
    qkv[:, :, 0, :, 0] = 1.0
    up = torch.where((kv // 4 % 4 == quarter) & (kv % 4 == 1), (kv // 64 + 1.0) * rise * d ** 0.5 * np.log(2.0), 0.0)
    qkv[:, :, 1, :, 0] = up[None, :, None]
    qkv = qkv.bfloat16()
    o = torch.full((B, S, H), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((B, nh, S), float("nan"), dtype=torch.float32, device="cuda")
    taw.taw_op_attn_fwd(I.BF16, B, S, nh, d, qkv, o, lse, taw.TAW_IMPL_MFMA)
    q, k, v = qkv.double().permute(2, 0, 3, 1, 4).contiguous()
    scores = (q @ k.transpose(-1, -2).contiguous()) * d ** -0.5
    scores.masked_fill_(kv[None, :] > kv[:, None], -float("inf"))
    ref = (torch.softmax(scores, -1) @ v).permute(0, 2, 1, 3).reshape(B, S, H)
    assert float((o.double() - ref).abs().max()) <= 3 * 2.0 ** -9 * float(v.abs().max())
    assert float((lse.double() - torch.logsumexp(scores, -1)).abs().max()) <= 2.0 ** -8


@pytest.mark.parametrize("form,B,S,nh,shape", [("fused", 2, 1500, 3, None), ("stored", 2, 1500, 3, (64, 4, 1)),      # one grid: nothing stored
                                               ("stored", 1, 1100, 15, (64, 4, 0)), ("stored", 1, 1100, 29, (128, 2, 0)), ("stored", 1, 600, 52, (128, 1, 0)),
                                               ("stored", 2, 700, 45, (256, 1, 0))])
def test_attention_backward_forms_without_atomics_are_reproducible(taw, form, B, S, nh, shape):
    """The fused backward with slots adds its dQ partial sums in a fixed order, and the form with stored dS reads back only
    what it wrote: runs over scratch with different stale contents give the same bits."""
    import torch
    d = 128
    H = nh * d
    assert shape is None or tuple(taw.taw_diag_attn_shape(1, B, S, nh).values()) == shape
    qkv = I.device_normal((B * S, 3 * H), seed=5, std=0.7)
    dO = I.device_normal((B * S, H), seed=6, std=1.0)
    o = torch.empty((B * S, H), dtype=torch.bfloat16, device="cuda")
    lse = torch.empty(B * nh * S, dtype=torch.float32, device="cuda")
    taw.taw_op_attn_fwd(I.BF16, B, S, nh, d, qkv, o, lse, taw.TAW_IMPL_MFMA)
    outs = []
    for fill in (0.0, 1e30, float("nan")):
        scratch = torch.full((taw.taw_op_attn_bwd_scratch_floats(B, S, nh),), fill, dtype=torch.float32, device="cuda")   # stale contents must not matter
        dqkv = torch.full_like(qkv, fill)
        taw.taw_op_attn_bwd(I.BF16, B, S, nh, d, qkv, o, dO, lse, dqkv, scratch, None, BWD_FORMS[form])
        torch.cuda.synchronize()
        outs.append(dqkv)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("n", [1, 7, 4096, 4499, 1 << 20])           # 4499: whole workgroups, a partly filled one and a scalar tail
def test_optimizer_step(taw, dtype, n):
    """Three AdamW steps over a shard against the oracle: master weights, both moments, the chunk in its
    storage type, and the zeroed gradient shard."""
    import torch
    rng = np.random.default_rng(n)
    w = rng.standard_normal(n).astype(np.float32)
    master = torch.from_numpy(w.copy()).cuda()
    m = torch.zeros(n, dtype=torch.float32, device="cuda")
    v = torch.zeros(n, dtype=torch.float32, device="cuda")
    chunk = U.empty_dev((n,), dtype)
    w64, m64, v64 = w.astype(np.float64), np.zeros(n), np.zeros(n)
    hp = dict(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-6, weight_decay=0.1, grad_scale=0.25)
    for t in range(1, 4):
        g = rng.standard_normal(n).astype(np.float32)
        G = torch.from_numpy(g.copy()).cuda()
        taw.taw_optimizer_step(chunk, dtype, master, m, v, G, n, t, zero_grad=(t == 3), **hp)
        w64, m64, v64 = O.adamw_step(w64, m64, v64, g.astype(np.float64), t, hp["lr"], hp["beta1"], hp["beta2"], hp["eps"],
                                     hp["weight_decay"], hp["grad_scale"])
        torch.cuda.synchronize()
        assert torch.count_nonzero(G).item() == (0 if t == 3 else np.count_nonzero(g))
    assert U.tensor_scale_err(U.from_dev(master), w64) < 1e-6
    assert U.tensor_scale_err(U.from_dev(m), m64) < 1e-6 and U.tensor_scale_err(U.from_dev(v), v64) < 1e-6
    assert U.tensor_scale_err(U.from_dev(chunk), w64) < (4e-3 if dtype == I.BF16 else 1e-6)
    if dtype == I.BF16:   # the chunk is exactly the master weights rounded to bf16
        assert np.array_equal(I.to_storage(master.cpu().numpy(), dtype), chunk.view(torch.int16).cpu().numpy().view(np.uint16))


@pytest.mark.parametrize("dtype,n", [(I.BF16, (1 << 27) + 2050), (I.BF16, (136 << 20) + 2050), (I.F32, (1 << 26) + 1027)], ids=["bf16", "bf16-272MiB", "fp32"])
def test_optimizer_step_on_a_chunk_past_the_cache(taw, dtype, n):
    """A bf16 chunk of more than 272 MiB is stored past the caches, a row of 256 x 16 bytes to a workgroup: the first and last elements against the oracle (bounds as in
    test_optimizer_step), and the whole of it against the same update of its halves, which take the other way: the same bits in every array."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(n)
    w, m, v, G = (torch.empty(n, device="cuda").normal_(0, s, generator=gen) for s in (1.0, 0.1, 0.1, 1.0))
    v.square_()
    tdt = torch.bfloat16 if dtype == I.BF16 else torch.float32
    hp = dict(lr=1e-2, beta1=0.9, beta2=0.95, eps=1e-6, weight_decay=0.1, grad_scale=0.25)
    at = torch.cat([torch.arange(4100), torch.arange(n - 4100, n)]).cuda()
    before = [x[at].double().cpu().numpy() for x in (w, m, v, G)]
    halves = [x.clone() for x in (w, m, v, G)] + [torch.empty(n, dtype=tdt, device="cuda")]
    chunk = torch.empty(n, dtype=tdt, device="cuda")
    taw.taw_optimizer_step(chunk, dtype, w, m, v, G, n, 3, zero_grad=True, **hp)
    cut = n // 2 // 1024 * 1024
    for lo, hi in ((0, cut), (cut, n)):
        hw, hm, hv, hG, hc = (x[lo:hi] for x in halves)
        taw.taw_optimizer_step(hc, dtype, hw, hm, hv, hG, hi - lo, 3, zero_grad=True, **hp)
    torch.cuda.synchronize()
    for x, y in zip((w, m, v, G, chunk), halves):
        assert torch.equal(x, y)
    ref = O.adamw_step(*before, 3, hp["lr"], hp["beta1"], hp["beta2"], hp["eps"], hp["weight_decay"], hp["grad_scale"])
    for x, r in zip((w, m, v), ref):
        assert U.tensor_scale_err(x[at].double().cpu().numpy(), r) < 1e-6
    assert torch.count_nonzero(G).item() == 0 and torch.equal(chunk, w.to(tdt))


@pytest.mark.parametrize("mode,f32,M,N", [(0, 1, 300, 264), (0, 1, 257, 263), (0, 1, 129, 130), (1, 0, 300, 264), (1, 0, 385, 520), (1, 1, 513, 8), (2, 0, 264, 136),
                                          (2, 1, 8, 392)])
@pytest.mark.parametrize("pad", [0, 8, 3])
def test_gemm_mfma_edges_of_large_tiles(taw, mode, f32, M, N, pad):
    """256 x 256 tiles that reach over the edge of C by rows, by columns, by whole wavefronts' blocks; results and residuals inside larger matrices with
    aligned and unaligned rows, nothing outside them touched.  Bounds as in test_linear_tile_shapes."""
    import torch
    K, dt = 136, torch.float32 if f32 else torch.bfloat16
    A, B = (I.device_normal(s, seed=i, std=1.0) for i, s in enumerate(((K, M) if mode == 2 else (M, K), (N, K) if mode == 0 else (K, N))))
    ref = (A.double().t() if mode == 2 else A.double()) @ (B.double().t() if mode == 0 else B.double())
    for residual, acc in ((0, 0), (1, 0), (0, 1), (1, 1)):
        C = torch.full((M + 2, N + pad), 7.0, dtype=dt, device="cuda")
        R = I.device_normal((M, N + pad), seed=5, std=1.0, dtype=dt) if residual else None
        taw.taw_op_gemm(I.BF16, mode, M, N, K, A, A.shape[1], B, B.shape[1], C, N + pad, I.F32 if f32 else I.BF16, acc, R, N + pad, taw.TAW_IMPL_MFMA)
        want = ref + 7.0 * acc + (R[:, :N].double() if residual else 0.0)
        err = float((C[:M, :N].double() - want).abs().max() / want.abs().max())
        assert err < (2e-6 if f32 else 2.0 ** -8), (residual, acc, err)
        assert bool((C[M:] == 7).all()) and bool((C[:, N:] == 7).all())


@pytest.mark.parametrize("M,N", [(1, 1), (63, 8), (65, 24), (33, 40), (129, 130), (70, 63), (66, 263)])
@pytest.mark.parametrize("pad", [0, 8, 3])
def test_gemm_mfma_edges_of_small_tiles(taw, M, N, pad):
    """64 x 64 tiles are stored from the accumulators, 8 columns of bf16 from a lane and a line from a pair of lanes: results that end inside a lane's columns,
    a pair's and a group of 32, with aligned and unaligned rows; nothing outside them touched.  Bounds as in test_linear_tile_shapes."""
    import torch
    K = 136
    p = taw.taw_diag_gemm_plan(0, M, N, K)
    assert (p["tile_m"], p["tile_n"]) == (64, 64)
    A, B = I.device_normal((M, K), seed=1, std=1.0), I.device_normal((N, K), seed=2, std=1.0)
    ref = A.double() @ B.double().t()
    for residual, acc in ((0, 0), (1, 0), (0, 1), (1, 1)):
        C = torch.full((M + 2, N + pad), 7.0, dtype=torch.bfloat16, device="cuda")
        R = I.device_normal((M, N + pad), seed=5, std=1.0) if residual else None
        taw.taw_op_gemm(I.BF16, 0, M, N, K, A, K, B, K, C, N + pad, I.BF16, acc, R, N + pad, taw.TAW_IMPL_MFMA)
        want = ref + 7.0 * acc + (R[:, :N].double() if residual else 0.0)
        err = float((C[:M, :N].double() - want).abs().max() / want.abs().max())
        assert err < 2.0 ** -8, (residual, acc, err)
        assert bool((C[M:] == 7).all()) and bool((C[:, N:] == 7).all())


# every tile shape (rows, columns, stages of its ring) of the product and of its backward, each with remainders in rows, columns and contraction:
# less than one step, a whole one, one more
S64, S128D, S128, S192, S256 = (64, 64, 4), (128, 128, 2), (128, 128, 4), (128, 256, 3), (256, 256, 2)


@pytest.mark.parametrize("T,N,K,fwd,bwd", [(1, 8, 8, S64, S64), (65, 72, 8, S64, S64), (333, 264, 136, S64, S64), (2100, 2056, 264, S128D, S64),
                                           (1501, 1032, 1032, S64, S128), (1000, 4104, 2056, S192, S192), (2050, 2056, 2056, S192, S256),
                                           (333, 6152, 136, S128, S64), (1300, 6152, 72, S256, S64), (777, 520, 3080, S64, S128D)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_linear_tile_shapes(taw, T, N, K, fwd, bwd):
    """y = x W^T (+ residual) and its backward at every tile shape against fp64 products of the same bf16 operands.  bf16 results: one
    rounding, 2^-9 of the element, so below 2^-8 of the tensor's scale; fp32 ones: accumulation order only, as in
    test_gemm_mfma_fp32_output_is_accurate.  The weight gradient starts from values it has to keep or to forget."""
    for backward, want in ((0, fwd), (1, bwd)):
        p = taw.taw_diag_gemm_plan(backward, T, N, K)
        assert (p["tile_m"], p["tile_n"], p["stages"]) == want, (backward, p)
    import torch
    x, W, dy = (I.device_normal(s, seed=i, std=d) for i, (s, d) in enumerate((((T, K), 1.0), ((N, K), 0.02), ((T, N), 1.0))))
    R = I.device_normal((T, N), seed=9, std=1.0)
    y = torch.full((T, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    taw.taw_op_gemm(I.BF16, 0, T, N, K, x, K, W, K, y, N, I.BF16, 0, R, N, taw.TAW_IMPL_MFMA)
    x64, W64, dy64 = x.double(), W.double(), dy.double()
    refs = {"y": (y, x64 @ W64.t() + R.double(), 2.0 ** -8)}
    n_scr = taw.taw_op_linear_bwd_scratch_floats(T, N, K)
    scratch = torch.full((n_scr,), float("nan"), dtype=torch.float32, device="cuda") if n_scr else None
    G0 = I.device_normal((N, K), seed=11, std=1.0, dtype=torch.float32)
    for acc in (0, 1):
        dx = torch.full((T, K), float("nan"), dtype=torch.bfloat16, device="cuda")
        G = G0.clone()
        taw.taw_op_linear_bwd(I.BF16, T, N, K, dy, W, x, dx, G, acc, taw.TAW_IMPL_MFMA, scratch=scratch)
        refs[f"dx{acc}"] = (dx, dy64 @ W64, 2.0 ** -8)
        refs[f"G{acc}"] = (G, dy64.t() @ x64 + acc * G0.double(), 2e-6)
    torch.cuda.synchronize()
    for k, (got, ref, tol) in refs.items():
        err = float((got.double() - ref).abs().max() / ref.abs().max())
        assert err < tol, (k, err)


# cut contractions of a linear's backward on every tile shape: the input gradient's (ranges of N), the weight gradient's (of T), both
@pytest.mark.parametrize("T,N,K,tile,cut_dx,cut_g", [(16, 2056, 72, S64, 4, 1), (520, 4104, 520, S128D, 8, 1), (777, 4104, 264, S128, 4, 1),
                                                     (1030, 5640, 520, S192, 4, 1), (1030, 2056, 2824, S256, 2, 1), (2050, 72, 72, S64, 1, 4),
                                                     (4100, 520, 520, S128D, 1, 8), (4100, 1032, 264, S128, 1, 4), (4100, 520, 2056, S192, 1, 2),
                                                     (2050, 1032, 2824, S256, 1, 2), (600, 2056, 8, S64, 4, 2)], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_linear_backward_cut_contractions(taw, T, N, K, tile, cut_dx, cut_g):
    """Both gradients against fp64 products of the same bf16 operands (bounds as in test_linear_tile_shapes), over scratch with stale contents, with
    the last range ragged; and against the call without scratch, which cuts nothing: fp32 sums in another order, so G by a few 2^-24 of
    what was summed and dx by a bf16 rounding here and there."""
    import torch
    p = taw.taw_diag_gemm_plan(1, T, N, K)
    assert ((p["tile_m"], p["tile_n"], p["stages"]), p["splits_dx"], p["splits"]) == (tile, cut_dx, cut_g)
    x, W, dy = (I.device_normal(s, seed=i, std=d) for i, (s, d) in enumerate((((T, K), 1.0), ((N, K), 0.02), ((T, N), 1.0))))
    G0 = I.device_normal((N, K), seed=11, std=1.0, dtype=torch.float32)
    n_scr = taw.taw_op_linear_bwd_scratch_floats(T, N, K)
    assert n_scr == p["scratch_floats"] > 0
    scratch = torch.full((n_scr + 1024,), float("nan"), dtype=torch.float32, device="cuda")
    got = {}
    for scr in (scratch, None):
        dx, G = torch.full((T, K), float("nan"), dtype=torch.bfloat16, device="cuda"), G0.clone()
        taw.taw_op_linear_bwd(I.BF16, T, N, K, dy, W, x, dx, G, 1, taw.TAW_IMPL_MFMA, scratch=scr)
        got[scr is None] = dx.double(), G.double()
    torch.cuda.synchronize()
    assert bool(scratch[n_scr:].isnan().all()) and not bool(scratch[:n_scr].isnan().any())
    refs = dy.double() @ W.double(), dy.double().t() @ x.double() + G0.double()
    for a, b, ref, tol in zip(got[False], got[True], refs, (2.0 ** -8, 2e-6)):
        scale = float(ref.abs().max())
        assert float((a - ref).abs().max()) < tol * scale and float((a - b).abs().max()) < tol * scale


@pytest.mark.parametrize("dtype", [I.F32, I.BF16])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_gemm_generic_large_tiles(taw, dtype, mode):
    """More than 2048 tiles of 16 x 16: the generic product takes 64 x 64 ones, ragged at every edge and in K, the result's last column or row alone
    or one of a pair (operands contiguous along it are loaded in pairs)."""
    _gemm_case(taw, dtype, mode, 1025, 1089, 131, taw.TAW_IMPL_GENERIC)
    _gemm_case(taw, dtype, mode, 1026, 1090, 13, taw.TAW_IMPL_GENERIC)
    _gemm_case(taw, dtype, mode, 650, 641, 100, taw.TAW_IMPL_GENERIC)          # 1681 tiles: 64 x 64 up to K = 128, split beyond
    _gemm_case(taw, dtype, mode, 650, 641, 129, taw.TAW_IMPL_GENERIC)
    _gemm_case(taw, dtype, mode, 1, 40000, 17, taw.TAW_IMPL_GENERIC)          # a single row or column has no pair
    _gemm_case(taw, dtype, mode, 40000, 1, 17, taw.TAW_IMPL_GENERIC)
    _gemm_case(taw, dtype, mode, 40001, 2, 5, taw.TAW_IMPL_GENERIC)
    _gemm_case(taw, dtype, mode, 1030, 1051, 70, taw.TAW_IMPL_GENERIC, residual=True)
    _gemm_case(taw, dtype, mode, 1030, 1052, 33, taw.TAW_IMPL_GENERIC, c_f32=True, accumulate=True)


@pytest.mark.parametrize("S", [1, 64, 65, 128, 129, 257, 333, 385, 640])
def test_attn_mfma_few_and_many_tiles_agree(taw, S):
    """Few tiles run on 128-row workgroups of 4 wavefronts, many on 256-row workgroups of 8.  A wavefront does the same arithmetic in the same
    order in both, so a batch of many sequences has to equal its sequences one by one, bit for bit."""
    import torch
    nh, B = 4, -(-600 // (4 * ((S + 255) // 256)))
    H = nh * 128
    g = torch.Generator(device="cuda").manual_seed(S)
    draw = lambda *shape: torch.empty(shape, device="cuda").normal_(generator=g).bfloat16()
    qkv, dO = draw(B, S, 3 * H), draw(B, S, H)

    def both(qkv, dO):
        b = qkv.shape[0]
        o, dqkv = torch.empty_like(dO), torch.empty_like(qkv)
        lse = torch.empty(b * nh * S, dtype=torch.float32, device="cuda")
        taw.taw_op_attn_fwd(I.BF16, b, S, nh, 128, qkv, o, lse, taw.TAW_IMPL_MFMA)
        scratch = torch.full((taw.taw_op_attn_bwd_scratch_floats(b, S, nh),), float("nan"), dtype=torch.float32, device="cuda")
        taw.taw_op_attn_bwd(I.BF16, b, S, nh, 128, qkv, o, dO, lse, dqkv, scratch, None, taw.TAW_IMPL_MFMA_STORED)
        return o, lse.view(b, -1), dqkv

    many = both(qkv, dO)
    for i in (0, B // 2, B - 1):
        for a, b in zip(both(qkv[i:i + 1].contiguous(), dO[i:i + 1].contiguous()), many):
            assert torch.equal(a[0], b[i])


@pytest.mark.parametrize("B,S,nh", [(1, 700, 47), (1, 1024, 33), (3, 320, 7)])
def test_attn_mfma_pairs_that_the_xcds_do_not_divide(taw, B, S, nh):
    """(batch, head) pairs beyond the last multiple of 8 are dealt out tile by tile, in front of the others: every tile of every pair is done once."""
    _attn_case(taw, I.BF16, B, S, nh, 128, taw.TAW_IMPL_MFMA, seed=S, bwd_impl=taw.TAW_IMPL_MFMA_STORED)


# shapes of the workgroups (rows, parts of a row's sum) and of the backward (both kernels in one grid, nothing stored): all that there are
F256, F128, F128P, F64P = (256, 1, 0), (128, 1, 0), (128, 2, 0), (64, 4, 0)
PAIR128, PAIR64P, ST256, ST128, ST128P, ST64P = (128, 1, 1), (64, 4, 1), (256, 1, 0), (128, 1, 0), (128, 2, 0), (64, 4, 0)


@pytest.mark.parametrize("B,S,nh,fwd,bwd", [(1, 641, 3, F64P, PAIR64P), (1, 704, 1, F64P, PAIR64P), (2, 705, 1, F64P, PAIR64P), (1, 767, 2, F64P, PAIR64P), (1, 897, 1, F64P, PAIR64P),
                                            (1, 1000, 9, F64P, PAIR64P), (1, 4096, 1, F64P, PAIR64P), (1, 4161, 1, F64P, PAIR64P), (1, 1100, 14, F64P, PAIR64P),
                                            (1, 641, 23, F64P, PAIR64P), (1, 1100, 15, F64P, ST64P), (3, 1025, 11, F128P, ST128P), (1, 1100, 29, F128P, ST128P),
                                            (1, 1153, 28, F128P, ST128P), (1, 1100, 48, F128, ST128P), (1, 1024, 24, F64P, PAIR128), (1, 600, 51, F128, PAIR128),
                                            (1, 600, 52, F128, ST128), (2, 704, 23, F128, ST128), (2, 700, 45, F256, ST256)], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("rotated", [False, True])
def test_attn_mfma_parted_rows(taw, B, S, nh, fwd, bwd, rotated):
    """Where there are few tiles several wavefronts share a row (a key): every row at the ends of tiles of 64 and 128, with parts that hold no key a row
    sees, and head counts that the 8 XCDs do not divide; whole rows beyond 640 tokens; the rotary backward inside each."""
    assert tuple(taw.taw_diag_attn_shape(0, B, S, nh).values()) == fwd and tuple(taw.taw_diag_attn_shape(1, B, S, nh).values()) == bwd
    _attn_case(taw, I.BF16, B, S, nh, 128, taw.TAW_IMPL_MFMA, seed=S, bwd_impl=taw.TAW_IMPL_MFMA_STORED, rotated=rotated)


@pytest.mark.parametrize("S,nh,shape", [(700, 2, F64P), (1088, 2, F64P), (1100, 29, F128P)], ids=["700", "1088", "1100-2parts"])
def test_attn_mfma_parted_rows_far_scores(taw, S, nh, shape):
    """One part of a row's keys far above or below the others, -inf among its scores: what the parts are scaled by when they meet is the row's maximum.
    Head 0: the keys of every second block of 32 score about +-300; head 1: they overflow to -inf for the later half of the rows."""
    import torch
    assert tuple(taw.taw_diag_attn_shape(0, 1, S, nh).values()) == shape
    H = nh * 128
    rng = np.random.default_rng(S)
    qkv, _ = draw(rng, (S, 3 * H), I.BF16)
    q64 = I.to_f64(qkv, I.BF16)
    part = (np.arange(S) // 32) % 2 == 1
    q64[:, 0] = np.where(np.arange(S) % 3 == 0, 60.0, -60.0)
    q64[:, H] = np.where(part, 60.0, 0.0)
    q64[:, 128] = np.where(np.arange(S) >= S // 2, 2.0 ** 100, 0.0)
    q64[:, H + 128] = np.where(part & (np.arange(S) < S // 2), -(2.0 ** 100), 0.0)
    qkv = I.to_storage(q64.astype(np.float32), I.BF16)
    q, k, v = (I.to_f64(qkv, I.BF16)[:, i * H:(i + 1) * H].reshape(S, nh, 128) for i in range(3))
    o, lse = U.empty_dev((S, H), I.BF16), torch.empty(nh * S, dtype=torch.float32, device="cuda")
    taw.taw_op_attn_fwd(I.BF16, 1, S, nh, 128, U.to_dev(qkv, I.BF16), o, lse, taw.TAW_IMPL_MFMA)
    got_o, got_l = U.from_dev(o).reshape(S, nh, 128), U.from_dev(lse).reshape(nh, S)
    for h in range(2):
        oref, lref = O.attention_fwd_rows(q[:, h], k[:, h], v[:, h], np.arange(S))      # exp(-2^196) is 0, as exp(-inf)
        assert U.tensor_scale_err(got_o[:, h], oref) < U.TOL[I.BF16]
        assert np.max(np.abs(got_l[h] - lref)) < 2e-2


@pytest.mark.parametrize("B,S,nh,shape", [(1, 64, 1, PAIR128), (1, 600, 51, PAIR128), (1, 1024, 24, PAIR128), (1, 641, 3, PAIR64P), (1, 1024, 16, PAIR64P), (2, 700, 8, PAIR64P),
                                          (1, 4161, 1, PAIR64P), (1, 600, 52, ST128), (1, 1100, 15, ST64P), (1, 4096, 5, ST64P), (1, 1100, 29, ST128P),
                                          (3, 1153, 11, ST128P), (1, 700, 100, ST256), (2, 1301, 30, ST256)], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
@pytest.mark.parametrize("rotated", [False, True])
def test_attn_bwd_stored_equals_recomputed(taw, B, S, nh, shape, rotated):
    """The default form and the pair that recomputes the scores form the same sums in the same order whatever shape the workgroups take: the same bits in dq, dk
    and dv, over scratch of NaN."""
    assert tuple(taw.taw_diag_attn_shape(1, B, S, nh).values()) == shape
    import torch
    H = nh * 128
    qkv, dO = I.device_normal((B * S, 3 * H), seed=S, std=1.0), I.device_normal((B * S, H), seed=nh, std=1.0)
    table = None
    if rotated:
        table = torch.empty(S * 128, dtype=torch.float32, device="cuda")
        taw.taw_rope_table_init(taw.make_desc(I.BF16, B, S, H, nh, 128, 8), table)
    o, lse = torch.empty_like(dO), torch.empty(B * nh * S, dtype=torch.float32, device="cuda")
    taw.taw_op_attn_fwd(I.BF16, B, S, nh, 128, qkv, o, lse, taw.TAW_IMPL_MFMA)
    out = []
    for form in (taw.TAW_IMPL_MFMA, taw.TAW_IMPL_MFMA_STORED):
        dqkv = torch.full_like(qkv, float("nan"))
        scratch = torch.full((taw.taw_op_attn_bwd_scratch_floats(B, S, nh),), float("nan"), dtype=torch.float32, device="cuda")
        taw.taw_op_attn_bwd(I.BF16, B, S, nh, 128, qkv, o, dO, lse, dqkv, scratch, table, form)
        out.append(dqkv)
    assert torch.equal(*out)
