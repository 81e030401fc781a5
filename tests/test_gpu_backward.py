"""GPU parity of the straight-through backward of the grouped W4A16 GEMM (section 3.1, item 2) against the oracle:
dX = dY What (bit-exact on one-hot gradients and in the exact-integer regime) and dW = dY^T X."""
import numpy as np
import pytest
import torch

from paper_2604_07853_amd import synth
from gpu_util import np_bits, norm_err, norm_err_bf16

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-3
TOL_F32 = 2e-5       # dW: bf16 x bf16 products are exact in fp32; accumulation order only
# dX is a 16-bit backward: the scaled gradient dY * s is rounded to bf16 once before the contraction (as a BF16
# trainer rounds the dequantized weight).  Each of the N terms is off by up to half a bf16 ulp, between 2^-9 and 2^-8
# of its size depending on where it lies in its binade (rms about 1.7e-3 of the term), independently, so the sum is
# off by about 1.7e-3 of its rms whatever N is; over 10^5 .. 10^7 outputs the largest deviation is 4 to 5 times
# that.  One-hot gradients and the exact-integer regime are exact (tests above).
TOL_DX_F32 = 1e-2
TOL_DX_RMS = 2.5e-3  # the rms itself


@pytest.fixture(scope="module")
def q():
    from paper_2604_07853_amd import binding
    binding.lib()
    return binding


def _i32(a):
    return torch.tensor(np.asarray(a), dtype=torch.int32, device="cuda")


def test_one_hot_gradient_bit_exact(q, oracle):
    E, N, K = 2, 128, 256
    w = synth.normal_bf16((E, N, K), 0.02, seed=81)
    codes, scales = oracle.quantize_int4(np_bits(w))
    deq = oracle.dequant_int4(codes, scales)
    qw = q.qarl_quantize_weights(w.cuda())
    eye = torch.eye(N).to(torch.bfloat16)
    dy = torch.cat([eye, eye]).cuda()
    dx = q.qarl_qgemm_grouped_dx(qw, dy, _i32([0, N, 2 * N]), 2 * N, out_dtype=q.QARL_OUT_F32).cpu().numpy()
    assert np.array_equal(dx[:N], deq[0]) and np.array_equal(dx[N:], deq[1])


@pytest.mark.parametrize("N", [128, 256])
def test_exact_integer_regime_bit_exact(q, oracle, N):
    rng = np.random.default_rng(82)
    E, K, rows = 3, 256, (40, 0, 75)
    M = sum(rows)
    qi = rng.integers(-7, 8, size=(E, N, K))
    qi[:, :, ::128] = 7
    ex = rng.integers(-3, 2, size=(E, N, K // 128))
    w = torch.tensor(qi * np.repeat(2.0 ** ex, 128, axis=2), dtype=torch.float32).to(torch.bfloat16)
    dy = torch.tensor(rng.integers(-4, 5, size=(M, N)), dtype=torch.float32).to(torch.bfloat16)
    x = torch.tensor(rng.integers(-4, 5, size=(M, K)), dtype=torch.float32).to(torch.bfloat16)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    rm = rng.permutation(M).astype(np.int32)
    codes, scales = oracle.quantize_int4(np_bits(w))
    qw = q.qarl_quantize_weights(w.cuda())
    dx = q.qarl_qgemm_grouped_dx(qw, dy.cuda(), _i32(off), M, out_dtype=q.QARL_OUT_F32)
    assert np.array_equal(dx.cpu().numpy().astype(np.float64), oracle.qgemm_w4a16_dx(np_bits(dy), codes, scales, off))
    dw = q.qarl_grouped_dw(dy.cuda(), x.cuda(), _i32(off), E, row_map=_i32(rm), out_dtype=q.QARL_OUT_F32)
    assert np.array_equal(dw.cpu().numpy().astype(np.float64), oracle.grouped_dw(np_bits(dy), np_bits(x), off, E, rm))
    assert bool((dw[1] == 0).all())                                  # the expert without rows gets zeros


@pytest.mark.parametrize("E,N,K,rows", [(3, 256, 384, (37, 0, 300)), (2, 128, 128, (1, 129)), (4, 384, 1024, (128, 256, 5, 64)),
                                        (2, 256, 512, (70, 129)), (3, 512, 256, (0, 200, 63)),    # several tiles along n and k, an expert without rows
                                        (2, 512, 1024, (130, 65))])   # 2 x 4 tiles of 256 x 256 per expert: one per XCD, three stages and a ragged one
def test_general_data_both_gradients(q, oracle, E, N, K, rows):
    seed = 8300 + N + K
    rng = np.random.default_rng(seed)
    M = int(sum(rows))
    w = synth.normal_bf16((E, N, K), 0.02, seed=seed)
    dy = synth.normal_bf16((M, N), 1.0, seed=seed + 1)
    x = synth.normal_bf16((M + 7, K), 1.0, seed=seed + 2)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    rm = rng.permutation(M + 7)[:M].astype(np.int32)
    scatter = rng.permutation(M).astype(np.int32)
    codes, scales = oracle.quantize_int4(np_bits(w))
    qw = q.qarl_quantize_weights(w.cuda())
    dx_ref = oracle.qgemm_w4a16_dx(np_bits(dy), codes, scales, off)
    dx = q.qarl_qgemm_grouped_dx(qw, dy.cuda(), _i32(off), M, out_dtype=q.QARL_OUT_F32)
    assert norm_err(dx.cpu().numpy(), dx_ref) <= TOL_DX_F32
    assert np.sqrt(((dx.cpu().numpy() - dx_ref) ** 2).mean() / (dx_ref ** 2).mean()) <= TOL_DX_RMS
    dxb = torch.full((M, K), float("nan"), dtype=torch.bfloat16, device="cuda")
    q.qarl_qgemm_grouped_dx(qw, dy.cuda(), _i32(off), M, out_row_map=_i32(scatter), out=dxb)
    want = np.empty_like(dx_ref)
    want[scatter] = dx_ref                                           # row i of the problem lands in row scatter[i]
    assert norm_err(dxb.float().cpu().numpy(), want) <= TOL_DX_F32 + 2.0 ** -8     # plus the output's own rounding
    dw_ref = oracle.grouped_dw(np_bits(dy), np_bits(x), off, E, rm)
    dw = q.qarl_grouped_dw(dy.cuda(), x.cuda(), _i32(off), E, row_map=_i32(rm), out_dtype=q.QARL_OUT_F32)
    assert norm_err(dw.cpu().numpy(), dw_ref) <= TOL_F32
    dwb = q.qarl_grouped_dw(dy.cuda(), x.cuda(), _i32(off), E, row_map=_i32(rm))
    assert norm_err_bf16(dwb.float().cpu().numpy(), dw_ref) <= TOL_BF16
    # without a row map the activation rows are the problem's rows themselves
    dw_id = q.qarl_grouped_dw(dy.cuda(), x.cuda(), _i32(off), E, out_dtype=q.QARL_OUT_F32)
    assert norm_err(dw_id.cpu().numpy(), oracle.grouped_dw(np_bits(dy), np_bits(x), off, E)) <= TOL_F32
    # the adjoint identity on the GPU's own results: <dY, Y> = <dX, X> = <dW, What>
    y = q.qarl_qgemm_grouped(qw, x.cuda(), _i32(off), M, row_map=_i32(rm), out_dtype=q.QARL_OUT_F32).double()
    a = float((dy.cuda().double() * y).sum())
    b = float((dx.double() * x.cuda().double()[torch.tensor(rm, dtype=torch.long, device="cuda")]).sum())
    c = float((dw.double() * torch.tensor(oracle.dequant_int4(codes, scales), device="cuda").double()).sum())
    scale = float(dy.double().norm() * y.norm().cpu())
    assert abs(a - b) <= 2e-3 * scale and abs(a - c) <= 1e-4 * scale


def test_backward_full_size_gate_up_sampled(q, oracle):
    """The gate_up matrices of the full layer (128 experts, N = 1536, K = 2048) at 2048 tokens with a Zipf router:
    dX on sampled rows, dW on the most and least loaded expert and one in between."""
    E, H, I, TOPK = synth.E, synth.H, synth.I, synth.TOPK
    N, K, T = 2 * I, H, 2048
    gu, _ = synth.expert_weights(E, H, I, seed=8400, device="cuda")
    qw = q.qarl_quantize_weights(gu)
    codes, scales = oracle.quantize_int4(np_bits(gu))
    del gu
    lg = synth.router_logits(T, E, seed=8401, device="cuda", zipf_s=1.1)
    r = q.qarl_moe_route(lg, TOPK)
    M = T * TOPK
    off = r.offsets.cpu().numpy()
    tok = r.tokens.cpu().numpy()
    x = synth.normal_bf16((T, K), 1.0, seed=8402, device="cuda")
    dy = synth.normal_bf16((M, N), 1.0, seed=8403, device="cuda")
    dx = q.qarl_qgemm_grouped_dx(qw, dy, r.offsets, M, out_dtype=q.QARL_OUT_F32)
    dw = q.qarl_grouped_dw(dy, x, r.offsets, E, row_map=r.tokens, out_dtype=q.QARL_OUT_F32)
    counts = np.diff(off)
    rng = np.random.default_rng(8404)
    rows = np.unique(np.concatenate([off[:-1][counts > 0], off[1:][counts > 0] - 1, rng.integers(0, M, 48)]))
    # the oracle on the sampled rows only: one sub-problem whose offsets count the sampled rows per expert
    exp_of = np.searchsorted(off, rows, side="right") - 1
    sub = np.concatenate([[0], np.cumsum(np.bincount(exp_of, minlength=E))]).astype(np.int32)
    dx_ref = oracle.qgemm_w4a16_dx(np_bits(dy)[rows], codes, scales, sub)
    assert norm_err(dx[torch.from_numpy(rows).cuda()].cpu().numpy(), dx_ref) <= TOL_DX_F32
    order = np.argsort(counts)
    for e in (int(order[-1]), int(order[0]), int(order[E // 2])):
        lo, hi = off[e], off[e + 1]
        ref = oracle.grouped_dw(np_bits(dy)[lo:hi], np_bits(x), np.array([0, hi - lo], dtype=np.int32), 1, tok[lo:hi])
        assert norm_err(dw[e].cpu().numpy(), ref[0]) <= TOL_F32, e


@pytest.mark.parametrize("E,N,K,heavy,rest", [(256, 512, 1536, (700, 300), 9),      # tiles chained, one list, experts not looked at
                                              (130, 1536, 2048, (3, 0, 900), 12),   # ... three lists' worth of tiles per expert, one list per XCD
                                              (256, 512, 1536, (700, 300), 30),     # the same, ranked in 256 places
                                              (130, 1536, 2048, (3, 0, 900), 40),
                                              (5, 512, 1024, (1300, 0), 400),       # one tile per workgroup, no order
                                              (128, 512, 1024, (1500,), 250),       # ranked, one tile per workgroup
                                              (300, 512, 512, (400,), 200),         # too many experts to rank
                                              (65, 512, 1024, (64, 0), 30)])        # few rows: the 128 x 128 tiles
def test_dw_in_every_order_of_the_experts(q, E, N, K, heavy, rest):
    """Popular experts first, tiles of the others in chains: every expert's gradient against 64-bit sums."""
    rng = np.random.default_rng(E + N)
    rows = rng.integers(0, rest, E)
    rows[rng.permutation(E)[:len(heavy)]] = heavy
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    M = int(off[-1])
    dy = synth.normal_bf16((M, N), 1.0, seed=8501, device="cuda")
    x = synth.normal_bf16((M + 5, K), 1.0, seed=8502, device="cuda")
    rm = torch.from_numpy(rng.permutation(M + 5)[:M].astype(np.int64)).cuda()
    dw = torch.full((E, N, K), float("nan"), dtype=torch.float32, device="cuda")
    q.qarl_grouped_dw(dy, x, _i32(off), E, row_map=rm.to(torch.int32), out_dtype=q.QARL_OUT_F32, out=dw)
    for e in range(E):
        lo, hi = int(off[e]), int(off[e + 1])
        want = dy[lo:hi].double().t() @ x[rm[lo:hi]].double()
        err = (dw[e].double() - want).abs() / (want.abs() + max(1.0, float(hi - lo)) ** 0.5)
        assert float(err.max()) <= TOL_F32, (e, hi - lo)


def test_backward_errors(q):
    w = synth.normal_bf16((1, 64, 128), 0.02, seed=85).cuda()
    qw = q.qarl_quantize_weights(w)                                  # N = 64: not a multiple of 128
    dy = torch.zeros((4, 64), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(q.QarlError) as ei:
        q.qarl_qgemm_grouped_dx(qw, dy, _i32([0, 4]), 4)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED
    q8 = q.qarl_quantize_weights(synth.normal_bf16((1, 128, 128), 0.02, seed=86).cuda(), q.QARL_FP8_E4M3_CH)
    with pytest.raises(q.QarlError) as ei:
        q.qarl_qgemm_grouped_dx(q8, torch.zeros((4, 128), dtype=torch.bfloat16, device="cuda"), _i32([0, 4]), 4)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED
    with pytest.raises(q.QarlError) as ei:
        q.qarl_grouped_dw(dy, torch.zeros((4, 128), dtype=torch.bfloat16, device="cuda"), _i32([0, 4]), 1)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED


@pytest.mark.parametrize("E,N,K,rows", [(2, 128, 4096, (6401, 5888)),             # two stages, a tile of one row, a last tile that is full
                                        (3, 1536, 4096, (0, 6100, 6144 - 192)),   # an expert without rows, last tiles of 212 and 64 rows
                                        (1, 384, 12288, (4101,)),                 # a tile of five rows
                                        (1, 3840, 4096, (12300,)), (1, 3968, 4096, (12300,))])    # the longest contraction whose scales fit LDS, and one more
def test_dx_of_many_rows(q, oracle, E, N, K, rows):
    """From 512 rows per expert and three rounds of workgroups on: 256 x 256 tiles where the scales fit LDS.  Against 64-bit sums
    of the same operands (the scaled gradients rounded to bf16), so that only the order of the sums is left.  The sums of
    a (q + 24) and of -24 a each have about 24 / 2.6 = 10 times the rms of their difference (q of normal weights has an rms of 2.6),
    and a chain of N fp32 additions is off by up to about sqrt(N) half ulps of such a value: 10 * 2^-24 * sqrt(N)."""
    seed = 8700 + N + K
    M = sum(rows)
    assert M >= 512 * E and (M // 256 + E // 2) * (K // 256) >= 768
    rng = np.random.default_rng(seed)
    w = synth.normal_bf16((E, N, K), 0.02, seed=seed, device="cuda")
    dy = synth.normal_bf16((M, N), 1.0, seed=seed + 1, device="cuda")
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    scatter = _i32(rng.permutation(M).astype(np.int32))
    qw = q.qarl_quantize_weights(w)
    codes = oracle.dequant_int4(*oracle.quantize_int4(np_bits(w)))            # s*q
    sc = qw.scales.float()                                                    # [E][N][K / 128]
    dx = q.qarl_qgemm_grouped_dx(qw, dy, _i32(off), M, out_dtype=q.QARL_OUT_F32)
    for e in range(E):
        lo, hi = off[e], off[e + 1]
        deq = torch.from_numpy(codes[e]).cuda()
        for g in range(K // 128):
            s = sc[e, :, g]
            a = (dy[lo:hi].float() * s).to(torch.bfloat16).double()
            ref = a @ torch.round(deq[:, g * 128:(g + 1) * 128].double() / s[:, None].double())
            got = dx[lo:hi, g * 128:(g + 1) * 128].double()
            if hi > lo:
                err = float(((got - ref).abs() / (ref.abs() + ref.pow(2).mean().sqrt())).max())
                assert err <= max(TOL_F32, 10 * 2.0 ** -24 * N ** 0.5), (e, g)
    dxb = torch.full((M + 1, K), 7.0, dtype=torch.bfloat16, device="cuda")
    q.qarl_qgemm_grouped_dx(qw, dy, _i32(off), M, out_row_map=scatter, out=dxb)
    assert torch.equal(dxb[scatter.long()], dx.to(torch.bfloat16)) and bool((dxb[M] == 7).all())
    # gradients with one element per row return rows of s*q bit for bit
    n = torch.from_numpy(rng.integers(0, N, M)).cuda()
    hot = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    hot[torch.arange(M, device="cuda"), n] = 1.0
    dx = q.qarl_qgemm_grouped_dx(qw, hot, _i32(off), M, out_dtype=q.QARL_OUT_F32)
    for e in range(E):
        assert torch.equal(dx[off[e]:off[e + 1]], torch.from_numpy(codes[e]).cuda().float()[n[off[e]:off[e + 1]]])


@pytest.mark.parametrize("N", [2048, 3840])
def test_dx_is_as_exact_on_either_tile_size(q, N):
    """The same rows on the 256 x 256 tiles (one call) and on the 128 x 128 ones (calls of fewer than 512 rows), each against 64-bit sums of
    the rounded operands.  Both add the same products in the same matrix instructions and form a row sum in sixteen chains of N / 32
    additions, so the 2-norms of their errors agree but for which rounding hits which row, about 1 / sqrt(M) = 1 %
    of the row sums' share, itself a tenth: 0.2 % is asked for.  Chains of N / 4 are 0.7 % off."""
    K, M = 4096, 12300
    w, dy = synth.normal_bf16((1, N, K), 0.02, seed=N, device="cuda"), synth.normal_bf16((M, N), 1.0, seed=N + 1, device="cuda")
    qw = q.qarl_quantize_weights(w)
    wide = q.qarl_qgemm_grouped_dx(qw, dy, _i32([0, M]), M, out_dtype=q.QARL_OUT_F32)
    small = torch.cat([q.qarl_qgemm_grouped_dx(qw, dy[r:r + 500].contiguous(), _i32([0, min(500, M - r)]), min(500, M - r), out_dtype=q.QARL_OUT_F32)
                       for r in range(0, M, 500)])
    shifts = 4 * torch.arange(8, device="cuda", dtype=torch.int32)
    codes = (((q.qarl_codes_to_canonical(qw)[0, :, :, None] >> shifts) & 15) - 8).reshape(N, K).double()
    err = {"wide": 0.0, "small": 0.0}
    for g in range(K // 128):
        c = slice(g * 128, (g + 1) * 128)
        ref = (dy.float() * qw.scales[0, :, g].float()).to(torch.bfloat16).double() @ codes[:, c]
        for name, got in (("wide", wide), ("small", small)):
            err[name] += float((got[:, c].double() - ref).pow(2).sum())
    assert (err["wide"] / err["small"]) ** 0.5 <= 1.002
