"""GPU parity of the grouped quantized GEMM against the oracle: bit-exact where the result
does not depend on summation order (one-hot probe, exact-integer regime), within the stated
tolerance on general data; both kernel paths on the same codes and scales."""
import numpy as np
import pytest
import torch

from paper_2604_07853_amd import synth
from gpu_util import np_bits, norm_err, norm_err_bf16, flip_fraction

pytestmark = pytest.mark.gpu

# Tolerance for bf16 outputs (2e-3, the stated bar): max (|d| - half_ulp_bf16(ref))+ / (|ref| + rms(ref)),
# i.e. the error of the value before it is rounded to the 8-bit-significand output format; a bf16
# rounding alone is up to 2^-8 = 3.9e-3 relative, so it is discounted and checked separately through
# the fraction of outputs whose bits differ from the oracle's own bf16 rounding.
TOL_BF16 = 2e-3
TOL_F32 = 2e-5       # fp32 outputs: accumulation-order noise only
MAX_FLIPS = 0.02     # bf16 outputs that may land on the neighbouring value
# e4m3 x e4m3 MFMA: products are exact, but inside one instruction the matrix core aligns them to the
# largest product's exponent and keeps about 15 bits below it, truncating (measured: next to a
# product of 448*448 = 2^17.6 a product of 14 arrives as 8, one below 8 as 0).  The result is an error
# of 4e-5..2e-4 of rms whatever K is, identical in both kernel paths, so fp32 outputs of the FP8
# format get a wider bar, still inside the 2e-3 one.
TOL_F32_FP8 = 1e-3
MAX_FLIPS_FP8 = 0.06
# FP8 layer end to end against the oracle's own chain: one moved e4m3 code of the intermediate changes one of I
# products by up to 2^-3 of its size, a moved row scale a few per cent of them; after the down projection and the
# combine that is a few 1e-3 of the output's rms on the rows it hits; a row whose largest element moved gets
# another scale and a few per cent new codes, which is worth up to 1e-1 of the rms on that token.
FP8_E2E_MAX = 5e-2
FP8_E2E_MAX_SCALE = 0.2   # tokens with a pair-row whose scale moved by one bf16 step of its largest element


@pytest.fixture(scope="module")
def q():
    from paper_2604_07853_amd import binding
    binding.lib()
    return binding


def _paths(q):
    return [q.QARL_PATH_DECODE, q.QARL_PATH_PREFILL]


def _i32(a):
    return torch.tensor(np.asarray(a), dtype=torch.int32, device="cuda")


def test_dense_w4a16_config1(q, oracle):
    """Config 1: x [16,2048] N(0,1), W [768,2048] N(0,0.02), W4A16 g128, fp32 out."""
    g = torch.Generator().manual_seed(0)                           # the config's seed 0: x first, then W, one stream
    x = torch.randn((16, 2048), generator=g).to(torch.bfloat16)
    w = (torch.randn((1, 768, 2048), generator=g) * 0.02).to(torch.bfloat16)
    codes, scales = oracle.quantize_int4(np_bits(w))
    off = np.array([0, 16], dtype=np.int32)
    ref = oracle.qgemm_w4a16(np_bits(x), codes, scales, off)
    qw = q.qarl_quantize_weights(w.cuda())
    for path in _paths(q):
        y = q.qarl_qgemm_grouped(qw, x.cuda(), _i32(off), 16, out_dtype=q.QARL_OUT_F32, path=path)
        e = norm_err(y.cpu().numpy(), ref)
        assert e <= TOL_F32, (path, e)
        yb = q.qarl_qgemm_grouped(qw, x.cuda(), _i32(off), 16, out_dtype=q.QARL_OUT_BF16, path=path)
        eb = norm_err_bf16(yb.float().cpu().numpy(), ref)
        assert eb <= TOL_BF16, (path, eb)
        fl = flip_fraction(np_bits(yb), oracle.bf16_from_f64(ref))
        assert fl <= MAX_FLIPS, (path, fl)


@pytest.mark.parametrize("K,N", [(256, 64), (768, 32), (4096, 32)])
def test_one_hot_probe_bit_exact_both_paths(q, oracle, K, N):
    """x = rows of the identity: the output is the dequantized weight s*q itself; both paths
    must reproduce it exactly (identical dequantized numerics)."""
    E = 2
    w = synth.normal_bf16((E, N, K), 0.02, seed=7)
    codes, scales = oracle.quantize_int4(np_bits(w))
    deq = oracle.dequant_int4(codes, scales)                       # [E, N, K] fp32
    eye = torch.eye(K).to(torch.bfloat16)
    x = torch.cat([eye, eye]).cuda()
    off = _i32([0, K, 2 * K])
    qw = q.qarl_quantize_weights(w.cuda())
    for path in _paths(q):
        y = q.qarl_qgemm_grouped(qw, x, off, 2 * K, out_dtype=q.QARL_OUT_F32, path=path).cpu().numpy()
        assert np.array_equal(y[:K], deq[0].T) and np.array_equal(y[K:], deq[1].T), path


def test_exact_integer_regime_bit_exact(q, oracle):
    rng = np.random.default_rng(7)
    E, N, K, M = 3, 64, 512, 75
    qi = rng.integers(-7, 8, size=(E, N, K))
    qi[:, :, ::128] = 7
    ex = rng.integers(-3, 2, size=(E, N, K // 128))
    w = torch.tensor(qi * np.repeat(2.0 ** ex, 128, axis=2), dtype=torch.float32).to(torch.bfloat16)
    x = torch.tensor(rng.integers(-4, 5, size=(M, K)), dtype=torch.float32).to(torch.bfloat16)
    off = np.array([0, 40, 40, 75], dtype=np.int32)                # expert 1 is empty
    rm = rng.permutation(M).astype(np.int32)
    codes, scales = oracle.quantize_int4(np_bits(w))
    ref = oracle.qgemm_w4a16(np_bits(x), codes, scales, off, rm)
    qw = q.qarl_quantize_weights(w.cuda())
    for path in _paths(q):
        y = q.qarl_qgemm_grouped(qw, x.cuda(), _i32(off), M, row_map=_i32(rm), out_dtype=q.QARL_OUT_F32, path=path)
        assert np.array_equal(y.cpu().numpy().astype(np.float64), ref), path


def _moe_case(q, oracle, E, H, I, T, topk, seed, zipf, path, fmt="int4"):
    gu, dn = synth.expert_weights(E, H, I, seed)
    x = synth.normal_bf16((T, H), 1.0, seed + 2)
    lg = synth.router_logits(T, E, seed + 3, zipf_s=zipf)
    r = q.qarl_moe_route(lg.cuda(), topk)
    ids, w = oracle.route(np_bits(lg), topk)
    counts, offsets, pairs = oracle.group(ids, E)
    assert np.array_equal(r.pairs.cpu().numpy(), pairs)
    M = T * topk
    tok = (pairs // topk).astype(np.int32)
    if fmt == "int4":
        guc, gus = oracle.quantize_int4(np_bits(gu))
        dnc, dns = oracle.quantize_int4(np_bits(dn))
        qgu = q.qarl_quantize_weights(gu.cuda())
        qdn = q.qarl_quantize_weights(dn.cuda())
        # stage 1: gate_up + SiLU*mul
        a_gpu = q.qarl_qgemm_grouped(qgu, x.cuda(), r.offsets, M, row_map=r.tokens, epilogue=q.QARL_EPI_SILU_MUL, path=path)
        gu_ref = oracle.qgemm_w4a16(np_bits(x), guc, gus, offsets, tok)
        a_ref_bits, a_ref = oracle.silu_mul(gu_ref)
        a_gpu_bits = np_bits(a_gpu)
        ea = norm_err_bf16(a_gpu.float().cpu().numpy(), a_ref)
        assert ea <= TOL_BF16, ea
        fl = flip_fraction(a_gpu_bits, a_ref_bits)
        assert fl <= MAX_FLIPS, fl
        # stage 2: down on the GPU's own a, Y in fp32 (NONE epilogue)
        y_gpu = q.qarl_qgemm_grouped(qdn, a_gpu, r.offsets, M, out_dtype=q.QARL_OUT_F32, path=path)
        y_ref = oracle.qgemm_w4a16(a_gpu_bits, dnc, dns, offsets)
        ey = norm_err(y_gpu.cpu().numpy(), y_ref)
        assert ey <= TOL_F32, ey
        # stage 3: down + combine, bf16 out, against the oracle on the GPU's a
        out_gpu = q.qarl_qgemm_grouped(qdn, a_gpu, r.offsets, M, epilogue=q.QARL_EPI_COMBINE, combine_w=r.w,
                                       sorted_pairs=r.pairs, T=T, topk=topk, path=path)
        out_ref, out_ref_bits = oracle.combine(y_ref, pairs, w, T, topk)
        eo = norm_err_bf16(out_gpu.float().cpu().numpy(), out_ref)
        assert eo <= TOL_BF16, eo
        fl = flip_fraction(np_bits(out_gpu), out_ref_bits)
        assert fl <= MAX_FLIPS, fl
        # end to end against the oracle's own chain
        full = oracle.moe_ffn_w4a16(np_bits(x), np_bits(lg), guc, gus, dnc, dns, topk)
        layer = q.MoELayer(qgu, qdn, T, topk, path)
        out2 = layer.forward(x.cuda(), lg.cuda())
        e2e = norm_err_bf16(out2.float().cpu().numpy(), full["out"])
        assert e2e <= TOL_BF16, e2e                                # includes the rare one-ulp flips of a
        assert np.array_equal(np_bits(out2), np_bits(out_gpu))     # same kernels, same result
    else:
        guq, gus = oracle.quantize_fp8_rows(np_bits(gu))
        dnq, dns = oracle.quantize_fp8_rows(np_bits(dn))
        qgu = q.qarl_quantize_weights(gu.cuda(), q.QARL_FP8_E4M3_CH)
        qdn = q.qarl_quantize_weights(dn.cuda(), q.QARL_FP8_E4M3_CH)
        xq, sx = q.qarl_quantize_rows_fp8(x.cuda())
        xq_ref, sx_ref = oracle.quantize_fp8_rows(np_bits(x))
        assert np.array_equal(xq.cpu().numpy(), xq_ref) and np.array_equal(sx.cpu().numpy(), sx_ref)
        a_gpu = q.qarl_qgemm_grouped(qgu, xq, r.offsets, M, row_map=r.tokens, x_scales=sx,
                                     epilogue=q.QARL_EPI_SILU_MUL, path=path)
        gu_ref = oracle.qgemm_fp8(xq_ref, sx_ref, guq, gus, offsets, tok)
        a_ref_bits, a_ref = oracle.silu_mul(gu_ref)
        ea = norm_err_bf16(a_gpu.float().cpu().numpy(), a_ref)
        assert ea <= TOL_BF16, ea
        fl = flip_fraction(np_bits(a_gpu), a_ref_bits)
        assert fl <= MAX_FLIPS_FP8, fl
        aq, sa = q.qarl_quantize_rows_fp8(a_gpu)
        aq_ref, sa_ref = oracle.quantize_fp8_rows(np_bits(a_gpu))   # oracle on the GPU's own a
        assert np.array_equal(aq.cpu().numpy(), aq_ref) and np.array_equal(sa.cpu().numpy(), sa_ref)
        y_gpu = q.qarl_qgemm_grouped(qdn, aq, r.offsets, M, x_scales=sa, out_dtype=q.QARL_OUT_F32, path=path)
        y_ref = oracle.qgemm_fp8(aq_ref, sa_ref, dnq, dns, offsets)
        ey = norm_err(y_gpu.cpu().numpy(), y_ref)
        assert ey <= TOL_F32_FP8, ey
        out_gpu = q.qarl_qgemm_grouped(qdn, aq, r.offsets, M, x_scales=sa, epilogue=q.QARL_EPI_COMBINE,
                                       combine_w=r.w, sorted_pairs=r.pairs, T=T, topk=topk, path=path)
        out_ref, _ = oracle.combine(y_ref, pairs, w, T, topk)
        eo = norm_err_bf16(out_gpu.float().cpu().numpy(), out_ref)
        assert eo <= TOL_BF16, eo
        layer = q.MoELayer(qgu, qdn, T, topk, path)
        out2 = layer.forward(x.cuda(), lg.cuda())
        assert np.array_equal(np_bits(out2), np_bits(out_gpu))
        # end to end against the oracle's own chain.  The activation quantizer of eq. (2) is discontinuous: an
        # intermediate that lands on the neighbouring bf16 value can move an e4m3 code by a whole step (2^-4
        # relative), and if it is the row's largest element the row's scale and a few per cent of its codes.  So
        # the stages above carry the parity bar; here the size of that effect is reported and bounded.
        full = oracle.moe_ffn_fp8(np_bits(x), np_bits(lg), guq, gus, dnq, dns, topk)
        a_rows = int((np_bits(a_gpu) != full["a"]).any(axis=1).sum())
        code_rows = int(((aq.cpu().numpy() != full["aq"]).any(axis=1) | (sa.cpu().numpy() != full["sa"])).sum())
        scale_rows = int((sa.cpu().numpy() != full["sa"]).sum())
        ref = full["out"]
        rms = np.sqrt((ref ** 2).mean())
        d = np.abs(out2.float().cpu().numpy().astype(np.float64) - ref) / (np.abs(ref) + rms)
        # tokens one of whose pair-rows got another row scale (their whole row of codes is requantized)
        tok_moved = np.zeros(T, dtype=bool)
        tok_moved[tok[sa.cpu().numpy() != full["sa"]]] = True
        e_same = float(d[~tok_moved].max()) if (~tok_moved).any() else 0.0
        e_moved = float(d[tok_moved].max()) if tok_moved.any() else 0.0
        e_9999, e_med = float(np.quantile(d, 0.9999)), float(np.median(d))
        print("fp8 end to end: T=%d path=%d max %.2e (tokens with a moved row scale: %.2e) p99.99 %.2e median %.2e; "
              "rows of a moved %d / %d, rows with codes or scale moved %d (scale %d)"
              % (T, path, e_same, e_moved, e_9999, e_med, a_rows, M, code_rows, scale_rows))
        assert e_med <= TOL_BF16 and e_same <= FP8_E2E_MAX and e_moved <= FP8_E2E_MAX_SCALE, (e_med, e_same, e_moved)
        assert scale_rows <= max(2, 0.02 * M), scale_rows


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("T,zipf", [(40, 0.0), (301, 1.1)])
def test_moe_layer_small_w4a16(q, oracle, T, zipf, path):
    """Scaled-down layer (E=64, H=512, I=256): ragged expert loads, empty experts, several tiles."""
    _moe_case(q, oracle, 64, 512, 256, T, 4, seed=20 + T, zipf=zipf, path=path)


@pytest.mark.parametrize("path", [1, 2])
@pytest.mark.parametrize("T,zipf", [(40, 0.0), (301, 1.1)])
def test_moe_layer_small_fp8(q, oracle, T, zipf, path):
    _moe_case(q, oracle, 64, 512, 256, T, 4, seed=40 + T, zipf=zipf, path=path, fmt="fp8")


def test_fp8_one_hot_probe(q, oracle):
    """x rows = 448*e_k: s_x = 1 exactly, so the output is s_w * decode(w_q) with no accumulation."""
    K, N = 256, 64
    w = synth.normal_bf16((1, N, K), 0.02, seed=8)
    wq, sw = oracle.quantize_fp8_rows(np_bits(w))
    qw = q.qarl_quantize_weights(w.cuda(), q.QARL_FP8_E4M3_CH)
    x = (torch.eye(K) * 448).to(torch.bfloat16).cuda()
    xq, sx = q.qarl_quantize_rows_fp8(x)
    assert bool((sx == 1.0).all())
    want = (oracle.e4m3_decode(wq[0]) * 448.0 * sw[0][:, None].astype(np.float64)).T
    for path in _paths(q):
        y = q.qarl_qgemm_grouped(qw, xq, _i32([0, K]), K, x_scales=sx, out_dtype=q.QARL_OUT_F32, path=path)
        assert np.array_equal(y.cpu().numpy().astype(np.float64), want.astype(np.float32).astype(np.float64)), path


def _fp8_codes_of(oracle, values):
    return oracle.e4m3_encode(np.asarray(values, dtype=np.float64))


@pytest.mark.parametrize("K", [256, 512])
def test_fp8_matrix_core_truncation_bound(q, oracle, K):
    """One product of 448 * 448 beside many small ones in the same k-block.  Products of two e4m3 values are
    exact, but the matrix core sums the products of one instruction after aligning them to the largest product's
    exponent E and dropping what lies below 2^(E-14).  The oracle sums exactly; the difference must stay below the
    bound that this model gives per output, sum over the 64-k blocks of 63 * 2^(E_block - 14) (+ fp32
    accumulation), in both kernel paths, and must not vanish on this input (else the wider FP8 bar is not needed)."""
    rng = np.random.default_rng(11 + K)
    N, M = 64, 48
    xv = rng.integers(-7, 8, size=(M, K)).astype(np.float64)
    wv = rng.integers(-7, 8, size=(1, N, K)).astype(np.float64)
    xv[:, ::64] = 448.0                                   # first element of every 64-k block of every token row
    wv[0, :, ::64] = 448.0
    xv[M // 2:, 64:] = rng.integers(-7, 8, size=(M - M // 2, K - 64))   # lower half: the big product in block 0 only
    xq, wq = _fp8_codes_of(oracle, xv), _fp8_codes_of(oracle, wv)
    assert np.array_equal(oracle.e4m3_decode(xq), xv) and np.array_equal(oracle.e4m3_decode(wq), wv)
    sx, sw = np.ones(M, dtype=np.float32), np.ones((1, N), dtype=np.float32)
    off = np.array([0, M], dtype=np.int32)
    ref = oracle.qgemm_fp8(xq, sx, wq, sw, off)
    prod = np.abs(xv[:, None, :] * wv[0][None, :, :]).reshape(M, N, K // 64, 64)
    top = prod.max(axis=3)
    Eb = np.floor(np.log2(np.maximum(top, 1.0)))
    bound = (63.0 * 2.0 ** (Eb - 14)).sum(axis=2) + K * 2.0 ** -24 * prod.sum(axis=(2, 3))
    qw = q.QWeight(q.QARL_FP8_E4M3_CH, 1, N, K, torch.tensor(wq, device="cuda"), torch.tensor(sw, device="cuda"))
    for path in _paths(q):
        y = q.qarl_qgemm_grouped(qw, torch.tensor(xq, device="cuda"), _i32(off), M,
                                 x_scales=torch.tensor(sx, device="cuda"), out_dtype=q.QARL_OUT_F32, path=path)
        d = np.abs(y.cpu().numpy().astype(np.float64) - ref)
        print("fp8 truncation K=%d path=%d: max |d| %.1f (bound there %.1f), mean |d| %.2f, rel. to rms %.2e"
              % (K, path, d.max(), bound.flat[d.argmax()], d.mean(), d.max() / np.sqrt((ref ** 2).mean())))
        assert np.all(d <= bound), (path, float((d - bound).max()))
        assert d.max() > 0, path


def test_moe_decode_config2_full_size(q, oracle):
    """Config 2 at full size: 256 tokens, 128 experts, H 2048, I 768, top-8, W4A16, decode path."""
    _moe_case(q, oracle, synth.E, synth.H, synth.I, 256, synth.TOPK, seed=1, zipf=0.0, path=1)


def test_empty_and_error_paths(q):
    w = synth.normal_bf16((2, 32, 128), 0.02, seed=1).cuda()
    qw = q.qarl_quantize_weights(w)
    x = torch.zeros((4, 128), dtype=torch.bfloat16, device="cuda")
    off = _i32([0, 0, 0])
    y = q.qarl_qgemm_grouped(qw, x, off, 0, out_dtype=q.QARL_OUT_F32)          # M = 0: no-op
    assert y.shape == (0, 32)
    with pytest.raises(q.QarlError) as ei:                                      # COMBINE without workspace
        q.lib().qarl_qgemm_grouped
        q._check(q.lib().qarl_qgemm_grouped(q.C.byref(qw.desc), q._ptr(x), None, 4, None, q._ptr(off), 4,
                                            q.QARL_EPI_COMBINE, q._ptr(x), q._ptr(off), 1, 4, q._ptr(x), 0, 0,
                                            None, 0, None))
    assert ei.value.status == q.QARL_ERR_WORKSPACE
    with pytest.raises(q.QarlError) as ei:
        q.qarl_qgemm_grouped(qw, x, off, 4, epilogue=q.QARL_EPI_SILU_MUL, out_dtype=q.QARL_OUT_F32)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED


@pytest.mark.parametrize("fmt", ["int4", "fp8"])
@pytest.mark.parametrize("E,N,K,rows", [(3, 96, 128, (37, 0, 5)), (2, 288, 384, (300, 129)), (1, 32, 128, (1,)),
                                        (2, 544, 768, (64, 257))])
def test_ragged_shapes_both_paths(q, oracle, fmt, E, N, K, rows):
    """Shapes that leave partial column tiles (N not a multiple of the tile width), a single 128-k stage,
    empty experts, one-row experts and experts spanning several token tiles; plain epilogue, fp32 out."""
    seed = 700 + N + K
    w = synth.normal_bf16((E, N, K), 0.02, seed=seed)
    M = int(sum(rows))
    x = synth.normal_bf16((M, K), 1.0, seed=seed + 1)
    off = np.concatenate([[0], np.cumsum(rows)]).astype(np.int32)
    if fmt == "int4":
        codes, scales = oracle.quantize_int4(np_bits(w))
        ref = oracle.qgemm_w4a16(np_bits(x), codes, scales, off)
        qw = q.qarl_quantize_weights(w.cuda())
        xin, xs, tol = x.cuda(), None, TOL_F32
    else:
        wq, sw = oracle.quantize_fp8_rows(np_bits(w))
        xq_ref, sx_ref = oracle.quantize_fp8_rows(np_bits(x))
        ref = oracle.qgemm_fp8(xq_ref, sx_ref, wq, sw, off)
        qw = q.qarl_quantize_weights(w.cuda(), q.QARL_FP8_E4M3_CH)
        xin, xs = q.qarl_quantize_rows_fp8(x.cuda())
        tol = TOL_F32_FP8
    for path in _paths(q):
        try:
            y = q.qarl_qgemm_grouped(qw, xin, _i32(off), M, x_scales=xs, out_dtype=q.QARL_OUT_F32, path=path)
        except q.QarlError as err:      # the streaming path takes W4A16 only with K a multiple of 256
            assert path == q.QARL_PATH_DECODE and err.status == q.QARL_ERR_UNSUPPORTED and fmt == "int4" and K % 256
            continue
        e = norm_err(y.cpu().numpy(), ref)
        assert e <= tol, (path, e)


@pytest.mark.parametrize("E,N,K,T,topk", [(8, 64, 2048, 600, 3),     # row maps too large to sit beside the LDS tile
                                          (3, 96, 4096, 50, 2),      # K beyond 2048: 16-row LDS tile, several row blocks
                                          (4, 512, 2048, 60, 3),     # 64-row blocks over a K-chunked tile, one pair per wavefront
                                          (4, 1024, 2048, 200, 3),   # the same with two pairs and several row blocks
                                          (4, 64, 512, 37, 3),       # M = 111: last quad of the map is partial
                                          (16, 32, 256, 1500, 3),    # M = 4500: maps stay in global memory
                                          (6, 96, 768, 171, 5)])     # 64-row blocks (K fits), M = 855
def test_decode_row_map_paths(q, oracle, E, N, K, T, topk):
    """Decode path with the gather map (routed tokens) and the scatter map (pair order of the combine):
    every way the kernel fetches its row ids (copied to LDS next to the tile, into the tile region, or read
    from global memory), experts that need several row blocks and several passes, M not a multiple of 4."""
    seed = 900 + K + T
    w = synth.normal_bf16((E, N, K), 0.02, seed=seed)
    x = synth.normal_bf16((T, K), 1.0, seed=seed + 1)
    lg = synth.router_logits(T, E, seed + 2, zipf_s=1.1)
    ids, wts = oracle.route(np_bits(lg), topk)                     # the router kernel takes E % 64 == 0 only:
    counts, offsets, pairs = oracle.group(ids, E)                  # the oracle's routing is this test's input
    M = T * topk
    tok = (pairs // topk).astype(np.int32)
    d_off, d_tok, d_pairs = _i32(offsets), _i32(tok), _i32(pairs)
    d_w = torch.tensor(np.asarray(wts, dtype=np.float32), device="cuda")
    codes, scales = oracle.quantize_int4(np_bits(w))
    qw = q.qarl_quantize_weights(w.cuda())
    # gather only: rows of x picked through row_map, fp32 out in sorted order
    y_ref = oracle.qgemm_w4a16(np_bits(x), codes, scales, offsets, tok)
    y = q.qarl_qgemm_grouped(qw, x.cuda(), d_off, M, row_map=d_tok, out_dtype=q.QARL_OUT_F32,
                             path=q.QARL_PATH_DECODE)
    assert norm_err(y.cpu().numpy(), y_ref) <= TOL_F32
    # gather + scatter: the same product through the combine epilogue (out_row_map = sorted pairs)
    xg = x[torch.tensor(tok, dtype=torch.long)].contiguous()       # rows already in sorted order
    y2_ref = oracle.qgemm_w4a16(np_bits(xg), codes, scales, offsets)
    out_ref, out_ref_bits = oracle.combine(y2_ref, pairs, wts, T, topk)
    out = q.qarl_qgemm_grouped(qw, xg.cuda(), d_off, M, epilogue=q.QARL_EPI_COMBINE, combine_w=d_w,
                               sorted_pairs=d_pairs, T=T, topk=topk, path=q.QARL_PATH_DECODE)
    assert norm_err_bf16(out.float().cpu().numpy(), out_ref) <= TOL_BF16
    assert flip_fraction(np_bits(out), out_ref_bits) <= MAX_FLIPS


@pytest.mark.parametrize("E,N,K,T,topk", [(8, 64, 2048, 500, 3),      # several row blocks per expert, partial last quad of ids
                                          (4, 512, 2048, 60, 3),      # 64-row blocks over a K-chunked tile
                                          (4, 1024, 2048, 200, 3),    # ... two pairs per wavefront, several row blocks
                                          (4, 64, 512, 37, 3),        # 111 pairs
                                          (6, 96, 768, 171, 5),       # 64-row blocks
                                          (128, 64, 256, 512, 8)])    # the largest routed batch: 512 tokens, 4096 pairs
def test_routed_mode_equals_grouped_decode(q, oracle, E, N, K, T, topk):
    """qarl_qgemm_routed (every workgroup lists its expert's pairs from the router's ids) against the oracle and,
    bit for bit, against the grouped decode path fed with the grouping of the same ids: plain epilogue with x per
    token, SiLU*mul, and the combine on rows in pair order."""
    seed = 1300 + K + T
    w = synth.normal_bf16((E, N, K), 0.02, seed=seed)
    x = synth.normal_bf16((T, K), 1.0, seed=seed + 1)
    lg = synth.router_logits(T, E, seed + 2, zipf_s=1.1)
    ids, wts = oracle.route(np_bits(lg), topk)
    counts, offsets, pairs = oracle.group(ids, E)
    M = T * topk
    tok = (pairs // topk).astype(np.int32)
    d_ids = _i32(np.asarray(ids).reshape(-1))
    d_off, d_tok, d_pairs = _i32(offsets), _i32(tok), _i32(pairs)
    d_w = torch.tensor(np.asarray(wts, dtype=np.float32), device="cuda")
    codes, scales = oracle.quantize_int4(np_bits(w))
    qw = q.qarl_quantize_weights(w.cuda())
    inv = torch.tensor(pairs, dtype=torch.long, device="cuda")     # sorted position i holds pair pairs[i]
    # plain epilogue, activation row = token: row pr of the routed result is row i of the grouped one, pairs[i] = pr
    y_ref = oracle.qgemm_w4a16(np_bits(x), codes, scales, offsets, tok)
    y_grp = q.qarl_qgemm_grouped(qw, x.cuda(), d_off, M, row_map=d_tok, out_dtype=q.QARL_OUT_F32,
                                 path=q.QARL_PATH_DECODE)
    y_rt = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    q.qarl_qgemm_routed(qw, x.cuda(), d_ids, T, topk, True, out=y_rt, out_dtype=q.QARL_OUT_F32)
    assert norm_err(y_rt[inv].cpu().numpy(), y_ref) <= TOL_F32
    assert torch.equal(y_rt[inv], y_grp)
    # SiLU*mul
    a_grp = q.qarl_qgemm_grouped(qw, x.cuda(), d_off, M, row_map=d_tok, epilogue=q.QARL_EPI_SILU_MUL,
                                 path=q.QARL_PATH_DECODE)
    a_rt = q.qarl_qgemm_routed(qw, x.cuda(), d_ids, T, topk, True, epilogue=q.QARL_EPI_SILU_MUL)
    assert np.array_equal(np_bits(a_rt[inv]), np_bits(a_grp))
    # combine: activation row = pair id
    xp = x[torch.tensor(np.arange(M) // topk, dtype=torch.long)].contiguous()   # one row per pair, pair order
    xg = xp[torch.tensor(pairs, dtype=torch.long)].contiguous()                 # the same rows in sorted order
    out_grp = q.qarl_qgemm_grouped(qw, xg.cuda(), d_off, M, epilogue=q.QARL_EPI_COMBINE, combine_w=d_w,
                                   sorted_pairs=d_pairs, T=T, topk=topk, path=q.QARL_PATH_DECODE)
    out_rt = q.qarl_qgemm_routed(qw, xp.cuda(), d_ids, T, topk, False, epilogue=q.QARL_EPI_COMBINE, combine_w=d_w)
    y2_ref = oracle.qgemm_w4a16(np_bits(xg), codes, scales, offsets)
    out_ref, _ = oracle.combine(y2_ref, pairs, wts, T, topk)
    assert norm_err_bf16(out_rt.float().cpu().numpy(), out_ref) <= TOL_BF16
    assert np.array_equal(np_bits(out_rt), np_bits(out_grp))


_ROUTED_QX_SHAPES = [(8, 64, 2048, 500, 3),      # several row blocks per expert, partial last quad of ids
                     (4, 512, 2048, 60, 3),      # two token tiles per block
                     (4, 64, 512, 37, 3),        # 111 pairs
                     (6, 96, 768, 171, 5),       # ring depth 3; rows with 1.5 chunks per lane
                     (3, 64, 4096, 50, 2),       # eight chunks per lane and row
                     (128, 64, 256, 512, 8)]     # the largest routed batch: 512 tokens, 4096 pairs


# (the int4 decode kernel's routed mode takes K % 256 == 0 up to 2048: W4A8 runs the shapes it accepts)
@pytest.mark.parametrize("fmt_name,E,N,K,T,topk", [(f,) + sh for f in ("fp8", "fp4", "w4a8") for sh in _ROUTED_QX_SHAPES
                                                   if f != "w4a8" or (sh[2] % 256 == 0 and sh[2] <= 2048)])
def test_routed_mode_quantizes_its_rows_like_the_row_quantizer(q, oracle, fmt_name, E, N, K, T, topk):
    """qarl_qgemm_routed on the e4m3-activation formats takes 16-bit rows and quantizes what it gathers: bit for bit
    the row quantizer followed by the grouped decode path on the grouping of the same ids, and within tolerance of
    the oracle's quantizer + GEMM.  Plain epilogue with x per token, SiLU*mul, and the combine on rows in pair
    order."""
    fmt = {"fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    seed = 1700 + K + T
    w = synth.normal_bf16((E, N, K), 0.02, seed=seed)
    x = synth.normal_bf16((T, K), 1.0, seed=seed + 1)
    x[T // 2] = 0                                                  # a zero row: scale 0, codes 0, output 0
    lg = synth.router_logits(T, E, seed + 2, zipf_s=1.1)
    ids, wts = oracle.route(np_bits(lg), topk)
    counts, offsets, pairs = oracle.group(ids, E)
    M = T * topk
    tok = (pairs // topk).astype(np.int32)
    d_ids = _i32(np.asarray(ids).reshape(-1))
    d_off, d_tok, d_pairs = _i32(offsets), _i32(tok), _i32(pairs)
    d_w = torch.tensor(np.asarray(wts, dtype=np.float32), device="cuda")
    qw = q.qarl_quantize_weights(w.cuda(), fmt)
    inv = torch.tensor(pairs, dtype=torch.long, device="cuda")     # sorted position i holds pair pairs[i]
    xq, sx = q.qarl_quantize_rows_fp8(x.cuda())
    y_grp = q.qarl_qgemm_grouped(qw, xq, d_off, M, row_map=d_tok, x_scales=sx, out_dtype=q.QARL_OUT_F32,
                                 path=q.QARL_PATH_DECODE)
    y_rt = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    q.qarl_qgemm_routed(qw, x.cuda(), d_ids, T, topk, True, out=y_rt, out_dtype=q.QARL_OUT_F32)
    assert torch.equal(y_rt[inv], y_grp)
    xq_ref, sx_ref = oracle.quantize_fp8_rows(np_bits(x))
    if fmt_name == "fp8":
        wc, wsc = oracle.quantize_fp8_rows(np_bits(w).reshape(E * N, K))
        y_ref = oracle.qgemm_fp8(xq_ref, sx_ref, wc.reshape(E, N, K), wsc.reshape(E, N), offsets, tok)
    elif fmt_name == "fp4":
        wc, wsc = oracle.quantize_fp4_rows(np_bits(w).reshape(E * N, K))
        y_ref = oracle.qgemm_fp4w(xq_ref, sx_ref, wc.reshape(E, N, K), wsc.reshape(E, N), offsets, tok)
    else:
        c4, s4 = oracle.quantize_int4(np_bits(w))
        y_ref = oracle.qgemm_w4a8(xq_ref, sx_ref, c4, s4, offsets, tok)
    assert norm_err(y_rt[inv].cpu().numpy(), y_ref) <= (TOL_F32 if fmt_name == "w4a8" else TOL_F32_FP8)
    # SiLU*mul
    a_grp = q.qarl_qgemm_grouped(qw, xq, d_off, M, row_map=d_tok, x_scales=sx, epilogue=q.QARL_EPI_SILU_MUL,
                                 path=q.QARL_PATH_DECODE)
    a_rt = q.qarl_qgemm_routed(qw, x.cuda(), d_ids, T, topk, True, epilogue=q.QARL_EPI_SILU_MUL)
    assert np.array_equal(np_bits(a_rt[inv]), np_bits(a_grp))
    # combine: activation row = pair id
    xp = x[torch.tensor(np.arange(M) // topk, dtype=torch.long)].contiguous()   # one row per pair, pair order
    xg = xp[torch.tensor(pairs, dtype=torch.long)].contiguous()                 # the same rows in sorted order
    xgq, sxg = q.qarl_quantize_rows_fp8(xg.cuda())
    out_grp = q.qarl_qgemm_grouped(qw, xgq, d_off, M, x_scales=sxg, epilogue=q.QARL_EPI_COMBINE, combine_w=d_w,
                                   sorted_pairs=d_pairs, T=T, topk=topk, path=q.QARL_PATH_DECODE)
    out_rt = q.qarl_qgemm_routed(qw, xp.cuda(), d_ids, T, topk, False, epilogue=q.QARL_EPI_COMBINE, combine_w=d_w)
    assert np.array_equal(np_bits(out_rt), np_bits(out_grp))


# Few pairs (T * topk <= 64) can take kernels of their own: one pair, one token with eight slots, several column blocks with a
# remainder, the most pairs, 16 slots (the most the fused combine takes) and 32 (two launches), one pair too many.
_FEW_PAIRS = [(64, 32, 256, 1, 1), (64, 96, 2048, 1, 8), (64, 1056, 1024, 3, 8), (64, 544, 768, 8, 8), (64, 64, 1280, 4, 16),
              (64, 64, 512, 2, 32), (64, 160, 512, 13, 5)]


@pytest.mark.parametrize("fmt_name,E,N,K,T,topk", [(f,) + sh for f in ("w4a16", "w4a8", "fp8", "fp4") for sh in _FEW_PAIRS])
def test_routed_mode_of_few_pairs_equals_grouped_decode(q, fmt_name, E, N, K, T, topk):
    """Bit for bit the grouped decode path (itself held against the oracle) on the grouping of the same ids: plain
    epilogue fp32 and bf16, SiLU*mul, the combine in fp32 and bf16 with rows per pair and per token."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    _few_pairs_case(q, fmt, synth.normal_bf16((E, N, K), 0.02, seed=K + T).cuda(), T, topk, None)


def _few_pairs_case(q, fmt, w, T, topk, fused):
    E, N, K = w.shape
    x = synth.normal_bf16((T, K), 1.0, seed=K + T + 1).cuda()
    qw = q.qarl_quantize_weights(w, fmt)
    r = q.qarl_moe_route(synth.router_logits(T, E, K + T + 2).cuda(), topk)
    M, inv = T * topk, r.pairs.long()
    ws = torch.full((M * (N + K),), -777.0, dtype=torch.float32, device="cuda")

    def grouped(rows, **kw):
        if fmt != q.QARL_W4A16_G128:
            rows, kw["x_scales"] = q.qarl_quantize_rows_fp8(rows)
        return q.qarl_qgemm_grouped(qw, rows, r.offsets, M, path=q.QARL_PATH_DECODE, **kw)

    for dt in (q.QARL_OUT_F32, q.QARL_OUT_BF16):
        got = q.qarl_qgemm_routed(qw, x, r.ids, T, topk, True, out_dtype=dt)
        assert torch.equal(got[inv], grouped(x, row_map=r.tokens, out_dtype=dt))
    got = q.qarl_qgemm_routed(qw, x, r.ids, T, topk, True, epilogue=q.QARL_EPI_SILU_MUL)
    assert torch.equal(got[inv], grouped(x, row_map=r.tokens, epilogue=q.QARL_EPI_SILU_MUL))
    xp = synth.normal_bf16((M, K), 1.0, seed=K + T + 3).cuda()           # one row per pair, pair order
    kw = dict(epilogue=q.QARL_EPI_COMBINE, combine_w=r.w)
    for dt in (q.QARL_OUT_F32, q.QARL_OUT_BF16):
        for per_token, rows, ordered in ((False, xp, xp[inv]), (True, x, x[r.tokens.long()])):
            got = q.qarl_qgemm_routed(qw, rows, r.ids, T, topk, per_token, out_dtype=dt, ws=ws, **kw)
            assert torch.equal(got, grouped(ordered.contiguous(), sorted_pairs=r.pairs, T=T, topk=topk, out_dtype=dt, **kw))
    if fused is not None:                            # no staging rows: the kernel for few pairs ran
        assert bool((ws == -777.0).all()) == fused


# Shapes whose combine runs on the kernels for few pairs (asserted), where these can go wrong.  int4: one pair, several units
# of columns per workgroup with a remainder, the most pairs, a chunk of x beyond the registers and more than 64 KiB of LDS (16
# slots).  FP8 / FP4: rows of more than four chunks per lane, a second pass over the slots and more than 64 KiB of LDS.
_FUSED = ([(f,) + sh for f in ("w4a16", "w4a8") for sh in ((64, 32, 256, 1, 1), (64, 2080, 768, 16, 4), (64, 544, 768, 8, 8),
                                                           (64, 4096, 2048, 1, 16))] +
          [(f,) + sh for f in ("fp8", "fp4") for sh in ((64, 32, 256, 1, 1), (64, 1056, 1024, 3, 8), (64, 96, 3968, 3, 8),
                                                        (256, 1056, 512, 15, 4), (64, 2048, 4096, 1, 16))])


@pytest.mark.parametrize("fmt_name,E,N,K,T,topk", _FUSED)
def test_fused_combine_of_few_pairs_equals_grouped_decode(q, fmt_name, E, N, K, T, topk):
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    _few_pairs_case(q, fmt, synth.normal_bf16((E, N, K), 0.02, seed=K + T, device="cuda"), T, topk, True)


@pytest.mark.parametrize("E,N,K,T,topk", [(128, 1056, 512, 15, 4), (64, 2048, 512, 6, 4), (128, 1024, 384, 10, 4)])
def test_fp8_combine_past_the_few_pair_line_takes_the_staging_rows(q, E, N, K, T, topk):
    """Where the streaming kernel and a combine launch are the faster by their estimate, short rows take them as long ones do."""
    _few_pairs_case(q, q.QARL_FP8_E4M3_CH, synth.normal_bf16((E, N, K), 0.02, seed=K + T, device="cuda"), T, topk, False)


def _stream_fp8_launches(call):
    """call's result, and (16-row tiles of a block, weight ring in LDS) of its qgemm_stream_fp8_kernel launches."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
        r = call()
        torch.cuda.synchronize()
    args = [e.name.split("qgemm_stream_fp8_kernel<")[1].split(">")[0].split(", ") for e in prof.events() if "qgemm_stream_fp8_kernel<" in e.name]
    return r, [(int(a[1]), a[5] != "0") for a in args]   # <epilogue, tiles, ring depth, e2m1, routed, ring, shares>


@pytest.mark.parametrize("fmt_name", ["fp8", "fp4"])
@pytest.mark.parametrize("E,N,K,T,topk,tiles,ring", [   # ring: the formats that keep it in LDS
    (16, 96, 128, 100, 2, 2, ()),                       # fewer stages than the ring in LDS has: registers
    (16, 96, 256, 100, 2, 2, ("fp8",)),                 # as many (FP4: fewer)
    (16, 64, 384, 60, 2, 2, ("fp8",)),                  # one more (FP4: half a stage, registers)
    (16, 544, 768, 65, 1, 1, ("fp8", "fp4")),           # 16-row blocks, slices of six and five pairs
    (128, 1056, 768, 20, 4, 1, ("fp8", "fp4")),         # slices of 17 and 16 pairs: a wavefront's second and third pair; six stages, FP4 three
    (128, 1056, 640, 100, 4, 1, ("fp8",)),              # ... five stages
    (128, 1056, 1280, 300, 4, 2, ("fp8", "fp4")),       # ... blocks of 32 rows, ten stages, FP4 five
    (128, 1056, 640, 300, 8, 4, ("fp8",)),              # ... of 64 rows, five stages
    (128, 1056, 1280, 300, 8, 4, ("fp8", "fp4")),       # ... ten, FP4 five
    (128, 512, 768, 300, 8, 4, ("fp8", "fp4")),         # 64-row blocks, a pair per wavefront
    (16, 32, 1024, 500, 2, 2, ("fp8", "fp4")),          # several row blocks of 32: temporal copies
    (3, 64, 2048, 90, 2, 2, ("fp8", "fp4"))])           # a token tile that fills most of the LDS
def test_routed_ring_in_lds_equals_the_register_ring(q, fmt_name, E, N, K, T, topk, tiles, ring):
    """The grouped decode call keeps its weight ring in registers.  Every output kind, bit for bit, and no row in front of the
    output or behind it: rows past an expert's end are stored out of the bounds of a buffer that ends with the output."""
    fmt = q.QARL_FP8_E4M3_CH if fmt_name == "fp8" else q.QARL_FP4_E2M1_CH
    M = T * topk
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=K + N, device="cuda"), fmt)
    x = synth.normal_bf16((T, K), 1.0, seed=K + T, device="cuda")
    r = q.qarl_moe_route(synth.router_logits(T, 64 * ((E + 63) // 64), T, device="cuda"), topk)
    ids = (r.ids % E).reshape(-1).contiguous()
    pairs = torch.argsort(ids, stable=True)
    off = _i32(np.concatenate([[0], np.cumsum(np.bincount(ids.cpu().numpy(), minlength=E))]))
    xq, sx = q.qarl_quantize_rows_fp8(x)
    for epi, dt in ((q.QARL_EPI_NONE, q.QARL_OUT_F32), (q.QARL_EPI_NONE, q.QARL_OUT_BF16), (q.QARL_EPI_SILU_MUL, q.QARL_OUT_BF16)):
        want = q.qarl_qgemm_grouped(qw, xq, off, M, row_map=(pairs // topk).int(), x_scales=sx, epilogue=epi, out_dtype=dt,
                                    path=q.QARL_PATH_DECODE)
        buf = torch.full((M + 2, want.shape[1]), 7.0, dtype=want.dtype, device="cuda")
        _, ran = _stream_fp8_launches(lambda: q.qarl_qgemm_routed(qw, x, ids, T, topk, True, epilogue=epi, out=buf[1:1 + M], out_dtype=dt))
        assert ran == [(tiles, fmt_name in ring)]
        assert torch.equal(buf[1:1 + M][pairs], want)
        assert bool((buf[0] == 7).all()) and bool((buf[M + 1] == 7).all())


@pytest.mark.parametrize("K,tiles", [(2048, 2), (1920, 4), (1408, 4), (384, 4), (256, 4)])
def test_fp4_block_height_follows_the_ring(q, K, tiles):
    """More than 32 rows per expert to expect: two blocks of 32 rows only where that makes room for the ring in LDS (K = 2048).
    An odd number of 128-k groups, or fewer stages than the ring has, never takes it and keeps one block of 64.  Same bits."""
    E, N, T, topk = 128, 512, 300, 8
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=K, device="cuda"), q.QARL_FP4_E2M1_CH)
    x = synth.normal_bf16((T, K), 1.0, seed=T, device="cuda")
    r = q.qarl_moe_route(synth.router_logits(T, E, T, device="cuda"), topk)
    xq, sx = q.qarl_quantize_rows_fp8(x)
    want = q.qarl_qgemm_grouped(qw, xq, r.offsets, T * topk, row_map=r.tokens, x_scales=sx, out_dtype=q.QARL_OUT_F32, path=q.QARL_PATH_DECODE)
    got, ran = _stream_fp8_launches(lambda: q.qarl_qgemm_routed(qw, x, r.ids, T, topk, True, out_dtype=q.QARL_OUT_F32))
    assert torch.equal(got[r.pairs.long()], want)
    assert [t for t, _ in ran] == [tiles]


@pytest.mark.parametrize("fmt_name,T", [("fp8", 40), ("w4a8", 40), ("fp8", 8), ("w4a8", 8), ("fp4", 8)])   # 80 and 16 pairs
def test_routed_mode_rows_outside_the_fast_division_range(q, oracle, fmt_name, T):
    """Rows whose scale leaves the range of the corrected-reciprocal division (absmax near 2^-100 and near 2^100),
    a zero row, negative zeros and a row of one repeated value: the kernel that quantizes its own rows must fall back
    to the IEEE division exactly where the row quantizer does, so routed and grouped results stay bit-identical, and
    the codes the grouped path consumed are the oracle's."""
    fmt = {"fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    E, N, K, topk = 4, 64, 512, 2
    w = synth.normal_bf16((E, N, K), 0.02, seed=1901)
    x = synth.normal_bf16((T, K), 1.0, seed=1902).float()
    x[0] *= 2.0 ** -110
    x[1] *= 2.0 ** 115
    x[2] = 0
    x[3] = 0.375
    x[4, :9] = -0.0
    x[5] *= 2.0 ** -126            # bf16 subnormals
    x = x.to(torch.bfloat16)
    lg = synth.router_logits(T, E, 1903)
    ids, _ = oracle.route(np_bits(lg), topk)
    counts, offsets, pairs = oracle.group(ids, E)
    M = T * topk
    tok = (pairs // topk).astype(np.int32)
    qw = q.qarl_quantize_weights(w.cuda(), fmt)
    xq, sx = q.qarl_quantize_rows_fp8(x.cuda())
    xq_ref, sx_ref = oracle.quantize_fp8_rows(np_bits(x))
    assert np.array_equal(xq.cpu().numpy(), xq_ref) and np.array_equal(sx.cpu().numpy(), sx_ref)
    y_grp = q.qarl_qgemm_grouped(qw, xq, _i32(offsets), M, row_map=_i32(tok), x_scales=sx, out_dtype=q.QARL_OUT_F32,
                                 path=q.QARL_PATH_DECODE)
    y_rt = q.qarl_qgemm_routed(qw, x.cuda(), _i32(np.asarray(ids).reshape(-1)), T, topk, True, out_dtype=q.QARL_OUT_F32)
    inv = torch.tensor(pairs, dtype=torch.long, device="cuda")
    assert torch.equal(y_rt[inv].view(torch.int32), y_grp.view(torch.int32))


def test_routed_mode_errors_and_route_only(q):
    w = synth.normal_bf16((64, 32, 256), 0.02, seed=3).cuda()
    qw = q.qarl_quantize_weights(w)
    x = synth.normal_bf16((600, 256), 1.0, seed=4).cuda()
    ids = torch.zeros((600 * 8,), dtype=torch.int32, device="cuda")
    with pytest.raises(q.QarlError) as ei:                       # more than 512 tokens
        q.qarl_qgemm_routed(qw, x, ids, 600, 8, True)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED
    with pytest.raises(q.QarlError) as ei:                       # more than 4096 pairs
        q.qarl_qgemm_routed(qw, x, ids, 500, 9, True)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED
    q8 = q.qarl_quantize_weights(synth.normal_bf16((4, 32, 4096), 0.02, seed=5).cuda(), q.QARL_W4A8_G128)
    with pytest.raises(q.QarlError) as ei:                       # the int4 kernels' routed mode stops at K = 2048
        q.qarl_qgemm_routed(q8, synth.normal_bf16((16, 4096), 1.0, seed=6).cuda(), ids, 16, 8, True)
    assert ei.value.status == q.QARL_ERR_UNSUPPORTED
    out = q.qarl_qgemm_routed(qw, x, ids, 0, 8, True)            # T = 0: nothing to do
    assert out.shape[0] == 0
    # the router without its grouping pass writes the same ids and weights
    lg = synth.router_logits(300, 64, 9).cuda()
    r1 = q.qarl_moe_route(lg, 4)
    r2 = q.qarl_moe_route(lg, 4, group=False)
    assert torch.equal(r1.ids, r2.ids) and torch.equal(r1.w, r2.w)


@pytest.mark.parametrize("path", [1, 2])
def test_layer_is_reproducible_run_to_run(q, path):
    """Wavefronts draw their weight tiles dynamically and workgroups finish in any order; no result may depend on
    it: repeated runs of one layer give the same bits, interleaved with a different batch in between."""
    E, H, I, T, topk = 64, 512, 256, 301, 4
    gu, dn = synth.expert_weights(E, H, I, seed=77)
    layer = q.MoELayer(q.qarl_quantize_weights(gu.cuda()), q.qarl_quantize_weights(dn.cuda()), T, topk, path)
    x = synth.normal_bf16((T, H), 1.0, 78).cuda()
    lg = synth.router_logits(T, E, 79, zipf_s=1.1).cuda()
    x2 = synth.normal_bf16((T, H), 1.0, 80).cuda()
    lg2 = synth.router_logits(T, E, 81).cuda()
    first = layer.forward(x, lg).clone()
    for _ in range(5):
        layer.forward(x2, lg2)
        again = layer.forward(x, lg)
        assert torch.equal(first.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("fmt_name,T", [(f, T) for f in ("w4a16", "w4a8", "fp8", "fp4") for T in (20, 200)])   # few pairs and many
def test_routed_mode_ids_outside_the_expert_range_leave_their_rows_alone(q, oracle, fmt_name, T):
    """Pairs whose id is not an expert (negative, >= E) select no weight matrix: their output rows keep what the
    buffer held, every other row is unaffected."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    E, N, K, topk = 4, 64, 256, 2
    w = synth.normal_bf16((E, N, K), 0.02, seed=31)
    x = synth.normal_bf16((T, K), 1.0, seed=32)
    rng = np.random.default_rng(33)
    ids = rng.integers(0, E, size=(T, topk)).astype(np.int32)
    ids[:, 1] = (ids[:, 0] + 1) % E                               # a token lists an expert at most once
    good = ids.copy()
    ids[2, 0], ids[7, 1], ids[19, 1] = -1, E, 1000
    qw = q.qarl_quantize_weights(w.cuda(), fmt)
    M = T * topk
    y = torch.full((M, N), -777.0, dtype=torch.float32, device="cuda")
    q.qarl_qgemm_routed(qw, x.cuda(), _i32(ids.reshape(-1)), T, topk, True, out=y, out_dtype=q.QARL_OUT_F32)
    y2 = torch.full((M, N), -777.0, dtype=torch.float32, device="cuda")
    q.qarl_qgemm_routed(qw, x.cuda(), _i32(good.reshape(-1)), T, topk, True, out=y2, out_dtype=q.QARL_OUT_F32)
    skipped = [2 * topk + 0, 7 * topk + 1, 19 * topk + 1]
    keep = np.ones(M, dtype=bool)
    keep[skipped] = False
    assert bool((y[skipped] == -777.0).all())
    assert torch.equal(y[torch.tensor(keep)], y2[torch.tensor(keep)])


@pytest.mark.parametrize("fmt_name", ["w4a16", "w4a8", "fp8", "fp4"])
def test_routed_combine_written_over_its_own_input(q, fmt_name):
    """The combined rows may land on top of x or of the ids: they are written when every workgroup has read both."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    E, N, K, T, topk = 64, 512, 512, 8, 8
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=61).cuda(), fmt)
    x = synth.normal_bf16((T, K), 1.0, seed=62).cuda()
    r = q.qarl_moe_route(synth.router_logits(T, E, 63).cuda(), topk)
    kw = dict(epilogue=q.QARL_EPI_COMBINE, combine_w=r.w)
    want = q.qarl_qgemm_routed(qw, x, r.ids, T, topk, True, **kw)
    over_x = x.clone()
    q.qarl_qgemm_routed(qw, over_x, r.ids, T, topk, True, out=over_x, **kw)
    assert torch.equal(over_x, want)
    buf = torch.zeros((T * N * 2,), dtype=torch.uint8, device="cuda")
    ids = buf.view(torch.int32)[:T * topk]
    ids.copy_(r.ids.reshape(-1))
    over_ids = buf.view(torch.bfloat16).reshape(T, N)
    q.qarl_qgemm_routed(qw, x, ids, T, topk, True, out=over_ids, **kw)
    assert torch.equal(over_ids, want)


@pytest.mark.parametrize("fmt_name,T", [(f, T) for f in ("w4a16", "w4a8", "fp8", "fp4") for T in (3, 200)])   # few pairs and many
def test_routed_rows_written_over_their_own_input(q, fmt_name, T):
    """256 experts: an expert's rows are read and written by one workgroup, so the rows of the plain and of the SiLU*mul epilogue
    may replace the rows of x they come from (as wide as these in bf16)."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    E, K, topk = 256, 512, 8
    ids = q.qarl_moe_route(synth.router_logits(T, E, 91).cuda(), topk).ids
    x = synth.normal_bf16((T * topk, K), 1.0, seed=92).cuda()
    for N, epi in ((K, q.QARL_EPI_NONE), (2 * K, q.QARL_EPI_SILU_MUL)):
        qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=93).cuda(), fmt)
        want = q.qarl_qgemm_routed(qw, x, ids, T, topk, False, epilogue=epi)
        over = x.clone()
        q.qarl_qgemm_routed(qw, over, ids, T, topk, False, epilogue=epi, out=over)
        assert torch.equal(over, want)


@pytest.mark.parametrize("fmt_name,T", [(f, T) for f in ("w4a16", "w4a8", "fp8", "fp4") for T in (8, 200)])
def test_routed_combine_counts_ids_outside_the_expert_range_as_zeros(q, fmt_name, T):
    """Few and many pairs, whatever the workspace and the weights of such slots hold, also with out on top of the ids: the
    same as with a weight of zero on a row that exists."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    E, N, K, topk = 64, 160, 512, 4
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=71).cuda(), fmt)
    x = synth.normal_bf16((T * topk, K), 1.0, seed=72).cuda()
    r = q.qarl_moe_route(synth.router_logits(T, E, 73).cuda(), topk)
    ids, w = r.ids.clone(), r.w.clone()
    for t, slot, bad in ((0, 0, -1), (2, 3, E), (3, 1, 2 ** 31 - 1), (T - 1, 2, -2 ** 31)):
        ids[t, slot] = bad
        w[t, slot] = 0.0
    ids[5] = -1
    w[5] = 0.0
    kw = dict(epilogue=q.QARL_EPI_COMBINE, out_dtype=q.QARL_OUT_F32)
    want = q.qarl_qgemm_routed(qw, x, r.ids, T, topk, False, combine_w=w, **kw)
    ws = torch.full((T * topk * (N + K // 128 + K),), float("nan"), dtype=torch.float32, device="cuda")
    got = q.qarl_qgemm_routed(qw, x, ids, T, topk, False, combine_w=r.w, ws=ws, **kw)
    assert torch.equal(got, want) and bool((got[5] == 0).all())
    ws.fill_(float("nan"))
    buf = torch.zeros((T, N), dtype=torch.float32, device="cuda")
    over = buf.view(torch.int32).view(-1)[:T * topk]
    over.copy_(ids.reshape(-1))
    q.qarl_qgemm_routed(qw, x, over, T, topk, False, combine_w=r.w, ws=ws, out=buf, **kw)
    assert torch.equal(buf, want)


@pytest.mark.parametrize("fmt_name,E,N,K,T,topk,staged", [
    ("w4a16", 6, 4096, 2048, 10, 6, True), ("w4a8", 6, 4096, 2048, 10, 6, True), ("fp8", 6, 4096, 2048, 4, 6, True),
    ("fp4", 6, 4096, 2048, 10, 6, True), ("fp8", 1, 1024, 512, 64, 1, True), ("fp4", 128, 2048, 768, 64, 1, True),
    ("w4a16", 128, 2048, 768, 8, 8, False), ("w4a8", 1, 512, 256, 1, 1, False), ("fp8", 128, 2048, 768, 2, 8, False),
    ("fp4", 6, 1024, 512, 1, 6, False)])
def test_routed_combine_of_few_pairs_reads_shared_weights_once(q, fmt_name, E, N, K, T, topk, staged):
    """Pairs that share their experts' weights go through the kernel that reads a matrix once for all of its rows, which stages
    its rows in the workspace; few pairs of many experts don't touch it.  The same bits as grouped decode either way."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=81).cuda(), fmt)
    M = T * topk
    x = synth.normal_bf16((M, K), 1.0, seed=82).cuda()
    rng = np.random.default_rng(83)
    ids = torch.tensor(np.stack([rng.permutation(E)[:topk] for _ in range(T)]).astype(np.int32), device="cuda")
    w = torch.tensor(rng.random((T, topk)).astype(np.float32), device="cuda")
    ws = torch.full((M * (N + K),), -777.0, dtype=torch.float32, device="cuda")
    kw = dict(epilogue=q.QARL_EPI_COMBINE, combine_w=w, out_dtype=q.QARL_OUT_F32)
    got = q.qarl_qgemm_routed(qw, x, ids, T, topk, False, ws=ws, **kw)
    assert bool((ws[:M * N] != -777.0).all()) == staged and (staged or bool((ws == -777.0).all()))
    pairs = torch.argsort(ids.view(-1), stable=True)
    off = torch.zeros((E + 1,), dtype=torch.int32, device="cuda")
    off[1:] = torch.cumsum(torch.bincount(ids.view(-1).long(), minlength=E), 0)
    rows = x[pairs].contiguous()
    if fmt != q.QARL_W4A16_G128:
        rows, kw["x_scales"] = q.qarl_quantize_rows_fp8(rows)
    want = q.qarl_qgemm_grouped(qw, rows, off, M, sorted_pairs=pairs.int(), T=T, topk=topk, path=q.QARL_PATH_DECODE, **kw)
    assert torch.equal(got, want)


@pytest.mark.parametrize("fmt_name", ["w4a16", "w4a8"])
@pytest.mark.parametrize("T,topk", [(64, 5), (80, 4)])   # no expert can pass the grid's 64 rows; one could (the kernels with shares)
@pytest.mark.parametrize("N,K", [(512, 2048), (96, 768), (288, 1024)])   # 64-row blocks: K-chunked tile, rings of three and four
def test_int4_row_blocks_at_the_edge_of_a_row_tile(q, fmt_name, N, K, T, topk):
    """64-row blocks run one or two row tiles, by the expert's rows: 64, 33, 32, 31, 1 and 0 rows, and some between, give bit for bit what the
    kernel of 32-row blocks gives on at most 16 rows at a time."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    E, M = 16, T * topk
    mean = M / E
    assert mean + 3.75 * mean ** 0.5 > 32 >= mean + 2.6 * mean ** 0.5    # blocks of 64 rows, one row tile allowed
    t = torch.arange(T)
    fill = [[6], [7], [8, 9, 10], [11, 12, 13], [14, 15]]                # the experts of a slot that none of the six takes
    ids = torch.stack([torch.tensor(fill[s])[t % len(fill[s])] for s in range(topk)], 1)
    ids[:64, 0] = 0
    ids[:33, 1], ids[33:64, 1] = 1, 3        # 33 and 31
    ids[:32, 2], ids[32, 2] = 2, 4           # 32 and 1
    counts = torch.bincount(ids.flatten(), minlength=E).tolist()
    assert counts[:6] == [64, 33, 32, 31, 1, 0] and max(counts) == 64
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=K + N, device="cuda"), fmt)
    x = synth.normal_bf16((T, K), 1.0, seed=T, device="cuda")
    pairs = torch.argsort(ids.flatten(), stable=True).cuda()
    tok, d_ids = (pairs // topk).int(), ids.int().flatten().cuda()
    rows, kw = x, {}
    if fmt != q.QARL_W4A16_G128:
        rows, kw["x_scales"] = q.qarl_quantize_rows_fp8(x)
    off = torch.tensor([0] + np.cumsum(counts).tolist(), dtype=torch.int32, device="cuda")
    for epi, dt in ((q.QARL_EPI_NONE, q.QARL_OUT_F32), (q.QARL_EPI_SILU_MUL, q.QARL_OUT_BF16)):
        routed = q.qarl_qgemm_routed(qw, x, d_ids, T, topk, True, epilogue=epi, out_dtype=dt)[pairs]
        grouped = q.qarl_qgemm_grouped(qw, rows, off, M, row_map=tok, epilogue=epi, out_dtype=dt, path=q.QARL_PATH_DECODE, **kw)
        for e, n in enumerate(counts):
            for r0 in range(0, n, 16):
                n16, at = min(16, n - r0), sum(counts[:e]) + r0
                one = torch.tensor([0 if i <= e else n16 for i in range(E + 1)], dtype=torch.int32, device="cuda")
                want = q.qarl_qgemm_grouped(qw, rows, one, n16, row_map=tok[at:at + n16].contiguous(), epilogue=epi, out_dtype=dt,
                                            path=q.QARL_PATH_DECODE, **kw)
                assert torch.equal(routed[at:at + n16], want) and torch.equal(grouped[at:at + n16], want)


@pytest.mark.parametrize("fmt_name", ["w4a16", "w4a8"])
@pytest.mark.parametrize("T", [257, 266, 267])        # 128 experts top-8: 32-row blocks with dealt shares end at 266 tokens
@pytest.mark.parametrize("N,K,zipf", [(512, 2048, 0.0), (512, 2048, 1.1), (96, 768, 1.1)])
def test_int4_block_height_of_many_experts(q, fmt_name, T, N, K, zipf):
    """Blocks of 32 or 64 rows, by the routed call's expected rows: bit for bit the grouped call's results."""
    fmt, E, topk = {"w4a16": q.QARL_W4A16_G128, "w4a8": q.QARL_W4A8_G128}[fmt_name], 128, 8
    M = T * topk
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=K + N, device="cuda"), fmt)
    x = synth.normal_bf16((T, K), 1.0, seed=T, device="cuda")
    r = q.qarl_moe_route(synth.router_logits(T, E, T, device="cuda", zipf_s=zipf), topk)
    ids = r.ids.reshape(-1).contiguous()
    pairs = torch.argsort(ids, stable=True)
    off = _i32(np.concatenate([[0], np.cumsum(np.bincount(ids.cpu().numpy(), minlength=E))]))
    rows, kw = x, {}
    if fmt != q.QARL_W4A16_G128:
        rows, kw["x_scales"] = q.qarl_quantize_rows_fp8(x)
    for epi, dt in ((q.QARL_EPI_NONE, q.QARL_OUT_F32), (q.QARL_EPI_SILU_MUL, q.QARL_OUT_BF16)):
        want = q.qarl_qgemm_grouped(qw, rows, off, M, row_map=(pairs // topk).int(), epilogue=epi, out_dtype=dt, path=q.QARL_PATH_DECODE, **kw)
        got = q.qarl_qgemm_routed(qw, x, ids, T, topk, True, epilogue=epi, out_dtype=dt)[pairs]
        assert torch.equal(got, want)


@pytest.mark.parametrize("fmt_name,E,N,K,T,topk,named", [
    ("w4a16", 16, 64, 512, 512, 4, 4),         # every token names the same experts: the others' workgroups take their row blocks
    ("w4a16", 3, 96, 256, 200, 2, 3),          # no workgroup without rows, a slice of three pairs of tiles
    ("w4a16", 256, 32, 256, 512, 8, 9),        # as many experts as the counts hold, one pair of tiles per slice
    ("w4a16", 257, 32, 256, 512, 8, 9),        # one more: further blocks are passes
    ("w4a16", 70, 1536, 2048, 512, 4, 40),     # 64-row blocks over a K-chunked tile, three pairs per wavefront, shares of one
    ("fp8", 96, 544, 2048, 512, 8, 60), ("fp4", 70, 512, 512, 512, 4, 70),   # blocks of 64 rows, slices that are no multiple of eight pairs
    ("w4a8", 8, 288, 1024, 150, 3, 3), ("fp8", 8, 288, 2048, 100, 3, 4), ("fp8", 5, 64, 128, 17, 2, 2),
    ("fp4", 64, 96, 512, 512, 8, 8), ("fp4", 64, 512, 256, 37, 8, 20)])
@pytest.mark.parametrize("twice", [False, True])
def test_routed_row_blocks_of_popular_experts_equal_grouped_decode(q, fmt_name, E, N, K, T, topk, named, twice):
    """Bit for bit the grouped decode path where only the first `named` experts have rows; twice: every token names its first
    expert in its last slot too, so that an expert may have more rows than there are tokens (up to the 512 the call lists)."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    g = torch.Generator().manual_seed(E + N + K + T)
    ids = torch.stack([torch.randperm(named, generator=g)[:topk] for _ in range(T)])
    if twice:
        ids[:, -1] = ids[:, 0]
        if int(torch.bincount(ids.flatten()).max()) > 512:
            pytest.skip("an expert lists at most 512 rows")
    M = T * topk
    pairs = torch.argsort(ids.flatten(), stable=True)
    off = torch.zeros(E + 1, dtype=torch.int32)
    off[1:] = torch.cumsum(torch.bincount(ids.flatten(), minlength=E), 0)
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=K + N, device="cuda"), fmt)
    x = synth.normal_bf16((T, K), 1.0, seed=T, device="cuda")
    rows, kw = x, {}
    if fmt != q.QARL_W4A16_G128:
        rows, kw["x_scales"] = q.qarl_quantize_rows_fp8(x)
    d_ids, d_tok, d_pairs = ids.int().flatten().cuda(), (pairs // topk).int().cuda(), pairs.cuda()
    for epi, dt in ((q.QARL_EPI_NONE, q.QARL_OUT_F32), (q.QARL_EPI_SILU_MUL, q.QARL_OUT_BF16)):
        want = q.qarl_qgemm_grouped(qw, rows, off.cuda(), M, row_map=d_tok, epilogue=epi, out_dtype=dt, path=q.QARL_PATH_DECODE, **kw)
        got = torch.full_like(want, float("nan"))
        q.qarl_qgemm_routed(qw, x, d_ids, T, topk, True, epilogue=epi, out=got, out_dtype=dt)
        assert torch.equal(got[d_pairs], want)


@pytest.mark.parametrize("fmt_name", ["w4a16", "w4a8", "fp8", "fp4"])
@pytest.mark.parametrize("E,N,K,T,topk,named", [(64, 544, 512, 256, 8, 12),    # slices of 9 and 8 pairs, two shares each: the last one has none
                                                (2, 4128, 256, 100, 2, 2),     # 129 pairs in 16 slices of nine: the last slice has none
                                                (4, 4128, 256, 100, 1, 1)])    # ... and takes a share of the popular expert's
def test_shares_and_slices_without_columns(q, oracle, fmt_name, E, N, K, T, topk, named):
    """The last `named` experts have all the rows, so a workgroup that counted past its last pair of weight tiles would look
    behind the codes and scales.  Routed and grouped decode path bit for bit, W4A16 against the oracle too."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    g = torch.Generator().manual_seed(E + N)
    ids = torch.stack([E - 1 - torch.randperm(named, generator=g)[:topk] for _ in range(T)])
    M = T * topk
    pairs = torch.argsort(ids.flatten(), stable=True)
    off = torch.zeros(E + 1, dtype=torch.int32)
    off[1:] = torch.cumsum(torch.bincount(ids.flatten(), minlength=E), 0)
    w, x = synth.normal_bf16((E, N, K), 0.02, seed=N), synth.normal_bf16((T, K), 1.0, seed=T)
    qw, xd, kw = q.qarl_quantize_weights(w.cuda(), fmt), x.cuda(), {}
    rows = xd
    if fmt != q.QARL_W4A16_G128:
        rows, kw["x_scales"] = q.qarl_quantize_rows_fp8(xd)
    y = q.qarl_qgemm_grouped(qw, rows, off.cuda(), M, row_map=(pairs // topk).int().cuda(), out_dtype=q.QARL_OUT_F32,
                             path=q.QARL_PATH_DECODE, **kw)
    got = torch.full_like(y, float("nan"))
    q.qarl_qgemm_routed(qw, xd, ids.int().flatten().cuda(), T, topk, True, out=got, out_dtype=q.QARL_OUT_F32)
    assert torch.equal(got[pairs.cuda()], y)
    if fmt == q.QARL_W4A16_G128:
        ref = oracle.qgemm_w4a16(np_bits(x), *oracle.quantize_int4(np_bits(w)), off.numpy(), (pairs // topk).numpy().astype(np.int32))
        assert norm_err(y.cpu().numpy(), ref) <= TOL_F32


@pytest.mark.parametrize("fmt_name", ["w4a16", "w4a8", "fp8", "fp4"])
@pytest.mark.parametrize("E,rows", [(64, 8), (64, 9), (64, 16), (64, 17), (64, 64), (48, 17), (48, 64), (3, 8), (3, 9), (257, 20)])
def test_auto_path_by_rows_per_expert(q, fmt_name, E, rows):
    """Bit for bit the path the rule names; the streaming one where the workspace does not hold the tiled path's, or out is x."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    tiled = rows > 8 if fmt_name == "fp8" else E >= 64 and rows > 16
    if E > 256:
        tiled = None
    N = K = 256
    M = E * rows
    cut = np.sort(np.random.default_rng(E + rows).integers(0, M + 1, E - 1))
    off = _i32(np.concatenate([[0], cut, [M]]))
    qw = q.qarl_quantize_weights(synth.normal_bf16((E, N, K), 0.02, seed=E, device="cuda"), fmt)
    x, kw = synth.normal_bf16((M, K), 1.0, seed=rows, device="cuda"), {}
    if fmt != q.QARL_W4A16_G128:
        x, kw["x_scales"] = q.qarl_quantize_rows_fp8(x)
    by = {p: q.qarl_qgemm_grouped(qw, x, off, M, path=p, out_dtype=q.QARL_OUT_F32, **kw) for p in _paths(q)
          if tiled is not None or p == q.QARL_PATH_DECODE}                    # (the tiled path takes at most 256 experts)
    got = q.qarl_qgemm_grouped(qw, x, off, M, out_dtype=q.QARL_OUT_F32, **kw)
    assert torch.equal(got, by[q.QARL_PATH_PREFILL if tiled else q.QARL_PATH_DECODE])
    if fmt == q.QARL_W4A16_G128:
        none = torch.empty((16,), dtype=torch.uint8, device="cuda")
        assert torch.equal(q.qarl_qgemm_grouped(qw, x, off, M, out_dtype=q.QARL_OUT_F32, ws=none), by[q.QARL_PATH_DECODE])
        over = x.clone()                                                      # K = N: row i of the result on top of row i of x
        q.qarl_qgemm_grouped(qw, over, off, M, out=over)
        assert torch.equal(over, q.qarl_qgemm_grouped(qw, x, off, M, path=q.QARL_PATH_DECODE))


@pytest.mark.parametrize("fmt_name", ["w4a16", "w4a8", "fp8", "fp4"])
@pytest.mark.parametrize("E,T,topk", [(64, 1, 1), (128, 1, 8), (192, 3, 5), (256, 8, 8), (128, 5, 16), (128, 40, 8)])
def test_layer_in_one_call_equals_its_three_calls(q, fmt_name, E, T, topk):
    """Few tokens: gate_up routes its tokens itself; many: the router is launched in front.  Bit for bit, ids and weights too,
    equal logits included; also where an output lies on an input, which keeps the router's launch."""
    fmt = {"w4a16": q.QARL_W4A16_G128, "fp8": q.QARL_FP8_E4M3_CH, "fp4": q.QARL_FP4_E2M1_CH, "w4a8": q.QARL_W4A8_G128}[fmt_name]
    H = I = 256
    gu, dn = synth.expert_weights(E, H, I, seed=E + T, device="cuda")
    gu, dn = q.qarl_quantize_weights(gu, fmt), q.qarl_quantize_weights(dn, fmt)
    x = synth.normal_bf16((T, H), 1.0, seed=T, device="cuda")
    lg = synth.router_logits(T, E, seed=E, device="cuda")
    lg[:, 1::2] = lg[:, ::2]                                       # every logit twice: the lower id wins
    for renorm in (1, 0):
        r = q.qarl_moe_route(lg, topk, bool(renorm))
        a = q.qarl_qgemm_routed(gu, x, r.ids, T, topk, True, epilogue=q.QARL_EPI_SILU_MUL)
        want = q.qarl_qgemm_routed(dn, a, r.ids, T, topk, False, epilogue=q.QARL_EPI_COMBINE, combine_w=r.w)
        for shared in (False, True):
            ids = torch.full((T * topk,), -7, dtype=torch.int32, device="cuda")
            w = torch.full((T * topk,), float("nan"), device="cuda")
            got_a, out = torch.full_like(a, float("nan")), torch.full_like(want, float("nan"))
            logits = lg.clone()
            if shared:                                             # the ids are written over the logits they come from
                if T * topk * 4 > logits.numel() * 2:
                    continue
                ids = logits.view(torch.int32).flatten()[:T * topk]
            ws = torch.empty((max(q.qarl_qgemm_workspace_bytes(dn, T * topk, T * topk, q.QARL_EPI_COMBINE), 16),), dtype=torch.uint8, device="cuda")
            q._check(q.lib().qarl_moe_layer_routed(q.C.byref(gu.desc), q.C.byref(dn.desc), x.data_ptr(), logits.data_ptr(), T, topk, renorm,
                                                   ids.data_ptr(), w.data_ptr(), got_a.data_ptr(), out.data_ptr(), q.QARL_OUT_BF16,
                                                   ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream))
            assert torch.equal(ids, r.ids.flatten()) and torch.equal(w, r.w.flatten())
            assert torch.equal(got_a, a) and torch.equal(out, want)
    layer = q.MoELayer(gu, dn, T, topk, q.QARL_PATH_DECODE)
    r = q.qarl_moe_route(lg, topk)
    assert torch.equal(layer.forward(x, lg), q.qarl_qgemm_routed(dn, q.qarl_qgemm_routed(gu, x, r.ids, T, topk, True, epilogue=q.QARL_EPI_SILU_MUL),
                                                                 r.ids, T, topk, False, epilogue=q.QARL_EPI_COMBINE, combine_w=r.w))


def test_layer_in_one_call_errors(q):
    gu, dn = synth.expert_weights(64, 256, 256, seed=1, device="cuda")
    gu, dn = q.qarl_quantize_weights(gu), q.qarl_quantize_weights(dn)
    t = torch.zeros((1 << 16,), dtype=torch.uint8, device="cuda")

    def call(g, d, T, topk, logits=True, ws=t.numel()):
        p = t.data_ptr()
        with pytest.raises(q.QarlError) as ei:
            q._check(q.lib().qarl_moe_layer_routed(q.C.byref(g.desc), q.C.byref(d.desc), p, p if logits else None, T, topk, 1, p, p, p, p, 0, p, ws, None))
        return ei.value.status
    assert call(dn, dn, 1, 8) == q.QARL_ERR_INVALID_ARG            # the second matrices do not follow the first
    assert call(gu, dn, 1, 65) == q.QARL_ERR_UNSUPPORTED           # the router's limits
    assert call(gu, dn, -1, 8) == q.QARL_ERR_INVALID_ARG
    assert call(gu, dn, 1, 8, logits=False) == q.QARL_ERR_INVALID_ARG
    assert call(gu, dn, 513, 1) == q.QARL_ERR_UNSUPPORTED          # the routed GEMMs' limits


def test_layer_in_one_call_is_refused_before_it_writes(q):
    """What only the second GEMM is refused for leaves ids, weights and intermediate rows as they were."""
    gu, dn = synth.expert_weights(64, 256, 256, seed=1, device="cuda")
    w4 = q.qarl_quantize_weights(gu), q.qarl_quantize_weights(dn)
    narrow = synth.expert_weights(64, 256, 128, seed=1, device="cuda")              # int4 down: K = 128 is no multiple of 256
    narrow = [q.qarl_quantize_weights(w) for w in narrow]
    for T in (1, 40):                                                               # the router inside gate_up, and in front of it
        x, lg = synth.normal_bf16((T, 256), 1.0, seed=2, device="cuda"), synth.router_logits(T, 64, seed=3, device="cuda")
        need = T * 8 * 256 * 4
        ws = torch.empty((need + 256,), dtype=torch.uint8, device="cuda")
        for (g, d), ws_at, ws_bytes, out_at, dt, status in ((w4, 0, need - 1, 0, 0, q.QARL_ERR_WORKSPACE), (w4, 8, need, 0, 0, q.QARL_ERR_WORKSPACE),
                                                            (w4, 0, need, 2, 0, q.QARL_ERR_ALIGNMENT), (w4, 0, need, 0, 7, q.QARL_ERR_INVALID_ARG),
                                                            (narrow, 0, need, 0, 0, q.QARL_ERR_UNSUPPORTED)):
            ids = torch.full((T * 8,), -7, dtype=torch.int32, device="cuda")
            w, a = torch.full((T * 8,), -7.0, device="cuda"), torch.full((T * 8, 256), -7.0, dtype=torch.bfloat16, device="cuda")
            out = torch.full((T + 1, 256), -7.0, dtype=torch.bfloat16, device="cuda")
            with pytest.raises(q.QarlError) as ei:
                q._check(q.lib().qarl_moe_layer_routed(q.C.byref(g.desc), q.C.byref(d.desc), x.data_ptr(), lg.data_ptr(), T, 8, 1, ids.data_ptr(),
                                                       w.data_ptr(), a.data_ptr(), out.data_ptr() + out_at, dt, ws.data_ptr() + ws_at, ws_bytes,
                                                       torch.cuda.current_stream().cuda_stream))
            assert ei.value.status == status
            assert all(bool((t == -7).all()) for t in (ids, w, a, out)), (T, status)
