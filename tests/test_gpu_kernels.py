"""Kernel-level parity on the GPU: MFMA lane layout, the bf16 GEMM and the
tile-local flash attention against the CPU oracle's steps."""
import math

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import epd_oracle as O
from paper_2501_05460_amd import binding as B
from gpu_util import rel_err

pytestmark = pytest.mark.gpu


def _bf16_grid(rng, shape, scale=1.0):
    return wl.to_bf16_grid((rng.standard_normal(shape) * scale).astype(np.float32))


def test_mfma_lane_layout():
    rng = np.random.default_rng(0)
    a = _bf16_grid(rng, (32, 16))
    b = _bf16_grid(rng, (16, 32))
    d = B.op_mfma_probe(B.to_device(a, True), B.to_device(b, True))
    torch.cuda.synchronize()
    want = a.astype(np.float64) @ b.astype(np.float64)
    np.testing.assert_allclose(d.cpu().numpy(), want, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("M,N,K", [(256, 128, 128), (512, 256, 256), (768, 384, 384), (256, 1152, 1152), (2560, 640, 640),
                                   (1024, 4352, 1152), (2048, 1024, 4096)])
def test_gemm_bf16_vs_oracle_linear(M, N, K):
    rng = np.random.default_rng(M + N + K)
    a = _bf16_grid(rng, (M, K))
    w = _bf16_grid(rng, (N, K), 0.05)
    bias = rng.standard_normal(N).astype(np.float32)
    c, _ = B.op_gemm_bf16(B.to_device(a, True), B.to_device(w, True), torch.from_numpy(bias).cuda())
    torch.cuda.synchronize()
    want = O.linear(a, w, bias)
    # fp32 accumulation, one bf16 rounding of the result: 2^-9 relative per element
    got = c.float().cpu().numpy()
    assert rel_err(got, want) < 6e-3
    np.testing.assert_allclose(got, want, rtol=2 ** -7, atol=2 ** -7 * np.abs(want).max() * 0.05)


def _scaled_q(q, hd):
    """The attention kernel takes its logits in the log2 domain straight from q . k: q carries the factor
    log2(e) / sqrt(hd) (the library folds it into the q projection).  Returns that q on the bf16 grid, and the
    q the oracle has to be given so that its logits q . k / sqrt(hd) are the same numbers."""
    c = math.log2(math.e) / math.sqrt(hd)
    qs = torch.from_numpy(np.asarray(q * c, np.float32)).bfloat16().float().numpy()
    return qs, qs.astype(np.float64) / c


def _attention_case(n_slices, n_tok, heads, hd, hd_pad, qk_scale, seed):
    rng = np.random.default_rng(seed)
    M = n_slices * n_tok
    D = heads * hd
    q = _bf16_grid(rng, (M, D), qk_scale)
    k = _bf16_grid(rng, (M, D), qk_scale)
    v = _bf16_grid(rng, (M, D))
    Dq = heads * hd_pad

    def pad_heads(x):
        out = np.zeros((M, Dq), np.float32)
        for h in range(heads):
            out[:, h * hd_pad:h * hd_pad + hd] = x[:, h * hd:(h + 1) * hd]
        return out

    q_dev, q = _scaled_q(q, hd)
    qk = np.concatenate([pad_heads(q_dev), pad_heads(k)], axis=1)          # [M, 2*Dq]
    vt = pad_heads(v).reshape(n_slices, n_tok, heads, hd_pad).transpose(0, 2, 3, 1).copy()
    qk_d = B.to_device(qk, True)
    o = B.op_attention_bf16(qk_d, qk_d[:, Dq:], B.to_device(vt, True), n_slices, n_tok, heads, hd_pad, 2 * Dq)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy().reshape(M, heads, hd_pad)
    assert np.all(got[:, :, hd:] == 0.0)
    got = got[:, :, :hd].reshape(M, D)
    want = np.concatenate([O.attention(q[s * n_tok:(s + 1) * n_tok], k[s * n_tok:(s + 1) * n_tok],
                                       v[s * n_tok:(s + 1) * n_tok], heads) for s in range(n_slices)])
    return got, want


@pytest.mark.parametrize("n_slices,n_tok,heads,hd,hd_pad", [
    (1, 64, 1, 64, 64), (2, 256, 3, 64, 64), (3, 1024, 2, 64, 64), (2, 1024, 2, 72, 96),
    (2, 1024, 2, 128, 128), (1, 192, 2, 32, 64), (2, 1024, 2, 72, 72), (1, 128, 3, 72, 72),
    (1, 256, 2, 80, 96)])
@pytest.mark.parametrize("qk_scale", [0.25, 1.0])
def test_attention_bf16_vs_oracle(n_slices, n_tok, heads, hd, hd_pad, qk_scale):
    # N(0,1) q/k give logits with std ~ 1..3 after scaling by 1/sqrt(hd) * hd^0.5:
    # sharp softmax rows, so a wrong key set or a cross-slice leak is visible
    got, want = _attention_case(n_slices, n_tok, heads, hd, hd_pad, qk_scale, seed=n_tok + hd)
    assert rel_err(got, want) < 1.5e-2


@pytest.mark.parametrize("n_tok,n_keys,heads,hd,hd_pad", [
    (128, 65, 2, 64, 64), (320, 257, 1, 64, 64), (1088, 1025, 2, 64, 64), (64, 1, 1, 64, 64),
    (128, 96, 2, 72, 72), (256, 197, 2, 128, 128), (192, 129, 1, 80, 96)])
def test_attention_bf16_ignores_rows_past_n_keys(n_tok, n_keys, heads, hd, hd_pad):
    """A slice owns n_tok rows but only n_keys of them are tokens (class token + patches, padded to the
    key block): the real queries see exactly the real keys, whatever the padding rows hold (here: large
    values that would take all the softmax weight if they leaked in)."""
    rng = np.random.default_rng(n_tok + n_keys + hd)
    n_slices = 2
    M = n_slices * n_tok
    D, Dq = heads * hd, heads * hd_pad
    q = _bf16_grid(rng, (M, D), 0.5)
    k = _bf16_grid(rng, (M, D), 0.5)
    v = _bf16_grid(rng, (M, D))
    real = (np.arange(M) % n_tok) < n_keys
    k[~real] *= 16.0
    v[~real] = 100.0

    def pad_heads(x):
        out = np.zeros((M, Dq), np.float32)
        for h in range(heads):
            out[:, h * hd_pad:h * hd_pad + hd] = x[:, h * hd:(h + 1) * hd]
        return out

    q_dev, q = _scaled_q(q, hd)
    qk = np.concatenate([pad_heads(q_dev), pad_heads(k)], axis=1)
    vt = pad_heads(v).reshape(n_slices, n_tok, heads, hd_pad).transpose(0, 2, 3, 1).copy()
    qk_d = B.to_device(qk, True)
    o = B.op_attention_bf16(qk_d, qk_d[:, Dq:], B.to_device(vt, True), n_slices, n_tok, heads, hd_pad,
                            2 * Dq, n_keys=n_keys)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy().reshape(M, heads, hd_pad)[:, :, :hd].reshape(M, D)
    assert np.isfinite(got).all()
    for s in range(n_slices):
        r = slice(s * n_tok, s * n_tok + n_keys)
        want = O.attention(q[r], k[r], v[r], heads)
        assert rel_err(got[r], want) < 1.5e-2, s


@pytest.mark.parametrize("paired", [False, True])
@pytest.mark.parametrize("hd", [64, 72, 96, 128])
@pytest.mark.parametrize("n_tok,n_keys", [(1024, 1024), (1088, 1025), (1024, 1000), (128, 33), (64, 32), (192, 129)])
def test_attention_bf16_of_few_and_many_slices_agrees_bit_for_bit(n_tok, n_keys, hd, paired):
    """In either order of summation: one slice runs 16 queries per wave, the fewest slices that take 32 those: the same bits either way,
    with reference moves (logits of up to about 30) in both.  Padding rows hold large values and NaN."""
    g = torch.Generator().manual_seed(n_tok * 131 + n_keys + hd)
    heads = 8
    many = next(n for n in range(2, 300) if B.op_attention_queries(n, n_tok, heads, hd, paired) == 32)
    assert B.op_attention_queries(1, n_tok, heads, hd, paired) == 16
    D = heads * hd
    qk = torch.randn(many, n_tok, 2 * D, generator=g)
    qk[:, :, :D] *= 6.0 * hd ** -0.5
    vt = torch.randn(many, D, n_tok, generator=g)
    qk[:, n_keys:, D:] = 1e4
    vt[:, :, n_keys:] = float("nan")
    # a last block reaches past the slice: rows and elements behind it belong to the buffers
    qk_d = torch.zeros(many * n_tok + 64, 2 * D, dtype=torch.bfloat16, device="cuda")
    qk_d[:many * n_tok] = qk.reshape(-1, 2 * D).to("cuda", torch.bfloat16)
    vt_d = torch.zeros(many * D * n_tok + 64, dtype=torch.bfloat16, device="cuda")
    vt_d[:many * D * n_tok] = vt.reshape(-1).to("cuda", torch.bfloat16)
    whole = B.op_attention_bf16(qk_d, qk_d[:, D:], vt_d, many, n_tok, heads, hd, 2 * D, n_keys=n_keys, paired=paired)
    whole = whole.view(many, n_tok, D)[:, :n_keys]
    assert torch.isfinite(whole.float()).all()
    for t in (0, many - 1):
        one = B.op_attention_bf16(qk_d[t * n_tok:], qk_d[t * n_tok:, D:], vt_d[t * D * n_tok:], 1, n_tok, heads, hd, 2 * D,
                                  n_keys=n_keys, paired=paired)
        assert torch.equal(one[:n_keys], whole[t])
    # and the values are the softmax's: bf16 weights and outputs, 2^-9 each on a handful of effective keys
    q, k = qk_d[:n_keys, :hd].double().cpu(), qk_d[:n_keys, D:D + hd].double().cpu()
    v = vt_d[:hd * n_tok].view(hd, n_tok)[:, :n_keys].double().cpu()
    want = torch.softmax(q @ k.T * np.log(2.0), -1) @ v.T
    got = whole[0, :, :hd].double().cpu()
    assert float((got - want).norm() / want.norm()) < 6e-3


def _attention_run(q, k, v, n_slices, n_tok, heads, hd):
    """q, k, v [M, heads * hd] on the bf16 grid -> kernel output and oracle output, both [M, heads * hd]."""
    M, D = q.shape
    q_dev, q = _scaled_q(q, hd)
    qk = np.concatenate([q_dev, k], axis=1).astype(np.float32)
    vt = v.reshape(n_slices, n_tok, heads, hd).transpose(0, 2, 3, 1).copy().astype(np.float32)
    qk_d = B.to_device(qk, True)
    o = B.op_attention_bf16(qk_d, qk_d[:, D:], B.to_device(vt, True), n_slices, n_tok, heads, hd, 2 * D)
    torch.cuda.synchronize()
    got = o.float().cpu().numpy().reshape(M, D)
    want = np.concatenate([O.attention(q[s * n_tok:(s + 1) * n_tok], k[s * n_tok:(s + 1) * n_tok],
                                       v[s * n_tok:(s + 1) * n_tok], heads) for s in range(n_slices)])
    return got, want


def _snap_bf16(x):
    return torch.from_numpy(np.asarray(x, np.float32)).bfloat16().float().numpy()


@pytest.mark.parametrize("hd", [64, 72, 128])
@pytest.mark.parametrize("kind", ["all_low", "rising", "falling", "wide"])
def test_attention_bf16_extreme_logits(kind, hd):
    """Logits far from zero and running maxima that move by large steps: the kernel shifts the logits
    by a reference value that follows the running maximum lazily, and every move rescales what has
    been accumulated.  all_low: every logit is -128 (closed form: the mean of V); rising: the
    maximum grows by ~11 (log2 units) per 32 keys, so the reference moves at every step; falling:
    the first key dominates and the later weights underflow; wide: random logits with std ~ 9."""
    n_slices, n_tok, heads = 2, 1024, 2
    M, D = n_slices * n_tok, heads * hd
    rng = np.random.default_rng(7 + hd)
    v = _bf16_grid(rng, (M, D))
    pos = (np.arange(M) % n_tok).astype(np.float32)[:, None]
    if kind == "all_low":
        q = np.full((M, D), 4.0, np.float32) * math.sqrt(64.0 / hd)
        k = -q
    elif kind in ("rising", "falling"):
        q = np.ones((M, D), np.float32)
        ramp = pos / n_tok if kind == "rising" else 1.0 - pos / n_tok
        k = np.broadcast_to(ramp * 32.0 * math.sqrt(64.0 / hd), (M, D)).copy()
    else:
        q = _bf16_grid(rng, (M, D), 3.0)
        k = _bf16_grid(rng, (M, D), 3.0)
    q, k = _snap_bf16(q), _snap_bf16(k)
    got, want = _attention_run(q, k, v, n_slices, n_tok, heads, hd)
    assert np.isfinite(got).all()
    assert rel_err(got, want) < 1.5e-2
    if kind == "all_low":
        mean_v = np.concatenate([np.broadcast_to(v[s * n_tok:(s + 1) * n_tok].mean(axis=0), (n_tok, D))
                                 for s in range(n_slices)])
        assert np.abs(got - mean_v).max() < 1e-2 * np.abs(v).max()


@pytest.mark.parametrize("epi,abs_err", [(1, 2.7e-4), (2, 2e-6)])
def test_gemm_gelu_epilogues_vs_oracle(epi, abs_err):
    """The activation inside the product's epilogue, element by element: pre-activations spread over
    +-5; the erf form is a fitted logistic with |error| <= 2.7e-4 against x Phi(x), the tanh form is
    exact up to fp32 rounding; on top of either comes one bf16 rounding of the output (at most 2^-8 relative)."""
    rng = np.random.default_rng(90 + epi)
    M, N, K = 640, 256, 256
    a = _bf16_grid(rng, (M, K), 1.0)
    w = _bf16_grid(rng, (N, K), 0.1)
    bias = (rng.standard_normal(N) * 0.5).astype(np.float32)
    out = B.op_gemm_bf16_form(B.to_device(a, True), B.to_device(w, True), torch.from_numpy(bias).cuda(), epi, 0)
    torch.cuda.synchronize()
    got = out.float().cpu().numpy().astype(np.float64)
    pre = O.linear(a, w, bias)
    assert np.abs(pre).max() > 4.0 and (np.abs(pre) < 0.5).mean() > 0.1    # both tails and the middle are sampled
    want = O.gelu_erf(pre) if epi == 1 else O.gelu_tanh(pre)
    # fp32 accumulation of K = 256 products adds ~1e-6 to the pre-activation: far below either term
    bound = abs_err + 1e-5 + 2.0 ** -8 * np.abs(want)   # half a bf16 step is 2^-8 relative at the bottom of a binade
    excess = np.abs(got - want) - bound
    assert excess.max() <= 0.0, (float(excess.max()), float(pre.flat[excess.argmax()]))


@pytest.mark.parametrize("M,N,K", [(256, 256, 128), (1000, 512, 256), (2304, 1024, 1024), (77, 256, 384)])
@pytest.mark.parametrize("epi", [0, 1, 2, 3])
def test_gemm_forms_agree_bit_for_bit(M, N, K, epi):
    """The plain loop, the pipelined loop (weights straight into LDS, fragments one k-step ahead) and
    the persistent kernel order every sum the same way: identical bits, ragged M included; the
    256x128, 128x128 and 64x64 tiles too."""
    rng = np.random.default_rng(M + N + K + epi)
    A = B.to_device(_bf16_grid(rng, (M, K), 0.5), True)
    W = B.to_device(_bf16_grid(rng, (N, K), 0.05), True)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32) * 0.1).cuda()
    r0 = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda()

    def run(form):
        R = r0.clone() if epi == 3 else None
        out = B.op_gemm_bf16_form(A, W, bias, epi, form, R)
        torch.cuda.synchronize()
        return out.view(torch.int16 if epi != 3 else torch.int32).cpu().numpy()

    ref = run(6)
    forms = [0, 1, 7, 8, 11, 13, 14] + ([9] if epi != 3 else [10])
    for form in forms:
        assert np.array_equal(run(form), ref), form
    if epi == 0:   # and the value itself, against the oracle
        want = O.linear(A.float().cpu().numpy(), W.float().cpu().numpy(), bias.cpu().numpy())
        got = B.op_gemm_bf16_form(A, W, bias, 0, 0).float().cpu().numpy()
        assert rel_err(got, want) < 6e-3


@pytest.mark.parametrize("M,N,K", [(1, 128, 128), (77, 384, 128), (130, 128, 256), (1000, 1152, 384), (3096, 256, 640), (4100, 1152, 128)])
@pytest.mark.parametrize("epi", [0, 2, 3])
def test_ring_tiles_agree_bit_for_bit(M, N, K, epi):
    """The ring kernel's three tiles (64x64, 128x64, 128x128) leave the bits of the 256x128 form: contractions shorter
    than the ring (two slabs), of one and of several turns of it, ragged rows, widths of odd multiples of 128."""
    rng = np.random.default_rng(M + N + K + epi)
    A = B.to_device(_bf16_grid(rng, (M, K), 0.5), True)
    W = B.to_device(_bf16_grid(rng, (N, K), 0.05), True)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32) * 0.1).cuda()
    r0 = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda()

    def run(form):
        out = B.op_gemm_bf16_form(A, W, bias, epi, form, r0.clone() if epi == 3 else None)
        torch.cuda.synchronize()
        return out.view(torch.int16 if epi != 3 else torch.int32).cpu().numpy()

    ref = run(1)
    for form in (11, 13, 14, 0):
        assert np.array_equal(run(form), ref), form


@pytest.mark.parametrize("epi,M,N,K,form", [
    (3, 961, 1152, 128, 11), (3, 1344, 1152, 384, 11), (3, 1345, 1152, 128, 11),      # 64 x 96: 16 rows of tiles, whole rounds, one too many for a round
    (3, 1793, 1152, 128, 13), (3, 2560, 1152, 640, 13), (3, 2688, 1152, 1664, 13),    # 128 x 96: ragged, full as far as a short K goes, a long one
    (2, 897, 4352, 128, 14), (1, 1025, 4096, 256, 14), (1, 1408, 4352, 384, 14),      # 128 x 192: the last column of tiles begins inside the one before
])
def test_ring_tiles_half_as_wide_again_agree_bit_for_bit(epi, M, N, K, form):
    """Tiles of 96 and 192 columns, in one round where 64 and 128 wide ones are in two: the bits of the 256 x 128 form, and
    rows past M are not written."""
    g = torch.Generator().manual_seed(M + N + K)
    A, W = torch.randn(M, K, generator=g).mul_(0.5).bfloat16().cuda(), torch.randn(N, K, generator=g).mul_(0.05).bfloat16().cuda()
    bias = torch.randn(N, generator=g).mul_(0.1).cuda()
    r0 = torch.randn(M, N, generator=g).cuda() if epi == 3 else None
    got, want = (B.op_gemm_bf16_form(A, W, bias, epi, f, None if r0 is None else r0.clone()) for f in (form, 1))
    assert torch.equal(got, want)


@pytest.mark.parametrize("epi,M,N,K,form", [
    (3, 9200, 1152, 256, 12),     # 256 x 192 tiles
    (3, 2600, 1152, 1152, 14),    # ring tiles over nine columns of 128, the tenth all padding
    (3, 3570, 1152, 256, 13),     # 128 x 64: eighteen of twenty
    (3, 14600, 1152, 1152, 5),    # whole rounds, the rows behind on ring tiles
    (3, 9400, 3584, 640, 5),
    (0, 15000, 2304, 640, 5),
    (2, 4800, 3584, 1152, 5),
    (3, 5000, 3200, 128, 18),     # whole 256-wide tile columns, the last 128 columns apart
    (3, 6700, 3200, 1152, 15),    # 224 x 256 tiles
    (1, 2400, 3584, 128, 15),
    (0, 3000, 2304, 1152, 1),     # one round of 256 x 128 tiles
    (3, 2300, 3200, 4096, 1),
    (2, 1500, 4608, 2048, 1),
    (0, 14600, 2304, 128, 1),     # several
    (3, 11500, 1152, 640, 10),    # 256 x 256 tiles
    (1, 11500, 1152, 640, 9),
    (0, 28, 1152, 128, 11),
])
def test_what_the_library_picks_leaves_the_bits_of_one_form(epi, M, N, K, form):
    """The dispatch over weights padded as the library pads them (1152 columns to 1280, 3200 to 3328): every form that runs is
    reached, and leaves the bits of 256 x 128 tiles and of 128 x 128 ring tiles, two different kernels, over unpadded weights."""
    assert B.op_gemm_bf16_shape(M, N, K, epi) == form
    rng = np.random.default_rng(M + N + K + epi)
    A = B.to_device(_bf16_grid(rng, (M, K), 0.5), True)
    W = B.to_device(_bf16_grid(rng, (N, K), 0.05), True)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32) * 0.1).cuda()
    r0 = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda() if epi == 3 else None
    got, *wanted = (B.op_gemm_bf16_form(A, W, bias, epi, f, None if r0 is None else r0.clone()) for f in (0, 1, 14))
    torch.cuda.synchronize()
    as_int = torch.int32 if epi == 3 else torch.int16
    for want in wanted:
        assert torch.equal(got.view(as_int), want.view(as_int))


@pytest.mark.parametrize("K", [128, 256, 640])
@pytest.mark.parametrize("epi,M,N,forms", [
    (0, 16536, 1024, (9, 1)), (1, 16536, 1024, (9, 1)), (2, 16536, 1024, (9, 1)),   # 260 tiles of 256 x 256, 520 of 256 x 128
    (3, 16537, 1024, (10, 1)), (4, 16536, 1024, (9, 1)), (5, 16536, 1024, (9, 1)),
    (3, 11100, 2304, (12, 10, 1)),                                                  # 528 of 256 x 192, 396 of 256 x 256
    (4, 1240, 1152, (1, 13)), (5, 1240, 1152, (1, 13)), (4, 8200, 1152, (0, 1)), (5, 8200, 1152, (0, 1))])
def test_persistent_tiles_beyond_the_first_agree_bit_for_bit(epi, M, N, forms, K):
    """More tiles than CUs, so that workgroups go on to a second tile, whose first slabs and stream rows are fetched under the last
    products of the one before; two slabs (K = 128: all of a tile's are its last) and more, a ragged last tile row, every
    epilogue.  Reference: one workgroup per tile on the 32-wide instruction (form 6), ring tiles where a width is no multiple
    of 256; the patch embedding and the value projection against fp64 too."""
    n_tok = {16536: 312, 1240: 248, 8200: 200}.get(M, 0)
    g = torch.Generator().manual_seed(M + N + K + epi)
    A, W = torch.randn(M, K, generator=g).mul_(0.5).bfloat16().cuda(), torch.randn(N, K, generator=g).mul_(0.05).bfloat16().cuda()
    bias = torch.randn(N, generator=g).mul_(0.1).cuda()
    r0 = torch.randn(M, N, generator=g).cuda() if epi == 3 else None
    pos = torch.randn(n_tok, N, generator=g).cuda() if epi == 4 else None
    run = lambda form: B.op_gemm_bf16_form(A, W, bias, epi, form, None if r0 is None else r0.clone(), pos=pos, n_tok=n_tok)
    ref = run(6 if N % 256 == 0 else 14)
    for form in forms:
        assert torch.equal(run(form), ref), form
    if epi in (4, 5):
        want = A.double().cpu() @ W.double().cpu().T + bias.double().cpu()
        if epi == 4:
            want, got = want + pos.double().cpu().repeat(M // n_tok, 1), ref
        else:
            got = ref.permute(0, 2, 1).reshape(M, N)
        # fp32 sums of K products; the transposed values leave in bf16 (2^-9)
        assert float((got.double().cpu() - want).norm() / want.norm()) < (1e-5 if epi == 4 else 4e-3)


@pytest.mark.parametrize("epi,M,N,K", [(1, 1, 256, 128), (2, 224, 512, 256), (3, 225, 256, 128), (3, 1000, 512, 384), (1, 7300, 2048, 128),
                                       (3, 14600, 1024, 128), (3, 14592, 1024, 640)])
def test_224_row_tiles_agree_bit_for_bit(epi, M, N, K):
    """Tiles of a height that does not divide 256: the last one computes rows of the tile above again, which a residual product must
    add once.  One tile, a last tile of one row, whole and ragged rows, more tiles than CUs."""
    g = torch.Generator().manual_seed(M + N + K + epi)
    A, W = torch.randn(M, K, generator=g).mul_(0.5).bfloat16().cuda(), torch.randn(N, K, generator=g).mul_(0.05).bfloat16().cuda()
    bias = torch.randn(N, generator=g).mul_(0.1).cuda()
    r0 = torch.randn(M, N, generator=g).cuda() if epi == 3 else None
    run = lambda form: B.op_gemm_bf16_form(A, W, bias, epi, form, None if r0 is None else r0.clone())
    assert torch.equal(run(15), run(6))


@pytest.mark.parametrize("M,N,n2,K,n_tok", [(8, 256, 256, 128, 8), (248, 256, 384, 128, 248), (1032, 2304, 1152, 256, 1032), (2400, 768, 384, 128, 600),
                                            (1736, 512, 256, 640, 248), (7344, 2304, 1152, 128, 816), (10240, 2048, 1024, 128, 1024),
                                            (7344, 2304, 1152, 640, 816), (7392, 2304, 1152, 640, 1056), (7624, 2048, 1024, 768, 7624)])
def test_two_products_in_one_launch_agree_bit_for_bit(M, N, n2, K, n_tok):
    """Every tile of the pair: ring tiles, 256, 224, 192 and 160 x 256 and 256 x 192.  One tile and more than CUs, slices that end inside a
    tile, value columns that leave a last tile half empty; the last three: workgroups that go from a q/k tile on to a value tile over more
    than two slabs, and last tile rows of 160 and 192 (7392 rows) and of 224 (7624) that lie over the one above.  Reference: the two
    products in a launch each, on the kernels with one workgroup per tile."""
    g = torch.Generator().manual_seed(M + N + K)
    A, W = torch.randn(M, K, generator=g).mul_(0.5).bfloat16().cuda(), torch.randn(N + n2, K, generator=g).mul_(0.05).bfloat16().cuda()
    bias = torch.randn(N + n2, generator=g).mul_(0.1).cuda()
    c = B.op_gemm_bf16_form(A, W[:N], bias[:N], 0, 6)
    v = B.op_gemm_bf16_form(A, W[N:].contiguous(), bias[N:].contiguous(), 5, 14, n_tok=n_tok)
    for form in (9, 11, 13, 14, 15, 16, 17) + ((12,) if N % 192 == 0 and n2 % 192 == 0 else ()):
        got_c, got_v = B.op_gemm_bf16_pair(A, W, bias, N, n_tok, form)
        assert torch.equal(got_c, c) and torch.equal(got_v, v), form


@pytest.mark.parametrize("epi,N,forms,rows,more", [(0, 4096, (9, 1), 21970, 32), (1, 4096, (9, 15, 1), 21970, 32), (2, 4352, (9, 15), 20672, 32),
                                                   (3, 1024, (10, 15, 1), 18300, 32), (3, 1152, (12,), 16270, 32), (5, 2048, (9, 1), 43936, 16)])
def test_outputs_that_stay_in_the_cache_and_larger_ones_agree_bit_for_bit(epi, N, forms, rows, more):
    """Either side of the size from which a product's output is streamed past the caches (90 million bf16 elements, 18.75 million of the
    stream): kernels of their own, the same bits in the rows they share.  The transposed store in slices of 16 rows."""
    g = torch.Generator().manual_seed(N + epi)
    M, K = rows + more, 128
    assert (rows * N <= 18.75e6 < M * N) if epi == 3 else (rows * N <= 90e6 < M * N)
    A, W = torch.randn(M, K, generator=g).mul_(0.5).bfloat16().cuda(), torch.randn(N, K, generator=g).mul_(0.05).bfloat16().cuda()
    bias = torch.randn(N, generator=g).mul_(0.1).cuda()
    r0 = torch.randn(M, N, generator=g).cuda() if epi == 3 else None
    for form in forms:
        near, far = (B.op_gemm_bf16_form(A[:m], W, bias, epi, form, None if r0 is None else r0[:m].clone(), n_tok=16 if epi == 5 else 0)
                     for m in (rows, M))
        assert torch.equal(near, far[:len(near)]), form


@pytest.mark.parametrize("M,N,K", [(256, 384, 128), (1000, 1152, 256), (2900, 1152, 1152), (77, 384, 384), (11100, 1152, 128)])
def test_gemm_192_wide_tiles_agree_bit_for_bit(M, N, K):
    """The residual product on 256 x 192 tiles (widths that are whole multiples of 192 and not of 256) leaves the
    bits of the other tile shapes: whole and ragged M, one tile and several per workgroup, and a launch with more
    tiles than CUs (the persistent walk takes a second tile)."""
    rng = np.random.default_rng(M + N + K)
    A = B.to_device(_bf16_grid(rng, (M, K), 0.5), True)
    W = B.to_device(_bf16_grid(rng, (N, K), 0.05), True)
    bias = torch.from_numpy(rng.standard_normal(N).astype(np.float32) * 0.1).cuda()
    r0 = torch.from_numpy(rng.standard_normal((M, N)).astype(np.float32)).cuda()

    def run(form):
        R = r0.clone()
        B.op_gemm_bf16_form(A, W, bias, 3, form, R)
        torch.cuda.synchronize()
        return R.view(torch.int32).cpu().numpy()

    ref = run(1)
    assert np.array_equal(run(12), ref)
    assert np.array_equal(run(2), ref)
    assert np.array_equal(run(0), ref)          # whichever form the library picks for this shape
    want = r0.cpu().numpy().astype(np.float64) + O.linear(A.float().cpu().numpy(), W.float().cpu().numpy(), bias.cpu().numpy())
    assert rel_err(ref.view(np.float32), want) < 1e-4


def test_measurement_probes_run_and_report_sane_figures():
    """The probes behind `bench.py --roof` (no part of the encode path): the register-resident MFMA loop stays below the
    nominal bf16 peak and above a fifth of it, the streaming copy below the nominal HBM rate, and a SIMD that runs a
    wave of MFMAs and a wave of exp + fma pairs together takes longer than either alone and less than both in turn
    (the partial overlap the attention kernel's floor is derived from)."""
    for shape in (32, 16):
        t = B.op_mfma_peak(True, iters=500, reps=2, shape=shape)
        assert 500.0 < t < 2600.0, (shape, t)
    g = B.op_copy_peak(1 << 28, reps=2)
    assert 1000.0 < g < 8000.0, g
    m, v, both = B.op_coissue(1, 1000, 1250, 2), B.op_coissue(2, 1000, 1250, 2), B.op_coissue(3, 1000, 1250, 2)
    assert m > 0 and v > 0 and max(m, v) * 0.98 <= both <= (m + v) * 1.02, (m, v, both)
