"""GPU parity of the decoder block around the BitLinear products (include/bitlinear_decoder.h) against
oracle/decoder.py.

Stage by stage: each kernel gets seeded inputs and is compared with the oracle's fp64 formula within a
tolerance that its fp32 arithmetic explains; what a kernel decides in integers or stores rounded (the int8
activations, the bf16 cache) is compared bit for bit with the oracle's decision taken on the kernel's own fp32
values.  End to end (a token through layers) the two sides' quantizers see inputs that differ in the last
bits, so an occasional code differs by one: that comparison is a bound, not an identity.
"""
import numpy as np
import pytest

import oracle
from oracle import decoder as D
from paper_2410_16144_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def mods():
    from paper_2410_16144_amd import binding, decoder, ops
    binding.lib()
    return binding, decoder, ops


def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _t(a, dev):
    return torch.from_numpy(np.ascontiguousarray(a)).to(dev)


# ------------------------------------------------------------------------------------------ norm + quantizer

NORM_SHAPES = [(1, 768), (1, 3200), (1, 8640), (3, 4096), (1, 45568), (2, 67), (1, 1), (1, 1000), (5, 4100), (1, 49152)]


WIDE_SHAPES = [(1, 16384), (1, 24576), (1, 45568), (2, 49152), (3, 16388), (1, 20001)]


@pytest.mark.parametrize("mode", ["plain", "residual", "residual_no_delta", "gated"])
@pytest.mark.parametrize("M,K,wide", [s + (False,) for s in NORM_SHAPES] + [s + (True,) for s in WIDE_SHAPES])
def test_norm_quant_parity(dev, mods, mode, M, K, wide):
    B, dec, ops = mods
    scratch = torch.empty(M * B.BL_NORM_SCRATCH_BYTES, dtype=torch.uint8, device=dev) if wide else None
    r = _rng(31000 + 7 * K + M)
    gamma = r.uniform(0.5, 1.5, K).astype(np.float32)
    a = synth.activations(r, M, K, outlier_frac=0.01)
    b = synth.activations(r, M, K)
    h = synth.activations(r, M, K)
    eps = 1e-5
    y_t = torch.empty((M, K), dtype=torch.float32, device=dev)
    qa = ops.alloc_quant(M, K, dev)
    qa.q.fill_(77)                                        # the layout's padding must be written as zero
    qa.q_sum.fill_(12345)
    if mode == "plain":
        dec.norm_quant(B.BL_NORM_PLAIN, _t(gamma, dev), eps, a=_t(a, dev), out=qa, y=y_t, scratch=scratch)
        x64 = a.astype(np.float64)
    elif mode.startswith("residual"):
        h_t = _t(h, dev)
        delta = None if mode == "residual_no_delta" else _t(a, dev)
        dec.norm_quant(B.BL_NORM_RESIDUAL, _t(gamma, dev), eps, a=delta, h=h_t, out=qa, y=y_t, scratch=scratch)
        want_h = h if delta is None else h + a            # one fp32 addition per element: exact agreement
        np.testing.assert_array_equal(h_t.cpu().numpy(), want_h)
        x64 = want_h.astype(np.float64)
    else:
        dec.norm_quant(B.BL_NORM_GATED, _t(gamma, dev), eps, a=_t(a, dev), b=_t(b, dev), out=qa, y=y_t, scratch=scratch)
        x64 = D.gated_ffn_input(a, b)
    torch.cuda.synchronize()
    y = y_t.cpu().numpy()
    want = D.rmsnorm(x64, gamma, eps)
    # fp32: a tree sum of K squares (relative error ~ 1e-7 log K), one division, root, two products; the gate adds
    # expf and a division.  3e-6 of the row's largest value covers it with margin.
    tol = 3e-6 * np.abs(want).max(axis=1, keepdims=True) + 1e-30
    assert np.all(np.abs(y - want) <= tol), float(np.abs(y - want).max())
    # the quantizer's decisions, taken on the kernel's own fp32 y, bit for bit
    q, a_scale, q_sum = oracle.quant_act(y)
    got_q = qa.q.cpu().numpy()
    np.testing.assert_array_equal(got_q[:, :K], q)
    assert not got_q[:, K:].any()
    np.testing.assert_array_equal(qa.a_scale.cpu().numpy().view(np.uint32), a_scale.view(np.uint32))
    np.testing.assert_array_equal(qa.q_sum.cpu().numpy(), q_sum)


@pytest.mark.parametrize("mode,M,K", [("plain", 1, 2048), ("residual", 2, 2052), ("gated", 1, 8192), ("plain", 2, 8196),
                                      ("gated", 511, 8200), ("gated", 512, 8200), ("gated", 512, 12288), ("gated", 512, 12292)])
def test_norm_quant_at_the_edges_of_the_thread_counts(dev, mods, mode, M, K):
    """256, 512 and 1024 threads per row: the longest row of each and the first beyond, and the gated form's change at 512
    rows.  Tolerance: the same derivation as above."""
    test_norm_quant_parity(dev, mods, mode, M, K, False)


def _norm_of_1024_threads(x, gamma, eps):
    """The plain norm in fp32, its sum of squares added up in the kernels' one order: element 4 (t + 1024 i) + j belongs to
    thread t of 1024, which adds its own up in turn; the 64 of a wave by the tree of wave_sum_f; the waves one after another."""
    M, K = x.shape
    padded = np.zeros((M, -(-K // 4096) * 4096), np.float32)
    padded[:, :K] = x
    sq = (padded * padded).reshape(M, -1, 1024, 4)
    ss = np.zeros((M, 1024), np.float32)
    for i in range(sq.shape[1]):
        for j in range(4):
            ss = ss + sq[:, i, :, j]
    lanes = np.arange(64)
    w = ss.reshape(M, 16, 64)
    for partner in (lanes ^ 1, lanes ^ 2, lanes ^ 7, lanes ^ 15):
        w = w + w[:, :, partner]
    w = (w[:, :, 0] + w[:, :, 16]) + (w[:, :, 32] + w[:, :, 48])
    total = np.zeros(M, np.float32)
    for i in range(16):
        total = total + w[:, i]
    r = np.float32(1.0) / np.sqrt(total / np.float32(K) + np.float32(eps))
    return (x * gamma) * r[:, None]


@pytest.mark.parametrize("K", [5, 768, 1030, 2048, 2052, 4096, 6000, 8192, 8200, 12032, 20000])
def test_norm_quant_adds_up_in_one_order(dev, mods, K):
    """Rows that 256, 512 and 1024 threads take, all the bits of the norm as 1024 threads add them up."""
    B, dec, ops = mods
    r = _rng(7100 + K)
    x, gamma = r.standard_normal((37, K)).astype(np.float32), r.uniform(0.5, 1.5, K).astype(np.float32)
    y = torch.empty(x.shape, device=dev)
    dec.norm_quant(B.BL_NORM_PLAIN, _t(gamma, dev), 1e-5, a=_t(x, dev), y=y)
    np.testing.assert_array_equal(y.cpu().numpy(), _norm_of_1024_threads(x, gamma, 1e-5))


@pytest.mark.parametrize("K", [8200, 12032, 12288])
def test_norm_quant_rows_do_not_depend_on_their_batch(dev, mods, K):
    """The gated form changes its thread count with the number of rows: the same row, the same bits."""
    B, dec, ops = mods
    M = 2048
    a, b = (torch.randn((M, K), device=dev, generator=torch.Generator(dev).manual_seed(K + i)) for i in range(2))
    gamma = torch.rand(K, device=dev) + 0.5
    y = torch.empty_like(a)
    whole = dec.norm_quant(B.BL_NORM_GATED, gamma, 1e-5, a=a, b=b, y=y)
    for M1 in (1, 100, 511):
        y1 = torch.empty((M1, K), device=dev)
        part = dec.norm_quant(B.BL_NORM_GATED, gamma, 1e-5, a=a[:M1], b=b[:M1], y=y1)
        assert torch.equal(y1, y[:M1]) and torch.equal(part.q, whole.q[:M1])
        assert torch.equal(part.a_scale, whole.a_scale[:M1]) and torch.equal(part.q_sum, whole.q_sum[:M1])


@pytest.mark.parametrize("M,K", [(1, 4096), (1, 100), (3, 2050), (37, 2048), (2, 8196), (5, 12288), (1, 49152)])
@pytest.mark.parametrize("pos_set", [None, 0, 77])
def test_final_norm_is_the_residual_norm_with_the_position(dev, mods, M, K, pos_set):
    """bl_final_norm: the bits of bl_norm_quant's residual form, the sum where it is wanted and nowhere else, the position's step."""
    B, dec, ops = mods
    g = torch.Generator(dev).manual_seed(K + M)
    h, delta = (torch.randn((M, K), device=dev, generator=g) for _ in range(2))
    gamma = torch.rand(K, device=dev, generator=g) + 0.5
    for d in (delta, None):
        ref_h, ref_y = h.clone(), torch.empty_like(h)
        dec.norm_quant(B.BL_NORM_RESIDUAL, gamma, 1e-5, a=d, h=ref_h, y=ref_y, quantize=False)
        for where in ("nowhere", "other", "itself"):
            src, other = h.clone(), torch.full_like(h, 3.0)
            out = {"nowhere": None, "other": other, "itself": src}[where]
            y = torch.empty_like(h)
            pos = torch.full((1,), 41, dtype=torch.int32, device=dev)
            assert dec.final_norm(src, d, gamma, 1e-5, y, pos, pos_set=pos_set, h_out=out) is y
            assert torch.equal(y, ref_y) and pos.item() == (42 if pos_set is None else pos_set)
            assert torch.equal(src, ref_h if where == "itself" else h)
            assert torch.equal(other, ref_h if where == "other" and d is not None else torch.full_like(h, 3.0))


@pytest.mark.parametrize("K", [512, 45056])
def test_norm_quant_gate_of_any_size(dev, mods, K):
    """The gate's two ways of computing silu meet at a size of 80: waves below it, waves with one element at or above it, and
    waves far beyond, where exp overflows.  The row's largest value sets the scale of the comparison (3e-6, as above), so
    each size gets a row of its own."""
    B, dec, ops = mods
    r = _rng(77)
    sizes = [1e-30, 1e-3, 1.0, 20.0, 79.99, 80.0, 87.5, 100.0, 1e4]
    a = r.uniform(-1.0, 1.0, (len(sizes), K)).astype(np.float32)
    for i, v in enumerate(sizes):
        a[i] *= np.float32(v)
        a[i, 0], a[i, K - 1] = v, -v
    b = r.uniform(0.5, 1.0, a.shape).astype(np.float32)
    gamma = r.uniform(0.5, 1.5, K).astype(np.float32)
    y = torch.empty(a.shape, device=dev)
    scratch = torch.empty(len(sizes) * B.BL_NORM_SCRATCH_BYTES, dtype=torch.uint8, device=dev)
    for use_scratch in (False, True):
        dec.norm_quant(B.BL_NORM_GATED, _t(gamma, dev), 1e-5, a=_t(a, dev), b=_t(b, dev), y=y, scratch=scratch if use_scratch else None)
        with np.errstate(over="ignore"):
            want = D.rmsnorm(D.gated_ffn_input(a, b), gamma, 1e-5)
        tol = 3e-6 * np.abs(want).max(axis=1, keepdims=True) + 1e-30
        assert np.all(np.abs(y.cpu().numpy() - want) <= tol)


def test_norm_quant_zero_row_and_no_quantizer(dev, mods):
    B, dec, ops = mods
    K = 512
    gamma = torch.ones(K, device=dev)
    qa = dec.norm_quant(B.BL_NORM_PLAIN, gamma, 1e-5, a=torch.zeros((1, K), device=dev))
    torch.cuda.synchronize()
    assert not qa.q.any() and float(qa.a_scale[0]) == 0.0 and int(qa.q_sum[0]) == 0
    # the final norm of a model: residual add and y only
    r = _rng(5)
    h, d = synth.activations(r, 1, K), synth.activations(r, 1, K)
    h_t, y_t = _t(h, dev), torch.empty((1, K), device=dev)
    assert dec.norm_quant(B.BL_NORM_RESIDUAL, gamma, 1e-5, a=_t(d, dev), h=h_t, y=y_t, quantize=False) is None
    torch.cuda.synchronize()
    np.testing.assert_array_equal(h_t.cpu().numpy(), h + d)
    np.testing.assert_allclose(y_t.cpu().numpy(), D.rmsnorm((h + d).astype(np.float64), np.ones(K), 1e-5), rtol=3e-6, atol=1e-6)


def test_norm_quant_feeds_the_product(dev, mods):
    """q, a_scale, q_sum as written by bl_norm_quant go straight into bl_gemv: the product equals the oracle's
    on the same y."""
    B, dec, ops = mods
    N, K = 200, 3200
    r = _rng(41)
    w = synth.ternary_weights(r, N, K)
    pw = ops.pack_ternary(_t(w, dev), 0.03)
    y_t = torch.empty((1, K), device=dev)
    qa = dec.norm_quant(B.BL_NORM_PLAIN, _t(r.uniform(0.5, 1.5, K).astype(np.float32), dev), 1e-5,
                        a=_t(synth.activations(r, 1, K), dev), y=y_t)
    out, acc = ops.gemv(pw, qa, want_acc=True)
    torch.cuda.synchronize()
    q, a_scale, _ = oracle.quant_act(y_t.cpu().numpy())
    ref_acc = oracle.matmul_i32(q, w)
    np.testing.assert_array_equal(acc.cpu().numpy(), ref_acc)
    np.testing.assert_allclose(out.cpu().numpy(), oracle.dequant(ref_acc, np.float32(0.03), a_scale), rtol=1e-6)


# ------------------------------------------------------------------------------------------ rotary table

@pytest.mark.parametrize("head_dim,max_pos,theta", [(64, 300, 10000.0), (120, 2048, 10000.0), (2, 5, 3.0), (256, 17, 500000.0)])
def test_rope_table(dev, mods, head_dim, max_pos, theta):
    B, dec, ops = mods
    t = dec.rope_table(head_dim, max_pos, dev, theta).cpu().numpy()
    ang = D.rope_angles(head_dim, max_pos, theta)
    # fp64 arithmetic rounded to fp32: half an ulp of values <= 1, plus the fp64 angle's rounding (~ pos * 1e-16)
    assert np.abs(t[..., 0] - np.cos(ang)).max() <= 6.1e-8
    assert np.abs(t[..., 1] - np.sin(ang)).max() <= 6.1e-8
    assert np.all(t[0, :, 0] == 1.0) and np.all(t[0, :, 1] == 0.0)


# ------------------------------------------------------------------------------------------ attention

def _bf16(x):
    return synth.bf16_bits_to_f32(synth.to_bf16_bits(np.asarray(x, np.float32)))


def _bits_as_bf16_tensor(bits, dev):
    return torch.from_numpy(bits.view(np.int16)).to(dev).view(torch.bfloat16)


@pytest.mark.parametrize("n_heads,head_dim,max_pos,positions", [
    (3, 64, 600, [0, 1, 2, 255, 256, 257, 511, 512, 599]),
    (20, 128, 300, [0, 77, 299]),
    (32, 120, 1024, [5, 700, 1023]),
    (32, 48, 512, [0, 300]),
    (2, 8, 256, [0, 255]),
    (32, 100, 300, [0, 100, 299]),
    (3, 4, 40, [7]),
    (1, 256, 260, [3, 259]),
])
def test_attn_decode_parity(dev, mods, n_heads, head_dim, max_pos, positions):
    B, dec, ops = mods
    hidden = n_heads * head_dim
    r = _rng(52000 + hidden + max_pos)
    table = dec.rope_table(head_dim, max_pos, dev)
    q_t, k_t, v_t = (torch.empty((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, table)
    # a cache already filled up to max_pos with seeded bf16 values; each call overwrites its own row
    kc = _bf16(r.standard_normal((max_pos, hidden)))
    vc = _bf16(r.standard_normal((max_pos, hidden)))
    att.k_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(kc), dev))
    att.v_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(vc), dev))
    kc64, vc64 = kc.astype(np.float64), vc.astype(np.float64)
    for pos in positions:
        ql, kl, vl = (3.0 * r.standard_normal(hidden).astype(np.float32) for _ in range(3))
        q_t.copy_(_t(ql[None], dev)); k_t.copy_(_t(kl[None], dev)); v_t.copy_(_t(vl[None], dev))
        pos_t.fill_(pos)
        out = att.launch()
        torch.cuda.synchronize()
        # the appended row: values are a plain rounding (bit-exact); keys go through an fp32 rotation first, so
        # a rounding decision may fall the other way now and then -- by one bf16 step at most
        got_k = att.k_cache[pos].view(torch.int16).cpu().numpy().view(np.uint16)
        got_v = att.v_cache[pos].view(torch.int16).cpu().numpy().view(np.uint16)
        np.testing.assert_array_equal(got_v, synth.to_bf16_bits(vl))
        want_k = D.round_to_bf16(D.rope(kl, pos, n_heads))
        k_f = synth.bf16_bits_to_f32(got_k).astype(np.float64)
        step = np.maximum(np.abs(want_k), 1e-30) * 2.0 ** -7
        assert np.all(np.abs(k_f - want_k) <= step)
        assert np.mean(k_f == want_k) >= 0.99
        # attention over rows 0 .. pos with the row the kernel stored
        kc64[pos], vc64[pos] = k_f, synth.bf16_bits_to_f32(got_v).astype(np.float64)
        want = D.attention_decode(D.rope(ql, pos, n_heads), kc64[:pos + 1], vc64[:pos + 1], n_heads)
        got = out.cpu().numpy()[0]
        assert np.abs(got - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), float(np.abs(got - want).max())
    # rows that no call addressed are untouched
    untouched = [j for j in range(max_pos) if j not in positions]
    got_all = att.k_cache.view(torch.int16).cpu().numpy().view(np.uint16)
    np.testing.assert_array_equal(got_all[untouched], synth.to_bf16_bits(kc)[untouched])


@pytest.mark.parametrize("groups", [1, 2, 3, 5])
@pytest.mark.parametrize("n_heads,head_dim", [(3, 64), (2, 100), (1, 256), (2, 132), (5, 4), (3, 128), (2, 256)])
def test_attn_decode_several_chunks_per_workgroup(dev, mods, groups, n_heads, head_dim):
    """A cache longer than the launch has workgroups for: each of a head's `groups` workgroups walks every groups-th
    chunk and folds them into one running maximum, sum and weighted values before the merge.  Positions that put the
    appended row into the first, a middle and the last chunk a workgroup walks, a ragged last chunk, one chunk only;
    every output against the fp64 softmax over the cache as stored, the counters back at zero."""
    B, dec, ops = mods
    max_pos, hidden = 700, n_heads * head_dim
    r = _rng(53000 + hidden + groups)
    table = dec.rope_table(head_dim, max_pos, dev)
    q_t, k_t, v_t = (torch.empty((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, table)
    kc = _bf16(r.standard_normal((max_pos, hidden)))
    vc = _bf16(r.standard_normal((max_pos, hidden)))
    att.k_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(kc), dev))
    att.v_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(vc), dev))
    kc64, vc64 = kc.astype(np.float64), vc.astype(np.float64)
    B.bl_set_tuning("attn_groups", groups)
    try:
        for pos in (0, 63, 64, 130, 320, 447, 448, 640, 699):
            ql, kl, vl = (3.0 * r.standard_normal(hidden).astype(np.float32) for _ in range(3))
            q_t.copy_(_t(ql[None], dev)); k_t.copy_(_t(kl[None], dev)); v_t.copy_(_t(vl[None], dev))
            pos_t.fill_(pos)
            out = att.launch()
            torch.cuda.synchronize()
            kc64[pos] = att.k_cache[pos].float().cpu().numpy().astype(np.float64)
            vc64[pos] = att.v_cache[pos].float().cpu().numpy().astype(np.float64)
            np.testing.assert_array_equal(att.v_cache[pos].view(torch.int16).cpu().numpy().view(np.uint16), synth.to_bf16_bits(vl))
            want = D.attention_decode(D.rope(ql, pos, n_heads), kc64[:pos + 1], vc64[:pos + 1], n_heads)
            got = out.cpu().numpy()[0]
            assert np.abs(got - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), (pos, float(np.abs(got - want).max()))
            assert not att.scratch[-4 * n_heads:].view(torch.int32).any()
    finally:
        B.bl_set_tuning("attn_groups", 0)


@pytest.mark.parametrize("n_heads,head_dim,groups", [(32, 128, 8), (26, 80, 9), (60, 100, 4), (28, 160, 9), (200, 88, 1), (40, 72, 12), (27, 156, 18),
                                                     (90, 128, 5), (32, 48, 16), (16, 96, 16), (8, 36, 32)])
def test_attn_decode_one_round_or_two(dev, mods, n_heads, head_dim, groups):
    """The workgroups that a call takes by itself: one round of the units (cache rows with few idle lanes, 72 % of the units filled)
    or more, each walking one chunk, several of them, and the last one in part; some heads against the fp64 softmax on the cache as
    it lies there."""
    B, dec, ops = mods
    hidden, max_pos = n_heads * head_dim, 64 * 20 - 7
    r = _rng(53900 + hidden)
    table = dec.rope_table(head_dim, max_pos, dev)
    q_t, k_t, v_t = (torch.empty((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, table)
    for c in (att.k_cache, att.v_cache):
        c.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(r.standard_normal((max_pos, hidden)).astype(np.float32)), dev))
    heads = sorted({0, n_heads // 2, n_heads - 1})
    cols = np.concatenate([np.arange(h * head_dim, (h + 1) * head_dim) for h in heads])
    for pos in sorted({0, 63, 64, 64 * groups - 1, 64 * groups, 64 * groups + 63, 64 * 19 + 5, max_pos - 1}):
        if pos >= max_pos:
            continue
        ql, kl, vl = (3.0 * r.standard_normal(hidden).astype(np.float32) for _ in range(3))
        q_t.copy_(_t(ql[None], dev)); k_t.copy_(_t(kl[None], dev)); v_t.copy_(_t(vl[None], dev))
        pos_t.fill_(pos)
        got = att.launch().cpu().numpy()[0]
        kc, vc = (c[:pos + 1].float().cpu().numpy().astype(np.float64)[:, cols] for c in (att.k_cache, att.v_cache))
        want = D.attention_decode(D.rope(ql[cols], pos, len(heads)), kc, vc, len(heads))
        assert np.abs(got[cols] - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), (pos, float(np.abs(got[cols] - want).max()))


def test_attn_decode_long_walk_is_as_exact_as_a_short_one(dev, mods):
    """52 heads have four workgroups each: at 10 000 positions every one adds up 39 chunks.  Sums of n terms one behind the other are off
    by about sqrt(n / 3) roundings, and with the scores' own error the walk's output was 1.31 times as far from 64 bits as at 1000
    positions (4 chunks per workgroup); in blocks of four chunks the longest run of roundings is 4 + 10, measured 1.20."""
    B, dec, ops = mods
    n_heads, d, max_pos = 52, 128, 10001
    hidden = n_heads * d
    table = dec.rope_table(d, max_pos, dev)
    g = torch.Generator(dev).manual_seed(5)
    lin = [torch.randn((1, hidden), device=dev, generator=g) for _ in range(3)]
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, d, max_pos, *lin, pos_t, table)
    for c in (att.k_cache, att.v_cache):
        c.copy_(torch.randn((max_pos, hidden), device=dev, generator=g))
    err = []
    for pos in (1000, max_pos - 1):
        pos_t.fill_(pos)
        got = att.launch()[0].double().view(n_heads, d)
        cos, sin = table[pos, :, 0].double(), table[pos, :, 1].double()
        q = lin[0].double().view(n_heads, d)
        q = torch.cat([q[:, :d // 2] * cos - q[:, d // 2:] * sin, q[:, :d // 2] * sin + q[:, d // 2:] * cos], 1)
        k, v = (c[:pos + 1].view(pos + 1, n_heads, d).transpose(0, 1).double().contiguous() for c in (att.k_cache, att.v_cache))
        w = torch.softmax((k * q[:, None]).sum(2) / d ** 0.5, 1)
        want = (w[:, :, None] * v).sum(1)
        err.append(float((got - want).norm() / want.norm()))
    assert err[1] <= 1.25 * err[0], err


@pytest.mark.parametrize("n_heads,head_dim", [(2, 64), (1, 256), (2, 36)])
def test_attn_decode_merges_of_every_size(dev, mods, n_heads, head_dim):
    """The last workgroup reads up to 16 or up to 64 deposits in one round: positions that leave 2, 16, 17 and 64 deposits, in a
    cache whose counters lie behind the deposits and in a longer one whose counters lie between them; twice each (the counters
    must be back at zero) and with fewer workgroups in between, against the fp64 softmax."""
    for chunks in (64, 66):
        _merges_of_every_size(dev, mods, n_heads, head_dim, chunks)


def _merges_of_every_size(dev, mods, n_heads, head_dim, chunks):
    B, dec, ops = mods
    hidden = n_heads * head_dim
    max_pos = 64 * chunks
    r = _rng(53500 + hidden)
    table = dec.rope_table(head_dim, max_pos, dev)
    q_t, k_t, v_t = (torch.empty((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, table)
    for c in (att.k_cache, att.v_cache):
        c.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(r.standard_normal((max_pos, hidden)).astype(np.float32)), dev))
    try:
        for used in (2, 16, 17, 64):
            B.bl_set_tuning("attn_groups", 1000)
            pos = 64 * used - 1 - used % 3
            ql, kl, vl = (3.0 * r.standard_normal(hidden).astype(np.float32) for _ in range(3))
            q_t.copy_(_t(ql[None], dev)); k_t.copy_(_t(kl[None], dev)); v_t.copy_(_t(vl[None], dev))
            pos_t.fill_(pos)
            first = att.launch().clone()
            B.bl_set_tuning("attn_groups", 3)
            fewer = att.launch().clone()
            B.bl_set_tuning("attn_groups", 1000)
            again = att.launch()
            torch.cuda.synchronize()
            assert torch.equal(first, again) and float((fewer - again).abs().max()) <= 2e-5 * max(1.0, float(again.abs().max()))
            kc64, vc64 = (c[:pos + 1].float().cpu().numpy().astype(np.float64) for c in (att.k_cache, att.v_cache))
            want = D.attention_decode(D.rope(ql, pos, n_heads), kc64, vc64, n_heads)
            assert np.abs(again.cpu().numpy()[0] - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), used
    finally:
        B.bl_set_tuning("attn_groups", 0)


@pytest.mark.parametrize("n_heads,head_dim", [(2, 64), (1, 200), (2, 36), (3, 4)])
def test_attn_decode_every_position_of_a_short_cache(dev, mods, n_heads, head_dim):
    """One chunk per workgroup, waves and steps without a row, then the first two-chunk positions; token after token, against the
    fp64 softmax."""
    B, dec, ops = mods
    hidden, max_pos = n_heads * head_dim, 140
    r = _rng(53900 + hidden)
    table = dec.rope_table(head_dim, max_pos, dev)
    lin = [torch.empty((1, hidden), device=dev) for _ in range(3)]
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, *lin, pos_t, table)
    for pos in range(max_pos):
        vals = [(3.0 * r.standard_normal(hidden)).astype(np.float32) for _ in range(3)]
        for t, v in zip(lin, vals):
            t.copy_(_t(v[None], dev))
        pos_t.fill_(pos)
        out = att.launch().cpu().numpy()[0]
        kc64, vc64 = (c[:pos + 1].float().cpu().numpy().astype(np.float64) for c in (att.k_cache, att.v_cache))
        want = D.attention_decode(D.rope(vals[0], pos, n_heads), kc64, vc64, n_heads)
        assert np.abs(out - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), pos


@pytest.mark.parametrize("pattern", [0x7FC0, 0x7F80, 0xFF80])
@pytest.mark.parametrize("n_heads,head_dim,groups", [(3, 64, 0), (2, 128, 3), (1, 256, 2)])
def test_attn_decode_cache_rows_beyond_the_token_may_hold_anything(dev, mods, pattern, n_heads, head_dim, groups):
    """The caches are the caller's memory and only rows 0 .. pos have ever been written: the rows from `pos` on hold
    NaN or infinity patterns here (row `pos` too, until this launch appends it).  Outputs must be those of the fp64
    softmax over rows 0 .. pos, untouched by what lies behind them."""
    B, dec, ops = mods
    max_pos, hidden = 200, n_heads * head_dim
    r = _rng(54000 + hidden + pattern)
    table = dec.rope_table(head_dim, max_pos, dev)
    q_t, k_t, v_t = (torch.empty((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, table)
    kc = _bf16(r.standard_normal((max_pos, hidden)))
    vc = _bf16(r.standard_normal((max_pos, hidden)))
    B.bl_set_tuning("attn_groups", groups)
    try:
        for pos in (0, 5, 63, 64, 100, 191):
            kb, vb = synth.to_bf16_bits(kc), synth.to_bf16_bits(vc)
            kb[pos:], vb[pos:] = pattern, pattern
            att.k_cache.copy_(_bits_as_bf16_tensor(kb, dev))
            att.v_cache.copy_(_bits_as_bf16_tensor(vb, dev))
            ql, kl, vl = (3.0 * r.standard_normal(hidden).astype(np.float32) for _ in range(3))
            q_t.copy_(_t(ql[None], dev)); k_t.copy_(_t(kl[None], dev)); v_t.copy_(_t(vl[None], dev))
            pos_t.fill_(pos)
            out = att.launch()
            torch.cuda.synchronize()
            kc64, vc64 = kc[:pos + 1].astype(np.float64), vc[:pos + 1].astype(np.float64)
            kc64[pos] = att.k_cache[pos].float().cpu().numpy().astype(np.float64)
            vc64[pos] = att.v_cache[pos].float().cpu().numpy().astype(np.float64)
            want = D.attention_decode(D.rope(ql, pos, n_heads), kc64, vc64, n_heads)
            got = out.cpu().numpy()[0]
            assert np.all(np.isfinite(got)), pos
            assert np.abs(got - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), (pos, float(np.abs(got - want).max()))
    finally:
        B.bl_set_tuning("attn_groups", 0)


def test_attn_decode_long_context_as_launched(dev, mods):
    """The 7B shape's attention (32 heads of 128) on a cache of 4096 positions, in the launch configuration the token
    loop uses: 32 workgroups per head, two chunks each near the end of the cache.  Sampled positions against the fp64
    softmax."""
    B, dec, ops = mods
    n_heads, head_dim, max_pos = 32, 128, 4096
    hidden = n_heads * head_dim
    r = _rng(54000)
    table = dec.rope_table(head_dim, max_pos, dev)
    q_t, k_t, v_t = (torch.empty((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, table)
    g = torch.Generator(device=dev).manual_seed(54001)
    att.k_cache.copy_(torch.randn((max_pos, hidden), device=dev, generator=g))
    att.v_cache.copy_(torch.randn((max_pos, hidden), device=dev, generator=g))
    for pos in (2047, 2048, 3000, 4095):
        ql, kl, vl = (3.0 * r.standard_normal(hidden).astype(np.float32) for _ in range(3))
        q_t.copy_(_t(ql[None], dev)); k_t.copy_(_t(kl[None], dev)); v_t.copy_(_t(vl[None], dev))
        pos_t.fill_(pos)
        out = att.launch()
        torch.cuda.synchronize()
        kc64 = att.k_cache[:pos + 1].float().cpu().numpy().astype(np.float64)
        vc64 = att.v_cache[:pos + 1].float().cpu().numpy().astype(np.float64)
        want = D.attention_decode(D.rope(ql, pos, n_heads), kc64, vc64, n_heads)
        got = out.cpu().numpy()[0]
        assert np.abs(got - want).max() <= 2e-5 * max(1.0, np.abs(want).max()), (pos, float(np.abs(got - want).max()))
    assert not att.scratch[-4 * n_heads:].view(torch.int32).any()


def test_attn_prefill_long_prompt_sampled(dev, mods):
    """A piece of 1000 tokens behind 700 cached ones (8 heads of 128: 16 blocks of 64 tokens per head, up to 27 chunks
    each): sampled tokens against the fp64 softmax over the cache as stored."""
    B, dec, ops = mods
    n_heads, head_dim, max_pos, pos0, M = 8, 128, 1700, 700, 1000
    hidden = n_heads * head_dim
    r = _rng(54100)
    table = dec.rope_table(head_dim, max_pos, dev)
    g = torch.Generator(device=dev).manual_seed(54101)
    k_cache = torch.randn((max_pos, hidden), device=dev, generator=g).to(torch.bfloat16)
    v_cache = torch.randn((max_pos, hidden), device=dev, generator=g).to(torch.bfloat16)
    lin = [3.0 * r.standard_normal((M, hidden)).astype(np.float32) for _ in range(3)]
    lin_t = [_t(v, dev) for v in lin]
    out = torch.empty((M, hidden), device=dev)
    scratch = torch.zeros(B.bl_attn_prefill_scratch_bytes(n_heads, head_dim, pos0, M), dtype=torch.uint8, device=dev)
    B.bl_attn_prefill(lin_t[0].data_ptr(), lin_t[1].data_ptr(), lin_t[2].data_ptr(), table.data_ptr(), k_cache.data_ptr(),
                      v_cache.data_ptr(), out.data_ptr(), scratch.data_ptr(), n_heads, head_dim, max_pos, pos0, M,
                      torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    kc64, vc64 = k_cache.float().cpu().numpy().astype(np.float64), v_cache.float().cpu().numpy().astype(np.float64)
    got = out.cpu().numpy()
    assert np.isfinite(got).all()
    for m in (0, 63, 64, 500, 959, 960, 999):
        want = D.attention_decode(D.rope(lin[0][m], pos0 + m, n_heads), kc64[:pos0 + m + 1], vc64[:pos0 + m + 1], n_heads)
        assert np.abs(got[m] - want).max() <= PREFILL_BLOCK_TOL * max(1.0, np.abs(want).max()), m
    want_v = synth.to_bf16_bits(lin[2][M - 1])
    np.testing.assert_array_equal(v_cache[pos0 + M - 1].view(torch.int16).cpu().numpy().view(np.uint16), want_v)


def test_attn_decode_out_of_range_position_does_nothing(dev, mods):
    B, dec, ops = mods
    n_heads, head_dim, max_pos = 2, 64, 16
    hidden = n_heads * head_dim
    q_t, k_t, v_t = (torch.ones((1, hidden), device=dev) for _ in range(3))
    pos_t = torch.full((1,), max_pos, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, q_t, k_t, v_t, pos_t, dec.rope_table(head_dim, max_pos, dev))
    att.out.fill_(-5.0)
    att.launch()
    pos_t.fill_(-1)
    att.launch()
    torch.cuda.synchronize()
    assert torch.all(att.out == -5.0) and not att.k_cache.any() and not att.v_cache.any()


def test_pos_advance(dev, mods):
    B, dec, ops = mods
    pos = torch.full((1,), 41, dtype=torch.int32, device=dev)
    for _ in range(3):
        B.bl_pos_advance(pos.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert int(pos[0]) == 44


# ------------------------------------------------------------------------------------------ layers, tokens

def _make_layers(seed, hidden, ffn, n_layers):
    r = _rng(seed)
    layers = []
    for _ in range(n_layers):
        layer = {}
        for name, (n, k) in {"q": (hidden, hidden), "k": (hidden, hidden), "v": (hidden, hidden), "o": (hidden, hidden),
                             "gate": (ffn, hidden), "up": (ffn, hidden), "down": (hidden, ffn)}.items():
            layer[name] = synth.ternary_weights(r, n, k)
            layer["s_" + name] = synth.draw_w_scale(r)
        for g, k in (("g_in", hidden), ("g_attn", hidden), ("g_post", hidden), ("g_ffn", ffn)):
            layer[g] = r.uniform(0.5, 1.5, k).astype(np.float32)
        layers.append(layer)
    return layers, r.uniform(0.5, 1.5, hidden).astype(np.float32)


def _to_device(layers, dev, dec, ops, gated=False):
    out = []
    for l in layers:
        proj = {n: ops.pack_ternary(_t(l[n], dev), float(l["s_" + n])) for n in ("q", "k", "v", "o", "gate", "up", "down")}
        if gated:
            proj["gate_up"] = dec.pack_gate_up(_t(l["gate"], dev), _t(l["up"], dev), float(l["s_gate"]))
        out.append(dec.LayerWeights(proj, *(_t(l[g], dev) for g in ("g_in", "g_attn", "g_post", "g_ffn")),
                                    s_up=float(l["s_up"])))
    return out


def _codes_close(got, y64, K):
    """The int8 codes of a row against the oracle's quantizer on the fp64 normalised row: equal except where the
    fp32 value sits within rounding error of a tie (then one step apart); at most a handful of those per row."""
    q, _, _ = oracle.quant_act(y64.astype(np.float32)[None, :])
    diff = np.abs(got[0, :K].astype(np.int32) - q[0].astype(np.int32))
    assert diff.max() <= 1 and np.count_nonzero(diff) <= max(2, K // 500), (int(diff.max()), int(np.count_nonzero(diff)))


def _product_of(qa, K, w, s):
    """The oracle's product on the GPU's own quantized row."""
    q = qa.q.cpu().numpy()[:, :K]
    return oracle.dequant(oracle.matmul_i32(q, w), np.float32(s), qa.a_scale.cpu().numpy())[0].astype(np.float64)


@pytest.mark.parametrize("hidden,ffn,n_heads,pos", [(1536, 4096, 16, 3), (768, 3072, 12, 0), (3200, 8640, 32, 300)])
def test_layer_stage_by_stage(dev, mods, hidden, ffn, n_heads, pos):
    """One layer, one token, every intermediate buffer: each stage against the oracle applied to the GPU's OWN
    output of the stage before, so that no difference is carried along.  Products are bit-exact in their integer
    sums; normalisations and attention hold their fp32 tolerance; codes differ only at ties."""
    B, dec, ops = mods
    max_pos = 512
    (l,), _ = _make_layers(63000 + hidden, hidden, ffn, 1)
    r = _rng(64000 + hidden)
    h0, delta = synth.activations(r, 1, hidden), synth.activations(r, 1, hidden)
    h_t, pos_t = _t(h0, dev), torch.full((1,), pos, dtype=torch.int32, device=dev)
    table = dec.rope_table(hidden // n_heads, max_pos, dev)
    layer = dec.DecoderLayer(_to_device([l], dev, dec, ops)[0], n_heads, max_pos, h_t, torch.empty_like(h_t), _t(delta, dev),
                             pos_t, table, fold_norm=False)
    kc = _bf16(r.standard_normal((max_pos, hidden)))
    vc = _bf16(r.standard_normal((max_pos, hidden)))
    layer.attn.k_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(kc), dev))
    layer.attn.v_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(vc), dev))
    # the launches one by one, so that the residual stream can be read between its two updates
    w = layer.w
    dec.norm_quant(B.BL_NORM_RESIDUAL, w.g_in, layer.eps, a=layer.delta_in, h=layer.h, out=layer.q1)
    h1 = h_t.cpu().numpy()
    np.testing.assert_array_equal(h1, h0 + delta)
    _codes_close(layer.q1.q.cpu().numpy(), D.rmsnorm(h1[0].astype(np.float64), l["g_in"], 1e-5), hidden)
    layer.qkv.launch()
    lin = {}
    for name, out in zip("qkv", layer.qkv.outs):
        lin[name] = out.cpu().numpy()[0]
        np.testing.assert_allclose(lin[name], _product_of(layer.q1, hidden, l[name], l["s_" + name]), rtol=1e-6)
    layer.attn.launch()
    k_row = layer.attn.k_cache[pos].float().cpu().numpy().astype(np.float64)
    v_row = layer.attn.v_cache[pos].float().cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(v_row, D.round_to_bf16(lin["v"]))
    want_k = D.round_to_bf16(D.rope(lin["k"], pos, n_heads))
    assert np.all(np.abs(k_row - want_k) <= np.maximum(np.abs(want_k), 1e-30) * 2.0 ** -7) and np.mean(k_row == want_k) >= 0.99
    kc64, vc64 = kc.astype(np.float64), vc.astype(np.float64)
    kc64[pos], vc64[pos] = k_row, v_row
    attn = layer.attn.out.cpu().numpy()[0]
    want = D.attention_decode(D.rope(lin["q"], pos, n_heads), kc64[:pos + 1], vc64[:pos + 1], n_heads)
    assert np.abs(attn - want).max() <= 2e-5 * max(1.0, np.abs(want).max())
    dec.norm_quant(B.BL_NORM_PLAIN, w.g_attn, layer.eps, a=layer.attn.out, out=layer.q2)
    _codes_close(layer.q2.q.cpu().numpy(), D.rmsnorm(attn.astype(np.float64), l["g_attn"], 1e-5), hidden)
    layer.o.launch()
    o = layer.o.outs[0].cpu().numpy()
    np.testing.assert_allclose(o[0], _product_of(layer.q2, hidden, l["o"], l["s_o"]), rtol=1e-6)
    dec.norm_quant(B.BL_NORM_RESIDUAL, w.g_post, layer.eps, a=layer.o.outs[0], h=layer.h, out=layer.q3)
    h2 = h_t.cpu().numpy()
    np.testing.assert_array_equal(h2, h1 + o)
    _codes_close(layer.q3.q.cpu().numpy(), D.rmsnorm(h2[0].astype(np.float64), l["g_post"], 1e-5), hidden)
    layer.gate_up.launch()
    gate, up = (t.cpu().numpy()[0] for t in layer.gate_up.outs)
    np.testing.assert_allclose(gate, _product_of(layer.q3, hidden, l["gate"], l["s_gate"]), rtol=1e-6)
    np.testing.assert_allclose(up, _product_of(layer.q3, hidden, l["up"], l["s_up"]), rtol=1e-6)
    dec.norm_quant(B.BL_NORM_GATED, w.g_ffn, layer.eps, a=layer.gate_up.outs[0], b=layer.gate_up.outs[1], out=layer.q4)
    _codes_close(layer.q4.q.cpu().numpy(), D.rmsnorm(D.gated_ffn_input(gate, up), l["g_ffn"], 1e-5), ffn)
    layer.down.launch()
    torch.cuda.synchronize()
    np.testing.assert_allclose(layer.delta_out.cpu().numpy()[0], _product_of(layer.q4, ffn, l["down"], l["s_down"]), rtol=1e-6)


# ------------------------------------------------------------------------------------------ norm folded into the product

def _run_norm_decode(dev, mods, r, K, Ns, with_delta, use_workspace):
    B, dec, ops = mods
    ws = [synth.ternary_weights(r, N, K) for N in Ns]
    scales = [float(synth.draw_w_scale(r)) for _ in Ns]
    x = synth.activations(r, 1, K, outlier_frac=0.01)
    delta = synth.activations(r, 1, K) if with_delta else None
    gamma = r.uniform(0.5, 1.5, K).astype(np.float32)
    pws = [ops.pack_ternary(_t(w, dev), s) for w, s in zip(ws, scales)]
    h_out = torch.full((1, K), -7.0, device=dev) if with_delta else None
    grp = dec.NormDecodeGroup(pws, _t(x, dev), _t(gamma, dev), 1e-5, delta=_t(delta, dev) if with_delta else None,
                              h_out=h_out, want_acc=True, want_quant=True, use_workspace=use_workspace)
    outs = [o.cpu().numpy()[0] for o in grp.launch()]
    torch.cuda.synchronize()
    return ws, scales, x, delta, gamma, grp, outs, h_out


@pytest.mark.parametrize("K,Ns,with_delta,use_workspace", [
    (200, (70,), True, False), (768, (768, 768, 768), True, True), (1536, (1536,), False, True),
    (3200, (3200, 3200, 3200), True, True), (4096, (11008, 11008), True, True), (8192, (8192, 8192, 8192), True, True),
    (8192, (8192,), False, False), (16384, (640,), True, True), (4096, (4096,), False, True), (8, (3,), True, False),
    (8192, (45568,), True, True)])   # the last: one of the 100B shape's gate/up matrices (Appendix A)
def test_decode_norm_batch_parity(dev, mods, K, Ns, with_delta, use_workspace):
    """RMSNorm folded into the fused quantizer: codes, scale and sums against the oracle's quantizer on
    z = (x + delta) * gamma formed with the same two fp32 operations; the scale carries the norm's scalar; the
    integer sums are exact; against the textbook order (normalise, then quantize) codes differ at ties only."""
    B, dec, ops = mods
    ws, scales, x, delta, gamma, grp, outs, h_out = _run_norm_decode(dev, mods, _rng(71000 + K + len(Ns)), K, Ns, with_delta, use_workspace)
    xp = x + delta if with_delta else x                                   # one fp32 addition
    if with_delta:
        np.testing.assert_array_equal(h_out.cpu().numpy(), xp)
    z = xp * gamma                                                        # one fp32 product
    q, a_z, q_sum = oracle.quant_act(z)
    r64 = 1.0 / np.sqrt(np.mean(xp.astype(np.float64) ** 2) + 1e-5)
    y64 = D.rmsnorm(xp[0].astype(np.float64), gamma, 1e-5)
    for i, (w, s) in enumerate(zip(ws, scales)):
        qa = grp.quants[i]
        np.testing.assert_array_equal(qa.q.cpu().numpy()[:, :K], q)
        assert not qa.q.cpu().numpy()[:, K:].any()
        np.testing.assert_array_equal(qa.q_sum.cpu().numpy(), q_sum)
        a_got = float(qa.a_scale[0])
        assert abs(a_got - float(a_z[0]) * r64) <= 3e-6 * float(a_z[0]) * r64      # fp32 tree sum of K squares, root, division
        acc = oracle.matmul_i32(q, w)
        np.testing.assert_array_equal(grp.accs[i].cpu().numpy(), acc)
        np.testing.assert_allclose(outs[i], oracle.dequant(acc, np.float32(s), np.float32([a_got]))[0], rtol=1e-6)
        _codes_close(qa.q.cpu().numpy(), y64, K)
        q_txt, a_txt, _ = oracle.quant_act(y64.astype(np.float32)[None, :])
        if np.array_equal(q_txt, q):                                      # no tie fell the other way: the textbook product
            want = oracle.dequant(acc, np.float32(s), a_txt)[0]
            assert np.abs(outs[i] - want).max() <= 5e-6 * np.abs(want).max()


def test_decode_norm_batch_zero_row(dev, mods):
    B, dec, ops = mods
    K, N = 1024, 300
    pw = ops.pack_ternary(_t(synth.ternary_weights(_rng(3), N, K), dev), 0.02)
    grp = dec.NormDecodeGroup([pw], torch.zeros((1, K), device=dev), torch.ones(K, device=dev), want_quant=True)
    out = grp.launch()[0]
    torch.cuda.synchronize()
    assert not out.any() and float(grp.quants[0].a_scale[0]) == 0.0 and not grp.quants[0].q.any()


@pytest.mark.parametrize("F,K", [(32, 64), (96, 200), (4096, 1536), (224, 3200)])
def test_pack_gate_up_layout(dev, mods, F, K):
    """bl_pack_gate_up is bl_pack_ternary of the two matrices interleaved by 32 rows: unpacking gives gate rows
    32 b .. 32 b + 31 in rows 64 b .. 64 b + 31 and the up rows of the same outputs behind them; non-ternary inputs
    of either matrix are counted and stored as 0."""
    B, dec, ops = mods
    r = _rng(56000 + F + K)
    wg, wu = synth.ternary_weights(r, F, K), synth.ternary_weights(r, F, K, p_zero=0.5)
    pw = dec.pack_gate_up(_t(wg, dev), _t(wu, dev), 0.03)
    back = ops.unpack_ternary(pw).cpu().numpy().reshape(F // 32, 2, 32, K)
    np.testing.assert_array_equal(back[:, 0].reshape(F, K), wg)
    np.testing.assert_array_equal(back[:, 1].reshape(F, K), wu)
    both = np.stack([wg.reshape(F // 32, 32, K), wu.reshape(F // 32, 32, K)], axis=1).reshape(2 * F, K)
    ref = ops.pack_ternary(_t(both, dev), 0.03)
    assert torch.equal(ref.blob, pw.blob)
    wg2, wu2 = wg.copy(), wu.copy()
    wg2[0, 0], wu2[F - 1, K - 1], wu2[3, 1] = 2, -2, 77
    bad = torch.zeros(1, dtype=torch.int32, device=dev)
    desc = B.bl_packed_desc_init(2 * F, K, 0.03)
    blob = torch.empty(int(desc.bytes), dtype=torch.uint8, device=dev)
    wg2_d, wu2_d = _t(wg2, dev), _t(wu2, dev)
    B.bl_pack_gate_up(wg2_d.data_ptr(), wu2_d.data_ptr(), desc, blob.data_ptr(), bad.data_ptr(),
                      int(torch.cuda.current_stream().cuda_stream))
    assert int(bad[0]) == 3
    back = ops.unpack_ternary(ops.PackedWeight(blob, desc)).cpu().numpy().reshape(F // 32, 2, 32, K)
    assert back[0, 0, 0, 0] == 0 and back[-1, 1, -1, -1] == 0 and back[0, 1, 3, 1] == 0


@pytest.mark.parametrize("waves", [4, 8, 16])
def test_gated_launch_with_forced_waves_per_row_block(dev, mods, waves):
    """The gated epilogue when a workgroup holds one, two or four row blocks."""
    B, dec, ops = mods
    B.bl_set_tuning("gemv_waves", waves)
    try:
        test_gated_launch_and_its_consumer(dev, mods, 4096, 12032, True)
        test_gated_launch_and_its_consumer(dev, mods, 768, 3072, False)
    finally:
        B.bl_set_tuning("gemv_waves", 0)


@pytest.mark.parametrize("K,F,with_delta", [(768, 3072, True), (4096, 12032, True), (1536, 4096, False), (64, 32, True),
                                          (3200, 8640, True), (512, 20000, True), (8192, 45568, False)])
def test_gated_launch_and_its_consumer(dev, mods, K, F, with_delta):
    """Gate and up interleaved in one matrix: the launch's epilogue leaves silu(gate) * up * g_ffn and the pieces of
    sum((silu(gate) * up)^2); the down projection quantizes that row as it is.  Integer sums exact; the gate and up
    values reproduced with the kernel's own two fp32 products; the rest within fp32 tolerance of the fp64 formulas."""
    _gated_case(dev, mods, K, F, with_delta)


@pytest.mark.parametrize("split", [1, 2, 3])
@pytest.mark.parametrize("K,F,with_delta", [(4096, 12032, True), (1536, 9216, False), (2560, 6912, True), (64, 32, True),
                                          (5120, 13824, True), (192, 2080, False)])
def test_gated_launch_work_balanced(dev, mods, split, K, F, with_delta):
    """The same launch in the work-balanced form (forced: `split` workgroups per compute unit): row blocks cut across
    workgroups are finished by whichever of them draws the block's last ticket, all 64 rows in one wave.  Run twice, so
    that the second launch finds the workspace as the first left it; the launch taken is the balanced one."""
    B, dec, ops = mods
    B.bl_set_tuning("decode_split", split)
    try:
        before = B.bl_get_stat("split_launches")
        for _ in range(2):
            _gated_case(dev, mods, K, F, with_delta)
        if K * F >= 2048 * 2048 * split:   # at least 8 tiles per workgroup: the balanced form is planned
            assert B.bl_get_stat("split_launches") > before
        assert not ops.workspace(dev).any(), "the workspace must be left zero"
    finally:
        B.bl_set_tuning("decode_split", 0)


def _gated_case(dev, mods, K, F, with_delta):
    B, dec, ops = mods
    r = _rng(81000 + K + F)
    wg, wu, wd = synth.ternary_weights(r, F, K), synth.ternary_weights(r, F, K), synth.ternary_weights(r, 200, F)
    sg, su, sd = (float(synth.draw_w_scale(r)) for _ in range(3))
    x = synth.activations(r, 1, K, outlier_frac=0.01)
    delta = synth.activations(r, 1, K) if with_delta else None
    g_post, g_ffn = (r.uniform(0.5, 1.5, n).astype(np.float32) for n in (K, F))
    pw = dec.pack_gate_up(_t(wg, dev), _t(wu, dev), sg)
    assert pw.N == 2 * F
    h_out = torch.empty((1, K), device=dev) if with_delta else None
    up_grp = dec.NormDecodeGroup([pw], _t(x, dev), _t(g_post, dev), 1e-5, delta=_t(delta, dev) if with_delta else None,
                                 h_out=h_out, want_acc=True, want_quant=True, glu=(su, _t(g_ffn, dev)))
    z_t = up_grp.launch()[0]
    pwd = ops.pack_ternary(_t(wd, dev), sd)
    folded_down = dec.can_fold_norm(F)
    if folded_down:
        down = dec.NormDecodeGroup([pwd], z_t, None, 1e-5, pieces=up_grp.pieces, want_acc=True, want_quant=True)
        out = down.launch()[0].cpu().numpy()[0]
        down_q, down_acc = down.quants[0], down.accs[0]
    else:   # a row too long for the product's quantizer: bl_norm_quant on the same pieces, twice (the word behind
            # the pieces must be back at zero), then the plain product
        y_t = torch.empty((1, F), device=dev)
        for _ in range(2):
            down_q = ops.alloc_quant(1, F, dev)
            down_q.q_sum.fill_(777)
            dec.norm_quant(B.BL_NORM_PREMULTIPLIED, None, 1e-5, a=z_t, out=down_q, y=y_t, scratch=up_grp.pieces, pieces=F // 32)
        out_t, down_acc = ops.gemv(pwd, down_q, want_acc=True)
        out = out_t.cpu().numpy()[0]
    torch.cuda.synchronize()
    # the gated launch
    xp = x + delta if with_delta else x
    q, a_z, _ = oracle.quant_act(xp * g_post)
    np.testing.assert_array_equal(up_grp.quants[0].q.cpu().numpy()[:, :K], q)
    acc = up_grp.accs[0].cpu().numpy()[0].reshape(F // 32, 2, 32)
    np.testing.assert_array_equal(acc[:, 0, :].reshape(F), oracle.matmul_i32(q, wg)[0])
    np.testing.assert_array_equal(acc[:, 1, :].reshape(F), oracle.matmul_i32(q, wu)[0])
    a_got = up_grp.quants[0].a_scale.cpu().numpy()[0]
    gate = acc[:, 0, :].reshape(F).astype(np.float32) * (np.float32(sg) * a_got)      # the kernel's two fp32 products
    up = acc[:, 1, :].reshape(F).astype(np.float32) * (np.float32(su) * a_got)
    prod = D.gated_ffn_input(gate, up)
    z = z_t.cpu().numpy()[0]
    assert np.abs(z - prod * g_ffn).max() <= 3e-6 * np.abs(prod * g_ffn).max()
    pairs = up_grp.pieces.cpu().numpy()
    assert not pairs[-1].any()                                          # the word behind the pieces is (back at) zero
    pieces, maxima = pairs[:-1, 0], pairs[:-1, 1]
    want_pieces = (prod ** 2).reshape(F // 32, 32).sum(axis=1)
    assert np.all(np.abs(pieces - want_pieces) <= 1e-5 * want_pieces.max())
    np.testing.assert_array_equal(maxima, np.abs(z).reshape(F // 32, 32).max(axis=1))
    r64 = 1.0 / np.sqrt(np.sum(pieces.astype(np.float64)) / F + 1e-5)
    a_d = float(down_q.a_scale[0])
    if folded_down:   # the consumer quantizes z as it is; the scalar from the pieces goes into the scale
        qz, az, sz = oracle.quant_act(z[None, :])
        assert abs(a_d - float(az[0]) * r64) <= 3e-6 * float(az[0]) * r64
    else:             # ... or forms y = z * r and quantizes that: codes against the oracle's quantizer on the kernel's own y
        y = y_t.cpu().numpy()
        assert np.abs(y[0] - z.astype(np.float64) * r64).max() <= 3e-6 * np.abs(z).max() * r64
        qz, az, sz = oracle.quant_act(y)
        assert a_d == float(az[0])
    np.testing.assert_array_equal(down_q.q.cpu().numpy()[:, :F], qz)
    assert not down_q.q.cpu().numpy()[:, F:].any()
    np.testing.assert_array_equal(down_q.q_sum.cpu().numpy(), sz)
    acc_d = oracle.matmul_i32(qz, wd)
    np.testing.assert_array_equal(down_acc.cpu().numpy(), acc_d)
    np.testing.assert_allclose(out, oracle.dequant(acc_d, np.float32(sd), np.float32([a_d]))[0], rtol=1e-6)
    # ... and against the textbook order: normalise silu(gate) * up, then quantize -- codes differ at ties only
    _codes_close(down_q.q.cpu().numpy(), D.rmsnorm(prod, g_ffn, 1e-5), F)


@pytest.mark.parametrize("hidden,ffn,n_heads,n_layers,use_graph,fold", [
    (768, 3072, 12, 2, False, True), (1536, 4096, 16, 2, True, True), (200, 328, 5, 3, True, True),
    (768, 3072, 12, 2, False, False), (1536, 4096, 16, 3, True, False), (768, 3072, 12, 2, True, "gated"),
    (200, 320, 5, 3, False, "gated")])
def test_token_loop_against_oracle(dev, mods, hidden, ffn, n_heads, n_layers, use_graph, fold):
    """Tokens through a small stack (125M- and 700M-shape layers of Appendix A): the final-normalised hidden state and
    the caches against the oracle's layer step, token after token; the captured graph gives the eager bits."""
    B, dec, ops = mods
    max_pos, n_tokens = 8, 5
    layers, g_final = _make_layers(61000 + hidden, hidden, ffn, n_layers)
    gated, fold = fold == "gated", bool(fold)
    stack = dec.DecoderStack(_to_device(layers, dev, dec, ops, gated), _t(g_final, dev), n_heads, max_pos, dev, fold_norm=fold)
    assert all(l.fold == fold and l.gated == gated for l in stack.layers)
    eager = (dec.DecoderStack(_to_device(layers, dev, dec, ops, gated), _t(g_final, dev), n_heads, max_pos, dev, fold_norm=fold)
             if use_graph else None)
    if use_graph:
        stack.capture()
    r = _rng(62000 + hidden)
    kcs = [np.zeros((max_pos, hidden)) for _ in layers]
    vcs = [np.zeros((max_pos, hidden)) for _ in layers]
    for pos in range(n_tokens):
        x = r.standard_normal((1, hidden)).astype(np.float32)
        stack.h.copy_(_t(x, dev))
        y = stack.step()
        torch.cuda.synchronize()
        assert int(stack.pos[0]) == pos + 1
        if use_graph:
            eager.h.copy_(_t(x, dev))
            y2 = eager.step()
            torch.cuda.synchronize()
            assert torch.equal(y, y2)
            for a, b in zip(stack.layers, eager.layers):
                assert torch.equal(a.attn.k_cache.view(torch.int16), b.attn.k_cache.view(torch.int16))
        h = x[0].astype(np.float64)
        for i, l in enumerate(layers):
            h = D.decoder_layer_step(h, pos, l, kcs[i], vcs[i], n_heads)
        want = D.rmsnorm(h, g_final, 1e-5)
        got = y.cpu().numpy()[0].astype(np.float64)
        # A bound, not an identity: the two sides' quantizers see inputs that differ in the last bits (fp32 against
        # fp64), and one code that falls the other way moves every output of its product.  The oracle ALONE, run
        # twice on this stack with 1e-6 relative noise added to the residual stream between layers, differs from
        # itself by 1e-6 on most tokens and by 1e-2 on the tokens where a code flips; test_layer_stage_by_stage
        # is the comparison without that carry-over.
        assert np.linalg.norm(got - want) <= 5e-2 * np.linalg.norm(want), np.linalg.norm(got - want) / np.linalg.norm(want)
        for i, layer in enumerate(stack.layers):
            got_v = layer.attn.v_cache[pos].float().cpu().numpy().astype(np.float64)
            assert np.linalg.norm(got_v - vcs[i][pos]) <= 5e-2 * np.linalg.norm(vcs[i][pos])


def test_stack_refuses_a_token_beyond_the_cache(dev, mods):
    B, dec, ops = mods
    layers, g_final = _make_layers(65000, 64, 128, 1)
    stack = dec.DecoderStack(_to_device(layers, dev, dec, ops), _t(g_final, dev), 2, 3, dev)
    for _ in range(3):
        stack.step()
    torch.cuda.synchronize()
    assert int(stack.pos[0]) == 3
    with pytest.raises(RuntimeError):
        stack.step()
    stack.set_position(1)
    stack.step()
    torch.cuda.synchronize()
    assert int(stack.pos[0]) == 2


def test_long_token_loop_graph_equals_eager_across_chunk_boundaries(dev, mods):
    """140 tokens through a small stack, as replays of one captured graph and as eager launches: the same bits on
    every token, across the 64- and 128-row chunk boundaries of the attention kernel (whose per-head ticket counters
    must be back at zero after every launch), and finite throughout."""
    B, dec, ops = mods
    hidden, ffn, n_heads, n_layers, max_pos, n_tokens = 256, 512, 4, 2, 160, 140
    layers, g_final = _make_layers(66000, hidden, ffn, n_layers)
    a = dec.DecoderStack(_to_device(layers, dev, dec, ops, True), _t(g_final, dev), n_heads, max_pos, dev)
    b = dec.DecoderStack(_to_device(layers, dev, dec, ops, True), _t(g_final, dev), n_heads, max_pos, dev)
    a.capture()
    x = torch.randn((n_tokens, 1, hidden), device=dev, generator=torch.Generator(device=dev).manual_seed(5))
    for t in range(n_tokens):
        a.h.copy_(x[t])
        b.h.copy_(x[t])
        ya, yb = a.step(), b.step()
        if t in (0, 63, 64, 65, 127, 128, 129, n_tokens - 1):
            torch.cuda.synchronize()
            assert torch.equal(ya, yb) and bool(torch.isfinite(ya).all()), t
    torch.cuda.synchronize()
    for la, lb in zip(a.layers, b.layers):
        assert torch.equal(la.attn.k_cache.view(torch.int16), lb.attn.k_cache.view(torch.int16))
        assert torch.equal(la.attn.v_cache.view(torch.int16), lb.attn.v_cache.view(torch.int16))
        counters = la.attn.scratch[-4 * n_heads:].view(torch.int32)
        assert not counters.any()
    assert int(a.pos[0]) == n_tokens == int(b.pos[0])


# A prompt's attention against the fp64 softmax.  Head sizes up to 128 go through the matrix cores with the fp32 queries
# and weights as sums of two bf16 numbers: each carries a relative error below 2^-17 (the remainder of a nearest bf16 is
# below 2^-9 of the value and is itself rounded to 2^-9 of that, plus the fp32 subtraction), so a score is off by at
# most 2^-17 sum|q_i k_i| / sqrt(d) -- a few 1e-5 at the value range used here (queries of spread 3) -- which moves
# every weight by that relative amount, and the weights' own split adds 2^-17 once more.
PREFILL_BLOCK_TOL = 2e-5


@pytest.mark.parametrize("n_heads,head_dim,max_pos,pos0,M", [(3, 64, 300, 0, 70), (3, 64, 300, 130, 100), (20, 128, 80, 5, 9),
                                                           (5, 40, 70, 0, 70), (2, 256, 200, 63, 2), (4, 100, 400, 37, 300),
                                                           (2, 120, 200, 0, 130), (2, 48, 100, 10, 64), (1, 16, 70, 63, 1), (3, 4, 140, 5, 130),
                                                           (2, 36, 90, 0, 65)])
def test_attn_prefill_parity(dev, mods, n_heads, head_dim, max_pos, pos0, M):
    """A prompt's attention: token m against cache rows 0 .. pos0 + m.  The appended rows as in the one-token call, bit
    for bit; every token's output against the fp64 softmax over the cache as stored, and against what M one-token calls
    give (bit for bit where the head size takes the same kernel, above 128)."""
    B, dec, ops = mods
    hidden = n_heads * head_dim
    r = _rng(95000 + hidden + M)
    table = dec.rope_table(head_dim, max_pos, dev)
    kc = _bf16(r.standard_normal((max_pos, hidden)))
    vc = _bf16(r.standard_normal((max_pos, hidden)))
    lin = [3.0 * r.standard_normal((M, hidden)).astype(np.float32) for _ in range(3)]
    lin_t = [_t(v, dev) for v in lin]
    k_cache = _bits_as_bf16_tensor(synth.to_bf16_bits(kc), dev).clone()
    v_cache = _bits_as_bf16_tensor(synth.to_bf16_bits(vc), dev).clone()
    out = torch.empty((M, hidden), device=dev)
    scratch = torch.zeros(B.bl_attn_prefill_scratch_bytes(n_heads, head_dim, pos0, M), dtype=torch.uint8, device=dev)
    for _ in range(2):   # twice: the counters in the scratch memory must be back at zero
        B.bl_attn_prefill(lin_t[0].data_ptr(), lin_t[1].data_ptr(), lin_t[2].data_ptr(), table.data_ptr(), k_cache.data_ptr(),
                          v_cache.data_ptr(), out.data_ptr(), scratch.data_ptr(), n_heads, head_dim, max_pos, pos0, M,
                          torch.cuda.current_stream().cuda_stream)
    # the same tokens one at a time
    one = [torch.empty((1, hidden), device=dev) for _ in range(3)]
    pos_t = torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, *one, pos_t, table)
    att.k_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(kc), dev))
    att.v_cache.copy_(_bits_as_bf16_tensor(synth.to_bf16_bits(vc), dev))
    outs = []
    for m in range(M):
        for t, v in zip(one, lin_t):
            t.copy_(v[m:m + 1])
        pos_t.fill_(pos0 + m)
        outs.append(att.launch().clone())
    torch.cuda.synchronize()
    assert torch.equal(k_cache.view(torch.int16), att.k_cache.view(torch.int16))
    assert torch.equal(v_cache.view(torch.int16), att.v_cache.view(torch.int16))
    stepwise = torch.cat(outs)
    if head_dim > 128:
        assert torch.equal(out, stepwise)
    tol = 2e-5 if head_dim > 128 else PREFILL_BLOCK_TOL
    assert float((out - stepwise).abs().max()) <= tol * max(1.0, float(stepwise.abs().max()))
    if head_dim > 128:
        assert not scratch.view(torch.int32).view(M, -1)[:, -n_heads:].any()
    else:
        assert scratch.numel() == 16 and not scratch.any()
    kc64, vc64 = k_cache.float().cpu().numpy().astype(np.float64), v_cache.float().cpu().numpy().astype(np.float64)
    got = out.cpu().numpy()
    worst = 0.0
    for m in range(M):
        want = D.attention_decode(D.rope(lin[0][m], pos0 + m, n_heads), kc64[:pos0 + m + 1], vc64[:pos0 + m + 1], n_heads)
        err = np.abs(got[m] - want).max() / max(1.0, np.abs(want).max())
        worst = max(worst, err)
        assert err <= tol, (m, err)
    print(f"attn_prefill heads={n_heads} d={head_dim} pos0={pos0} M={M}: worst error {worst:.2e}", flush=True)
    want_k = D.round_to_bf16(D.rope(lin[1][M - 1], pos0 + M - 1, n_heads))
    assert np.all(np.abs(kc64[pos0 + M - 1] - want_k) <= np.maximum(np.abs(want_k), 1e-30) * 2.0 ** -7)


def test_attn_prefill_head_size_above_128_behind_many_chunks(dev, mods):
    """More deposits (a forced workgroup per 64 cache rows and token) than are read in one round, against the fp64 softmax."""
    B, dec, ops = mods
    head_dim, pos0, M, max_pos = 256, 64 * 65 - 1, 2, 64 * 66
    r = _rng(96000)
    table = dec.rope_table(head_dim, max_pos, dev)
    k_cache, v_cache = (_bits_as_bf16_tensor(synth.to_bf16_bits(r.standard_normal((max_pos, head_dim)).astype(np.float32)), dev).clone()
                        for _ in range(2))
    lin = [3.0 * r.standard_normal((M, head_dim)).astype(np.float32) for _ in range(3)]
    lin_t, out = [_t(v, dev) for v in lin], torch.empty((M, head_dim), device=dev)
    scratch = torch.zeros(B.bl_attn_prefill_scratch_bytes(1, head_dim, pos0, M), dtype=torch.uint8, device=dev)
    B.bl_set_tuning("attn_groups", 1000)
    try:
        for _ in range(2):
            B.bl_attn_prefill(*(t.data_ptr() for t in lin_t), table.data_ptr(), k_cache.data_ptr(), v_cache.data_ptr(), out.data_ptr(),
                              scratch.data_ptr(), 1, head_dim, max_pos, pos0, M, torch.cuda.current_stream().cuda_stream)
    finally:
        B.bl_set_tuning("attn_groups", 0)
    torch.cuda.synchronize()
    kc64, vc64 = (c.float().cpu().numpy().astype(np.float64) for c in (k_cache, v_cache))
    for m in range(M):
        want = D.attention_decode(D.rope(lin[0][m], pos0 + m, 1), kc64[:pos0 + m + 1], vc64[:pos0 + m + 1], 1)
        assert np.abs(out[m].cpu().numpy() - want).max() <= 2e-5 * max(1.0, np.abs(want).max())


@pytest.mark.parametrize("n_heads,head_dim,pos0,M", [(2, 8, 31, 33), (2, 24, 0, 32), (2, 32, 127, 65), (3, 72, 128, 1), (2, 80, 96, 64),
                                                     (2, 88, 33, 31), (2, 96, 0, 129), (1, 104, 255, 66), (2, 112, 160, 40), (9, 128, 129, 95)])
def test_attn_prefill_every_head_size_class(dev, mods, n_heads, head_dim, pos0, M):
    """Each instance of the transposed-score kernel that the cases above leave out (head sizes in sixteens, whole and half),
    at the edges of its 32-row chunks, of the four sets that share them out (a set without a chunk, a step with fewer
    chunks than sets) and of its 64-token blocks.  Tolerance: the same derivation as above."""
    test_attn_prefill_parity(dev, mods, n_heads, head_dim, pos0 + M + 3, pos0, M)


def test_prompt_then_tokens(dev, mods):
    """A prompt in two pieces through DecoderStack.prefill (products as bl_gemm over all rows, attention on the matrix
    cores), then single tokens: the caches and hidden states follow those of the same tokens taken one at a time through
    the unfolded one-token path, and the oracle."""
    B, dec, ops = mods
    hidden, ffn, n_heads, n_layers, max_pos = 256, 512, 4, 2, 160
    layers, g_final = _make_layers(67000, hidden, ffn, n_layers)
    a = dec.DecoderStack(_to_device(layers, dev, dec, ops), _t(g_final, dev), n_heads, max_pos, dev, fold_norm=False)
    b = dec.DecoderStack(_to_device(layers, dev, dec, ops), _t(g_final, dev), n_heads, max_pos, dev, fold_norm=False)
    x = torch.randn((103, hidden), device=dev, generator=torch.Generator(device=dev).manual_seed(9))
    ya = torch.cat([a.prefill(x[:70].contiguous()), a.prefill(x[70:100].contiguous())])
    yb = []
    for t in range(103):
        b.h.copy_(x[t:t + 1])
        yb.append(b.step().clone())
        if t >= 100:
            a.h.copy_(x[t:t + 1])
            ya = torch.cat([ya, a.step()])
    torch.cuda.synchronize()
    assert int(a.pos[0]) == 103 == int(b.pos[0])
    yb = torch.cat(yb)
    # the prompt's attention sums in another order than the one-token kernel: the first layer's cache rows are the same
    # bits, everything behind an attention agrees to the bound of the end-to-end comparisons
    assert torch.equal(a.layers[0].attn.k_cache.view(torch.int16), b.layers[0].attn.k_cache.view(torch.int16))
    assert torch.equal(a.layers[0].attn.v_cache.view(torch.int16), b.layers[0].attn.v_cache.view(torch.int16))
    assert float(torch.linalg.norm(ya - yb)) <= 5e-2 * float(torch.linalg.norm(yb))
    assert bool(torch.isfinite(ya).all())
    # the oracle, token by token, on the first tokens
    kcs = [np.zeros((max_pos, hidden)) for _ in layers]
    vcs = [np.zeros((max_pos, hidden)) for _ in layers]
    xs = x.cpu().numpy()
    for t in range(6):
        h = xs[t].astype(np.float64)
        for i, l in enumerate(layers):
            h = D.decoder_layer_step(h, t, l, kcs[i], vcs[i], n_heads)
        want = D.rmsnorm(h, g_final, 1e-5)
        got = ya[t].cpu().numpy().astype(np.float64)
        assert np.linalg.norm(got - want) <= 5e-2 * np.linalg.norm(want)


@pytest.mark.parametrize("n_heads,head_dim,pos0,M", [(3, 64, 351, 33), (3, 64, 352, 33), (2, 128, 990, 33), (1, 72, 500, 1), (2, 96, 0, 400),
                                                     (40, 16, 0, 225), (40, 24, 0, 257), (60, 16, 10, 300), (33, 128, 31, 250)])
def test_attn_prefill_waves_and_block_order(dev, mods, n_heads, head_dim, pos0, M):
    """The matrix-core attention around its rules: four and eight waves per workgroup (384 positions and one more; few and many
    workgroups), blocks of 32 tokens in falling order and in pairs (even and odd numbers of blocks), last blocks of one token.
    Every token against the fp64 softmax over the cache as stored."""
    B, dec, ops = mods
    hidden, max_pos = n_heads * head_dim, pos0 + M
    r = _rng(96000 + hidden + M)
    table = dec.rope_table(head_dim, max_pos, dev)
    g = torch.Generator(device=dev).manual_seed(96000 + hidden)
    k_cache, v_cache = (torch.randn((max_pos, hidden), device=dev, generator=g).to(torch.bfloat16) for _ in range(2))
    lin = [3.0 * r.standard_normal((M, hidden)).astype(np.float32) for _ in range(3)]
    lin_t = [_t(v, dev) for v in lin]
    out = torch.full((M, hidden), float("nan"), device=dev)
    scratch = torch.zeros(B.bl_attn_prefill_scratch_bytes(n_heads, head_dim, pos0, M), dtype=torch.uint8, device=dev)
    B.bl_attn_prefill(lin_t[0].data_ptr(), lin_t[1].data_ptr(), lin_t[2].data_ptr(), table.data_ptr(), k_cache.data_ptr(),
                      v_cache.data_ptr(), out.data_ptr(), scratch.data_ptr(), n_heads, head_dim, max_pos, pos0, M,
                      torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    q = torch.from_numpy(np.stack([D.rope(lin[0][m], pos0 + m, n_heads) for m in range(M)])).view(M, n_heads, head_dim)
    k, v = (c.cpu().double().view(max_pos, n_heads, head_dim) for c in (k_cache, v_cache))
    seen = torch.arange(max_pos)[None] <= torch.arange(pos0, max_pos)[:, None]
    for h in range(n_heads):
        s = (q[:, h].double() @ k[:, h].t()) / head_dim ** 0.5
        want = torch.softmax(s.masked_fill(~seen, -float("inf")), 1) @ v[:, h]
        got = out[:, h * head_dim:(h + 1) * head_dim].cpu().double()
        assert (got - want).abs().max() <= PREFILL_BLOCK_TOL * max(1.0, float(want.abs().max())), h


@pytest.mark.parametrize("n_heads,head_dim,max_pos,pos0,M", [(22, 72, 90, 5, 70), (32, 48, 70, 0, 33), (12, 128, 100, 31, 3), (9, 168, 40, 1, 20)])
def test_attn_prefill_parity_wide_rows(dev, mods, n_heads, head_dim, max_pos, pos0, M):
    """Rows long enough for the append that takes sixteen bytes at a time: head sizes whose quarters are odd numbers of pieces, and one
    beyond the matrix-core attention."""
    test_attn_prefill_parity(dev, mods, n_heads, head_dim, max_pos, pos0, M)


@pytest.mark.parametrize("n_heads,head_dim,max_pos,pos0,M", [(40, 160, 1300, 1250, 3), (150, 136, 330, 326, 3), (2, 132, 4400, 4220, 2), (300, 256, 700, 640, 2),
                                                             (28, 160, 2100, 2000, 4), (13, 164, 3000, 2900, 3), (7, 136, 130, 126, 4)])
def test_attn_prefill_equals_tokens_beyond_one_chunk_per_workgroup(dev, mods, n_heads, head_dim, max_pos, pos0, M):
    """Head sizes above 128 in caches whose chunks outnumber a head's workgroups (12, 3, 64 and 5; 9 and 19 that do not fill rounds of the dies with their heads, and one
    cache of as few chunks as workgroups): a prompt's tokens add up their
    chunks in the one-token call's order, bit for bit."""
    B, dec, ops = mods
    hidden = n_heads * head_dim
    table = dec.rope_table(head_dim, max_pos, dev)
    g = torch.Generator(device=dev).manual_seed(97000 + hidden)
    kc, vc = (torch.randn((max_pos, hidden), device=dev, generator=g).to(torch.bfloat16) for _ in range(2))
    lin = [3.0 * torch.randn((M, hidden), device=dev, generator=g) for _ in range(3)]
    k_cache, v_cache, out = kc.clone(), vc.clone(), torch.empty((M, hidden), device=dev)
    scratch = torch.zeros(B.bl_attn_prefill_scratch_bytes(n_heads, head_dim, pos0, M), dtype=torch.uint8, device=dev)
    one, pos_t = [torch.empty((1, hidden), device=dev) for _ in range(3)], torch.zeros(1, dtype=torch.int32, device=dev)
    att = dec.Attention(n_heads, head_dim, max_pos, *one, pos_t, table)
    att.k_cache.copy_(kc)
    att.v_cache.copy_(vc)
    for _ in range(2):   # twice: the counters in the scratch memory must be back at zero
        B.bl_attn_prefill(*(t.data_ptr() for t in lin), table.data_ptr(), k_cache.data_ptr(), v_cache.data_ptr(), out.data_ptr(),
                          scratch.data_ptr(), n_heads, head_dim, max_pos, pos0, M, torch.cuda.current_stream().cuda_stream)
        for m in range(M):
            for t, v in zip(one, lin):
                t.copy_(v[m:m + 1])
            pos_t.fill_(pos0 + m)
            assert torch.equal(att.launch()[0], out[m]), m
    assert torch.equal(k_cache.view(torch.int16), att.k_cache.view(torch.int16))
    assert not scratch.view(torch.int32).view(M, -1)[:, -n_heads:].any()
