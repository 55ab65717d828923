"""The sizes at which a kernel's tiles, splits and dispatch rules change, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from oracle import fp8_oracle as f8
from helpers import check_fp8_against_model_oracle, f64, max_abs, rmse
from paper_2407_08608_amd import binding, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N", [31, 32, 33, 64, 65, 96, 97, 127, 128, 130, 255, 257, 513, 700])
def test_fp32_tile_and_split_edges(N, causal):
    # 64-row workgroups of two 32-row slabs; four waves of a slab split every 128-key block, so at 31..130 keys
    # some splits see no key at all, or (causal) none that a given row may see
    q = inputs.normal_tensor(300 + N, "q", (1, 6, N, 64), "f32")
    k, v = (inputs.normal_tensor(300 + N, n, (1, 2, N, 64), "f32") for n in ("k", "v"))
    o, lse = binding.fa_fwd_gqa(q.cuda(), k.cuda(), v.cuda(), 0.125, causal)
    o_ref, l_ref = oracle.attention_fwd_gqa(f64(q), f64(k), f64(v), 0.125, causal)
    assert max_abs(f64(o), o_ref) <= 2e-5 and max_abs(f64(lse), l_ref) <= 2e-5  # fp32 sums of at most 700 terms


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("H,H_kv,N", [(1, 1, 1), (3, 3, 2), (6, 2, 7), (4, 1, 16), (9, 9, 31), (10, 5, 32), (700, 700, 9), (5, 5, 33)])
def test_fp32_short_sequences(H, H_kv, N, causal):
    # up to 32 keys a wave does a head by itself, four to a workgroup: head counts that fill it and do not
    q = inputs.normal_tensor(320 + N, "q", (1, H, N, 64), "f32")
    k, v = (inputs.normal_tensor(320 + N, n, (1, H_kv, N, 64), "f32") for n in ("k", "v"))
    o, lse = binding.fa_fwd_gqa(q.cuda(), k.cuda(), v.cuda(), 0.125, causal)
    o_ref, l_ref = oracle.attention_fwd_gqa(f64(q), f64(k), f64(v), 0.125, causal)
    assert max_abs(f64(o), o_ref) <= 1e-5 and max_abs(f64(lse), l_ref) <= 1e-5  # fp32 sums of at most 64 terms


def test_fp32_more_heads_than_one_launch_takes():
    # a launch of 512-thread workgroups takes 2^23 - 1 of them: here a few heads more, of 33 rows (q is zero but for the
    # heads at the seam and at the end, so that L = log(33) and O = mean(V) elsewhere)
    H, N, seam = 2 ** 23 + 5, 33, 2 ** 23 - 1
    if torch.cuda.mem_get_info()[0] < 180 * 2 ** 30:
        pytest.skip("needs 150 GB of device memory")
    q = torch.zeros((1, H, N, 64), device="cuda")
    o, lse = torch.empty_like(q), torch.empty((1, H, N), device="cuda")
    q[:, seam - 2:] = inputs.normal_tensor(340, "q", (1, H - seam + 2, N, 64), "f32").cuda()
    k, v = (inputs.normal_tensor(340, n, (1, 1, N, 64), "f32") for n in ("k", "v"))
    binding.fa_fwd_gqa(q, k.cuda(), v.cuda(), 0.125, False, o=o, lse=lse)
    for h in (slice(0, 2), slice(seam // 2, seam // 2 + 2), slice(seam - 2, H)):
        o_ref, l_ref = oracle.attention_fwd_gqa(f64(q[:, h]), f64(k), f64(v), 0.125, False)
        assert max_abs(f64(o[:, h]), o_ref) <= 2e-5 and max_abs(f64(lse[:, h]), l_ref) <= 2e-5
    del q, o, lse
    torch.cuda.empty_cache()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("N,hidden", [(20, 20), (100, 100), (100, 40), (300, 300), (300, 64)])
def test_fp32_rows_whose_every_score_is_minus_infinity(N, hidden, causal):
    # keys hidden through -inf in one component: a row that sees only such keys has L = -inf (and no output), others
    # are untouched by them
    q = inputs.normal_tensor(330, "q", (1, 2, N, 64), "f32")
    k, v = (inputs.normal_tensor(330, n, (1, 2, N, 64), "f32") for n in ("k", "v"))
    q[..., 0] = 1.0
    k[:, :, :hidden, 0] = -np.inf
    o, lse = (t.cpu().double() for t in binding.fa_fwd(q.cuda(), k.cuda(), v.cuda(), 0.125, causal))
    s = torch.matmul(q.double(), k.double().transpose(-1, -2).contiguous()) * 0.125
    if causal:
        s = s.masked_fill(torch.ones(N, N, dtype=torch.bool).triu(1), -np.inf)
    ref = torch.logsumexp(s, dim=-1)
    seen = torch.isfinite(ref)
    assert (lse[~seen] == -np.inf).all() and torch.isnan(o[~seen]).all()
    assert float(torch.where(seen, lse - ref, 0.0).abs().max()) <= 2e-5
    o_ref = torch.matmul(torch.softmax(s, dim=-1), v.double())
    assert float(torch.where(seen[..., None], o - o_ref, 0.0).abs().max()) <= 2e-5  # fp32 sums of at most 300 terms


@pytest.mark.parametrize("causal", [False, True])
def test_fp32_splits_merge_when_their_maxima_differ(causal):
    # scores rise to 80 nats over the sequence: the splits of a row end with different maxima.  A raw score of up
    # to 640 in sums of 64 terms carries about 8 roundings of 2^-24 * 640, times 1 / 8: 4e-5 relative in P, and
    # |V| reaches 4.
    q, k, v = inputs.rising_maximum_qkv(310, 1, 2, 600, 64, "f32")
    o, lse = binding.fa_fwd(q.cuda(), k.cuda(), v.cuda(), 0.125, causal)
    o_ref, l_ref = oracle.attention_fwd(f64(q), f64(k), f64(v), 0.125, causal)
    assert max_abs(f64(o), o_ref) <= 2e-4 and max_abs(f64(lse), l_ref) <= 2e-4


REL_RMSE, REL_MAXABS = 1e-2, 5e-2  # 2^-9 (bf16) rounding of P, dS and the outputs in sums over the sequence


def _check_backward(seed, B, H, H_kv, N, d, causal, dtype, kv_heads=None):
    # against the oracle: everything, or the key/value heads `kv_heads` and their groups
    q, dout = (inputs.normal_tensor(seed, n, (B, H, N, d), dtype) for n in ("q", "do"))
    k, v = (inputs.normal_tensor(seed, n, (B, H_kv, N, d), dtype) for n in ("k", "v"))
    qg, kg, vg, dog = (t.cuda() for t in (q, k, v, dout))
    o, lse = binding.fa_fwd_gqa(qg, kg, vg, d ** -0.5, causal)
    got = binding.fa_bwd_gqa(qg, kg, vg, o, lse, dog, d ** -0.5, causal)
    torch.cuda.synchronize()
    for h in [slice(0, H_kv)] if kv_heads is None else [slice(i, i + 1) for i in kv_heads]:
        group = slice(h.start * (H // H_kv), h.stop * (H // H_kv))
        ref = oracle.attention_bwd_gqa(f64(q[:, group]), f64(k[:, h]), f64(v[:, h]), f64(dout[:, group]), d ** -0.5, causal)
        for name, t in zip(("dq", "dk", "dv"), got):
            g, r = f64(t[:, group if name == "dq" else h]), ref[name]
            assert np.isfinite(g).all(), name
            # the floors: with one visible key dS = P (dP - D) is exactly 0 and what is left are the roundings of two fp32
            # sums of d products (2^-24 * sqrt(d) * |dO| |V| ~ 2e-6), times |K| * scale
            ref_rms = float(np.sqrt(np.mean(r * r)))
            assert rmse(g, r) <= REL_RMSE * ref_rms + 1e-5 and max_abs(g, r) <= REL_MAXABS * np.abs(r).max() + 1e-4, name


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,N,H", [(128, 2, 1200), (128, 33, 300), (128, 63, 300), (128, 65, 260), (128, 127, 220), (128, 128, 220), (128, 129, 160),
                                   (128, 191, 150), (128, 321, 110)] + [(256, n, 4) for n in (2, 31, 32, 63, 64, 65, 127, 129, 321)])
def test_backward_shared_score_tiles(d, N, H, causal, dtype):
    # key blocks of 128 (64 at d = 256) in 32-key tiles, query tiles of 64 in two sub-tiles whose P and dS the waves
    # exchange; an odd and an even number of query tiles, and two query heads per K/V head walking the ring twice.  At
    # d = 128 with so many heads that the pass takes these tiles
    _check_backward(500 + N, 1, H, H // 2, N, d, causal, dtype, None if N < 100 or d == 256 else (0, H // 2 - 1))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("H,H_kv,N", [(1, 1, 1), (2, 2, 31), (2, 1, 33), (4, 1, 64), (3, 3, 97), (8, 2, 129), (1, 1, 130),
                                      (4, 2, 333), (2, 2, 1025)])
@pytest.mark.parametrize("d", [64, 128])
def test_backward_query_split_for_few_key_blocks(d, H, H_kv, N, causal, dtype):
    # 32-key workgroups whose four waves take every fourth 32-query tile of the group's heads: fewer tiles than waves,
    # ragged last tiles of queries and of keys, tile numbers that carry over to the next query head
    _check_backward(700 + N + d, 1, H, H_kv, N, d, causal, dtype)


def _check_both_sides(seed, d, causal, N, group, most, dtype):
    # the most key/value heads that take one form of the backward, and one more, which take another
    for H_kv in (most, most + 1):
        _check_backward(seed + H_kv, 1, H_kv * group, H_kv, N, d, causal, dtype, None if N < 100 else (0, H_kv - 1))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,causal,N,group,most", [(64, False, 40, 4, 144), (64, True, 40, 2, 156), (128, False, 30, 2, 228), (128, True, 40, 1, 127)])
def test_backward_on_both_sides_of_the_key_split_rule(d, causal, N, group, most, dtype):
    # the dK/dV pass in its 32-key form by itself, and large
    _check_both_sides(800, d, causal, N, group, most, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,causal,N,group,H_kv", [(64, False, 333, 8, 23), (64, True, 513, 16, 27), (128, False, 333, 8, 17), (128, True, 513, 8, 17)])
def test_backward_32_key_workgroups_by_themselves(d, causal, N, group, H_kv, dtype):
    # behind the large dQ pass, over more tiles than a wave keeps in its stages, ragged
    _check_backward(880 + N, 1, H_kv * group, H_kv, N, d, causal, dtype, (0, H_kv - 1))


@pytest.mark.parametrize("d,causal,N,group,most", [(64, False, 70, 1, 75), (64, False, 70, 4, 17), (64, False, 70, 8, 9), (64, True, 70, 1, 54),
                                                   (64, True, 97, 4, 1), (64, True, 170, 8, 1), (128, False, 70, 1, 42), (128, False, 70, 4, 1),
                                                   (128, False, 170, 8, 1), (128, True, 70, 1, 39), (128, True, 97, 4, 1), (128, True, 170, 8, 1)])
def test_backward_on_both_sides_of_the_rule_of_128_queries(d, causal, N, group, most):
    # one launch with the dQ work in 32-query workgroups, and in 128-query ones ahead of the key blocks and behind them
    _check_both_sides(900, d, causal, N, group, most, "f16")


@pytest.mark.parametrize("d,causal,N,most", [(64, False, 40, 172), (64, False, 70, 144), (64, True, 40, 181), (64, True, 70, 204),
                                             (128, False, 30, 192), (128, False, 70, 128), (128, True, 40, 105), (128, True, 70, 132)])
def test_backward_on_both_sides_of_the_one_launch_rule(d, causal, N, most):
    # one launch, and two
    _check_both_sides(850, d, causal, N, 1, most, "bf16")


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,H", [(64, 2), (64, 300), (128, 2), (128, 300), (256, 2)])
def test_backward_with_a_very_low_logsumexp(d, H, causal):
    # scores near -140 (-200 in log2 units) everywhere: exp2 of a padding key's zero score against such an L overflows, and
    # must not reach dQ through the zero rows past N (N = 70 leaves 26 of them).  Few and many workgroups.
    N = 70
    q, k, v = (inputs.normal_tensor(950, n, (1, H, N, d), "f32") for n in ("q", "k", "v"))
    q, k = q * 0.1 + 10.0, k * 0.1 - 14.0 / d ** 0.5
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    dout = inputs.normal_tensor(951, "do", (1, H, N, d), "bf16")
    o, lse = binding.fa_fwd(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
    assert float(lse.max()) < -100.0
    got = binding.fa_bwd(q.cuda(), k.cuda(), v.cuda(), o, lse, dout.cuda(), d ** -0.5, causal)
    assert all(torch.isfinite(t).all() for t in got)
    for h in (0, H - 1):
        # K and Q are nearly constant over the rows, so dQ and dK are small differences of large sums and each element
        # gets the bound of its own sum: P, dS and the outputs are rounded to 2^-9 (2^-8 leaves as much again for the
        # fp32 scores of up to 2^12, whose roundings move P by less than 2^-10), and D carries the rounding of O
        q64, k64, v64, do64 = (f64(t[0, h]) for t in (q, k, v, dout))
        s = q64 @ k64.T * d ** -0.5
        if causal:
            s = np.where(np.tri(N, dtype=bool), s, -np.inf)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        p /= p.sum(axis=1, keepdims=True)
        out = p @ v64
        ds = p * (do64 @ v64.T - (do64 * out).sum(axis=1, keepdims=True))
        d_err = p * (np.abs(do64) * np.abs(out)).sum(axis=1, keepdims=True)
        dp_err = p * (np.abs(do64) @ np.abs(v64).T)
        ds_err = 2.0 ** -8 * (np.abs(ds) + d_err) + 2.0 ** -10 * dp_err
        for g, ref, err in ((got[0], ds @ k64 * d ** -0.5, ds_err @ np.abs(k64) * d ** -0.5),
                            (got[1], ds.T @ q64 * d ** -0.5, ds_err.T @ np.abs(q64) * d ** -0.5),
                            (got[2], p.T @ do64, 2.0 ** -8 * p.T @ np.abs(do64))):
            assert (np.abs(f64(g[0, h]) - ref) <= err + 2.0 ** -8 * np.abs(ref)).all()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,N", [(64, 127), (64, 129), (64, 290), (128, 33), (128, 128), (128, 130), (128, 260)])
def test_backward_four_wave_query_tiles(d, N, causal):
    # enough heads that neither pass takes its few-workgroup form: 128-query tiles with 32-key blocks, ragged in both
    _check_backward(960 + N, 2, 200, 100, N, d, causal, "bf16")


@pytest.mark.parametrize("d,causal,N", [(64, True, 3072), (64, True, 3073), (128, True, 1536), (128, True, 1537), (64, False, 1280),
                                        (128, False, 1281)])
def test_backward_query_tile_rule_edges(d, causal, N):
    # on both sides of the length up to which the 128-query tiles are used, with more heads than the few-workgroup forms
    # take (one of them against the oracle)
    _check_backward(990, 1, 32, 32, N, d, causal, "bf16", (5,))


@pytest.mark.parametrize("heads,N,d", [(64, 1500, 128), (128, 1500, 128), (512, 100, 128), (384, 200, 128), (100, 300, 128),
                                       (7, 1409, 128), (256, 129, 256), (300, 300, 256), (5, 700, 256), (9, 1300, 64),
                                       (11, 200, 64), (3, 2048, 64), (3, 2049, 64), (3, 1664, 128), (3, 1665, 128), (5, 1408, 128), (5, 1536, 128), (5, 1537, 128),
                                       (61, 1700, 128), (62, 1700, 128), (255, 300, 128), (256, 300, 128), (127, 300, 256),
                                       (128, 300, 256), (359, 512, 64), (360, 512, 64), (10, 4100, 64), (11, 4100, 64), (250, 300, 256), (10, 4100, 256), (11, 4100, 256),
                                       (64, 2048, 128), (65, 2048, 128), (51, 2300, 128), (64, 2300, 128), (19, 6400, 64), (16, 6400, 64), (24, 4100, 256)])
@pytest.mark.parametrize("fp8", [False, True])
def test_causal_forward_paired_and_single_tiles(heads, N, d, fp8):
    # head counts on both sides of the rule that pairs causal query tiles, with odd and even tile counts (few heads of a long
    # sequence are divided by keys instead); every row of the first, a middle and the last head against the oracle
    pick = sorted({0, heads // 2, heads - 1})
    q = inputs.normal_tensor(1000 + N, "q", (1, heads, N, d), "bf16")
    k, v = (inputs.normal_tensor(1000 + N, n, (1, 1, N, d), "bf16") for n in ("k", "v"))
    if fp8:
        dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (q, k, v)]
        o, lse = binding.fa_fwd_fp8_gqa(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, True)
        codes = [[a.cpu().numpy() for a in p] for p in dev]
        for h in pick:
            (qc, qs), kc, vc = codes[0], codes[1], codes[2]
            check_fp8_against_model_oracle(o[:, h:h + 1], lse[:, h:h + 1], (qc[:, h:h + 1], kc[0], vc[0]),
                                           (qs[:, h:h + 1], kc[1], vc[1]), d ** -0.5, True, kv_heads=1)
        return
    o, lse = binding.fa_fwd_gqa(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, True)
    for h in pick:
        o_ref, l_ref = oracle.attention_fwd(f64(q[:, h:h + 1]), f64(k), f64(v), d ** -0.5, True)
        assert max_abs(f64(o[:, h:h + 1]), o_ref) <= 2e-2 and rmse(f64(o[:, h:h + 1]), o_ref) <= 3e-3
        assert max_abs(f64(lse[:, h:h + 1]), l_ref) <= 2e-3


@pytest.mark.parametrize("d,causal,N,group,most", [(64, False, 70, 8, 59), (64, False, 70, 2, 136), (64, True, 70, 4, 156), (64, True, 70, 2, 186),
                                                   (128, False, 70, 4, 73), (128, False, 70, 2, 102), (128, True, 70, 3, 78), (128, True, 70, 2, 112)])
def test_backward_both_passes_in_one_launch(d, causal, N, group, most):
    # shared heads on both sides of the rule that lets both passes share a launch: beyond it large, or the dK/dV pass alone in
    # its 32-key form
    _check_both_sides(1100, d, causal, N, group, most, "bf16")


@pytest.mark.parametrize("d,N", [(64, 511), (64, 512), (64, 640), (64, 641), (64, 769), (64, 768), (64, 1408), (64, 1409), (128, 640),
                                 (128, 641), (128, 704), (128, 705), (128, 897), (128, 1152), (128, 1153)])
@pytest.mark.parametrize("fp8", [False, True])
def test_forward_tile_rule_edges(d, N, fp8):
    # where the unmasked forward changes between 128- and 256-row workgroups, and odd and even numbers of 128-row tiles, with
    # two heads: all but d = 128 with FP8 to 128 keys are divided by keys (with many heads: test_forward_main_loops)
    q, k, v = inputs.qkv(1200 + N, 1, 2, N, d, "bf16")
    if fp8:
        dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (q, k, v)]
        o, lse = binding.fa_fwd_fp8(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, False)
        codes = [[a.cpu().numpy() for a in p] for p in dev]
        check_fp8_against_model_oracle(o, lse, [c[0] for c in codes], [c[1] for c in codes], d ** -0.5, False)
        return
    o, lse = binding.fa_fwd(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, False)
    o_ref, l_ref = oracle.attention_fwd(f64(q), f64(k), f64(v), d ** -0.5, False)
    assert max_abs(f64(o), o_ref) <= 2e-2 and rmse(f64(o), o_ref) <= 3e-3 and max_abs(f64(lse), l_ref) <= 2e-3


@pytest.mark.parametrize("over", ["q", "dout"])
@pytest.mark.parametrize("d,H,N,causal", [(64, 2, 100, True), (128, 2, 300, False), (128, 200, 140, True), (256, 4, 200, True),
                                          (64, 200, 140, False)])
def test_backward_writes_dq_over_an_input(d, H, N, causal, over):
    # the calls that reuse Q's or dO's memory for dQ: every form of the two passes, against separate buffers (D is summed
    # in another order there: at most a rounding of the outputs apart)
    q, k, v, dout = (inputs.normal_tensor(1300 + N, n, (1, H, N, d), "bf16").cuda() for n in ("q", "k", "v", "do"))
    o, lse = binding.fa_fwd(q, k, v, d ** -0.5, causal)
    ref = binding.fa_bwd(q, k, v, o, lse, dout, d ** -0.5, causal)
    t = {"q": q.clone(), "dout": dout.clone()}
    got = binding.fa_bwd(t["q"], k, v, o, lse, t["dout"], d ** -0.5, causal, dq=t[over])
    for a, b in zip(got, ref):
        assert rmse(f64(a), f64(b)) <= 2.0 ** -9 * float(np.sqrt(np.mean(f64(b) ** 2)))


# (d, H, H_kv, N, causal) for every form of the two passes: one launch that computes D for itself and one behind the row sums, with
# 32-query workgroups and with 128-query ones ahead of the key blocks and behind them, the dK/dV pass alone in its 32-key form, large
# with 128- and 256-query tiles, d = 256
_FORMS = [(64, 2, 2, 333, False), (128, 2, 2, 100, True), (64, 2, 2, 1000, True), (128, 2, 2, 300, False), (64, 100, 100, 70, False), (128, 60, 60, 70, True),
          (64, 88, 88, 170, True), (128, 12, 12, 2000, False), (64, 16, 2, 511, False), (128, 24, 3, 288, False), (64, 520, 65, 70, False),
          (128, 284, 71, 70, True), (64, 400, 400, 140, False), (128, 200, 200, 140, True), (64, 30, 30, 1400, False), (128, 32, 32, 1537, True),
          (256, 4, 4, 200, True), (256, 40, 40, 300, False)]


def _forms_inputs(seed, d, H, H_kv, N, causal):
    q, dout = (inputs.normal_tensor(seed + N, n, (1, H, N, d), "bf16").cuda() for n in ("q", "do"))
    k, v = (inputs.normal_tensor(seed + N, n, (1, H_kv, N, d), "bf16").cuda() for n in ("k", "v"))
    o, lse = binding.fa_fwd_gqa(q, k, v, d ** -0.5, causal)
    return q, k, v, o, lse, dout


@pytest.mark.parametrize("over", ["dq", "dk", "dv", "dq one head on", "dk one head on"])
@pytest.mark.parametrize("d,H,H_kv,N,causal", _FORMS)
def test_backward_writes_a_gradient_over_the_output(d, H, H_kv, N, causal, over):
    # O is not needed once D is known, so a caller may hand its memory to a gradient, also shifted against O by a head:
    # against separate buffers (D may be summed in another order: at most a rounding of the outputs apart)
    q, k, v, o, lse, dout = _forms_inputs(1500, d, H, H_kv, N, causal)
    ref = binding.fa_bwd_gqa(q, k, v, o, lse, dout, d ** -0.5, causal)
    pool = torch.empty((1, H + 1, N, d), device="cuda", dtype=torch.bfloat16)
    pool[:, :H] = o
    first, heads = int("head" in over), H if over.startswith("dq") else H_kv
    out = {over.split()[0]: pool[:, first:first + heads]}
    got = binding.fa_bwd_gqa(q, k, v, pool[:, :H], lse, dout, d ** -0.5, causal, **out)
    for a, b in zip(got, ref):
        assert rmse(f64(a), f64(b)) <= 2.0 ** -9 * float(np.sqrt(np.mean(f64(b) ** 2)))


@pytest.mark.parametrize("dq_over", ["q", "dout"])
@pytest.mark.parametrize("d,H,H_kv,N,causal", _FORMS)
def test_backward_writes_dq_over_an_input_and_dv_over_the_output(d, H, H_kv, N, causal, dq_over):
    # dV replaces O before dQ, which goes over an input of the dK/dV pass, is computed
    q, k, v, o, lse, dout = _forms_inputs(1520, d, H, H_kv, N, causal)
    ref = binding.fa_bwd_gqa(q, k, v, o, lse, dout, d ** -0.5, causal)
    got = binding.fa_bwd_gqa(q, k, v, o, lse, dout, d ** -0.5, causal, dq=q if dq_over == "q" else dout, dv=o[:, :H_kv])
    for a, b in zip(got, ref):
        assert rmse(f64(a), f64(b)) <= 2.0 ** -9 * float(np.sqrt(np.mean(f64(b) ** 2)))


@pytest.mark.parametrize("H,H_kv,N", [(4, 2, 100), (8, 2, 700), (260, 65, 140)])
def test_backward_writes_shared_head_gradients_inside_the_output(H, H_kv, N):
    # dK and dV of shared heads are smaller than O: both fit into it, dV behind dK
    q, dout = (inputs.normal_tensor(1550 + N, n, (1, H, N, 64), "f16").cuda() for n in ("q", "do"))
    k, v = (inputs.normal_tensor(1550 + N, n, (1, H_kv, N, 64), "f16").cuda() for n in ("k", "v"))
    o, lse = binding.fa_fwd_gqa(q, k, v, 0.125, True)
    ref = binding.fa_bwd_gqa(q, k, v, o, lse, dout, 0.125, True)
    got = binding.fa_bwd_gqa(q, k, v, o, lse, dout, 0.125, True, dk=o[:, :H_kv], dv=o[:, H_kv:2 * H_kv])
    for a, b in zip(got, ref):
        assert rmse(f64(a), f64(b)) <= 2.0 ** -12 * float(np.sqrt(np.mean(f64(b) ** 2)))


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,N,H,H_kv", [(64, 512, 2, 2), (64, 513, 2, 2), (64, 128, 8, 2), (64, 129, 8, 2), (128, 192, 2, 2),
                                        (128, 193, 2, 2), (128, 96, 4, 2), (128, 97, 4, 2), (128, 3, 2, 1), (64, 70, 128, 128),
                                        (64, 70, 129, 129), (128, 70, 64, 64), (128, 70, 65, 65)])
def test_backward_row_sums_inside_the_one_launch(d, N, H, H_kv, causal):
    # on both sides of the numbers of tiles and of workgroups up to which the one launch computes D for itself, ragged and not
    _check_backward(1400 + N, 1, H, H_kv, N, d, causal, "bf16")


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("H,H_kv,N", [(1, 1, 65), (3, 1, 96), (8, 2, 97), (2, 2, 129), (5, 5, 255), (6, 3, 333), (16, 4, 641), (3, 3, 1025),
                                      (4, 1, 1409), (2, 2, 2100), (12, 12, 1056)])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_forward_with_the_keys_split_over_the_waves(d, H, H_kv, N, causal, dtype):
    # 32-query workgroups of four and eight waves: as many tiles as waves, fewer, ragged last tiles of keys and of queries,
    # and every way the tiles of a head are dealt to the XCDs (heads a multiple of 8, 4, 2 or odd, short and long)
    q = inputs.normal_tensor(1600 + N, "q", (1, H, N, d), dtype)
    k, v = (inputs.normal_tensor(1600 + N, n, (1, H_kv, N, d), dtype) for n in ("k", "v"))
    o, lse = binding.fa_fwd_gqa(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
    o_ref, l_ref = oracle.attention_fwd_gqa(f64(q), f64(k), f64(v), d ** -0.5, causal)
    assert max_abs(f64(o), o_ref) <= 2e-2 and rmse(f64(o), o_ref) <= 3e-3 and max_abs(f64(lse), l_ref) <= 2e-3


@pytest.mark.parametrize("d,causal,N,most", [(64, False, 100, 69), (64, False, 100, 80), (64, True, 100, 97), (64, False, 1024, 26),
                                             (128, False, 100, 64), (128, False, 256, 56), (128, True, 512, 33), (128, False, 2048, 12),
                                             (256, False, 300, 25), (256, True, 1024, 12)])
def test_forward_on_both_sides_of_the_key_split_rule(d, causal, N, most):
    # the most heads (a multiple of 8 or not) that are divided so, and the next ones that are not: the same rows
    # either way, against the oracle and, as P~ is rounded relative to different references, to one another
    q = inputs.normal_tensor(1700 + N, "q", (1, most + 16, N, d), "bf16")
    k, v = (inputs.normal_tensor(1700 + N, n, (1, 1, N, d), "bf16") for n in ("k", "v"))
    o_ref, l_ref = oracle.attention_fwd(f64(q[:, :1]), f64(k), f64(v), d ** -0.5, causal)
    for H in (most, most + 1, most + 16):
        o, lse = binding.fa_fwd_gqa(q[:, :H].contiguous().cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
        assert max_abs(f64(o[:, :1]), o_ref) <= 2e-2 and rmse(f64(o[:, :1]), o_ref) <= 3e-3
        assert max_abs(f64(lse[:, :1]), l_ref) <= 2e-3


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("d,N", [(64, 600), (128, 600), (128, 1500), (256, 600)])
def test_forward_key_splits_merge_when_their_references_differ(d, N, causal):
    # every row's maximum rises over the sequence by 80 nats, so the waves of a workgroup end with different references and
    # raise them in most tiles; a raw score s of up to 80 sqrt(d) is a sum of d fp32 products, error below 2^-20 s scale in
    # the exponent, and the outputs carry the 16-bit roundings of P~ and O
    q, k, v = inputs.rising_maximum_qkv(1800, 1, 2, N, d, "bf16")
    o, lse = binding.fa_fwd(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
    o_ref, l_ref = oracle.attention_fwd(f64(q), f64(k), f64(v), d ** -0.5, causal)
    assert max_abs(f64(o), o_ref) <= 2e-2 + 2.0 ** -8 * np.abs(o_ref).max() and max_abs(f64(lse), l_ref) <= 2e-3


@pytest.mark.parametrize("d", [64, 128, 256])
def test_forward_key_splits_with_scores_of_minus_infinity(d):
    # keys hidden through -inf in one component of K: waves whose tiles hold nothing else add nothing to a row
    N, hidden = 300, 200
    q, k, v = inputs.qkv(1810, 1, 2, N, d, "bf16")
    q[..., 0] = 1.0
    k[:, :, :hidden, 0] = -np.inf
    o, lse = binding.fa_fwd(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, False)
    k[..., 0] = torch.where(torch.isinf(k[..., 0]), torch.zeros_like(k[..., 0]), k[..., 0])
    s = q.double() @ k.double().transpose(-1, -2).contiguous() * d ** -0.5
    s[..., :hidden] = -np.inf
    assert max_abs(f64(lse), torch.logsumexp(s, -1).numpy()) <= 2e-3
    assert max_abs(f64(o), (torch.softmax(s, -1) @ v.double()).numpy()) <= 2e-2


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("H,H_kv,N", [(1, 1, 65), (3, 1, 127), (8, 2, 129), (2, 2, 160), (5, 5, 255), (6, 3, 333), (16, 4, 641), (3, 3, 1025),
                                      (4, 1, 1409), (2, 2, 2100)])
@pytest.mark.parametrize("d", [64, 128, 256])
def test_fp8_forward_with_the_keys_split_over_the_waves(d, H, H_kv, N, causal):
    # 32-query workgroups of four and eight waves over 64-key tiles: fewer tiles than waves and more, ragged last tiles of keys
    # and of queries, tiles that share a 128-row scale block, every way the tiles of a head are dealt to the XCDs
    q = inputs.normal_tensor(1900 + N, "q", (1, H, N, d), "bf16")
    k, v = (inputs.normal_tensor(1900 + N, n, (1, H_kv, N, d), "bf16") for n in ("k", "v"))
    v[:, :, N // 2:] *= 30.0  # block scales that differ between the splits
    dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (q, k, v)]
    o, lse = binding.fa_fwd_fp8_gqa(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, causal)
    codes = [[a.cpu().numpy() for a in p] for p in dev]
    check_fp8_against_model_oracle(o, lse, [c[0] for c in codes], [c[1] for c in codes], d ** -0.5, causal, kv_heads=H_kv)


@pytest.mark.parametrize("d,causal,N,most", [(64, False, 256, 57), (64, True, 512, 57), (64, False, 1024, 32), (128, False, 256, 56), (128, True, 512, 30),
                                             (128, False, 2048, 16), (256, False, 300, 44), (256, True, 1024, 21)])
def test_fp8_forward_on_both_sides_of_the_key_split_rule(d, causal, N, most):
    # the most heads (a multiple of 8 or not) that are divided so, and the next ones that are not: the first head against the oracle
    q = inputs.normal_tensor(1950 + N, "q", (1, most + 16, N, d), "bf16")
    k, v = (inputs.normal_tensor(1950 + N, n, (1, 1, N, d), "bf16") for n in ("k", "v"))
    for H in (most, most + 1, most + 16):
        dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (q[:, :H].contiguous(), k, v)]
        o, lse = binding.fa_fwd_fp8_gqa(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, causal)
        (qc, qs), kc, vc = [[a.cpu().numpy() for a in p] for p in dev]
        check_fp8_against_model_oracle(o[:, :1], lse[:, :1], (qc[:, :1], kc[0], vc[0]), (qs[:, :1], kc[1], vc[1]), d ** -0.5, causal, kv_heads=1)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("d,N,H", [(64, 1, 1300), (64, 63, 1300), (64, 65, 1300), (64, 128, 600), (64, 129, 600), (64, 321, 300), (64, 641, 300),
                                   (128, 1, 1300), (128, 64, 1300), (128, 127, 1300), (128, 193, 600), (128, 256, 600), (128, 577, 300)])
def test_forward_shared_tiles(d, N, H, rising, causal):
    # many heads, so 128 or 256 queries a workgroup: one key block, the second stage, an odd and an even number of blocks
    # before a causal pair's second tile, ragged last blocks of keys and of queries; with rising maxima a block's scores
    # are computed a second time, from either stage of K, while the next tiles arrive
    dtype = "f16" if H == 600 else "bf16"
    pick = [0, H // 2, H - 1]
    q, k, v = inputs.rising_maximum_qkv(1900 + N, 1, 1, N, d, dtype) if rising else inputs.qkv(1900 + N, 1, 1, N, d, dtype)
    o_ref, l_ref = oracle.attention_fwd(f64(q), f64(k), f64(v), d ** -0.5, causal)
    o, lse = binding.fa_fwd_gqa(q.expand(1, H, N, d).contiguous().cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
    assert torch.equal(o, o[:, :1].expand_as(o)) and torch.equal(lse, lse[:, :1].expand_as(lse))  # every head alike
    for h in pick:
        assert max_abs(f64(o[:, h:h + 1]), o_ref) <= 2e-2 + (2.0 ** -8 * np.abs(o_ref).max() if rising else 0)  # roundings of P~ and O
        assert max_abs(f64(lse[:, h:h + 1]), l_ref) <= 2e-3


@pytest.mark.parametrize("d,causal,N,heads", [(64, False, 700, (8, 16)), (64, True, 2049, (8, 16)), (64, True, 3000, (5, 6, 7)), (64, True, 6144, (2, 8)),
                                              (64, True, 6145, (2,)), (64, False, 897, (16,)), (128, False, 700, (8, 16)), (128, True, 1409, (4, 12)),
                                              (128, True, 1920, (3, 16)), (128, True, 1921, (3,)), (128, False, 897, (4,))])
def test_forward_key_splits_of_four_and_eight_waves(d, causal, N, heads):
    # head counts on both sides of the rule that gives the key-split workgroups of the four-wave kernels eight waves, and
    # both sides of the lines between the kernels
    q = inputs.normal_tensor(1960 + N, "q", (1, max(heads), N, d), "bf16")
    k, v = (inputs.normal_tensor(1960 + N, n, (1, 1, N, d), "bf16") for n in ("k", "v"))
    o_ref, l_ref = oracle.attention_fwd(f64(q[:, :1]), f64(k), f64(v), d ** -0.5, causal)
    for H in heads:
        o, lse = binding.fa_fwd_gqa(q[:, :H].contiguous().cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
        assert max_abs(f64(o[:, :1]), o_ref) <= 2e-2 and rmse(f64(o[:, :1]), o_ref) <= 3e-3
        assert max_abs(f64(lse[:, :1]), l_ref) <= 2e-3


@pytest.mark.parametrize("d,causal,N,H", [(64, False, 700, 85), (64, False, 129, 333), (128, False, 300, 61), (128, False, 700, 67), (64, True, 957, 107),
                                          (64, True, 2100, 41), (128, True, 1024, 83), (128, True, 300, 94), (64, True, 512, 381),
                                          (128, True, 512, 255), (128, True, 650, 420)])
def test_forward_tiles_of_a_head_on_one_xcd(d, causal, N, H):
    # heads and work items that are no multiple of 8, without a mask, as single causal tiles and as pairs: every tile of every
    # head is done (the outputs start as NaN), and by itself (every head has the same rows)
    q, k, v = inputs.qkv(2000 + N, 1, 1, N, d, "bf16")
    o_ref, l_ref = oracle.attention_fwd(f64(q), f64(k), f64(v), d ** -0.5, causal)
    o = torch.full((1, H, N, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((1, H, N), float("nan"), device="cuda")
    binding.fa_fwd_gqa(q.expand(1, H, N, d).contiguous().cuda(), k.cuda(), v.cuda(), d ** -0.5, causal, o=o, lse=lse)
    assert torch.equal(o, o[:, :1].expand_as(o)) and torch.equal(lse, lse[:, :1].expand_as(lse))
    assert max_abs(f64(o[:, :1]), o_ref) <= 2e-2 and rmse(f64(o[:, :1]), o_ref) <= 3e-3 and max_abs(f64(lse[:, :1]), l_ref) <= 2e-3


# (fp8, d, causal, N, heads, kernel): enough heads that no key split is made, so that the kernel's own loop runs; checked
# against the rules on the CPU in test_division_host.py
MAIN_LOOPS = ([(False, 128, False, N, 24, "fa_fwd_pingpong_kernel") for N in (897, 1024, 1031, 1100, 1152, 1153, 1345, 2049)] +
              [(False, 128, True, N, H, "fa_fwd_pingpong_kernel") for N, H in ((1921, 24), (4096, 16), (4129, 16), (4200, 17))] +
              [(False, 64, False, N, 48, "fa_fwd_16bit_kernel<bf16_tag, 64, 64, 8,") for N in (897, 1031, 1408, 1409)] +
              [(False, 64, True, N, H, "fa_fwd_16bit_kernel<bf16_tag, 64, 64, 8,") for N, H in ((6145, 16), (6273, 19), (6400, 19))] +
              [(False, 64, False, N, 48, "fa_fwd_16bit_kernel<bf16_tag, 64, 64, 4,") for N in (640, 641, 768, 769, 896)] +
              [(False, 128, False, N, 48, "fa_fwd_16bit_kernel<bf16_tag, 128, 64, 4,") for N in (640, 641, 704, 705, 896)] +
              [(False, 64, True, 6144, 16, "fa_fwd_16bit_kernel<bf16_tag, 64, 64, 4,"),
               (False, 128, True, 1920, 24, "fa_fwd_16bit_kernel<bf16_tag, 128, 64, 4,")] +
              [(False, 256, False, N, H, "fa_fwd_d256_kernel") for N, H in ((65, 200), (300, 60), (1000, 24), (1031, 24), (2049, 16))] +
              [(False, 256, True, N, H, "fa_fwd_d256_kernel") for N, H in ((300, 60), (1031, 24), (2100, 24))] +
              [(True, 64, False, N, H, "fa_fwd_fp8_kernel<64, 64, 4,") for N, H in ((130, 130), (511, 64))] +
              [(True, 64, False, N, 48, "fa_fwd_fp8_async_kernel<64,") for N in (512, 641, 1409)] +
              [(True, 128, False, N, 48, "fa_fwd_fp8_kernel<128, 64, 4,") for N in (640, 704)] +
              [(True, 128, False, N, 48, "fa_fwd_fp8_async_kernel<128,") for N in (705, 897, 1153)] +
              [(True, 256, False, N, H, "fa_fwd_fp8_async_kernel<256,") for N, H in ((300, 64), (700, 48), (1031, 48))] +
              [(True, 64, True, N, H, "fa_fwd_fp8_kernel<64, 64, 4,") for N, H in ((700, 65), (2500, 64))] +
              [(True, 128, True, 1000, 48, "fa_fwd_fp8_kernel<128, 64, 4,"), (True, 128, True, 2000, 25, "fa_fwd_fp8_async_kernel<128,"),
               (True, 256, True, 700, 48, "fa_fwd_fp8_async_kernel<256,")])


@pytest.mark.parametrize("rising", [False, True])
@pytest.mark.parametrize("fp8,d,causal,N,H", [c[:5] for c in MAIN_LOOPS])
def test_forward_main_loops(fp8, d, causal, N, H, rising):
    # every kernel's own loop on both sides of the lengths between the kernels: whole and ragged tiles and key blocks, odd and
    # even numbers of tiles, the causal diagonal; with rising maxima the references move in every block of a row, one block
    # behind the scores in the pipelined kernels.  Every head has the same rows.
    q, k, v = inputs.rising_maximum_qkv(2100 + N, 1, 1, N, d, "bf16") if rising else inputs.qkv(2100 + N, 1, 1, N, d, "bf16")
    many = q.expand(1, H, N, d).contiguous()
    if fp8:
        dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (many, k, v)]
        o, lse = binding.fa_fwd_fp8_gqa(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, causal)
        (qc, qs), kc, vc = [[a.cpu().numpy() for a in p] for p in dev]
        check_fp8_against_model_oracle(o[:, :1], lse[:, :1], (qc[:, :1], kc[0], vc[0]), (qs[:, :1], kc[1], vc[1]), d ** -0.5, causal, kv_heads=1)
    else:
        o, lse = binding.fa_fwd_gqa(many.cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
        o_ref, l_ref = oracle.attention_fwd(f64(q), f64(k), f64(v), d ** -0.5, causal)
        # (rising: scores of up to 80 nats are sums of d fp32 products, and few keys carry a row: the roundings of P~ and O)
        assert max_abs(f64(o[:, :1]), o_ref) <= 2e-2 + (2.0 ** -8 * np.abs(o_ref).max() if rising else 0)
        assert rmse(f64(o[:, :1]), o_ref) <= (6e-3 if rising else 3e-3) and max_abs(f64(lse[:, :1]), l_ref) <= 2e-3
    assert torch.equal(o, o[:, :1].expand_as(o)) and torch.equal(lse, lse[:, :1].expand_as(lse))


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("d,causal,N,H", [c[1:5] for c in MAIN_LOOPS if c[0]])
def test_fp8_main_loops_with_and_without_scales(d, causal, N, H, scaled):
    # block scales of V and K that jump up and down from block to block, by factors on both sides of the lazy-raise threshold,
    # with an all-zero V block (scale 1) among them; and the instantiations that take the codes at unit scale
    if scaled:
        q, k, v = inputs.qkv(2300 + N, 1, 1, N, d, "bf16")
        for t, f in enumerate([1.0, 64.0, 0.02, 0.0, 3.0, 1.5, 0.001, 200.0] * (N // 1024 + 1)):
            v[:, :, t * 128:(t + 1) * 128] *= f
            k[:, :, t * 128:(t + 1) * 128] *= 0.25 * (1 + t % 4)
        dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (q.expand(1, H, N, d).contiguous(), k, v)]
        o, lse = binding.fa_fwd_fp8_gqa(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, causal)
        (qc, qs), (kc, ks), (vc, vs) = [[a.cpu().numpy() for a in p] for p in dev]
    else:
        rng = np.random.default_rng(2300 + N + d)
        qc, kc, vc = (f8.e4m3_encode(rng.standard_normal((1, 1, N, d))) for _ in range(3))
        qs = ks = vs = np.ones((1, 1, -(-N // 128)), dtype=np.float32)
        dev = [torch.from_numpy(c).cuda() for c in (qc, kc, vc)]
        o, lse = binding.fa_fwd_gqa(dev[0].expand(1, H, N, d).contiguous(), *dev[1:], d ** -0.5, causal, dtype=binding.FA_FP8_E4M3)
    check_fp8_against_model_oracle(o[:, :1], lse[:, :1], (qc[:, :1], kc, vc), (qs[:, :1], ks, vs), d ** -0.5, causal)
    assert torch.equal(o, o[:, :1].expand_as(o)) and torch.equal(lse, lse[:, :1].expand_as(lse))


# (fp8, d, causal, N, B, H, H_kv): shared heads in the kernels' own loops
SHARED_HEADS = [(False, 64, False, 700, 2, 24, 6), (False, 64, False, 1031, 2, 24, 8), (False, 64, True, 700, 3, 32, 4), (False, 128, False, 300, 2, 33, 11),
                (False, 128, False, 1100, 2, 16, 4), (False, 128, True, 1000, 2, 32, 8), (False, 128, True, 2300, 2, 16, 2), (False, 256, False, 600, 2, 24, 6),
                (False, 256, True, 600, 2, 24, 3), (True, 64, False, 700, 2, 32, 8), (True, 64, True, 700, 3, 32, 4), (True, 128, False, 600, 2, 32, 8),
                (True, 128, False, 1100, 2, 24, 6), (True, 128, True, 2000, 2, 16, 2), (True, 256, False, 700, 2, 24, 6)]


@pytest.mark.parametrize("fp8,d,causal,N,B,H,H_kv", SHARED_HEADS)
def test_main_loops_with_shared_heads(fp8, d, causal, N, B, H, H_kv):
    # the first and the last group of every batch against the oracle
    q = inputs.normal_tensor(2400 + N, "q", (B, H, N, d), "bf16")
    k, v = (inputs.normal_tensor(2400 + N, n, (B, H_kv, N, d), "bf16") for n in ("k", "v"))
    n = H // H_kv
    groups = [(b, g) for b in (0, B - 1) for g in (0, H_kv - 1)]
    if fp8:
        dev = [binding.fa_fp8_quant_hadamard(t.cuda()) for t in (q, k, v)]
        o, lse = binding.fa_fwd_fp8_gqa(*(p[0] for p in dev), *(p[1] for p in dev), d ** -0.5, causal)
        (qc, qs), kc, vc = [[a.cpu().numpy() for a in p] for p in dev]
        for b, g in groups:
            of, kv = (slice(b, b + 1), slice(g * n, g * n + n)), (slice(b, b + 1), slice(g, g + 1))
            check_fp8_against_model_oracle(o[of], lse[of], (qc[of], kc[0][kv], vc[0][kv]), (qs[of], kc[1][kv], vc[1][kv]), d ** -0.5, causal, kv_heads=1)
        return
    o, lse = binding.fa_fwd_gqa(q.cuda(), k.cuda(), v.cuda(), d ** -0.5, causal)
    for b, g in groups:
        of, kv = (slice(b, b + 1), slice(g * n, g * n + n)), (slice(b, b + 1), slice(g, g + 1))
        o_ref, l_ref = oracle.attention_fwd_gqa(f64(q[of]), f64(k[kv]), f64(v[kv]), d ** -0.5, causal)
        assert max_abs(f64(o[of]), o_ref) <= 2e-2 and rmse(f64(o[of]), o_ref) <= 3e-3 and max_abs(f64(lse[of]), l_ref) <= 2e-3


def _bits(t):
    return t.view(torch.int16 if t.dtype != torch.float32 else torch.int32)


# (dtype, d, N, heads): key splits of four and eight waves, the 128- and 256-row loops, d = 256, both fp32 kernels, FP8
_FORMS_FWD = [("bf16", 64, 300, 2), ("f16", 64, 700, 2), ("bf16", 128, 300, 2), ("bf16", 128, 1500, 2), ("bf16", 256, 300, 2), ("f16", 64, 300, 300),
              ("bf16", 128, 300, 200), ("f16", 128, 2300, 24), ("bf16", 64, 1500, 48), ("bf16", 256, 300, 60), ("f32", 64, 20, 3), ("f32", 64, 300, 3),
              ("fp8", 64, 300, 2), ("fp8", 64, 300, 120), ("fp8", 64, 700, 60), ("fp8", 128, 300, 2), ("fp8", 128, 300, 100), ("fp8", 128, 1500, 24),
              ("fp8", 256, 300, 2), ("fp8", 256, 300, 64)]


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("dtype,d,N,H", _FORMS_FWD)
def test_forward_rows_with_scores_of_nan_or_infinity(dtype, d, N, H, causal):
    # a NaN in a query's row, or a key whose score is NaN or +inf for the rows that see it: those rows have no output and no
    # logsumexp (inf - inf in the softmax), every other row keeps its bits
    q = inputs.normal_tensor(2200 + N, "q", (1, H, N, d), "bf16" if dtype == "fp8" else dtype).cuda()
    k, v = (inputs.normal_tensor(2200 + N, n, (1, 1, N, d), "bf16" if dtype == "fp8" else dtype).cuda() for n in ("k", "v"))
    q[..., 0] = 1.0
    if dtype == "fp8":
        (q, qs), (k, ks), (v, vs) = (binding.fa_fp8_quant_hadamard(t) for t in (q, k, v))
        run = lambda q, k: binding.fa_fwd_fp8_gqa(q, k, v, qs, ks, vs, d ** -0.5, causal)  # noqa: E731
        nan, kinds = 0x7F, ("nan",)  # (e4m3 has no infinity)
    else:
        run = lambda q, k: binding.fa_fwd_gqa(q, k, v, d ** -0.5, causal)  # noqa: E731
        nan, kinds = float("nan"), ("nan", "inf")
    o, lse = run(q, k)
    assert torch.isfinite(o).all() and torch.isfinite(lse).all()

    def check(o2, l2, hit):
        assert torch.isnan(o2[hit]).all() and not torch.isfinite(l2[hit]).any()
        assert torch.equal(_bits(o2[~hit]), _bits(o[~hit])) and torch.equal(_bits(l2[~hit]), _bits(lse[~hit]))

    for i in (0, N // 2, N - 1):
        q2, hit = q.clone(), torch.zeros((1, H, N), dtype=torch.bool, device="cuda")
        q2[:, ::2, i, 5], hit[:, ::2, i] = nan, True
        check(*run(q2, k), hit)
    for j in (0, 40 % N, N - 1):
        for kind in kinds:
            k2, hit = k.clone(), torch.zeros((1, H, N), dtype=torch.bool, device="cuda")
            k2[:, :, j, 0], hit[:, :, j if causal else 0:] = nan if kind == "nan" else float("inf"), True
            check(*run(q, k2), hit)


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("d,causal,N,H,H_kv", [(128, True, 129, 30, 30), (128, True, 256, 32, 32), (128, False, 160, 32, 32), (128, False, 97, 60, 60),
                                               (64, True, 257, 56, 56), (64, False, 385, 40, 20), (64, False, 160, 64, 64), (64, False, 159, 110, 55),
                                               (128, True, 161, 48, 6), (128, False, 288, 24, 3), (64, True, 193, 32, 8), (64, True, 193, 48, 6), (64, False, 511, 16, 2)])
def test_backward_128_query_workgroups_beside_key_blocks(d, causal, N, H, H_kv, dtype):
    # one launch whose dQ work has 128 queries to a workgroup, ahead of the key blocks (groups up to four) and behind them: a
    # last workgroup of one row, of one and of four waves, fewer tiles than are staged ahead, ragged last tiles, waves that end up to
    # three tiles before the others; (64, False, 160, 64): D computed in this launch
    _check_backward(2500 + N, 1, H, H_kv, N, d, causal, dtype, (0, H_kv - 1))
