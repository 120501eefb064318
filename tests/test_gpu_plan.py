"""The attention's work plan at the edges of its rules: a unit cut into more
than 32 parts, cost-ordered items over more than one plan workgroup, and more
units than the plan keeps costs of in LDS. The plan only decides where and when
a part runs, so without splits an output equals that of any other call that
holds the sequence, bit for bit, and with planned splits it equals the unsplit
one within the output tolerance (parts are merged by their log-sum-exp)."""
import numpy as np
import pytest
import torch

import paper_2608_19758_amd as fp2
import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


def _attend(wl, mask, splits):
    d = gu.device_tensors(wl)
    p = gu.params_for(wl, 0.5, kv_splits=splits)
    out, lse = fp2.attend(p, d["q"], d["k_cache"], d["v_cache"], d["cu_seqlens"],
                          torch.from_numpy(mask).cuda(), d["block_table"],
                          cu_seqlens_host=wl.cu_seqlens, q_scale=d["q_scale"],
                          k_scale=d["k_scale"], v_scale=d["v_scale"], want_lse=True,
                          **gu.kv_args(wl, d))
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), lse.cpu().numpy()


# Planned against unsplit outputs, beside the largest difference: every part
# rounds its probabilities against its own reference, and a rounding to p bits of
# mantissa is uniform within 2^-(p+1) of the power of two below, 0.41 * 2^-p of the
# value in the mean square (e4m3, p = 3: 0.0255, two of them 0.036; bf16, p = 7:
# 0.0016 and 0.0023, as much again for the outputs' own rounding). The relative
# gates of the parity tests lie just above: 0.04 and 0.005.
def _same_within_rounding(o0, l0, o1, l1, dtype):
    rel = np.linalg.norm(o0 - o1) / np.linalg.norm(o1)
    print("planned against unsplit: out %.3g, relative %.3g, lse %.3g"
          % (np.abs(o0 - o1).max(), rel, np.abs(l0 - l1).max()))
    assert np.isfinite(o1).all() and np.abs(o1).max() > 0
    assert np.abs(o0 - o1).max() <= gu.TOL[dtype] and rel <= gu.REL_GATE[dtype]
    assert np.abs(l0 - l1).max() <= gu.LSE_TOL[dtype]


# (new tokens, prefix, query heads, KV heads): one tail block whose dense head
# takes 644 steps (more parts than the lanes of a half-wave; fp8 41, of 16 steps), and
# 1028 steps (64 parts, the most, of 17 steps, where the smallest budget asks for
# more); 1280 units in two plan workgroups
@pytest.mark.parametrize("n,prefix,hq,hkv", [(128, 40960, 8, 2), (128, 65536, 8, 2),
                                             (20480, 0, 16, 8)])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_one_dense_head(dtype, n, prefix, hq, hkv):
    print("case", dtype, n, prefix, hq, hkv, flush=True)
    wl = synth.generate(synth.Spec("plan", [n], hq, hkv, dtype=dtype, page_size=64, seed=5,
                                   prefix=[prefix] if prefix else None))
    nq, nk = (n + 127) // 128, (n + prefix + 127) // 128
    last = prefix // 128 + np.arange(nq)[:, None]
    j = np.arange(nk)[None, :]
    mask = np.zeros((1, hkv, nq, nk), np.uint8)
    mask[0] = (j == 0) | ((j <= last) & (j > last - 2))
    mask[0, 1] = j <= last                        # the dense head
    _same_within_rounding(*_attend(wl, mask, 0), *_attend(wl, mask, 1), dtype)


# the same among 34056 units, past the 32768 whose costs the plan keeps: 33
# sequences bounded by the longest, whose dense head weighs up to 260 steps where a
# workgroup's share is some 100, so that units are cut and put in order of cost
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_parts_among_more_units_than_cached_costs(dtype):
    print("case", dtype, flush=True)
    lens, hq, hkv = [16500] + [40] * 32, 16, 8
    wl = synth.generate(synth.Spec("plan_many", lens, hq, hkv, dtype=dtype, page_size=64, seed=13))
    i = np.arange(129)
    mask = np.zeros((33, hkv, 129, 129), np.uint8)
    mask[1:, :, 0, 0] = 1
    mask[0] = (i[None, :] == 0) | ((i[None, :] <= i[:, None]) & (i[None, :] > i[:, None] - 2))
    mask[0, 1] = i[None, :] <= i[:, None]         # the dense head
    _same_within_rounding(*_attend(wl, mask, 0), *_attend(wl, mask, 1), dtype)


# a call whose entries leave half of the workgroups idle takes each as two items
# of 128 rows, one bounded by many more units as one of 256: g = 2, 4 and 8, the
# last query block partial, at most 3 key blocks so that neither call splits a
# unit (the default plan)
@pytest.mark.parametrize("hq,hkv", [(4, 2), (4, 1), (8, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("n", [130, 380])
def test_few_units_take_narrow_items(dtype, hq, hkv, n):
    print("case", dtype, hq, hkv, n, flush=True)
    wl = synth.generate(synth.Spec("plan_few", [n], hq, hkv, dtype=dtype, page_size=64, seed=8))
    p = gu.params_for(wl, 0.0, score_splits=1)
    out, mask, lse = gu.gpu_prefill(wl, p)
    d = gu.device_tensors(wl)
    b = 512 // hkv
    cu = np.minimum(np.arange(b + 1), 1).astype(np.int32) * n
    p.batch = b
    table = d["block_table"].repeat(b, 1).contiguous()
    o, m, l = fp2.prefill(p, d["q"], d["k_cache"], d["v_cache"], torch.from_numpy(cu).cuda(), table,
                          cu_seqlens_host=cu, q_scale=d["q_scale"], k_scale=d["k_scale"],
                          v_scale=d["v_scale"], want_lse=True)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(m.cpu().numpy()[:1], mask)
    np.testing.assert_array_equal(o.float().cpu().numpy(), out)
    np.testing.assert_array_equal(l.cpu().numpy(), lse)


# rows taken as the two halves of an entry (a call whose entries leave half of the
# workgroups idle) and as whole entries (one bounded by more units) give the same
# numbers, with and without parts: g = 2, 4 and 8, the last query block partial,
# a prefix that is not a multiple of the block, pruned blocks corrected
@pytest.mark.parametrize("hq,hkv", [(4, 2), (4, 1), (8, 1)])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("splits", [1, 3])
def test_half_entries(dtype, hq, hkv, splits):
    print("case", dtype, hq, hkv, splits, flush=True)
    wl = synth.generate(synth.Spec("plan_half", [200], hq, hkv, dtype=dtype, page_size=64, seed=12,
                                   prefix=[1100]))
    p = gu.params_for(wl, 0.97, kv_splits=splits, score_splits=1)
    d = gu.device_tensors(wl)
    out, mask, lse = gu.gpu_prefill(wl, p, d)
    b = 264 // hkv
    p.batch = b
    first = np.minimum(np.arange(b + 1), 1).astype(np.int32)
    cu, cuk = first * 200, first * 1300
    o, m, l = fp2.prefill(p, d["q"], d["k_cache"], d["v_cache"], torch.from_numpy(cu).cuda(),
                          d["block_table"].repeat(b, 1).contiguous(), cu_seqlens_host=cu,
                          cu_seqlens_k=torch.from_numpy(cuk).cuda(), cu_seqlens_k_host=cuk,
                          q_scale=d["q_scale"], k_scale=d["k_scale"], v_scale=d["v_scale"],
                          want_lse=True)
    torch.cuda.synchronize()
    assert 0 < (mask & 1).sum() < mask.size
    np.testing.assert_array_equal(m.cpu().numpy()[:1], mask)
    np.testing.assert_array_equal(o.float().cpu().numpy(), out)
    np.testing.assert_array_equal(l.cpu().numpy(), lse)


# a few tokens whose unit keeps all of its key blocks and takes 2 * blocks + 2
# steps: whole up to the smallest budget (16 steps; 8 in bf16 for calls of so few
# entries), then in ceil(steps / budget) parts, and with the same numbers as under
# that fixed count of parts. fp8 units are not cut finer: each cut rounds the
# probabilities anew.
@pytest.mark.parametrize("hq,hkv", [(8, 2), (32, 8), (16, 16)])
@pytest.mark.parametrize("dtype,budget", [("bf16", 8), ("fp8", 16)])
@pytest.mark.parametrize("blocks", [3, 4, 7, 8, 15, 16])
def test_parts_of_a_short_extend(dtype, budget, hq, hkv, blocks):
    print("case", dtype, hq, hkv, blocks, flush=True)
    wl = synth.generate(synth.Spec("plan_extend", [18], hq, hkv, dtype=dtype, page_size=64, seed=11,
                                   prefix=[128 * blocks - 40]))
    d = gu.device_tensors(wl)
    parts = -(-(2 * blocks + 2) // budget)
    o0, m0, l0 = gu.gpu_prefill(wl, gu.params_for(wl, 0.0), d)
    o1, m1, l1 = gu.gpu_prefill(wl, gu.params_for(wl, 0.0, kv_splits=parts), d)
    assert (m0 & 1).sum() == hkv * blocks and np.isfinite(o0).all()
    np.testing.assert_array_equal(m0, m1)
    np.testing.assert_array_equal(o0, o1)
    np.testing.assert_array_equal(l0, l1)


# sequences of 3, 7 and 8 key blocks that keep them all, in calls of few and of
# many entries: on both sides of the bounds (8 and 16 steps, two a block and two
# an entry) below which no unit can be split and no merge is launched
@pytest.mark.parametrize("heads", [1, 32])
@pytest.mark.parametrize("n", [384, 896, 1024])
def test_no_merge_below_the_smallest_budget(heads, n):
    print("case", heads, n, flush=True)
    wl = synth.generate(synth.Spec("plan_short", [n], heads, heads, page_size=0, seed=9))
    d = gu.device_tensors(wl)
    o0, m0, l0 = gu.gpu_prefill(wl, gu.params_for(wl, 0.0), d)
    o1, m1, l1 = gu.gpu_prefill(wl, gu.params_for(wl, 0.0, kv_splits=1), d)
    np.testing.assert_array_equal(m0, m1)
    assert np.isfinite(o0).all() and np.abs(o0 - o1).max() <= gu.TOL["bf16"]
    assert np.abs(l0 - l1).max() <= gu.LSE_TOL["bf16"]


def test_more_units_than_cached_costs():
    """33 sequences bounded by 16500 tokens and 8 KV heads make 34056 units (the
    plan keeps 32768 costs): the rows of the longest and of a short sequence
    equal those of calls that hold it alone."""
    lens = [16500] + [40] * 32
    wl = synth.generate(synth.Spec("plan_many", lens, 8, 8, page_size=0, seed=6))
    alpha = 0.99
    out, _, lse = gu.gpu_prefill(wl, gu.params_for(wl, alpha, kv_splits=1, score_splits=1))
    d = gu.device_tensors(wl)
    for b in (0, 32):
        r0, r1 = int(wl.cu_seqlens[b]), int(wl.cu_seqlens[b + 1])
        cu = np.array([0, r1 - r0], np.int32)
        p = fp2.make_params(batch=1, num_q_heads=8, num_kv_heads=8, max_seq_len=r1 - r0, alpha=alpha,
                            sink_blocks=1, window_blocks=2, kv_splits=1, score_splits=1)
        o, _, l = fp2.prefill(p, d["q"][r0:r1].contiguous(), d["k_cache"][r0:r1].contiguous(),
                              d["v_cache"][r0:r1].contiguous(), torch.from_numpy(cu).cuda(),
                              cu_seqlens_host=cu, want_lse=True)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(o.float().cpu().numpy(), out[r0:r1])
        np.testing.assert_array_equal(l.cpu().numpy(), lse[r0:r1])
