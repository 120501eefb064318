"""GPU tests of the block-means cache (fp2_prefill_cached): a chunked prefill
that keeps the pooled means of complete blocks between its calls.

A sequence is prefilled in two calls over one paged KV pool: the first chunk
(positions [0, P)), then the rest with P tokens of prefix. The cache starts
poisoned (NaN bf16 everywhere); the first call pools every block it sees and
writes it to its slot, the second copies the P // 128 complete blocks and
pools the rest. Bars: the second call's mask, outputs and LSE equal those of
fp2_prefill without a cache bit for bit; the cache then holds, in every block's
slot, exactly the means fp2_pool computes over the whole sequence; a
pooled_blocks beyond the complete blocks is clamped (same results again).
"""
import numpy as np
import pytest
import torch

import paper_2608_19758_amd as fp2
import synth
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

B = 128
NAN_BF16 = 0x7FC0


def spec(lens, page, hq=8, hkv=2, dtype="bf16", seed=31):
    pool = sum((L + page - 1) // page for L in lens) + 9
    return synth.Spec("meanscache", list(lens), hq, hkv, dtype=dtype, page_size=page,
                      page_order="permuted", pool_pages=pool, salient_frac=0.1, salient_min=2,
                      sink_blocks=1, window_blocks=2, recent_blocks=0, mean_correction=1,
                      seed=seed)


def slot(wl, b, J):
    """The documented slot of key block J of sequence b."""
    p = wl.spec.page_size
    t = J * B
    return int(wl.block_table[b][t // p]) * ((p + B - 1) // B) + (t % p) // B


def call(wl, d, rows, kv_lens, q_lens, alpha, cache=None, pooled=None):
    """fp2_prefill(_cached) for the query rows `rows` (per sequence, a slice of
    that sequence's positions) against the first kv_lens[b] tokens of the pool."""
    sp = wl.spec
    cu_q = np.concatenate([[0], np.cumsum(q_lens)]).astype(np.int32)
    cu_k = np.concatenate([[0], np.cumsum(kv_lens)]).astype(np.int32)
    q = torch.cat([d["q"][int(wl.cu_seqlens[b]) + r.start:int(wl.cu_seqlens[b]) + r.stop]
                   for b, r in enumerate(rows)])
    p = fp2.make_params(batch=sp.batch, num_q_heads=sp.num_q_heads, num_kv_heads=sp.num_kv_heads,
                        max_seq_len=max(q_lens), page_size=sp.page_size,
                        max_pages_per_seq=wl.max_pages, alpha=alpha,
                        sink_blocks=sp.sink_blocks, window_blocks=sp.window_blocks,
                        recent_blocks=sp.recent_blocks, mean_correction=1, dtype=sp.dtype,
                        max_kv_len=max(kv_lens))
    mc = None
    if cache is not None:
        mc = (cache[0], cache[1], torch.tensor(pooled, dtype=torch.int32, device="cuda"))
    out, mask, lse = fp2.prefill(p, q, d["k_cache"], d["v_cache"], torch.from_numpy(cu_q).cuda(),
                                 d["block_table"], cu_seqlens_host=cu_q,
                                 cu_seqlens_k=torch.from_numpy(cu_k).cuda(), cu_seqlens_k_host=cu_k,
                                 q_scale=d["q_scale"], k_scale=d["k_scale"], v_scale=d["v_scale"],
                                 want_lse=True, means_cache=mc)
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), mask.cpu().numpy(), lse.cpu().numpy()


CASES = [
    dict(lens=[1500, 700], cut=[640, 300], page=64, dtype="bf16"),
    dict(lens=[1300], cut=[1024], page=16, dtype="fp8"),
    dict(lens=[900, 1800], cut=[129, 1], page=200, dtype="bf16"),
    dict(lens=[2000, 333], cut=[1000, 128], page=128, dtype="fp8"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "p%d_%s_%s" % (c["page"], c["dtype"],
                                                                      "_".join(map(str, c["cut"]))))
def test_chunked_with_means_cache(case):
    print("means-cache case", case, flush=True)
    lens, cut = case["lens"], case["cut"]
    wl = synth.generate(spec(lens, case["page"], dtype=case["dtype"]))
    d = gu.device_tensors(wl)
    sp = wl.spec
    alpha = 0.98
    pnum = int(wl.num_pages)
    slots = fp2.means_cache_slots(gu.params_for(wl, alpha), pnum)
    assert slots == pnum * ((sp.page_size + B - 1) // B)
    kh = torch.full((slots, sp.num_kv_heads, 128), 0, dtype=torch.int16, device="cuda")
    kh.fill_(NAN_BF16)
    vb = kh.clone()
    cache = (kh.view(torch.bfloat16), vb.view(torch.bfloat16))
    # first chunk: positions [0, cut), KV = the same tokens; nothing cached yet
    r1 = [range(0, c) for c in cut]
    call(wl, d, r1, cut, cut, alpha, cache, [0] * len(lens))
    # second chunk with and without the cache
    r2 = [range(c, L) for c, L in zip(cut, lens)]
    q2 = [L - c for c, L in zip(cut, lens)]
    want = call(wl, d, r2, lens, q2, alpha)
    got = call(wl, d, r2, lens, q2, alpha, cache, [c // B for c in cut])
    for a, g in zip(want, got):
        np.testing.assert_array_equal(a, g)
    # the cache now holds the means of every block of the whole sequences
    p = gu.params_for(wl, alpha)
    khat, vbar = fp2.pool(p, d["k_cache"], d["v_cache"], d["cu_seqlens"], d["block_table"],
                          cu_seqlens_host=wl.cu_seqlens, k_scale=d["k_scale"],
                          v_scale=d["v_scale"])
    torch.cuda.synchronize()
    khat = khat.view(torch.int16).cpu().numpy()
    vbar = vbar.view(torch.int16).cpu().numpy()
    khc, vbc = kh.cpu().numpy(), vb.cpu().numpy()
    for b, L in enumerate(lens):
        for J in range((L + B - 1) // B):
            s = slot(wl, b, J)
            np.testing.assert_array_equal(khc[s], khat[b, :, J])
            np.testing.assert_array_equal(vbc[s], vbar[b, :, J])
    # pooled_blocks past the complete blocks is clamped
    again = call(wl, d, r2, lens, q2, alpha, cache, [10 ** 6] * len(lens))
    for a, g in zip(want, again):
        np.testing.assert_array_equal(a, g)


# cached blocks around the copy group of 16, and far more uncached blocks than
# the call's new tokens could make; a short and a long sequence
@pytest.mark.parametrize("held", [0, 3, 15, 16, 17])
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
def test_short_extend_with_partly_filled_cache(dtype, held):
    print("partly filled", dtype, held, flush=True)
    lens, q_lens = [2300, 130], [60, 2]
    wl = synth.generate(spec(lens, 64, dtype=dtype, seed=32))
    d = gu.device_tensors(wl)
    alpha = 0.98
    slots = fp2.means_cache_slots(gu.params_for(wl, alpha), int(wl.num_pages))
    kh = torch.full((slots, 2, 128), NAN_BF16, dtype=torch.int16, device="cuda")
    cache = (kh.view(torch.bfloat16), kh.clone().view(torch.bfloat16))
    rows = [range(L - q, L) for L, q in zip(lens, q_lens)]
    want = call(wl, d, rows, lens, q_lens, alpha)
    call(wl, d, rows, lens, q_lens, alpha, cache, [0, 0])    # fills every slot
    for b in range(2):                                       # and the slots from `held` on are lost
        for J in range(held, (lens[b] + B - 1) // B):
            cache[0].view(torch.int16)[slot(wl, b, J)] = NAN_BF16
            cache[1].view(torch.int16)[slot(wl, b, J)] = NAN_BF16
    got = call(wl, d, rows, lens, q_lens, alpha, cache, [held, held])
    for a, g in zip(want, got):
        np.testing.assert_array_equal(a, g)


# more sequences than a wave has lanes, each with another share of its blocks in
# the cache: none, some, all, more than it has
@pytest.mark.parametrize("dtype", ["bf16", "fp8"])
@pytest.mark.parametrize("batch", [5, 64, 65, 130])
def test_batch_of_partly_cached_sequences(dtype, batch):
    print("partly cached batch", dtype, batch, flush=True)
    rng = np.random.RandomState(batch)
    lens = [int(x) for x in rng.randint(1, 700, batch)]
    lens[batch // 2] = 5000
    q_lens = [min(L, int(x)) for L, x in zip(lens, rng.randint(1, 90, batch))]
    held = [int(rng.randint(0, L // B + 2)) for L in lens]
    wl = synth.generate(spec(lens, 64, dtype=dtype, seed=33))
    d = gu.device_tensors(wl)
    alpha = 0.98
    slots = fp2.means_cache_slots(gu.params_for(wl, alpha), int(wl.num_pages))
    kh = torch.full((slots, 2, 128), NAN_BF16, dtype=torch.int16, device="cuda")
    cache = (kh.view(torch.bfloat16), kh.clone().view(torch.bfloat16))
    rows = [range(L - q, L) for L, q in zip(lens, q_lens)]
    want = call(wl, d, rows, lens, q_lens, alpha)
    call(wl, d, rows, lens, q_lens, alpha, cache, [0] * batch)
    full = [c.view(torch.int16).clone() for c in cache]
    for b in range(batch):                       # the slots from `held` on are lost
        lost = [slot(wl, b, J) for J in range(min(held[b], lens[b] // B), (lens[b] + B - 1) // B)]
        for c in cache:
            c.view(torch.int16)[lost] = NAN_BF16
    got = call(wl, d, rows, lens, q_lens, alpha, cache, held)
    for a, g in zip(want, got):
        np.testing.assert_array_equal(a, g)
    for c, f in zip(cache, full):
        assert torch.equal(c.view(torch.int16), f)


def test_a_cache_without_the_prefix_costs_no_more_than_none():
    """A token after 57K: with a cache that holds nothing yet the call pools the
    prefix as fast as one without a cache (an eighth of the chip took 14 times
    as long)."""
    from paper_2608_19758_amd import serving
    pre, page = 57343, 64
    pages = (pre + 1 + page - 1) // page
    be = serving.PrefillBackend(serving.BackendConfig(
        num_q_heads=32, num_kv_heads=8, page_size=page, max_batch=1, max_extend_len=1,
        max_kv_len=pre + 1, alpha=0.98))
    table = torch.arange(pages, dtype=torch.int32).view(1, -1).cuda()
    kv = torch.randn((pages * page, 8, 128), device="cuda").bfloat16()
    q = torch.randn((1, 32, 128), device="cuda").bfloat16()
    meta = be.init_forward_metadata([1], [pre], table, cached_prefix_lens=[0])
    means = be.alloc_means_cache(pages)

    def median_us(**kw):
        ts = []
        for _ in range(21):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            be.forward_extend(q, kv, kv, meta, **kw)
            b.record()
            torch.cuda.synchronize()
            ts.append(a.elapsed_time(b) * 1e3)
        return sorted(ts)[10]

    median_us()
    none, empty = median_us(), median_us(means_cache=means)
    print("no cache %.0f us, empty cache %.0f us" % (none, empty), flush=True)
    assert empty <= 3 * none
