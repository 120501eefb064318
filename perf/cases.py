"""The calls whose speed this library is measured by: listed ones, and a draw
of more of the same ranges.

Every case is one layer's attention call as a serving engine or a model makes
it, through the public entry points, on inputs resident in HBM. Inputs have
the structure of the synthetic workloads in ``synth/``: N(0, 1) queries, keys
and values, a direction per KV head added to the keys of a few salient blocks
and to the queries of every other block, bf16 or e4m3 codes with per-head
scales, K/V in a paged pool. They are made on the GPU.
"""
import math
import random

import numpy as np
import torch

import paper_2608_19758_amd as fp2
from paper_2608_19758_amd import serving

D = 128          # head dimension
B = 128          # selection block

# threshold alpha for an expected share of kept causal blocks on these inputs
# (long sequences; the forced blocks come on top in short ones)
_ALPHA_OF = [(0.0086, 0.9935), (0.0163, 0.9877), (0.042, 0.9793), (0.09, 0.9724), (0.17, 0.9700),
             (0.60, 0.9500)]


def _case(name, op, lens, **kw):
    c = dict(name=name, op=op, lens=lens, prefix="", hq=32, hkv=8, dtype="bf16", page=64,
             permuted=False, alpha=0.97, kept=0.17, sink=1, window=2, corr=True, tile=0,
             cached=False, lse=False, salient=0.01)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: one 2K sequence of a small layer, contiguous K/V;
        # launches and latency count
        _case("prompt_2k", "prefill", "2048", hq=4, hkv=1, page=0, alpha=0.991371465, kept=0.30,
              window=1, salient=0.19),
        # a short prompt of an 8B-sized layer at the engine's forced set, most
        # blocks kept; odd length
        _case("prompt_4k_dense", "prefill", "4003", alpha=0.95, kept=0.62, sink=2, window=4),
        # the ordinary long prompt: 32K in bf16, paged
        _case("prompt_32k", "prefill", "32768", alpha=0.970053076, kept=0.163),
        # the long-context layer in fp8
        _case("prompt_128k_fp8", "prefill", "131072", dtype="fp8", alpha=0.979329735, kept=0.042),
        # a continuous batch of fresh prompts of uneven length on a scattered
        # page pool, with the log-sum-exp a context-parallel merge needs
        _case("ragged_batch_8", "prefill", "12840,7399,30893,18608,17958,23275,40237,4986",
              permuted=True, alpha=0.970228848, kept=0.174, lse=True),
        # twice the query heads, very sparse: the selection stage and the mean
        # correction weigh most here
        _case("wide_128k_fp8", "prefill", "131072", hq=64, dtype="fp8", alpha=0.99268689,
              kept=0.0089, salient=0.005),
        # one chunk of a chunked prefill through the serving backend, block
        # means of the prefix cached by the chunks before
        _case("chunk_8k_at_56k", "extend", "8192", prefix="57344", alpha=0.972, kept=0.10,
              cached=True),
        # the last few tokens of a long fp8 prompt (prefix-cache hit): latency
        _case("tail_128_at_128k_fp8", "extend", "128", prefix="130944", dtype="fp8",
              alpha=0.979329735, kept=0.042, cached=True),
        # four requests at different stages in one forward, ragged, fp8
        _case("mixed_extends_fp8", "extend", "8192,8192,4096,1000", prefix="0,32768,90112,130048",
              dtype="fp8", permuted=True, alpha=0.979329735, kept=0.05, cached=True),
        # selection per 128 packed rows instead of per query block
        _case("tiles_32k_fp8", "prefill", "32768", dtype="fp8", tile=128, alpha=0.975, kept=0.09),
        # attention under a caller's own mask: multi-head layer (no grouping),
        # pages of 16 tokens, correction on
        _case("own_mask_16k_mha", "attend", "16001", hq=16, hkv=16, page=16, permuted=True,
              alpha=0.0, kept=0.15, lse=True),
        # the selection alone, as an engine calls it to reuse the mask over
        # several layers
        _case("select_64k", "estimate", "65536", alpha=0.972, kept=0.10),
    ]


def _lens(text):
    return [int(x) for x in text.split(",")] if text else []


def _shape(case):
    lens = _lens(case["lens"])
    pre = _lens(case["prefix"]) or [0] * len(lens)
    return lens, pre, [p + n for p, n in zip(pre, lens)]


def _alpha_for(kept):
    """Threshold for an expected share of kept blocks (log-linear between the
    calibrated points)."""
    x = math.log(kept)
    for (k0, a0), (k1, a1) in zip(_ALPHA_OF, _ALPHA_OF[1:]):
        if x <= math.log(k1):
            t = (x - math.log(k0)) / (math.log(k1) - math.log(k0))
            return round(a0 + t * (a1 - a0), 6)
    return _ALPHA_OF[-1][1]


def _between(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; half of them odd sizes,
    half multiples of 128 where that is possible."""
    n = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    return max(128, n // 128 * 128) if rng.random() < 0.5 and n >= 128 else n


def _cost(case):
    """Score-and-value products of the kept blocks in units of bf16 work."""
    lens, pre, kv = _shape(case)
    pairs = sum(n * (p + n / 2.0) for n, p in zip(lens, pre))
    nb = max(1.0, sum(kv) / len(kv) / B)
    kept = min(1.0, case["kept"] + 2.0 * (case["sink"] + case["window"]) / nb + 1.0 / B)
    return case["hq"] * pairs * kept * (0.5 if case["dtype"] == "fp8" else 1.0)


def draw(rng):
    """One more call of the ranges above. Its attention work stays below half
    of the largest listed case's."""
    most = 0.5 * max(_cost(c) for c in listed())
    while True:
        op = rng.choices(["prefill", "extend", "attend", "estimate"], [5, 4, 2, 1])[0]
        hq, hkv = rng.choice([(32, 8), (32, 8), (32, 8), (64, 8), (32, 4), (16, 8), (16, 16), (4, 1)])
        dtype = rng.choice(["bf16", "fp8"])
        kept = math.exp(rng.uniform(math.log(0.01), math.log(0.3)))
        kw = dict(hq=hq, hkv=hkv, dtype=dtype, page=rng.choice([64, 64, 64, 16, 128]),
                  permuted=rng.random() < 0.5, kept=round(kept, 4), alpha=_alpha_for(kept),
                  corr=rng.random() < 0.85, lse=rng.random() < 0.25)
        if rng.random() < 0.4:
            kw.update(sink=2, window=4)
        if op == "extend":
            n = rng.choice([1, 1, 2, 4])
            lens = [_between(rng, 16, 8192) for _ in range(n)]
            pre = [_between(rng, 64, 122880) for _ in range(n)]
            kw.update(prefix=",".join(map(str, pre)), cached=rng.random() < 0.7)
        else:
            n = rng.choice([1, 1, 1, 2, 6])
            lens = [_between(rng, 512, 131072) for _ in range(n)]
            if rng.random() < 0.2:
                kw.update(page=0, permuted=False)
        if op == "attend":
            kw.update(kept=round(max(kept, 0.02), 4), alpha=0.0)
        if op == "prefill" and hq > hkv and rng.random() < 0.15:
            kw.update(tile=128)
        c = _case("drawn", op, ",".join(map(str, lens)), **kw)
        del c["name"]
        if sum(lens) <= 131072 and _cost(c) <= most:
            return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _tokens(case, seed):
    """Queries, keys and values in storage type with their scales, on the GPU:
    q [queries, hq, D], k and v [KV tokens, hkv, D], scales per head."""
    lens, pre, kv = _shape(case)
    hq, hkv = case["hq"], case["hkv"]
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(1 + 2 * seed)
    r = random.Random(1000003 * seed + 7)
    q = torch.randn((sum(lens), hq, D), generator=g, device=dev)
    k = torch.randn((sum(kv), hkv, D), generator=g, device=dev)
    v = torch.randn((sum(kv), hkv, D), generator=g, device=dev)
    v += 0.05 * torch.randn((hkv, D), generator=g, device=dev)
    u = torch.randn((hkv, D), generator=g, device=dev)
    u = u / u.norm(dim=1, keepdim=True)
    uq = 2.0 * u.repeat_interleave(hq // hkv, dim=0)
    q0 = k0 = 0
    for n, p, t in zip(lens, pre, kv):
        even = (torch.arange(p, p + n, device=dev) // B) % 2 == 0     # biased query blocks
        q[q0:q0 + n] += even[:, None, None] * uq
        nb = (t + B - 1) // B
        planted = np.zeros((hkv, nb), np.float32)
        for h in range(hkv):
            planted[h, 0] = 1.0
            if nb > 1:
                picks = min(nb - 1, max(1, round(case["salient"] * nb)))
                planted[h, r.sample(range(1, nb), picks)] = 1.0
        at = torch.from_numpy(planted).to(dev).repeat_interleave(B, dim=1)[:, :t]
        k[k0:k0 + t] += 3.0 * at.t()[:, :, None] * u
        q0, k0 = q0 + n, k0 + t
    if case["dtype"] == "bf16":
        one = torch.ones(max(hq, hkv), device=dev)
        return dict(q=q.bfloat16(), k=k.bfloat16(), v=v.bfloat16(), q_scale=one[:hq],
                    k_scale=one[:hkv], v_scale=one[:hkv])
    res = {}
    for name, x in (("q", q), ("k", k), ("v", v)):
        s = (x.abs().amax(dim=(0, 2)) / 448.0).contiguous()
        res[name] = (x / s[None, :, None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn)
        res[name + "_scale"] = s
    return res


def _own_mask(case, seed, nq, nk):
    """A caller's mask [batch, hkv, nq, nk]: sink, diagonal window and random
    blocks of the expected share."""
    lens, pre, _ = _shape(case)
    g = torch.Generator(device="cuda").manual_seed(5 + 2 * seed)
    m = torch.rand((len(lens), case["hkv"], nq, nk), generator=g, device="cuda") < case["kept"]
    j = torch.arange(nk, device="cuda")
    for b, (n, p) in enumerate(zip(lens, pre)):
        first = p + torch.arange(nq, device="cuda") * B
        last = (p + torch.clamp(torch.arange(1, nq + 1, device="cuda") * B, max=n) - 1) // B
        m[b] |= (j[None, :] < case["sink"]) | (last[:, None] - j[None, :] < case["window"])
        m[b] &= (j[None, :] <= last[:, None]) & (first[:, None] < p + n)
    return m.to(torch.uint8)


def prepare(case, seed):
    """A program's state before the call: the layer's queries, its paged cache
    with page table, lengths, and the buffers and backend it keeps."""
    lens, pre, kv = _shape(case)
    x = _tokens(case, seed)
    hq, hkv, page = case["hq"], case["hkv"], case["page"]
    fp8 = case["dtype"] == "fp8"
    dev = torch.device("cuda")
    raw = (lambda t: t.view(torch.uint8)) if fp8 else (lambda t: t)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    cu_k = np.concatenate([[0], np.cumsum(kv)]).astype(np.int32)
    if page:
        npg = [(t + page - 1) // page for t in kv]
        total = sum(npg) + (sum(npg) // 4 + 1 if case["permuted"] else 0)
        order = torch.arange(total, dtype=torch.int32)
        if case["permuted"]:
            order = torch.randperm(total, generator=torch.Generator().manual_seed(9 + seed)).int()
        table = torch.zeros((len(kv), max(npg)), dtype=torch.int32)
        at = 0
        slots = []
        for b, (m, t) in enumerate(zip(npg, kv)):
            table[b, :m] = order[at:at + m]
            s = order[at:at + m].long()[:, None] * page + torch.arange(page)[None, :]
            slots.append(s.reshape(-1)[:t])
            at += m
        slots = torch.cat(slots).to(dev)
        table = table.to(dev)
        pools = []
        for name in ("k", "v"):
            pool = torch.zeros((total * page, hkv, D), dtype=raw(x[name]).dtype, device=dev)
            pool.index_copy_(0, slots, raw(x[name]))
            pools.append(pool)
        kc, vc = pools
        pages = int(table.shape[1])
    else:
        kc, vc, table, pages, total = raw(x["k"]), raw(x["v"]), None, 0, 0
    st = dict(case=case, q=raw(x["q"]), k=kc, v=vc, table=table, cu=torch.from_numpy(cu).to(dev),
              cu_host=cu, scales=({s: x[s] for s in ("q_scale", "k_scale", "v_scale")} if fp8 else {}))
    knobs = dict(alpha=case["alpha"], sink_blocks=case["sink"], window_blocks=case["window"])
    if case["op"] == "extend":
        cfg = serving.BackendConfig(num_q_heads=hq, num_kv_heads=hkv, page_size=page,
                                    max_batch=len(lens), max_extend_len=max(lens),
                                    max_kv_len=max(kv), dtype=case["dtype"],
                                    mean_correction=case["corr"], **knobs)
        be = serving.PrefillBackend(cfg)
        st["backend"] = be
        st["means"] = None
        if case["cached"]:
            # what the forwards over the prefix left: the means of its blocks
            st["means"] = be.alloc_means_cache(total)
            fill = be.init_forward_metadata([1] * len(pre), [max(0, p - 1) for p in pre], table)
            be.forward_extend(st["q"][:len(pre)].contiguous(), kc, vc, fill, means_cache=st["means"],
                              **st["scales"])
        st["meta"] = be.init_forward_metadata(lens, pre, table,
                                              cached_prefix_lens=pre if case["cached"] else None)
        return st
    p = fp2.make_params(batch=len(lens), num_q_heads=hq, num_kv_heads=hkv, max_seq_len=max(lens),
                        page_size=page, max_pages_per_seq=pages, dtype=case["dtype"],
                        mean_correction=int(case["corr"]), query_tile_rows=case["tile"], **knobs)
    st["p"] = p
    st["workspace"] = fp2.alloc_workspace(p)
    out, mask, lse = fp2.alloc_outputs(p, sum(lens), want_lse=case["lse"])
    st["mask"] = mask
    if case["op"] == "attend":
        st["mask"] = _own_mask(case, seed, mask.shape[2], mask.shape[3])
    if case["op"] != "estimate":
        st["out"], st["lse"] = out, lse
    return st


def run(state):
    """One layer's call."""
    case = state["case"]
    if case["op"] == "extend":
        out, lse = state["backend"].forward_extend(state["q"], state["k"], state["v"], state["meta"],
                                                   means_cache=state["means"],
                                                   want_lse=case["lse"], **state["scales"])
        return {"out": out, "lse": lse}
    if case["op"] == "estimate":
        mask, _ = fp2.estimate(state["p"], state["q"], state["k"], state["v"], state["cu"],
                               state["table"], cu_seqlens_host=state["cu_host"],
                               block_mask=state["mask"], workspace=state["workspace"],
                               **state["scales"])
        return {"mask": mask}
    if case["op"] == "attend":
        out, lse = fp2.attend(state["p"], state["q"], state["k"], state["v"], state["cu"],
                              state["mask"], state["table"], cu_seqlens_host=state["cu_host"],
                              out=state["out"], lse=state["lse"], workspace=state["workspace"],
                              **state["scales"])
        return {"out": out, "lse": lse}
    out, mask, lse = fp2.prefill(state["p"], state["q"], state["k"], state["v"], state["cu"],
                                 state["table"], cu_seqlens_host=state["cu_host"],
                                 out=state["out"], lse=state["lse"], block_mask=state["mask"],
                                 workspace=state["workspace"], **state["scales"])
    return {"out": out, "mask": mask, "lse": lse}


# ---------------------------------------------------------------------------
# What a pass cannot do without, how far results may differ, and the exact ones
# ---------------------------------------------------------------------------

def work(case):
    lens, pre, kv = _shape(case)
    hq, hkv = case["hq"], case["hkv"]
    esz = 1 if case["dtype"] == "fp8" else 2
    tq = B if not case["tile"] else case["tile"] * hkv // hq
    nq, nk = (max(lens) + tq - 1) // tq, (max(kv) + B - 1) // B
    bytes_ = sum(lens) * hq * D * esz
    flops = 0.0
    if case["cached"]:   # complete prefix blocks: their means instead of their keys and values
        fresh = sum(t - p // B * B for t, p in zip(kv, pre))
        bytes_ += fresh * hkv * D * 2 * esz + sum(p // B for p in pre) * hkv * D * 4
    else:
        bytes_ += sum(kv) * hkv * D * 2 * esz
    if case["op"] == "estimate" or case["op"] == "prefill" or case["op"] == "extend":
        bytes_ += len(lens) * hkv * nq * nk
    if case["op"] == "attend":
        bytes_ += len(lens) * hkv * nq * nk
    if case["op"] != "estimate":
        bytes_ += sum(lens) * hq * (2 * D + (4 if case["lse"] else 0))
    for n, p, t in zip(lens, pre, kv):
        pairs = n * (p + (n + 1) / 2.0)                  # visible (query, key) pairs
        if case["op"] != "attend":
            flops += 2.0 * D * hq * pairs / B            # block scores
        if case["op"] != "estimate":
            flops += 4.0 * D * hq * pairs * case["kept"]
            if case["corr"]:
                flops += 4.0 * D * hq * pairs / B * (1.0 - case["kept"])
    return {"bytes": float(bytes_), "flops": flops}


def tolerance(case):
    """bf16: probabilities and outputs are rounded to 8 bits of mantissa; fp8:
    probabilities are rounded to 4 bits, against a reference that depends on
    the order of the keys. A block whose energy lies at the threshold may be
    selected by one implementation and not by another (``differ``)."""
    if case["op"] == "estimate":
        return {"rel": 1e-5, "differ": 2e-4}
    if case["dtype"] == "fp8":
        return {"rel": 0.03, "max": 0.99, "differ": 2e-4}
    return {"rel": 0.008, "max": 0.2, "differ": 2e-4}


def exact(case, seed):
    """The same results in 64 bits: means, block energies, selection, and the
    softmax over kept keys and pruned blocks' means."""
    if case["op"] == "estimate":
        return None
    x = _tokens(case, seed)
    lens, pre, kv = _shape(case)
    hq, hkv = case["hq"], case["hkv"]
    g = hq // hkv
    tq = B if not case["tile"] else case["tile"] // g     # positions per selection tile
    scale = 1.0 / math.sqrt(D)
    nqm, nkm = (max(lens) + tq - 1) // tq, (max(kv) + B - 1) // B
    given = _own_mask(case, seed, nqm, nkm) if case["op"] == "attend" else None
    out = torch.zeros((sum(lens), hq, D), dtype=torch.float64, device="cuda")
    lse = torch.zeros((sum(lens), hq), dtype=torch.float64, device="cuda")
    q0 = k0 = 0
    for b, (n, p, t) in enumerate(zip(lens, pre, kv)):
        nb, nt = (t + B - 1) // B, (n + tq - 1) // tq
        cnt = torch.full((nb,), B, dtype=torch.float64, device="cuda")
        cnt[-1] = t - (nb - 1) * B
        ja = (p + torch.arange(nt) * tq) // B                              # block of a tile's first row
        jb = (p + torch.clamp(torch.arange(1, nt + 1) * tq, max=n) - 1) // B    # and of its last
        for h in range(hkv):
            pad = lambda name: torch.nn.functional.pad(                    # noqa: E731
                x[name][k0:k0 + t, h].double() * x[name + "_scale"][h].double(),
                (0, 0, 0, nb * B - t)).view(nb, B, D)
            k, v = pad("k"), pad("v")
            kbar, vbar = k.sum(1) / cnt[:, None], v.sum(1) / cnt[:, None]
            khat = kbar.bfloat16().double()
            qs = x["q"][q0:q0 + n, h * g:(h + 1) * g].double() * \
                x["q_scale"][h * g:(h + 1) * g].double()[None, :, None]
            if given is not None:
                keep = given[b, h, :nt, :nb].cpu().numpy() != 0
            else:
                ell = torch.empty((nt, nb), dtype=torch.float64, device="cuda")
                step = max(1, (1 << 26) // (tq * g * nb))
                for i0 in range(0, nt, step):
                    i1 = min(nt, i0 + step)
                    r = qs[i0 * tq:min(n, i1 * tq)].reshape(-1, D)
                    s = (r @ khat.t()) * scale
                    s = torch.nn.functional.pad(s, (0, 0, 0, (i1 - i0) * tq * g - s.shape[0]),
                                                value=-math.inf)
                    ell[i0:i1] = torch.logsumexp(s.view(i1 - i0, tq * g, nb), dim=1)
                jj, a, z = torch.arange(nb)[None, :], ja[:, None], jb[:, None]
                seen = (jj <= z).cuda()
                ell.masked_fill_(~seen, -math.inf)
                forced = ((jj < case["sink"]) | (z - jj < case["window"]) | (jj >= a)).cuda() & seen
                keep = forced | (ell >= ell.amax(1, keepdim=True) + math.log(case["alpha"]))
                keep = (keep & seen).cpu().numpy()
            for i in range(nt):
                r0, r1 = i * tq, min(n, (i + 1) * tq)
                r = qs[r0:r1].reshape(-1, D)
                a = int(ja[i])
                kept = torch.from_numpy(np.nonzero(keep[i, :int(jb[i]) + 1])[0]).cuda()
                s = (r @ k[kept].view(-1, D).t()) * scale
                key = (kept[:, None] * B + torch.arange(B, device="cuda")[None, :]).view(-1)
                pos = (p + torch.arange(r0, r1, device="cuda")).repeat_interleave(g)
                s.masked_fill_(key[None, :] > pos[:, None], -math.inf)
                vals = v[kept].view(-1, D)
                if case["corr"] and a > 0:
                    cut = torch.from_numpy(np.nonzero(~keep[i, :a])[0]).cuda()
                    s = torch.cat([s, (r @ kbar[cut].t()) * scale + math.log(B)], dim=1)
                    vals = torch.cat([vals, vbar[cut]], dim=0)
                z = torch.logsumexp(s, dim=1)
                o = torch.exp(s - z[:, None]) @ vals
                out[q0 + r0:q0 + r1, h * g:(h + 1) * g] = o.view(r1 - r0, g, D)
                lse[q0 + r0:q0 + r1, h * g:(h + 1) * g] = z.view(r1 - r0, g)
        q0, k0 = q0 + n, k0 + t
    res = {"out": out, "lse": lse if case["lse"] else None}
    if case["op"] == "prefill":
        res["mask"] = None
    return res
