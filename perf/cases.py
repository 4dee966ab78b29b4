"""The calls whose speed this repository is judged by: one attention layer of
cached diffusion-LLM serving, from a single request to a long-context batch.

A case is a dict of plain values:

  op        "attend"   one attention call over a planned batch, as each layer
                       of a serving iteration makes it: the plan, the page
                       table and the output buffers are in hand
            "iterate"  the same call with its planning and the upload of plan
                       and page table, as the first layer of an iteration
            "handoff"  export of the requests' KV from one paged pool and
                       import into another under an unrelated page table
  hq, hkv, d           query heads, KV heads, head dim
  decodes              block decodes in the batch; their prompts are drawn
                       from LN(ln prompt, sigma), clipped to [16, longest],
                       and followed by resp masked response positions
  block                query rows of a decode (32 in block decoding)
  scattered            a decode recomputes `block` scattered response
                       positions (per-token caching) instead of one block
  prefills             total lengths of the whole prefills, "2304,3328"
  layout               seed of the prompt lengths, so that they belong to the
                       case; block offsets, pages and values come from the
                       seed that prepare() gets

Head shapes are LLaDA-8B's (32/32), Dream-7B's (28/4) and smaller groups at
both head dims; batch recipes are those of the repository's workloads.
"""
import math

import numpy as np
import torch

from paper_2607_04206_amd import attn, kv

PAGE = 16


def _case(name, op, hq, hkv, d, *, decodes=0, prompt=500, sigma=0.8, longest=4096, resp=256, block=32,
          scattered=False, prefills="", layout=0):
    return dict(name=name, op=op, hq=hq, hkv=hkv, d=d, decodes=decodes, prompt=prompt, sigma=sigma, longest=longest,
                resp=resp, block=block, scattered=scattered, prefills=prefills, layout=layout)


def listed():
    return [
        # one request alone on the GPU, between its prefills: launch latency and the length of a serial chain of stages
        _case("one_decode_mha", "attend", 32, 32, 128, decodes=1, prompt=795, sigma=0.0, resp=256),
        # a lightly loaded decode worker of the GQA model
        _case("few_decodes_gqa", "attend", 28, 4, 128, decodes=8),
        # a busy decode worker of each model (the ShareGPT-like prompts of the decode workloads)
        _case("decodes_mha", "attend", 32, 32, 128, decodes=32, prompt=300, longest=2048),
        _case("decodes_gqa", "attend", 28, 4, 128, decodes=48),
        # many requests over long cached contexts: bound by HBM, some contexts split
        _case("long_decodes_mha", "attend", 32, 32, 128, decodes=256, prompt=1200, sigma=1.0, longest=32768, resp=512),
        # per-token cached decodes: scattered rows over their whole cached context
        _case("token_decodes_mha", "attend", 32, 32, 128, decodes=32, prompt=300, scattered=True),
        # the mixed microbatch of a colocated worker: decodes seated first, whole prefills admitted under the budget
        _case("mixed_gqa", "attend", 28, 4, 128, decodes=48, prefills="2304,3328"),
        # the same kind of batch for the MHA model with 1024 appended masks (odd lengths)
        _case("mixed_mha", "attend", 32, 32, 128, decodes=16, prompt=795, resp=1024, prefills="1819,1201", layout=1),
        # a typical iteration of the serving loop with everything it does on the host
        _case("iteration_gqa", "iterate", 28, 4, 128, decodes=14, prefills="1093", layout=2),
        # a dedicated prefill worker on long documents
        _case("long_prefills_gqa", "attend", 28, 4, 128, prefills="4846,11772,6273,5701,9127,7415,6914,9520"),
        # small-head model, grouped four to one: prefills, decodes and odd tails at head dim 64
        _case("mixed_d64", "attend", 32, 8, 64, decodes=24, prompt=400, prefills="1001,2048,517", layout=3),
        # disaggregated serving: the KV of a decode batch moves between two pools
        _case("handoff_mha", "handoff", 32, 32, 128, decodes=32, prompt=300, longest=2048),
    ]


def draw(rng):
    """One more case of the same ranges; costs at most what the largest listed ones do (about 6e12 flop, 10 GB)."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        hq, hkv, d = rng.choice([(32, 32, 128), (32, 32, 128), (28, 4, 128), (28, 4, 128), (32, 8, 128), (32, 8, 64), (16, 2, 128), (8, 8, 64)])
        kind = rng.choice(["decode", "decode", "decode", "mixed", "mixed", "prefill", "handoff"])
        op = "handoff" if kind == "handoff" else "iterate" if kind == "mixed" and rng.random() < 0.25 else "attend"
        decodes = 0 if kind == "prefill" else log_int(1, 128)
        prompt = log_int(100, 2000)
        resp = rng.choice([256, 512, 1024])
        # whole blocks of 32 mostly; a cut-off last block, or larger blocks, now and then
        block = rng.choice([32, 32, 32, 32, 32, 17, 64]) if kind in ("decode", "mixed") else 32
        scattered = block <= 32 and kind in ("decode", "mixed") and rng.random() < 0.15
        count = 0 if kind in ("decode", "handoff") else rng.randint(1, 4 if kind == "mixed" else 8)
        prefills = ",".join(str(log_int(200, 4500 if kind == "mixed" else 12000)) for _ in range(count))
        c = dict(op=op, hq=hq, hkv=hkv, d=d, decodes=decodes, prompt=prompt, sigma=rng.choice([0.4, 0.8, 1.0]),
                 longest=rng.choice([2048, 4096, 16384]), resp=resp, block=block, scattered=scattered, prefills=prefills,
                 layout=rng.randrange(1 << 20))
        w = work(c)
        if w["flops"] <= 6e12 and w["bytes"] <= 8e9:
            return c


# ------------------------------------------------------------------ layout
def _decode_lengths(case):
    rng = np.random.default_rng(case["layout"])
    p = rng.normal(math.log(case["prompt"]), case["sigma"], size=case["decodes"])
    return np.clip(np.rint(np.exp(p)), 16, case["longest"]).astype(np.int64)


def _prefill_lengths(case):
    return [int(x) for x in case["prefills"].split(",") if x]


def _layout(case, seed):
    """Lengths, row positions and page table of the batch: decodes first, then prefills."""
    rng = np.random.default_rng([case["layout"], seed])
    prompts = _decode_lengths(case)
    kv_len = [int(p) + case["resp"] for p in prompts]
    rows, first = [], []
    for p in prompts:
        if case["scattered"]:
            pos = int(p) + np.sort(rng.choice(case["resp"], size=case["block"], replace=False))
        else:
            pos = int(p) + case["block"] * int(rng.integers(0, case["resp"] // case["block"])) + np.arange(case["block"])
        rows.append(pos)
        first.append(int(pos[0]))
    for n in _prefill_lengths(case):
        kv_len.append(n)
        rows.append(np.arange(n))
        first.append(0)
    pages = [-(-n // PAGE) for n in kv_len]
    pool = sum(pages) + sum(pages) // 8 + 1
    table = rng.permutation(pool)[:sum(pages)].astype(np.int32)
    indptr = lambda sizes: np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)  # noqa: E731
    return dict(q_indptr=indptr([len(r) for r in rows]), q_offset=np.asarray(first, np.int32), kv_len=np.asarray(kv_len, np.int32),
                page_indptr=indptr(pages), page_ids=table, rows=rows, pool=pool, other=rng.permutation(pool)[:sum(pages)].astype(np.int32))


def _normal(gen, *shape):
    """N(0, 1) in bf16 (projected activations are of that order after the norm before them)."""
    out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    flat = out.view(-1)
    for at in range(0, flat.numel(), 1 << 28):
        part = flat[at:at + (1 << 28)]
        part.normal_(generator=gen)
    return out


def _plan_args(case, lay):
    return dict(q_indptr=lay["q_indptr"], q_offset=lay["q_offset"], kv_len=lay["kv_len"], page_indptr=lay["page_indptr"],
                page_ids=lay["page_ids"], num_q_heads=case["hq"], num_kv_heads=case["hkv"], head_dim=case["d"],
                num_pool_pages=lay["pool"], sm_scale=float(np.float32(1.0 / math.sqrt(case["d"]))),
                q_pos=np.concatenate(lay["rows"]).astype(np.int32) if case["scattered"] else None)


def _tensors(case, lay, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + case["layout"])
    pool = (lay["pool"], case["hkv"], PAGE, case["d"])
    t = dict(k_cache=_normal(gen, *pool), v_cache=_normal(gen, *pool))
    if case["op"] != "handoff":
        n = int(lay["q_indptr"][-1])
        t.update(q=_normal(gen, n, case["hq"], case["d"]), k_new=_normal(gen, n, case["hkv"], case["d"]),
                 v_new=_normal(gen, n, case["hkv"], case["d"]))
    return t


def prepare(case, seed):
    lay = _layout(case, seed)
    t = _tensors(case, lay, seed)
    state = dict(case=case, lay=lay, t=t)
    dev = t["k_cache"].device
    if case["op"] == "handoff":
        n, hkv, d = int(lay["kv_len"].sum()), case["hkv"], case["d"]
        table = dict(kv_len=lay["kv_len"], page_indptr=lay["page_indptr"], num_kv_heads=hkv, head_dim=d, num_pool_pages=lay["pool"])
        state.update(send=kv.plan(page_ids=lay["page_ids"], device=dev, **table), receive=kv.plan(page_ids=lay["other"], device=dev, **table),
                     packed=[torch.empty((n, hkv, d), dtype=torch.bfloat16, device=dev) for _ in range(2)],
                     pools=[torch.zeros_like(t["k_cache"]), torch.zeros_like(t["v_cache"])])
        return state
    rows = int(lay["q_indptr"][-1])
    state.update(args=_plan_args(case, lay), out=torch.empty((rows, case["hq"], case["d"]), dtype=torch.bfloat16, device=dev),
                 lse=torch.empty((rows, case["hq"]), dtype=torch.float32, device=dev))
    if case["op"] == "attend":
        state.update(plan=attn.plan(device=dev, **state["args"]), page_ids=torch.from_numpy(lay["page_ids"]).to(dev))
    return state


def run(state):
    t = state["t"]
    if "send" in state:
        k, v = kv.kv_export(state["send"], t["k_cache"], t["v_cache"], *state["packed"])
        kv.kv_import(state["receive"], k, v, *state["pools"])
        return [k, v, *state["pools"]]
    if "plan" in state:
        plan, page_ids = state["plan"], state["page_ids"]
    else:
        dev = t["q"].device
        plan = attn.plan(device=dev, **state["args"])
        page_ids = torch.from_numpy(state["lay"]["page_ids"]).to(dev, non_blocking=True)
    out, lse = attn.forward(plan, t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], page_ids,
                            out=state["out"], lse=state["lse"])
    return [out, lse, t["k_cache"], t["v_cache"]]


def work(case):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    lengths = [int(p) + case["resp"] for p in _decode_lengths(case)]
    items = [(case["block"], n) for n in lengths] + [(n, n) for n in _prefill_lengths(case)]
    if case["op"] == "handoff":  # K and V, each read and written by the export and by the import
        return {"bytes": 16.0 * d * hkv * sum(n for _, n in items), "flops": 0.0}
    # K and V of the context once, the fresh rows' write into the cache, Q, O, the page ids and the LSE
    bytes_ = sum(4.0 * d * hkv * (n + r) + 4.0 * d * hq * r + 4.0 * -(-n // PAGE) + 4.0 * hq * r for r, n in items)
    return {"bytes": bytes_, "flops": sum(4.0 * r * n * d * hq for r, n in items)}


def tolerance(case):
    if case["op"] == "handoff":
        return "exact"
    # bf16 outputs and bf16-rounded softmax weights: against 64 bits the call shows 2.3e-3 (2-norm) in every case
    return {"rel": 1e-2, "max": 5e-2}


def exact(case, seed):
    """out and lse in 64 bits, and the pools as the call leaves them."""
    if case["op"] == "handoff":
        return None
    lay = _layout(case, seed)
    t = _tensors(case, lay, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    scale = float(np.float32(1.0 / math.sqrt(d)))
    kc, vc = t["k_cache"], t["v_cache"]
    out = torch.empty((int(lay["q_indptr"][-1]), hq, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((int(lay["q_indptr"][-1]), hq), dtype=torch.float64, device="cuda")
    for i, pos in enumerate(lay["rows"]):
        a, b = int(lay["q_indptr"][i]), int(lay["q_indptr"][i + 1])
        pages = torch.from_numpy(lay["page_ids"][lay["page_indptr"][i]:lay["page_indptr"][i + 1]].astype(np.int64)).cuda()
        at = torch.from_numpy(np.asarray(pos, np.int64)).cuda()
        for pool, fresh in ((kc, t["k_new"]), (vc, t["v_new"])):
            pool[pages[at // PAGE], :, at % PAGE] = fresh[a:b]
        n = int(lay["kv_len"][i])
        seq = [p[pages].transpose(1, 2).reshape(-1, hkv, d)[:n] for p in (kc, vc)]
        heads = max(1, min(hq // hkv, int(2e9 // ((b - a) * n))))
        for g in range(hkv):
            k, v = (s[:, g].double() for s in seq)
            kt = k.t().contiguous()
            for h in range(g * (hq // hkv), (g + 1) * (hq // hkv), heads):
                to = min(h + heads, (g + 1) * (hq // hkv))
                q = t["q"][a:b, h:to].double().reshape(-1, d)
                for r in range(0, q.shape[0], 16384):
                    s = (q[r:r + 16384] @ kt) * scale
                    m = torch.logsumexp(s, 1, keepdim=True)
                    o = torch.exp(s - m) @ v
                    flat = torch.arange(r, r + s.shape[0], device="cuda")
                    out[a + flat // (to - h), h + flat % (to - h)] = o
                    lse[a + flat // (to - h), h + flat % (to - h)] = m[:, 0]
    return [out, lse, kc, vc]
