"""The decode-attention work a program has this library do: one call, or one step of calls,
of each route through the public entry points, over the sizes the routes are used at.

A case is a dict of plain values:
  route    one_launch  pkv_plan_decode: plan, attend and merge in one launch
           noalloc     pkv_plan_decode_noalloc: the same with the library's own scratch
           layers      pkv_plan once, then pkv_decode (fused merge) for each layer of a model
           separate    pkv_plan, then pkv_decode with a separate merge kernel
           rect        pkv_decode_rect over the whole batch
           buckets     pkv_decode_buckets with coarse length buckets
  batch    rows of the batch, `free` of them empty slots of a serving batch (length 0)
  family   how the row lengths are drawn from [lo, hi]: "uniform", "bimodal" (half the rows
           short, half long), "zipf" (multiples of lo, heavy-tailed) or "equal" (all hi)
  lengths  seed of the row lengths: they belong to the case, so its work is known
  hq, hkv  query and KV heads (G = hq / hkv query heads share a KV head)
  split_min, split_max   the planner's bounds
  layers   decode calls of a pass (1 except on the layers route)
  scaled   the queries are stored with 1/sqrt(d) folded in (else sm_scale carries it)

K, V and Q values, page order and holes come from the seed that prepare() gets.
"""
import math
import random

import torch

import paper_2606_26666_amd as pkv
from paper_2606_26666_amd import costmodel

D = 128      # head dimension
PAGE = 16    # tokens per KV page
STEPS = 32   # decode steps a row's block table has room for
ROUTES = ("one_launch", "noalloc", "layers", "separate", "rect", "buckets")
MAX_KV_BYTES = 1.6e9  # K and V bytes of the largest drawn case
MAX_TOKENS = 65536    # the longest row (the longest prompts of the request traces)


def _case(name, route, batch, family, lo, hi, hkv, *, hq=32, lengths=1, split_min=16, split_max=64, layers=1,
          free=0, scaled=True):
    c = dict(route=route, batch=batch, free=free, family=family, lo=lo, hi=hi, lengths=lengths, hq=hq, hkv=hkv,
             split_min=split_min, split_max=split_max, layers=layers, scaled=scaled)
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # the smallest call: one short chat turn, one split per head; latency and launch only
        _case("tiny", "one_launch", 1, "equal", 512, 512, 8, split_min=1, split_max=1),
        # a few short interactive rows of odd lengths (single tokens among them) on a model
        # with 8 query heads per KV head, from a caller that keeps no workspace
        _case("b4_short_g8", "noalloc", 4, "uniform", 1, 2048, 4, scaled=False),
        # one long document being read: the benchmark's B1 configuration
        _case("b1_32k", "one_launch", 1, "equal", 32769, 32769, 8),
        # the longest context of the request traces, 8 query heads per KV head
        _case("b1_64k_g8", "one_launch", 1, "equal", 65531, 65531, 4),
        # short and long rows together: the benchmark's B8 bimodal configuration
        _case("b8_bimodal", "one_launch", 8, "bimodal", 256, 32768, 8, lengths=20260623),
        # no grouping (each query head has its own KV head)
        _case("b4_bimodal_g1", "one_launch", 4, "bimodal", 256, 32768, 32, lengths=3),
        # two query heads per KV head, heavy-tailed lengths
        _case("b8_zipf_g2", "one_launch", 8, "zipf", 256, 32768, 16, lengths=5),
        # a serving batch of chats, some slots free
        _case("b64_chat", "one_launch", 64, "uniform", 128, 4096, 8, free=5, scaled=False),
        # many short rows: more rows than the planner's one-wave path takes
        _case("b256_short_g8", "one_launch", 256, "uniform", 16, 1024, 8, hq=64),
        # the largest call: a full batch of long ragged rows
        _case("b32_uniform", "one_launch", 32, "uniform", 1024, 32768, 8, lengths=7),
        # a model's decode step: one plan, reused by the attention of four layers
        _case("b16_layers", "layers", 16, "uniform", 256, 8192, 8, layers=4, lengths=11),
        # the rectangular kernels through the length-bucket route
        _case("b8_buckets", "buckets", 8, "uniform", 1024, 32768, 8, lengths=20260623),
    ]


def draw(rng):
    """One more case: the route, the heads, the batch (1..256, or 1..6 where the library's
    scratch holds the states, evenly over its logarithm) and the row lengths (the longest up
    to MAX_TOKENS, evenly over its logarithm)."""
    route = rng.choice(("one_launch",) * 6 + ("noalloc", "layers", "layers", "separate", "rect", "buckets"))
    hq, hkv = rng.choice(((32, 8), (32, 8), (32, 8), (32, 4), (64, 8), (32, 16), (32, 32)))
    layers = rng.randint(2, 4) if route == "layers" else 1
    token_bytes = 4 * D * hkv * layers
    batch = round(math.exp(rng.uniform(0.0, math.log(6 if route == "noalloc" else 256))))
    family = rng.choice(("uniform", "uniform", "bimodal", "zipf", "equal"))
    top = min(MAX_TOKENS, MAX_KV_BYTES / token_bytes / batch)
    hi = round(math.exp(rng.uniform(math.log(min(256, top)), math.log(top))))
    lo = min(hi, rng.choice((1, 16, 200, max(1, hi // 16))))
    free = rng.randint(0, batch // 4) if rng.random() < 0.3 else 0
    return _case(None, route, batch, family, lo, hi, hkv, hq=hq, lengths=rng.randrange(1 << 30),
                 layers=layers, free=free, scaled=rng.random() < 0.7)


def _lengths(case):
    """Row lengths: a function of the case alone."""
    r = random.Random(case["lengths"])
    lo, hi, n = case["lo"], case["hi"], case["batch"]
    if case["family"] == "uniform":
        lens = [r.randint(lo, hi) for _ in range(n)]
    elif case["family"] == "bimodal":
        short = [r.randint(lo, max(lo, hi // 16)) for _ in range(n // 2)]
        lens = short + [r.randint(max(lo, hi // 2), hi) for _ in range(n - n // 2)]
        r.shuffle(lens)
    elif case["family"] == "zipf":
        lens = [min(hi, int(lo * r.paretovariate(0.5))) for _ in range(n)]
    else:
        lens = [hi] * n
    for i in r.sample(range(n), case["free"]):
        lens[i] = 0
    return lens


def _inputs(case, seed):
    """Inputs on the GPU, from the seed: page pools with one page in eight unowned, block
    table and queries."""
    lens = _lengths(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    pages = [-(-(n + STEPS) // PAGE) for n in lens]
    total = sum(pages)
    pool = total + total // 8 + 1
    perm = torch.randperm(pool, generator=gen, device="cuda", dtype=torch.int32)
    table = torch.full((len(lens), max(pages)), -1, dtype=torch.int32, device="cuda")
    at = 0
    for i, n in enumerate(pages):
        table[i, :n] = perm[at:at + n]
        at += n
    shape = (pool, PAGE, case["hkv"], D)
    caches = [tuple(torch.randn(shape, generator=gen, device="cuda", dtype=torch.float16) for _ in "kv")
              for _ in range(case["layers"])]
    q = [torch.randn((len(lens), case["hq"], D), generator=gen, device="cuda") for _ in range(case["layers"])]
    q = [(x / math.sqrt(D) if case["scaled"] else x).half() for x in q]
    return lens, table, caches, q


def _sm_scale(case):
    return 1.0 if case["scaled"] else 1.0 / math.sqrt(D)


def prepare(case, seed):
    lens, table, caches, q = _inputs(case, seed)
    hq, hkv, route = case["hq"], case["hkv"], case["route"]
    target = costmodel.default_target(lens, hkv, hq=hq)
    params = pkv.make_params(hkv, case["split_min"], case["split_max"], target, policy=pkv.PKV_SPLIT_QUOTA)
    s = dict(case=case, table=table, caches=caches, q=q, params=params, host_lens=lens,
             lens=torch.tensor(lens, dtype=torch.int32, device="cuda"), scale=_sm_scale(case))
    s["out"] = [torch.zeros_like(x) for x in q]
    if route == "rect":
        active = sum(n > 0 for n in lens)
        s["S"] = costmodel.rect_split_count(active, hkv, params)
    if route == "noalloc":
        n = pkv.pkv_max_tasks(len(lens), hkv, case["split_max"])
        s["plan"] = (torch.zeros((n, 5), dtype=torch.int32, device="cuda"),
                     torch.zeros(len(lens) + 1, dtype=torch.int32, device="cuda"),
                     torch.zeros(1, dtype=torch.int32, device="cuda"))
        s["err"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    else:
        s["bufs"] = b = pkv.DecodeBuffers(len(lens), hq, hkv, D, case["split_max"], "cuda")
        s["plan"] = (b.tasks, b.split_offsets, b.num_tasks)
    return s


def run(s):
    route, table, lens, params, out, scale = s["case"]["route"], s["table"], s["lens"], s["params"], s["out"], s["scale"]
    (k, v), q = s["caches"][0], s["q"][0]
    tasks, offsets, count = s["plan"]
    if route == "one_launch":
        pkv.pkv_plan_decode(q, k, v, table, lens, params, tasks, offsets, count, scale, out[0], s["bufs"].ws)
    elif route == "noalloc":
        pkv.pkv_plan_decode_noalloc(q, k, v, table, lens, params, tasks, offsets, count, scale, out[0], s["err"])
    elif route == "rect":
        pkv.pkv_decode_rect(q, k, v, table, lens, s["S"], params.tile_tokens, scale, out[0], s["bufs"].ws)
    elif route == "buckets":
        pkv.pkv_decode_buckets(q, k, v, table, lens, s["host_lens"], costmodel.COARSE_BUCKET_TOKENS, params, scale,
                               out[0], s["bufs"].ws)
    else:
        ws = s["bufs"].ws
        pkv.pkv_plan(lens, None, k.shape[0], params, tasks, offsets, count, ws, max_pages_per_row=table.shape[1])
        for (k, v), q, o in zip(s["caches"], s["q"], out):
            pkv.pkv_decode(q, k, v, table, lens, tasks, offsets, count, scale, o, ws, fused=route == "layers")
    if route in ("rect", "buckets"):
        return {"out": out}
    return {"out": out, "tasks": tasks, "split_offsets": offsets, "num_tasks": count}


def work(case):
    """K, V, queries, lengths and page ids read once, outputs written once."""
    lens = _lengths(case)
    tokens, rows, layers = sum(lens), len(lens), case["layers"]
    pages = sum(-(-n // PAGE) for n in lens)
    kv = tokens * case["hkv"] * D * 2 * 2
    qo = rows * case["hq"] * D * 2 * 2
    return {"bytes": layers * (kv + qo) + 4 * pages + 4 * rows, "flops": layers * 4 * case["hq"] * D * tokens}


def tolerance(case):
    """fp16 outputs of fp32 sums: each rounds to within half an fp16 unit (2^-11 of the value),
    a relative 2-norm of 2.1e-4 against 64 bits as measured on every case. The plan (integers)
    is exact."""
    return {"rel": 1e-3, "max": 4e-3}


def exact(case, seed):
    lens, table, caches, q = _inputs(case, seed)
    hq, hkv = case["hq"], case["hkv"]
    outs = []
    for (k, v), ql in zip(caches, q):
        out = torch.zeros((len(lens), hq, D), dtype=torch.float64, device="cuda")
        for i, n in enumerate(lens):
            if n == 0:
                continue
            ids = table[i, : -(-n // PAGE)].long()
            kr, vr = (x[ids].reshape(-1, hkv, D)[:n].double().transpose(0, 1).contiguous() for x in (k, v))
            qr = ql[i].double().reshape(hkv, hq // hkv, D)
            p = torch.softmax(torch.bmm(qr, kr.transpose(1, 2).contiguous()) * _sm_scale(case), dim=-1)
            out[i] = torch.bmm(p, vr).reshape(hq, D)
        outs.append(out)
    if case["route"] in ("rect", "buckets"):
        return {"out": outs}
    return {"out": outs, "tasks": None, "split_offsets": None, "num_tasks": None}
