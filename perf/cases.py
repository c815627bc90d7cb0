"""The workloads this library's speed is measured on.

One case is one decode step of one attention layer (or the merge that a
weight node runs on the partials it received), made through the C-ABI
bindings of ``paper_2606_29207_amd.kf``.  A case names a batch:

* ``mode``    how the step is called: ``step`` (kf_decode_step), ``no_alloc``
  (kf_decode_step_no_alloc), ``calls`` (append, partial attention and merge as
  three calls), ``static`` (partial attention and merge of a context that
  takes no token), ``query_first`` (historical routes on one stream while the
  tails append and attend on a second one) or ``merge`` (kf_merge_partials
  alone);
* ``seqs``, ``q_heads``, ``kv_heads`` and the resident tokens per sequence,
  log-uniform in ``ctx_lo .. ctx_hi`` (``lens`` seeds the lengths, so that a
  case always has the same ones), cut into routes of ``part`` tokens;
* ``fp8`` pools (E4M3 codes, one scale per page and KV head) or bf16,
  ``head_major`` pools or page-major, ``permuted`` page ids (a serving pool
  after some churn) or contiguous ones (pages handed out in pairs).

An appending step writes one token per sequence into its tail page.  As in a
serving loop, the step's route table is copied into the bound buffer first,
so that every pass is the same step.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2606_29207_amd import kf

PAGE, DIM = 16, 128
RESERVE = 192            # tokens a tail's reserved pages hold beyond its resident ones
SCALE = 1.0 / math.sqrt(DIM)
DEVICE = "cuda"


def _case(name, mode, seqs, q_heads, kv_heads, ctx_lo, ctx_hi, part, *, fp8=False,
          head_major=False, permuted=False, lens=1):
    return {"name": name, "mode": mode, "seqs": seqs, "q_heads": q_heads, "kv_heads": kv_heads,
            "ctx_lo": ctx_lo, "ctx_hi": ctx_hi, "part": part, "fp8": fp8,
            "head_major": head_major, "permuted": permuted, "lens": lens}


def listed():
    return [
        # the smallest call: one short conversation on a small layer, 4 MB of K/V,
        # where launches and latency count
        _case("tiny", "static", 1, 8, 2, 4096, 4096, 2048),
        # a few interactive chats on a Llama-3.1-8B layer, one route each
        _case("chat_8", "step", 8, 32, 8, 300, 3000, 8192, permuted=True),
        # a full continuous batch of short requests on an fp8 GQA-8 layer
        _case("short_fp8_64", "step", 64, 64, 8, 128, 4096, 16384, fp8=True, permuted=True),
        # multi-head attention (one query head per KV head), a large batch of
        # short requests, the step as its three calls
        _case("mha_192", "calls", 192, 32, 32, 65, 1100, 8192, permuted=True),
        # wide groups (16 query heads per KV head) over medium ragged contexts
        _case("gqa16_24", "step", 24, 64, 4, 1500, 12000, 4096, permuted=True),
        # a tensor-parallel shard with 2 KV heads, head-major pools, under a
        # harness that cannot allocate
        _case("shard_2kv", "no_alloc", 48, 8, 2, 8192, 8192, 4096, head_major=True),
        # an attention node's query-first schedule over 16K contexts
        _case("query_first_8", "query_first", 8, 32, 8, 16384, 16384, 4096),
        # a weight node merging the partials of million-token requests
        _case("merge_128", "merge", 32, 32, 8, 128 * 8192, 128 * 8192, 8192),
        # a Llama-3.1-8B layer at 32K tokens, the benchmark's default workload
        _case("llama8b_32k", "step", 16, 32, 8, 32768, 32768, 8192),
        # agentic serving: lengths 2K .. 128K in one permuted pool
        _case("agentic_mix", "step", 64, 32, 8, 2048, 131072, 16384, permuted=True),
        # a 70B-like layer (64/8 heads) with fp8 K/V at 64K tokens
        _case("wide_gqa_fp8", "step", 32, 64, 8, 65536, 65536, 16384, fp8=True),
        # four million-token contexts, 17 GB of K/V
        _case("million_ctx", "static", 4, 32, 8, 1048576, 1048576, 65536),
    ]


_HEADS = ((8, 2), (16, 2), (32, 8), (64, 8), (32, 32), (40, 8), (24, 8), (64, 4), (8, 1), (16, 16))


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        mode = rng.choice(("step", "step", "step", "no_alloc", "calls", "static", "query_first",
                           "merge"))
        q_heads, kv_heads = rng.choice(_HEADS)
        lo = spread(100, 100000)
        c = _case("", mode, spread(1, 256), q_heads, kv_heads, lo,
                  lo if rng.random() < 0.3 else min(262144, spread(lo, 40 * lo)),
                  rng.choice((2048, 4096, 8192, 16384, 65536)), fp8=rng.random() < 0.35,
                  head_major=rng.random() < 0.25, permuted=rng.random() < 0.6,
                  lens=rng.randrange(1 << 20))
        del c["name"]
        if mode == "merge":
            c.update(fp8=False, head_major=False, permuted=False)
        # the library's fixed scratch array serves groups of up to 8 query heads
        if mode == "no_alloc" and q_heads // kv_heads > 4:
            continue
        if 2e6 <= work(c)["bytes"] <= 8e9:
            return c


# ------------------------------------------------------------------- tables
def _lengths(case):
    """Resident tokens of each sequence."""
    lo, hi = case["ctx_lo"], case["ctx_hi"]
    rng = random.Random(case["lens"])
    return [min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))
            for _ in range(case["seqs"])]


def _appends(case):
    return case["mode"] in ("step", "no_alloc", "calls", "query_first")


def _table(case):
    """Route rows [seq, part, tok_begin, tok_end, page_base, page_cap], the CSR
    rows of the sequences and their tail routes (-1 where nothing is appended)."""
    rows, begin, tails, base = [], [0], [], 0
    for b, n in enumerate(_lengths(case)):
        for k, t0 in enumerate(range(0, n, case["part"])):
            t1 = min(t0 + case["part"], n)
            grow = RESERVE if t1 == n and _appends(case) else 0
            cap = -(-(t1 - t0 + grow) // PAGE)
            rows.append([b, k, t0, t1, base, cap])
            base += cap
        tails.append(len(rows) - 1 if _appends(case) else -1)
        begin.append(len(rows))
    return rows, begin, tails


def _page_ids(case, caps, gen):
    """Page ids of the routes, route after route, and the pool's page count."""
    total = sum(caps)
    if case["permuted"]:
        return torch.randperm(total, generator=gen, device=DEVICE).to(torch.int32), total
    ids, first = [], 0
    for c in caps:
        ids.append(torch.arange(first, first + c, dtype=torch.int32))
        first += c + (c & 1)
    return torch.cat(ids).to(DEVICE), first


# ------------------------------------------------------------------- inputs
def _pages(case, pool):
    """The pool indexed by page first, whatever its layout."""
    return pool.transpose(0, 1) if case["head_major"] else pool


def _encode(x):
    """E4M3 codes and scales of pages x [n, heads, ...], the page's largest at 448."""
    amax = x.abs().amax(dim=(2, 3))
    scale = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    return _code(x / scale[:, :, None, None]), scale


def _code(x):
    return x.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)


def _decode(codes):
    return codes.view(torch.float8_e4m3fn).float()


def _pool(case, P, inner, gen):
    """A pool of N(0, 1) values in its storage layout, and its scales (fp8)."""
    H = case["kv_heads"]
    lead = (H, P) if case["head_major"] else (P, H)
    if not case["fp8"]:
        return torch.randn(lead + inner, generator=gen, device=DEVICE, dtype=torch.bfloat16), None
    pool = torch.empty(lead + inner, device=DEVICE, dtype=torch.uint8)
    scale = torch.empty((P, H), device=DEVICE)
    step = max(1, (1 << 27) // (H * PAGE * DIM))
    for p in range(0, P, step):
        n = min(step, P - p)
        codes, scale[p:p + n] = _encode(torch.randn((n, H) + inner, generator=gen, device=DEVICE))
        _pages(case, pool)[p:p + n] = codes
    return pool, scale


def _inputs(case, seed):
    """The step's inputs on the GPU, from the seed alone."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    rows, begin, tails = _table(case)
    B, Hq, H = case["seqs"], case["q_heads"], case["kv_heads"]
    x = {"routes": torch.tensor(rows, dtype=torch.int32, device=DEVICE),
         "seq_route_begin": torch.tensor(begin, dtype=torch.int32, device=DEVICE)}
    if case["mode"] == "merge":
        x["o_part"] = torch.randn((len(rows), Hq, DIM), generator=gen, device=DEVICE) * 0.02
        x["lse_part"] = 9.5 + 0.1 * torch.randn((len(rows), Hq), generator=gen, device=DEVICE)
        return x
    x["tail_route"] = torch.tensor(tails, dtype=torch.int32, device=DEVICE)
    x["page_ids"], P = _page_ids(case, [r[5] for r in rows], gen)
    x["q"] = torch.randn((B, Hq, DIM), generator=gen, device=DEVICE, dtype=torch.bfloat16)
    for n in ("k_new", "v_new"):
        x[n] = torch.randn((B, H, DIM), generator=gen, device=DEVICE, dtype=torch.bfloat16)
    x["k_pool"], x["k_scale"] = _pool(case, P, (PAGE, DIM), gen)
    x["v_pool"], x["v_scale"] = _pool(case, P, (DIM, PAGE), gen)
    # an attention sink: the first token of each sequence scores about 7 for every head
    sink = 0.6 * x["q"].view(B, H, Hq // H, DIM).float().sum(2)
    first = x["page_ids"][torch.tensor([rows[r][4] for r in begin[:-1]], device=DEVICE)].long()
    pages = _pages(case, x["k_pool"])
    if case["fp8"]:
        k = _decode(pages[first]) * x["k_scale"][first][:, :, None, None]
        k[:, :, 0] = sink
        pages[first], x["k_scale"][first] = _encode(k)
    else:
        pages[first, :, 0] = sink.to(torch.bfloat16)
    return x


# --------------------------------------------------------------------- step
def prepare(case, seed):
    x = _inputs(case, seed)
    B, Hq, R = case["seqs"], case["q_heads"], x["routes"].shape[0]
    st = {"mode": case["mode"], "inputs": x,
          "out": torch.empty((B, Hq, DIM), device=DEVICE),
          "lse": torch.empty((B, Hq), device=DEVICE),
          "err": torch.zeros(1, dtype=torch.int32, device=DEVICE)}
    if case["mode"] == "merge":
        st["merge"] = kf.bind_merge_partials(B, x["o_part"], x["lse_part"], x["seq_route_begin"],
                                             st["out"], st["lse"], st["err"])
        return st
    layout = kf.KV_HEAD_MAJOR if case["head_major"] else kf.KV_PAGE_MAJOR
    shape = kf.shape_of(x["q"], x["k_pool"], x["page_ids"], SCALE, layout)
    most = int(x["routes"][:, 5].max())
    st["routes"] = x["routes"].clone()
    st["o_part"] = torch.empty((R, Hq, DIM), device=DEVICE)
    st["lse_part"] = torch.empty((R, Hq), device=DEVICE)
    scales = {"k_scale": x["k_scale"], "v_scale": x["v_scale"]}
    if case["mode"] in ("step", "no_alloc"):
        ws = kf.alloc_workspace(shape, R, most, DEVICE) if case["mode"] == "step" else None
        st["step"] = kf.bind_decode_step(
            shape, x["q"], x["k_pool"], x["v_pool"], st["routes"], x["tail_route"], most,
            x["page_ids"], x["seq_route_begin"], st["o_part"], st["lse_part"], st["out"],
            st["lse"], ws, st["err"], **scales)
        return st
    st["append"] = kf.bind_kv_append(shape, x["k_pool"], x["v_pool"], st["routes"],
                                     x["tail_route"], x["page_ids"], st["err"], **scales)
    st["merge"] = kf.bind_merge_partials(B, st["o_part"], st["lse_part"], x["seq_route_begin"],
                                         st["out"], st["lse"], st["err"])

    def partial(route_list=None):
        return kf.bind_partial_attn(shape, x["q"], x["k_pool"], x["v_pool"], st["routes"], most,
                                    x["page_ids"], st["o_part"], st["lse_part"],
                                    kf.alloc_workspace(shape, R, most, DEVICE), st["err"],
                                    route_list=route_list, **scales)

    if case["mode"] != "query_first":
        st["partial"] = partial()
        return st
    tails = set(x["tail_route"].tolist())
    lists = ([r for r in range(R) if r not in tails], sorted(tails))
    st["hist"], st["tail"] = (partial(torch.tensor(v, dtype=torch.int32, device=DEVICE))
                              if v else None for v in lists)
    st["second"] = torch.cuda.Stream()
    st["ready"], st["done"] = torch.cuda.Event(), torch.cuda.Event()
    return st


def run(st):
    x, mode = st["inputs"], st["mode"]
    if mode == "merge":
        st["merge"]()
        return {"out": st["out"], "lse": st["lse"]}
    if mode == "static":
        st["partial"]()
        st["merge"]()
        return {n: st[n] for n in ("out", "lse", "o_part", "lse_part")}
    st["routes"].copy_(x["routes"])   # the step's route table
    if mode in ("step", "no_alloc"):
        st["step"](x["k_new"], x["v_new"])
    elif mode == "calls":
        st["append"](x["k_new"], x["v_new"])
        st["partial"]()
        st["merge"]()
    else:
        cur, second = torch.cuda.current_stream(), st["second"]
        st["ready"].record(cur)
        second.wait_event(st["ready"])
        if st["hist"] is not None:
            st["hist"](cur)
        st["append"](x["k_new"], x["v_new"], second)
        st["tail"](second)
        st["done"].record(second)
        cur.wait_event(st["done"])
        st["merge"](cur)
    got = {n: st[n] for n in ("out", "lse", "o_part", "lse_part", "routes")}
    got.update((n, x[n]) for n in ("k_pool", "v_pool", "k_scale", "v_scale") if x[n] is not None)
    return got


def work(case):
    Hq, H, B = case["q_heads"], case["kv_heads"], case["seqs"]
    lens = _lengths(case)
    routes = sum(-(-n // case["part"]) for n in lens)
    outs = B * Hq * (DIM + 1) * 4
    partials = routes * Hq * (DIM + 1) * 4
    if case["mode"] == "merge":
        return {"bytes": partials + outs + 4 * (B + 1), "flops": 2 * routes * Hq * DIM}
    tokens = sum(lens) + (B if _appends(case) else 0)
    pages = sum(-(-n // PAGE) for n in lens)
    elem = 1 if case["fp8"] else 2
    data = tokens * H * 2 * DIM * elem + (pages * H * 8 if case["fp8"] else 0)
    if _appends(case):
        data += B * H * 2 * DIM * (2 + elem)   # the new token read, and written to its page
    tables = 4 * pages + 24 * routes + 8 * B
    return {"bytes": data + tables + B * Hq * DIM * 2 + partials + outs,
            "flops": 4 * tokens * Hq * DIM}


def tolerance(case):
    # 32-bit scores, sums and weights; p enters the second product as a bf16
    # pair (2^-17): 6e-6 is measured for fp8 pools, 1e-6 for bf16 ones.  The
    # tables and pools are the same values.
    return {"rel": 2e-5}


# -------------------------------------------------------------------- exact
def _append_exact(case, x, rows, tails):
    """The step's tokens written to their pages; route rows with the new ends."""
    B, rows = case["seqs"], [list(r) for r in rows]
    at = [(rows[r][4] + (rows[r][3] - rows[r][2]) // PAGE, (rows[r][3] - rows[r][2]) % PAGE)
          for r in tails]
    page = x["page_ids"][torch.tensor([p for p, _ in at], device=DEVICE)].long()
    slot = torch.tensor([s for _, s in at], device=DEVICE)
    for r in tails:
        rows[r][3] += 1
    b = torch.arange(B, device=DEVICE)
    for n, is_v in (("k", False), ("v", True)):
        pool, new = _pages(case, x[n + "_pool"]), x[n + "_new"]
        pages = pool[page]                                # [B, H, 16, 128] or [B, H, 128, 16]
        pages = pages.transpose(2, 3).contiguous() if is_v else pages
        if not case["fp8"]:
            pages[b, :, slot] = new
        else:
            # the first token of a page sets scale = amax/28; a later one that
            # does not fit under 448 * scale re-encodes the page to amax/28
            new = new.float()
            amax, old = new.abs().amax(-1), x[n + "_scale"][page]
            fresh = amax / torch.full_like(amax, 28.0)   # a true division, as the rule says
            start = (slot == 0)[:, None]
            over = ~start & (amax > 448.0 * old)
            scale = torch.where(start, torch.where(amax > 0, fresh, torch.ones_like(fresh)),
                                torch.where(over, fresh, old))
            wide = _code(_decode(pages) * old[:, :, None, None] / fresh[:, :, None, None])
            before = torch.arange(PAGE, device=DEVICE)[None, :] < slot[:, None]
            redo = over[:, :, None, None] & before[:, None, :, None]
            pages = torch.where(redo, wide, pages)
            pages[b, :, slot] = _code(new / scale[:, :, None])
            x[n + "_scale"][page] = scale
        pool[page] = pages.transpose(2, 3) if is_v else pages
    return rows


def _merge_exact(o, lse, begin):
    out, total = [], []
    for r0, r1 in zip(begin[:-1], begin[1:]):
        total.append(torch.logsumexp(lse[r0:r1], 0))
        out.append((torch.exp(lse[r0:r1] - total[-1])[:, :, None] * o[r0:r1]).sum(0))
    return torch.stack(out), torch.stack(total)


def exact(case, seed):
    x = _inputs(case, seed)
    rows, begin, tails = _table(case)
    if case["mode"] == "merge":
        out, lse = _merge_exact(x["o_part"].double(), x["lse_part"].double(), begin)
        return {"out": out, "lse": lse}
    if _appends(case):
        rows = _append_exact(case, x, rows, tails)
    H, G = case["kv_heads"], case["q_heads"] // case["kv_heads"]
    o_part, lse_part = [], []
    for b, _, t0, t1, base, _ in rows:
        n = t1 - t0
        ids = x["page_ids"][base:base + -(-n // PAGE)].long()
        k, v = _pages(case, x["k_pool"])[ids], _pages(case, x["v_pool"])[ids]
        if case["fp8"]:
            k, v = _decode(k), _decode(v)
        k, v = k.double(), v.double()
        if case["fp8"]:
            k *= x["k_scale"][ids][:, :, None, None]
            v *= x["v_scale"][ids][:, :, None, None]
        k = k.transpose(0, 1).reshape(H, -1, DIM)[:, :n]
        v = v.permute(1, 0, 3, 2).reshape(H, -1, DIM)[:, :n]
        s = torch.matmul(x["q"][b].view(H, G, DIM).double(), k.transpose(1, 2)) * SCALE
        lse = torch.logsumexp(s, -1)
        o_part.append(torch.matmul(torch.exp(s - lse[:, :, None]), v).reshape(H * G, DIM))
        lse_part.append(lse.reshape(H * G))
    o_part, lse_part = torch.stack(o_part), torch.stack(lse_part)
    out, lse = _merge_exact(o_part, lse_part, begin)
    got = {"out": out, "lse": lse, "o_part": o_part, "lse_part": lse_part}
    if _appends(case):
        got["routes"] = torch.tensor(rows, dtype=torch.int32, device=DEVICE)
        got.update((n, x[n]) for n in ("k_pool", "v_pool", "k_scale", "v_scale")
                   if x[n] is not None)
    return got
