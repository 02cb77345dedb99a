"""The calls this framework is timed on: what a serving loop that keeps a Hard-KV Cascade Cache
does on one GPU, through the package's public entry points.

A case is one of seven kinds of call:

  decode   Decoder.attend: one layer's paged decode attention
  loop     DecodeLoop.step: one token of several layers (append, then attention per layer)
  select   Compressor.score + select: the scoring half of a compression
  mixed    the same with the sampled-redundancy metric beside the attention mass
  rewrite  Compressor.compact: the Cascade-Cache rewrite under a given selection
  step     Compressor.step: a whole compression
  budget   BudgetCompressor.select: the hard budget's selection with Cautious Update votes

Calls that change the cache first put its metadata (tables, masks, counts, allocator: one
buffer) back, as the benchmark does, so that every pass does the same work.
"""
from __future__ import annotations

import math

import torch

from paper_2606_28831_amd import Allocator, PagedKV
from paper_2606_28831_amd.pipeline import BudgetCompressor, Compressor, DecodeLoop, Decoder

PAGE = 16
DTYPE = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(name, kind, NS, Hq, Hkv, D, dtype, N, **more):
    """N: the longest row in tokens; lo: the shortest row as a share of it (rows lie evenly
    between, one length per sequence, or per head with `ragged`, as after a head-adaptive
    budget); table: page-table width in tokens (a serving cache is as wide as its longest
    allowed row); holes: share of masked slots (a sparse tier); tau: window queries
    sharpened or flattened per head by up to this factor; keep: mean share of the slots a
    rewrite keeps."""
    c = dict(name=name, kind=kind, NS=NS, Hq=Hq, Hkv=Hkv, D=D, dtype=dtype, N=N, lo=1.0,
             ragged=False, table=0, holes=0.0, W=32, p=0.9, tau=1.0, L_dense=0, L_sparse=0,
             n_ref=0, lse_in=False, keep_c=False, keep=0.5, L_upper=4096, L=1)
    c.update(more)
    return c


def listed():
    return [
        # one user's request decoding a compressed context: the launch-latency end
        _case("decode_one_sequence", "decode", 1, 32, 8, 128, "bf16", 1999, table=12288, lo=0.6,
              ragged=True, holes=0.2),
        # a batch at the end of its prompts: the largest plain decode launch (one layer)
        _case("decode_batch_full_rows", "decode", 64, 32, 8, 128, "bf16", 8192, table=12288),
        # a few long contexts with 7 query heads per KV head, before their first compression
        _case("decode_long_rows_g7", "decode", 4, 28, 4, 128, "bf16", 32761, lo=0.7, table=32768),
        # the steady state of a decode loop: compressed rows of every length, 4 layers
        _case("decode_loop_compressed", "loop", 256, 32, 8, 128, "bf16", 5600, L=4, lo=0.14,
              ragged=True, holes=0.1, table=12288),
        # the smallest compression: an fp32 cache of two heads, all stages
        _case("step_small_f32", "step", 1, 8, 2, 64, "f32", 2048, W=16),
        # one user's request reaching a compression point
        _case("select_one_sequence", "select", 1, 32, 8, 128, "bf16", 8187, tau=10.0, keep_c=True),
        # a small batch of long prompts
        _case("select_batch8_16k", "select", 8, 32, 8, 128, "bf16", 16384, p=0.95, tau=10.0),
        # a large batch of 32k contexts with 7 query heads per KV head: the headline compression
        _case("select_batch32_32k_g7", "select", 32, 28, 4, 128, "bf16", 32768, tau=10.0),
        # a compression inside the decode loop: the row LSEs come from the decode steps, the
        # rows are already compressed, the newest tokens stay dense; 2 layers of 64 sequences
        _case("select_decode_lse", "select", 128, 32, 8, 128, "bf16", 3100, lo=0.4, ragged=True,
              table=12288, L_dense=512, lse_in=True),
        # two metrics, dense and sparse tiers; 2 layers of 16 sequences
        _case("mixed_two_layers_16k", "mixed", 32, 32, 8, 128, "bf16", 16384, L_dense=512,
              L_sparse=2048, n_ref=256),
        # the rewrite of a large batch: budgets differ by head
        _case("rewrite_batch32_32k", "rewrite", 32, 28, 4, 128, "bf16", 32768, L_dense=512,
              L_sparse=2048, keep=0.6),
        # the hard budget over a large batch: every window row votes
        _case("budget_batch32_32k_g7", "budget", 32, 28, 4, 128, "bf16", 32768, tau=10.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "loop", "select", "select", "select", "mixed",
                       "rewrite", "rewrite", "step", "budget"])
    if kind == "step":
        Hkv, G, W = rng.choice([1, 2, 4]), rng.choice([1, 2, 4]), rng.choice([8, 16, 32])
        return _case("", "step", 1, Hkv * G, Hkv, rng.choice([64, 128]), "f32", _log(rng, 300, 4096), W=W,
                     p=round(rng.uniform(0.8, 0.95), 3))
    dtype = "bf16" if kind in ("mixed", "budget") or rng.random() < 0.85 else "f32"
    D = 128 if rng.random() < 0.75 else 64
    G = rng.choice([1, 2, 4, 4, 7, 8])
    Hkv = rng.choice([2, 4, 8])
    W = 32 if rng.random() < 0.7 else rng.choice([8, 16, 24])
    # slots (heads x tokens) at most: a drawn call costs no more than the largest listed ones
    most = {"decode": 1 << 22, "loop": 1 << 23, "select": 1 << 22, "mixed": 1 << 22,
            "rewrite": 1 << 22, "budget": 1 << 21}[kind]
    if dtype == "f32":
        most >>= 1 if kind in ("decode", "loop", "rewrite") else 4
    N = _log(rng, {"rewrite": 3000, "mixed": 2000}.get(kind, 500),
             {"select": 131072, "decode": 65536, "budget": 40000}.get(kind, 32768))
    NS = max(1, min(_log(rng, 1, 128), most // (N * Hkv)))
    table = rng.choice([0, 0, 12288, 32768])
    more = dict(W=W, lo=round(rng.uniform(0.2, 1.0), 2), ragged=rng.random() < 0.5,
                table=table if N <= table else 0)
    if kind in ("decode", "loop"):
        more.update(holes=rng.choice([0.0, 0.0, 0.3]))
        if kind == "loop":
            L = rng.choice([2, 3, 4])
            NS = L * max(1, min(NS, most // (N * Hkv)) // L)
            more.update(L=L)
    elif kind == "rewrite":
        more.update(keep=round(rng.uniform(0.05, 0.8), 2), L_dense=rng.choice([0, 512]),
                    L_sparse=rng.choice([0, 2048]))
    else:
        more.update(p=round(rng.uniform(0.8, 0.95), 3), tau=rng.choice([1.0, 10.0]))
        if kind == "select":
            more.update(keep_c=rng.random() < 0.5, lse_in=rng.random() < 0.3,
                        L_dense=rng.choice([0, 0, 512]))
        elif kind == "mixed":
            more.update(n_ref=rng.choice([64, 200, 256]), L_dense=512)
        else:
            more.update(L_upper=_log(rng, 512, 8192), L_dense=rng.choice([0, 512]))
    return _case("", kind, NS, Hkv * G, Hkv, D, dtype, N, **more)


# ---------------------------------------------------------------------------------- inputs
def _lens(case):
    """Row lengths, one per head: evenly spread over [lo * N, N] in golden-ratio order."""
    NS, Hkv, N, lo = case["NS"], case["Hkv"], case["N"], case["lo"]
    n = NS * Hkv if case["ragged"] else NS
    at = [N - int((1.0 - lo) * N * ((i * 0.6180339887498949) % 1.0)) for i in range(n)]
    return at if case["ragged"] else [x for x in at for _ in range(Hkv)]


def _randn(shape, gen, dtype):
    """N(0, 1) draws, made in pieces so that the fp32 draw of a large pool is never whole."""
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 28):
        piece = flat[i:i + (1 << 28)]
        piece.copy_(torch.randn(piece.shape, generator=gen, device="cuda"))
    return out


def _cache(case, gen):
    """A paged cache whose pages lie scattered over a pool with room for a rewrite, its
    allocator, and a copy of the buffer that holds both's metadata."""
    dev = "cuda"
    lens = torch.tensor(_lens(case), dtype=torch.int64, device=dev)
    H = lens.numel()
    n_pages = (lens + PAGE - 1) // PAGE
    width = max(int(n_pages.max()), -(-case["table"] // PAGE)) + (1 if case["kind"] == "loop" else 0)
    width += width % 2
    used = int(n_pages.sum())
    rewrites = case["kind"] in ("rewrite", "step")
    pool = used + (used if rewrites else used // 8) + H + 16
    perm = torch.randperm(pool, generator=gen, device=dev).to(torch.int32)
    slot = torch.arange(width, device=dev)[None, :]
    live = slot < n_pages[:, None]
    table = torch.full((H, width), -1, dtype=torch.int32, device=dev)
    table[live] = perm[:used]
    filled = (lens[:, None] - slot * PAGE).clamp(0, PAGE)
    mask = ((1 << filled) - 1) * live
    if case["holes"]:
        bits = torch.rand((H, width, PAGE), generator=gen, device=dev) >= case["holes"]
        keep = (bits.to(torch.int64) << torch.arange(PAGE, device=dev)).sum(-1)
        newest = slot == n_pages[:, None] - 1
        mask = torch.where(newest, mask, mask & keep)
    free = torch.zeros(pool, dtype=torch.int32, device=dev)
    free[:pool - used] = torch.sort(perm[used:]).values
    top = torch.tensor([pool - used], dtype=torch.int32, device=dev)
    parts = [table, mask.to(torch.int16), n_pages.to(torch.int32), free, top]
    at, total = [], 0
    for t in parts:
        at.append(total)
        total += -(-t.numel() * t.element_size() // 256) * 256
    meta = torch.zeros(total, dtype=torch.uint8, device=dev)
    views = []
    for t, o in zip(parts, at):
        v = meta[o:o + t.numel() * t.element_size()].view(t.dtype).view(t.shape)
        v.copy_(t)
        views.append(v)
    dt = DTYPE[case["dtype"]]
    k = _randn((pool, PAGE, case["D"]), gen, dt)
    v = _randn((pool, PAGE, case["D"]), gen, dt)
    kv = PagedKV(k, v, views[0], views[1], views[2])
    return dict(kv=kv, alloc=Allocator(views[3], views[4]), meta=meta, meta0=meta.clone())


def _queries(case, gen, W):
    NS, Hq, Hkv, D = case["NS"], case["Hq"], case["Hkv"], case["D"]
    q = torch.randn((W, NS, Hq, D), generator=gen, device="cuda")
    if case["tau"] > 1.0:
        u = torch.rand((NS, Hkv), generator=gen, device="cuda") * 2.0 - 1.0
        q /= torch.pow(torch.tensor(case["tau"], device="cuda"), u).repeat_interleave(Hq // Hkv, 1)[None, :, :, None]
    return q.to(DTYPE[case["dtype"]])


def _bits(mask, width):
    """[H, 16 * width] truth values of the page masks."""
    m = mask.to(torch.int32)[:, :width, None] >> torch.arange(PAGE, device=mask.device, dtype=torch.int32)
    return (m & 1).bool().reshape(mask.shape[0], -1)


def _rows(st, h, which="k"):
    """(rows [n_pages * 16, D], valid [n_pages * 16]) of one head, from the tables as they are."""
    kv = st["kv"]
    n = int(kv.n_pages[h])
    pool = kv.k_pool if which == "k" else kv.v_pool
    rows = pool[kv.page_table[h, :n].long()].reshape(-1, pool.shape[-1])
    return rows, _bits(kv.page_mask[h:h + 1], n)[0]


def _row_lse(case, st, q, dtype):
    """Log-sum-exp of every window row over its head's valid keys, [W, NS, Hq]."""
    NS, Hq, Hkv, D = case["NS"], case["Hq"], case["Hkv"], case["D"]
    G, W = Hq // Hkv, q.shape[0]
    out = torch.empty((W, NS, Hq), dtype=dtype, device="cuda")
    for h in range(NS * Hkv):
        s, g = h // Hkv, (h % Hkv) * G
        k, ok = _rows(st, h)
        z = q[:, s, g:g + G].reshape(-1, D).to(dtype) @ k.to(dtype).t() / math.sqrt(D)
        out[:, s, g:g + G] = torch.logsumexp(z.masked_fill(~ok, -math.inf), 1).view(W, G)
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    kind, NS, Hq, Hkv, D, W = (case[k] for k in ("kind", "NS", "Hq", "Hkv", "D", "W"))
    st = dict(kind=kind, **_cache(case, gen))
    kv, dt = st["kv"], DTYPE[case["dtype"]]
    f32 = dict(dtype=torch.float32, device="cuda")
    if kind == "decode":
        st["dec"] = Decoder(NS, Hq, Hkv, D, kv, st["alloc"])
        st["q"] = _queries(case, gen, 1)[0]
        st["o"], st["lse"] = torch.empty((NS, Hq, D), **f32), torch.empty((NS, Hq), **f32)
    elif kind == "loop":
        st["loop"] = DecodeLoop(case["L"], NS // case["L"], Hq, Hkv, D, W, kv, st["alloc"], case["p"],
                                case["L_dense"], keep_c=False)
        st["q"] = _queries(case, gen, 1)[0]
        st["k_new"], st["v_new"] = (torch.randn((NS, Hkv, D), generator=gen, device="cuda").to(dt) for _ in "kv")
        st["lse"] = torch.empty((NS, Hq), **f32)
    elif kind == "budget":
        st["comp"] = BudgetCompressor(NS, Hq, Hkv, D, W, kv, st["alloc"], case["p"], case["L_upper"] // 2,
                                      case["L_upper"], L_dense=case["L_dense"], n_sink=4)
        st["q"] = _queries(case, gen, W)
    else:
        comp = st["comp"] = Compressor(NS, Hq, Hkv, D, W, kv, st["alloc"], case["p"], L_dense=case["L_dense"],
                                       L_sparse=case["L_sparse"], metric="attn+red" if kind == "mixed" else "attn",
                                       n_ref=case["n_ref"], keep_c=case["keep_c"])
        if kind == "rewrite":
            # the selection of a head keeps its own share of the slots
            H, S = comp.n_heads, comp.S_max
            share = torch.rand((H, 1), generator=gen, device="cuda") * 2.0 * case["keep"]
            word = torch.zeros((H, S // 32), dtype=torch.int64, device="cuda")
            for b in range(32):
                word |= (torch.rand((H, S // 32), generator=gen, device="cuda") < share).to(torch.int64) << b
            comp.buf.sel_bits.copy_(torch.where(word >= 1 << 31, word - (1 << 32), word))
        else:
            st["q"] = _queries(case, gen, W)
            st["lse_in"] = _row_lse(case, st, st["q"], torch.float32) if case["lse_in"] else None
        if kind == "mixed":
            H, mp = kv.page_mask.shape
            key = torch.rand((H, mp * PAGE), generator=gen, device="cuda").masked_fill(~_bits(kv.page_mask, mp), -1.0)
            least = min(_lens(case))
            comp.n_ref = min(case["n_ref"], least)
            st["ref"] = torch.sort(torch.topk(key, comp.n_ref, dim=1).indices, dim=1).values.to(torch.int32)
            # the redundancy temperature is solved once per head, at the first compression
            comp.score(st["q"], ref_slots=st["ref"])
            comp.select()
    return st


def run(st):
    kind, kv, alloc = st["kind"], st["kv"], st["alloc"]
    if kind in ("loop", "rewrite", "step"):
        st["meta"].copy_(st["meta0"])
    tables = dict(page_table=kv.page_table, page_mask=kv.page_mask, n_pages=kv.n_pages,
                  free_ids=alloc.free_ids, free_top=alloc.free_top, k_pool=kv.k_pool, v_pool=kv.v_pool)
    if kind == "decode":
        st["dec"].attend(st["q"], st["o"], st["lse"])
        return dict(o=st["o"], lse=st["lse"])
    if kind == "loop":
        loop = st["loop"]
        loop.step(st["q"], st["k_new"], st["v_new"], st["lse"])
        return dict(o=loop.o, lse=st["lse"], status=loop.status, **tables)
    comp, b = st["comp"], st["comp"].buf
    if kind == "budget":
        comp.select(st["q"])
        return {k: b[k] for k in ("row_lse", "votes", "sel_bits", "k", "head_mode", "k_cap", "cand_len", "status")}
    if kind == "rewrite":
        comp.compact()
        return dict(status=b.status, **tables)
    if kind == "step":
        comp.step(st["q"])
        return dict(s_attn=b.s_attn, row_lse=b.row_lse, sel_bits=b.sel_bits, k=b.k, status=b.status, **tables)
    comp.score(st["q"], ref_slots=st.get("ref"), row_lse_in=st["lse_in"])
    comp.select()
    out = dict(s_attn=b.s_attn, cand_len=b.cand_len, sel_bits=b.sel_bits, k=b.k, status=b.status)
    if st["lse_in"] is None:
        out["row_lse"] = b.row_lse
    if comp.keep_c:
        out["c"] = b.c
    if kind == "mixed":
        out["x_red"] = b.x_red
    return out


# ------------------------------------------------------------------------- what it must cost
def _cond(case, n):
    """Pages of a row of n pages before the dense and the sparse tier."""
    nd = min(n, -(-case["L_dense"] // PAGE))
    return n - nd - min(n - nd, case["L_sparse"] // PAGE)


def work(case):
    kind, Hq, Hkv, D, W = (case[k] for k in ("kind", "Hq", "Hkv", "D", "W"))
    e = 4 if case["dtype"] == "f32" else 2
    G, H, lens = Hq // Hkv, case["NS"] * Hkv, _lens(case)
    pages = [-(-n // PAGE) for n in lens]
    width = max(max(pages), -(-case["table"] // PAGE))
    S, slots = width * PAGE, sum(lens)
    heads = 6 * sum(pages)                            # live table and mask entries
    valid = slots * (1.0 - case["holes"])
    if kind in ("decode", "loop"):
        rows = case["NS"] * Hq
        new = 4 * H * D * e if kind == "loop" else 0  # k, v of the step, read and written
        return dict(bytes=2 * valid * D * e + rows * (D * (e + 4) + 4) + heads + new, flops=4 * valid * G * D)
    moved = sum(min(n, _cond(case, g) * PAGE) for n, g in zip(lens, pages)) * 4 * D * e * case["keep"]
    if kind == "rewrite":
        return dict(bytes=moved + 2 * heads + H * S // 8, flops=0)
    R = G * W
    b = slots * D * e + case["NS"] * W * Hq * (D * e + 4) + heads + H * S * 4 + H * S // 8
    f = 2 * R * slots * D
    if kind == "mixed":
        b, f = b + H * S * 4, f + 2 * case["n_ref"] * slots * D
    if kind == "budget":
        b -= H * S * 2                                # votes are 16 bits, scores 32
    if kind == "step":
        b += moved * 1.6                              # p near 0.9 of the mass keeps about 4 of 5 slots
    if case["keep_c"]:
        b += H * S * 4
    return dict(bytes=b, flops=f)


def tolerance(case):
    """About four times the error of the computed outputs against 64 bits: 2.4e-7 for attention
    outputs, 9e-8 for log scores, 1.6e-6 for calibrated probabilities (a relative error there is
    an absolute one of a log score).  A slot at the Top-p threshold can fall on either side, so a
    few words of a selection bitmap, counts or votes may differ; a rewrite moves bytes."""
    if case["kind"] == "rewrite":
        return "exact"
    if case["kind"] in ("decode", "loop"):
        return {"rel": 1e-6, "max": 4e-5}
    return {"rel": 8e-6 if case["keep_c"] else 1e-6, "max": 1e-4, "differ": 1e-3}


# ------------------------------------------------------------------------- in 64 bits
def exact(case, seed):
    kind, NS, Hq, Hkv, D = (case[k] for k in ("kind", "NS", "Hq", "Hkv", "D"))
    if kind == "rewrite":
        return None
    st = prepare(case, seed)
    kv, G, d = st["kv"], Hq // Hkv, torch.float64
    q = st["q"]
    if kind in ("decode", "loop"):
        o = torch.zeros((NS, Hq, D), dtype=d, device="cuda")
        lse = torch.full((NS, Hq), -math.inf, dtype=d, device="cuda")
        for h in range(NS * Hkv):
            s, g = h // Hkv, (h % Hkv) * G
            (k, ok), (v, _) = _rows(st, h), _rows(st, h, "v")
            k, v = k[ok].to(d), v[ok].to(d)
            if kind == "loop":
                k = torch.cat([k, st["k_new"][s, h % Hkv][None].to(d)])
                v = torch.cat([v, st["v_new"][s, h % Hkv][None].to(d)])
            z = q[s, g:g + G].to(d) @ k.t() / math.sqrt(D)
            lse[s, g:g + G] = torch.logsumexp(z, 1)
            o[s, g:g + G] = torch.softmax(z, 1) @ v
        names = () if kind == "decode" else ("status", "page_table", "page_mask", "n_pages", "free_ids", "free_top",
                                             "k_pool", "v_pool")
        return dict(o=o, lse=lse, **dict.fromkeys(names))
    lse = st.get("lse_in")
    given = lse is not None
    lse = lse.to(d) if given else _row_lse(case, st, q, d)
    if kind == "budget":
        return dict(row_lse=lse, votes=None, sel_bits=None, k=None, head_mode=None, k_cap=None, cand_len=None, status=None)
    H, S, W = NS * Hkv, kv.max_pages * PAGE, q.shape[0]
    sa = torch.full((H, S), -math.inf, dtype=d, device="cuda")
    x = sa.clone() if kind == "mixed" else None
    for h in range(H):
        s, g = h // Hkv, (h % Hkv) * G
        k, ok = _rows(st, h)
        n = max(0, int(kv.n_pages[h]) - -(-case["L_dense"] // PAGE)) * PAGE
        k = k.to(d)
        z = q[:, s, g:g + G].reshape(-1, D).to(d) @ k[:n].t() / math.sqrt(D)
        z = torch.logsumexp(z - lse[:, s, g:g + G].reshape(-1, 1), 0) - math.log(G * W)
        sa[h, :n] = z.masked_fill(~ok[:n], -math.inf)
        if kind == "mixed":
            ref = st["ref"][h].long()
            norm = k.norm(dim=1)
            cos = (k[:n] / norm[:n, None]) @ (k[ref] / norm[ref, None]).t()
            cos.masked_fill_(torch.arange(n, device="cuda")[:, None] == ref[None, :], -math.inf)
            x[h, :n] = (-cos.amax(1)).masked_fill(~ok[:n], -math.inf)
    out = dict(s_attn=sa, cand_len=None, sel_bits=None, k=None, status=None)
    if not given:
        out["row_lse"] = lse
    if kind == "mixed":
        out["x_red"] = x
    if case["keep_c"]:
        out["c"] = torch.softmax(sa, 1).nan_to_num(0.0)   # a head without candidates: 0
    if kind == "step":
        del out["cand_len"]
        out.update(dict.fromkeys(("page_table", "page_mask", "n_pages", "free_ids", "free_top", "k_pool", "v_pool")))
    return out
