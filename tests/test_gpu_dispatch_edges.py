"""Edges of the kernels' launch rules on the GPU: the sizes where a launch changes shape
(splits per row, rows per workgroup, chunk lengths), against the CPU oracle."""
import math

import numpy as np
import pytest
import torch

import oracle as O
import workload as WL
from hk_testlib import RTOL, HostCache, check_lse, check_log_scores, check_prob, np64, q_rows, unpack_bits

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _decode_against_oracle(cfg, lens, max_pages, hole_prob=0.1, n_split=None, q_scale=2.0, heads=None):
    import paper_2606_28831_amd as hk
    w = WL.make_workload(cfg, DEV, hole_prob=hole_prob, head_lens=lens, max_pages=max_pages)
    kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    d = hk.dims(w.NS, cfg["Hq"], cfg["Hkv"], cfg["D"])
    if n_split is not None:
        assert hk.hk_decode_plan(d, w.max_pages)[0] == n_split
    gen = torch.Generator(device=DEV).manual_seed(31)
    q = (torch.randn(w.NS, cfg["Hq"], cfg["D"], generator=gen, device=DEV) * q_scale).to(w.k_pool.dtype)
    o = torch.full((w.NS, cfg["Hq"], cfg["D"]), float("nan"), device=DEV)
    lse = torch.full((w.NS, cfg["Hq"]), float("nan"), device=DEV)
    scale = 1 / math.sqrt(cfg["D"])
    ws = hk.workspace(hk.OP_DECODE, d, w.max_pages, DEV)
    ws.fill_(255)                      # NaN in every float an idle split leaves unwritten
    hk.hk_decode_attn(d, q, kv, scale, o, lse, ws)
    torch.cuda.synchronize()
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages, heads=heads)
    qn, on, ln = np64(q), np64(o), np64(lse)
    G, rtol = cfg["Hq"] // cfg["Hkv"], RTOL[cfg["dtype"]]
    for h in range(w.n_heads) if heads is None else heads:
        s, kvh = divmod(h, cfg["Hkv"])
        K, valid = host.head(h)
        V, _ = host.head_v(h)
        ref_o, ref_l = O.decode_head(qn[s, kvh * G:(kvh + 1) * G], K, V, valid, scale)
        for g in range(G):
            check_prob(on[s, kvh * G + g], ref_o[g], rtol, f"o head {h} g {g}")
        check_lse(ln[s, kvh * G:(kvh + 1) * G], ref_l, rtol, f"lse head {h}")


# splits per row: 1, the most one wave per query head merges (8), one more, several loads of
# the four-wave form; query heads that are no multiple of the four a workgroup merges
@pytest.mark.parametrize("D,G,dtype,pages", [(128, 7, "bf16", 16), (64, 1, "f32", 128), (64, 7, "bf16", 144),
                                             (128, 1, "bf16", 144), (128, 2, "f32", 560), (64, 8, "bf16", 600)])
def test_decode_merge_shapes(D, G, dtype, pages):
    cfg = dict(L=1, B=3, Hq=G, Hkv=1, D=D, N=pages * 16, dtype=dtype, W=8, seed=41, recipe="normal")
    _decode_against_oracle(cfg, [pages * 16, 0, pages * 8 + 5], pages, n_split=-(-pages // 16))


# more query heads than the merge gives four waves each: one wave at 9 to 32 splits, four above
@pytest.mark.parametrize("D,dtype,pages", [(128, "bf16", 1156), (64, "f32", 1156), (64, "bf16", 4096),
                                           (128, "bf16", 4228)])
def test_decode_merge_many_heads(D, dtype, pages):
    H = 1030
    cfg = dict(L=1, B=H, Hq=1, Hkv=1, D=D, N=pages * 16, dtype=dtype, W=8, seed=71, recipe="normal")
    lens = [(i * 37) % 301 for i in range(H)]            # some of no page at all
    lens[5], lens[77], lens[500], lens[H - 1] = 18000, 16 * pages, 4100, 9 * 128 * 16 + 1
    heads = [0, 1, 5, 77, 255, 500, 511, 512, H - 2, H - 1]
    _decode_against_oracle(cfg, lens, pages, n_split=-(-pages // 128), heads=heads)


# the second pass's chunks of 16 pages up to 128: few rows take short ones; rows that end before,
# at and past a chunk's edge, or hold nothing.  A workspace below the size asked for is refused.
@pytest.mark.parametrize("D,G,dtype,pages,lens", [
    (64, 4, "f32", 130, [2080, 256, 257, 0]), (128, 4, "bf16", 130, [2080, 255, 16, 1]),
    (128, 7, "bf16", 40, [640, 512, 513, 300]), (64, 8, "bf16", 66, [1056, 1, 1024, 1025])])
def test_score_chunk_lengths(D, G, dtype, pages, lens):
    import paper_2606_28831_amd as hk
    W, NS, Hkv = 16, 2, 2
    cfg = dict(L=1, B=NS, Hq=Hkv * G, Hkv=Hkv, D=D, N=pages * 16, dtype=dtype, W=W, seed=43, recipe="normal")
    w = WL.make_workload(cfg, DEV, hole_prob=0.1, head_lens=lens, max_pages=pages)
    kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    d = hk.dims(NS, Hkv * G, Hkv, D, W)
    H = NS * Hkv
    ws = hk.workspace(hk.OP_SCORE, d, w.max_pages, DEV)
    ws.fill_(255)
    s = torch.full((H, w.S_max), 7.0, device=DEV)
    cl = torch.empty(H, dtype=torch.int32, device=DEV)
    lse = torch.empty(W, NS, Hkv * G, device=DEV)
    scale = 1 / math.sqrt(D)
    hk.hk_score(d, w.q_obs, kv, 48, scale, s, cl, row_lse_out=lse, ws=ws)
    with pytest.raises(hk.HardKVError):
        hk.hk_score(d, w.q_obs, kv, 48, scale, s, cl, row_lse_out=lse, ws=ws[:ws.numel() - 256])
    torch.cuda.synchronize()
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    qn, sn, ln, rtol = np64(w.q_obs), np64(s), np64(lse), RTOL[dtype]
    for h in range(H):
        sq, kvh = divmod(h, Hkv)
        K, valid = host.head(h)
        n_cand = 16 * max(0, int(w.n_pages[h]) - 3)
        assert int(cl[h]) == n_cand
        ref_s, ref_l = O.score_head(q_rows(qn, h, Hkv, G), K, valid, n_cand, scale)
        full = np.full(w.S_max, -np.inf)
        full[:len(ref_s)] = ref_s
        check_log_scores(sn[h], full, rtol, f"s head {h}")
        check_lse(ln[:, sq, kvh * G:(kvh + 1) * G].reshape(-1), ref_l, rtol, f"lse head {h}")


# more workgroups than run at once: chunks past a row's candidates are skipped, and rows of up
# to 12288 slots in more heads than CUs finish in 512-thread workgroups; row ends at, before
# and past a 2048-slot chunk's edge, ties at the threshold
@pytest.mark.parametrize("H,S", [(400, 12288), (300, 12320), (257, 16384), (700, 6176)])
@pytest.mark.parametrize("ties", [False, True])
def test_wide_select_skips_dead_chunks(H, S, ties):
    import paper_2606_28831_amd as hk
    gen = torch.Generator(device=DEV).manual_seed(H + S)
    ends = torch.tensor([0, 1, 2047, 2048, 2049, 4096, S - 1, S, 16], device=DEV)
    cl = ends[torch.arange(H, device=DEV) % len(ends)].to(torch.int32)
    x = torch.randn((H, S), generator=gen, device=DEV) * 2
    if ties:
        x = x.round()
    mask = torch.randint(-2 ** 15, 2 ** 15, (H, S // 16), generator=gen, device=DEV).to(torch.int16)
    mask[:, ::3] = -1
    new = lambda *s, dtype=torch.float32: torch.full(s, 7, dtype=dtype, device=DEV)
    c1, c2, l1, l2 = new(H, S), new(H, S), new(H, 1), new(H, 1)
    bits = [new(H, S // 32, dtype=torch.int32) for _ in range(2)]
    k = [new(H, dtype=torch.int32) for _ in range(2)]
    m = [new(H) for _ in range(2)]
    ws = hk.select_workspace(H, S, DEV)
    ws.fill_(255)
    hk.hk_calibrate_topp_ws(H, S, cl, mask, [x], None, [1.0], 0.9, bits[0], k[0], ws, c_out=c1, lse_out=l1,
                            sel_mass=m[0])
    hk.hk_calibrate(H, S, cl, mask, [x], None, [1.0], c2, lse_out=l2)
    torch.cuda.synchronize()
    none = torch.isneginf(l2)
    assert torch.equal(none, torch.isneginf(l1))
    torch.testing.assert_close(l1[~none], l2[~none], rtol=1e-6, atol=2e-6)
    torch.testing.assert_close(c1, c2, rtol=1e-5, atol=0)      # 2e-6 of a log-sum-exp near 10
    # the selection of the c it computed, bit for bit, by the single-workgroup selector
    hk.hk_topp_select(H, S, cl, mask, c1, 0.9, bits[1], k[1], sel_mass=m[1])
    torch.cuda.synchronize()
    assert torch.equal(bits[0], bits[1]) and torch.equal(k[0], k[1]) and torch.equal(m[0], m[1])
    ws.fill_(255)
    bits[0].fill_(7)
    hk.hk_topp_select_ws(H, S, cl, mask, c1, 0.9, bits[0], k[0], ws, sel_mass=m[0], k_max=900)
    hk.hk_topp_select(H, S, cl, mask, c1, 0.9, bits[1], k[1], sel_mass=m[1], k_max=900)
    torch.cuda.synchronize()
    assert torch.equal(bits[0], bits[1]) and torch.equal(k[0], k[1]) and torch.equal(m[0], m[1])


def _vote_row(kind, n, rng):
    if kind == "no_weight":                        # every value below 2^-40: nothing to reach
        return np.exp2(-41.0 - rng.integers(0, 4, n)).astype(np.float32)
    if kind == "around_weight":                    # both sides of 2^-40, the smallest weight
        return np.exp2(-36.0 - 8.0 * rng.random(n)).astype(np.float32)
    if kind == "peak":                             # one value of most of the mass, a long tail
        a = np.exp2(-10.0 - 60.0 * rng.random(n)).astype(np.float32)
        a[rng.integers(0, n)] = 0.75
        return a
    if kind == "binades":                          # both sides of 2^-8, where weights take a second half
        return (np.exp2(-6.0 - 4.0 * rng.random(n))).astype(np.float32)
    # one digit of the first round holds nearly every key (more than a wave's list), others far away
    a = np.float32(2.0 ** -12) * (1.0 + rng.integers(0, 1 << 10, n) * np.float32(2.0 ** -22))
    a[:: max(1, n // 40)] = 2.0 ** -30
    a[0] = 0.5
    return a.astype(np.float32)


@pytest.mark.parametrize("S", [96, 8192, 32768, 40960])
@pytest.mark.parametrize("kind", ["no_weight", "around_weight", "peak", "binades", "one_digit"])
def test_vote_rows_weights_and_lists(kind, S):
    import paper_2606_28831_amd as hk
    rng = np.random.default_rng(S)
    H, R, p = 4, 2, 0.9
    cl = np.array([S, S - 5, S // 3, 0], np.int32)
    mask = np.full((H, S // 16), 0xFFFF, np.int64)
    mask[1, ::5] = 0x7FFE
    a = np.empty((H, R, S), np.float32)
    a[:, :, ::2], a[:, :, 1::2] = np.nan, 5.0      # what is no candidate is not looked at
    cand = [O.candidate_mask(((mask[h][:, None] >> np.arange(16)) & 1).reshape(-1).astype(bool), int(cl[h]))
            for h in range(H)]
    for h in range(H):
        for r in range(R):
            if cand[h].any():
                a[h, r, cand[h]] = _vote_row(kind, int(cand[h].sum()), rng)
    votes = torch.full((H, S), 7, dtype=torch.int16, device=DEV)
    row_sel = torch.full((H, R, S // 32), 7, dtype=torch.int32, device=DEV)
    row_k = torch.empty(H, R, dtype=torch.int32, device=DEV)
    st = torch.zeros(1, dtype=torch.int32, device=DEV)
    hk.hk_vote_topp(H, R, S, torch.tensor(cl, device=DEV),
                    torch.tensor(mask.astype(np.uint16).view(np.int16), device=DEV), torch.tensor(a, device=DEV), p,
                    votes, row_sel, row_k=row_k, status=st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    got = row_sel.cpu().numpy()
    for h in range(H):
        ref_v, ref_k, ref_sel = O.vote_head(np.where(cand[h], a[h], 0), cand[h], p)
        for r in range(R):
            assert int(row_k[h, r]) == ref_k[r], (kind, h, r)
            assert np.array_equal(unpack_bits(got[h, r], S), ref_sel[r]), (kind, h, r)
        assert np.array_equal(votes[h].cpu().numpy().astype(np.int64) & 0xFFFF, ref_v), (kind, h)


# pairs of pages per wave: odd page counts, a last page alone, one slot, ranges that leave waves
# without a pair; every group size; scores that climb by far more than 2^16 from page to page (a
# new reference each time) and fall by as much
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("G", [1, 2, 4, 7, 8])
def test_decode_bf16_page_pairs(D, G):
    cfg = dict(L=1, B=6, Hq=G, Hkv=1, D=D, N=33 * 16, dtype="bf16", W=8, seed=47, recipe="normal")
    _decode_against_oracle(cfg, [33 * 16, 16 * 16 + 1, 1, 17 * 16, 3 * 16 - 1, 0], 34)


@pytest.mark.parametrize("G", [4, 7])
def test_decode_bf16_extreme_scores(G):
    import paper_2606_28831_amd as hk
    D, pages, H = 128, 20, 4
    cfg = dict(L=1, B=H, Hq=G, Hkv=1, D=D, N=pages * 16, dtype="bf16", W=8, seed=53, recipe="normal")
    w = WL.make_workload(cfg, DEV, max_pages=pages)
    n = pages * 16
    gen = torch.Generator(device=DEV).manual_seed(53)
    step = torch.arange(n, device=DEV, dtype=torch.float32)
    gain = torch.stack([step * 0.2, (n - step) * 0.2, torch.where(step % 37 == 0, 60.0, -60.0), step * 0])
    u = torch.ones(D, device=DEV)
    for h in range(H):
        k = (torch.randn(n, D, generator=gen, device=DEV) * 0.1 + gain[h][:, None] * u / D ** 0.5).to(torch.bfloat16)
        w.k_pool[w.page_table[h].long()] = k.view(pages, 16, D)
    w.v_pool[w.page_table[3, 3].long(), 5, 7] = float("inf")      # a key of every weight but 0
    kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    d = hk.dims(H, G, 1, D)
    q = (torch.randn(H, G, D, generator=gen, device=DEV) * 0.1 + u).to(torch.bfloat16)
    o, lse = torch.empty(H, G, D, device=DEV), torch.empty(H, G, device=DEV)
    hk.hk_decode_attn(d, q, kv, 1 / math.sqrt(D), o, lse, hk.workspace(hk.OP_DECODE, d, w.max_pages, DEV))
    torch.cuda.synchronize()
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    for h in range(H):
        K, valid = host.head(h)
        V, _ = host.head_v(h)
        on = np64(o[h])
        if h == 3:
            assert np.all(np.isposinf(on[:, 7]))
            V = np.where(np.isinf(V), 0.0, V)
            on[:, 7] = 0.0
        ref_o, ref_l = O.decode_head(np64(q[h]), K, V, valid, 1 / math.sqrt(D))
        if h == 3:
            ref_o[:, 7] = 0.0
        for g in range(G):
            check_prob(on[g], ref_o[g], RTOL["bf16"], f"o head {h} g {g}")
        check_lse(np64(lse[h]), ref_l, RTOL["bf16"], f"lse head {h}")


# Values near the end of the fp32 range: their sums hold against the largest score of a row, also
# where that score comes late and lies above the earlier ones by less than 2^16; beside them a head
# of ordinary values.
@pytest.mark.parametrize("D,G", [(64, 7), (128, 4)])
def test_decode_bf16_large_values(D, G):
    import paper_2606_28831_amd as hk
    pages, H = 20, 3
    cfg = dict(L=1, B=H, Hq=G, Hkv=1, D=D, N=pages * 16, dtype="bf16", W=8, seed=59, recipe="normal")
    w = WL.make_workload(cfg, DEV, max_pages=pages)
    n = pages * 16
    gen = torch.Generator(device=DEV).manual_seed(59)
    late = torch.zeros(n, device=DEV)
    late[139:] = 10.0                                   # e^10 = 2^14.4 times the weight of the others
    for h, big in enumerate([2.0 ** 118, 2.0 ** 110, 1.0]):
        k = (torch.randn(n, D, generator=gen, device=DEV) * 0.05 + late[:, None] / D).to(torch.bfloat16)
        v = (big * (1.0 + torch.rand(n, D, generator=gen, device=DEV))).to(torch.bfloat16)
        w.k_pool[w.page_table[h].long()] = k.view(pages, 16, D)
        w.v_pool[w.page_table[h].long()] = v.view(pages, 16, D)
    kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    d = hk.dims(H, G, 1, D)
    q = torch.ones(H, G, D, device=DEV).to(torch.bfloat16)
    o, lse = torch.empty(H, G, D, device=DEV), torch.empty(H, G, device=DEV)
    hk.hk_decode_attn(d, q, kv, 1.0, o, lse, hk.workspace(hk.OP_DECODE, d, w.max_pages, DEV))
    torch.cuda.synchronize()
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    for h in range(H):
        K, valid = host.head(h)
        V, _ = host.head_v(h)
        ref_o, ref_l = O.decode_head(np64(q[h]), K, V, valid, 1.0)
        for g in range(G):
            check_prob(np64(o[h])[g], ref_o[g], RTOL["bf16"], f"o head {h} g {g}")
        check_lse(np64(lse[h]), ref_l, RTOL["bf16"], f"lse head {h}")


# Infinite values give infinite sums, also in the last page of an odd number of pages (which the
# pair of pages repeats with an empty mask), beside sums that stay finite and ones that are large.
@pytest.mark.parametrize("D,G", [(64, 1), (128, 7)])
@pytest.mark.parametrize("n_pages", [1, 2, 5, 7, 15, 17, 33])
def test_decode_bf16_infinite_values_last_page(D, G, n_pages):
    import paper_2606_28831_amd as hk
    H, n = 2, n_pages * 16 - 3                          # the last page holds 13 slots
    cfg = dict(L=1, B=H, Hq=G, Hkv=1, D=D, N=n, dtype="bf16", W=8, seed=61, recipe="normal")
    w = WL.make_workload(cfg, DEV, head_lens=[n, n], max_pages=34)
    last = w.page_table[:, n_pages - 1].long()
    w.v_pool[last, 4, 7] = float("inf")
    w.v_pool[last[0], 12, 9] = float("-inf")
    w.v_pool[last[1], 2, 11] = 2.0 ** 126
    kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    d = hk.dims(H, G, 1, D)
    gen = torch.Generator(device=DEV).manual_seed(61)
    q = torch.randn(H, G, D, generator=gen, device=DEV).to(torch.bfloat16)
    o, lse = torch.empty(H, G, D, device=DEV), torch.empty(H, G, device=DEV)
    hk.hk_decode_attn(d, q, kv, 1 / math.sqrt(D), o, lse, hk.workspace(hk.OP_DECODE, d, w.max_pages, DEV))
    torch.cuda.synchronize()
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    for h in range(H):
        K, valid = host.head(h)
        V, _ = host.head_v(h)
        on, inf = np64(o[h]), np.isinf(V).any(0)
        assert np.all(np.isposinf(on[:, 7])) and (h == 1 or np.all(np.isneginf(on[:, 9])))
        ref_o, ref_l = O.decode_head(np64(q[h]), K, np.where(np.isinf(V), 0.0, V), valid, 1 / math.sqrt(D))
        large = np.abs(ref_o[0]) > 1e30                  # its own scale: the others are near 1
        for g in range(G):
            check_prob(on[g][~inf & ~large], ref_o[g][~inf & ~large], RTOL["bf16"], f"o head {h} g {g}")
            check_prob(on[g][large], ref_o[g][large], RTOL["bf16"], f"large o head {h} g {g}")
        check_lse(np64(lse[h]), ref_l, RTOL["bf16"], f"lse head {h}")


# A head's row LSEs, log scores and redundancy are the same bits whoever shares its launch (few
# heads take shorter chunks in the second pass) and however much workspace there is, its row LSEs
# also whether or not the redundancy is asked for.
@pytest.mark.parametrize("D,G,dtype,pages", [(128, 4, "bf16", 520), (64, 7, "bf16", 300), (64, 2, "f32", 160)])
def test_score_of_a_head_does_not_depend_on_the_batch(D, G, dtype, pages):
    import paper_2606_28831_amd as hk
    W, NS, Hkv, n_ref = 8, 26, 2, 33
    lens = [pages * 16 - 37 * (i % 11) for i in range(NS * Hkv)]
    cfg = dict(L=1, B=NS, Hq=Hkv * G, Hkv=Hkv, D=D, N=pages * 16, dtype=dtype, W=W, seed=67, recipe="normal")
    w = WL.make_workload(cfg, DEV, head_lens=lens, max_pages=pages)
    ref = (torch.arange(n_ref, device=DEV, dtype=torch.int32) * (min(lens) // n_ref)).expand(NS * Hkv, n_ref)

    def score(seqs, red, more_ws=0):
        n, H = len(seqs), len(seqs) * Hkv
        rows = slice(seqs[0] * Hkv, (seqs[-1] + 1) * Hkv)
        kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table[rows].clone(), w.page_mask[rows].clone(),
                        w.n_pages[rows].clone())
        d = hk.dims(n, Hkv * G, Hkv, D, W)
        ws = hk.workspace(hk.OP_SCORE, d, w.max_pages, DEV)
        ws = torch.full((ws.numel() + more_ws,), 255, dtype=torch.uint8, device=DEV)
        s, x = (torch.full((H, w.S_max), 7.0, device=DEV) for _ in "sx")
        cl, lse = torch.empty(H, dtype=torch.int32, device=DEV), torch.empty(W, n, Hkv * G, device=DEV)
        more = dict(ref_slots=ref[rows].contiguous(), n_ref=n_ref, x_red=x) if red else {}
        hk.hk_score(d, w.q_obs[:, seqs[0]:seqs[-1] + 1].contiguous(), kv, 48, 1 / math.sqrt(D), s, cl,
                    row_lse_out=lse, ws=ws, **more)
        torch.cuda.synchronize()
        return s, lse, x

    all_of = {red: score(range(NS), red) for red in (False, True)}
    for seqs in (range(NS), range(3), range(17, 18)):
        rows, at = slice(seqs[0] * Hkv, (seqs[-1] + 1) * Hkv), slice(seqs[0], seqs[-1] + 1)
        for red, more_ws in ((True, 0), (False, 0), (False, 1 << 24)):
            s, lse, x = score(seqs, red, more_ws)
            assert all(torch.equal(lse, a[1][:, at]) for a in all_of.values()), (list(seqs), red, more_ws)
            assert torch.equal(s, all_of[red][0][rows]) and torch.equal(x, all_of[red][2][rows])


# The redundancy pass takes shorter chunks with few heads (2 x 2) and 512-page ones where every CU
# has a workgroup (64 x 4).
@pytest.mark.parametrize("NS,Hkv,pages", [(2, 2, 520), (64, 4, 34)])
def test_redundancy_chunk_lengths(NS, Hkv, pages):
    import paper_2606_28831_amd as hk
    D, G, W, n_ref = 64, 2, 8, 33
    H, least = NS * Hkv, pages * 16 - 40
    lens = [pages * 16 - 8 * (i % 6) for i in range(H)]
    cfg = dict(L=1, B=NS, Hq=Hkv * G, Hkv=Hkv, D=D, N=pages * 16, dtype="bf16", W=W, seed=47, recipe="normal")
    w = WL.make_workload(cfg, DEV, head_lens=lens, max_pages=pages)
    kv = hk.PagedKV(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    d = hk.dims(NS, Hkv * G, Hkv, D, W)
    ref = (torch.arange(n_ref, device=DEV, dtype=torch.int32) * (least // n_ref)).expand(H, n_ref).contiguous()
    s, x = (torch.full((H, w.S_max), 7.0, device=DEV) for _ in "sx")
    cl, lse = torch.empty(H, dtype=torch.int32, device=DEV), torch.empty(W, NS, Hkv * G, device=DEV)
    hk.hk_score(d, w.q_obs, kv, 48, 1 / math.sqrt(D), s, cl, row_lse_out=lse, ref_slots=ref, n_ref=n_ref, x_red=x,
                ws=hk.workspace(hk.OP_SCORE, d, w.max_pages, DEV))
    torch.cuda.synchronize()
    x = np64(x)
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    for h in (0, H - 1):
        K, valid = host.head(h)
        n = 16 * (int(w.n_pages[h]) - 3)
        K = np.asarray(K, np.float64) / np.linalg.norm(K, axis=1, keepdims=True).clip(1e-30)
        r = ref[h].cpu().numpy()
        cos = K[:n] @ K[r].T
        cos[r[r < n], np.nonzero(r < n)[0]] = -np.inf
        # bf16 products are exact, fp32 sums over D and an fp32 norm: 1e-5 absolute on a cosine
        assert np.abs(x[h, :n] + cos.max(1))[valid[:n].astype(bool)].max() < 1e-5
        assert np.isneginf(x[h, n:]).all()
