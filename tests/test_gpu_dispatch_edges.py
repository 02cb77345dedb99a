"""Edges of the kernels' launch rules on the GPU: the sizes where a launch changes shape
(splits per row, rows per workgroup, chunk lengths), against the CPU oracle."""
import math

import pytest
import torch

import oracle as O
import workload as WL
from hk_testlib import RTOL, HostCache, check_lse, check_prob, np64

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _decode_against_oracle(cfg, lens, max_pages, hole_prob=0.1, n_split=None, q_scale=2.0):
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
    host = HostCache(w.k_pool, w.v_pool, w.page_table, w.page_mask, w.n_pages)
    qn, on, ln = np64(q), np64(o), np64(lse)
    G, rtol = cfg["Hq"] // cfg["Hkv"], RTOL[cfg["dtype"]]
    for h in range(w.n_heads):
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
