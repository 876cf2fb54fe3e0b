"""fp32 attention and state at the edges of their tiles, pieces and pointers:
64-query blocks, 32-key tiles (the window at a page's end, pages shorter than a tile),
items cut into pieces or not (by the scratch the workspace leaves), operands
aligned to 4 bytes only, and infinite values. Against the fp64 oracle with the
repository's fp32 bar."""
import numpy as np
import pytest

from synth_inputs import make_case
from synth_inputs.configs import Workload

from hsa_testlib import F32_TOL, assert_close, run_oracle, say, to_host, upload

pytestmark = pytest.mark.gpu

BASE = Workload("attn_f32", batch=1, heads=2, head_dim=64, n_q=65, page_size=40, n_cand=5,
                n_cur=2, k_h=(3, 1), dtype="f32", seed=71, value_scale=0.35, gates=True)


def _layer(wl, dev):
    from paper_2609_34606_amd import HsaLayer
    import torch
    layer = HsaLayer(wl.batch, wl.heads, wl.head_dim, wl.page_size, torch.float32, "cuda:0",
                     k_pool=dev["k_pool"], v_pool=dev["v_pool"], page_table=dev["page_table"])
    layer.fold(0, wl.n_pages)
    return layer


def _oracle(case, wl):
    return run_oracle(dict(q=case.q, k_pool=case.k_pool, v_pool=case.v_pool,
                           page_table=case.page_table, g_lin=case.g_lin, g_sp=case.g_sp), wl,
                      wl.budgets())


@pytest.mark.parametrize("n_q,P,n_cand,n_cur,k_h,d,B", [
    (1, 8, 3, 1, (2, 0), 64, 1),          # one query, pages shorter than a tile, one-page list
    (63, 24, 5, 2, (3, 1), 128, 2),       # 24-key pages: every tile clamped
    (64, 32, 5, 2, (3, 1), 128, 1),       # whole tiles and blocks
    (65, 40, 5, 2, (3, 1), 128, 3),       # 8-key windows, a block of one query
    (257, 392, 9, 1, (8, 2), 64, 1),      # pieces of unequal lists
    (300, 1560, 6, 3, (6, 1), 128, 1)])
def test_edges_with_full_and_smallest_workspace(n_q, P, n_cand, n_cur, k_h, d, B):
    import torch
    from paper_2609_34606_amd import config, hsa_forward, hsa_forward_workspace_size
    wl = BASE.replace(n_q=n_q, page_size=P, n_cand=n_cand, n_cur=n_cur, k_h=k_h, head_dim=d, batch=B)
    say(f"[case] f32 attention edges {wl}")
    case = make_case(wl)
    dev = upload(case)
    layer = _layer(wl, dev)
    ref = _oracle(case, wl)["O"]
    k_max = max(k_h)
    full = hsa_forward_workspace_size(layer.cfg, n_q, k_max, n_cur)
    # the bytes a call needs: the query sums and the selection (a bf16 config
    # differs by its split partials only), and the pieces' scratch after them
    need = -(-n_q // 32) * wl.heads * d * 8 * B
    need = -(-need // 256) * 256 + 256
    assert full > need
    for nbytes in (full, need, need + (full - need) // 2):
        o = torch.full_like(dev["q"], float("nan"))
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
        hsa_forward(layer.cfg, dev["q"], n_q, layer.pool, n_cand, n_cur, list(k_h), k_max,
                    layer.kv_state, layer.k_state, layer.page_kmean, dev["g_lin"], dev["g_sp"], o, ws=ws)
        torch.cuda.synchronize()
        assert_close(f"O ({nbytes} bytes)", to_host(o), ref, **F32_TOL)
    st = hsa_forward(layer.cfg, dev["q"], n_q, layer.pool, n_cand, n_cur, list(k_h), k_max,
                     layer.kv_state, layer.k_state, layer.page_kmean, dev["g_lin"], dev["g_sp"], o,
                     ws=torch.empty(need - 256, dtype=torch.uint8, device="cuda:0"), check=False)
    assert st == 4  # HSA_ERR_WORKSPACE below what a call needs, as for bf16


def test_operands_aligned_to_four_bytes():
    import torch
    wl = BASE.replace(n_q=130, page_size=200, head_dim=128, seed=72)
    say(f"[case] f32 unaligned {wl}")
    case = make_case(wl)
    dev = upload(case)

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        v = buf[1:].view(t.shape)
        v.copy_(t)
        assert v.data_ptr() % 16 == 4
        return v

    layer = _layer(wl, dev)
    layer.k_pool, layer.v_pool = shifted(dev["k_pool"]), shifted(dev["v_pool"])
    layer.kv_state, layer.k_state = shifted(layer.kv_state), shifted(layer.k_state)
    out = shifted(torch.zeros_like(dev["q"]))
    # the query sums of the page selection read 16 bytes at a time: the queries
    # keep their alignment in hsa_forward, and lose it in the sparse branch
    layer.forward(dev["q"], wl.n_cand, wl.n_cur, list(wl.budgets()), g_lin=dev["g_lin"],
                  g_sp=dev["g_sp"], out=out)
    torch.cuda.synchronize()
    ref = _oracle(case, wl)
    assert_close("O", to_host(out), ref["O"], **F32_TOL)
    from paper_2609_34606_amd import hsa_sparse_attn
    sel = torch.from_numpy(np.ascontiguousarray(ref["sel"])).to("cuda:0").to(torch.int32)
    o_sp = shifted(torch.zeros_like(dev["q"]))
    hsa_sparse_attn(layer.cfg, shifted(dev["q"]), wl.n_q, layer.pool, sel, sel.shape[-1],
                    list(wl.budgets()), wl.n_cand, wl.n_cur, o_sp)
    torch.cuda.synchronize()
    assert_close("O_sp", to_host(o_sp), ref["O_sp"], **F32_TOL)


@pytest.mark.parametrize("P,n_pages,H,d,B,shift", [(8, 1, 1, 64, 1, 0), (24, 3, 2, 128, 1, 1),
                                                    (40, 30, 3, 64, 2, 0), (392, 9, 8, 128, 1, 1),
                                                    (1560, 3, 1, 128, 1, 0)])
def test_state_and_index_of_some_pages(P, n_pages, H, d, B, shift):
    # pages [1, 1 + n_pages) folded on top of a state, the pool aligned to 4
    # bytes only where shift is 1; 64-bit numpy sums. The state's terms are
    # fp32 products added in fp32: 1e-5 as in the parity tests.
    import torch
    from paper_2609_34606_amd import HsaLayer
    say(f"[case] f32 state P={P} pages={n_pages} H={H} d={d} B={B} shift={shift}")
    r = np.random.default_rng(74)
    slots = B * (n_pages + 2)
    k = r.standard_normal((slots, H, P, d)).astype(np.float32)
    v = r.standard_normal((slots, H, d, P)).astype(np.float32)
    table = r.permutation(slots).reshape(B, n_pages + 2).astype(np.int32)

    def up(a):
        buf = torch.empty(a.size + shift, dtype=torch.float32, device="cuda:0")
        t = buf[shift:].view(a.shape)
        t.copy_(torch.from_numpy(a))
        return t

    layer = HsaLayer(B, H, d, P, torch.float32, "cuda:0", k_pool=up(k), v_pool=up(v),
                     page_table=torch.from_numpy(table).to("cuda:0"))
    layer.kv_state.fill_(0.5)
    layer.k_state.fill_(0.25)
    layer.fold(1, n_pages)
    torch.cuda.synchronize()
    pages = table[:, 1:1 + n_pages]
    kk = k[pages].astype(np.float64)                      # [B, n, H, P, d]
    f = np.where(kk > 0, kk + 1.0, np.exp(np.minimum(kk, 0.0)))
    S = 0.5 + np.matmul(v[pages].astype(np.float64), f).sum(1)   # [B, H, d(v), d(k)]
    assert_close("kv_state", to_host(layer.kv_state), S, max_abs=np.inf, rel_l2=1e-5)
    assert_close("k_state", to_host(layer.k_state), 0.25 + f.sum((1, 3)), max_abs=np.inf, rel_l2=1e-5)
    mean = to_host(layer.page_kmean)
    np.testing.assert_allclose(mean[:, :, 1:1 + n_pages], kk.mean(3).swapaxes(1, 2), rtol=1e-12, atol=1e-15)
    assert (mean[:, :, 0] == 0).all() and (mean[:, :, -1] == 0).all()


def test_infinite_value_stays_in_its_page_and_dimension():
    # a value of +inf makes its (head, dimension) infinite and nothing else,
    # also where a masked window re-reads the key that holds it (page 40: keys
    # 8..31 are read again by the window of keys 32..39)
    import torch
    from paper_2609_34606_amd import hsa_sparse_attn
    wl = BASE.replace(n_cand=0, k_h=(0, 0), n_cur=2, n_q=20, seed=73)
    say(f"[case] f32 infinite value {wl}")
    case = make_case(wl)
    dev = upload(case)
    slot = int(case.page_table[0, 1])
    dev["v_pool"][slot, 1, 5, 20] = float("inf")
    layer = _layer(wl, dev)
    o_sp = torch.zeros((1, wl.n_q, wl.heads, wl.head_dim), dtype=torch.float32, device="cuda:0")
    hsa_sparse_attn(layer.cfg, dev["q"], wl.n_q, layer.pool, None, 0, None, 0, 2, o_sp)
    torch.cuda.synchronize()
    got = to_host(o_sp)
    assert np.isposinf(got[0, :, 1, 5]).all()
    got[0, :, 1, 5] = 0.0
    assert np.isfinite(got).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("adaptive", [False, True])
def test_scores_round_less_than_one_chain_over_d(d, adaptive):
    # Terms of one sign make the partial sums grow along d, so each rounding
    # counts. Key 0 has all the weight, and the LSE is its score: its error
    # against 64 bits must stay below what one fp32 chain over d shows for the
    # same numbers (emulated: the product of two floats is exact in 64 bits, the
    # sum is rounded to 32). Measured on that emulation, in units of 2^-24: one
    # chain 2.0 (d = 64) and 3.0, two halves 1.2 and 1.5; the LSE's scaling and
    # addition round at most three times more (0.3 each, added in squares).
    import torch
    from paper_2609_34606_amd import HsaLayer, hsa_sparse_attn, hsa_sparse_attn_adaptive
    say(f"[case] f32 score rounding d={d} adaptive={adaptive}")
    H, n_q, P = 4, 256, 8
    r = np.random.default_rng(75)
    q = np.abs(r.standard_normal((n_q, H, d))).astype(np.float32)
    k = -np.abs(r.standard_normal((1, H, P, d))).astype(np.float32)
    k[:, :, 0] *= -1
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    layer = HsaLayer(1, H, d, P, torch.float32, "cuda:0", k_pool=up(k),
                     v_pool=up(np.ones((1, H, d, P), dtype=np.float32)),
                     page_table=torch.zeros((1, 1), dtype=torch.int32, device="cuda:0"), sm_scale=1.0)
    o = torch.zeros((1, n_q, H, d), dtype=torch.float32, device="cuda:0")
    lse = torch.zeros((1, H, n_q), dtype=torch.float32, device="cuda:0")
    if adaptive:
        hsa_sparse_attn_adaptive(layer.cfg, up(q)[None], n_q, layer.pool, None, 0, None, 0, 1, o, lse=lse,
                                 tau_min=1.0, tau_max=1.0)
    else:
        hsa_sparse_attn(layer.cfg, up(q)[None], n_q, layer.pool, None, 0, None, 0, 1, o, lse=lse)
    torch.cuda.synchronize()
    q64, k64 = q.astype(np.float64), k[0, :, 0].astype(np.float64)
    ref = np.einsum("qhd,hd->hq", q64, k64)
    assert ref.min() > 8  # the other keys' scores are as far below zero
    chain = np.zeros((H, n_q), dtype=np.float32)
    for i in range(d):
        chain = (chain.astype(np.float64) + q64[:, :, i].T * k64[:, None, i]).astype(np.float32)
    rms = lambda x: float(np.sqrt((((x - ref) / ref) ** 2).mean()))
    assert rms(to_host(lse)[0]) <= 0.8 * rms(chain)
