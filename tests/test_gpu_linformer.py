"""GPU parity of the Linformer linear branch against the fp64 oracle.

Compared on the same seeded inputs and projections:
  * compressed pages: each element within one rounding of the pool type
    (bf16: 2^-8 relative, fp32: 1e-5) of the oracle's fp64 E^T X;
  * the branch output (hsa_sparse_attn over the compressed pool) and the
    whole forward (hsa_forward_linformer) within the bf16 / fp32 bars of
    hsa_testlib, with the page selection bit-exact.
"""
import numpy as np
import pytest

from synth_inputs import WORKLOADS, make_case, make_projections
from synth_inputs.configs import Workload

from hsa_testlib import BF16_TOL, F32_TOL, assert_close, elementwise_gates, gate_dims_of, say, to_host, upload
from oracle import hsa_blocks_oracle as BO
from oracle import hsa_linformer_oracle as LO
from oracle import hsa_oracle as O

pytestmark = pytest.mark.gpu

SMALL = Workload("small_linformer", batch=1, heads=3, head_dim=128, n_q=300, page_size=200,
                 n_cand=7, n_cur=2, k_h=(0, 3, 9), dtype="bf16", seed=71, gates=True)


def _layer(wl, dev, e_k, e_v):
    import torch
    from paper_2609_34606_amd import HsaLayer
    B, n_q, H, d = dev["q"].shape
    layer = HsaLayer(B, H, d, wl.page_size, dev["q"].dtype, dev["q"].device, k_pool=dev["k_pool"],
                     v_pool=dev["v_pool"], page_table=dev["page_table"],
                     gate_dims=gate_dims_of(dev))
    dt = dev["q"].dtype
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev["q"].device).to(dt)
    layer.set_projections(to(e_k), to(e_v))
    return layer


def _check_compressed(layer, host, e_k, e_v, wl, pages):
    ck, cv = to_host(layer.ck), to_host(layer.cv)
    rel = 2.0 ** -8 if wl.dtype == "bf16" else 1e-5
    worst = 0.0
    for b in range(wl.batch):
        for p in pages:
            slot = int(host["page_table"][b, p])
            for h in range(wl.heads):
                k_page, v_page = O.page_kv(host["k_pool"], host["v_pool"], host["page_table"], b, h, p)
                rk = LO.compress(e_k[h], k_page)
                rv = LO.compress(e_v[h], v_page)
                for got, ref in ((ck[slot, h], rk), (cv[slot, h].T, rv)):
                    scale = np.sqrt(np.mean(ref ** 2)) + 1e-30
                    err = np.abs(got - ref) - rel * np.abs(ref)
                    worst = max(worst, float(err.max() / scale))
                    assert (err <= 1e-5 * scale).all(), (b, p, h, float(err.max()), scale)
    say(f"  compressed pages: worst excess over one rounding {worst:.2e} (rms units)")


def _run(wl, rank=64, kind="gaussian", tau=(BO.TAU_MIN, BO.TAU_MAX), query_blocks=None, host=None,
         dev=None):
    import torch
    from paper_2609_34606_amd import hsa_sparse_attn
    from paper_2609_34606_amd import config as mkcfg
    from paper_2609_34606_amd import kv_pool
    say(f"[case] linformer {wl} rank={rank} {kind} tau={tau}")
    if host is None:
        case = make_case(wl)
        host = dict(q=case.q, k_pool=case.k_pool, v_pool=case.v_pool, page_table=case.page_table,
                    g_lin=case.g_lin, g_sp=case.g_sp)
        dev = upload(case)
        k_h = list(case.k_h)
    else:
        k_h = list(dev["k_h"])
    e_k, e_v = make_projections(wl, rank, kind)
    B, n_q, H, d = dev["q"].shape
    k_max = max(1, max(k_h))
    layer = _layer(wl, dev, e_k, e_v)
    layer.fold(0, wl.n_pages)
    layer.compress(0, wl.n_pages)
    sel = torch.full((B, H, k_max), -7, dtype=torch.int32, device=dev["q"].device)
    o = layer.forward_linformer(dev["q"], wl.n_cand, wl.n_cur, k_h, k_max=k_max, tau_min=tau[0],
                                tau_max=tau[1], g_lin=dev.get("g_lin"), g_sp=dev.get("g_sp"),
                                sel_out=sel)
    # the branch alone: sparse attention over the compressed pool
    crank = mkcfg(B, H, d, rank, dev["q"].dtype)
    cpool = kv_pool(layer.ck, layer.cv, dev["page_table"], crank)
    o_lin = torch.zeros((B, n_q, H, d), dtype=torch.float32, device=dev["q"].device)
    lse = torch.zeros((B, H, n_q), dtype=torch.float32, device=dev["q"].device)
    hsa_sparse_attn(crank, dev["q"], n_q, cpool, sel, k_max, k_h, wl.n_cand, wl.n_cur, o_lin, lse=lse)
    torch.cuda.synchronize()
    _check_compressed(layer, host, e_k, e_v, wl, range(wl.n_pages) if wl.n_pages <= 12 else
                      sorted(set(range(wl.n_cand, wl.n_pages)) | set(to_host(sel).ravel()[to_host(sel).ravel() >= 0].tolist()))[:16])
    ref = LO.hsa_forward_linformer(host["q"], host["k_pool"], host["v_pool"], host["page_table"],
                                   e_k, e_v, wl.n_cand, wl.n_cur, k_h, tau[0], tau[1],
                                   host.get("g_lin"), host.get("g_sp"), query_blocks=query_blocks)
    tol = BF16_TOL if wl.dtype == "bf16" else F32_TOL
    gsel = to_host(sel)
    w = min(gsel.shape[-1], ref["sel"].shape[-1])
    np.testing.assert_array_equal(gsel[:, :, :w], ref["sel"][:, :, :w])
    rows = ref["rows"]
    assert_close("O_lin", to_host(o_lin)[:, rows], ref["O_lin"], **tol)
    np.testing.assert_allclose(to_host(lse)[:, :, rows], ref["lse_lin"],
                               atol=2e-3 if wl.dtype == "bf16" else 1e-4)
    assert_close("O", to_host(o)[:, rows], ref["O"], **tol)
    return layer, ref


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("rank", [32, 64, 128])
def test_small_ragged_bf16(d, rank):
    # pages of 200 tokens (a partial last tile), 5 query blocks with a ragged tail
    _run(SMALL.replace(head_dim=d), rank=rank)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("P,n_pages,H", [(8, 3, 1), (64, 300, 1), (72, 2, 1), (136, 131, 2), (200, 1, 5),
                                           (264, 90, 3), (392, 40, 7), (520, 3, 2)])
def test_compression_over_tile_and_item_counts(P, n_pages, H, d):
    # one to nine 64-token tiles per page, whole pages and parts of them, and
    # item counts that the eight XCDs share unevenly: every page of a head is
    # written once, by the right item
    wl = SMALL.replace(page_size=P, n_cand=n_pages, n_cur=0, heads=H, k_h=(1,) * H, head_dim=d, n_q=64, seed=73)
    say(f"[case] compression {wl}")
    case = make_case(wl)
    host = dict(k_pool=case.k_pool, v_pool=case.v_pool, page_table=case.page_table)
    e_k, e_v = make_projections(wl, 32, "gaussian")
    layer = _layer(wl, upload(case), e_k, e_v)
    layer.ck.fill_(float("nan"))
    layer.cv.fill_(float("nan"))
    layer.compress(0, n_pages)
    import torch
    torch.cuda.synchronize()
    _check_compressed(layer, host, e_k, e_v, wl, range(n_pages))


@pytest.mark.parametrize("n_pages,parts", [(1, True), (86, False)])
def test_compressed_pages_at_an_odd_element(n_pages, parts):
    # ck and cv one element past an aligned address: pages summed from parts
    # (3 pairs of page and head) and written whole (258 of them)
    import torch
    from paper_2609_34606_amd import hsa_linformer_compress_workspace_size
    wl = SMALL.replace(n_cand=n_pages, n_cur=0, seed=72)
    say(f"[case] compressed pages at an odd element {wl}")
    case = make_case(wl)
    host = dict(k_pool=case.k_pool, v_pool=case.v_pool, page_table=case.page_table)
    e_k, e_v = make_projections(wl, 64, "gaussian")
    layer = _layer(wl, upload(case), e_k, e_v)
    assert (hsa_linformer_compress_workspace_size(layer.cfg, 64, n_pages) > 0) == parts
    shifted = lambda t: torch.full((t.numel() + 1,), float("nan"), dtype=t.dtype, device=t.device)[1:].view(t.shape)
    layer.ck, layer.cv = shifted(layer.ck), shifted(layer.cv)
    assert layer.ck.data_ptr() % 4 == 2 and layer.cv.data_ptr() % 4 == 2
    layer.compress(0, n_pages)
    torch.cuda.synchronize()
    _check_compressed(layer, host, e_k, e_v, wl, sorted({0, n_pages // 2, n_pages - 1}))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_elementwise_gates_linformer(dtype):
    wl = SMALL.replace(dtype=dtype, seed=26)
    case = make_case(wl)
    elementwise_gates(case, seed=26)
    host = dict(q=case.q, k_pool=case.k_pool, v_pool=case.v_pool, page_table=case.page_table,
                g_lin=case.g_lin, g_sp=case.g_sp)
    dev = upload(case)
    dev["k_h"] = list(case.k_h)
    _run(wl, rank=64, host=host, dev=dev)


def test_fp32_tiny():
    _run(WORKLOADS["c1"], rank=32)


@pytest.mark.parametrize("P,rank,d", [(8, 128, 128), (64, 32, 64), (72, 64, 128), (136, 128, 64),
                                      (200, 64, 64), (328, 128, 128), (392, 32, 128)])
def test_compress_whole_pages(P, rank, d):
    # enough pages and heads that pages are not split into parts: walks of one
    # to seven 64-token tiles per product, ragged last tiles, every rank and d
    # (rank 32 at d = 64 leaves two waves of a workgroup without output tiles)
    import torch
    wl = SMALL.replace(page_size=P, head_dim=d, heads=8, k_h=(1,) * 8, n_cand=33, n_q=1, seed=74)
    say(f"[case] compress whole pages P={P} rank={rank} d={d}")
    case = make_case(wl)
    dev = upload(case)
    e_k, e_v = make_projections(wl, rank)
    layer = _layer(wl, dev, e_k, e_v)
    layer.ck.fill_(float("nan"))
    layer.cv.fill_(float("nan"))
    layer.compress(0, wl.n_pages)
    torch.cuda.synchronize()
    _check_compressed(layer, dict(k_pool=case.k_pool, v_pool=case.v_pool, page_table=case.page_table),
                      e_k, e_v, wl, (0, 17, wl.n_pages - 1))


def test_small_pages_and_meanpool():
    _run(SMALL.replace(page_size=8, n_cand=11, k_h=(1, 4, 6), seed=72), rank=32)
    _run(SMALL.replace(page_size=256, seed=73), rank=64, kind="meanpool")


def test_identity_projection_full_coverage_is_twice_the_page_attention():
    # rank = P and E = I: the compressed pages are the pages; with tau = 1 both
    # branches are the page-level sparse branch, so O_lin equals its output
    import torch
    from paper_2609_34606_amd import hsa_sparse_attn
    wl = SMALL.replace(page_size=64, seed=74)
    case = make_case(wl)
    dev = upload(case)
    eye = np.stack([np.eye(64, dtype=np.float32)] * wl.heads)
    layer = _layer(wl, dev, eye, eye)
    layer.fold(0, wl.n_pages)
    layer.compress(0, wl.n_pages)
    torch.cuda.synchronize()
    assert torch.equal(layer.ck.view(torch.int16)[case.page_table.ravel()],
                       dev["k_pool"].view(torch.int16)[case.page_table.ravel()])
    B, n_q, H, d = dev["q"].shape
    k_h = list(case.k_h)
    k_max = max(k_h)
    sel = torch.empty((B, H, k_max), dtype=torch.int32, device="cuda:0")
    o = layer.forward_linformer(dev["q"], wl.n_cand, wl.n_cur, k_h, tau_min=1.0, tau_max=1.0,
                                sel_out=sel)
    o_sp = torch.empty((B, n_q, H, d), dtype=torch.float32, device="cuda:0")
    hsa_sparse_attn(layer.cfg, dev["q"], n_q, layer.pool, sel, k_max, k_h, wl.n_cand, wl.n_cur, o_sp)
    torch.cuda.synchronize()
    # gates NULL: o = 0.5 O_lin + 0.5 O_sp = O_sp up to the bf16 rounding of o
    diff = np.abs(to_host(o) - to_host(o_sp))
    say(f"  identity projection: max |o - O_sp| {diff.max():.3e}")
    assert diff.max() <= 1.6e-2


def _full_size(name, qb_k=4):
    import torch
    from synth_inputs import make_case_torch
    wl = WORKLOADS[name]
    dev = make_case_torch(wl, "cuda:0")
    torch.cuda.synchronize()
    host = {k: dev[k].float().cpu().numpy() for k in ("q", "k_pool", "v_pool")}
    host["page_table"] = dev["page_table"].cpu().numpy()
    n_qb = -(-wl.n_q // 64)
    qbs = sorted(set([0, n_qb - 1] + np.random.default_rng(8).choice(n_qb, qb_k, replace=False).tolist()))
    _run(wl, rank=64, query_blocks=qbs, host=host, dev=dev)


def test_c2_linformer_full_size():
    _full_size("c2")


def test_c3_linformer_full_size():
    _full_size("c3")
