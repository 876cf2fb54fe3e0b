"""Keys whose scores are -inf (a -inf key channel, or a product that overflows
fp32): they get no weight wherever in the list they stand, also where a whole
tile, key stream or piece of an item holds no other keys. Against 64-bit sums
over the remaining keys, with the repository's bars for the sparse branch."""
import numpy as np
import pytest

from hsa_testlib import BF16_TOL, F32_TOL, assert_close, say, to_host

pytestmark = pytest.mark.gpu

# masked(i, n): is key i of a list of n keys masked?
MASKS = {
    "first": lambda i, n: i < 64,                        # the walk's first tile
    "odd": lambda i, n: i // 32 % 2 == 1,                # every second 32-key tile
    "middle": lambda i, n: (i >= n // 4) & (i < n - 8),  # first tiles of later pieces
    "most": lambda i, n: i < n - 8,                      # all but eight keys
    "blocks": lambda i, n: (i >= 128) & (i < 256) | (i >= n - 64),
    "all": lambda i, n: i >= 0,
}


def _inputs(r, H, d, n_q, P, n_pages, mask, kind):
    """q [n_q, H, d], k and v [H, n, d] (float32, exact in bf16) and the mask
    [n_q, n]. kind "inf": -inf in channel 0 of a masked key; "overflow": -1e30
    there, against 1e30 in the query (every third query holds 0 instead and
    masks nothing)."""
    import torch
    n = P * n_pages
    bf = lambda *s: torch.from_numpy(r.standard_normal(s).astype(np.float32)).bfloat16().float().numpy()
    q, k, v = bf(n_q, H, d), bf(H, n, d), bf(H, n, d)
    m = np.broadcast_to(MASKS[mask](np.arange(n), n), (n_q, n)).copy()
    big = float(torch.tensor(1e30).bfloat16())
    k[:, :, 0] = 0.0
    if kind == "inf":
        q[:, :, 0] = np.abs(q[:, :, 0]) + 0.5
        q = torch.from_numpy(q).bfloat16().float().numpy()
        k[:, m[0], 0] = -np.inf
    else:
        q[:, :, 0] = big
        q[::3, :, 0] = 0.0
        k[:, m[0], 0] = -big
        m[::3] = False
    return q, k, v, m


def _reference(q, k, v, m, scale=0.0):
    q, k, v = q.astype(np.float64), k.astype(np.float64), v.astype(np.float64)
    k0 = np.where(np.isinf(k[:, :, :1]), 0.0, k[:, :, :1])
    k = np.concatenate([k0 * 0.0, k[:, :, 1:]], axis=2)  # channel 0 only masks
    s = np.einsum("qhd,hkd->hqk", q, k) * (scale or q.shape[-1] ** -0.5)
    s = np.where(m[None], -np.inf, s)
    mx = s.max(-1, keepdims=True)
    e = np.exp(s - np.where(np.isinf(mx), 0.0, mx))
    z = e.sum(-1, keepdims=True)
    o = np.einsum("hqk,hkd->qhd", e / np.where(z > 0, z, 1.0), v)
    with np.errstate(divide="ignore"):
        return o, np.log(z[..., 0]) + np.where(np.isinf(mx), 0.0, mx)[..., 0]


def _run(dtype, q, k, v, P, ws_bytes=None, scale=0.0, adaptive=False):
    import torch
    from paper_2609_34606_amd import (HsaLayer, hsa_sparse_attn, hsa_sparse_attn_adaptive,
                                      hsa_sparse_attn_workspace_size)
    n_q, H, d = q.shape
    n_pages = k.shape[1] // P
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0").to(dt)
    kp = k.reshape(H, n_pages, P, d).transpose(1, 0, 2, 3)
    vp = v.reshape(H, n_pages, P, d).transpose(1, 0, 3, 2)
    layer = HsaLayer(1, H, d, P, dt, "cuda:0", k_pool=up(kp), v_pool=up(vp),
                     page_table=torch.arange(n_pages, dtype=torch.int32, device="cuda:0")[None],
                     sm_scale=scale)
    o = torch.full((1, n_q, H, d), float("nan"), dtype=torch.float32, device="cuda:0")
    lse = torch.full((1, H, n_q), float("nan"), dtype=torch.float32, device="cuda:0")
    nbytes = hsa_sparse_attn_workspace_size(layer.cfg, n_q, 0, n_pages) if ws_bytes is None else ws_bytes
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0") if nbytes else None
    if adaptive:
        hsa_sparse_attn_adaptive(layer.cfg, up(q)[None], n_q, layer.pool, None, 0, None, 0, n_pages, o,
                                 lse=lse, tau_min=1.0, tau_max=1.0)
    else:
        hsa_sparse_attn(layer.cfg, up(q)[None], n_q, layer.pool, None, 0, None, 0, n_pages, o, lse=lse, ws=ws)
    torch.cuda.synchronize()
    return to_host(o)[0], to_host(lse)[0]


# fp32: items cut into pieces with the workspace of the size query, whole with
# none; bf16: 33 tiles of one item are cut into two ranges, 8 are not
@pytest.mark.parametrize("dtype,d,n_q,P,n_pages,ws_bytes", [
    ("f32", 64, 70, 40, 9, None), ("f32", 128, 70, 392, 5, None), ("f32", 128, 70, 392, 5, 0),
    ("bf16", 64, 300, 128, 4, None), ("bf16", 128, 70, 200, 8, None), ("bf16", 128, 70, 40, 33, None)])
@pytest.mark.parametrize("kind", ["inf", "overflow"])
@pytest.mark.parametrize("mask", ["first", "odd", "middle", "most"])
def test_masked_keys_get_no_weight(dtype, d, n_q, P, n_pages, ws_bytes, kind, mask):
    say(f"[case] masked scores {dtype} d={d} n_q={n_q} P={P} pages={n_pages} ws={ws_bytes} {kind} {mask}")
    q, k, v, m = _inputs(np.random.default_rng(91), 2, d, n_q, P, n_pages, mask, kind)
    o, lse = _run(dtype, q, k, v, P, ws_bytes)
    ref_o, ref_lse = _reference(q, k, v, m)
    assert_close("O_sp", o, ref_o, **(BF16_TOL if dtype == "bf16" else F32_TOL))
    np.testing.assert_allclose(lse, ref_lse, atol=2e-3 if dtype == "bf16" else 1e-4)


@pytest.mark.parametrize("dtype,P,n_pages", [("f32", 392, 5), ("bf16", 40, 33)])
@pytest.mark.parametrize("scale", [0.0, 0.75])  # 0.75 log2(e) > 1: a lower starting reference
def test_a_query_with_no_weights(dtype, P, n_pages, scale):
    # every score of two thirds of the queries is -inf: zeros and an LSE of
    # -inf, as for an empty list; the other queries are not touched
    say(f"[case] no weights {dtype} P={P} scale={scale}")
    q, k, v, m = _inputs(np.random.default_rng(92), 2, 64, 70, P, n_pages, "all", "overflow")
    o, lse = _run(dtype, q, k, v, P, scale=scale)
    ref_o, ref_lse = _reference(q, k, v, m, scale)
    none = m.all(1)
    assert (o[none] == 0).all() and np.isneginf(lse[:, none]).all()
    assert_close("O_sp", o[~none], ref_o[~none], **(BF16_TOL if dtype == "bf16" else F32_TOL))
    np.testing.assert_allclose(lse[:, ~none], ref_lse[:, ~none], atol=2e-3 if dtype == "bf16" else 1e-4)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mask", ["first", "blocks"])
def test_masked_blocks_of_the_tile_lists(dtype, mask):
    # threshold 1: a block of masked keys (weight 0) is kept or not by the
    # rounding of the running weight, and no key of it has a weight either way
    say(f"[case] masked blocks {dtype} {mask}")
    q, k, v, m = _inputs(np.random.default_rng(93), 2, 64, 300, 128, 5, mask, "inf")
    o, lse = _run(dtype, q, k, v, 128, adaptive=True)
    ref_o, ref_lse = _reference(q, k, v, m)
    assert_close("O_sp", o, ref_o, **(BF16_TOL if dtype == "bf16" else F32_TOL))
    np.testing.assert_allclose(lse, ref_lse, atol=2e-3 if dtype == "bf16" else 1e-4)


@pytest.mark.parametrize("d,n_q,P,n_pages,ws_bytes", [(64, 70, 40, 9, None), (128, 70, 392, 5, None),
                                                      (128, 70, 392, 5, 0)])
def test_huge_fp32_scores(d, n_q, P, n_pages, ws_bytes):
    # a few keys, in different tiles, streams and pieces, whose scores reach
    # 1e20 and more: the largest takes all the weight (no two are near each
    # other), whichever sign and order they have
    say(f"[case] huge scores d={d} P={P} pages={n_pages} ws={ws_bytes}")
    r = np.random.default_rng(94)
    n = P * n_pages
    q, k, v = (r.standard_normal(s).astype(np.float32) for s in ((n_q, 2, d), (2, n, d), (2, n, d)))
    at = np.linspace(1, n - 2, 7).astype(int)
    k[:, at, 0] = np.float32(1e21) * np.array([1.5, -4.0, 3.0, 8.0, -7.0, 0.25, -0.5], dtype=np.float32)
    o, lse = _run("f32", q, k, v, P, ws_bytes)
    s = np.einsum("qhd,hkd->hqk", q.astype(np.float64), k.astype(np.float64)) / np.sqrt(d)
    best = s.argmax(-1)
    assert (s.max(-1) > 1e15).all()
    for h in range(2):
        np.testing.assert_array_equal(o[:, h], v[h, best[h]])
    np.testing.assert_allclose(lse, s.max(-1), rtol=1e-5)
