"""What a call finds in its workspace must not matter: launches that cut their
items clear the arrival counters first and write every partial before they read
it. Each call runs twice in one workspace, filled with ones beforehand, once in
one filled with zeros, and (fp32) with the smallest workspace the call takes;
equal bits where the plan is the same, the fp64 oracle otherwise."""
import ctypes

import numpy as np
import pytest

from synth_inputs import make_case, make_projections, make_prompts
from synth_inputs.configs import Workload

from hsa_testlib import BF16_TOL, F32_TOL, assert_close, say, to_host, upload
from oracle import hsa_blocks_oracle as BO
from oracle import hsa_hkv_oracle as HK
from oracle import hsa_linformer_oracle as LO
from oracle import hsa_oracle as O

pytestmark = pytest.mark.gpu

# lists of 11, 3 and 7 pages: every call cuts the long ones
WL = Workload("workspace", batch=1, heads=3, head_dim=128, n_q=300, page_size=200, n_cand=9,
              n_cur=2, k_h=(9, 1, 5), dtype="bf16", seed=95, gates=True)
RANK = 64


def _up256(n):
    return -(-n // 256) * 256


def _f32_scratch_bytes(cfg, n_q):
    """What the size queries count for pieces of fp32 items: two slots per
    range and a counter per item of 64 queries."""
    items = cfg.batch * cfg.num_heads * -(-n_q // 64)
    ranges = min(16 * items, 256 if cfg.head_dim == 128 else 512)
    return 2 * ranges * 8 * (cfg.head_dim // 8 + 2) * 64 * 4 + _up256(4 * items)


class _Call:
    """One call of `kind` on a case, with the workspace given to run()."""

    def __init__(self, kind, wl):
        import torch
        from paper_2609_34606_amd import HsaLayer
        import paper_2609_34606_amd as hsa
        self.hsa, self.kind, self.wl = hsa, kind, wl
        c = self.case = make_case(wl)
        self.host = dict(q=c.q, k_pool=c.k_pool, v_pool=c.v_pool, page_table=c.page_table,
                         g_lin=c.g_lin, g_sp=c.g_sp)
        self.dev = upload(c)
        self.k_h, self.k_max = list(c.k_h), max(c.k_h)
        self.layer = HsaLayer(wl.batch, wl.heads, wl.head_dim, wl.page_size, self.dev["q"].dtype,
                              "cuda:0", k_pool=self.dev["k_pool"], v_pool=self.dev["v_pool"],
                              page_table=self.dev["page_table"])
        self.layer.fold(0, wl.n_pages)
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
        if kind == "linformer":
            self.e = make_projections(wl, RANK, "gaussian")
            self.layer.set_projections(*(t(x).to(self.dev["q"].dtype) for x in self.e))
            self.layer.compress(0, wl.n_pages)
        if kind == "retrieval":
            # one chunk of all candidates beside one of a page, so that the
            # chosen one keeps the long lists
            pe, ce, cf = make_prompts(wl, 100)
            ce, cf = ce[:, :2], np.array([[0, wl.n_cand - 1, wl.n_cand]], dtype=np.int32)
            pe = ce[:, 0] + 0.1 * pe
            self.prompts = pe.astype(np.float32), np.ascontiguousarray(ce), cf
            self.prompts_dev = [t(x) for x in self.prompts]
        size = dict(forward=hsa.hsa_forward_workspace_size, adaptive=hsa.hsa_adaptive_workspace_size,
                    linformer=hsa.hsa_linformer_workspace_size,
                    retrieval=hsa.hsa_retrieval_workspace_size)[kind]
        self.full = size(self.layer.cfg, wl.n_q, self.k_max, wl.n_cur)

    def launch(self, ws):
        """Enqueues the call: (o, sel, the chosen chunk or None)."""
        import torch
        L, wl, dev, hsa = self.layer, self.wl, self.dev, self.hsa
        chunk = None
        o = torch.full_like(dev["q"], float("nan"))
        sel = torch.full((wl.batch, wl.heads, self.k_max), -7, dtype=torch.int32, device="cuda:0")
        head = (L.cfg, dev["q"], wl.n_q, L.pool)
        tail = (L.page_kmean, dev["g_lin"], dev["g_sp"], o)
        state = (L.kv_state, L.k_state)
        if self.kind == "forward":
            hsa.hsa_forward(*head, wl.n_cand, wl.n_cur, self.k_h, self.k_max, *state, *tail, sel_out=sel, ws=ws)
        elif self.kind == "adaptive":
            hsa.hsa_forward_adaptive(*head, wl.n_cand, wl.n_cur, self.k_h, self.k_max, *state, *tail,
                                     sel_out=sel, ws=ws)
        elif self.kind == "linformer":
            hsa.hsa_forward_linformer(*head, L.ck, L.cv, RANK, wl.n_cand, wl.n_cur, self.k_h, self.k_max,
                                      *tail, sel_out=sel, ws=ws)
        else:
            pe, ce, cf = self.prompts_dev
            chunk = torch.full((wl.batch,), -7, dtype=torch.int32, device="cuda:0")
            hsa.hsa_forward_retrieval(*head, pe, ce, ce.shape[2], ce.shape[1], cf, wl.n_cand, wl.n_cur,
                                      self.k_h, self.k_max, *state, *tail, chunk_out=chunk, sel_out=sel, ws=ws)
        return o, sel, chunk

    def run(self, ws):
        import torch
        o, sel, chunk = self.launch(ws)
        torch.cuda.synchronize()
        assert chunk is None or chunk.tolist() == [0]
        return o, to_host(sel)

    def reference(self):
        h, wl = self.host, self.wl
        pools = (h["q"], h["k_pool"], h["v_pool"], h["page_table"])
        gates = (h["g_lin"], h["g_sp"])
        if self.kind == "forward":
            return O.hsa_forward(*pools, wl.n_cand, wl.n_cur, self.k_h, *gates, sm_scale=None,
                                 k_max=self.k_max, query_rows=None, heads=None)
        if self.kind == "adaptive":
            return BO.hsa_forward_adaptive(*pools, wl.n_cand, wl.n_cur, self.k_h, BO.TAU_MIN, BO.TAU_MAX, *gates)
        if self.kind == "linformer":
            return LO.hsa_forward_linformer(*pools, *self.e, wl.n_cand, wl.n_cur, self.k_h, BO.TAU_MIN,
                                            BO.TAU_MAX, *gates)
        return HK.hsa_forward_retrieval(*pools, *self.prompts, wl.n_cur, self.k_h, *gates, k_max=self.k_max,
                                        query_rows=None)


@pytest.mark.parametrize("kind", ["forward", "adaptive", "linformer", "retrieval"])
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
def test_contents_of_the_workspace_do_not_matter(kind, dtype, d):
    import torch
    wl = WL.replace(dtype=dtype, head_dim=d)
    say(f"[case] workspace {kind} {wl}")
    call = _Call(kind, wl)
    cfg = call.layer.cfg
    if dtype == "bf16" and kind in ("forward", "retrieval"):
        most = ctypes.c_int32()
        lens = (ctypes.c_int32 * wl.heads)(*[min(k, wl.n_cand) + wl.n_cur for k in wl.k_h])
        assert call.hsa.lib().hsa_attention_plan(ctypes.byref(cfg), wl.n_q, lens, 0, None, None,
                                                 ctypes.byref(most)) == 0
        assert most.value > 1  # items are cut
    tol = F32_TOL if dtype == "f32" else BF16_TOL
    ref = call.reference()
    ws = torch.full((call.full,), 255, dtype=torch.uint8, device="cuda:0")
    bits = torch.int16 if dtype == "bf16" else torch.int32
    a, sel = call.run(ws)
    np.testing.assert_array_equal(sel[..., :ref["sel"].shape[-1]], ref["sel"])
    assert_close("O", to_host(a), ref["O"], **tol)
    runs = [call.run(ws), call.run(torch.zeros_like(ws))]
    if dtype == "f32":
        # one workgroup per item below the pieces' scratch: other bits, the same bar
        need = call.full - _f32_scratch_bytes(cfg, wl.n_q)
        whole = call.run(torch.full((need,), 255, dtype=torch.uint8, device="cuda:0"))[0]
        assert_close("O (whole items)", to_host(whole), ref["O"], **tol)
        # more than the size query asks for changes nothing
        runs.append(call.run(torch.full((call.full + 4096,), 255, dtype=torch.uint8, device="cuda:0")))
    for b, s in runs:
        assert torch.equal(a.view(bits), b.view(bits)), "outputs differ in some bits"
        np.testing.assert_array_equal(s, sel)


@pytest.mark.parametrize("kind", ["forward", "adaptive", "linformer", "retrieval"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_captured_calls_replay(kind, dtype):
    # a captured call clears its own arrival counters: every replay gives the
    # eager call's bits, whatever is left in the workspace in between
    import torch
    wl = WL.replace(dtype=dtype)
    say(f"[case] captured {kind} {wl}")
    call = _Call(kind, wl)
    bits = torch.int16 if dtype == "bf16" else torch.int32
    ws = torch.zeros(call.full, dtype=torch.uint8, device="cuda:0")
    ref, sel = call.run(ws)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        o, s, _ = call.launch(ws)
    for fill in (255, 0, 1, None):
        if fill is not None:
            ws.fill_(fill)
        call.run(torch.full_like(ws, 255))  # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o.view(bits), ref.view(bits)), f"replay after {fill} differs in some bits"
        np.testing.assert_array_equal(to_host(s), sel)
