"""Decode and extend captured in a HIP graph (torch.cuda.CUDAGraph) after the
workspace of the capture stream is reserved: every replay, with new query values
copied into the captured input and eager work and synchronisations in between,
must equal the eager call on the same inputs bit for bit (the same kernels, the
same work split). A call that would have to grow the workspace while the stream
is captured fails with RL_ERR_WORKSPACE instead of allocating.
"""

import pytest
import torch

from paper_2609_08368_amd import rl_attn as ra
from paper_2609_08368_amd import workloads as wl
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _replay_and_compare(g, q_static, fresh, eager, outs, what, oracle=None):
    for rep in range(4):
        q_new = fresh(rep)
        q_static.copy_(q_new)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        ref = eager(q_new)                      # eager call on the default stream, in between
        torch.cuda.synchronize()
        for got, want in zip(outs, ref):
            assert torch.equal(got.view(torch.int16) if got.dtype == torch.bfloat16 else got,
                               want.view(torch.int16) if want.dtype == torch.bfloat16 else want), \
                f"{what}: replay {rep} differs from the eager call"
        H.say(f"  {what}: replay {rep} equal")
    if oracle is not None:                      # the last replay against the oracle as well
        ref_o, ref_l = oracle(q_static)
        H.compare(outs[0].reshape(ref_o.shape), ref_o, outs[1].reshape(ref_l.shape), ref_l, what=f"{what} vs oracle")


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("n", [1, 4])
@pytest.mark.parametrize("warm", [True, False], ids=["warm", "reserve_only"])
def test_decode_graph_replays_equal_eager(fp8, n, warm):
    lens = [700, 4, 3000, 129, 64]
    w = wl.custom(401, "extend" if n > 1 else "decode", lens, q_lens=[n] * len(lens) if n > 1 else None,
                  hq=16, hkv=2, page_size=64)
    t = (wl.materialize_fp8 if fp8 else wl.materialize)(w, DEV)
    B, hq = w.batch, w.hq
    shape = (B, n, hq, 128) if n > 1 else (B, hq, 128)
    H.say(f"graph decode fp8={fp8} n={n}")

    def call(q, out, lse, stream=None):
        args = (t["k_pages"], t["v_pages"])
        if fp8:
            ra.decode_fp8(q, *args, t["k_scale"], t["v_scale"], t["block_table"], t["kv_lens"], t["scale"], out=out,
                          lse=lse, stream=stream)
        else:
            ra.decode(q, *args, t["block_table"], t["kv_lens"], t["scale"], out=out, lse=lse, stream=stream)

    def fresh(rep):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(500 + rep)
        return torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)

    def eager(q):
        out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
        lse = torch.empty(shape[:-1], dtype=torch.float32, device=DEV)
        call(q, out, lse)
        return out, lse

    s = torch.cuda.Stream()
    ra.reserve_workspace(ra.decode_workspace_size(B, hq, w.hkv, t["block_table"].shape[1], w.page_size,
                                                  query_tokens=n), stream=s)
    q_static = fresh(99)
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    lse = torch.empty(shape[:-1], dtype=torch.float32, device=DEV)
    if warm:
        with torch.cuda.stream(s):
            call(q_static, out, lse, stream=s)    # warm-up on the capture stream
    else:
        # the capture stream's first call is the captured one: its reserved
        # workspace must suffice (an eager call elsewhere loads the kernels)
        call(q_static, out, lse)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call(q_static, out, lse, stream=s)
    torch.cuda.synchronize()
    oracle = (lambda q: H.oracle_full(w, dict(t, q=q.reshape(t["q"].shape)))) if n > 1 else \
        (lambda q: H.oracle_full(w, dict(t, q=q)))
    _replay_and_compare(g, q_static, fresh, eager, (out, lse), f"decode fp8={fp8} n={n}", oracle)
    ra.check_device_errors()


def test_extend_graph_replays_equal_eager():
    w = wl.custom(402, "extend", [700, 300, 90], q_lens=[300, 1, 90], hq=16, hkv=2, page_size=64)
    t = wl.materialize(w, DEV)
    shape = tuple(t["q"].shape)
    H.say("graph extend")

    def call(q, out, lse, stream=None):
        ra.extend(q, t["qo_indptr"], t["k_pages"], t["v_pages"], t["block_table"], t["kv_lens"], t["scale"],
                  out=out, lse=lse, stream=stream)

    def fresh(rep):
        gen = torch.Generator(device=DEV)
        gen.manual_seed(600 + rep)
        return torch.randn(shape, generator=gen, device=DEV).to(torch.bfloat16)

    def eager(q):
        out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
        lse = torch.empty(shape[:-1], dtype=torch.float32, device=DEV)
        call(q, out, lse)
        return out, lse

    s = torch.cuda.Stream()
    ra.reserve_workspace(ra.extend_workspace_size(w.batch, w.total_q, w.hq, w.hkv, t["block_table"].shape[1],
                                                  w.page_size), stream=s)
    q_static = fresh(99)
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    lse = torch.empty(shape[:-1], dtype=torch.float32, device=DEV)
    with torch.cuda.stream(s):
        call(q_static, out, lse, stream=s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        call(q_static, out, lse, stream=s)
    torch.cuda.synchronize()
    _replay_and_compare(g, q_static, fresh, eager, (out, lse), "extend", lambda q: H.oracle_full(w, dict(t, q=q)))
    ra.check_device_errors()


def test_capture_without_reserved_workspace_is_refused():
    """A fresh stream has no workspace: the captured call reports RL_ERR_WORKSPACE and
    launches nothing; the capture is then ended and discarded."""
    w = wl.custom(403, "decode", [100, 40], hq=8, hkv=2, page_size=16)
    t = wl.materialize(w, DEV)
    s = torch.cuda.Stream()
    out = torch.empty_like(t["q"])
    g = torch.cuda.CUDAGraph()
    err = None
    with torch.cuda.graph(g, stream=s):
        out.zero_()                             # a fill kernel, so the captured graph is not empty
        try:
            ra.decode(t["q"], t["k_pages"], t["v_pages"], t["block_table"], t["kv_lens"], t["scale"], out=out,
                      stream=s)
        except ra.RlAttnError as e:
            err = e
    torch.cuda.synchronize()
    assert err is not None and err.status == "RL_ERR_WORKSPACE"


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_capture_with_room_for_the_list_only(fp8):
    """A workspace that holds a call's work list, but no partials of split keys, is enough under
    capture: units stay whole, with the bits of the eager call that splits them."""
    hq, hkv, ps, lens = 16, 2, 64, [20000, 40000, 300]
    n = [40, 3, 300]
    w = wl.custom(407, "extend", lens, q_lens=n, hq=hq, hkv=hkv, page_size=ps)
    H.say(f"capture with a list-only workspace fp8={fp8}")
    t = (wl.materialize_fp8 if fp8 else wl.materialize)(w, DEV)
    pages = (t["k_pages"], t["v_pages"]) + ((t["k_scale"], t["v_scale"]) if fp8 else ())
    width = t["block_table"].shape[1]
    plan = ra.diag_extend_plan(lens, hq, hkv, width * ps, qo_indptr=w.qo_indptr)
    assert plan["split_seqs"] > 0
    need = ra.extend_workspace_size(w.batch, w.total_q, hq, hkv, 1, ps)       # the list alone
    assert need < ra.extend_workspace_size(w.batch, w.total_q, hq, hkv, width, ps)
    ext = ra.extend_fp8 if fp8 else ra.extend
    dec = ra.decode_fp8 if fp8 else ra.decode
    q1 = t["q"][:w.batch].contiguous()

    def calls(out_e, out_d, stream=None):
        ext(t["q"], t["qo_indptr"], *pages, t["block_table"], t["kv_lens"], t["scale"], out=out_e, stream=stream)
        dec(q1, *pages, t["block_table"], t["kv_lens"], t["scale"], out=out_d, deterministic=True, stream=stream)

    want_e, want_d = torch.empty_like(t["q"]), torch.empty_like(q1)
    calls(want_e, want_d)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    ra.reserve_workspace(need, stream=s)
    out_e, out_d = torch.empty_like(t["q"]), torch.empty_like(q1)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        calls(out_e, out_d, stream=s)
    for rep in range(3):
        out_e.zero_()
        out_d.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_e.view(torch.int16), want_e.view(torch.int16)), f"extend, replay {rep}"
        assert torch.equal(out_d.view(torch.int16), want_d.view(torch.int16)), f"deterministic decode, replay {rep}"
    ref_o, _ = H.oracle_full(w, t)
    H.compare(out_e, ref_o, what="captured whole units")
    ra.check_device_errors(s)


def test_workspace_of_the_largest_batch_serves_smaller_captured_ones():
    """Reserved once for 1,100 sequences (more than the planner splits), used by a captured call of 3."""
    hq, hkv, ps, n = 16, 2, 64, [1, 50, 100]
    w = wl.custom(408, "extend", [17000, 33000, 100], q_lens=n, hq=hq, hkv=hkv, page_size=ps)
    H.say("workspace of a larger batch")
    t = wl.materialize(w, DEV)
    width = t["block_table"].shape[1]
    s = torch.cuda.Stream()
    ra.reserve_workspace(ra.extend_workspace_size(1100, w.total_q, hq, hkv, width, ps), stream=s)
    assert ra.diag_extend_plan(w.kv_lens, hq, hkv, width * ps, qo_indptr=w.qo_indptr)["split_seqs"] > 0
    want, _ = H.run_extend(w, t)
    out = torch.empty_like(t["q"])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ra.extend(t["q"], t["qo_indptr"], t["k_pages"], t["v_pages"], t["block_table"], t["kv_lens"], t["scale"],
                  out=out, stream=s)
    for rep in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), f"replay {rep}"
    ra.check_device_errors(s)


def test_profiling_skips_captured_calls():
    """With kernel timing on, a call captured into a graph is not timed (its events
    would only be recorded at replay); eager calls still are."""
    w = wl.custom(404, "decode", [300, 64], hq=8, hkv=2, page_size=16)
    t = wl.materialize(w, DEV)
    s = torch.cuda.Stream()
    ra.reserve_workspace(ra.decode_workspace_size(w.batch, w.hq, w.hkv, t["block_table"].shape[1], w.page_size),
                         stream=s)
    out = torch.empty_like(t["q"])
    ra.profile_read("decode")
    ra.profile_enable(True)
    try:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            ra.decode(t["q"], t["k_pages"], t["v_pages"], t["block_table"], t["kv_lens"], t["scale"], out=out,
                      stream=s)
        g.replay()
        ra.decode(t["q"], t["k_pages"], t["v_pages"], t["block_table"], t["kv_lens"], t["scale"])
        torch.cuda.synchronize()
        launches, ms = ra.profile_read("decode")
    finally:
        ra.profile_enable(False)
    assert launches == 1 and ms > 0, (launches, ms)
    ref_o, _ = H.oracle_full(w, t)
    H.compare(out, ref_o, what="captured decode with profiling on")


def test_graph_survives_workspace_growth():
    """A graph keeps the address of its stream's workspace: a later, larger eager call
    on the same stream grows the workspace but keeps the captured buffer, so the graph
    still replays correctly; rl_attn_release() then frees both."""
    w = wl.custom(405, "decode", [300, 64], hq=8, hkv=2, page_size=16)
    t = wl.materialize(w, DEV)
    big = wl.custom(406, "decode", [40] * 4000, hq=8, hkv=2, page_size=16)
    tb = wl.materialize(big, DEV)
    s = torch.cuda.Stream()
    ra.reserve_workspace(ra.decode_workspace_size(w.batch, w.hq, w.hkv, t["block_table"].shape[1], w.page_size),
                         stream=s)
    out = torch.empty_like(t["q"])
    lse = torch.empty(t["q"].shape[:-1], dtype=torch.float32, device=DEV)
    H.say("graph then workspace growth on the capture stream")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ra.decode(t["q"], t["k_pages"], t["v_pages"], t["block_table"], t["kv_lens"], t["scale"], out=out, lse=lse,
                  stream=s)
    torch.cuda.synchronize()
    out_big = torch.empty_like(tb["q"])
    with torch.cuda.stream(s):
        ra.decode(tb["q"], tb["k_pages"], tb["v_pages"], tb["block_table"], tb["kv_lens"], tb["scale"], out=out_big,
                  stream=s)                     # needs a larger workspace: it grows here
    torch.cuda.synchronize()
    want_o, want_l = H.run_decode(w, t)
    for rep in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want_o.view(torch.int16)) and torch.equal(lse, want_l), \
            f"replay {rep} after the workspace grew differs from the eager call"
    ref_o, ref_l = H.oracle_full(w, t)
    H.compare(out, ref_o, lse, ref_l, what="graph replay after workspace growth")
    ref_bo, ref_bl = H.oracle_full(big, tb)
    H.compare(out_big, ref_bo, what="larger call on the capture stream")
    ra.check_device_errors(s)
    del g
    ra.release()
