"""Calls captured into a graph: work lists that no eager call has built yet, graphs that outlive the
cache's entries, and the no-allocation backward, whose lists the graph copies again. Every replay, with
eager work on other packs between, gives bitwise what the eager calls give. All buffers are those of
the call itself, and every list that could take a captured one's place is of a smaller pack."""
import numpy as np
import pytest

from paper_2607_01701_amd import _lib
from paper_2607_01701_amd.workload import make_pack

from gpu_util import dev_inputs, log, run_hip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def step(pack, d, r, noalloc):
    """Forward and backward into the tensors of r."""
    import torch
    from paper_2607_01701_amd import attn_bwd, attn_fwd
    attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, pack.scale, out=r["out"], lse=r["lse"])
    if not noalloc:
        attn_bwd(d["q"], d["k"], d["v"], r["out"], r["lse"], d["dout"], pack.cu_seqlens, pack.scale, dq=r["dq"],
                 dk=r["dk"], dv=r["dv"])
        return
    st = _lib.t2v_attn_bwd_noalloc(
        d["q"].data_ptr(), d["k"].data_ptr(), d["v"].data_ptr(), r["out"].data_ptr(), r["lse"].data_ptr(),
        np.ascontiguousarray(pack.cu_seqlens, dtype=np.int32), len(pack.cu_seqlens) - 1, pack.heads, pack.head_dim,
        pack.scale, d["dout"].data_ptr(), r["dq"].data_ptr(), r["dk"].data_ptr(), r["dv"].data_ptr(),
        torch.cuda.current_stream().cuda_stream)
    assert st == 0, _lib.t2v_last_error()


@pytest.mark.parametrize("warm", [False, True], ids=["new_lists", "cached_lists"])
@pytest.mark.parametrize("noalloc", [False, True], ids=["bwd", "bwd_noalloc"])
def test_replays_after_other_packs(noalloc, warm):
    import torch
    from paper_2607_01701_amd import t2v_release_cache
    pack = make_pack([700, 129, 1500], 3, 128, seed=95)
    d = dev_inputs(pack)
    log(f"case captured step noalloc={noalloc} warm={warm}")
    want = {k: v.clone() for k, v in run_hip(pack, d).items()}
    r = {k: torch.empty_like(v) for k, v in want.items()}
    if not warm:
        t2v_release_cache()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(pack, d, r, noalloc)
    eager = run_hip(pack, d)  # before the graph has run
    assert all(torch.equal(eager[k], want[k]) for k in want), "eager call after the capture"
    for i in range(3):
        for j in range(70):  # more packs than the cache holds; at most 40 + 70 rows, one or two tiles
            p = make_pack([40 + j], 1, 64, seed=96 + j)
            run_hip(p)
        for x in r.values():
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(r[k], want[k]) for k in want), f"replay {i}"
    t2v_release_cache()


def test_capture_waits_for_a_list_still_in_flight():
    """A list whose upload is queued behind other work of an eager call's stream: it is on the device
    when the capture on another stream ends, since the graph's launches wait for nothing outside the graph."""
    import torch
    from paper_2607_01701_amd import attn_fwd, t2v_release_cache
    pack = make_pack([300, 129], 2, 128, seed=97)
    d = dev_inputs(pack)
    want, want_lse = (x.clone() for x in attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, pack.scale))
    out, lse, out2, lse2 = (torch.empty_like(x) for x in (want, want_lse, want, want_lse))
    x = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    y = x @ x
    t2v_release_cache()
    log("case capture with the list in flight")
    busy, side, behind = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(busy):
        for _ in range(100):
            torch.mm(x, x, out=y)
        behind.record()
        attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, pack.scale, out=out2, lse=lse2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        graph.capture_begin()
        attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, pack.scale, out=out, lse=lse)
        graph.capture_end()
    assert behind.query(), "the captured call returned before the list was on the device"
    for i in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.equal(lse, want_lse), f"replay {i}"
    assert torch.equal(out2, want) and torch.equal(lse2, want_lse)
    t2v_release_cache()
