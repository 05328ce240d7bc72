"""The one-pass backward for cross-attention to short key segments (at most 256 keys each, many
queries): gradients against the float64 oracle and the general path at the edges of its tiles
(key counts around 32, 64, 128 and 256; query counts around its 32-query steps, its three LDS
stages and its pieces), bitwise reproducible also while other streams run it, and delta_ws
holding -Delta and lse * log2(e) as after the general path."""
import numpy as np
import pytest

import oracle
from paper_2607_01701_amd.workload import bf16_bits_to_f32, make_pack_qk

from gpu_util import assert_within, dev_inputs, log, rel_err

pytestmark = pytest.mark.gpu

LQ = [3000, 1, 31, 33, 96, 97, 2049, 1500, 64, 65]
LK = [1, 32, 33, 128, 129, 256, 255, 64, 65, 100]
HEADS = 64


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _backward(d, pack, out, lse):
    import torch
    from paper_2607_01701_amd import attn_bwd
    ws = torch.full((2, pack.heads, pack.total_tokens), float("nan"), dtype=torch.float32, device="cuda")
    g = attn_bwd(d["q"], d["k"], d["v"], out, lse, d["dout"], pack.cu_seqlens, pack.scale, delta_ws=ws,
                 cu_seqlens_k=pack.cu_seqlens_k)
    return dict(zip(("dq", "dk", "dv"), g), ws=ws)


def test_short_key_backward(monkeypatch, capfd):
    import torch
    from paper_2607_01701_amd import attn_fwd, t2v_release_cache
    pack = make_pack_qk(LQ, LK, HEADS, 128, seed=91)
    log(f"case one-pass backward lq={LQ} lk={LK} H={HEADS}")
    d = dev_inputs(pack)
    out, lse = attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, pack.scale, cu_seqlens_k=pack.cu_seqlens_k)
    t2v_release_cache()
    monkeypatch.setenv("T2V_LOG", "1")
    a = _backward(d, pack, out, lse)
    torch.cuda.synchronize()
    err = capfd.readouterr().err
    assert "256-row tiles" in err and "loops split at" in err, err
    monkeypatch.delenv("T2V_LOG")
    streams = [torch.cuda.Stream() for _ in range(3)]
    again = []
    for s in streams:  # concurrent calls have partial slots of their own
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            again.append(_backward(d, pack, out, lse))
    torch.cuda.synchronize()
    for b in again:
        for n in a:
            assert torch.equal(a[n], b[n]), f"{n} is not reproducible"
    monkeypatch.setenv("T2V_SHORT", "off")
    g = _backward(d, pack, out, lse)
    torch.cuda.synchronize()
    # fp32 sums of the same products in another order (128 terms of order 1)
    assert torch.allclose(a["ws"], g["ws"], rtol=1e-5, atol=1e-4)
    heads = [0, HEADS - 1]
    f = {n: bf16_bits_to_f32(np.ascontiguousarray(getattr(pack, n)[:, heads])) for n in ("q", "k", "v", "dout")}
    ref = oracle.attention(f["q"], f["k"], f["v"], f["dout"], pack.cu_seqlens, pack.scale,
                           cu_seqlens_k=pack.cu_seqlens_k)
    errs = {"out": 0.0, "lse": 0.0}
    for n in ("dq", "dk", "dv"):
        got = a[n][:, heads].double().cpu().numpy()
        errs[n] = rel_err(got, ref[n])
        # The general path rounds P, dS and the result at the same places; each is within 2^-8 of the exact result.
        assert rel_err(a[n].double().cpu().numpy(), g[n].double().cpu().numpy()) <= 2e-2, n
    log(f"  errors {errs}")
    assert_within(errs)


def test_few_queries_and_equal_offsets_keep_the_general_path(monkeypatch, capfd):
    """Too few queries to fill the CUs, a segment of 257 keys, or offsets equal to the queries'
    (self-attention): bitwise what T2V_SHORT=off gives."""
    import torch
    from paper_2607_01701_amd import attn_fwd
    for lq, lk, H in (([3000, 500], [100, 256], 2), ([20000, 500], [100, 257], 20), ([200] * 40, [200] * 40, 64)):
        pack = make_pack_qk(lq, lk, H, 128, seed=92)
        log(f"case general path lq={lq[:2]} lk={lk[:2]} H={H}")
        d = dev_inputs(pack)
        out, lse = attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, pack.scale, cu_seqlens_k=pack.cu_seqlens_k)
        monkeypatch.delenv("T2V_SHORT", raising=False)
        a = _backward(d, pack, out, lse)
        monkeypatch.setenv("T2V_SHORT", "off")
        b = _backward(d, pack, out, lse)
        torch.cuda.synchronize()
        for n in a:
            assert torch.equal(a[n], b[n]), n


def test_partial_sums_share_one_buffer_and_stay_bounded(monkeypatch, capfd):
    """Calls enqueued in a row on one stream share one buffer; with more than 2,048 pieces of 2,048
    queries the pieces grow instead (512 heads x 10,000 queries: 2,560), and the gradients are
    those of the general path."""
    import torch
    from paper_2607_01701_amd import attn_bwd, attn_fwd, t2v_release_cache
    H, lq, lk = 512, [6000, 4000], [77, 200]
    log(f"case bounded partial sums lq={lq} lk={lk} H={H}")
    cu, ck = np.array([0, 6000, 10000], np.int32), np.array([0, 77, 277], np.int32)
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v, dout = (torch.randn((n, H, 128), generator=g, device="cuda", dtype=torch.bfloat16)
                     for n in (10000, 277, 277, 10000))
    out, lse = attn_fwd(q, k, v, cu, 0.1, cu_seqlens_k=ck)
    ws = torch.empty((2, H, 10000), dtype=torch.float32, device="cuda")
    grads = [torch.empty_like(x) for x in (q, k, v)]

    def backward():
        attn_bwd(q, k, v, out, lse, dout, cu, 0.1, *grads, delta_ws=ws, cu_seqlens_k=ck)

    t2v_release_cache()
    monkeypatch.setenv("T2V_LOG", "1")
    backward()
    assert "loops split at 2560" in capfd.readouterr().err
    monkeypatch.delenv("T2V_LOG")
    free = torch.cuda.mem_get_info()[0]
    for _ in range(8):
        backward()
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] >= free - (64 << 20)  # a buffer per call would be 8 x 640 MiB
    one_pass = [x.clone() for x in grads]
    monkeypatch.setenv("T2V_SHORT", "off")
    backward()
    torch.cuda.synchronize()
    for n, a, b in zip(("dq", "dk", "dv"), one_pass, grads):
        # both round P, dS and the result at the same places; each is within 2^-8 of the exact result
        d = (a.float() - b.float()).abs().max().item() / b.float().abs().max().item()
        assert d <= 2e-2, (n, d)
    t2v_release_cache()


def _cross_inputs(lq, lk, heads, seed):
    import torch
    from paper_2607_01701_amd import attn_fwd
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v, dout = (torch.randn((n, heads, 128), generator=g, device="cuda", dtype=torch.bfloat16)
                     for n in (sum(lq), sum(lk), sum(lk), sum(lq)))
    cu, ck = (np.concatenate([[0], np.cumsum(x)]).astype(np.int32) for x in (lq, lk))
    out, lse = attn_fwd(q, k, v, cu, 0.1, cu_seqlens_k=ck)
    return q, k, v, out, lse, dout, cu, ck


def test_path_does_not_depend_on_what_is_in_flight():
    """Packs that grow, enqueued without waiting (their partial sums would take 384, 480 and 576 MiB
    at once), give bitwise what each gives on an idle GPU."""
    import torch
    from paper_2607_01701_amd import attn_bwd
    log("case growing packs in flight")
    packs = [_cross_inputs([t // 16] * 16, [200] * 16, 24, 6) for t in (100000, 140000, 170000)]

    def backward(p):
        return attn_bwd(*p[:6], p[6], 0.1, cu_seqlens_k=p[7])[1:]

    torch.cuda.synchronize()
    in_flight = [backward(p) for p in packs]
    torch.cuda.synchronize()
    for p, g in zip(packs, in_flight):
        alone = backward(p)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(g, alone))


def test_workspace_sizes_give_the_same_bits():
    """t2v_attn_bwd_qk_ws: no workspace is refused with the sizes it could use and nothing written; the
    least (a head at a time), an uneven one (5 of 41 heads) and the most give bitwise equal gradients and
    never write past their size; t2v_attn_bwd_qk takes the general path."""
    import torch
    from paper_2607_01701_amd import _lib, attn_bwd
    H, lq, lk = 41, [6000, 0, 700, 4099], [77, 0, 31, 256]
    q, k, v, out, lse, dout, cu, ck = _cross_inputs(lq, lk, H, 7)
    ws = torch.empty((2, H, sum(lq)), dtype=torch.float32, device="cuda")
    log(f"case workspace sizes lq={lq} lk={lk} H={H}")

    def call(nbytes):
        g = [torch.full_like(x, 3.0) for x in (q, k, v)]
        buf = torch.full((nbytes + 4096,), 77, dtype=torch.uint8, device="cuda")
        r = _lib.t2v_attn_bwd_qk_ws(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(), cu, ck,
                                    len(lq), H, 128, 0.1, dout.data_ptr(), *(x.data_ptr() for x in g),
                                    ws.data_ptr(), buf.data_ptr() if nbytes else None, nbytes,
                                    torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert bool((buf[nbytes:] == 77).all()), "written past the workspace"
        return r, g

    (st, least, most), g = call(0)
    assert st == _lib.T2V_ERR_WORKSPACE and 0 < least and most == H * least
    assert all(bool((x == 3.0).all()) for x in g)
    assert call(least - 16)[0][0] == _lib.T2V_ERR_WORKSPACE
    (st, *_), full = call(most)
    assert st == _lib.T2V_OK
    for nbytes in (least, 5 * least + 256):
        (st, *_), g = call(nbytes)
        assert st == _lib.T2V_OK and all(torch.equal(a, b) for a, b in zip(g, full)), nbytes
    bound = attn_bwd(q, k, v, out, lse, dout, cu, 0.1, cu_seqlens_k=ck)
    assert all(torch.equal(a, b) for a, b in zip(bound, full))


def test_entry_without_workspace_takes_the_general_path(monkeypatch):
    import torch
    from paper_2607_01701_amd import _lib, attn_bwd
    H = 41
    q, k, v, out, lse, dout, cu, ck = _cross_inputs([6000, 4099], [77, 256], H, 8)
    ws = torch.empty((2, H, 10099), dtype=torch.float32, device="cuda")
    g = [torch.empty_like(x) for x in (q, k, v)]
    log("case cross backward without workspace")
    st = _lib.t2v_attn_bwd_qk(q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), lse.data_ptr(), cu, ck, 2, H,
                              128, 0.1, dout.data_ptr(), *(x.data_ptr() for x in g), ws.data_ptr(),
                              torch.cuda.current_stream().cuda_stream)
    assert st == 0, _lib.t2v_last_error()
    monkeypatch.setenv("T2V_SHORT", "off")
    want = attn_bwd(q, k, v, out, lse, dout, cu, 0.1, cu_seqlens_k=ck)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(g, want))


@pytest.mark.parametrize("lq,lk,one_pass", [
    ([33] * 300, [16] * 300, False), ([79] * 150, [200] * 150, False), ([80] * 150, [200] * 150, True),
    ([1] * 200 + [12000, 0], [31] * 201 + [0], False), ([1] * 150 + [20000, 0], [31] * 151 + [0], True),
], ids=["33_queries", "79_queries", "80_queries", "ones_and_one_long", "ones_and_one_longer"])
def test_short_query_sequences_keep_the_general_path(lq, lk, one_pass, capfd, monkeypatch):
    """With pieces of fewer than 80 queries in the mean an item's fixed part outweighs the saved pass."""
    import torch
    from paper_2607_01701_amd import attn_bwd, t2v_release_cache
    H = 40
    cu, ck = (np.concatenate([[0], np.cumsum(x)]).astype(np.int32) for x in (lq, lk))
    x, y = (torch.zeros((n, H, 128), dtype=torch.bfloat16, device="cuda") for n in (sum(lq), sum(lk)))
    lse = torch.zeros((H, sum(lq)), dtype=torch.float32, device="cuda")
    log(f"case path of short query sequences n={len(lq)} lq={lq[0]}")
    t2v_release_cache()
    monkeypatch.setenv("T2V_LOG", "1")
    attn_bwd(x, y, y, x, lse, x, cu, 0.1, cu_seqlens_k=ck)
    torch.cuda.synchronize()
    lists = capfd.readouterr().err.count("t2v: work list")
    assert lists == (1 if one_pass else 2)  # the general path has one for dK/dV and one for dQ


@pytest.mark.parametrize("case,scale", [("negative_scale", -0.2), ("zero_scale", 0.0), ("special_values", 0.1)])
def test_other_scales_orders_and_values(case, scale, monkeypatch):
    """The one-pass backward on negative and zero scales against the oracle; NaN and infinities come out
    where the general path has them, and leave the other sequences and heads as they were; pack
    order changes nothing."""
    import torch
    from paper_2607_01701_amd import attn_bwd, attn_fwd
    lq, lk, H = [3000, 2049, 96], [77, 256, 33], 65
    pack = make_pack_qk(lq, lk, H, 128, seed=93)
    log(f"case one-pass backward {case}")
    d = dev_inputs(pack)

    def backward(**env):
        for name, value in env.items():
            monkeypatch.setenv(name, value)
        out, lse = attn_fwd(d["q"], d["k"], d["v"], pack.cu_seqlens, scale, cu_seqlens_k=pack.cu_seqlens_k)
        g = attn_bwd(d["q"], d["k"], d["v"], out, lse, d["dout"], pack.cu_seqlens, scale, cu_seqlens_k=pack.cu_seqlens_k)
        torch.cuda.synchronize()
        for name in env:
            monkeypatch.delenv(name)
        return dict(zip(("dq", "dk", "dv"), g))

    clean = backward()
    for n, x in backward(T2V_ORDER="natural").items():
        assert torch.equal(x, clean[n]), n
    if case != "special_values":
        heads = [0, H - 1]
        f = {n: bf16_bits_to_f32(np.ascontiguousarray(getattr(pack, n)[:, heads])) for n in ("q", "k", "v", "dout")}
        ref = oracle.attention(f["q"], f["k"], f["v"], f["dout"], pack.cu_seqlens, scale, cu_seqlens_k=pack.cu_seqlens_k)
        assert_within({"out": 0.0, "lse": 0.0, **{n: rel_err(x[:, heads].double().cpu().numpy(), ref[n])
                                                  for n, x in clean.items()}})
        return
    d["q"][40, 0, 3] = float("nan")        # sequence 0, head 0
    d["dout"][3005, 1, 7] = float("inf")   # sequence 1, head 1
    d["k"][340, 2, 0] = float("nan")       # sequence 2, head 2
    a, g = backward(), backward(T2V_SHORT="off")
    for n in a:
        assert torch.equal(a[n].isnan(), g[n].isnan()) and torch.equal(a[n].isinf(), g[n].isinf()), n
        same = a[n] == clean[n]
        c = np.cumsum([0] + (lq if n == "dq" else lk))
        for s in range(3):
            rest = [h for h in range(H) if h != s]
            assert bool(same[c[s]:c[s + 1], rest].all()), (n, s)
    assert bool(a["dk"][:77, 0].isnan().all()) and bool(a["dq"][5049:, 2].isnan().all())


def test_captured_call_gives_the_same_bits():
    """A backward call captured into a graph takes the same path as an eager one: each replay, with eager
    calls between, writes what the eager call wrote."""
    import torch
    from paper_2607_01701_amd import attn_bwd
    log("case captured one-pass backward")
    q, k, v, out, lse, dout, cu, ck = _cross_inputs([6000, 4099], [77, 256], 41, 9)
    grads = [torch.empty_like(x) for x in (q, k, v)]
    ws = torch.empty((2, 41, 10099), dtype=torch.float32, device="cuda")

    def backward():
        attn_bwd(q, k, v, out, lse, dout, cu, 0.1, *grads, delta_ws=ws, cu_seqlens_k=ck)

    backward()
    torch.cuda.synchronize()
    want = [x.clone() for x in grads]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        backward()
    for i in range(4):
        for x in grads:
            x.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(grads, want)), f"replay {i}"
        backward()
        assert all(torch.equal(a, b) for a, b in zip(grads, want)), f"eager call after replay {i}"
