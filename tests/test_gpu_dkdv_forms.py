"""The dK/dV kernel's 64-keys-per-wave form (256-key tiles, hand-scheduled steps) gives bitwise
what the 32-keys-per-wave form gives, at the edges of its tiles: key counts around 32, 64 and
256, query loops shorter than its LDS stages, of exactly as many steps, and ragged by one; and
both match the float64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2607_01701_amd.workload import make_pack_qk

from gpu_util import assert_within, compare_full, dev_inputs, log, run_hip, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


PACKS = [
    # (query lengths, key lengths, heads): the kernel keeps 5 stages of 32 queries
    ([1, 31, 32, 33, 64], [1, 31, 32, 33, 64], 2),
    ([127, 128, 129, 159, 160, 161], [63, 65, 255, 256, 257, 513], 2),
    ([300, 192, 193, 1000], [300, 700, 129, 1000], 3),
]


@pytest.mark.parametrize("lq,lk,H", PACKS, ids=["one_stage", "stage_edges", "several_tiles"])
def test_wide_form_is_bitwise_equal(lq, lk, H, monkeypatch):
    import torch
    pack = make_pack_qk(lq, lk, H, 128, seed=81)
    log(f"case dK/dV forms lq={lq} lk={lk} H={H}")
    d = dev_inputs(pack)
    monkeypatch.setenv("T2V_KVTILE", "narrow")
    a = {k: v.clone() for k, v in run_hip(pack, d).items()}
    monkeypatch.setenv("T2V_KVTILE", "wide")
    b = run_hip(pack, d)
    for k in a:
        assert torch.equal(a[k], b[k]), f"{k} differs between the two forms"
    ref = oracle.attention(pack.f32("q"), pack.f32("k"), pack.f32("v"), pack.f32("dout"), pack.cu_seqlens, pack.scale,
                           cu_seqlens_k=pack.cu_seqlens_k)
    errs, _ = compare_full(to_np(b), ref, pack.cu_seqlens, "wide dK/dV", cu_k=pack.cu_seqlens_k)
    assert_within(errs)


@pytest.mark.parametrize("heads,lens,rows", [(24, [4096] * 8, 256), (12, [1024] * 8, 128), (3, [6912], 128)])
def test_form_is_chosen_from_the_pack(heads, lens, rows, capfd, monkeypatch):
    """The form follows the predicted time (the plan log names the tile rows)."""
    import torch
    from paper_2607_01701_amd import attn_bwd, t2v_release_cache
    T = sum(lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    x = torch.zeros((T, heads, 128), dtype=torch.bfloat16, device="cuda")
    lse = torch.zeros((heads, T), dtype=torch.float32, device="cuda")
    t2v_release_cache()
    monkeypatch.setenv("T2V_LOG", "1")
    attn_bwd(x, x, x, x, lse, x, cu, 0.1)
    torch.cuda.synchronize()
    err = capfd.readouterr().err
    log(f"case form choice heads={heads} lens={lens[:2]}")
    assert err.splitlines()[0].split("heads, ")[1].startswith(f"{rows}-row tiles"), err


@pytest.mark.parametrize("case,scale,order", [("negative_scale", -0.2, None), ("zero_scale", 0.0, None),
                                              ("pack_order", 0.1, "natural"), ("special_values", 0.1, None)])
def test_wide_form_on_other_scales_orders_and_values(case, scale, order, monkeypatch):
    """Bitwise equal there too; NaN and infinities come out where the other form has them."""
    import torch
    pack = make_pack_qk([300, 129, 160], [300, 257, 64], 2, 128, seed=82)
    log(f"case dK/dV forms {case}")
    d = dev_inputs(pack)
    if case == "special_values":
        d["q"][40, 0, 3] = float("nan")
        d["dout"][305, 1, 7] = float("inf")
        d["v"][560, 0, 0] = -float("inf")
    if order is not None:
        monkeypatch.setenv("T2V_ORDER", order)
    monkeypatch.setenv("T2V_KVTILE", "narrow")
    a = {k: v.clone() for k, v in run_hip(pack, d, scale).items()}
    monkeypatch.setenv("T2V_KVTILE", "wide")
    b = run_hip(pack, d, scale)
    for k in a:
        assert bool(((a[k] == b[k]) | (a[k].isnan() & b[k].isnan())).all()), k
    if case == "special_values":
        assert bool(a["dk"][:300, 0].isnan().all()) and not bool(a["dk"][:300, 1].isnan().any())
        assert not bool(a["dv"][300:557, 1, 7].isfinite().all()) and not bool(a["dk"][557:, 0].isfinite().all())
    else:
        ref = oracle.attention(pack.f32("q"), pack.f32("k"), pack.f32("v"), pack.f32("dout"), pack.cu_seqlens, scale,
                               cu_seqlens_k=pack.cu_seqlens_k)
        errs, _ = compare_full(to_np(b), ref, pack.cu_seqlens, "wide dK/dV", cu_k=pack.cu_seqlens_k)
        assert_within(errs)
