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
