"""Which kernel sequence a decode step takes, read back through the stage names of a profile: the sides
of every line that a dispatch rule draws.  (What the sequences compute is compared elsewhere.)"""
import pytest
import torch

from paper_2406_02542_amd import api

pytestmark = pytest.mark.gpu
DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def stages(dtype, B, Hq, Hkv, S, d, k, mode, append=False, paged=False):
    """Names of the kernels that one step launches."""
    dt, D = DT[dtype], 128
    lay = api.make_layout(B, Hq, Hkv, D, d, S, dt)
    per = -(-S // 256)
    lead = (B * per, Hkv, 256) if paged else (B, Hkv, S)
    klo, khi, v = (torch.zeros((*lead, w), dtype=dt, device="cuda") for w in (d, D - d, D))
    q = torch.randn((B, Hq, D), device="cuda").to(dt)
    P = torch.eye(D, device="cuda").repeat(Hkv, 1, 1)
    step = {}
    if append:
        step["k_new"], step["v_new"] = (torch.zeros((B, Hkv, D), dtype=dt, device="cuda") for _ in range(2))
    if paged:
        step["page_table"] = torch.arange(B * per, dtype=torch.int32, device="cuda").reshape(B, per)
        step["page_rows"], step["n_pages"] = 256, B * per
    ws = api.alloc_workspace(lay, S, d, k, mode)
    out = torch.empty_like(q)
    prof = api.Profile()
    prof.attach()
    try:
        api.loki_decode_step(lay, q, P, klo, khi if d < D else None, v, S, d, k, mode, ws, out, **step)
    finally:
        prof.detach()
    torch.cuda.synchronize()
    names = [n for n, _ in prof.read()]
    print(dtype, B, Hq, Hkv, S, d, k, hex(mode), append, paged, names, flush=True)
    assert torch.all(out == 0)  # (the values are zeros)
    return names


@pytest.mark.parametrize("one_launch,dtype,B,Hq,Hkv,S,d,k,mode", [
    (True, "bf16", 1, 32, 32, 4096, 32, 1024, 0), (True, "bf16", 2, 32, 8, 2048, 64, 512, 1), (True, "f32", 1, 32, 8, 1000, 64, 100, 1),
    (False, "bf16", 16, 32, 32, 700, 32, 100, 0),   # 512 units of one head: 16 blocks per CU
    (False, "bf16", 64, 64, 8, 600, 64, 150, 0),    # 512 units, eight heads and two passes in every block
    (False, "bf16", 64, 32, 8, 600, 48, 150, 1),    # the same on the vector units
    (False, "f32", 2, 32, 8, 600, 128, 150, 1)])    # fp32 rows of over 64 columns: would spill
def test_rotation_inside_the_scoring(one_launch, dtype, B, Hq, Hkv, S, d, k, mode):
    names = stages(dtype, B, Hq, Hkv, S, d, k, mode | api.PATH_SPLIT)
    assert (names[0] == "rotate_score") == one_launch
    assert one_launch or names[:2] == ["rotate_query", "score"]
