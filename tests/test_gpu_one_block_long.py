"""Selection by one block at 8193 to 16384 rows, where a thread holds up to 32 keys: inside the
one-block-per-head launch (which, on a contiguous cache, looks a selected row's score up by its
position) and inside the attention launch of the split path.  The library takes these routes only with
many heads, so the cases are made on the GPU and compared in 64 bits on a few heads: every number of
lanes per slab row (1 to 16 bf16, 4 to 32 fp32), appended, paged, ragged, grouped."""
import numpy as np
import pytest
import torch

from paper_2406_02542_amd import api
from tests.parity import TORCH_DT, check_index_set, check_out

pytestmark = pytest.mark.gpu


def check_step(dtype, B, Hq, Hkv, S, d, k, append, paged, ragged, path, stages):
    dt, D, G = TORCH_DT[dtype], 128, Hq // Hkv
    where = f"{dtype} B {B} {Hq}/{Hkv} S {S} d {d} k {k} append {append} paged {paged} ragged {ragged}"
    print("case", where, flush=True)
    g = torch.Generator(device="cuda").manual_seed(S + d)
    sigma = torch.sqrt(torch.exp(-torch.arange(D, device="cuda") / 20.0) ** 2 + 0.01)
    per = -(-S // 256)
    pages = torch.randperm(B * per + 5, generator=torch.Generator().manual_seed(d))[:B * per].to(torch.int32).reshape(B, per).cuda()
    lead = (B * per + 5, Hkv, 256) if paged else (B, Hkv, S)
    kh = (torch.randn((*lead, D), generator=g, device="cuda") * sigma).to(dt)
    klo, khi = kh[..., :d].contiguous(), (kh[..., d:].contiguous() if d < D else None)
    del kh
    v = torch.randn((*lead, D), generator=g, device="cuda").to(dt)
    q, k_new, v_new = (torch.randn((B, h, D), generator=g, device="cuda").to(dt) for h in (Hq, Hkv, Hkv))
    P = torch.linalg.qr(torch.randn((Hkv, D, D), generator=g, device="cuda", dtype=torch.float64))[0].float().contiguous()
    lens = np.full(B, S, np.int64)
    if ragged:
        lens[1:] = np.random.default_rng(S).integers(1, S + 1, B - 1)
        lens[1] = 1
    ks = np.maximum(1, lens * k // S)
    step = {}
    if ragged:
        step["seq_lens"], step["ks"] = (torch.from_numpy(x.astype(np.int32)).cuda() for x in (lens, ks))
    if append:
        step["k_new"], step["v_new"] = k_new, v_new
    if paged:
        step.update(page_table=pages, page_rows=256, n_pages=lead[0])
    lay = api.make_layout(B, Hq, Hkv, D, d, S, dt)
    ws = api.alloc_workspace(lay, S, d, k, 0)
    out = torch.full_like(q, float("nan"))
    idx = torch.full((B, Hq, k), -7, dtype=torch.int32, device="cuda")
    prof = api.Profile()
    prof.attach()
    try:
        api.loki_decode_step(lay, q, P, klo, khi, v, S, d, k, path, ws, out, idx, **step)
    finally:
        prof.detach()
    torch.cuda.synchronize()
    assert [n for n, _ in prof.read()][-len(stages):] == stages
    worst = 0.0
    for b, hq in {(0, 0), (1, Hq - 1), (B // 2, Hq // 2), (B - 1, 1), (B - 1, Hq - 1)}:
        h, n, kk = hq // G, int(lens[b]), int(ks[b])

        def rows(t):
            if t is None:
                return torch.empty((n, 0), dtype=torch.float64)
            t = t[pages[b].long(), h].reshape(-1, t.shape[-1]) if paged else t[b, h]
            return t[:n].double().cpu()
        kr, vr = torch.cat([rows(klo), rows(khi)], dim=1), rows(v)
        Ph = P[h].double().cpu()
        if append:  # the row as it lies in the cache: 2^-8 of it and 128 fp32 products (bf16), 2e-6 of its norm (fp32)
            ref = k_new[b, h].double().cpu() @ Ph
            err = (kr[n - 1] - ref).abs()
            assert bool((err <= (2.0 ** -8 * ref.abs() + 1e-5 if dtype == "bf16" else 2e-6 * ref.norm())).all()), (where, b, h)
            assert torch.equal(vr[n - 1], v_new[b, h].double().cpu())
        qh = q[b, hq].double().cpu() @ Ph
        scores = (kr[:, :d] @ qh[:d]).numpy()
        got = idx[b, hq].cpu().numpy()
        assert np.all(got[kk:] == -1)
        check_index_set(got[:kk], np.sort(np.argsort(-scores, kind="stable")[:kk]), scores, n, kk, f"{where} b {b} head {hq}")
        sel = torch.from_numpy(got[:kk].astype(np.int64))
        w = torch.softmax(kr[sel] @ qh / D ** 0.5, dim=0)
        worst = max(worst, check_out(out[b, hq].double().cpu().numpy(), (w @ vr[sel]).numpy(), dtype, f"{where} b {b} head {hq}"))
    print(f"   max_err {worst:.3e}", flush=True)


@pytest.mark.parametrize("dtype,B,Hq,Hkv,S,d,k,append,paged,ragged", [
    ("bf16", 16, 32, 8, 12345, 32, 1543, False, False, False), ("bf16", 9, 32, 16, 10001, 64, 1250, False, True, True),
    ("bf16", 16, 8, 8, 8193, 8, 1, True, False, False), ("bf16", 16, 8, 8, 8193, 16, 700, True, False, True),
    ("bf16", 16, 8, 8, 12000, 32, 1500, True, False, False), ("bf16", 16, 8, 8, 16384, 64, 2048, True, True, True),
    ("bf16", 16, 8, 8, 9001, 128, 500, True, False, False), ("bf16", 16, 8, 8, 9001, 96, 2048, False, True, False),
    ("f32", 16, 8, 8, 8193, 16, 300, True, False, True), ("f32", 16, 8, 8, 10240, 32, 1000, False, True, False),
    ("f32", 16, 8, 8, 9000, 64, 2000, True, True, False), ("f32", 16, 8, 8, 8200, 128, 2048, True, False, False)])
def test_one_block_per_head_long_rows(dtype, B, Hq, Hkv, S, d, k, append, paged, ragged):
    check_step(dtype, B, Hq, Hkv, S, d, k, append, paged, ragged, 0, ["fused_decode"])


@pytest.mark.parametrize("dtype,B,Hq,Hkv,S,d,k,append,paged,ragged", [
    ("bf16", 33, 8, 8, 8193, 16, 300, True, True, True), ("f32", 17, 16, 8, 12000, 32, 1500, True, False, False),
    ("bf16", 9, 32, 8, 16384, 64, 2048, False, True, False), ("bf16", 5, 64, 8, 9001, 128, 700, True, False, True)])
def test_selection_inside_the_attention_long_rows(dtype, B, Hq, Hkv, S, d, k, append, paged, ragged):
    check_step(dtype, B, Hq, Hkv, S, d, k, append, paged, ragged, api.PATH_SPLIT, ["select_attend"])
