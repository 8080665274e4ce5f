"""Page tables of more than 64 pages per sequence, through the single-launch kernels: the pages of long rows
(Algorithm 1 on several blocks per unit, up to 131072 rows on 256-row pages), and tables wider than the rows there
are.  A paged call selects and returns what the contiguous call does, with an appended row in the last page; the
entries past the sequence's pages are out of the pool and must not be used."""
import pytest
import torch

from paper_2406_02542_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,S,d,k,width,group,last_stage", [
    (1, 8, 2, 16640, 32, 2080, 65, 1, "fused_decode"),      # the first length with 65 pages, full
    (3, 8, 2, 16385, 32, 1000, 70, 1, "fused_decode"),      # one row in page 65, a wider table
    (1, 16, 2, 131072, 16, 8192, 512, 1, "fused_decode"),   # the longest
    (1, 4, 2, 130817, 64, 4000, 600, 1, "fused_decode"),    # one row in page 512, a table wider than a block
    (40, 16, 2, 12500, 32, 1500, 200, 1, "fused_decode"),    # several blocks per unit, two of them
    (140, 8, 2, 700, 32, 170, 128, 1, "fused_decode"),      # one block per unit
    (20, 8, 8, 2100, 32, 500, 100, 0, "fused_decode"),      # one block per head, every head its own KV head
    (16, 32, 8, 3000, 32, 400, 65, 0, "fused_decode"),      # one block per head of a group
    (1, 4, 4, 20000, 32, 900, 90, 0, "gather_attend"),      # the split path as before
])
def test_paged_equals_contiguous(B, Hq, Hkv, S, d, k, width, group, last_stage):
    print("case", B, Hq, Hkv, S, d, k, width, group, flush=True)
    gen = torch.Generator(device="cuda").manual_seed(S + width)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    dt, per, n_pages = torch.bfloat16, -(-S // 256), B * -(-S // 256) + 3
    P = torch.linalg.qr(rnd(Hkv, 128, 128).double())[0].float().contiguous()
    scale = torch.exp(-torch.arange(128, device="cuda") / 20.0) + 0.1
    kh = (rnd(B, Hkv, per * 256, 128) * scale).to(dt)
    v, q = rnd(B, Hkv, per * 256, 128).to(dt), rnd(B, Hq, 128).to(dt)
    k_new, v_new = rnd(B, Hkv, 128).to(dt), rnd(B, Hkv, 128).to(dt)
    slabs = [kh[..., :d].contiguous(), kh[..., d:].contiguous(), v]
    perm = torch.randperm(n_pages, generator=torch.Generator().manual_seed(width))[:B * per].to(torch.int32).reshape(B, per)
    table = torch.full((B, width), 0x7fffffff, dtype=torch.int32)
    table[:, :per] = perm
    at = perm.flatten().long().cuda()

    def to_pool(t):
        pool = torch.full((n_pages, Hkv, 256, t.shape[-1]), 3e4, dtype=dt, device="cuda")
        pool[at] = t.reshape(B, Hkv, per, 256, -1).transpose(1, 2).reshape(B * per, Hkv, 256, -1)
        return pool

    def call(layout, kl, kv_hi, vv, **step):
        ws = api.alloc_workspace(layout, S, d, k, group)
        out = torch.full((B, Hq, 128), float("nan"), dtype=dt, device="cuda")
        idx = torch.full((B, Hkv if group else Hq, k), -7, dtype=torch.int32, device="cuda")
        prof = api.Profile()
        prof.attach()
        try:
            api.loki_decode_step(layout, q, P, kl, kv_hi, vv, S, d, k, group, ws, out, idx, k_new=k_new, v_new=v_new, **step)
        finally:
            prof.detach()
        torch.cuda.synchronize()
        return out, idx, prof.read()[-1][0]

    pools = [to_pool(t) for t in slabs]
    lay = api.make_layout(B, Hq, Hkv, 128, d, per * 256, dt)
    out, idx, stage = call(lay, *pools, page_table=table.cuda(), page_rows=256, n_pages=n_pages)
    ref, ref_idx, _ = call(lay, *slabs)
    assert stage == last_stage
    assert torch.equal(idx, ref_idx)
    # the same rows in another order of fp32 sums where the two calls take different kernels, one rounding to bf16
    assert float((out.float() - ref.float()).norm() / ref.float().norm()) < 2e-3
    for pool, slab in zip(pools, slabs):  # the appended row, and nothing else
        back = pool[at].reshape(B, per, Hkv, 256, -1).transpose(1, 2).reshape(slab.shape)
        assert torch.equal(back, slab)
        assert float(pool[sorted(set(range(n_pages)) - set(at.tolist()))].float().min()) == float(torch.tensor(3e4, dtype=dt))


@pytest.mark.parametrize("path", [api.PATH_FUSED, api.PATH_CLUSTER])
def test_pinned_paths_refuse_wide_tables(path):
    B, Hq, Hkv, S, d, k = 1, 8, 2, 2000, 32, 200
    z = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16, device="cuda")
    lay = api.make_layout(B, Hq, Hkv, 128, d, 2048, torch.bfloat16)
    ws = api.alloc_workspace(lay, S, d, k, 1)
    P, q, out = torch.zeros((Hkv, 128, 128), device="cuda"), z(B, Hq, 128), z(B, Hq, 128)
    for width, ok in ((64, True), (65, False)):
        table = torch.zeros((B, width), dtype=torch.int32, device="cuda")
        args = (lay, q, P, z(1, Hkv, 256, d), z(1, Hkv, 256, 128 - d), z(1, Hkv, 256, 128), S, d, k, 1 | path, ws, out)
        step = dict(page_table=table, page_rows=256, n_pages=1)
        if ok:
            api.loki_decode_step(*args, **step)
        else:
            with pytest.raises(api.LokiError) as e:
                api.loki_decode_step(*args, **step)
            assert e.value.status == 2
    torch.cuda.synchronize()
