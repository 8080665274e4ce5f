"""loki_rotate_keys at the edges of its tiles and of its dealing out of rows to blocks, against a
float64 product (Algorithm 1 lines 3-4 of arXiv 2406.02542)."""
import pytest
import torch

from paper_2406_02542_amd import api

pytestmark = pytest.mark.gpu
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


def check(B, H, n, pos, cap, d, dtype, scale=1.0, page_rows=0):
    print(f"case B={B} H={H} n={n} pos={pos} cap={cap} d={d} {dtype} scale={scale} pages={page_rows}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B * 1000003 + H * 1009 + n * 31 + d)
    P = torch.linalg.qr(torch.randn((min(H, 4), 128, 128), generator=gen, device="cuda", dtype=torch.float64))[0].float()
    P = P.repeat(-(-H // min(H, 4)), 1, 1)[:H].contiguous()
    k = (torch.randn((B, H, n, 128), generator=gen, device="cuda") * scale).to(DT[dtype])
    lay = api.make_layout(B, H, H, 128, d, cap, DT[dtype])
    if page_rows:
        per = -(-cap // page_rows)
        table = torch.randperm(B * per + 2, generator=torch.Generator().manual_seed(n))[:B * per].to(torch.int32).reshape(B, per)
        lead = (B * per + 2, H, page_rows)
    else:
        lead = (B, H, cap)
    klo = torch.full((*lead, d), 5.0, dtype=DT[dtype], device="cuda")
    khi = torch.full((*lead, 128 - d), 5.0, dtype=DT[dtype], device="cuda") if d < 128 else None
    if page_rows:
        api.loki_rotate_keys_paged(lay, k, P, klo, khi, table.cuda(), page_rows, lead[0], pos, n)
    else:
        api.loki_rotate_keys(lay, k, P, klo, khi, pos, n)
    torch.cuda.synchronize()
    rows = klo if khi is None else torch.cat([klo, khi], dim=-1)
    if page_rows:  # logical rows of every sequence; the pages of none stay as they were
        free = sorted(set(range(lead[0])) - set(table.flatten().tolist()))
        assert bool((rows[free] == 5.0).all())
        rows = rows[table.flatten().long().cuda()].reshape(B, per, H, page_rows, 128).transpose(1, 2).reshape(B, H, per * page_rows, 128)
    assert bool((rows[:, :, :pos] == 5.0).all()) and bool((rows[:, :, pos + n:] == 5.0).all())
    for h in range(H):
        x, Ph = k[:, h].double().reshape(-1, 128), P[h].double()
        got = rows[:, h, pos:pos + n].double().reshape(-1, 128)
        ref = x @ Ph
        # 128 fp32 multiply-adds in any order: 128 2^-24 of the sum of the magnitudes at the very worst, of
        # which sqrt(128) / 128 (7e-7) is what random signs leave; 2e-6 covers every order of the sums
        acc = 2e-6 * (x.abs() @ Ph.abs())
        if dtype == "bf16":  # and half an ulp of the one rounding, taken at the magnitude above
            bound = (ref.abs() + acc) * 2.0 ** -8 + acc
        else:  # (and a few units of the smallest denormal)
            bound = acc + 2.0 ** -146
        worst = float(((got - ref).abs() - bound).max())
        assert worst <= 0, (h, worst)


# a trip is 32 rows in bf16 and 16 in fp32
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,H,n,pos,d", [
    (1, 2, 1, 0, 32), (1, 2, 15, 3, 32), (1, 2, 16, 0, 64), (1, 1, 17, 0, 8), (1, 2, 31, 1, 32), (2, 2, 32, 0, 128),
    (3, 2, 33, 5, 16),                       # trips that cross a sequence
    (50, 2, 3, 2, 32), (64, 8, 1, 7, 32),    # many sequences in one trip
    (3, 5, 701, 0, 40), (2, 3, 4099, 2, 32)])
def test_tiles_and_sequences(B, H, n, pos, d, dtype):
    check(B, H, n, pos, pos + n + 3, d, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,n", [(256, 577), (128, 1025), (300, 261), (200, 290), (700, 33)])
def test_trips_per_block_and_rounds(H, n, dtype):
    """One to twenty trips a block (more than are on their way at once), one and several rounds of blocks."""
    check(1, H, n, 0, n, 32, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,pos", [(300, 250), (1, 511), (37, 1000)])
def test_pages(n, pos, dtype):
    check(3, 2, n, pos, 1280, 32, dtype, page_rows=256)


@pytest.mark.parametrize("scale", [2.0 ** -130, 2.0 ** 100])
def test_fp32_range(scale):
    """Denormal products and large ones keep fp32's range."""
    check(1, 2, 70, 0, 70, 32, "f32", scale=scale)
