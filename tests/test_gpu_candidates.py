"""Ranking of the candidates of the threshold's histogram bin in the single-launch kernels (grouped heads; one block per
head beyond 8192 rows) and in the attention launch of the split path: by one wave from registers or from LDS, or (too many of them) by further digits.  Scores are made exactly: the query is
(1, 1, 1, 0, ..) under P = 1 and a row holds (1, j 2^-10, i 2^-18), so that its score, 1 + j 2^-10 + i 2^-18 < 1.25, is exact in
fp32 and all such rows share the 11 leading key bits; rows above and below lie in other bins.  The index list
must be the stable one to the last entry, and the result the same whether or not it is asked for."""
import numpy as np
import pytest
import torch

from paper_2406_02542_amd import api
from tests.parity import check_out

pytestmark = pytest.mark.gpu


def _check(path, G, S, above, inside, chosen, kinds, first_rows, paged, copies=1, last_stage="fused_decode"):
    Hkv, D, d = 2, 128, 16  # (copies: of the two KV heads, where the route needs many)
    k = above + chosen
    print("case", path, G, S, above, inside, chosen, kinds, first_rows, paged, flush=True)
    rng = np.random.default_rng(S + inside + kinds)
    kh = np.zeros((Hkv, S, D), np.float32)
    kh[..., d:] = rng.standard_normal((Hkv, S, D - d)) * 0.1
    score = np.empty((Hkv, S))
    for h in range(Hkv):
        where = np.concatenate([np.arange(inside), inside + rng.permutation(S - inside)]) if first_rows else rng.permutation(S)
        a = np.full(S, 0.25)                       # below
        fine = np.zeros(S, np.int64)
        fine[where[:inside]] = rng.permutation(1 << 16)[:kinds][rng.integers(0, kinds, inside)] if kinds < inside else \
            rng.permutation(1 << 16)[:inside]
        a[where[:inside]] = 1.0
        a[where[inside:inside + above]] = 3.0
        kh[h, :, 0], kh[h, :, 1], kh[h, :, 2] = a, (fine >> 8) * 2.0 ** -10, (fine & 255) * 2.0 ** -18
        score[h] = a + fine * 2.0 ** -18
    dt = torch.bfloat16
    kd = torch.from_numpy(kh).cuda().to(dt)[None]
    v = torch.randn((1, Hkv, S, D), generator=torch.Generator(device="cuda").manual_seed(S), device="cuda").to(dt)
    kd, v, Hkv = kd.repeat(1, copies, 1, 1), v.repeat(1, copies, 1, 1), Hkv * copies
    q = torch.zeros((1, Hkv * G, D), device="cuda")
    q[..., :3] = 1.0
    q[:, 1::G, d:] = 0.5  # (ranks nothing: the slab has no such column)
    q = q.to(dt)
    P = torch.eye(D, device="cuda").repeat(Hkv, 1, 1).contiguous()
    step = {}
    klo, khi, vv = kd[..., :d].contiguous(), kd[..., d:].contiguous(), v
    if paged:
        n = -(-S // 256)
        table = torch.randperm(n + 2, generator=torch.Generator().manual_seed(S))[:n].to(torch.int32)[None].cuda()

        def to_pool(t):
            pool = torch.zeros((n + 2, Hkv, 256, t.shape[-1]), dtype=dt, device="cuda")
            for p in range(n):
                rows = t[0, :, 256 * p:min(S, 256 * (p + 1))]
                pool[int(table[0, p]), :, :rows.shape[1]] = rows
            return pool
        klo, khi, vv = to_pool(klo), to_pool(khi), to_pool(v)
        step = dict(page_table=table, page_rows=256, n_pages=n + 2)
    lay = api.make_layout(1, Hkv * G, Hkv, D, d, S, dt)
    mode = 1 if G > 1 else 0
    ws = api.alloc_workspace(lay, S, d, k, mode)
    idx = torch.full((1, Hkv, k), -7, dtype=torch.int32, device="cuda")
    outs = []
    prof = api.Profile()
    prof.attach()
    try:
        for want in (idx, None):
            out = torch.full((1, Hkv * G, D), float("nan"), dtype=dt, device="cuda")
            api.loki_decode_step(lay, q, P, klo, khi, vv, S, d, k, mode | path, ws, out, want, **step)
            outs.append(out)
    finally:
        prof.detach()
    torch.cuda.synchronize()
    assert prof.read()[-1][0] == last_stage
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(idx, idx[:, :2].repeat(1, copies, 1))
    for h in range(2):
        sel = np.sort(np.argsort(-score[h], kind="stable")[:k])
        assert np.array_equal(idx[0, h].cpu().numpy(), sel)
        rows, val = kd[0, h].double().cpu().numpy()[sel], v[0, h].double().cpu().numpy()[sel]
        for g in range(G):
            a = rows @ q[0, h * G + g].double().cpu().numpy() / np.sqrt(D)
            p = np.exp(a - a.max())
            check_out(outs[0][0, h * G + g].float().cpu().numpy(), (p / p.sum()) @ val, "bf16", f"head {h} {g}")


# candidates up to the limits of the register forms (256, 1024), of the list (2048 with 256 threads) and past them;
# all, one or some of them chosen; distinct, a few values, one value
@pytest.mark.parametrize("paged", [False, True])
@pytest.mark.parametrize("S,above,inside,chosen,kinds", [
    (700, 40, 3, 1, 9), (700, 40, 3, 3, 9), (2000, 0, 64, 63, 99), (3000, 500, 256, 100, 999), (3000, 33, 257, 256, 999),
    (4000, 300, 1024, 1, 9999), (4000, 300, 1025, 700, 9999), (8000, 100, 2048, 1000, 9999), (8000, 100, 2049, 1000, 9999),
    (8000, 900, 1500, 700, 3), (8000, 900, 1500, 700, 1), (4000, 0, 4000, 1300, 9999)])
def test_candidates_one_block(S, above, inside, chosen, kinds, paged):
    _check(api.PATH_FUSED, 4, S, above, inside, chosen, kinds, False, paged)


# several blocks: up to 1024 candidates of a unit are exchanged as a list, more take another histogram
@pytest.mark.parametrize("S,above,inside,chosen,kinds,first", [
    (2000, 40, 3, 2, 9, False), (16000, 1000, 1024, 500, 9999, False), (16000, 1000, 1025, 1024, 9999, True),
    (16000, 50, 5000, 2500, 9999, False), (16000, 50, 5000, 2500, 5, False), (40000, 100, 8192, 3000, 9999, False),
    (40000, 100, 8193, 3000, 9999, False), (40000, 100, 5000, 3000, 9999, True), (40000, 100, 9000, 3000, 2, True),
    (40000, 3000, 30000, 1, 30000, False)])
def test_candidates_several_blocks(S, above, inside, chosen, kinds, first):
    _check(api.PATH_CLUSTER, 8 if S < 10000 else 2, S, above, inside, chosen, kinds, first, S <= 16000 and chosen % 2 == 0)


# the same with lists whose rows take long: 64 units, as many candidates as there are rows in a unit's list, up to
# 8192 and 4096 of a block
@pytest.mark.parametrize("S,above,inside,chosen,kinds,first", [
    (17000, 100, 1025, 925, 9999, False), (17000, 100, 4000, 3900, 9999, False), (17000, 100, 4001, 3900, 9999, False),
    (17000, 2000, 4000, 2000, 3, True), (40000, 1192, 8192, 7000, 9999, False), (40000, 1192, 8193, 7000, 9999, False),
    (40000, 1192, 6000, 5000, 9999, True), (40000, 4000, 4096, 4096, 9999, True)])
def test_candidates_of_long_lists(S, above, inside, chosen, kinds, first):
    _check(api.PATH_CLUSTER, 2, S, above, inside, chosen, kinds, first, False, copies=32)


# one block per head, keys in LDS: lists of up to 2048 candidates
@pytest.mark.parametrize("S,above,inside,chosen,kinds,paged", [
    (8193, 0, 1, 1, 9, False), (9000, 700, 256, 255, 999, True), (9000, 700, 1024, 1, 9999, False), (12000, 64, 1025, 600, 9999, False),
    (9000, 64, 2048, 1000, 9999, True), (9000, 64, 2049, 1000, 9999, False), (9000, 900, 1900, 700, 2, False),
    (9000, 900, 1900, 1100, 1, False), (9000, 0, 9000, 2048, 9999, False)])
def test_candidates_one_block_per_head(S, above, inside, chosen, kinds, paged):
    _check(0, 1, S, above, inside, chosen, kinds, False, paged, copies=64)


# selection inside the attention launch, which begins with the certain rows from 2049 to 8192 rows on (S stays beside
# that line: both forms report the same stage): lists of up to 1024 candidates, shares with and without certain rows
@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("S,above,inside,chosen,kinds,paged", [
    (2049, 0, 1, 1, 9, False), (2500, 40, 3, 2, 9, True), (4000, 700, 256, 255, 999, True), (4097, 700, 1024, 1000, 9999, False),
    (8000, 64, 1024, 700, 3, True), (8000, 64, 1025, 700, 9999, False), (8191, 100, 1000, 900, 9999, False), (3001, 0, 1024, 1024, 999, False),
    (5001, 1500, 900, 500, 1, True), (8192, 0, 8192, 2500, 9999, True), (8192, 100, 3000, 2000, 2, False), (2050, 33, 1300, 1, 9999, False)])
def test_candidates_in_the_attention_launch(G, S, above, inside, chosen, kinds, paged):
    assert 2048 < S <= 8192
    _check(api.PATH_SPLIT, G, S, above, inside, chosen, kinds, False, paged, last_stage="select_attend")


# the same launch with the whole list before the attention, and the selection in a launch of its own
@pytest.mark.parametrize("G,S,above,inside,chosen,kinds,paged,last_stage", [
    (1, 700, 40, 3, 2, 9, True, "select_attend"), (4, 2048, 40, 1025, 700, 99, False, "select_attend"),
    (4, 12000, 900, 600, 300, 9999, True, "select_attend"), (4, 16384, 3000, 900, 500, 1, False, "select_attend"),
    (1, 12000, 0, 12000, 3000, 9999, False, "gather_attend")])
def test_candidates_before_the_attention(G, S, above, inside, chosen, kinds, paged, last_stage):
    assert S <= 2048 or S > 8192
    _check(api.PATH_SPLIT, G, S, above, inside, chosen, kinds, False, paged, last_stage=last_stage)
