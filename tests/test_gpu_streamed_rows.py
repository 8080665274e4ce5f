"""Calls that read enough of their caches to load past the last-level cache (streams_rows in
csrc/api.hip), one for each kernel that has such a form, against the same in 64 bits."""
import pytest
import torch

from paper_2406_02542_amd import api
from perf import cases as C

pytestmark = pytest.mark.gpu


def decode(*a, **kw):
    return C._decode("", *a, **kw)


CASES = {
    # one block per head: both types, row widths on both forms of the scoring, the append, pages, long rows
    "fused": decode(8, 32, 32, 1900, 32, 475, append=True),
    "fused_paged": decode(12, 32, 32, 2100, 64, 525, append=True, ragged=True, paged=True),
    "fused_f32": decode(3, 64, 64, 1100, 32, 333, dtype="f32"),
    "fused_wide_f32": decode(3, 64, 64, 1000, 96, 333, dtype="f32", append=True),
    "fused_long": decode(6, 32, 32, 8300, 16, 1001),
    "fused_grouped": decode(8, 32, 16, 4000, 32, 800),
    # one block per group, 512 and 256 threads, and several blocks per group
    "group_alone": decode(10, 32, 8, 5000, 32, 1250, mode="group", append=True),
    "group_two_per_cu": decode(34, 32, 8, 1900, 64, 475, mode="group", append=True),
    "group_paged": decode(46, 16, 8, 2000, 32, 700, mode="group", append=True, ragged=True, paged=True),
    "cluster": decode(4, 64, 8, 12000, 64, 3000, mode="group", append=True),
    "cluster_paged": decode(6, 32, 8, 11000, 16, 2750, mode="group", append=True, paged=True),
    # the same with the slab past the caches while it is scored (few rows kept beside 80 MB of slab and more)
    "group_alone_slab": decode(24, 32, 8, 9001, 32, 600, mode="group", append=True),
    "group_two_per_cu_slab": decode(64, 64, 8, 2801, 32, 170, mode="group", append=True),
    "group_paged_slab": decode(64, 16, 8, 4000, 32, 250, mode="group", append=True, ragged=True, paged=True),
    "cluster_slab": decode(8, 32, 8, 22001, 32, 1300, mode="group", append=True),
    "cluster_paged_slab": decode(4, 32, 8, 90001, 16, 2800, mode="group", append=True, paged=True),
    # selection and attention of the split path: one launch on the vector units and the matrix cores, two launches
    "tokens": decode(3, 32, 32, 5001, 32, 1250, append=True, tokens=2),
    "tokens_group": decode(8, 32, 8, 5001, 32, 1250, mode="group", append=True, tokens=2),
    "few_heads": decode(5, 8, 8, 16000, 32, 4000, append=True),
    "few_heads_f32": decode(5, 8, 8, 8000, 32, 3000, dtype="f32", append=True),
    "long_head": decode(2, 16, 16, 20000, 64, 2500, append=True),
    "long_group_f32": decode(2, 16, 8, 20000, 32, 2500, dtype="f32", mode="group"),
    "many_groups": decode(8, 128, 32, 3000, 8, 800, mode="group"),
    # dense attention: matrix cores and vector units, equal and unequal lengths
    "dense_mfma": {"kind": "dense", "B": 5, "Hq": 32, "Hkv": 8, "S": 5003, "dtype": "bf16", "ragged": False},
    "dense_mfma_ragged": {"kind": "dense", "B": 10, "Hq": 64, "Hkv": 8, "S": 5003, "dtype": "bf16", "ragged": True},
    "dense_f32": {"kind": "dense", "B": 3, "Hq": 32, "Hkv": 8, "S": 4001, "dtype": "f32", "ragged": False},
    "dense_ragged": {"kind": "dense", "B": 9, "Hq": 32, "Hkv": 32, "S": 1303, "dtype": "bf16", "ragged": True},
    # the Gram pass
    "fit": {"kind": "fit", "Hkv": 16, "N": 20001, "dtype": "bf16", "tau": 20.0},
}


@pytest.mark.parametrize("name", CASES)
def test_streamed(name):
    c = CASES[name]
    print(f"case {name} {c}", flush=True)
    assert C.work(c)["bytes"] > 5e7  # (unequal lengths: the rule counts 0.55 of what the longest makes)
    s = C.prepare(c, 5)
    got = {k: v.clone() for k, v in C.run(s).items()}
    torch.cuda.synchronize()
    del s
    ref = C.exact(c, 5)
    tol = C.tolerance(c)["rel"]
    for key, r in ref.items():
        g, r = got[key].double().cpu(), r.double().cpu()
        err = float((g - r).norm() / r.norm())
        print(f"  {key}: {err:.2e}", flush=True)
        assert err <= tol, (key, err)


@pytest.mark.parametrize("G,d", [(1, 32), (4, 40)])
def test_streamed_pca_attn(G, d):
    """Appendix E, Algorithm 2, on the vector units and the matrix cores."""
    B, H, S = 8, 8, 9001
    gen = torch.Generator(device="cuda").manual_seed(G)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device="cuda")
    P = torch.linalg.qr(rnd(H, 128, 128).double())[0].float().contiguous()
    klo, v, q = rnd(B, H, S, d).bfloat16(), rnd(B, H, S, 128).bfloat16(), rnd(B, H * G, 128).bfloat16()
    lay = api.make_layout(B, H * G, H, 128, d, S, torch.bfloat16)
    out = torch.empty_like(q)
    ws = api.alloc_workspace(lay, S, d, 0, -2)
    api.loki_pca_attn(lay, q, P, klo, v, S, d, ws, out)
    torch.cuda.synchronize()
    for b in range(B):
        for h in range(H):
            qh = q[b, h * G:(h + 1) * G].double() @ P[h].double()
            a = (qh[:, :d] @ klo[b, h].double().t().contiguous()) / 128 ** 0.5
            ref = torch.softmax(a, -1) @ v[b, h].double()
            err = float((out[b, h * G:(h + 1) * G].double() - ref).norm() / ref.norm())
            assert err < 6e-3, (b, h, err)
