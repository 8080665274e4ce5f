"""Calls that read enough of their caches to load past the last-level cache (row_loads in csrc/api.hip), one for each
kernel that has such a form, against the same in 64 bits; that they do so is asked of the library."""
import pytest
import torch

from paper_2406_02542_amd import api
from perf import cases as C

pytestmark = pytest.mark.gpu


def decode(*a, **kw):
    return C._decode("", *a, **kw)


ONE, SPLIT, TWO = ["fused_decode"], ["select_attend"], ["select", "gather_attend"]
# case, the kernels that load its rows (of the split path the last), and how these load its rows (0 through the caches, 1 past them, 2 the slab of a
# group too)
CASES = {
    # one block per head: both types, row widths on both forms of the scoring, the append, pages, long rows
    "fused": (decode(9, 32, 32, 1900, 32, 475, append=True), ONE, 1),
    "fused_paged": (decode(12, 32, 32, 2100, 64, 525, append=True, ragged=True, paged=True), ONE, 1),
    "fused_lengths": (decode(16, 32, 32, 2100, 32, 525, append=True, ragged=True), ONE, 1),
    "fused_short_lengths": (decode(10, 32, 32, 2100, 32, 525, append=True, ragged=True), ONE, 0),
    "fused_f32": (decode(3, 64, 64, 1400, 32, 333, dtype="f32"), ONE, 1),
    "fused_wide_f32": (decode(3, 64, 64, 1000, 96, 333, dtype="f32", append=True), ONE, 1),
    "fused_long": (decode(8, 32, 32, 8300, 16, 1001), ONE, 1),
    # one block per group, 512 and 256 threads, and several blocks per group
    "group_alone": (decode(13, 32, 8, 5000, 32, 1250, mode="group", append=True), ONE, 1),
    "group_two_per_cu": (decode(34, 32, 8, 1900, 64, 475, mode="group", append=True), ONE, 1),
    "group_paged": (decode(64, 16, 8, 2500, 32, 850, mode="group", append=True, ragged=True, paged=True), ONE, 1),
    "cluster": (decode(4, 64, 8, 12000, 64, 3000, mode="group", append=True), ONE, 1),
    "cluster_paged": (decode(7, 32, 8, 11000, 16, 2750, mode="group", append=True, paged=True), ONE, 1),
    # the same with the slab past the caches while it is scored (few rows kept beside 80 MB of slab and more)
    "group_alone_slab": (decode(24, 32, 8, 9001, 32, 600, mode="group", append=True), ONE, 2),
    "group_two_per_cu_slab": (decode(64, 64, 8, 2801, 32, 170, mode="group", append=True), ONE, 2),
    "group_paged_slab": (decode(64, 16, 8, 5000, 32, 310, mode="group", append=True, ragged=True, paged=True), ONE, 2),
    "cluster_slab": (decode(8, 32, 8, 22001, 32, 1300, mode="group", append=True), ONE, 2),
    "cluster_paged_slab": (decode(4, 32, 8, 90001, 16, 2800, mode="group", append=True, paged=True), ONE, 2),
    # selection and attention of the split path: one launch on the vector units and the matrix cores, two launches
    "tokens": (decode(3, 32, 32, 5001, 32, 1250, append=True, tokens=2), SPLIT, 1),
    "tokens_group": (decode(8, 32, 8, 5001, 32, 1250, mode="group", append=True, tokens=2), SPLIT, 1),
    "few_heads": (decode(5, 8, 8, 16000, 32, 4000, append=True), TWO, 1),
    "few_heads_f32": (decode(5, 8, 8, 8000, 32, 3000, dtype="f32", append=True), SPLIT, 1),
    "long_head": (decode(2, 16, 16, 20000, 64, 2500, append=True), TWO, 1),
    "long_group_f32": (decode(3, 16, 8, 20000, 32, 2500, dtype="f32", mode="group"), TWO, 1),
    "many_groups": (decode(8, 128, 32, 3000, 8, 800, mode="group"), SPLIT, 1),
    "group_heads": (decode(10, 64, 8, 8000, 64, 450), SPLIT, 1),  # every head of a group for itself
    # dense attention: matrix cores and vector units, equal and unequal lengths
    "dense_mfma": ({"kind": "dense", "B": 5, "Hq": 32, "Hkv": 8, "S": 5003, "dtype": "bf16", "ragged": False}, None, 1),
    "dense_mfma_ragged": ({"kind": "dense", "B": 10, "Hq": 64, "Hkv": 8, "S": 5003, "dtype": "bf16", "ragged": True}, None, 1),
    "dense_f32": ({"kind": "dense", "B": 3, "Hq": 32, "Hkv": 8, "S": 4001, "dtype": "f32", "ragged": False}, None, 1),
    "dense_ragged": ({"kind": "dense", "B": 11, "Hq": 32, "Hkv": 32, "S": 1303, "dtype": "bf16", "ragged": True}, None, 1),
    "dense_short_lengths": ({"kind": "dense", "B": 5, "Hq": 32, "Hkv": 32, "S": 1303, "dtype": "bf16", "ragged": True}, None, 0),
    # the Gram pass, which loads past the caches from 80 MB of keys on
    "fit": ({"kind": "fit", "Hkv": 16, "N": 20001, "dtype": "bf16", "tau": 20.0}, None, None),
}


def loads(s):
    """How the library says that this call loads its rows."""
    c, x = s["c"], s["x"]
    rows = float(x["lens"].sum())
    if c["kind"] == "dense":
        args = api.StepArgs(seq_lens=s["lens"].data_ptr()) if c["ragged"] else None
        return api.loki_debug_row_loads(s["lay"], c["S"], 128, c["S"], -1, args, rows, rows)
    step = dict(s["step"])
    table = step.pop("page_table", None)
    args = api.StepArgs(**{k: v.data_ptr() if isinstance(v, torch.Tensor) else v for k, v in step.items()})
    if table is not None:
        args.page_table, args.pages_per_seq = table.data_ptr(), table.shape[1]
    return api.loki_debug_row_loads(s["lay"], c["S"], c["d"], c["k"], s["mode"], args, rows, float(x["ks"].sum()))


@pytest.mark.parametrize("name", CASES)
def test_streamed(name):
    c, kernels, form = CASES[name]
    print(f"case {name} {c}", flush=True)
    s = C.prepare(c, 5)
    if form is not None:
        assert loads(s) == form
    else:
        assert C.work(c)["bytes"] > 8.1e7
    prof = api.Profile()
    prof.attach()
    try:
        got = {k: v.clone() for k, v in C.run(s).items()}
    finally:
        prof.detach()
    torch.cuda.synchronize()
    names = [n for n, _ in prof.read()]
    print(" ", names, flush=True)
    if kernels is not None:
        assert names[-len(kernels):] == kernels
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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("ragged", [False, True])
def test_the_form_does_not_change_results(dtype, ragged):
    """One block per head: a large batch past the caches, and its first sequences as a batch of their own through them,
    are the same bit for bit."""
    c = decode(16, 32, 32, 2701, 32, 500, dtype=dtype, ragged=ragged)
    s = C.prepare(c, 7)
    x, n, dt = s["x"], 3, C._dtype(c)
    if ragged:
        x["lens"].sort()  # the first sequences are the short ones
        x["ks"][:] = [max(1, int(r) * c["k"] // c["S"]) for r in x["lens"]]
        s["step"] = {k: torch.from_numpy(x[v]).cuda() for k, v in [("seq_lens", "lens"), ("ks", "ks")]}

    def loaded_and_out(B):
        lay = api.make_layout(B, 32, 32, 128, c["d"], x["cap"], dt)
        rows, kept = float(x["lens"][:B].sum()), float(x["ks"][:B].sum())
        step = {k: v[:B] for k, v in s["step"].items()}
        args = api.StepArgs(**{k: v.data_ptr() for k, v in step.items()}) if step else None
        form = api.loki_debug_row_loads(lay, c["S"], c["d"], c["k"], 0, args, rows, kept)
        ws = api.alloc_workspace(lay, c["S"], c["d"], c["k"], 0)
        out = torch.empty((B, 32, 128), dtype=dt, device="cuda")
        api.loki_decode_step(lay, x["q"][:B], x["P"], x["klo"][:B], x["khi"][:B], x["v"][:B], c["S"], c["d"], c["k"], 0, ws, out, **step)
        return form, out

    (form_all, all_), (form_few, few) = loaded_and_out(16), loaded_and_out(n)
    torch.cuda.synchronize()
    assert (form_all, form_few) == (1, 0)
    assert torch.equal(all_[:n], few)
