"""Whether a call loads its rows past the last-level cache: by the rows it holds, not by the longest it could hold."""
import itertools

import pytest
import torch

from paper_2406_02542_amd import api

SET = 256  # any address: only whether a pointer is set counts
DT = {"bf16": torch.bfloat16, "f32": torch.float32}


def form(B, Hq, Hkv, S, d, k, mode, lens=None, ks=None, tokens=1, dtype="bf16", paged=False):
    lay = api.make_layout(B, Hq, Hkv, 128, d, S, DT[dtype])
    if lens is None and not paged:
        return api.loki_debug_row_loads(lay, S, d, k, mode)
    args = api.StepArgs(queries_per_seq=tokens)
    if paged:
        args.page_table, args.page_rows, args.pages_per_seq, args.n_pages = SET, 256, -(-S // 256), B * -(-S // 256)
    if lens is None:
        return api.loki_debug_row_loads(lay, S, d, k, mode, args)
    args.seq_lens = SET
    if ks is not None:
        args.ks = SET
    kept = [min(x, k, n) for x, n in zip(ks if ks is not None else [k] * len(lens), lens)]
    return api.loki_debug_row_loads(lay, S, d, k, mode, args, sum(lens), sum(kept))


def test_short_sequences_in_a_long_cache_stay_in_the_caches():
    # 16 x 32 heads, k = S / 4: 16 x 32 x 512 rows of 64 bytes, and 128 kept of 448, 46 MB; by the longest 369 MB
    assert form(16, 32, 32, 4096, 32, 1024, 0, [512] * 16, [128] * 16) == 0
    assert form(16, 32, 32, 4096, 32, 1024, 0, [512] * 16, [128] * 16, paged=True) == 0
    assert form(16, 32, 32, 4096, 32, 1024, 0, [4096] * 16, [1024] * 16) == 1
    # dense attention, 16 x 8 KV heads: 512 bytes a row
    assert form(16, 32, 8, 16384, 128, 16384, -1, [1000] * 16) == 0
    assert form(16, 32, 8, 16384, 128, 16384, -1, [2000] * 16) == 1
    # one selection per group: 43 MB of slab and 42 of selected rows, then 268 and 184
    assert form(64, 64, 8, 8192, 32, 1024, 1, [1300] * 64, [160] * 64) == 0
    assert form(64, 64, 8, 8192, 32, 1024, 1, [8192] * 64, [700] * 64) == 2
    # two tokens of a sequence: each holds the sequence's rows
    assert form(4, 32, 32, 8192, 32, 2048, 0, [900] * 8, [220] * 8, tokens=2) == 0
    assert form(4, 32, 32, 8192, 32, 2048, 0, [8192] * 8, [2048] * 8, tokens=2) == 1


@pytest.mark.parametrize("dtype,mode,G", itertools.product(["bf16", "f32"], [-1, 0, 1], [1, 4]))
def test_equal_lengths_are_the_same_call(dtype, mode, G):
    """Sequences that all hold S rows load as they do without lengths, at every size."""
    seen = set()
    for B, S in itertools.product([2, 5, 8, 12, 16, 40], [1000, 1700, 2600, 4096, 9000, 16384]):
        Hkv, d, k = 8, 32 if mode >= 0 else 128, S // 8 if mode >= 0 else S
        if mode >= 0 and dtype == "bf16" and G == 4 and mode == 1 and S > 8192:
            continue  # (which launch a group takes there turns on whether it has lengths)
        a = form(B, G * Hkv, Hkv, S, d, k, mode, dtype=dtype)
        b = form(B, G * Hkv, Hkv, S, d, k, mode, [S] * B, [k] * B if mode >= 0 else None, dtype=dtype)
        assert a == b, (B, S, a, b)
        seen.add(a)
    assert len(seen) > 1  # both sides of the line


def test_the_line_lies_at_the_bytes_that_are_read():
    """Lengths of any mix: past the caches from 90 MB of slab and selected rows on."""
    import random
    rng = random.Random(3)
    both = set()
    for _ in range(400):
        B, S = rng.randrange(2, 65), rng.randrange(600, 8192)
        k = S // rng.choice([4, 8, 16])
        lens = [rng.randrange(1, S + 1) for _ in range(B)]
        ks = [max(1, n * k // S) for n in lens]
        mb = 32 * 2 * sum(32 * n + 224 * min(x, k, n) for n, x in zip(lens, ks)) / 1e6
        if abs(mb - 90) < 0.1:
            continue
        got = form(B, 32, 32, S, 32, k, 0, lens, ks)
        assert got == (1 if mb > 90 else 0), (B, S, k, mb)
        both.add(got)
    assert both == {0, 1}
