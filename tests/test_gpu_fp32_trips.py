"""One block per head, fp32: lists around the rows of a trip of the attention (64 and 128 rows), with up to 256
blocks and with more, against the same in 64 bits."""
import pytest
import torch

from perf import cases as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,S,k", [(1, 8, 8, 300, k) for k in (1, 63, 64, 65, 127, 128, 129, 255, 257, 300)] +
                         [(2, 160, 160, 330, k) for k in (1, 64, 129, 319, 320, 321)] + [(5, 64, 16, 400, k) for k in (129, 330)])
def test_lists(B, Hq, Hkv, S, k):
    c = C._decode("", B, Hq, Hkv, S, 32, k, dtype="f32", append=Hq == Hkv)
    print("case", c, flush=True)
    s = C.prepare(c, k)
    got = C.run(s)["out"].double()
    torch.cuda.synchronize()
    ref = C.exact(c, k)["out"]
    # 32-bit products and sums of up to 321 rows: 321 2^-24 at the worst, relative to the values' size
    assert float((got - ref).norm() / ref.norm()) < C.tolerance(c)["rel"]
