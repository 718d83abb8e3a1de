"""Binned Monte-Carlo placement where chromosomes hold very different numbers of
queries, so that workgroups take shares of the shuffles by cost: one or few of
many chromosomes loaded, chromosomes without length or without queries, one
just at and just past the cost at which shares are taken, several passes with
an uneven last one.  Totals against the query-ordered entry point."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1208_3407_amd import bits  # noqa: E402

DEV = torch.device("cuda", 0)


def up(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32)).to(DEV)


@pytest.mark.parametrize("lens,counts,shuffles,batch", [
    ([50_000_000] + [20_000] * 255, [20_000] + [0] * 255, 90, 90),
    ([50_000_000] + [20_000] * 255, [1] * 255 + [9_000], 300, 131),
    ([30_000_000, 0, 0, 40_000_000, 0, 10_000], [30_000, 0, 0, 10, 0, 0], 700, 300),
    ([10_000_000] * 24, [9_500] + [0] * 23, 1024, 1024),
    ([10_000_000] * 24, [0] * 12 + [4_000] * 12, 257, 200),
    ([10_000_000] * 64, [63 * 500] + [500] * 63, 200, 77),
    ([10_000_000] * 65, [1_000] * 64 + [5_000], 200, 200),
    ([100_000_000], [7_000], 1000, 999),
    ([20_000_000] * 2, [8_000, 7_999], 1024, 1000),
])
def test_totals(lens, counts, shuffles, batch):
    print("case:", len(lens), sum(counts), shuffles, batch, flush=True)
    rng = np.random.default_rng(len(lens) + shuffles)
    off = np.concatenate([[0], np.cumsum(lens)])
    s = np.concatenate([off[c] + rng.integers(0, lens[c] - 900, n) for c, n in enumerate(counts) if n])
    s = rng.permutation(s)
    b = rng.integers(0, int(off[-1]) - 400, 30_000)
    q = up(s), up(s + rng.integers(0, 900, len(s)))
    ref = bits.bits_sort_ref(up(b), up(b + 399))
    got = bits.bits_mc_binned(ref, *q, lens, 11, 5, 5 + shuffles, batch=batch)
    exp = bits.bits_mc_pvalue(ref, *q, lens, 11, 5, 5 + shuffles)
    assert torch.equal(got.totals.view(torch.int64), exp.totals.view(torch.int64))
    assert torch.equal(got.observed.view(torch.int64), exp.observed.view(torch.int64))
    assert bits.bits_get_status(ref) == 0
