"""The learned count's second search, looked for next to the first rank: which
queries take the search in full, read off the fallback counter of a reference
whose models all predict their leaf's first rank (a search in full then misses
its window for about half of the keys)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1208_3407_amd import bits  # noqa: E402

DEV = torch.device("cuda", 0)
N, STEP, LEN = 4_000_000, 700, 350   # B: [700 i, 700 i + 349]
SHAPES = [None] + [{"path": 2, "block": b, "qpl": q} for b in (256, 512) for q in (1, 2, 4)]


def up(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32)).to(DEV)


@pytest.fixture(scope="module")
def ref():
    s = np.arange(N, dtype=np.int64) * STEP
    r = bits.bits_sort_ref(up(s), up(s + LEN - 1), learned=True, train={"epochs": 0})
    raw = r.rmi_bytes()
    for a in range(2):
        base = a * bits.RMI_MODEL_BYTES + bits.RMI_HEADER_BYTES
        words = raw[base:base + 4096 * bits.RMI_LEAF_BYTES].view(torch.int32).view(4096, 32)
        for w in (2, 3, 6, 7, 9, 10, 11, 12, 14, 15):   # w1, b2, error bounds
            words[:, w] = 0
        words[:, 16:32] = 0                             # b1 and w2
    torch.cuda.synchronize()
    return r


def run(ref, rank, launch):
    """Queries [700 r, 700 r + 100]: r ends lie before each, one interval meets it.  Fallbacks of the count."""
    f0 = bits.bits_rmi_info(ref)["fallbacks"]
    counts, total = bits.bits_count_per_query(ref, up(rank * STEP), up(rank * STEP + 100), launch=launch)
    assert bool((counts.view(torch.int32) == 1).all()) and int(total.view(torch.int64)[0]) == len(rank)
    return bits.bits_rmi_info(ref)["fallbacks"] - f0


def test_ranks_on_line_boundaries(ref):
    """Four queries of a wave at ranks that are multiples of 32, the others in mid-line: no more full
    searches than with all of them in mid-line."""
    rng = np.random.default_rng(3)
    rank = rng.integers(1, N // 32 - 1, 64_000) * 32 + 5
    mid = [run(ref, rank, s) for s in SHAPES]
    assert len(set(mid)) == 1 and mid[0] > 10_000
    edge = rank - 5 * (np.arange(len(rank)) % 16 == 0)
    got = [run(ref, edge, s) for s in SHAPES]
    # the first search of a moved query can change leaves, the second must not run
    assert abs(got[0] - mid[0]) <= 100, (got, mid)


def test_looks_do_not_depend_on_the_wave(ref):
    """All ranks on line boundaries, so that every lane needs its second look: the searches that run in full
    are those of a mid-line set, at every launch shape."""
    rng = np.random.default_rng(4)
    rank = rng.integers(1, N // 32 - 1, 20_000) * 32
    mid = run(ref, rank + 5, None)
    got = [run(ref, rank, s) for s in SHAPES]
    assert len(set(got)) == 1 and abs(got[0] - mid) <= 600, (got, mid)   # 600: 3% of the first searches in other leaves


def test_batch_searches_as_the_count(ref):
    """A batch plan over references with models takes the same searches as a count of each pair: totals and
    fallbacks agree, references around the size where both searches of a query go in step among them."""
    rng = np.random.default_rng(5)
    q = [(up(s), up(s + 100)) for s in (rng.integers(0, N * STEP, n) for n in (1, 900, 5000))]
    refs = [ref]
    for n in (1, 32_767, 32_768, 32_769, 65_537):
        s = rng.integers(0, N * STEP, n)
        refs.append(bits.bits_sort_ref(up(s), up(s + LEN), learned=True, train={"epochs": 5, "max_points": 64}))

    def fallbacks():
        return [bits.bits_rmi_info(r)["fallbacks"] for r in refs]

    f0 = fallbacks()
    exp = torch.stack([torch.cat([bits.bits_count(r, *a).view(torch.int64) for r in refs]) for a in q])
    f1 = fallbacks()
    plan = bits.bits_batch_create(refs, q)
    assert torch.equal(bits.bits_batch_run(plan).view(torch.int64).view(len(q), len(refs)), exp)
    f2 = fallbacks()
    bits.bits_batch_destroy(plan)
    assert [b - a for a, b in zip(f0, f1)] == [c - b for b, c in zip(f1, f2)] and f2[0] > f1[0] > f0[0]
