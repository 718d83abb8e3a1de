"""The search without a model (LDS top tree, interpolated window of line heads
or keys, one line) at the sizes where its windows end: buckets of one window
and one key more, arrays of less than a line and of lines plus or minus one
key, both sides of the size where windows of keys give way to line heads, and
key patterns that a straight line does not predict (equal keys, runs far
apart, a curve).  Counts, first ranks, decisions and Monte-Carlo observed
totals against the oracle; the re-sorting Monte-Carlo, whose rounds are
searched the same way, against the other orientation."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1208_3407_amd import bits  # noqa: E402

DEV = torch.device("cuda", 0)
TOP = 2**32 - 1


def up(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32)).to(DEV)


def keys(kind, n, rng):
    if kind == "uniform":
        s = rng.integers(0, 2_900_000_000, n)
    elif kind == "equal":
        s = np.full(n, 1_000_000)
    elif kind == "runs":            # a few dense runs far apart
        s = rng.integers(0, 7, n) * 400_000_000 + rng.integers(0, 1 + n // 8, n)
    else:                           # "curve": density falls off steeply
        s = (2.9e9 * rng.random(n) ** 6).astype(np.int64)
    s = s.astype(np.int64)
    e = s + rng.integers(0, 1000, n)
    e[rng.random(n) < 0.001] = TOP
    return s.astype(np.uint32), e.astype(np.uint32)


@pytest.mark.parametrize("kind", ["uniform", "equal", "runs", "curve"])
@pytest.mark.parametrize("n", [1, 2, 3, 28, 29, 32, 33, 1000, 8193, 28 * 8192 + 1, 1 << 19, (1 << 19) + 1, 1_000_003])
def test_windows(kind, n):
    print("case:", kind, n, flush=True)
    rng = np.random.default_rng(n * 4 + len(kind))
    bs, be = keys(kind, n, rng)
    near = np.concatenate([bs, be])[rng.integers(0, 2 * n, 3000)].astype(np.int64) + rng.integers(-2, 3, 3000)
    a0 = np.clip(np.concatenate([near, rng.integers(0, 2**32, 1500), [0, 0, TOP]]), 0, TOP)
    a1 = np.minimum(a0 + np.concatenate([rng.integers(0, 2000, 4500), [0, TOP, 0]]), TOP)
    sbs, sbe = np.sort(bs), np.sort(be)
    exp, total = oracle.count_sorted(sbs, sbe, a0.astype(np.uint32), a1.astype(np.uint32))
    first = np.searchsorted(sbs, a1, side="right")
    ref = bits.bits_sort_ref(up(bs), up(be))
    qa = up(a0), up(a1)
    for launch in (None, {"path": 3, "depth": 0, "block": 256, "qpl": 1}, {"path": 3, "depth": 5, "qpl": 4},
                   {"path": 0, "depth": 1, "block": 512, "qpl": 2}):
        counts, tot = bits.bits_count_per_query(ref, *qa, launch=launch)
        assert np.array_equal(counts.cpu().numpy(), exp), launch
        assert int(tot.item()) == total, launch
    counts, got_first, offsets = bits.bits_enum_counts(ref, *qa)
    assert np.array_equal(got_first.cpu().numpy(), first)
    assert np.array_equal(offsets.cpu().numpy()[1:], np.cumsum(exp.astype(np.uint64)))
    found, witness = bits.bits_decide(ref, *qa)
    assert int(found.item()) == int(total > 0)
    if total:
        assert exp[int(witness.item())] > 0
    # one chromosome of the whole range: the observed total of the Monte-Carlo entry point
    inside = a1 < TOP
    mc = bits.bits_mc_pvalue(ref, up(a0[inside]), up(a1[inside]), [TOP], 7, 0, 2)
    assert int(mc.observed.item()) == int(exp[inside].astype(np.uint64).sum())
    assert bits.bits_get_status(ref) == 0


@pytest.mark.parametrize("nb,rounds,batch", [(1, 3, 2), (2, 9, 9), (31, 8, 8), (33, 17, 16), (100, 1, 1),
                                             (8193, 20, 12), (28 * 8192 + 5, 10, 10), ((1 << 19) + 37, 9, 9)])
def test_resort_rounds(nb, rounds, batch):
    print("case: resort", nb, rounds, batch, flush=True)
    rng = np.random.default_rng(nb)
    lens = [40_000_000, 300_000, 1_000]
    off = np.concatenate([[0], np.cumsum(lens)])

    def one(n):
        c = rng.integers(0, 3, n)
        L = rng.integers(1, 900, n)
        s = off[c] + (rng.random(n) * (np.array(lens)[c] - L)).astype(np.int64)
        return s, s + L - 1
    a, b = one(2500), one(nb)
    if nb > 50:
        b[1][7] += 50_000_000                    # outside its chromosome
    qa, qb = (up(a[0]), up(a[1])), (up(b[0]), up(b[1]))
    status = torch.zeros(1, dtype=torch.uint32, device=DEV)
    got = bits.bits_mc_resort(*qa, *qb, lens, 11, 3, 3 + rounds, batch=batch, status=status)
    exp = bits.bits_mc_pvalue(bits.bits_sort_ref(*qa), *qb, lens, 11, 3, 3 + rounds)
    for name in ("totals", "observed", "n_ge", "n_le"):
        assert torch.equal(getattr(got, name).view(torch.int64), getattr(exp, name).view(torch.int64)), name
    assert int(status.item()) == (bits.BITS_FLAG_CHROM if nb > 50 else 0)


def near_sets(n, rng):
    """References and queries that the second search's start near the first one's rank does not fit: long
    intervals on either side, many equal keys, intervals with start > end in B (not checked there: the
    difference of the two ranks then wraps), the first and last coordinates."""
    s = np.concatenate([rng.integers(0, 2_900_000_000, n - n // 2),
                        rng.normal(1_000_000_000, 40_000, n // 2).astype(np.int64)])
    e = s + np.where(rng.random(n) < 0.01, rng.integers(0, 3_000_000, n), rng.integers(0, 900, n))
    swap = rng.random(n) < 0.02
    s[swap], e[swap] = e[swap], s[swap]
    s[: n // 50] = 1_000_000_100
    m = 20_000
    a = rng.integers(0, 2_950_000_000, m)
    a[: m // 2] = rng.normal(1_000_000_000, 60_000, m // 2).astype(np.int64)
    z = a + np.where(rng.random(m) < 0.1, rng.integers(0, 100_000_000, m), rng.integers(0, 700, m))
    z[:3], a[1:4] = TOP, 0
    a[4:8], z[4:8] = 1_000_000_100, 1_000_000_100
    return s, e, a, np.minimum(z, TOP)


@pytest.mark.parametrize("n", [1, 33, 5_000, 300_007])
def test_second_rank_next_to_the_first(n):
    print("case: near", n, flush=True)
    s, e, a, z = near_sets(n, np.random.default_rng(n))
    exp = (np.searchsorted(np.sort(s), z, "right") - np.searchsorted(np.sort(e), a, "left")) % 2**32
    ref = bits.bits_sort_ref(up(s), up(e), learned=True, train={"epochs": 10})
    for launch in (None, {"path": 2, "block": 256, "qpl": 1}, {"path": 2, "qpl": 4}, {"path": 3}, {"path": 1}):
        counts, _ = bits.bits_count_per_query(ref, up(a), up(z), launch=launch)
        assert np.array_equal(counts.cpu().numpy().astype(np.int64), exp), launch


def test_second_rank_next_to_the_first_large():
    n = (1 << 24) + 77
    s, e, a, z = near_sets(n, np.random.default_rng(9))
    exp = (np.searchsorted(np.sort(s), z, "right") - np.searchsorted(np.sort(e), a, "left")) % 2**32
    ref = bits.bits_sort_ref(up(s), up(e))
    for launch in (None, {"path": 3, "depth": 0, "block": 256, "qpl": 2}, {"path": 3, "depth": 7}):
        counts, _ = bits.bits_count_per_query(ref, up(a), up(z), launch=launch)
        assert np.array_equal(counts.cpu().numpy().astype(np.int64), exp), launch
