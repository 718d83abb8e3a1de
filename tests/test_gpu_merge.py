"""The batch plan's sorted form (all query keys sorted once, walked in chunks
against 64 references at a time) against numpy's ranks: reference counts
around the 64 lanes, one to the most query sets, empty sets and references, a
single interval, equal keys, references far denser than the queries of a
chunk, ends of 2^32 - 1, and intervals with start > end (counted 0 and
flagged).  The plan is replayed with new queries in the same buffers."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1208_3407_amd import bits  # noqa: E402

DEV = torch.device("cuda", 0)
TOP = 2**32 - 1


def up(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32)).to(DEV)


def queries(rng, n, kind):
    s = rng.integers(0, 2_000_000_000, n) if kind == "wide" else rng.integers(1_000_000, 1_200_000, n)
    e = s + rng.integers(0, 50_000, n)
    if kind == "equal":
        s[:], e[:] = 1_100_000, 1_100_500
    if n > 10:
        e[0], s[1], e[1] = TOP, 0, 0
    return s, e


@pytest.mark.parametrize("n_q,n_ref,total,kind", [
    (1, 24, 1 << 20, "wide"), (3, 63, 270_000, "narrow"), (33, 64, 263_000, "wide"), (192, 65, 259_000, "wide"),
    (7, 130, 131_000, "equal"), (20, 200, 90_000, "narrow")])
def test_merged_pairs(n_q, n_ref, total, kind):
    print("case:", n_q, n_ref, total, kind, flush=True)
    rng = np.random.default_rng(n_q * 1000 + n_ref)
    cut = np.sort(rng.integers(0, total + 1, n_q - 1))
    na = np.diff(np.concatenate([[0], cut, [total]]))
    if n_q > 2:
        na[0], na[1] = 0, na[0] + na[1]      # an empty set
    sizes = np.rint(np.exp(rng.uniform(0, np.log(30_000), n_ref))).astype(np.int64)
    sizes[0], sizes[1], sizes[2] = 0, 1, 300_000
    refs, host = [], []
    for j, n in enumerate(sizes):
        s = rng.integers(0, 2_000_000_000, n) if j % 3 else rng.integers(1_000_000, 1_200_000, n)
        if j == 3:
            s[:] = 1_100_000
        e = s + rng.integers(0, 10_000, n)
        host.append((np.sort(s), np.sort(e)))
        refs.append((up(s), up(e)))
    refs = bits.bits_sort_refs(refs)
    sets = [queries(rng, int(n), kind) for n in na]
    dev = [(up(s), up(e)) for s, e in sets]
    plan = bits.bits_batch_create(refs, dev)
    for rnd in range(3):
        got = bits.bits_batch_run(plan).cpu().numpy().reshape(n_q, n_ref)
        exp = np.zeros((n_q, n_ref), np.uint64)
        for i, (s, e) in enumerate(sets):
            ok = s <= e
            for j, (bs, be) in enumerate(host):
                exp[i, j] = (np.searchsorted(bs, e[ok], "right").sum() - np.searchsorted(be, s[ok], "left").sum())
        assert np.array_equal(got, exp), rnd
        bad = any((s > e).any() for s, e in sets)
        assert bits.bits_get_status(refs[0]) == (bits.BITS_FLAG_INTERVAL if bad else 0)
        # new queries in the same buffers; the last replay has intervals with start > end
        for i, (s, e) in enumerate(sets):
            s, e = queries(rng, len(s), kind)
            if rnd == 1 and len(s) > 100:
                s[5:9], e[5:9] = e[5:9] + 1, s[5:9]
            sets[i] = s, e
            dev[i][0].copy_(up(s))
            dev[i][1].copy_(up(e))
    # the search per pair gives the same totals
    other = bits.bits_batch_create(refs, dev, launch={"path": bits.BITS_PATH_PLAIN})
    plan_totals = bits.bits_batch_run(plan).clone()
    assert torch.equal(plan_totals.view(torch.int64), bits.bits_batch_run(other).view(torch.int64))
