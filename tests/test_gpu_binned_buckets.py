"""The binned Monte-Carlo search's bucket tables, its walk over the shuffles of
a step and its loads several steps ahead: per-shuffle totals equal to the
oracle's, at the sizes where each can go wrong."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1208_3407_amd import bits  # noqa: E402

DEV = torch.device("cuda", 0)


def up(x):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(x, dtype=np.uint32))).to(DEV)


def check(lengths, a_s, a_e, b_s, b_e, shuffles, batch):
    print("case: na=%d nb=%d shuffles=%d" % (len(a_s), len(b_s), shuffles), flush=True)
    exp = oracle.mc_totals(np.sort(b_s), np.sort(b_e), oracle.mc_prepare(lengths, a_s, a_e), 11, 0, shuffles,
                           threads=8)
    ref = bits.bits_sort_ref(up(b_s), up(b_e))
    mc = bits.bits_mc_binned(ref, up(a_s), up(a_e), lengths, 11, 0, shuffles, batch=batch)
    torch.cuda.synchronize()
    assert np.array_equal(mc.totals.cpu().numpy(), exp)


def intervals(rng, lo, hi, n, longest):
    s = rng.integers(lo, hi - 1, n)
    return s, np.minimum(s + rng.integers(0, longest, n), hi - 1)


@pytest.mark.parametrize("per", [1, 2, 3, 4, 5, 6, 7, 12, 60])
def test_keys_per_bucket(per):
    """`per` keys at one coordinate (so in one bucket), with bare coordinates between, and a genome of
    fewer coordinates than the tables have buckets next to a longer one."""
    rng = np.random.default_rng(per)
    lengths = [900, 40_000]
    at = np.concatenate([np.arange(0, 900, 7), 900 + np.arange(0, 40_000, 61)])
    b_s = np.repeat(at, per)
    b_e = np.minimum(b_s + rng.integers(0, 5, len(b_s)), np.where(b_s < 900, 899, 40_899))
    a = [intervals(rng, 0, 900, 300, 6), intervals(rng, 900, 40_900, 4000, 90)]
    check(lengths, np.concatenate([a[0][0], a[1][0]]), np.concatenate([a[0][1], a[1][1]]), b_s, b_e, 9, 4)


@pytest.mark.parametrize("longest", [10, 20_000, 300_000, 3_000_000])
@pytest.mark.parametrize("gap", [False, True])
def test_ends_past_a_region(longest, gap):
    """Ends inside, an eighth past, and far past a region, over even keys and keys in clusters."""
    rng = np.random.default_rng(longest + gap)
    lengths = [5_000_000]
    s, e = intervals(rng, 0, 5_000_000, 60_000, 500)
    if gap:   # dense runs with nothing in between
        s = s // 500_000 * 500_000 + s % 500_000 // 25
        e = np.minimum(s + rng.integers(0, 500, len(s)), 4_999_999)
    a_s, a_e = intervals(rng, 0, 5_000_000, 3000, longest)
    check(lengths, a_s, a_e, s, e, 5, 5)


@pytest.mark.parametrize("na", [1, 2, 63, 64, 65, 1024, 4095, 4096, 4097, 9 * 1024 + 1, 20_000])
def test_steps_and_shuffles(na):
    """Records per wave around whole steps and rounds of loads; few records a shuffle leave many shuffles,
    and empty ones, in one step.  20000 keys: several workgroups a region; 400000: one."""
    for n_b in (20_000, 400_000):
        rng = np.random.default_rng(na + n_b)
        lengths = [3_000_000, 50_000]
        b_s, b_e = intervals(rng, 0, 3_000_000, n_b, 300)
        a_s, a_e = intervals(rng, 0, 3_000_000, na, 2000)
        shuffles = 200 if na <= 65 else 3
        check(lengths, a_s, a_e, b_s, b_e, shuffles, 128)


def test_top_of_the_coordinate_range():
    rng = np.random.default_rng(5)
    size = 0xFFFFFFFF
    lengths = [size - 70_000, 70_000]
    b_s, b_e = intervals(rng, size - 90_000, size, 30_000, 3000)
    a_s, a_e = intervals(rng, size - 70_000, size, 5000, 4000)
    check(lengths, a_s, a_e, b_s, b_e, 6, 6)


@pytest.mark.parametrize("na", [1, 1023, 5632, 5633, 8191, 8192, 8193, 11_265, 20_000])
@pytest.mark.parametrize("n_b", [3_000, 1_300_000])
def test_groups_of_several_shuffles(na, n_b):
    """One chromosome holds nearly all entries and 23 few or none, so that workgroups take several
    shuffles of a group held in registers (at most 8192 entries) and of one placed chunk by chunk (many
    regions) or entry by entry (few)."""
    rng = np.random.default_rng(na + n_b)
    lengths = [9_000_000] + [40_000] * 22 + [0]
    b_s, b_e = intervals(rng, 0, 9_000_000 + 22 * 40_000, n_b, 40)
    a_s, a_e = intervals(rng, 0, 9_000_000, na, 3000)
    b = [intervals(rng, 9_000_000 + 40_000 * k, 9_040_000 + 40_000 * k, k % 3, 100) for k in range(22)]
    a_s = np.concatenate([a_s] + [x[0] for x in b])
    a_e = np.concatenate([a_e] + [x[1] for x in b])
    check(lengths, a_s, a_e, b_s, b_e, 131, 128)


@pytest.mark.parametrize("na", [9_216, 10_240, 10_241, 15_872, 20_480, 20_481, 31_000])
def test_chunks_of_large_groups(na):
    """A single chromosome of more than 128 regions: chunks of 10240 entries, each staged in two windows
    of 5632, around whole chunks and windows."""
    rng = np.random.default_rng(na)
    b_s, b_e = intervals(rng, 0, 9_000_000, 700_000, 40)
    a_s, a_e = intervals(rng, 0, 9_000_000, na, 3000)
    check([9_000_000], a_s, a_e, b_s, b_e, 5, 3)


@pytest.mark.parametrize("na", [5, 63 * 40, 64 * 40, 65 * 40, 200 * 40])
@pytest.mark.parametrize("n_b", [30_000, 300_000])
def test_few_records_a_shuffle(na, n_b):
    """Around 64 records per region and shuffle, where a wave's walk over the shuffles changes form."""
    rng = np.random.default_rng(na + n_b)
    b_s, b_e = intervals(rng, 0, 4_000_000, n_b, 300)
    a_s, a_e = intervals(rng, 0, 4_000_000, na, 3000)
    check([4_000_000], a_s, a_e, b_s, b_e, 40, 33)
