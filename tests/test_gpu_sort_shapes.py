"""The radix sort at the sizes where its shape changes: segments one workgroup
sorts (up to 4096 and 8192 keys) and one key more, tiles of 4096, 7168, 12288
and 16384 keys and their neighbours, numbers of tiles at which the next shape
is taken; segments of one call whose digits vary in different passes, and
segments with all keys equal.  Sorted arrays, stable order, trees, line heads
and the words after the keys against numpy."""
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


def keys(rng, n, kind):
    """Keys whose digits vary in the passes `kind` (a bit mask) alone; 0: all equal."""
    x = np.full(n, 0x01020304, np.int64)
    for p in range(4):
        if kind >> p & 1:
            x = (x & ~(255 << 8 * p)) | (rng.integers(0, 256, n) << 8 * p)
    return x.astype(np.uint32)


def check_ref(ref, s, e):
    n, d = len(s), ref.depth
    for got, k, t in ((ref.sorted_starts(), s, 0), (ref.sorted_ends(), e, 1)):
        exp = np.sort(k)
        assert np.array_equal(got.cpu().numpy(), exp)
        tree = ref.tree().cpu().numpy().reshape(2, -1)[t]
        node = np.arange(1, 1 << d)
        level = np.floor(np.log2(node)).astype(np.int64)
        pos = (2 * (node - (1 << level)) + 1) * n >> (level + 1)
        assert np.array_equal(tree[1:], exp[pos - 1])
        hl = ref.heads_len()
        base = ref.c.heads + t * hl * 4
        heads = ref._view(base, hl, torch.uint32).cpu().numpy()
        assert np.array_equal(heads[:(n + 31) // 32], exp[::32]) and (heads[(n + 31) // 32:] == 2**32 - 1).all()
        line = (n + 31) // 32 * 32
        addr = ref.c.bs if t == 0 else ref.c.be
        assert (ref._view(addr, line, torch.uint32).cpu().numpy()[n:] == 2**32 - 1).all()


@pytest.mark.parametrize("n", [1, 31, 4095, 4096, 4097, 8191, 8192, 8193, 12289, 28673, 109 * 6144, 110 * 6144 + 1,
                               1_400_000])
def test_index(n):
    print("case: index", n, flush=True)
    rng = np.random.default_rng(n)
    s, e = keys(rng, n, 15), keys(rng, n, 9)
    check_ref(bits.bits_sort_ref(up(s), up(e)), s, e)


@pytest.mark.parametrize("sizes", [(3, 4096, 1), (0, 8192, 5000), (40_000, 0, 7, 9000), (700_000, 3, 300_001)])
def test_segments_with_their_own_digits(sizes):
    print("case: segments", sizes, flush=True)
    rng = np.random.default_rng(len(sizes))
    sets = [(keys(rng, n, 3 * i % 16), keys(rng, n, 5 * i % 16)) for i, n in enumerate(sizes)]
    refs = bits.bits_sort_refs([(up(s), up(e)) for s, e in sets])
    for r, (s, e) in zip(refs, sets):
        if len(s):
            check_ref(r, s, e)
        assert not r.status_words().cpu().numpy().any()


@pytest.mark.parametrize("n,kind", [(n, k) for n in (1, 4097, 8193, 7168 * 3, 200 * 7168 + 1)
                                    for k in (0, 1, 4, 10, 15)] + [(16384 * 730 - 5, 0), (16384 * 730 - 5, 15)])
def test_stable_values(n, kind):
    print("case: values", n, kind, flush=True)
    rng = np.random.default_rng(n + kind)
    s = keys(rng, n, kind)
    e = rng.integers(0, 2**32, n).astype(np.uint32)
    idx = bits.bits_enum_index_build(up(s), up(e))
    order = np.argsort(s, kind="stable")
    assert np.array_equal(idx.ids().cpu().numpy(), order.astype(np.uint32))
    assert np.array_equal(idx.starts().cpu().numpy(), s[order])
    assert np.array_equal(idx.ends().cpu().numpy(), e[order])


def test_fewer_rounds_fit_the_same_workspace():
    """A workspace for `batch` rounds holds every shorter last batch, whatever shape its sort takes."""
    rng = np.random.default_rng(5)
    n = 70_000
    s = np.sort(rng.integers(0, 9_000_000, n))
    a = up(s[:500]), up(s[:500] + 20)
    b = up(s), up(s + 50)
    ws = bits._scratch(bits.bits_mc_resort_workspace(n, 30), DEV)
    full = bits.bits_mc_resort(*a, *b, [10_000_000], 7, 0, 43, batch=30, workspace=ws)
    one = bits.bits_mc_resort(*a, *b, [10_000_000], 7, 0, 43, batch=1)
    assert torch.equal(full.totals.view(torch.int64), one.totals.view(torch.int64))
