"""Calls that sort accept a workspace sized for larger tiles than the sort would
like: 20480 keys (16384 with values along), one more histogram per segment and
rounds of a re-sorting batch end to end, the layout callers may have sized
theirs by.  Results are those of a workspace of the reported size."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_1208_3407_amd import bits  # noqa: E402

DEV = torch.device("cuda", 0)
SIZES = [1, 4097, 8193, 20_000, 100_003, 700_001, 1_400_000, 3_000_001]


def up(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32)).to(DEV)


def intervals(n):
    s = np.random.default_rng(n).integers(0, 2_900_000_000, n)
    return up(s), up(s + 300)


def a256(x):
    return (x + 255) // 256 * 256


def sort_bytes(ns, vals):
    tile = 16_384 if vals else 20_480
    tiles = sum((n + tile - 1) // tile for n in ns)
    k = len(ns)
    return (256 + a256(64 * k) + 2 * a256(4096 * k) + a256(2048 * tiles) + a256(4 * sum(ns))
            + (a256(4 * sum(ns)) if vals else 0))


def scratch(nbytes):
    return bits._scratch(nbytes, DEV)


@pytest.mark.parametrize("n", SIZES)
def test_index(n):
    b = intervals(n)
    ws = scratch(max(sort_bytes([n, n], False), bits.bits_sort_ref_workspace(0)))
    ref, exp = bits.bits_sort_ref(*b, workspace=ws), bits.bits_sort_ref(*b)
    assert torch.equal(ref.sorted_starts().view(torch.int32), exp.sorted_starts().view(torch.int32))
    assert torch.equal(ref.sorted_ends().view(torch.int32), exp.sorted_ends().view(torch.int32))
    assert bits.bits_get_status(ref) == 0


@pytest.mark.parametrize("n", SIZES)
def test_enumeration_index(n):
    b = intervals(n)
    exp = bits.bits_enum_index_build(*b)
    ws = scratch(sort_bytes([n], True))
    block = scratch(3 * a256(4 * n))
    rc = bits._lib.bits_enum_index_build(bits._ptr(b[0]), bits._ptr(b[1]), n, bits._ptr(block), block.numel(),
                                         bits._ptr(ws), ws.numel(), bits._stream())
    assert rc == 0
    q = intervals(1000)
    ref = bits.bits_sort_ref(*b)
    counts, first, offsets = bits.bits_enum_counts(ref, *q)
    pairs = bits.bits_enumerate(exp, *q, counts, offsets, first=first)
    ids = block[2 * a256(4 * n):][:4 * n].view(torch.int32)
    order = torch.sort(b[0].view(torch.int32).long() & 0xFFFFFFFF, stable=True).indices
    assert torch.equal(ids.long(), order)
    assert len(pairs[0]) == int(offsets.view(torch.int64)[-1])


@pytest.mark.parametrize("nb,batch", [(1, 1), (33, 3), (8193, 30), (20_001, 64), (100_003, 2), (700_001, 5)])
def test_resort(nb, batch):
    a, b = intervals(5000), intervals(nb)
    gen = [1_000_000_000, 1_000_000_000, 900_001_000]
    nbytes = 4 * a256(4 * nb) + 2 * 1024 + 256 + 4 * a256(4 * batch * nb) + a256(sort_bytes([nb] * (2 * batch), False))
    rounds = batch + 1
    got = bits.bits_mc_resort(*a, *b, gen, 7, 0, rounds, batch=batch, workspace=scratch(nbytes))
    exp = bits.bits_mc_resort(*a, *b, gen, 7, 0, rounds, batch=batch)
    assert torch.equal(got.totals.view(torch.int64), exp.totals.view(torch.int64))
    short = scratch(4 * a256(4 * nb) + 4 * a256(4 * batch * nb))
    with pytest.raises(bits.BitsError):
        bits.bits_mc_resort(*a, *b, gen, 7, 0, rounds, batch=batch, workspace=short)
