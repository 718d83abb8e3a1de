"""Which form a batch plan takes: a replay of the sorted form sorts the query
keys in the plan's workspace, one of the search per pair only reads it.  And
the sorted form's totals where the references' keys of one chunk of queries
are many: below and above the number that is placed key by key."""
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


def intervals(rng, n, lo=0, hi=2_000_000_000):
    s = rng.integers(lo, hi, n)
    return up(s), up(s + 500)


def sorts(plan):
    before = plan.workspace.clone()
    bits.bits_batch_run(plan)
    return not torch.equal(before, plan.workspace)


@pytest.mark.parametrize("n_q,n_ref,total,n,launch,expected", [
    (1, 64, 1 << 20, 20_000, None, True),
    (192, 65, 259_000, 20_000, None, True),
    (193, 65, 259_000, 20_000, None, False),            # more sets than accumulators
    (7, 64, 65_536, 20_000, None, False),               # the search is the faster form
    (7, 64, 65_535, 20_000, None, False),               # too few evaluations
    (7, 64, 1 << 20, 20_000, {"block": 1024}, False),   # a given shape
    (7, 64, 1 << 20, 20_000, {"path": 1}, False),       # a given path
])
def test_form(n_q, n_ref, total, n, launch, expected):
    rng = np.random.default_rng(n_q + n_ref)
    refs = bits.bits_sort_refs([intervals(rng, n) for _ in range(n_ref)])
    q = [intervals(rng, total // n_q + (i < total % n_q)) for i in range(n_q)]
    plan = bits.bits_batch_create(refs, q, launch=launch)
    assert sorts(plan) == expected
    bits.bits_batch_destroy(plan)


@pytest.mark.parametrize("n", [500, 520, 1_000, 1_030, 4_000, 4_200])
@pytest.mark.parametrize("n_ref", [24, 64, 66])
def test_dense_chunk(n, n_ref):
    """Every reference has n keys (half of the references twice that) between two queries of one chunk."""
    print("case: dense", n, n_ref, flush=True)
    rng = np.random.default_rng(n * n_ref)
    refs = bits.bits_sort_refs([intervals(rng, n << (j & 1), 1_000_000_000, 1_000_001_500) for j in range(n_ref)])
    q = [intervals(rng, 400_000) for _ in range(2)]
    q.append(intervals(rng, 500, 999_990_000, 1_000_010_000))
    plan = bits.bits_batch_create(refs, q)
    assert sorts(plan)
    other = bits.bits_batch_create(refs, q, launch={"path": bits.BITS_PATH_PLAIN})
    assert torch.equal(bits.bits_batch_run(plan).view(torch.int64), bits.bits_batch_run(other).view(torch.int64))
    for p in (plan, other):
        bits.bits_batch_destroy(p)
