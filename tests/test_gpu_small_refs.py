"""References around the sizes where the open path changes: 2^14 keys (bisected below, windows above;
12288 on average in a batch plan) and 2^16 keys with models (both searches in step below)."""
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
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32)).to(DEV)


def sets(rng, n):
    s = np.sort(rng.integers(0, 50_000_000, n))
    s[n // 2:] //= 64   # half of them dense
    return s, s + rng.integers(0, 4000, n)


@pytest.mark.parametrize("n", [1, 2, 31, 33, 16_383, 16_384, 16_385, 65_535, 65_536, 65_537])
@pytest.mark.parametrize("learned", [False, True])
@pytest.mark.parametrize("launch", [None, {"qpl": 1}, {"qpl": 2}, {"qpl": 4}])
def test_small_references(n, learned, launch):
    print("case:", n, learned, launch, flush=True)
    rng = np.random.default_rng(n)
    b_s, b_e = sets(rng, n)
    a_s, a_e = sets(rng, 5000)
    a_s[0], a_e[0], a_s[1], a_e[1] = 0, 2**32 - 1, 2**32 - 1, 2**32 - 1
    ref = bits.bits_sort_ref(up(b_s), up(b_e), learned=learned, train={"epochs": 10})
    counts, total = bits.bits_count_per_query(ref, up(a_s), up(a_e), launch=launch)
    found, witness = bits.bits_decide(ref, up(a_s[2:]), up(a_e[2:]), launch=launch)[:2]
    torch.cuda.synchronize()
    exp, tot = oracle.counter(a_s, a_e, b_s, b_e)
    assert np.array_equal(counts.cpu().numpy(), exp) and int(total.cpu()[0]) == tot
    assert bool(int(torch.as_tensor(found).cpu().reshape(-1)[0])) == bool(exp[2:].any())


@pytest.mark.parametrize("mean", [5_000, 12_288, 12_290, 16_500])
def test_small_reference_batches(mean):
    rng = np.random.default_rng(mean)
    refs, queries = [], []
    for n in (mean // 2, mean, 2 * mean - mean // 2):
        refs.append(sets(rng, n))
    for n in (0, 1, 700, 3000):
        queries.append(sets(rng, n))
    built = [bits.bits_sort_ref(up(s), up(e)) for s, e in refs]
    sent = [(up(s), up(e)) for s, e in queries]
    plan = bits.bits_batch_create(built, sent)
    got = bits.bits_batch_run(plan)
    torch.cuda.synchronize()
    got = got.cpu().numpy().reshape(len(queries), len(refs))
    for i, (a_s, a_e) in enumerate(queries):
        for j, (b_s, b_e) in enumerate(refs):
            assert int(got[i, j]) == (oracle.counter(a_s, a_e, b_s, b_e)[1] if len(a_s) else 0), (i, j)
