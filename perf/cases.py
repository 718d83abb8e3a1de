"""Timing cases of the library: what a program that uses it has it do.

Every case is one pass through the public entry points of
``paper_1208_3407_amd.bits`` on inputs that are already on the GPU.  The sizes
are those of the repository's own workloads (10,000 x 10,000 on one
chromosome, Table 1's 1e5 to 1e7 intervals, the 159-track screen's sets of
1e3 to 2e6, the 5e7 x 5e7 learned count with 1000 shuffles of 1e6), some of
them moved to odd numbers so that tiles and lines end raggedly.

Kinds of case (key "op"):
  count    one query set against one reference index: per-query counts and
           their total, or ("form": "total") the total alone; on a plain
           reference ("learned": False) or on one with the learned index
  index    chromosome-local intervals to a reference index: projection, sort,
           trees and heads, and with "learned" the trained models
  batch    one replay of the plan that counts every (query set, reference) pair
  mc       Monte-Carlo significance of one pair as the all-pairs screen runs
           it: shuffles binned by genome region, then the median of the totals
  ordered  the same shuffles by the query-ordered entry point
  resort   the paper's orientation: the database set re-placed, re-sorted and
           counted every round
  enum     every intersecting pair: index of B (when "build"), counts with
           offsets, pairs
"""
import math

import numpy as np
import torch

from paper_1208_3407_amd import bits

# 24 chromosomes, each 7% shorter than the one before it; or one of 10 Mbp.
GENOMES = {"g24": [249_200_000 * 93 ** k // 100 ** k for k in range(24)], "one": [10_000_000]}
N_CLUSTERS, CLUSTER_SIGMA = 20_000, 50_000.0
MC_SEED = 7
RECORD_BYTES_CAP = 4 << 30   # records of one binned pass, as the screen caps them


def listed():
    return [
        # two small annotation files of one chromosome: launches and host time decide
        {"name": "count_small", "op": "count", "na": 10_000, "nb": 10_000, "genome": "one", "learned": False,
         "form": "per_query"},
        # alignments of a whole genome against a large annotation, index without a model (the default)
        {"name": "count_genome", "op": "count", "na": 10_000_019, "nb": 9_999_991, "genome": "g24", "learned": False,
         "form": "per_query"},
        # the largest count of the repository's benchmark, through the learned index
        {"name": "count_learned", "op": "count", "na": 50_000_000, "nb": 50_000_000, "genome": "g24", "learned": True,
         "form": "per_query"},
        # one annotation track turned into an index
        {"name": "index_track", "op": "index", "nb": 100_003, "genome": "g24", "learned": False},
        # the benchmark's reference: index of 5e7 intervals with trained models
        {"name": "index_learned", "op": "index", "nb": 50_000_000, "genome": "g24", "learned": True, "epochs": 80,
         "points": 128},
        # observed counts of all pairs of a set of tracks (the screen's first step)
        {"name": "batch_tracks", "op": "batch", "nq": 32, "nr": 64, "lo": 1_000, "hi": 500_000},
        # significance of a small track against a small one
        {"name": "mc_small", "op": "mc", "na": 2_000, "nb": 20_000, "shuffles": 100},
        # significance of a track of 1e5 against one of 1e6
        {"name": "mc_track", "op": "mc", "na": 100_000, "nb": 1_000_000, "shuffles": 2_000},
        # the benchmark's Monte-Carlo run
        {"name": "mc_genome", "op": "mc", "na": 1_000_000, "nb": 50_000_000, "shuffles": 1_000},
        # few shuffles of a mid-sized set, query by query through the learned index
        {"name": "ordered_learned", "op": "ordered", "na": 100_003, "nb": 1_000_000, "shuffles": 100,
         "learned": True},
        # Table 1's loop at its smallest size
        {"name": "resort_table", "op": "resort", "na": 100_000, "nb": 100_000, "rounds": 64},
        # the pairs themselves, from the raw sets on
        {"name": "enum_pairs", "op": "enum", "na": 1_000_003, "nb": 5_000_011, "build": True},
    ]


def _size(rng, lo, hi):
    """Log-uniform whole number in [lo, hi]; odd more often than not."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n | 1 if rng.random() < 0.5 else n))


def draw(rng):
    op = rng.choice(["count", "count", "index", "batch", "mc", "mc", "ordered", "resort", "enum"])
    if op == "count":
        one = rng.random() < 0.2
        return {"op": op, "na": _size(rng, 1_000, 200_000 if one else 20_000_000),
                "nb": _size(rng, 1_000, 200_000 if one else 20_000_000), "genome": "one" if one else "g24",
                "learned": rng.random() < 0.35, "form": rng.choice(["per_query", "per_query", "total"])}
    if op == "index":
        case = {"op": op, "nb": _size(rng, 1_000, 20_000_000), "genome": "g24", "learned": rng.random() < 0.4}
        if case["learned"]:
            case["epochs"], case["points"] = rng.choice([(80, 128), (300, 256)])
        return case
    if op == "batch":
        return {"op": op, "nq": rng.randint(2, 32), "nr": rng.randint(2, 48), "lo": 1_000,
                "hi": _size(rng, 5_000, 400_000)}
    if op in ("mc", "ordered"):
        na, nb = _size(rng, 1_000, 500_000), _size(rng, 10_000, 10_000_000)
        most = (400_000_000 if op == "mc" else 30_000_000) // na
        case = {"op": op, "na": na, "nb": nb, "shuffles": _size(rng, 10, max(11, min(5_000, most)))}
        if op == "ordered":
            case["learned"] = rng.random() < 0.5
        return case
    if op == "resort":
        nb = _size(rng, 1_000, 1_000_000)
        return {"op": op, "na": _size(rng, 1_000, 1_000_000), "nb": nb,
                "rounds": rng.randint(2, max(3, min(128, 12_000_000 // nb)))}
    return {"op": op, "na": _size(rng, 1_000, 3_000_000), "nb": _size(rng, 1_000, 5_000_000),
            "build": rng.random() < 0.5}


# ------------------------------------------------------------------ inputs

def _rng(seed, role):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 1_000_003 + role) & 0x7FFFFFFFFFFFFFFF)


def _u32(x):
    return x.to(torch.int32).view(torch.uint32)   # int64 -> int32 keeps the low 32 bits


def _chroms(lens, n, gen):
    ends = torch.cumsum(lens, 0)
    return torch.searchsorted(ends, (torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
                                     * float(ends[-1])).long(), right=True).clamp_(max=len(lens) - 1)


def _intervals(n, genome, seed, role, mixture, median=200.0):
    """(chromosome, local start, local end), int64: starts uniform over the genome, or for a mixture the
    second half around Gaussian cluster centres that all roles of a seed share; log-normal lengths."""
    lens = torch.tensor(GENOMES[genome], dtype=torch.int64, device="cuda")
    gen = _rng(seed, role)
    z = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
    L = (torch.exp(z) * median).round_().clamp_(20, 100_000).long()
    c = _chroms(lens, n, gen)
    pos = (torch.rand(n, generator=gen, device="cuda", dtype=torch.float64) * lens[c]).long()
    if mixture:
        cg = _rng(seed, 0)
        cc = _chroms(lens, N_CLUSTERS, cg)
        mu = (torch.rand(N_CLUSTERS, generator=cg, device="cuda", dtype=torch.float64) * lens[cc]).long()
        k = n - n // 2
        j = torch.randint(0, N_CLUSTERS, (k,), generator=gen, device="cuda")
        c[n // 2:] = cc[j]
        pos[n // 2:] = mu[j] + (torch.randn(k, generator=gen, device="cuda", dtype=torch.float64)
                                * CLUSTER_SIGMA).long()
    s = torch.minimum(pos, lens[c] - L).clamp_(min=0)
    return c, s, s + L - 1


def _global(local, genome):
    c, s, e = local
    off = torch.tensor(np.concatenate([[0], np.cumsum(GENOMES[genome])[:-1]]), dtype=torch.int64, device="cuda")[c]
    return off + s, off + e


def _queries(case, seed, n=None, role=1):
    return _global(_intervals(n or case["na"], case.get("genome", "g24"), seed, role, False), case.get("genome", "g24"))


def _database(case, seed, n=None, role=2):
    return _global(_intervals(n or case["nb"], case.get("genome", "g24"), seed, role, True), case.get("genome", "g24"))


def _pairs(case):
    """Pairs of an enum case: 85% of what its sizes lead one to expect, less eight standard deviations."""
    mean = case["na"] * case["nb"] * 660 / sum(GENOMES["g24"])   # two mean lengths of 330 bp
    return max(0, int(0.85 * mean - 8 * math.sqrt(mean)))


def _enum_sets(case, seed):
    """Query set and database of an enum case.  Queries after the one that reaches the case's number of pairs
    are replaced by ones of the set that hit nothing (or, to make it exact, one interval), so that every seed's
    output has the same size."""
    a, b = _queries(case, seed), _database(case, seed)
    c = _counts(a, b)
    most = _pairs(case)
    before = torch.cumsum(c, 0)
    k = int((before <= most).sum())
    rest = most - (int(before[k - 1]) if k else 0)
    take = torch.arange(case["na"], device="cuda")
    take[k:] = torch.nonzero(c == 0)[0]
    take[k:k + rest] = torch.nonzero(c == 1)[:rest, 0]
    return (a[0][take], a[1][take]), b


def _dev(pair):
    return _u32(pair[0]), _u32(pair[1])


def _sets(case, seed):
    """Sizes of a batch's query sets and references: log-uniform, from the seed."""
    r = np.random.default_rng(int(seed))
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    return ([int(x) for x in np.rint(np.exp(r.uniform(lo, hi, case["nq"])))],
            [int(x) for x in np.rint(np.exp(r.uniform(lo, hi, case["nr"])))])


def _pass_batch(na, shuffles):
    return int(max(1, min(1000, shuffles, RECORD_BYTES_CAP // (8 * na))))


def _scratch(nbytes):
    raw = torch.empty(max(nbytes, 1) + 256, dtype=torch.uint8, device="cuda")
    off = -raw.data_ptr() % 256
    return raw[off:off + max(nbytes, 1)]


def prepare(case, seed):
    op, genome = case["op"], GENOMES[case.get("genome", "g24")]
    st = {"case": case, "genome": genome}
    if op == "index":
        st["b"] = [_u32(x) for x in _intervals(case["nb"], case["genome"], seed, 2, True)]
        st["train"] = {"epochs": case["epochs"], "max_points": case["points"]} if case["learned"] else None
        return st
    if op == "batch":
        nq, nr = _sets(case, seed)
        st["q"] = [_dev(_queries(case, seed, n, 10 + k)) for k, n in enumerate(nq)]
        st["refs"] = bits.bits_sort_refs([_dev(_database(case, seed, n, 100 + k)) for k, n in enumerate(nr)])
        st["plan"] = bits.bits_batch_create(st["refs"], st["q"])
        return st
    a, b = _enum_sets(case, seed) if op == "enum" else (_queries(case, seed), _database(case, seed))
    st["a"], b = _dev(a), _dev(b)
    if op == "resort":
        st["b"], st["batch"] = b, min(64, case["rounds"])
        st["ws"] = _scratch(bits.bits_mc_resort_workspace(case["nb"], st["batch"]))
        return st
    st["ref"] = bits.bits_sort_ref(*b, learned=bool(case.get("learned")),
                                   train={"epochs": 80, "max_points": 128} if case.get("learned") else None)
    if op == "mc":
        st["batch"] = _pass_batch(case["na"], case["shuffles"])
        st["ws"] = _scratch(bits.bits_mc_binned_workspace(case["na"], case["nb"], genome, st["batch"]))
    elif op == "ordered":
        st["ws"] = _scratch(bits.bits_mc_workspace(case["na"]))
    elif op == "enum":
        st["b"] = b
        st["index"] = None if case["build"] else bits.bits_enum_index_build(*b)
    return st


# ------------------------------------------------------------------ passes

def _i32(t):
    return t.view(torch.int32)


def _i64(t):
    return t.view(torch.int64)


def _models(ref):
    """The trained leaves of B_S and B_E as views: hidden weights, output weights with hidden biases, output bias."""
    rec = ref.rmi_bytes().view(2, -1, 128)[:, 1:]      # a 128-byte header, then 128-byte leaf records
    half = rec.view(torch.float16)
    return {"w1": half[..., :32].unflatten(-1, (4, 8))[..., 4:], "b1_w2": half[..., 32:],
            "b2": rec.view(torch.float32)[..., 9]}


def _mc(out):
    return {"totals": _i64(out.totals), "observed": _i64(out.observed), "n_ge": _i64(out.n_ge),
            "n_le": _i64(out.n_le)}


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "count":
        if case["form"] == "total":
            return {"total": _i64(bits.bits_count(st["ref"], *st["a"]))}
        counts, total = bits.bits_count_per_query(st["ref"], *st["a"])
        return {"counts": _i32(counts), "total": _i64(total)}
    if op == "index":
        ref = bits.bits_sort_ref(*bits.bits_project(st["genome"], *st["b"]), learned=case["learned"],
                                 train=st["train"])
        out = {"starts": _i32(ref.sorted_starts()), "ends": _i32(ref.sorted_ends())}
        return dict(out, **_models(ref)) if case["learned"] else out
    if op == "batch":
        return {"totals": _i64(bits.bits_batch_run(st["plan"]))}
    if op == "mc":
        out = bits.bits_mc_binned(st["ref"], *st["a"], st["genome"], MC_SEED, 0, case["shuffles"], batch=st["batch"],
                                  workspace=st["ws"])
        lo, hi = bits.bits_mc_median(out.totals)
        return dict(_mc(out), lo=_i64(lo), hi=_i64(hi))
    if op == "ordered":
        return _mc(bits.bits_mc_pvalue(st["ref"], *st["a"], st["genome"], MC_SEED, 0, case["shuffles"],
                                       workspace=st["ws"]))
    if op == "resort":
        return _mc(bits.bits_mc_resort(*st["a"], *st["b"], st["genome"], MC_SEED, 0, case["rounds"],
                                       batch=st["batch"], workspace=st["ws"]))
    index = bits.bits_enum_index_build(*st["b"]) if case["build"] else st["index"]
    counts, first, offsets = bits.bits_enum_counts(st["ref"], *st["a"])
    pa, pb = bits.bits_enumerate(index, *st["a"], counts, offsets, first=first)
    return {"counts": _i32(counts), "offsets": _i64(offsets), "pair_a": _i32(pa), "pair_b": _i32(pb)}


# ------------------------------------------------------------------ work

def _touched(na, nb):
    """Bytes of B_S and B_E that na queries cannot do without: all of both, or one 64-byte piece of each a query."""
    return min(8 * nb, 128 * na)


def work(case):
    """Bytes of inputs read once and outputs written once; whole-number operations where they are the larger
    part: ten Philox rounds of six operations and two rank searches a placement, two searches a query."""
    op = case["op"]

    def searches(n, nb):
        return 2 * n * math.log2(nb + 1)

    if op == "count":
        out = 4 * case["na"] if case["form"] == "per_query" else 8
        return {"bytes": 8 * case["na"] + out + _touched(case["na"], case["nb"]),
                "flops": searches(case["na"], case["nb"])}
    if op == "index":
        steps = case.get("epochs", 0) * case.get("points", 0)
        return {"bytes": 12 * case["nb"] + 8 * case["nb"] + (2 * 4096 * 128 if case["learned"] else 0),
                "flops": searches(case["nb"], case["nb"]) + 2 * min(4096 * steps, case.get("epochs", 0) * case["nb"]) * 300}
    if op == "batch":
        mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])   # mean log-uniform size
        return {"bytes": 8 * mean * (case["nq"] + case["nr"]) + 8 * case["nq"] * case["nr"],
                "flops": searches(mean * case["nq"] * case["nr"], mean)}
    if op in ("mc", "ordered"):
        n = case["na"] * case["shuffles"]
        return {"bytes": 8 * case["na"] + _touched(n, case["nb"]) + 8 * case["shuffles"],
                "flops": 60 * n + searches(n, case["nb"])}
    if op == "resort":
        n = case["nb"] * case["rounds"]
        return {"bytes": 8 * (case["na"] + case["nb"]) + 8 * case["rounds"],
                "flops": 60 * n + searches(n, case["nb"]) + searches(case["na"] * case["rounds"], case["nb"])}
    return {"bytes": 8 * case["na"] + 12 * case["na"] + 8 * _pairs(case) + (20 if case["build"] else 12) * case["nb"],
            "flops": searches(case["na"], case["nb"]) + (searches(case["nb"], case["nb"]) if case["build"] else 0)}


# ------------------------------------------------------------------ exact values

def _counts(a, b):
    """#{b.start <= a.end} - #{b.end < a.start} per query, int64."""
    bs, be = torch.sort(b[0]).values, torch.sort(b[1]).values
    return torch.searchsorted(bs, a[1], right=True) - torch.searchsorted(be, a[0])


def _philox(g):
    """The two low words of Philox-4x32-10 (Salmon et al., SC'11), counter (lo g, hi g, 0, 0), key (MC_SEED, 0);
    int64 tensors that hold 32-bit words."""
    m = 0xFFFFFFFF
    c0, c1 = g & m, (g >> 32) & m
    c2, c3 = torch.zeros_like(g), torch.zeros_like(g)
    k0, k1 = MC_SEED, 0
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # products mod 2^64
        c0, c1, c2, c3 = ((p1 >> 32) & m) ^ c1 ^ k0, p1 & m, ((p0 >> 32) & m) ^ c3 ^ k1, p0 & m
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c0, c1


def _shuffled(sets, genome, s):
    """The set with every interval at its place in shuffle s: uniform over the legal starts of its chromosome."""
    off = torch.tensor(np.concatenate([[0], np.cumsum(genome)]), dtype=torch.int64, device="cuda")
    a0, a1 = sets
    c = torch.searchsorted(off, a0, right=True) - 1
    L = a1 - a0 + 1
    span = off[c + 1] - off[c] - L + 1
    lo, hi = _philox(s * len(a0) + torch.arange(len(a0), device="cuda"))
    t = lo * span                                       # below 2^60: span < 2^28
    st = off[c] + ((hi * span + (t >> 32)) >> 32)
    return st, st + L - 1


def _tails(totals, observed):
    totals = torch.stack(totals)
    return {"totals": totals, "observed": observed.view(1), "n_ge": (totals >= observed).sum().view(1),
            "n_le": (totals <= observed).sum().view(1)}


def exact(case, seed):
    op = case["op"]
    if op == "count":
        c = _counts(_queries(case, seed), _database(case, seed))
        return {"total": c.sum().view(1)} if case["form"] == "total" else {"counts": c.int(), "total": c.sum().view(1)}
    if op == "index":
        s, e = _global(_intervals(case["nb"], case["genome"], seed, 2, True), case["genome"])
        out = {"starts": _i32(_u32(torch.sort(s).values)), "ends": _i32(_u32(torch.sort(e).values))}
        # the trained weights are what the optimiser leaves after its steps: no value in 64 bits stands for them
        return dict(out, w1=None, b1_w2=None, b2=None) if case["learned"] else out
    if op == "batch":
        nq, nr = _sets(case, seed)
        refs = [_database(case, seed, n, 100 + k) for k, n in enumerate(nr)]
        refs = [(torch.sort(s).values, torch.sort(e).values) for s, e in refs]
        got = []
        for k, n in enumerate(nq):
            a = _queries(case, seed, n, 10 + k)
            got += [(torch.searchsorted(s, a[1], right=True) - torch.searchsorted(e, a[0])).sum() for s, e in refs]
        return {"totals": torch.stack(got)}
    a, b = _enum_sets(case, seed) if op == "enum" else (_queries(case, seed), _database(case, seed))
    if op == "enum":
        c = _counts(a, b)
        offsets = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(c, 0)])
        return {"counts": c.int(), "offsets": offsets, "pair_a": torch.repeat_interleave(c).int(), "pair_b": None}
    n, moved = (case["rounds"], b) if op == "resort" else (case["shuffles"], a)
    if n * len(moved[0]) > 300_000_000 or n > 3_000:
        return None                                     # over 20 s
    genome = GENOMES["g24"]
    bs, be = torch.sort(b[0]).values, torch.sort(b[1]).values
    totals = []
    for s in range(n):
        m = _shuffled(moved, genome, s)
        if op == "resort":
            totals.append(_counts(a, m).sum())
        else:
            totals.append((torch.searchsorted(bs, m[1], right=True) - torch.searchsorted(be, m[0])).sum())
    out = _tails(totals, _counts(a, b).sum())
    if op == "mc":
        v = torch.sort(out["totals"]).values
        out["lo"], out["hi"] = v[(n - 1) // 2].view(1), v[n // 2].view(1)
    return out
