"""The filters over CSR entries (spans of consecutive entries, whatever pairs they belong to) on
hand-built records and connections: runs of empty pairs at both ends and between, a pair that
spans many spans, pairs of one entry, capacities below the entries, a range of a table's pairs,
against numpy."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_27612_amd import workloads as W  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_27612_amd import emr as m
    return m


def dev(x, dtype):
    return torch.tensor(np.ascontiguousarray(x, dtype=dtype)).cuda()


COUNTS = {
    "none": [0, 0, 0],
    "one": [1],
    "ends empty": [0] * 50 + [3] + [0] * 700 + [5, 1, 0, 0, 64, 65] + [0] * 300,
    "single entries": [1] * 5000,
    "long pair": [2, 0, 300000, 0, 0, 7, 63],
    "mixed": None,
    # a step of 64 entries over 63, 64, 65 and 5000 pairs, and tables of 64, 65, 4096 and 4097 pairs
    "63 pairs a step": [32, 32] + [0] * 61 + [1] * 3,
    "64 pairs": [5] + [0] * 62 + [70],
    "65 pairs": [0] * 63 + [70, 5],
    "4096 pairs": [64] + [0] * 4094 + [64],
    "4097 pairs": [0] + [1] + [0] * 4094 + [130],
    "sparse": [1 if k % 173 == 5 else 0 for k in range(20000)],
    "dense then sparse": [7] * 200 + [1 if k % 90 == 0 else 0 for k in range(9000)] + [500],
}


def counts_of(name):
    if COUNTS[name] is not None:
        return np.array(COUNTS[name], np.int64)
    r = np.random.default_rng(1)
    return np.where(r.random(3000) < 0.4, 0, (r.pareto(0.7, 3000) * 3).astype(np.int64) % 40000)


@pytest.mark.parametrize("name", sorted(COUNTS))
@pytest.mark.parametrize("share", [0.0, 0.3, 1.0])
def test_band_filter(emr, name, share):
    n = counts_of(name)
    off = np.concatenate([[0], np.cumsum(n)])
    total = int(off[-1])
    r = np.random.default_rng(2)
    band = np.where(r.random(total) < share, 1.0, np.where(r.random(total) < 0.1, np.nan, 0.0))
    cell, w = r.integers(1, 1 << 20, total), r.standard_normal(total)
    conn = {"cell": dev(np.append(cell, 0), np.int32), "w": dev(np.append(w, 0), np.float32),
            "pair_count": dev(n, np.int64), "pair_offset": dev(off, np.int64),
            "capacity": max(total, 1), "n_pairs": len(n), "total": total}
    keep = np.nan_to_num(band, nan=-1.0) > 0.5
    want = np.array([int(keep[a:b].sum()) for a, b in zip(off[:-1], off[1:])])
    out = emr.emr_band_filter(conn, dev(np.append(band, 0), np.float32), 0.5)
    assert out["total"] == int(keep.sum())
    np.testing.assert_array_equal(out["pair_count"].cpu().numpy(), want)
    np.testing.assert_array_equal(out["pair_offset"].cpu().numpy(),
                                  np.concatenate([[0], np.cumsum(want)]))
    np.testing.assert_array_equal(out["cell"].cpu().numpy()[:out["total"]], cell[keep])
    np.testing.assert_array_equal(out["w"].cpu().numpy()[:out["total"]], w[keep].astype(np.float32))
    if total > 10 and share == 1.0:  # entries beyond the capacity given are not read
        conn["capacity"] = total // 2
        cut = emr.emr_band_filter(conn, dev(np.append(band, 0), np.float32), 0.5,
                                  capacity=max(total, 1))
        half = np.minimum(off, total // 2)
        kept = np.array([int(keep[a:b].sum()) for a, b in zip(half[:-1], half[1:])])
        np.testing.assert_array_equal(cut["pair_count"].cpu().numpy(), kept)
        np.testing.assert_array_equal(cut["pair_offset"].cpu().numpy(),
                                      np.concatenate([[0], np.cumsum(kept)]))


def test_band_filter_reports_a_short_output(emr):
    n = counts_of("mixed")
    off = np.concatenate([[0], np.cumsum(n)])
    total = int(off[-1])
    conn = {"cell": dev(np.zeros(total), np.int32), "w": dev(np.zeros(total), np.float32),
            "pair_count": dev(n, np.int64), "pair_offset": dev(off, np.int64), "capacity": total,
            "n_pairs": len(n), "total": total}
    with pytest.raises(emr.EmrError) as e:
        emr.emr_band_filter(conn, torch.ones(total, device="cuda"), 0.5, capacity=total - 1)
    assert e.value.status == emr.EMR_E_CAPACITY and str(total) in str(e.value)


@pytest.mark.parametrize("name", sorted(COUNTS))
def test_chain_filter(emr, name):
    depth = 10
    Q = sum(4 ** k for k in range(depth))
    n = counts_of(name)
    off = np.concatenate([[0], np.cumsum(n)])
    r = np.random.default_rng(3)
    parent = np.concatenate([np.sort(r.choice(min(Q, max(4 * c, 8)), size=c, replace=False))
                             if c else np.zeros(0, np.int64) for c in n]).astype(np.int64)
    w4 = r.standard_normal((len(parent), 4)).astype(np.float32)
    rec = {"parent": dev(np.append(parent, 0), np.int32), "w4": dev(np.vstack([w4, np.zeros((1, 4))]),
                                                                   np.float32),
           "pair_count": dev(n, np.int64), "pair_offset": dev(off, np.int64),
           "capacity": max(int(off[-1]), 1), "n_pairs": len(n),
           "workspace": torch.empty(256, dtype=torch.uint8, device="cuda")}
    keep = np.zeros(len(parent), bool)
    for a, b in zip(off[:-1], off[1:]):
        kept = set()
        for i in range(a, b):
            if parent[i] == 0 or (parent[i] - 1) // 4 in kept:
                kept.add(int(parent[i]))
                keep[i] = True
    want = np.array([int(keep[a:b].sum()) for a, b in zip(off[:-1], off[1:])])
    out = emr.emr_chain_filter(rec, depth)
    np.testing.assert_array_equal(out["pair_count"].cpu().numpy()[:len(n)], want)
    np.testing.assert_array_equal(out["pair_offset"].cpu().numpy(),
                                  np.concatenate([[0], np.cumsum(want)]))
    k = int(want.sum())
    np.testing.assert_array_equal(out["parent"].cpu().numpy()[:k], parent[keep])
    np.testing.assert_array_equal(out["w4"].cpu().numpy()[:k], w4[keep])


@pytest.mark.parametrize("name", ["ends empty", "long pair", "mixed", "single entries", "sparse",
                                  "dense then sparse", "4097 pairs"])
def test_ranges_of_pairs(emr, name):
    """The pairs from k on (the offsets' tail, over the same entries) give the whole table's results
    for those pairs: the band filter and the chain rule, with the entries cut off by the capacity too."""
    n = counts_of(name)
    off = np.concatenate([[0], np.cumsum(n)])
    total, P = int(off[-1]), len(n)
    r = np.random.default_rng(4)
    band = r.random(total).astype(np.float32)
    cell = r.integers(1, 1 << 20, total)
    parent = np.concatenate([np.arange(c) for c in n])  # a prefix of the heap: every ancestor kept
    keep = np.concatenate([[0], np.cumsum(band > 0.5)])
    for k, last in ((1, P), (P // 2, P), (P - 1, P), (2, P - 1)):
        for cap in (total, total - total // 3):
            lo, hi = min(off[k], cap), min(off[last], cap)
            edge = np.minimum(off[k:last + 1], cap)
            conn = {"cell": dev(cell, np.int32), "w": dev(band, np.float32),
                    "pair_count": dev(n, np.int64)[k:], "pair_offset": dev(off, np.int64)[k:],
                    "capacity": cap, "n_pairs": last - k, "total": total}
            out = emr.emr_band_filter(conn, dev(band, np.float32), 0.5)
            want = keep[edge] - keep[lo]
            np.testing.assert_array_equal(out["pair_offset"].cpu().numpy(), want)
            np.testing.assert_array_equal(out["pair_count"].cpu().numpy(), np.diff(want))
            m = int(want[-1])
            assert out["total"] == m
            np.testing.assert_array_equal(out["cell"].cpu().numpy()[:m],
                                          cell[lo:hi][band[lo:hi] > 0.5])
            rec = {"parent": dev(parent, np.int32), "w4": dev(np.zeros((total, 4)), np.float32),
                   "pair_count": conn["pair_count"], "pair_offset": conn["pair_offset"],
                   "capacity": cap, "n_pairs": last - k,
                   "workspace": torch.empty(256, dtype=torch.uint8, device="cuda")}
            out = emr.emr_chain_filter(rec, 10, capacity=total)
            np.testing.assert_array_equal(out["pair_offset"].cpu().numpy(), edge - lo)
            np.testing.assert_array_equal(out["pair_count"].cpu().numpy()[:last - k], np.diff(edge))
            np.testing.assert_array_equal(out["parent"].cpu().numpy()[:hi - lo], parent[lo:hi])


@pytest.mark.parametrize("mask", [0, 1, 6, 15])
def test_express(emr, mask):
    """Against the same filter in numpy on the call's own records; pairs from none to every cell."""
    genomes = W.population(8, 60, 20, 60)
    subs = W.tabular_sources(4)
    depth = 6
    pop = emr.emr_pack_population(genomes)
    rec = emr.emr_discover_all(pop, subs, depth, 0.02)
    counts, recs = emr.records_to_host(rec)
    assert counts.max() > 64 and (counts == 0).any()
    xy = emr.emr_build_grids(depth).cpu().numpy()
    out = emr.emr_express(pop, subs, depth, rec, mask, 0.1)
    off = out["pair_offset"].cpu().numpy()
    cell, w = out["cell"].cpu().numpy(), out["w"].cpu().numpy()
    for r, (p, w4) in enumerate(recs):
        s = subs[r % len(subs)]
        c = (4 * p[:, None] + np.arange(1, 5)).ravel()
        x, y = xy[c - 1, 0], xy[c - 1, 1]
        up = s["y"] < y if s["dir"] == 0 else y < s["y"]
        kind = np.where((x == s["x"]) & (y == s["y"]), 8,
                        np.where(up, 1, np.where(y == s["y"], 4, 2)))
        keep = ((kind & mask) != 0) & (np.abs(w4.ravel()) > np.float32(0.1))
        np.testing.assert_array_equal(cell[off[r]:off[r + 1]], c[keep])
        np.testing.assert_array_equal(w[off[r]:off[r + 1]], w4.ravel()[keep])
    assert off[-1] == out["total"]
