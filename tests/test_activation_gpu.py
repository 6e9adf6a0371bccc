"""Activation's kernels against a float64 sum over the same edges: workgroups of 1, 2 and 4 pattern
groups, ragged pattern counts, hand-built genomes on both sides of every node-count class, and the
stepwise kernels (where a workgroup would take longer than the steps' launches, more nodes than the
LDS holds, more steps than one fused run)."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_27612_amd import workloads as W  # noqa: E402
from tests.test_oracle_pins import INPUTS, LIN, mk  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emr():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2608_27612_amd import emr as m
    return m


# The most nodes of a genome whose states (two buffers of 16 Q bytes a node, 4 bytes of edge offset)
# fit 80 KB of LDS for Q = 4, 2, 1 pattern groups, and 160 KB for Q = 1; above, it runs stepwise.
CLASS_NODES = [((kb << 10) - 4) // (32 * q + 4) for kb, q in ((80, 4), (80, 2), (80, 1), (160, 1))]


@pytest.fixture(scope="module")
def classes(emr):
    """Networks of one input, one output and k hidden nodes between them, for k around every class
    bound: the weights are s (x + e y) at a cell (x, y) for both ends, and those of magnitude over
    0.004 are expressed, so a genome's s sets its k. Weights stay small, and cells come in pairs of
    opposite weights, so no sigmoid saturates and a wrong state shows in the output."""
    depth, w_min, e = 6, 0.004, 0.0041
    xy = emr.emr_build_grids(depth).cpu().numpy().astype(np.float64)
    v = np.sort(np.abs(xy[:, 0] + e * xy[:, 1]))[::-1]
    want = [2, 40, 300] + [2 * ((b + d) // 2) - 2 for b in CLASS_NODES for d in (0, 2)] + [3000, 5000]
    genomes = []
    for k in want:
        assert v[k - 1] > v[k] * (1 + 1e-4)  # (the outputs' error is a few 1e-7 of them)
        s = w_min / np.sqrt(v[k - 1] * v[k])
        genomes.append(mk(INPUTS + [6], [0] * 5 + [LIN],
                          [(0, 5, s), (1, 5, s * e), (2, 5, s), (3, 5, s * e)]))
    subs = W.sources_array([(0.0, 0.0, 0), (0.0, 0.0, 1)])
    pop = emr.emr_pack_population(genomes)
    net = emr.emr_build_networks(pop, subs, depth, -1.0, 15, w_min, 0)
    nets = net.to_host()
    assert [len(n["cells"]) for n in nets] == want
    nodes = np.array(want) + 2
    for b in CLASS_NODES:
        assert (nodes == b - b % 2).any() and (nodes == b - b % 2 + 2).any()
    return net, nets


@pytest.mark.parametrize("patterns", [1, 4, 5, 8, 13, 16, 17, 33, 1200])
def test_every_node_count_class(classes, patterns):
    """Against float64; and bit for bit against calls of one pattern, which run stepwise (three steps'
    launches are shorter than one workgroup's run of thousands of nodes), where the call of 1200 patterns
    runs every genome fused that the LDS can hold."""
    net, nets = classes
    x = np.random.default_rng(patterns).uniform(-1, 1, (patterns, 1)).astype(np.float32)
    got = net.activate(x, 3)[:, :, 0]
    some = sorted({0, patterns // 2, patterns - 1})
    want = reference(nets, x[some].astype(np.float64), 3)
    assert np.ptp(want[-1]) > 0.01 or patterns == 1
    assert np.abs(got[:, some] - want).max() <= 4 * sum_bound(nets) + 1e-6
    for k in some:
        one = net.activate(x[k:k + 1], 3)[:, 0, 0]
        np.testing.assert_array_equal(one.view(np.uint32), got[:, k].copy().view(np.uint32))


@pytest.fixture(scope="module")
def built(emr):
    """Networks of 6 to 773 nodes (depth 6, every connection type), hidden nodes among themselves, the
    largest with 211,000 edges; and their edges."""
    genomes = W.population(3, 60, 20, 60)
    subs = W.tabular_sources(5)
    pop = emr.emr_pack_population(genomes)
    net = emr.emr_build_networks(pop, subs, 6, 0.02, 15, 0.1, 1)
    return net, net.to_host()


def reference(nets, x, steps):
    """[genomes, patterns] float64: the first sources are x's inputs, the next one the output."""
    out = np.zeros((len(nets), len(x)))
    m = x.shape[1]
    for g, net in enumerate(nets):
        n = m + 1 + len(net["cells"])
        s = np.zeros((n, len(x)))
        s[:m] = x.T
        order = np.argsort(net["dst"], kind="stable")
        src, dst, w = net["src"][order], net["dst"][order], net["w"][order].astype(np.float64)
        first = np.searchsorted(dst, np.arange(n + 1))
        for _ in range(steps):
            z = np.zeros_like(s)
            for v in np.unique(dst):
                a, b = first[v], first[v + 1]
                z[v] = w[a:b] @ s[src[a:b]]
            s = 1.0 / (1.0 + np.exp(-z))
            s[:m] = x.T
        out[g] = s[m]
    return out


def sum_bound(nets):
    """Error of one node's sum in units of 2^-24: |w| summed over its edges, times the depth of the
    summation (its chain of edges / 64 terms, a butterfly of 6), through a sigmoid of slope 1/4."""
    worst = 0.0
    for net in nets:
        if len(net["w"]):
            a = np.bincount(net["dst"], weights=np.abs(net["w"]))
            d = np.bincount(net["dst"])
            worst = max(worst, float((a * (d / 64 + 8)).max()))
    return worst * 2.0 ** -24


@pytest.mark.parametrize("patterns", [1, 4, 5, 8, 13, 16, 31, 33, 70])
def test_batches_match_float64_and_each_other(built, patterns):
    net, nets = built
    x = np.random.default_rng(patterns).uniform(-1, 1, (patterns, 5)).astype(np.float32)
    got = net.activate(x, 3)[:, :, 0]
    sizes = [6 + len(n["cells"]) for n in nets]
    assert min(sizes) < 10 and max(sizes) > CLASS_NODES[0]
    want = reference(nets, x.astype(np.float64), 3)
    # a saturated sigmoid hides its sum's error, so the bound is loose where sums are large
    assert np.abs(got - want).max() <= min(1e-3, 4 * sum_bound(nets) + 1e-6)
    # a pattern's outputs have the same bits in every batch
    for k in (0, patterns - 1):
        one = net.activate(x[k:k + 1], 3)[:, 0, 0]
        np.testing.assert_array_equal(one.view(np.uint32), got[:, k].copy().view(np.uint32))


def test_stepwise_and_fused_agree(built):
    """The heaviest genome runs stepwise in a call of 4 patterns and fused in one of 16384; a call
    of 1025 steps runs every genome stepwise, one of 1024 none of the small ones."""
    net, nets = built
    assert max(len(n["src"]) for n in nets) > 16384  # (twice the least that runs stepwise)
    x = np.random.default_rng(9).uniform(-1, 1, (16384, 5)).astype(np.float32)
    many = net.activate(x, 2)[:, :4, 0].copy()
    few = net.activate(x[:4], 2)[:, :, 0].copy()
    np.testing.assert_array_equal(many.view(np.uint32), few.view(np.uint32))
    a = net.activate(x[:3], 1024)[:, :, 0]
    b = net.activate(x[:3], 1025)[:, :, 0]
    # (two neighbouring steps of a settled or alternating network: compared with float64 instead)
    light = [g for g in range(len(nets)) if len(nets[g]["src"]) < 200]
    want = [reference([nets[g] for g in light], x[:3].astype(np.float64), s) for s in (1024, 1025)]
    settled = np.abs(want[0] - want[1]) < 1e-9
    assert settled.mean() > 0.5
    assert np.abs(a[light] - want[0])[settled].max() < 1e-5
    assert np.abs(b[light] - want[1])[settled].max() < 1e-5
