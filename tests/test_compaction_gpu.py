"""Compaction: one kernel for at most 16384 pairs, buckets of pairs above; tile groups with a few records and with
every record; ranges of one, two and more groups of 64 tiles; the two sets of totals taken in turn.
A pair's records are compared bit for bit with the raw outputs of its grid."""

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


def kept(raw, theta):
    """(parents, outputs) whose variance test passes, in the kernel's float32 operations."""
    w = raw.reshape(-1, 4)
    c, d = w[:, 0] - w[:, 1], w[:, 2] - w[:, 3]
    e = (w[:, 0] + w[:, 1]) - (w[:, 2] + w[:, 3])
    # the fused multiply-adds are exact products here: float64 holds them, rounded once per step
    s = np.float32(d.astype(np.float64) ** 2 + np.float32(c * c))
    s = np.float32(2.0 * s.astype(np.float64) + np.float32(e * e))
    p = np.nonzero(s > np.float32(16) * np.float32(theta))[0]
    return p, w[p]


def check(emr, genomes, subs, depth, theta, calls=3):
    pop = emr.emr_pack_population(genomes)
    raw = emr.emr_eval_raw(pop, subs, depth).cpu().numpy()
    pop = emr.emr_pack_population(genomes)
    want = [kept(r, theta) for r in raw]
    total = sum(len(p) for p, _ in want)
    res = emr.alloc_result(pop, subs, depth, capacity=max(1, total))
    for _ in range(calls):  # (the sets of totals in turn; interpreted, then compiled and listed)
        res["parent"].fill_(-1)
        emr.emr_discover(pop, subs, depth, theta, res=res)
        n, most = emr.emr_result_check(res)
        assert (n, most) == (total, max(len(p) for p, _ in want))
        _, got = emr.records_to_host(res)
        for (p, w), (gp, gw) in zip(want, got):
            np.testing.assert_array_equal(p, gp)
            np.testing.assert_array_equal(w.view(np.uint32), gw.view(np.uint32))


# depth 4: 2 tiles; 6: 22; 7: 86 (two groups); 8: 342 (marked groups)
@pytest.mark.parametrize("genomes,inputs,depth", [(1, 1, 4), (1, 2, 6), (2, 2, 7), (5, 3, 7),
                                                  (3, 2, 8), (33, 4, 6)])
@pytest.mark.parametrize("theta", [-1.0, 0.0, 0.03])
def test_records_are_the_grid_s(emr, genomes, inputs, depth, theta):
    check(emr, W.population(genomes + depth, genomes, 16, 50), W.tabular_sources(inputs + 1)[:inputs],
          depth, theta)


def test_one_kernel_and_two_agree(emr):
    """4096 genomes of 4 sources are the last call of one kernel; 4097 take buckets of pairs."""
    genomes = W.population(11, 4097, 8, 24)
    subs = W.xor_sources()
    out = []
    for n in (4096, 4097):
        pop = emr.emr_pack_population(genomes[:n])
        res = emr.alloc_result(pop, subs, 5, capacity=1 << 20)
        for _ in range(3):
            emr.emr_discover(pop, subs, 5, 0.02, res=res)
            emr.emr_result_check(res)
        off = res["pair_offset"].cpu().numpy()[:16385]
        k = int(off[-1])
        out.append((off, res["pair_count"].cpu().numpy()[:16384],
                    res["parent"][:k].cpu().numpy(), res["w4"][:k].cpu().numpy().view(np.uint32)))
    for x, y in zip(*out):
        np.testing.assert_array_equal(x, y)


def test_raw_outputs_into_an_unaligned_buffer(emr):
    genomes = W.population(3, 20, 16, 50)
    subs = W.xor_sources()
    pop = emr.emr_pack_population(genomes)
    want = emr.emr_eval_raw(pop, subs, 5)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    for shift in (1, 2, 3):
        buf = torch.full((want.numel() + 4,), 7.0, device="cuda")
        view = buf[shift:shift + want.numel()].view(want.shape)
        emr.emr_eval_raw_noalloc(pop, subs, 5, view, err)
        torch.cuda.synchronize()
        assert int(err.item()) == 0
        assert torch.equal(view.view(torch.int32), want.view(torch.int32))
        assert torch.all(buf[:shift] == 7.0) and torch.all(buf[shift + want.numel():] == 7.0)
