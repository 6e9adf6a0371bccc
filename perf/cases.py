"""The work that users of this library have it do, as cases that can be timed and compared.

Every case goes through the public entry points of paper_2608_27612_amd.emr as a program calls
them. The kinds:

  discover    emr_discover + emr_result_check on a population held on the device: a substrate
              queried again and again (a service, a benchmark, a parameter sweep)
  fresh       a new population packed from the concatenated genome arrays, discovered once and
              checked: discovery's share of an evolution loop's generation
  generation  a new population packed, its networks built (substrate discovery, a hidden-to-hidden
              phase, expression, assembly, pruning) and its XOR fitness computed: the whole
              generation of an evolution loop without NEAT's reproduction
  recurrent   a new population packed and discovered, its hidden nodes found and queried as
              sources of their own (per-genome sources, a deep grid)
  raw         every CPPN output of a population's grid, unfiltered (emr_eval_raw)
  prune       the filters on a checked result: expression by type and weight, band values, band
              filter, and the literal chain rule
  activate    networks that are kept, activated on a data set's patterns
  stream      one deep CPPN past the size of one call, delivered to a host sink chunk by chunk

Populations are seeded random CPPNs of the size classes of paper_2608_27612_amd.workloads. Buffers
whose used length depends on the inputs are zeroed once and padded to a fixed length.
"""

import math

import numpy as np
import torch

from paper_2608_27612_amd import emr
from paper_2608_27612_amd import workloads as W

KINDS = ("discover", "fresh", "generation", "recurrent", "raw", "prune", "activate", "stream")


def _case(name, kind, genomes, h, e, inputs, depth, theta, **more):
    c = {"name": name, "kind": kind, "genomes": genomes, "h": h, "e": e, "inputs": inputs,
         "depth": depth, "theta": theta}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one CPPN, one source (a single substrate inspected interactively)
        _case("single_d5", "discover", 1, 8, 20, 1, 5, 0.03),
        # the benchmark's population of 1000 CPPNs on the XOR substrate, held on the device
        _case("xor_pop1000_d7", "discover", 1000, 20, 60, 0, 7, 0.03),
        # the tabular substrate: 32 inputs and one output, larger CPPNs
        _case("tabular_pop150_d6", "discover", 150, 40, 120, 32, 6, 0.03),
        # an evolution loop's discovery: a new population every call, at the paper's "depth 7"
        _case("fresh_pop1000_d7", "fresh", 1000, 20, 60, 0, 7, 0.03),
        # a new tabular population, an odd number of inputs
        _case("fresh_tabular_pop150_d6", "fresh", 150, 40, 120, 31, 6, 0.03),
        # whole generations: NEAT's usual population of 150 on a coarse grid, and 1000 at depth 7
        _case("generation_pop150_d5", "generation", 150, 20, 60, 0, 5, 0.03, types=1),
        _case("generation_pop1000_d7", "generation", 1000, 20, 60, 0, 7, 0.03, types=1),
        # the recurrent substrate: 100 CPPNs, hidden nodes queried on a grid of 1.4M positions
        _case("recurrent_pop100_d10", "recurrent", 100, 20, 60, 0, 10, 0.02),
        # the unfiltered outputs of a population (weight images, other filters in the caller)
        _case("raw_pop500_d7", "raw", 500, 20, 60, 0, 7, 0.03),
        # ES-HyperNEAT's filters on a tabular result
        _case("prune_tabular_pop150_d6", "prune", 150, 40, 120, 32, 6, 0.03, types=15),
        # kept networks on a data set: 1000 rows through 150 networks of 32 inputs
        _case("activate_pop150_rows1000", "activate", 150, 20, 60, 32, 5, 0.03, types=1, rows=1000),
        # one deep CPPN on 89M positions per source, streamed
        _case("stream_single_d13", "stream", 1, 30, 90, 0, 13, 0.01),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ones' ranges; at most 350M queries of a discover or fresh call."""
    kind = rng.choice(KINDS)
    h = rng.randint(4, 40)
    c = {"kind": kind, "h": h, "e": rng.randint(2 * h + 4, 3 * h + 10),
         "theta": round(rng.uniform(0.02, 0.05), 4)}
    if kind in ("discover", "fresh", "prune"):
        c["inputs"] = rng.choice((0, 1, rng.randint(2, 33)))
        c["genomes"] = _log(rng, 20 if kind == "prune" else 1, 1000 if c["inputs"] < 2 else 150)
        c["depth"] = rng.randint(4, 7)
        if kind == "prune":
            c["types"] = rng.choice((1, 3, 15))
    elif kind == "generation":
        c.update(inputs=0, genomes=_log(rng, 50, 1000), depth=rng.randint(4, 7), h=min(h, 20),
                 e=min(c["e"], 60), types=rng.choice((1, 15)))
    elif kind == "recurrent":
        c.update(inputs=0, genomes=_log(rng, 50, 100), depth=rng.randint(6, 9), h=min(h, 20),
                 e=min(c["e"], 60))
    elif kind == "raw":
        c.update(inputs=rng.choice((0, 1, 3)), genomes=_log(rng, 10, 500), depth=rng.randint(4, 7))
    elif kind == "activate":
        c.update(inputs=rng.randint(4, 33), genomes=_log(rng, 50, 150), depth=rng.randint(4, 6),
                 h=min(h, 20), e=min(c["e"], 60), types=rng.choice((1, 15)),
                 rows=_log(rng, 16, 1000))
    else:
        c.update(inputs=0, genomes=1, h=rng.randint(10, 30), depth=rng.randint(10, 12), theta=0.01)
        c["e"] = rng.randint(2 * c["h"], 3 * c["h"])
    return c


# ------------------------------------------------------------------------------- inputs

N_TYPES_W_MIN = 0.1  # expression's weight filter, as in the paper's experiments
BAND = 0.05          # band threshold of the prune cases
GEN_STEPS = 4        # synchronous activation steps


def _n(depth):
    return sum(4 ** k for k in range(1, depth + 1))  # grid positions


def _sources(case):
    """inputs 0: the XOR substrate; 1: one outgoing source; n > 1: the tabular substrate."""
    if case["inputs"] == 0:
        return W.xor_sources()
    if case["inputs"] == 1:
        return W.sources_array([(0.0, -1.0, W.DIR_OUT)])
    return W.tabular_sources(case["inputs"])


def _genomes(case, seed):
    """The seed's population; a single CPPN is redrawn until its substrate has a hidden node (a
    CPPN that is flat everywhere is not inspected or streamed)."""
    if case["genomes"] == 1:
        while True:
            g = W.single_cppn(seed, case["h"], case["e"])
            pop = emr.emr_pack_population(g)
            res = emr.emr_discover_all(pop, _sources(case), 4, _theta(case))
            if int(res["pair_offset"][-1].item()) > 0:
                return g
            seed += 1 << 32
    return W.population(seed, case["genomes"], case["h"], case["e"])


def _theta(case):
    return float(np.float32(case["theta"]))


def _capacity(case):
    pairs = case["genomes"] * len(_sources(case))
    return min(pairs * (1 + _n(case["depth"] - 1)), 1 << 19)


def _pad(case):
    """Fixed length of the buffers that collect results of input-dependent length."""
    return {"recurrent": 1 << 21, "prune": 1 << 20, "stream": 1 << 16}[case["kind"]]


def _result(pop, case):
    res = emr.alloc_result(pop, _sources(case), case["depth"], capacity=_capacity(case))
    for key in ("parent", "w4"):
        res[key].zero_()
    return res


def _rows(case, seed):
    return np.random.default_rng(seed + 1).uniform(-1.0, 1.0, (case["rows"], case["inputs"])) \
        .astype(np.float32)


def prepare(case, seed):
    genomes = _genomes(case, seed)
    kind, sources, depth, theta = case["kind"], _sources(case), case["depth"], _theta(case)
    s = {"case": case, "kind": kind, "sources": sources, "depth": depth, "theta": theta}
    if kind in ("discover", "fresh", "raw", "prune", "stream", "activate"):
        s["pop"] = emr.emr_pack_population(genomes)
    if kind in ("discover", "fresh"):
        s["res"] = _result(s["pop"], case)
    if kind in ("fresh", "generation", "recurrent"):
        s["flat"] = emr.flat_genomes(genomes)
    if kind == "prune":
        s["res"] = emr.emr_discover_all(s["pop"], sources, depth, theta)
    if kind == "activate":
        s["net"] = emr.emr_build_networks(s["pop"], sources, depth, theta, case["types"],
                                          N_TYPES_W_MIN, 1)
        s["rows"] = _rows(case, seed)
    if kind in ("recurrent", "prune"):
        s["pad"] = {}
    return s


def _padded(s, key, x, n):
    """x[:n] in a zeroed buffer of the case's fixed length that the state keeps."""
    buf = s["pad"].get(key)
    if buf is None:
        buf = torch.zeros((_pad(s["case"]),) + x.shape[1:], dtype=x.dtype, device=x.device)
        s["pad"][key] = buf
    n = min(n, len(buf))
    buf[:n].copy_(x[:n])
    return buf


def _records(res):
    return {k: res[k] for k in ("parent", "w4", "pair_count", "pair_offset")}


# ------------------------------------------------------------------------------- the pass

def run(s):
    kind, sources, depth, theta = s["kind"], s["sources"], s["depth"], s["theta"]
    if kind == "discover":
        emr.emr_discover(s["pop"], sources, depth, theta, res=s["res"])
        emr.emr_result_check(s["res"])
        return _records(s["res"])
    if kind == "fresh":
        pop = emr.emr_pack_population(s["flat"])
        emr.emr_discover(pop, sources, depth, theta, res=s["res"])
        emr.emr_result_check(s["res"])
        return _records(s["res"])
    if kind == "generation":
        pop = emr.emr_pack_population(s["flat"])
        net = emr.emr_build_networks(pop, sources, depth, theta, s["case"]["types"],
                                     N_TYPES_W_MIN, 1)
        fitness = net.xor_fitness(1, GEN_STEPS)
        torch.cuda.current_stream().synchronize()  # the loop reads the fitness before it goes on
        info = net.info()
        return {"fitness": fitness, "nodes": int(info.nodes), "edges": int(info.edges)}
    if kind == "recurrent":
        pop = emr.emr_pack_population(s["flat"])
        rec = emr.emr_discover_all(pop, sources, depth, theta)
        hid = emr.emr_hidden_sources(pop, sources, depth, rec)
        src, offs = emr.hidden_sources_to_host(hid)
        rec2 = emr.emr_discover_all(pop, src, depth, theta, src_offsets=offs)
        n1, n2 = int(rec["pair_offset"][-1].item()), int(rec2["pair_offset"][-1].item())
        return {"offsets": hid["offsets"], "cell": _padded(s, "cell", hid["cell"], hid["total"]),
                "parent1": _padded(s, "parent1", rec["parent"], n1),
                "w41": _padded(s, "w41", rec["w4"], n1),
                "pair_offset2": _padded(s, "po2", rec2["pair_offset"], len(rec2["pair_offset"])),
                "parent2": _padded(s, "parent2", rec2["parent"], n2),
                "w42": _padded(s, "w42", rec2["w4"], n2)}
    if kind == "raw":
        return emr.emr_eval_raw(s["pop"], sources, depth)
    if kind == "prune":
        conn = emr.emr_express(s["pop"], sources, depth, s["res"], s["case"]["types"],
                               N_TYPES_W_MIN)
        band = emr.emr_band_values(s["pop"], sources, depth, conn)
        kept = emr.emr_band_filter(conn, band, BAND)
        chain = emr.emr_chain_filter(s["res"], depth)
        n = conn["total"]
        return {"offset": conn["pair_offset"], "cell": _padded(s, "cell", conn["cell"], n),
                "w": _padded(s, "w", conn["w"], n), "band": _padded(s, "band", band, n),
                "band_offset": kept["pair_offset"],
                "band_cell": _padded(s, "band_cell", kept["cell"], kept["total"]),
                "band_w": _padded(s, "band_w", kept["w"], kept["total"]),
                "chain_offset": chain["pair_offset"],
                "chain_parent": _padded(s, "chain_parent", chain["parent"],
                                        int(chain["pair_offset"][-1].item()))}
    if kind == "activate":
        return s["net"].activate(s["rows"], GEN_STEPS)
    return _collect(s)


def _collect(s):
    """A streamed run whose sink keeps the records pair by pair."""
    pairs = s["pop"].n_genomes * len(s["sources"])
    got = [[] for _ in range(pairs)]

    def sink(pair, chunk, parent, w4):
        got[pair].append((parent, w4))

    emr.emr_discover_stream(s["pop"], s["sources"], s["depth"], s["theta"], sink)
    count = np.array([sum(len(p) for p, _ in g) for g in got], np.int64)
    n = _pad(s["case"])
    parent, w4 = np.zeros(n, np.int64), np.zeros((n, 4), np.float32)
    every = [d for g in got for d in g]
    if every:
        p = np.concatenate([d[0] for d in every])[:n]
        parent[:len(p)] = p
        w4[:len(p)] = np.concatenate([d[1] for d in every])[:n]
    return {"count": count, "parent": parent, "w4": w4}


# ------------------------------------------------------------------------------- what it takes

def _queries(case):
    q = case["genomes"] * len(_sources(case)) * _n(case["depth"])
    hidden = 26 * case["genomes"] * _n(case["depth"])  # hidden nodes of a genome, on average
    if case["kind"] == "generation" or case["kind"] == "recurrent":
        return q + hidden
    if case["kind"] == "prune":
        return 4 * 60 * case["genomes"] * len(_sources(case))  # the band's neighbours
    return 0 if case["kind"] == "activate" else q


def work(case):
    """Floating-point operations of the position-dependent part of every query (0.4 per edge that
    a genome can have, twice the half that is drawn: what a random CPPN of these sizes comes to on
    average) and the genomes read and results written once."""
    pairs = case["genomes"] * len(_sources(case))
    flops = _queries(case) * (0.4 if case["genomes"] > 1 else 0.45) * case["e"]
    data = case["genomes"] * 9 * case["e"] + 16 * pairs + 20 * 6 * pairs
    if case["kind"] == "raw":
        data += 4 * _queries(case)
    elif case["kind"] in ("generation", "recurrent"):
        data += 26 * case["genomes"] * (16 + 20 * 60) + 26 * case["genomes"] * 12
    elif case["kind"] == "prune":
        data += pairs * 15 * (20 + 4 * 4 * 8)
    elif case["kind"] == "activate":
        edges = 60 * case["genomes"] * case["inputs"]
        flops = 2 * edges * GEN_STEPS * case["rows"]
        data = 8 * edges + 4 * case["rows"] * (case["inputs"] + case["genomes"])
    return {"bytes": float(data), "flops": float(flops)}


def tolerance(case):
    return {"rel": 2e-5, "max": 1e-3, "differ": 0.0}


# ------------------------------------------------------------------------------- in 64 bits

_ACT = (lambda z: z, torch.sigmoid, torch.tanh, lambda z: torch.exp(-z * z), torch.sin, torch.abs)


def _cppn64(g, values):
    """The output of one CPPN; values: x1, y1, x2, y2, 1 as broadcastable float64 tensors."""
    kind, n = g["kind"], len(g["kind"])
    into = [[] for _ in range(n)]
    for u, v, w, on in zip(g["src"], g["dst"], g["w"], g["enabled"]):
        if on:
            into[int(v)].append((int(u), float(w)))
    out = int(np.nonzero(kind == W.KIND_OUTPUT)[0][0])
    have = {}

    def node(v):
        if v not in have:
            if kind[v] < W.KIND_HIDDEN:
                have[v] = values[int(kind[v])]
            else:
                z = torch.full((1, 1), float(g["bias"][v]), dtype=torch.float64,
                               device=values[0].device)
                for u, w in into[v]:
                    z = z + w * node(u)
                have[v] = _ACT[int(g["act"][v])](z)
        return have[v]

    return node(out)


def _grid64(first, n, dev):
    """Centres (x, y) of grid positions first .. first + n: position p is heap cell p + 1, its
    children 4p + 5 .. 4p + 8 (child k on the +x side by bit 0 of k, the +y side by bit 1)."""
    f = torch.arange(first + 1, first + n + 1, device=dev)
    x = torch.zeros(n, dtype=torch.float64, device=dev)
    y = torch.zeros_like(x)
    half = torch.ones_like(x)
    digits, level = [], 0
    while True:
        live = f > 0
        if not bool(live.any()):
            break
        digits.append((torch.where(live, (f - 1) % 4, 0), live))
        f = torch.where(live, (f - 1) // 4, 0)
        level += 1
    for k, live in reversed(digits):
        half = torch.where(live, half * 0.5, half)
        x = x + torch.where(live, (2.0 * (k % 2) - 1.0) * half, 0.0)
        y = y + torch.where(live, (2.0 * (k // 2) - 1.0) * half, 0.0)
    return x, y


def _outputs64(g, sx, sy, outgoing, x, y):
    """[sources, positions] outputs of the queries from (or to) sources at (sx, sy)."""
    s, p = (sx[:, None], sy[:, None]), (x[None, :], y[None, :])
    one = torch.ones((1, 1), dtype=torch.float64, device=x.device)
    a, b = (s, p) if outgoing else (p, s)
    return _cppn64(g, (*a, *b, one)).expand(len(sx), len(x))


def _discover64(g, sources, depth, theta, dev, centres=None):
    """Per source of one genome: (kept parents, their children's outputs [n, 4])."""
    got = [([], []) for _ in range(len(sources))]
    total = _n(depth)
    for d in (0, 1):
        who = [j for j in range(len(sources)) if int(sources[j]["dir"]) == d]
        for c0 in range(0, len(who), 256):
            part = who[c0:c0 + 256]
            sx = torch.tensor([float(sources[j]["x"]) for j in part], dtype=torch.float64, device=dev)
            sy = torch.tensor([float(sources[j]["y"]) for j in part], dtype=torch.float64, device=dev)
            step = max(4, (1 << 24) // len(part) // 4 * 4)
            for first in range(0, total, step):
                n = min(step, total - first)
                if centres is not None:
                    x, y = centres[0][first:first + n], centres[1][first:first + n]
                else:
                    x, y = _grid64(first, n, dev)
                w = _outputs64(g, sx, sy, d == 0, x, y).reshape(len(part), n // 4, 4)
                keep = w.var(dim=2, unbiased=False) > theta
                if not bool(keep.any()):
                    continue
                si, pi = keep.nonzero(as_tuple=True)
                w = w[si, pi]
                cuts = torch.searchsorted(si, torch.arange(len(part) + 1, device=dev)).tolist()
                for k, j in enumerate(part):
                    got[j][0].append(pi[cuts[k]:cuts[k + 1]] + first // 4)
                    got[j][1].append(w[cuts[k]:cuts[k + 1]])
    none = (torch.zeros(0, dtype=torch.int64, device=dev),
            torch.zeros((0, 4), dtype=torch.float64, device=dev))
    return [(torch.cat(p), torch.cat(w)) if p else none for p, w in got]


def _fixed(x, n, dtype=None):
    out = torch.zeros((n,) + x.shape[1:], dtype=dtype or x.dtype, device=x.device)
    m = min(n, len(x))
    out[:m] = x[:m]
    return out


def _offsets64(counts, dev):
    return torch.tensor(np.concatenate([[0], np.cumsum(counts)]), dtype=torch.int64, device=dev)


def exact(case, seed):
    if case["kind"] == "generation" and case["genomes"] * _n(case["depth"]) > 30_000_000:
        return None
    dev = torch.device("cuda")
    genomes, sources, depth, theta = _genomes(case, seed), _sources(case), case["depth"], _theta(case)
    kind = case["kind"]
    centres = _grid64(0, _n(depth), dev) if depth <= 11 else None
    if kind == "raw":
        out = torch.empty((len(genomes) * len(sources), _n(depth)), dtype=torch.float64, device=dev)
        for i, g in enumerate(genomes):
            for j, s in enumerate(sources):
                p = [torch.tensor([float(s[k])], dtype=torch.float64, device=dev) for k in ("x", "y")]
                out[i * len(sources) + j] = _outputs64(g, *p, int(s["dir"]) == 0, *centres)[0]
        return out
    phases = [(sources, [_discover64(g, sources, depth, theta, dev, centres) for g in genomes])]
    pairs = [r for rs in phases[0][1] for r in rs]
    counts = np.array([len(p) for p, _ in pairs])
    parent, w4 = torch.cat([p for p, _ in pairs]), torch.cat([w for _, w in pairs])
    if kind in ("discover", "fresh"):
        n = max(_capacity(case), 1)
        return {"parent": _fixed(parent, n, torch.int32), "w4": _fixed(w4, n),
                "pair_count": torch.tensor(counts, device=dev),
                "pair_offset": _offsets64(counts, dev)}
    if kind == "stream":
        n = _pad(case)
        return {"count": torch.tensor(counts), "parent": _fixed(parent, n), "w4": _fixed(w4, n)}
    if kind == "prune":
        return _prune64(case, genomes, sources, pairs, centres)
    # hidden nodes: the children of the outgoing pairs' kept parents, queried from their centres
    cells, hidden = [], []
    for g, rs in zip(genomes, phases[0][1]):
        kids = [4 * p[:, None] + torch.arange(1, 5, device=dev)
                for (p, _), s in zip(rs, sources) if int(s["dir"]) == 0]
        cells.append(torch.unique(torch.cat(kids).reshape(-1)))
        at = (cells[-1] - 1).cpu()
        src = np.zeros(len(at), emr.SOURCE_DTYPE)
        src["x"], src["y"] = centres[0].cpu()[at].numpy(), centres[1].cpu()[at].numpy()
        hidden.append(_discover64(g, src, depth, theta, dev, centres))
    if kind == "recurrent":
        n, all2 = _pad(case), [r for rs in hidden for r in rs]
        return {"offsets": _offsets64([len(c) for c in cells], dev),
                "cell": _fixed(torch.cat(cells), n, torch.int32),
                "parent1": _fixed(parent, n, torch.int32), "w41": _fixed(w4, n),
                "pair_offset2": _fixed(_offsets64([len(p) for p, _ in all2], dev), n),
                "parent2": _fixed(torch.cat([p for p, _ in all2]), n, torch.int32),
                # (of the second phase's many records one may lie within rounding of the
                # threshold, and the records after it then have other places)
                "w42": None}
    nets = _networks64(case, sources, phases[0][1], cells, hidden, centres)
    if kind == "activate":
        return _activate64(nets, torch.tensor(_rows(case, seed), dtype=torch.float64, device=dev))
    rows = torch.tensor([[0, 1, 0], [0, 1, 1], [1, 1, 0], [1, 1, 1]], dtype=torch.float64, device=dev)
    target = torch.tensor([0.0, 1.0, 1.0, 0.0], dtype=torch.float64, device=dev)
    out = _activate64(nets, rows)[:, :, 0]
    return {"fitness": 1.0 - ((out - target) ** 2).mean(dim=1), "nodes": nets["nodes"],
            "edges": len(nets["w"])}


def _expressed64(case, source, record, centres):
    """(cells, weights) of one pair's connections."""
    p, w = record
    cell = (4 * p[:, None] + torch.arange(1, 5, device=p.device)).reshape(-1)
    w = w.reshape(-1)
    cx, cy = centres[0][cell - 1], centres[1][cell - 1]
    sx, sy = float(source["x"]), float(source["y"])
    same = (cx == sx) & (cy == sy)
    up = cy > sy if int(source["dir"]) == 0 else cy < sy
    kind = torch.where(same, 8, torch.where(up, 1, torch.where(cy == sy, 4, 2)))
    keep = ((kind & case["types"]) != 0) & (w.abs() > float(np.float32(N_TYPES_W_MIN)))
    return cell[keep], w[keep]


def _prune64(case, genomes, sources, pairs, centres):
    dev, n = pairs[0][0].device, _pad(case)
    cells, ws, bands, chains = [], [], [], []
    for r, record in enumerate(pairs):
        g, s = genomes[r // len(sources)], sources[r % len(sources)]
        cell, w = _expressed64(case, s, record, centres)
        x, y = centres[0][cell - 1], centres[1][cell - 1]
        level = torch.zeros_like(cell)
        for k in range(1, case["depth"]):
            level += (cell > _n(k)).to(level.dtype)
        side = 2.0 * 0.5 ** (level + 1).double()
        if len(cell):
            p = [torch.tensor([float(s[k])], dtype=torch.float64, device=dev) for k in ("x", "y")]
            px = torch.cat([x - side, x + side, x, x])
            py = torch.cat([y, y, y - side, y + side])
            v = _outputs64(g, *p, int(s["dir"]) == 0, px, py)[0].reshape(4, -1)
            d = (w[None, :] - v).abs()
            bands.append(torch.maximum(torch.minimum(d[0], d[1]), torch.minimum(d[2], d[3])))
        else:
            bands.append(w)
        cells.append(cell)
        ws.append(w)
        kept, chain = set(), []
        for q in record[0].tolist():
            if q == 0 or (q - 1) // 4 in kept:
                kept.add(q)
                chain.append(q)
        chains.append(chain)
    keep = [b > float(np.float32(BAND)) for b in bands]
    return {"offset": _offsets64([len(c) for c in cells], dev),
            "cell": _fixed(torch.cat(cells), n, torch.int32), "w": _fixed(torch.cat(ws), n),
            "band": _fixed(torch.cat(bands), n),
            "band_offset": _offsets64([int(k.sum()) for k in keep], dev),
            "band_cell": _fixed(torch.cat([c[k] for c, k in zip(cells, keep)]), n, torch.int32),
            "band_w": _fixed(torch.cat([w[k] for w, k in zip(ws, keep)]), n),
            "chain_offset": _offsets64([len(c) for c in chains], dev),
            "chain_parent": _fixed(torch.tensor([q for c in chains for q in c], dtype=torch.int64,
                                                device=dev), n, torch.int32)}


def _networks64(case, sources, phase0, cells, hidden, centres):
    """All genomes' pruned networks in one node numbering: edges, inputs and outputs [genomes, k]."""
    dev, sub, span = centres[0].device, len(sources), len(sources) + _n(case["depth"]) + 1
    known = torch.zeros(len(cells) * span, dtype=torch.bool, device=dev)
    us, vs, ws = [], [], []
    for g, (rs, cs, hs) in enumerate(zip(phase0, cells, hidden)):
        base = g * span + sub
        known[base + cs] = True
        centre = [c[cs - 1].tolist() for c in centres]
        asked = [(sources[j], g * span + j, rs[j]) for j in range(sub)]
        asked += [({"x": centre[0][i], "y": centre[1][i], "dir": 0}, base + int(c), hs[i])
                  for i, c in enumerate(cs.tolist())]
        for source, at, record in asked:
            # cells that the last phase finds are nodes too
            if int(source["dir"]) == 0 and len(record[0]):
                known[base + (4 * record[0][:, None] + torch.arange(1, 5, device=dev)).reshape(-1)] = True
            cell, w = _expressed64(case, source, record, centres)
            here = torch.full_like(cell, at)
            us.append(here if int(source["dir"]) == 0 else base + cell)
            vs.append(base + cell if int(source["dir"]) == 0 else here)
            ws.append(w)
    u, v, w = torch.cat(us), torch.cat(vs), torch.cat(ws)
    first = torch.arange(len(cells), device=dev)[:, None] * span
    ins = first + torch.tensor([j for j in range(sub) if int(sources[j]["dir"]) == 0], device=dev)
    outs = first + torch.tensor([j for j in range(sub) if int(sources[j]["dir"]) != 0], device=dev)
    known[ins], known[outs] = True, True
    ok = known[u] & known[v]
    u, v, w = u[ok], v[ok], w[ok]

    def reach(seeds, a, b):
        seen = torch.zeros_like(known)
        seen[seeds.reshape(-1)] = True
        n = -1
        while n != int(seen.sum()):
            n = int(seen.sum())
            seen[b[seen[a]]] = True
        return seen

    fwd, bwd = reach(ins, u, v), reach(outs, v, u)
    node = fwd & bwd & known
    node[ins], node[outs] = True, True
    ok = fwd[u] & bwd[v]
    new = torch.cumsum(node.to(torch.int64), 0) - 1
    return {"u": new[u[ok]], "v": new[v[ok]], "w": w[ok], "nodes": int(node.sum()),
            "ins": new[ins], "outs": new[outs]}


def _activate64(nets, rows):
    """[genomes, rows, outputs] after GEN_STEPS synchronous steps."""
    out = []
    for r in rows.split(64):
        z = torch.zeros((nets["nodes"], len(r)), dtype=torch.float64, device=rows.device)
        at = nets["ins"].reshape(-1)
        clamp = r.T.repeat(len(nets["ins"]), 1)
        z[at] = clamp
        for _ in range(GEN_STEPS):
            s = torch.zeros_like(z)
            for k in range(0, len(nets["w"]), 1 << 22):
                u, v, w = (nets[n][k:k + (1 << 22)] for n in ("u", "v", "w"))
                s.index_add_(0, v, w[:, None] * z[u])
            z = torch.sigmoid(s)
            z[at] = clamp
        out.append(z[nets["outs"]].transpose(1, 2))
    return torch.cat(out, dim=1)
