"""The measured calls of the k-hop retrieval library.

A case names a synthetic graph, a batch of queries and the call a program makes with them.  The
graphs have the shapes of the benchmark workloads (see ``kggen``), drawn on the GPU so that a new
graph costs a second:

``uniform``  subjects with out-degrees from P(d) ~ d^-2, objects uniform: a small curated graph.
``concept``  out- and in-degrees from P(d) ~ d^-alpha (1.8, cap 200,000), rank matched, relations by
             rank with p(r) ~ (r+1)^-1.1: biomedical concept graphs.
``hub``      0.01 % of the entities are the subject of 40 % and the object of 40 % of the triples.

Every call goes through the public entry points: ``Graph.khop`` and then what the program asked for
(``call``): ``lists`` (query-major entity / hop / predecessor lists), ``level`` (walk-exact search and
one level), ``triples`` (active triples of the last hop), ``paths`` (shortest paths of given pairs) or
``chains`` (bulk export of complete paths).  Results go to buffers that the program keeps, large enough
for any answer of the case; what lies behind an answer in them stays zero.  Everything a pass returns is
whole numbers.
"""
import math

import numpy as np
import torch

import paper_2604_18913_amd as lkg

CAP = 200_000  # largest degree of the power laws
PAGE = 1 << 20  # chains written at a time


def _case(name, call, graph, entities, triples, relations, queries, k, first=0, last=None, mask=False, seeds=5,
          live_seeds=False, shards=0):
    """``first`` / ``last``: the queries whose results are fetched (the batch is always expanded whole);
    ``seeds``: each query has 1 .. seeds of them; ``live_seeds``: drawn among the subjects only."""
    return {"name": name, "call": call, "graph": graph, "entities": entities, "triples": triples,
            "relations": relations, "queries": queries, "k": k, "first": first,
            "last": queries if last is None else last, "mask": mask, "seeds": seeds, "live_seeds": live_seeds,
            "shards": shards}


def listed():
    return [
        # one question to a small graph: nothing but latency, launches and read-backs
        _case("lookup_1q", "lists", "uniform", 10_000, 50_000, 20, 1, 2, live_seeds=True),
        # the first benchmark workload: 64 one-seed questions to the same graph
        _case("small_64q", "lists", "uniform", 10_000, 50_000, 20, 64, 2, seeds=1),
        # one interactive question to a graph of UMLS size (407K concepts, 3.4M triples), three hops
        _case("concept_1q", "lists", "concept", 407_000, 3_400_000, 500, 1, 3, live_seeds=True),
        # a service's batch of 200 questions with relation whitelists to that graph (four-word planes)
        _case("concept_200q_mask", "lists", "concept", 407_000, 3_400_000, 500, 200, 3, mask=True),
        # the headline workload: every list of a full batch at 30M triples
        _case("biomed_1024q", "lists", "concept", 3_000_000, 30_000_000, 500, 1024, 3),
        # the same graph, whitelists of 10 .. 50 relations, a batch that does not fill its last word
        _case("biomed_1000q_mask", "lists", "concept", 3_000_000, 30_000_000, 500, 1000, 3, mask=True),
        # ends of the walks of exactly three triples (the plain iteration) of a page of 96 queries
        _case("biomed_walk_level", "level", "concept", 3_000_000, 30_000_000, 500, 1024, 3, first=448, last=544),
        # active triples of the third hop with their components, for a page of 16 queries
        _case("biomed_triples_16q", "triples", "concept", 3_000_000, 30_000_000, 500, 1024, 3, last=16),
        # explanations: up to 16 shortest paths for 4,096 (query, reached entity) pairs, whitelists
        _case("biomed_paths_mask", "paths", "concept", 3_000_000, 30_000_000, 500, 1024, 2, mask=True),
        # complete paths of one question in bulk: count all chains of three triples, write a page of them
        _case("concept_chains", "chains", "concept", 407_000, 3_400_000, 500, 8, 3, first=3, last=4,
              live_seeds=True),
        # the hub-heavy workload, a full batch of one-seed questions, lists of one page of 64 queries
        _case("hub_1024q_page", "lists", "hub", 20_000_000, 300_000_000, 1000, 1024, 3, last=64, seeds=1),
        # a graph behind the shard cache (8 subject shards, every unit fits), lists of a ragged page
        _case("sharded_1024q_page", "lists", "concept", 5_000_000, 50_000_000, 2000, 1024, 3, first=100, last=163,
              seeds=3, shards=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["lists", "lists", "lists", "lists", "level", "triples", "paths", "chains"])
    graph = rng.choice(["uniform", "concept", "concept", "hub"])
    entities = _log_int(rng, 5_000, 407_000 if call == "chains" else 3_000_000)
    triples = int(entities * rng.uniform(4, 12))
    relations = rng.choice([20, 100, 500, 1000, 2000])
    queries = _log_int(rng, 1, 8 if call == "chains" else 1024)
    k = rng.choice([1, 2, 3, 3, 4]) if call in ("lists", "paths") else rng.choice([2, 3, 3])
    first, last = 0, queries
    if call == "chains":
        first = rng.randrange(queries)
        last = first + 1
    elif call == "triples":
        first = rng.randrange(queries)
        last = min(queries, first + rng.randint(1, 16))
    elif call == "level" or call == "lists" and rng.random() < 0.4:  # a page of the batch
        first = rng.randrange(queries)
        last = min(queries, first + _log_int(rng, 1, 256))
    mask = rng.random() < 0.4 and call != "level"
    shards = rng.randint(2, 8) if call == "lists" and queries > 64 and rng.random() < 0.25 else 0
    c = _case("", call, graph, entities, triples, relations, queries, k, first, last, mask, rng.choice([1, 3, 5]),
              call == "chains" or queries < 64 or rng.random() < 0.5, shards)
    del c["name"]
    return c


# ------------------------------------------------------------------------- inputs
def _degrees(gen, n, total, alpha, cap):
    """n degrees from the truncated power law on [dmin, cap], dmin the smallest whose mean gives `total`
    triples; the ones behind the running sum `total` are 0."""
    cap = max(1, min(cap, n - 1))
    d = np.arange(1, cap + 1, dtype=np.float64)
    w = d ** -alpha
    sw, sd = np.cumsum(w[::-1])[::-1], np.cumsum((d * w)[::-1])[::-1]
    enough = np.flatnonzero(sd / sw * n >= total)
    dmin = int(enough[0]) + 1 if enough.size else cap
    cdf = torch.from_numpy(np.cumsum(w[dmin - 1:]) / sw[dmin - 1]).cuda()
    u = torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)
    deg = (torch.searchsorted(cdf, u) + dmin).clamp_(max=cap)
    deg[torch.cumsum(deg, 0) > total] = 0
    return deg


def _randint(gen, hi, n):
    return torch.randint(0, hi, (n,), generator=gen, device="cuda")


def _stubs(ids, deg):
    return torch.repeat_interleave(ids, deg)


def _triples(case, gen):
    """(subject, relation, object) as host int32 arrays: pairs drawn from the two stub lists, distinct, in
    random order, so that triple ids carry no locality."""
    E, T, R, kind = case["entities"], case["triples"], case["relations"], case["graph"]
    perm = torch.randperm(E, generator=gen, device="cuda")
    if kind == "uniform":
        s_stubs = _stubs(perm, _degrees(gen, E, T, 2.0, E - 1))
        o_stubs = torch.arange(E, device="cuda")
    elif kind == "concept":
        d_out, d_in = (_degrees(gen, E, T, 1.8, CAP).sort(descending=True).values for _ in range(2))
        s_stubs, o_stubs = _stubs(perm, d_out), _stubs(perm, d_in)
    else:
        n_hub = max(2, round(E * 1e-4))
        hubs, rest = perm[:n_hub], perm[n_hub:]
        s_hub = hubs.repeat(int(T * 0.4) // n_hub + 1)
        s_stubs = torch.cat([s_hub, _stubs(rest, _degrees(gen, E - n_hub, T - s_hub.numel(), 2.2, CAP))])
        n_obj = int(T * 0.4)
        o_stubs = torch.cat([hubs[_randint(gen, n_hub, n_obj)], rest[_randint(gen, E - n_hub, T - n_obj)]])
    n = int(T * 1.5) + 16  # hub pairs repeat: what is left after dropping them is cut to T
    s, o = s_stubs[_randint(gen, s_stubs.numel(), n)], o_stubs[_randint(gen, o_stubs.numel(), n)]
    del s_stubs, o_stubs
    if kind == "concept":
        w = (torch.arange(R, device="cuda", dtype=torch.float64) + 1.0) ** -1.1
        cdf = torch.cumsum(w / w.sum(), 0)
        r = torch.searchsorted(cdf, torch.rand(n, generator=gen, device="cuda", dtype=torch.float64)).clamp_(max=R - 1)
    else:
        r = _randint(gen, R, n)
    key = torch.unique((s * R + r) * E + o)
    del s, r, o
    key = key[torch.randperm(key.numel(), generator=gen, device="cuda")[:T]]
    o = (key % E).to(torch.int32).cpu().numpy()
    key //= E
    return (key // R).to(torch.int32).cpu().numpy(), (key % R).to(torch.int32).cpu().numpy(), o


def _queries(case, gen, subj):
    """seed_off int64[Q+1], seeds int32 on the GPU; hub graphs seed every second query at a hub."""
    Q, E = case["queries"], case["entities"]
    counts = 1 + _randint(gen, case["seeds"], Q)
    off = torch.zeros(Q + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(counts, 0, out=off[1:])
    n = int(off[-1])
    pick = _randint(gen, len(subj), n).cpu().numpy()
    by_triple = torch.from_numpy(subj[pick]).to("cuda", torch.int64)  # a subject drawn by its triples: mostly hubs
    seeds = _randint(gen, E, n)
    if case["live_seeds"]:
        live = torch.zeros(E, dtype=torch.bool, device="cuda")
        live[torch.from_numpy(subj).cuda().long()] = True
        ids = live.nonzero().flatten()
        seeds = ids[_randint(gen, ids.numel(), n)]
    elif case["graph"] == "hub":
        owner = torch.repeat_interleave(torch.arange(Q, device="cuda"), counts)
        seeds = torch.where(owner % 2 == 0, by_triple, seeds)
    return off, seeds.to(torch.int32)


def _whitelists(case, gen):
    """int64[Q, ceil(R/64)]: 10 .. 50 relations of each query (at most half of a small relation set)."""
    Q, R = case["queries"], case["relations"]
    lo, hi = min(10, R // 4), min(50, R // 2)
    count = lo + _randint(gen, hi - lo + 1, Q)
    rank = torch.rand(Q, R, generator=gen, device="cuda").argsort(1).argsort(1)
    words = (R + 63) // 64
    bits = torch.zeros(Q, words * 64, dtype=torch.int64, device="cuda")
    bits[:, :R] = (rank < count[:, None]).long()
    return (bits.view(Q, words, 64) << torch.arange(64, device="cuda")).sum(2)


def _capacity(case):
    """Entries of the result buffers: a bound on the answers, whatever the inputs."""
    nq, E, T = case["last"] - case["first"], case["entities"], case["triples"]
    if case["call"] == "triples":
        return nq * T
    n = nq * E
    return n // 2 if case["graph"] == "concept" and n > 1 << 26 else n  # more than half are never an object


def _buffers(case):
    n, call = _capacity(case), case["call"]
    dtypes = {"lists": (torch.int32, torch.uint8, torch.int32), "level": (torch.int32,),
              "triples": (torch.int32,) * 4}.get(call)
    if dtypes:
        return [torch.zeros(n, dtype=d, device="cuda") for d in dtypes]
    if call == "chains":
        return [torch.zeros((PAGE, case["k"]), dtype=torch.int32, device="cuda"),
                torch.zeros(PAGE, dtype=torch.int32, device="cuda")]
    return []


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    subj, rel, obj = _triples(case, gen)
    graph = lkg.Graph(subj, rel, obj, case["entities"], case["relations"], num_shards=case["shards"])
    off, seeds = _queries(case, gen, subj)
    state = {"case": case, "graph": graph, "off": off, "seeds": seeds,
             "mask": _whitelists(case, gen) if case["mask"] else None, "buffers": _buffers(case)}
    if case["call"] == "paths":  # the pairs a program wants explained: entries of an earlier answer's lists
        res = graph.khop(off, seeds, case["k"], state["mask"])
        o = res.offsets()
        entity, _, _ = res.fetch(want_hop=False, want_pred=False)
        at = _randint(gen, int(o[-1]), 4096).sort().values
        state["query"] = (torch.searchsorted(torch.from_numpy(o).cuda(), at, right=True) - 1).to(torch.int32)
        state["target"] = entity[at].contiguous()
        torch.cuda.synchronize()
        res.close()
    torch.cuda.synchronize()
    return state


def run(state):
    case, g, buf = state["case"], state["graph"], state["buffers"]
    k, first, last, call = case["k"], case["first"], case["last"], case["call"]
    res = g.khop(state["off"], state["seeds"], k, state["mask"], walk_exact=call in ("level", "chains"))
    out = {"offsets": res.offsets()}
    if call == "lists":
        res.fetch(first, last, out=buf)
        out["entity"], out["hop"], out["pred"] = buf
    elif call == "level":
        out["level_offsets"], entity = res.level(k, first, last)
        buf[0][:entity.numel()] = entity
        out["entity"] = buf[0]
    elif call == "triples":
        out["triple_offsets"] = res.active_triples(k, first, last, out=buf)[0]
        out["triple"], out["subject"], out["relation"], out["object"] = buf
    elif call == "paths":
        out["count"], out["edges"] = g.paths(res, state["query"], state["target"], 16)
    else:
        total = res.walks_count(first, k)
        n = min(total, PAGE)  # the page in the middle of the list
        res.walks_fetch(first, k, (total - n) // 2, n, out=buf)
        out["total"] = total
        out["edges"], out["target"] = buf
    res.close()
    return out


# ------------------------------------------------------------------------- work, tolerance
def _reached_share(case):
    """Share of the (query, entity) pairs a search of k hops reaches, as measured on these shapes."""
    shares = SHARE[case["graph"]]
    k = min(case["k"], len(shares))
    share = shares[k - 1]
    return share * MASKED[min(k, len(MASKED)) - 1] if case["mask"] else share


SHARE = {"uniform": (5e-4, 3e-3, 0.02, 0.1), "concept": (1e-5, 0.02, 0.16, 0.25), "hub": (0.01, 0.4, 0.75, 0.9)}
MASKED = (0.1, 0.02, 0.05, 0.06)


def work(case):
    """Bytes of one pass: the graph's ids read once (4 per triple, relation ids with a whitelist), the
    outputs written once.  There is no arithmetic but bit operations."""
    T, E, k, call = case["triples"], case["entities"], case["k"], case["call"]
    nq = case["last"] - case["first"]
    read = T * (6 if case["mask"] else 4) + 8 * case["queries"]
    pairs = nq * E * _reached_share(case)
    if call == "lists":
        out = 9 * pairs
    elif call == "level":
        out = 4 * pairs
    elif call == "triples":
        out = 16 * nq * T * _triple_share(case)
    elif call == "paths":
        read, out = read + 4096 * 8, 4096 * (4 + 64 * k)
    else:
        read, out = read + 8 * k * T, (4 * k + 4) * PAGE
    return {"bytes": int(read + out), "flops": 0}


def _triple_share(case):
    """Share of a graph's triples that leave the last frontier of a query."""
    share = {"uniform": 0.01, "concept": 0.4, "hub": 0.7}[case["graph"]] if case["k"] > 2 else 0.02
    return share * 0.02 if case["mask"] else share


def tolerance(case):
    return "exact"
