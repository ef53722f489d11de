"""The work that a user of this package has it do, as timed cases.

Seven kinds of call, each through the package's public entry points:

  count     coact_build: dispatch and co-activation counts of a routing trace
  graph     reweight: family preferences and the task-modulated graph from such counts
  diagnose  gesr_scores, activation_distance and pair_jaccard of such counts
  rank      placement_load and group_objective of a set of candidate placements
  score     eval_placements and jain_index: costs, loads and balance of placements on a serving trace
  stats     eval_trace_stats: the per-token statistics of a default and a grouped placement
  online    eval_online: scoring with decayed per-GPU loads

Sizes are those of the presets in synth.CONFIGS (small to large backbones), of the README's example and of
bench.py; the token counts of the large ones are cut so that inputs are quick to make.  Traces follow the same
law as the presets' (planted family clusters and generic experts, Gumbel-top-k).
"""
import math

import numpy as np
import torch

import paper_2606_01007_amd as tacg
from paper_2606_01007_amd import synth

THETA = (3, 20)
RHO = 0.995
EXACT_WORK = 2e9  # placement-token-layers that the plain scoring below takes in a few seconds


def listed():
    return [
        # a unit-test sized calibration trace (the "tiny" preset): the smallest call, latency only
        dict(name="count_tiny", kind="count", E=8, k=2, L=2, F=3, N=3 * 2048, mix="uniform"),
        # a calibration trace of ordinary length on a 60-expert backbone, the README's 20000 tokens per family
        dict(name="count_60", kind="count", E=60, k=4, L=24, F=6, N=6 * 20000, mix="uniform"),
        # a long calibration trace on a 256-expert backbone, all layers
        dict(name="count_256", kind="count", E=256, k=8, L=58, F=16, N=(1 << 21) - 37, mix="uniform"),
        # the graph that the grouping step reads, for every layer of the 256-expert backbone
        dict(name="graph_256", kind="graph", E=256, k=8, L=58, F=16, n=4096),
        # choice of generic experts and the motivation diagnostics of the same counts
        dict(name="diagnose_256", kind="diagnose", E=256, k=8, L=58, F=16, n=4096, top=64),
        # a search's set of candidate placements: snapshot loads and grouping objective of each
        dict(name="rank_256", kind="rank", E=256, k=8, L=58, F=16, n=4096, P=1024, G=32),
        # the tiny preset's 16 placements: the smallest scoring call
        dict(name="score_tiny", kind="score", E=8, k=2, L=2, F=3, N=3 * 2048, mix="uniform", P=16, G=4, n_rep=0, R=0),
        # 512 placements of the 60-expert backbone on 6 GPUs, some experts replicated twice
        dict(name="score_60", kind="score", E=60, k=4, L=24, F=6, N=6 * 20000 + 7, mix="uniform", P=512, G=6, n_rep=4,
             R=2),
        # 1024 placements of the 128-expert backbone on one 8-GPU node, skewed serving mix
        dict(name="score_128", kind="score", E=128, k=8, L=48, F=16, N=1 << 18, mix="zipf", P=1024, G=8, n_rep=8, R=2),
        # 1024 placements of the 256-expert backbone on 32 GPUs, the benchmark's call at a sixteenth of its tokens
        dict(name="score_256", kind="score", E=256, k=8, L=58, F=16, N=1 << 19, mix="dirichlet", P=1024, G=32, n_rep=16,
             R=3),
        # the default against the grouped placement on a serving trace, as a placement report needs it
        dict(name="stats_256", kind="stats", E=256, k=8, L=58, F=16, N=1 << 19, mix="dirichlet", P=2, G=32, n_rep=16,
             R=3),
        # decayed-load scoring of 1024 placements on the start of a serving trace
        dict(name="online_256", kind="online", E=256, k=8, L=58, F=16, N=1 << 15, mix="dirichlet", P=1024, G=32,
             n_rep=16, R=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["count", "count", "graph", "diagnose", "rank", "score", "score", "score", "stats", "online"])
    E = _log(rng, 8, 256)
    k = rng.randint(2, min(10, E // 3))
    c = dict(kind=kind, E=E, k=k, L=_log(rng, 2, 58), F=rng.randint(2, 16))
    if kind in ("graph", "diagnose", "rank"):
        c["n"] = _log(rng, 256, 4096)
        if kind == "diagnose":
            c["top"] = rng.choice([16, 64, 200])
        if kind == "rank":
            c["P"], c["G"] = _log(rng, 2, 1024), rng.randint(2, min(32, E))
        return c
    c["mix"] = rng.choice(["uniform", "zipf", "dirichlet"])
    if kind == "count":
        most = (1 << 21) * 58 * 28 / (c["L"] * (k + k * (k - 1) / 2))
        c["N"] = _log(rng, 512, max(512, min(1 << 21, most)))
        return c
    c["G"] = rng.randint(2, min(32, E))
    c["R"] = rng.randint(0, min(3, c["G"] - 1))
    c["n_rep"] = rng.randint(1, max(1, min(16, E // 12))) if c["R"] else 0
    if kind == "stats":
        c["P"] = rng.randint(1, 8)
        c["N"] = _log(rng, 512, 1 << 19)
    elif kind == "online":
        c["P"] = _log(rng, 1, 1024)
        c["N"] = _log(rng, 512, 1 << 15)
    else:
        c["P"] = _log(rng, 1, 1024)
        most = (1 << 19) * 58 * 1024 * 10 / (c["L"] * (64 + c["P"]) * (k + 2))
        c["N"] = _log(rng, 512, max(512, min(1 << 19, most)))
    return c


# ---- inputs -------------------------------------------------------------------------------------

def _planted(c, seed):
    E = c["E"]
    size = max(1, min(10, E // 8))
    generic = c.get("n_rep") or max(1, E // 16)
    return synth.planted_logits(E, c["L"], c["F"], size, min(2, max(1, (E - generic) // size)), 1.5, generic, 1.0, seed)


def _trace(c, seed):
    pl = _planted(c, seed)
    shares = synth.mix_shares(c["mix"], c["F"], {"uniform": 0.0, "zipf": 1.1, "dirichlet": 0.3}[c["mix"]], seed)
    n = synth.largest_remainder(c["N"], shares)
    return synth.sample_trace(pl.mu, n, c["k"], seed, "cuda"), synth.fam_offsets(n), pl


def _placements(c, seed, gen):
    """P random placements of exact capacity, the first of them contiguous."""
    base = torch.as_tensor(synth.contiguous_placement(c["E"], synth.capacities(c["E"], c["G"], -(-c["E"] // c["G"]))),
                           device="cuda")
    out = torch.empty((c["P"], c["L"], c["E"]), dtype=torch.uint8, device="cuda")
    for l in range(c["L"]):
        out[:, l] = base[torch.argsort(torch.rand((c["P"], c["E"]), generator=gen, device="cuda"), dim=1)]
    out[0] = base
    return out


def _secondaries(c, primary, generic, gen):
    """R random GPUs other than its primary for each replicated expert; 0xFF elsewhere."""
    if not c["R"]:
        return None
    P, L, E = primary.shape
    sec = torch.full((P, L, E, c["R"]), 0xFF, dtype=torch.uint8, device="cuda")
    at = torch.as_tensor(generic, device="cuda")  # [L][n_rep]
    for l in range(L):
        key = torch.rand((P, at.shape[1], c["G"]), generator=gen, device="cuda")
        key.scatter_(2, primary[:, l, at[l]].long().unsqueeze(2), 2.0)
        sec[:, l, at[l]] = torch.argsort(key, dim=2)[..., :c["R"]].to(torch.uint8)
    return sec


def _dispatches(trace, off, E):
    """int64 [F][L][E]"""
    F, L = len(off) - 1, trace.shape[0]
    out = torch.zeros((F, L, E), dtype=torch.int64, device=trace.device)
    for f in range(F):
        part = trace[:, int(off[f]):int(off[f + 1])].reshape(L, -1).long()
        out[f].scatter_add_(1, part, torch.ones((1, 1), dtype=torch.int64, device=part.device).expand_as(part))
    return out


def _counts(trace, off, E):
    """D int32 [F][L][E] and C int32 [F][L][E][E] (diagonal D), from products of one-hot rows (exact in float32)."""
    F, (L, _, k) = len(off) - 1, trace.shape
    C = torch.zeros((F, L, E, E), dtype=torch.int32, device=trace.device)
    for f in range(F):
        for l in range(L):
            for t in range(int(off[f]), int(off[f + 1]), 1 << 20):
                ids = trace[l, t:min(t + (1 << 20), int(off[f + 1]))].long()
                x = torch.zeros((ids.shape[0], E), dtype=torch.float32, device=ids.device).scatter_(1, ids, 1.0)
                C[f, l] += torch.mm(x.t().contiguous(), x).round().to(torch.int32)
    return torch.diagonal(C, dim1=2, dim2=3).contiguous(), C


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed + 7)
    s = dict(case=c)
    if c["kind"] in ("graph", "diagnose", "rank"):
        trace, off, _ = _trace(dict(c, N=c["n"] * c["F"], mix="uniform"), seed)
        s["D"], s["C"] = _counts(trace, off, c["E"])
        if c["kind"] == "rank":
            pooled = (s.pop("C").double() / c["n"]).mean(0)
            pooled.diagonal(dim1=1, dim2=2).zero_()
            s["a"] = (pooled / pooled.amax((1, 2), keepdim=True)).float()
            s["primary"] = _placements(c, seed, gen)
        return s
    s["trace"], s["off"], pl = _trace(c, seed)
    if c["kind"] == "count":
        return s
    s["home"] = synth.home_bands(c["F"], c["G"])
    s["primary"] = _placements(c, seed, gen)
    s["secondary"] = _secondaries(c, s["primary"], pl.generic, gen)
    s["ref"] = None
    if c["R"]:
        d = _dispatches(s["trace"], s["off"], c["E"]).sum(0)  # [L][E]
        s["ref"] = torch.zeros((c["P"], c["L"], c["G"]), dtype=torch.int64, device="cuda")
        s["ref"].scatter_add_(2, s["primary"].long(), d.unsqueeze(0).expand(c["P"], -1, -1).contiguous())
    return s


# ---- one pass -----------------------------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    kind, E = c["kind"], c["E"]
    if kind == "count":
        D, C, err = tacg.coact_build(s["trace"], s["off"], E)
        return dict(D=D, C=C, err=err)
    if kind == "graph":
        pref, tilde, hat = tacg.reweight(s["D"], s["C"], c["k"], alpha=0.25, want_hat=True)
        return dict(pref=pref, tilde=tilde, hat=hat)
    if kind == "diagnose":
        cent, cons, spec = tacg.gesr_scores(s["D"], s["C"], c["k"])
        pairs, jac = tacg.pair_jaccard(s["C"], c["top"])
        return dict(cent=cent, cons=cons, spec=spec, dist=tacg.activation_distance(s["D"], c["k"]), pairs=pairs, jac=jac)
    if kind == "rank":
        return dict(load=tacg.placement_load(s["D"], s["primary"], c["G"]),
                    obj=tacg.group_objective(s["a"], s["primary"], c["G"]))
    args = (s["trace"], s["off"], E, s["home"][0], s["home"][1], c["G"], s["primary"], s["secondary"])
    if kind == "stats":
        return tacg.eval_trace_stats(*args, s["ref"], theta=THETA)
    if kind == "online":
        return tacg.eval_online(*args, rho=RHO, theta=THETA)
    out = tacg.eval_placements(*args, s["ref"], theta=THETA)
    out["jain"], out["maxvio"] = tacg.jain_index(out["load"])
    return out


def work(case):
    """Bytes: inputs once, outputs once.  Operations: for counting an add per pair of a token-layer's experts, for
    scoring an OR per expert, the difference with the anchor and two population counts, for the decayed loads a
    multiply-add and an addition per GPU too; for the rest the arithmetic of the formulas."""
    c = case
    E, k, L, F = (c[x] for x in ("E", "k", "L", "F"))
    if c["kind"] == "count":
        return dict(bytes=2 * c["N"] * L * k + 4 * F * L * E * (E + 1), flops=c["N"] * L * (k + k * (k - 1) // 2))
    if c["kind"] == "graph":
        return dict(bytes=4 * F * L * E * (E + 1) + 4 * L * E * F + 8 * L * E * E, flops=L * E * E * (4 * F + 5))
    if c["kind"] == "diagnose":
        return dict(bytes=4 * F * L * E * (E + 1) + 24 * L * E + 8 * F * F + 4 * F * L * c["top"] + 8 * L * F * F,
                    flops=F * L * E * E * 10)
    if c["kind"] == "rank":
        P, G = c["P"], c["G"]
        return dict(bytes=4 * F * L * E + P * L * E + 4 * L * E * E + 8 * P * L * (G + 1),
                    flops=P * L * E * (2 + max(0, -(-E // G) - 1)))
    P, G = c["P"], c["G"]
    ptl = P * c["N"] * L
    size = 2 * c["N"] * L * k + P * L * E * (1 + c["R"]) + (8 * P * L * G if c["R"] else 0) + 4 * P * L * G + 16 * P
    if c["kind"] == "online":
        return dict(bytes=size + 8 * P * F + 8 * P * L * G, flops=ptl * (k + 2 + 3 * G))
    return dict(bytes=size + (24 if c["kind"] == "stats" else 8) * P * F, flops=ptl * (k + 2))


def tolerance(case):
    # Counts, costs and loads are whole numbers.  The decayed loads are defined with one rounding a step in trace
    # order, and the statistics have no floating output.
    if case["kind"] in ("count", "stats", "online"):
        return "exact"
    # float32 values of 64-bit arithmetic: another order of the sums moves the last bit of a few of them
    if case["kind"] in ("graph", "score"):
        return {"rel": 1.5e-7, "max": 1e-6}
    return {"rel": 1e-12, "max": 1e-10}  # 64-bit sums


# ---- the same values from plain torch -------------------------------------------------------------

def exact(case, seed):
    c = case
    if c["kind"] == "online" or c["kind"] in ("score", "stats") and c["P"] * c["N"] * c["L"] > EXACT_WORK:
        return None
    s = prepare(case, seed)
    zero = torch.zeros(1, dtype=torch.int32, device="cuda")
    if c["kind"] == "count":
        D, C = _counts(s["trace"], s["off"], c["E"])
        return dict(D=D, C=C, err=zero)
    if c["kind"] == "graph":
        return _exact_graph(s["D"], s["C"], c["k"])
    if c["kind"] == "diagnose":
        return _exact_diagnose(s["D"], s["C"], c["k"], c["top"])
    if c["kind"] == "rank":
        return _exact_rank(s["D"], s["a"], s["primary"], c["G"])
    return _exact_score(s)


def _rows(D, C, k):
    """Per-family frequencies: usage [F][L][E] and A [F][L][E][E] with a zero diagonal."""
    n = D.double().sum(2) / k
    A = C.double() / n[:, :, None, None]
    A.diagonal(dim1=2, dim2=3).zero_()
    return D.double() / (n * k)[:, :, None], A


def _exact_graph(D, C, k, alpha=0.25, tau=1.0, eps=1e-8):
    u, A = _rows(D, C, k)
    F = D.shape[0]
    z = 0
    for x in (u, A.sum(3)):
        d = x - (x.sum(0, keepdim=True) - x) / (F - 1)
        z = z + (d - d.mean(2, keepdim=True)) / (d.std(2, keepdim=True, unbiased=False) + eps)
    pref = torch.softmax(z / tau, dim=0).permute(1, 2, 0).contiguous()
    bar = A.mean(0)
    hat = bar / bar.amax((1, 2), keepdim=True)
    task = pref @ pref.transpose(1, 2).contiguous()
    return dict(pref=pref, tilde=(1 - alpha) * hat + alpha * task * hat, hat=hat)


def _exact_diagnose(D, C, k, top):
    F, L, E = D.shape
    u, A = _rows(D, C, k)
    bar = A.mean(0)
    norm = A.norm(dim=3) * bar.norm(dim=2)
    cos = torch.where(norm > 0, (A * bar).sum(3) / norm, torch.zeros_like(norm))
    spec = (A - bar).norm(dim=3).amax(0)
    p = (u * k).reshape(F, -1)
    dist = torch.stack([(p - p[i]).norm(dim=1) for i in range(F)])
    a, b = torch.triu_indices(E, E, 1, device=D.device)
    tri = C[:, :, a, b]
    n = min(top, a.numel())
    order = torch.sort(tri, dim=2, descending=True, stable=True)
    keep, at = order.values[..., :n] > 0, order.indices[..., :n]
    big = E * E
    ids = torch.sort(torch.where(keep, (a * E + b)[at], torch.full_like(at, big)), dim=2).values
    pairs = torch.full((F, L, top), -1, dtype=torch.int32, device=D.device)
    pairs[..., :n] = torch.where(ids < big, ids, torch.full_like(ids, -1)).to(torch.int32)
    member = torch.zeros((F, L, a.numel()), dtype=torch.float64, device=D.device).scatter_(2, at, keep.double())
    member = member.transpose(0, 1).contiguous()  # [L][F][pairs]
    inter = member @ member.transpose(1, 2).contiguous()
    size = member.sum(2)
    union = size[:, :, None] + size[:, None, :] - inter
    jac = torch.where(union > 0, inter / union.clamp_min(1), torch.ones_like(union))
    return dict(cent=bar.sum(2), cons=cos.mean(0), spec=spec, dist=dist, pairs=pairs, jac=jac)


def _exact_rank(D, a, primary, G):
    P, L, E = primary.shape
    d = D.long().sum(0)
    load = torch.zeros((P, L, G), dtype=torch.int64, device=D.device)
    load.scatter_add_(2, primary.long(), d.unsqueeze(0).expand(P, -1, -1).contiguous())
    obj = torch.empty((P, L), dtype=torch.float64, device=D.device)
    gpus = torch.arange(G, device=D.device)
    for l in range(L):
        w = a[l].double()
        w.fill_diagonal_(0.0)
        for p in range(0, P, 256):
            x = (primary[p:p + 256, l, :, None] == gpus).double()
            obj[p:p + 256, l] = (x * torch.matmul(w, x)).sum((1, 2))
    return dict(load=load, obj=obj)


def _bits(m):
    """Population count of int64 values below 2^32."""
    m = m - ((m >> 1) & 0x55555555)
    m = (m & 0x33333333) + ((m >> 2) & 0x33333333)
    m = (m + (m >> 4)) & 0x0F0F0F0F
    return ((m * 0x01010101) & 0xFFFFFFFF) >> 24


def _exact_score(s):
    """The serving rule of eval_placements, token by token in integers."""
    c = s["case"]
    P, L, N, k, F, G, E = (c[x] for x in ("P", "L", "N", "k", "F", "G", "E"))
    dev, off = "cuda", s["off"]
    start, size = s["home"]
    fam = torch.as_tensor(np.repeat(np.arange(F), np.diff(off)), device=dev)
    t = torch.arange(N, device=dev) - torch.as_tensor(off[:-1], device=dev)[fam]
    hs, hz = torch.as_tensor(start, device=dev).long(), torch.as_tensor(size, device=dev).long()
    anchor = hs[fam] + t % hz[fam]
    band = ((torch.ones_like(hs) << hz) - 1) << hs  # [F] GPUs of each family's band
    bands = torch.unique(band)
    cost = {n: torch.zeros((P, F), dtype=torch.int64, device=dev) for n in ("home", "span", "cross", "mass")}
    load = torch.zeros((P, L, G), dtype=torch.int64, device=dev)
    step = max(1, int(2e7 // (N * k)))
    for l in range(L):
        ids = s["trace"][l].long()
        for p in range(0, P, step):
            prim = s["primary"][p:p + step, l].long()
            n = prim.shape[0]
            cand = torch.ones_like(prim) << prim
            best, many = prim, torch.zeros_like(prim, dtype=torch.bool)
            if c["R"]:
                sec = s["secondary"][p:p + step, l].long()
                cand = cand | torch.where(sec < G, torch.ones_like(sec) << sec.clamp_max(G), torch.zeros_like(sec)).sum(2)
                many = _bits(cand) > 1
                ref = s["ref"][p:p + step, l]
                ok = THETA[1] * G * ref <= (THETA[0] + THETA[1]) * ref.sum(1, keepdim=True)
                feas = (ok.long() << torch.arange(G, device=dev)).sum(1, keepdim=True)
                cand = torch.where(cand & feas != 0, cand & feas, cand)
                member = (cand.unsqueeze(2) >> torch.arange(G, device=dev)) & 1
                best = torch.argmin(torch.where(member == 1, ref.unsqueeze(1), torch.full_like(member, 1 << 62)), dim=2)
            flat = ids.reshape(1, -1).expand(n, -1)
            pick = lambda table: table.gather(1, flat).reshape(n, N, k)  # noqa: E731
            gpu, single = pick(prim), ~pick(many.long()).bool()
            cards = torch.zeros((n, N), dtype=torch.int64, device=dev)
            for q in range(k):
                cards |= torch.where(single[:, :, q], torch.ones_like(cards) << gpu[:, :, q], torch.zeros_like(cards))
            if c["R"]:
                fc, fall = pick(cand), pick(best)
                for q in range(k):
                    x = fc[:, :, q] & cards
                    low = _bits((x & -x) - 1)
                    alt = torch.where((fc[:, :, q] >> anchor) & 1 == 1, anchor.expand(n, -1), fall[:, :, q])
                    g = torch.where(single[:, :, q], gpu[:, :, q], torch.where(x != 0, low & 31, alt))
                    gpu[:, :, q] = g
                    cards |= torch.ones_like(cards) << g
            load[p:p + step, l].scatter_add_(1, gpu.reshape(n, -1), torch.ones((1, 1), dtype=torch.int64, device=dev)
                                             .expand(n, N * k))
            spans = sum(((cards.unsqueeze(0) & b) != 0).long().squeeze(0) for b in bands) > 1
            inside = ((band[fam].unsqueeze(1) >> gpu) & 1).sum(2)
            per = dict(home=_bits(cards & ~(torch.ones_like(anchor) << anchor)), span=_bits(cards) - 1, cross=spans.long(),
                       mass=inside)
            for name, v in per.items():
                cost[name][p:p + step].scatter_add_(1, fam.expand(n, -1), v)
    out = dict(cost_home=cost["home"].sum(1), cost_span=cost["span"].sum(1), load=load.to(torch.int32),
               err=torch.zeros(1, dtype=torch.int32, device=dev))
    if c["kind"] == "stats":
        return dict(out, span_fam=cost["span"], cross_fam=cost["cross"], home_mass_fam=cost["mass"])
    x = load.sum(1).double()
    mean = x.mean(1)
    return dict(out, cost_home_fam=cost["home"], jain=x.sum(1) ** 2 / (G * (x * x).sum(1)), maxvio=x.amax(1) / mean - 1)
