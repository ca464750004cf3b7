"""Measured cases of the memory-retrieval library: what an agent that keeps a value-driven memory has it do.

A case is one call, or the few calls that belong together in one step of the agent's loop, through the
MemoryBank binding (one thin layer over the C ABI).  Kinds:

  step     one iteration of the loop: append `new` entries (0: none), retrieve for `B` queries, fold rewards
           into the values of the returned entries (`zipf` > 0: of that many ids with heavy duplication instead)
  masked   typed retrieval: every query accepts some entry types and leaves one group of entries out
  eps      epsilon-greedy retrieval (the exploration policy of the drafting and refining stages)
  exact    retrieval by exhaustive selection, for queries whose pool has to be exact whatever the bank holds
  ingest   bulk append into an empty bank
  values   verifier outcomes -> normalised rewards -> value update -> start point of every task

Rows and queries are L2-normalised Gaussians, or (`clustered`) centre + 0.3 N(0,1) with queries near the
centres, which gives the narrow similarity bands that near-duplicate entries have.  Everything is drawn on
the GPU from the seed alone.
"""
import math

import numpy as np
import torch

from paper_2603_10846_amd.binding import MemoryBank

DEV = "cuda:0"
CHUNK = 65536                       # rows generated and appended at a time
TORCH_TYPE = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
BYTES = {"f32": 4, "bf16": 2, "f16": 2}
ALPHA = 0.1                         # step size of the value update
SIGMA_MIN, CLIP = 0.1, 3.0          # reward normalisation
N_TYPES = 4                         # entry types of a masked bank (tag & 0xff); groups = tag >> 8
N_GROUPS = 250
NO_GROUP = 0xFFFFFFFF


def _case(name, kind, dtype, N, d, B=0, k1=0, k2=0, lam=0.5, stage=0, clustered=False, new=0, zipf=0, M=0, sets=0, members=0, eps=0.0):
    c = dict(kind=kind, dtype=dtype, N=N, d=d, B=B, k1=k1, k2=k2, lam=lam, stage=stage, clustered=clustered, new=new, zipf=zipf,
             M=M, sets=sets, members=members, eps=eps)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a young memory and one query: the latency of a single agent's lookup
        _case("tiny_f32_b1", "step", "f32", 4096, 768, B=1, k1=32, k2=4),
        # a mid-size fp32 memory shared by 64 agents
        _case("mid_f32_b64", "step", "f32", 65536, 1024, B=64, k1=64, k2=8, stage=1),
        # one agent on a memory of a million near-duplicate-rich entries: the bandwidth-bound lookup
        _case("clustered_bf16_b1", "step", "bf16", 1048576, 1024, B=1, k1=128, k2=16, clustered=True),
        # the benchmark's step: 256 agents append, retrieve and update
        _case("clustered_bf16_b256", "step", "bf16", 1048576, 1024, B=256, k1=128, k2=16, clustered=True, new=256),
        # the largest batch on the largest bank in common use, then an update that names few entries very often
        _case("large_bf16_b1024", "step", "bf16", 4194304, 1536, B=1024, k1=128, k2=16, stage=1, zipf=16384),
        # a growing memory of long fp16 embeddings: a chunk of new entries, retrieval with a wide pool, update
        _case("stream_f16_b128", "step", "f16", 1048576, 4096, B=128, k1=256, k2=32, lam=0.7, new=65536),
        # sizes that fit no tile: few queries, odd bank, a dimension that is padded
        _case("ragged_f16_b7", "step", "f16", 30011, 200, B=7, k1=50, k2=5, lam=0.3, stage=1),
        # lookup restricted by entry type, held-out operators left out
        _case("masked_f16_b32", "masked", "f16", 300007, 384, B=32, k1=64, k2=8),
        # the pool-size study's widest over-retrieval (30 x 32), filled epsilon-greedily
        _case("pool960_bf16_b64", "eps", "bf16", 262144, 1024, B=64, k1=960, k2=32, lam=1.0, eps=0.1),
        # the always-exact answer for a handful of flagged queries
        _case("exact_bf16_b4", "exact", "bf16", 1048576, 1024, B=4, k1=128, k2=16, clustered=True),
        # building a bank: bulk append
        _case("ingest_f32", "ingest", "f32", 65536, 1024),
        # a round of verifier outcomes: rewards, update, start points
        _case("values_m8192", "values", "f32", 65536, 64, M=8192, sets=256, members=64, stage=1, eps=0.1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "masked", "eps", "exact", "ingest", "values"])
    dtype = rng.choice(["f32", "bf16", "f16"])
    d = 8 * _log(rng, 8, 512)                                   # 64 .. 4096, seldom a multiple of 64
    if kind == "values":
        M = _log(rng, 4, 20000)
        return _case(None, kind, dtype, _log(rng, 1000, 200000), 64, M=M, sets=_log(rng, 1, 2000), members=_log(rng, 2, 500),
                     stage=rng.randrange(2), eps=rng.choice([0.0, 0.1]))
    N = _log(rng, 1000, min(1200000, 1500000000 // d))
    if kind == "ingest":
        return _case(None, kind, dtype, min(N, 300000000 // d), d)
    B = _log(rng, 1, 16) if kind == "exact" else _log(rng, 1, 1024)
    if kind == "exact":
        N = min(N, 400000000 // d)
    B = max(1, min(B, int(1.5e12 / N / d)))
    k1 = _log(rng, 257, 2048) if kind == "eps" and rng.random() < 0.5 else _log(rng, 8, 256)
    k2 = min(_log(rng, 2, 32), k1)
    lam = round(rng.random(), 2)
    new = rng.choice([0, 0, B, _log(rng, 100, 20000)]) if kind == "step" else 0
    zipf = _log(rng, 1000, 16384) if kind == "step" and rng.random() < 0.2 else 0
    return _case(None, kind, dtype, N, d, B=B, k1=k1, k2=k2, lam=lam, stage=rng.randrange(2), clustered=rng.random() < 0.4, new=new,
                 zipf=zipf, eps=0.1 if kind == "eps" else 0.0)


# ----------------------------------------------------------------------------- inputs, from the seed alone

def _gen(seed, what, part=0):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + what * 4099 + part) % (1 << 62))


def _centres(c, seed):
    return torch.randn((min(256, max(1, c["N"] // 64)), c["d"]), device=DEV, generator=_gen(seed, 1)) if c["clustered"] else None


def _vectors(g, n, d, centres, noise):
    x = torch.randn((n, d), device=DEV, generator=g)
    if centres is not None:
        which = torch.randint(0, centres.shape[0], (n,), device=DEV, generator=g)
        x = x.mul_(noise).add_(centres[which])
    return x.div_(torch.linalg.vector_norm(x, dim=1, keepdim=True))


def _row_chunks(c, seed):
    """(first id, fp32 rows) of the bank before the pass, a chunk at a time."""
    centres = _centres(c, seed)
    for j, a in enumerate(range(0, c["N"], CHUNK)):
        yield a, _vectors(_gen(seed, 2, j), min(CHUNK, c["N"] - a), c["d"], centres, 0.3)


def _inputs(c, seed):
    g, kind = _gen(seed, 3), c["kind"]
    s = {"q0": torch.randn((2, c["N"] + c["new"]), device=DEV, generator=g).mul_(0.5).clamp_(-1.0, 1.0)}
    if c["new"]:
        s["new"] = _vectors(_gen(seed, 4), c["new"], c["d"], _centres(c, seed), 0.3)
    if c["B"]:
        s["queries"] = _vectors(_gen(seed, 5), c["B"], c["d"], _centres(c, seed), 0.1)
        s["rewards"] = (torch.rand(c["B"] * c["k2"], device=DEV, generator=g) < 0.3).float()
    if c["zipf"]:                                               # Zipf(1.1) ranks through an affine map of the ids
        u = torch.rand(c["zipf"], device=DEV, generator=g, dtype=torch.float64)
        cdf = torch.arange(1, c["N"] + 1, device=DEV, dtype=torch.float64).pow_(-1.1).cumsum_(0)
        ranks = torch.searchsorted(cdf / cdf[-1], u).clamp_(max=c["N"] - 1)
        s["zipf_ids"] = ((ranks * 2654435761 + 12345) % c["N"]).int()
        s["rewards"] = torch.rand(c["zipf"], device=DEV, generator=g)
    if kind == "masked":
        s["types"] = torch.randint(0, N_TYPES, (c["N"],), device=DEV, generator=g)
        s["groups"] = torch.randint(0, N_GROUPS, (c["N"],), device=DEV, generator=g)
        s["allow"] = torch.randint(1, 1 << N_TYPES, (c["B"],), device=DEV, generator=g)
        s["exclude"] = torch.randint(0, N_GROUPS, (c["B"],), device=DEV, generator=g)
        s["exclude"][::3] = NO_GROUP
    if kind == "values":
        M, G = c["M"], c["sets"]
        s["ids"] = torch.randint(0, c["N"], (M,), device=DEV, generator=g).int()
        s["feasible"] = (torch.rand(M, device=DEV, generator=g) < 0.7).to(torch.uint8)
        s["latency"] = torch.rand(M, device=DEV, generator=g).add_(0.1)
        s["best"] = torch.rand(M, device=DEV, generator=g).mul_(0.5).add_(0.1)
        sizes = torch.randint(1, 2 * c["members"], (G,), device=DEV, generator=g)
        s["offsets"] = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), sizes.cumsum(0)])
        s["set_ids"] = torch.randint(0, c["N"], (int(s["offsets"][-1]),), device=DEV, generator=g).int()
    return s


def prepare(c, seed):
    s = _inputs(c, seed)
    s["case"] = c
    total = c["N"] + c["new"]
    bank = MemoryBank(c["d"], c["dtype"], total, max_B=max(c["B"], 1), max_k1=max(c["k1"], 1), device=DEV)
    s["bank"] = bank
    if c["kind"] == "ingest":
        bank.store.zero_()                                      # rows past the end are part of the returned buffer
        s["rows"] = torch.cat([x for _, x in _row_chunks(c, seed)])
        return s
    for a, x in _row_chunks(c, seed):
        bank.append(x, s["q0"][0, a:a + x.shape[0]].contiguous(), s["q0"][1, a:a + x.shape[0]].contiguous())
    if c["new"]:
        s["new_q"] = s["q0"][:, c["N"]:].contiguous()
    if c["kind"] == "masked":
        bank.set_tags(0, s["types"] | (s["groups"] << 8))
    if c["B"]:                                                  # result buffers that such a program keeps
        s["out"] = (torch.empty((c["B"], c["k2"]), dtype=torch.int32, device=DEV),
                    torch.empty((c["B"], c["k2"]), dtype=torch.float32, device=DEV), None, None)
    return s


def run(s):
    c, bank = s["case"], s["bank"]
    kind, stage = c["kind"], c["stage"]
    if kind == "step":
        if c["new"]:
            bank.lib.mem_restore(bank.h, c["N"])                # the bank as it was before the step's entries
            bank.append(s["new"], s["new_q"][0], s["new_q"][1])
        ids, scores, _, _ = bank.retrieve(s["queries"], stage, c["k1"], c["k2"], c["lam"], out=s["out"])
        bank.update_q(s["zipf_ids"] if c["zipf"] else ids.view(-1), stage, s["rewards"], ALPHA)
        return {"ids": ids, "scores": scores, "q": bank.q[stage]}
    if kind == "masked":
        ids, scores, cand, sims = bank.retrieve_masked(s["queries"], stage, c["k1"], c["k2"], c["lam"], s["allow"], s["exclude"],
                                                       want_candidates=True)
        return {"ids": ids, "scores": scores, "cand_ids": cand, "cand_sims": sims}
    if kind == "eps":
        ids, scores, cand, sims, explored = bank.retrieve_eps(s["queries"], stage, c["k1"], c["k2"], c["lam"], c["eps"], 1234, 5,
                                                              want_candidates=True)
        return {"ids": ids, "scores": scores, "cand_ids": cand, "cand_sims": sims, "explored": explored}
    if kind == "exact":
        ids, scores, cand, sims = bank.retrieve_exact(s["queries"], stage, c["k1"], c["k2"], c["lam"], want_candidates=True)
        return {"ids": ids, "scores": scores, "cand_ids": cand, "cand_sims": sims}
    if kind == "ingest":
        bank.lib.mem_restore(bank.h, 0)
        bank.append(s["rows"], s["q0"][0], s["q0"][1])
        return {"store": bank.store.view(torch.int32), "invnorm": bank.invnorm[:c["N"]], "q": bank.q}
    rewards = bank.shape_rewards(stage, s["feasible"], s["latency"], s["best"], normalise=True, sigma_min=SIGMA_MIN, clip=CLIP)
    bank.update_q(s["ids"], stage, rewards, ALPHA)
    ids, vals, explored = bank.select_by_q(s["set_ids"], s["offsets"], stage, c["eps"], 77, 3)
    return {"rewards": rewards, "q": bank.q[stage], "ids": ids, "values": vals, "explored": explored}


def work(c):
    """Every stored row that the pass needs once, inputs and outputs once."""
    e, d, total = BYTES[c["dtype"]], c["d"], c["N"] + c["new"]
    if c["kind"] == "ingest":
        return {"bytes": c["N"] * (d * (4 + e) + 4 + 4 * 4), "flops": 2 * c["N"] * d}
    if c["kind"] == "values":
        return {"bytes": c["M"] * (1 + 4 + 4 + 4 + 4 + 4 + 8) + c["sets"] * (c["members"] * 8 + 8 + 9), "flops": 30 * c["M"]}
    M = c["zipf"] or c["B"] * c["k2"]
    b = total * d * e + c["B"] * (d * 4 + c["k1"] * 8 + c["k2"] * 8) + c["new"] * (d * 4 + 8)
    if c["kind"] == "step":
        b += M * 16
    if c["kind"] == "masked":
        b += total * 4
    return {"bytes": b, "flops": 2 * c["B"] * total * d}


def tolerance(c):
    # Similarities are accumulated in fp64 and scores formed in fp64, both rounded to fp32 once (6e-8); the
    # z-scores divide by the pool's spread, and values fold through fp32 recurrences.  Which of two entries is
    # named can only differ where their fp64 values tie to the last bits.  Measured against exact(): 3e-8 on
    # scores, similarities, inverse norms and normalised rewards, 1e-8 on values.
    if c["kind"] == "ingest":
        return {"rel": 2e-7, "max": 1e-6}
    return {"rel": 2e-7, "max": 8e-6, "differ": 1e-4}


# ----------------------------------------------------------------------------- the same results in 64 bits

def _stored(c, x):
    return x.to(TORCH_TYPE[c["dtype"]]).double()


def _fold(q, ids, rewards):
    for i, r in zip(ids.tolist(), rewards.tolist()):
        q[i] += float(np.float32(ALPHA)) * (r - q[i])
    return q


def _recall(c, s, seed):
    """(similarities desc [B, k1], ids) over the bank as the retrieve of the pass sees it."""
    q = _stored(c, s["queries"])
    q = q / q.norm(dim=1, keepdim=True)
    best = ids = None

    def fold(a, x):
        nonlocal best, ids
        x = _stored(c, x)
        sim = q @ (x / x.norm(dim=1, keepdim=True)).t()
        if c["kind"] == "masked":
            t, grp = s["types"][a:a + x.shape[0]], s["groups"][a:a + x.shape[0]]
            ok = ((s["allow"][:, None] >> t[None]) & 1).bool() & (grp[None] != s["exclude"][:, None])
            sim = sim.masked_fill(~ok, -math.inf)
        v, i = sim.topk(min(c["k1"], sim.shape[1]), dim=1)
        i = i + a
        if best is not None:
            v, i = torch.cat([best, v], 1), torch.cat([ids, i], 1)
            v, o = v.topk(min(c["k1"], v.shape[1]), dim=1)
            i = i.gather(1, o)
        best, ids = v, i

    for a, x in _row_chunks(c, seed):
        fold(a, x)
    if c["new"]:
        for a in range(0, c["new"], CHUNK):
            fold(c["N"] + a, s["new"][a:a + CHUNK])
    return best, ids


def _value_filter(c, s, sims, ids):
    """(scores desc, ids) of the k2 best of every pool."""
    q = s["q0"][c["stage"]].double()[ids]
    live = sims > -math.inf
    n = live.sum(1, keepdim=True).clamp(min=1)

    def z(v):
        v = torch.where(live, v, torch.zeros_like(v))
        dv = torch.where(live, v - v.sum(1, keepdim=True) / n, torch.zeros_like(v))
        return dv / ((dv * dv).sum(1, keepdim=True).div(n).sqrt() + 1e-6)

    lam = float(np.float32(c["lam"]))
    score = torch.where(live, (1 - lam) * z(sims) + lam * z(q), torch.full_like(sims, -math.inf))
    v, o = score.topk(min(c["k2"], score.shape[1]), dim=1)
    return v, ids.gather(1, o)


def _padded(v, k):
    return torch.cat([v, torch.full((v.shape[0], k - v.shape[1]), -math.inf, dtype=v.dtype, device=v.device)], 1)


def exact(c, seed):
    s = _inputs(c, seed)
    kind, stage = c["kind"], c["stage"]
    if kind == "ingest":
        inv = torch.cat([1.0 / _stored(c, x).norm(dim=1) for _, x in _row_chunks(c, seed)])
        return {"store": None, "invnorm": inv, "q": s["q0"].double()}
    if kind == "values":
        raw = torch.tanh(torch.log(s["best"].double()) - torch.log(s["latency"].double())) if stage else torch.ones(c["M"], dtype=torch.float64, device=DEV)
        raw = torch.where(s["feasible"] != 0, raw, -torch.ones_like(raw)).cpu().numpy()
        n = np.arange(raw.size, dtype=np.float64)
        before, before2 = np.cumsum(raw) - raw, np.cumsum(raw * raw) - raw * raw
        mu = before / np.maximum(n, 1)
        sigma = np.sqrt(np.maximum(before2 / np.maximum(n, 1) - mu * mu, 0.0))
        sigma_min, clip = float(np.float32(SIGMA_MIN)), float(np.float32(CLIP))
        r = np.clip((raw - mu) / np.maximum(sigma, sigma_min), -clip, clip)
        q = _fold(s["q0"][stage].double().cpu().numpy(), s["ids"].cpu().numpy(), r)
        return {"rewards": r, "q": q, "ids": None, "values": None, "explored": None}
    sims, ids = _recall(c, s, seed)
    scores, top = _value_filter(c, s, sims, ids)
    scores, sims = _padded(scores, c["k2"]), _padded(sims, c["k1"])
    if kind == "step":
        if not c["zipf"] and top.shape[1] < c["k2"]:
            return {"ids": None, "scores": scores, "q": None}
        named = s["zipf_ids"] if c["zipf"] else top.reshape(-1)
        q = _fold(s["q0"][stage].double().cpu().numpy(), named.cpu().numpy(), s["rewards"].double().cpu().numpy())
        return {"ids": None, "scores": scores, "q": q}
    out = {"ids": None, "scores": None if kind == "eps" else scores, "cand_ids": None, "cand_sims": sims}
    return dict(out, explored=None) if kind == "eps" else out
