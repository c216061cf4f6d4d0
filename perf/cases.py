"""What users of this library have it do, as timed cases.

Every case goes through the public binding: a KV pool, a prefix table and a
batch become a plan, and ``pfx_step`` runs one step of one layer (the append
of the new tokens and attention for every query row); prefixes move between
a host store and the pool through ``movement.Mover``.

A case is one batch recipe.  ``agents`` prefixes of log-uniform length in
[prefix_lo, prefix_hi]; ``decode`` requests of one new token each and
``extend`` requests whose ``rows`` last tokens are new (0: all of them),
suffix lengths uniform in [suffix_lo, suffix_hi] (decode) and
[extend_lo, extend_hi] (extend).  Requests go to the agents in turn, or by
Zipf(1.1) (``zipf``).  ``lens`` seeds the lengths, so that they belong to the
case; values and page placement come from the seed given to ``prepare``.
Values are N(0, 1) in bf16, as after a model's normalisations; pages are
scattered over the pool, as an allocator leaves them after a while.
"""

import math
import random

import numpy as np
import torch

from paper_2608_25523_amd import binding as B
from paper_2608_25523_amd import movement as M

PAGE = 16
DEFAULTS = dict(kind="step", layers=1, replan=False, hq=32, hkv=8, d=128, agents=1, prefix_lo=2048, prefix_hi=2048,
                decode=0, suffix_lo=1, suffix_hi=1, extend=0, extend_lo=1, extend_hi=1, rows=0, zipf=False, lens=0)


def _case(name=None, **kw):
    c = dict(DEFAULTS, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest steps: four requests over one short prefix in a small
        # model's layer, a decode step and the prefill before it.
        _case("tiny-decode", hq=8, hkv=2, d=64, prefix_lo=128, prefix_hi=128, decode=4, suffix_lo=33, suffix_hi=48),
        _case("tiny-extend", hq=8, hkv=2, d=64, prefix_lo=128, prefix_hi=128, extend=4, extend_lo=32, extend_hi=32),
        # One running request: an agent workflow in its sequential stage.
        _case("decode-one", decode=1, suffix_lo=288, suffix_hi=288),
        # One decode step of a whole 32-layer model for 16 requests of three
        # agents: the lengths grew, so the step is planned anew, then run on
        # every layer's pool.
        _case("model-decode-16", layers=32, replan=True, agents=3, prefix_lo=700, prefix_hi=3000, decode=16,
              suffix_lo=40, suffix_hi=600),
        # A full decode batch: 4 agents, 16 requests each.
        _case("decode-64", agents=4, decode=64, suffix_lo=64, suffix_hi=512, lens=2),
        # Ragged prefixes and skewed agents.
        _case("decode-hetero", agents=16, prefix_lo=512, prefix_hi=8192, decode=256, suffix_lo=32, suffix_hi=1024,
              zipf=True, lens=4),
        # The large decode batch at 64 query heads.
        _case("decode-448", hq=64, agents=8, prefix_lo=8192, prefix_hi=8192, decode=448, suffix_lo=64,
              suffix_hi=2048, lens=5),
        # A request is admitted: its prompt over its agent's prefix (the
        # engine prefills admitted requests one by one), short and long, at
        # both head sizes.
        _case("prefill-300", prefix_lo=4096, prefix_hi=4096, extend=1, extend_lo=300, extend_hi=300),
        _case("prefill-1999-d64", d=64, extend=1, extend_lo=1999, extend_hi=1999),
        # Many admissions at once.
        _case("extend-32", agents=3, prefix_lo=4096, prefix_hi=4096, extend=32, extend_lo=256, extend_hi=2048, lens=3),
        # The largest batch, prefills beside decodes.
        _case("mixed-480", hq=64, agents=8, prefix_lo=8192, prefix_hi=8192, decode=448, suffix_lo=64, suffix_hi=2048,
              extend=32, extend_lo=512, extend_hi=4096, lens=5),
        # An agent enters the resident set: its prefix comes from the host.
        _case("load-prefix", kind="load"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["decode", "decode", "decode", "extend", "extend", "extend", "mixed", "load"])
        hq, hkv, d = rng.choice([(8, 2, 64), (32, 8, 64), (32, 8, 128), (32, 8, 128), (64, 8, 128), (16, 16, 128),
                                 (32, 2, 128)])
        lo = _log_int(rng, 100, 8192)
        c = _case(hq=hq, hkv=hkv, d=d, agents=rng.randint(1, 8), prefix_lo=lo, prefix_hi=min(8192, lo * rng.randint(1, 4)),
                  lens=rng.randint(0, 1 << 20))
        if kind == "load":
            c.update(kind="load", agents=1)
            c["prefix_hi"] = c["prefix_lo"]
        if kind in ("decode", "mixed"):
            s = _log_int(rng, 1, 1024)
            c.update(decode=_log_int(rng, 1, 448), suffix_lo=s, suffix_hi=min(2048, s * rng.randint(1, 8)),
                     zipf=rng.random() < 0.3)
        if kind in ("extend", "mixed"):
            s = _log_int(rng, 32, 2048)
            c.update(extend=_log_int(rng, 1, 32), extend_lo=s, extend_hi=min(4096, s * rng.randint(1, 4)),
                     rows=rng.choice([0, 0, 0, _log_int(rng, 17, 512)]))
        w = work(c)
        if w["flops"] <= 5e12 and w["bytes"] <= 3e9:
            return c


# --------------------------------------------------------------------------- the batch of a case

def _pages(n):
    return (n + PAGE - 1) // PAGE


class _Batch:
    """Lengths and rows of a case (no values)."""

    def __init__(self, c):
        rng = random.Random(1000 + c["lens"])
        lo, hi = c["prefix_lo"], c["prefix_hi"]
        self.prefix = [int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))) if hi > lo else lo
                       for _ in range(c["agents"])]
        self.prefix = [min(max(p, lo), hi) for p in self.prefix]
        n = c["decode"] + c["extend"]
        if c["zipf"]:
            self.agent = rng.choices(range(c["agents"]), weights=[1.0 / (k + 1) ** 1.1 for k in range(c["agents"])], k=n)
        else:
            self.agent = [i % c["agents"] for i in range(n)]
        ext = [rng.randint(c["extend_lo"], c["extend_hi"]) for _ in range(c["extend"])]
        dec = [rng.randint(c["suffix_lo"], c["suffix_hi"]) for _ in range(c["decode"])]
        self.suffix = ext + dec
        self.rows = [min(s, c["rows"]) if c["rows"] else s for s in ext] + [1] * len(dec)
        self.need = sum(map(_pages, self.prefix)) + sum(map(_pages, self.suffix))
        self.num_pages = self.need + self.need // 4 + 8


def _csr(lists):
    ptr = np.zeros(len(lists) + 1, np.int32)
    ptr[1:] = np.cumsum([len(x) for x in lists])
    return ptr, (np.concatenate(lists) if lists else np.zeros(0)).astype(np.int32)


def _place(b, seed):
    order = np.random.Generator(np.random.PCG64(seed)).permutation(b.num_pages).astype(np.int32)
    cut = np.cumsum([_pages(n) for n in b.prefix + b.suffix])
    parts = np.split(order[:b.need], cut[:-1])
    return parts[:len(b.prefix)], parts[len(b.prefix):]


def _values(c, b, seed):
    """(k_pool, v_pool, q, k_new, v_new): pools [layers][pages][Hkv][16][d], rows [layers][tokens][heads][d]."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def randn(*shape):
        return torch.randn((c["layers"],) + shape, dtype=torch.bfloat16, device="cuda", generator=g)

    pool = (b.num_pages, c["hkv"], PAGE, c["d"])
    t = sum(b.rows)
    return (randn(*pool), randn(*pool), randn(t, c["hq"], c["d"]), randn(t, c["hkv"], c["d"]),
            randn(t, c["hkv"], c["d"]))


class _State:
    pass


def prepare(case, seed):
    c, b, s = case, _Batch(case), _State()
    s.c = c
    if c["kind"] == "load":
        n, shape = _pages(b.prefix[0]), (c["hkv"], PAGE, c["d"])
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        s.store = M.HostStore(n, c["hkv"], c["d"])
        for t in (s.store.k, s.store.v):
            t.copy_(torch.randn((n,) + shape, dtype=torch.bfloat16, device="cuda", generator=g))
        s.k = torch.zeros((b.num_pages,) + shape, dtype=torch.bfloat16, device="cuda")
        s.v = torch.zeros_like(s.k)
        s.mover = M.Mover(B.make_pool(b.num_pages, c["hkv"], c["d"], s.k, s.v), s.store, n)
        s.pages = _place(b, seed)[0][0]
        s.slots = s.store.alloc.alloc(n)
        return s
    pp, sp = _place(b, seed)
    s.k, s.v, s.q, s.kn, s.vn = _values(c, b, seed)
    s.o = torch.empty_like(s.q)
    s.lse = torch.empty(s.q.shape[:3], dtype=torch.float32, device="cuda")
    s.pools = [B.make_pool(b.num_pages, c["hkv"], c["d"], s.k[i], s.v[i]) for i in range(c["layers"])]
    # The arguments of a layer's call, made once by a program that keeps its buffers.
    s.calls = [(s.pools[i], s.kn[i], s.vn[i], s.q[i], s.o[i], s.lse[i]) for i in range(c["layers"])]
    mode = B.PFX_MODE_DECODE if not c["extend"] else B.PFX_MODE_MIXED if c["decode"] else B.PFX_MODE_EXTEND
    pptr, pids = _csr(pp)
    sptr, sids = _csr(sp)
    qptr = np.concatenate([[0], np.cumsum(b.rows)]).astype(np.int32)
    s.tables = (pptr, pids, np.asarray(b.prefix, np.int32), np.asarray(b.agent, np.int32), sptr, sids,
                np.asarray(b.suffix, np.int32), qptr, c["hq"], mode)
    s.plan = B.pfx_plan_create(s.pools[0], *s.tables).upload()
    return s


def run(s):
    c = s.c
    if c["kind"] == "load":
        s.mover.load(s.pages, s.slots)
        return s.k, s.v
    plan = s.plan
    if c["replan"]:
        plan = B.pfx_plan_create(s.pools[0], *s.tables).upload(workspace=s.plan.workspace)
    for pool, kn, vn, q, o, lse in s.calls:
        B.pfx_step(pool, plan, kn, vn, q, o, lse)
    return s.o, s.lse, s.k, s.v


def work(case):
    """K and V of every referenced prefix once and of every suffix once, the
    new rows, Q and O; causal-exact products."""
    c, b = case, _Batch(case)
    token = 4 * c["hkv"] * c["d"]
    if c["kind"] == "load":
        return {"bytes": 2 * token * b.prefix[0], "flops": 0}
    t = sum(b.rows)
    kv = sum(b.prefix[a] for a in set(b.agent)) + sum(b.suffix)
    visible = sum(n * (b.prefix[a] + s - n) + n * (n + 1) // 2 for a, s, n in zip(b.agent, b.suffix, b.rows))
    return {"bytes": c["layers"] * (token * (kv + t) + t * c["hq"] * (4 * c["d"] + 4)),
            "flops": c["layers"] * 4 * c["d"] * c["hq"] * visible}


def tolerance(case):
    if case["kind"] == "load":
        return "exact"
    return {"rel": 1.2e-2, "max": 0.3}


def exact(case, seed):
    """Attention by its definition in float64, request by request."""
    c, b = case, _Batch(case)
    if c["kind"] == "load":
        return None
    hq, hkv, d = c["hq"], c["hkv"], c["d"]
    G = hq // hkv
    pp, sp = _place(b, seed)
    k_pool, v_pool, q, kn, vn = _values(c, b, seed)
    o = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    lse = torch.empty(q.shape[:3], dtype=torch.float64, device="cuda")
    for layer in range(c["layers"]):
        at = 0
        for a, sp_r, L, n in zip(b.agent, sp, b.suffix, b.rows):
            def keys(pool, new):
                def tokens(pages, count):
                    x = pool[layer][torch.from_numpy(pages.astype(np.int64)).cuda()]
                    return x.transpose(1, 2).reshape(-1, hkv, d)[:count]
                x = torch.cat([tokens(pp[a], b.prefix[a]), tokens(sp_r, L - n), new[layer, at:at + n]])
                return x.double().transpose(0, 1).contiguous()
            K, V = keys(k_pool, kn), keys(v_pool, vn)
            K = K.transpose(1, 2).contiguous()
            total = K.shape[2]
            step = max(1, int(2e8 // (hq * total)))
            for i in range(0, n, step):
                m = min(step, n - i)
                x = q[layer, at + i:at + i + m].double().reshape(m, hkv, G, d).transpose(0, 1).reshape(hkv, m * G, d)
                sc = torch.bmm(x.contiguous(), K) / math.sqrt(d)
                if n > 1:
                    last = total - n + i + torch.arange(m, device="cuda")
                    hide = torch.arange(total, device="cuda")[None] > last[:, None]
                    sc.view(hkv, m, G, total).masked_fill_(hide[None, :, None], -math.inf)
                z = torch.logsumexp(sc, 2, keepdim=True)
                out = torch.bmm(sc.sub_(z).exp_(), V)
                o[layer, at + i:at + i + m] = out.view(hkv, m, G, d).transpose(0, 1).reshape(m, hq, d)
                lse[layer, at + i:at + i + m] = z.view(hkv, m, G).transpose(0, 1).reshape(m, hq)
            at += n
    return o, lse, None, None
