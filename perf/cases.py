"""The work that a user of this framework has it do, as cases that can be timed.

A case is a dict of plain values.  Five kinds of work:

  step    one draft step: (lexical drafts, on a second stream beside) top-k
          retrieval, gather of the continuations, root-first tree merge.
  query   top-k retrieval alone, every query with its own prompt excluded.
  ingest  finished traces enter a new store: raw verifier states are
          normalised (or quantised) into the key buffer.
  grow    a server's first requests: a new store takes one bulk append, then
          rounds of a few committed positions and one batch of queries.
  verify  what follows the verifier's forward: accept walk, the mask of the
          tree, rejected nodes into the session's ring, a lookup in the
          standing ring.

Inputs are seeded synthetic tool-calling traffic: 48-token calls copied from
templates with a few values minted per request; states cluster by call and
position; queries are stored states plus noise, a quarter of them (in batches)
random directions that retrieve nothing useful.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2608_03839_amd as oil

CALL = 48          # tokens per call (one trace = one prompt per call)
MINTED = 3         # of them minted per request
CTX = 16           # tokens of context for the lexical source
CHUNK = 32768      # rows generated at a time
THETA = 0.8


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest call: one request against a store that has just begun
        # (f32 states), all latency and launches
        dict(name="tiny_step", kind="step", n=4096, d=512, B=1, k=8, L=8, fmt="bf16", raw="f32", clusters=0,
             vocab=32000, lex=0, lex_len=0, lex_budget=0, sem_budget=32, hist=0, bands=False),
        # single-stream decode: one user, a store of some 1,400 calls
        dict(name="decode_64k", kind="step", n=65536, d=4096, B=1, k=16, L=16, fmt="bf16", raw="bf16", clusters=256,
             vocab=128256, lex=0, lex_len=0, lex_budget=0, sem_budget=64, hist=0, bands=False),
        # the paper's own configuration: one request, 320,000 positions, copy
        # depth by similarity band, three lexical branches beside
        dict(name="paper_320k", kind="step", n=320000, d=4096, B=1, k=8, L=48, fmt="bf16", raw="bf16", clusters=256,
             vocab=128256, lex=3, lex_len=32, lex_budget=44, sem_budget=16, hist=16384, bands=True),
        # the headline: a serving batch of 32 against 1M positions (a few
        # positions past 2^20, as a store that grows while it serves has)
        dict(name="batched_1m", kind="step", n=1048581, d=4096, B=32, k=32, L=8, fmt="bf16", raw="bf16",
             clusters=4096, vocab=128256, lex=0, lex_len=0, lex_budget=0, sem_budget=64, hist=0, bands=False),
        # the same against a quantised store, with a batch that is not full
        dict(name="batched_1m_fp8", kind="step", n=1000003, d=4096, B=27, k=32, L=8, fmt="fp8", raw="bf16",
             clusters=4096, vocab=128256, lex=0, lex_len=0, lex_budget=0, sem_budget=64, hist=0, bands=False),
        # the whole draft step of a large model at 64 requests, lexical drafts
        # over the store and each request's own history
        dict(name="full_step_8192", kind="step", n=524288, d=8192, B=64, k=32, L=12, fmt="bf16", raw="bf16",
             clusters=256, vocab=128256, lex=4, lex_len=12, lex_budget=48, sem_budget=16, hist=8192, bands=False),
        # a wide serving batch, ragged store and batch, own prompts excluded
        dict(name="wide_200", kind="query", n=400001, d=5120, B=200, k=16, fmt="bf16", raw="bf16", clusters=1024),
        # the widest batch the framework takes, on a quantised store
        dict(name="wide_512_fp8", kind="query", n=1048576, d=4096, B=512, k=32, fmt="fp8", raw="bf16", clusters=4096),
        # a day's traces loaded into a new store
        dict(name="ingest_bf16", kind="ingest", n=60001, d=4096, fmt="bf16", raw="bf16", clusters=256),
        # f32 states of a wider model into a quantised store
        dict(name="ingest_f32_fp8", kind="ingest", n=20011, d=5120, fmt="fp8", raw="f32", clusters=256),
        # a server's first requests: 8,000 positions, then four rounds of five
        # committed positions and 16 queries
        dict(name="grow_session", kind="grow", n=8000, d=4096, B=16, k=16, fmt="bf16", raw="bf16", clusters=64,
             rounds=4, add=5),
        # the step after the forward, 32 trees of up to 65 nodes
        dict(name="verify_32", kind="verify", n=65536, d=4096, B=32, k=32, L=8, raw="bf16", clusters=64,
             sem_budget=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "query", "query", "ingest", "ingest", "grow", "verify"])
    # widths of real models, and now and then one that is no multiple of anything
    d = rng.choice([512, 1024, 2048, 2880, 4096, 4096, 5120, 8192, rng.randrange(500, 4100)])
    raw = rng.choice(["bf16", "bf16", "bf16", "f32"])
    fmt = rng.choice(["bf16", "bf16", "fp8"])
    room = (1 << 32) // d  # elements of the largest listed store
    if kind == "step":
        n = _log(rng, 2000, min(1000000, room))
        lex = rng.choice([0, 0, 3, 4])
        lex_len = rng.choice([12, 32]) if lex else 0
        k = rng.choice([8, 16, 32, 48])
        L = rng.choice([8, 12, 16, 48])
        return dict(kind=kind, n=n, d=d, B=rng.choice([1, 1, 2, 3, 4, 5, 8, 16, 31, 32, 48, 64]), k=k, L=L, fmt=fmt,
                    raw=raw, clusters=max(1, n // CALL // rng.choice([5, 40])), vocab=128256, lex=lex,
                    lex_len=lex_len, lex_budget=(44 if lex else 0), sem_budget=rng.choice([16, 32, 64]),
                    hist=(_log(rng, 500, 16384) if lex else 0), bands=rng.random() < 0.3)
    if kind == "query":
        n = _log(rng, 10000, min(1000000, room))
        return dict(kind=kind, n=n, d=d, B=_log(rng, 33, 384), k=rng.choice([8, 16, 32, 64]), fmt=fmt, raw=raw,
                    clusters=max(1, n // CALL // 8))
    if kind == "ingest":
        n = _log(rng, 40, 80000 * 4096 // max(d, 4096))
        return dict(kind=kind, n=n, d=d, fmt=fmt, raw=raw, clusters=64)
    if kind == "grow":
        return dict(kind=kind, n=_log(rng, 500, 30000), d=d, B=rng.choice([1, 4, 8, 16, 32]), k=rng.choice([8, 16]),
                    fmt=fmt, raw=raw, clusters=32, rounds=4, add=rng.randrange(1, 9))
    B = rng.choice([1, 4, 16, 32, 64])
    return dict(kind=kind, n=_log(rng, 500, min(65536, 2000 * B)), d=d, B=B, k=16, L=8, raw=raw, clusters=64,
                sem_budget=rng.choice([16, 32, 64]))


# ------------------------------------------------------------------ inputs
def _gen(seed, device="cpu"):
    g = torch.Generator(device=device)
    g.manual_seed(seed & 0x7FFFFFFFFFFF)
    return g


def _dev():
    return torch.device("cuda")


class _Traffic:
    """Tokens, traces and raw states of a store of n positions."""

    def __init__(self, case, seed, n=None):
        self.n = n = case["n"] if n is None else n
        self.d, self.clusters, self.seed = case["d"], case["clusters"], seed
        self.vocab = case.get("vocab", 128256)
        self.dtype = torch.float32 if case["raw"] == "f32" else torch.bfloat16
        rng = np.random.default_rng(seed)
        calls = -(-n // CALL)
        if self.clusters:
            self.cluster = rng.integers(0, self.clusters, calls)
            self.templates = rng.integers(0, self.vocab, (self.clusters, CALL)).astype(np.int32)
            tok = self.templates[self.cluster]
            for _ in range(MINTED):
                tok[np.arange(calls), rng.integers(0, CALL, calls)] = rng.integers(0, self.vocab, calls)
        else:
            tok = rng.integers(0, self.vocab, (calls, CALL)).astype(np.int32)
        self.tokens = np.ascontiguousarray(tok.reshape(-1)[:n])
        self.traces = np.repeat(np.arange(calls, dtype=np.int32), CALL)[:n]
        self.rng = rng
        self._tables = None

    def labels(self):
        dev = _dev()
        return torch.from_numpy(self.tokens).to(dev), torch.from_numpy(self.traces).to(dev)

    def rows(self):
        """(first position, raw rows) chunk by chunk."""
        dev, n, d = _dev(), self.n, self.d
        if self.clusters and self._tables is None:
            g = _gen(self.seed * 1000003 + 1, dev)
            mu = torch.randn((self.clusters, d), generator=g, device=dev)
            mu /= mu.norm(dim=1, keepdim=True)
            off = torch.randn((self.clusters * CALL, d), generator=g, device=dev)
            # spread 0.1 of the norm, 64% of its variance by position in the call
            off = mu.repeat_interleave(CALL, dim=0).add_(off, alpha=0.08 / math.sqrt(d))
            self._tables = off
        for c, s in enumerate(range(0, n, CHUNK)):
            m = min(CHUNK, n - s)
            x = torch.randn((m, d), generator=_gen(self.seed * 1000003 + 7 + c, dev), device=dev)
            if self.clusters:
                at = np.arange(s, s + m)
                at = torch.from_numpy(self.cluster[at // CALL] * CALL + at % CALL).to(dev)
                x.mul_(0.06 / math.sqrt(d)).add_(self._tables[at])
            yield s, x.to(self.dtype)

    def drop_tables(self):
        self._tables = None


def _queries(case, seed, traffic, p_random):
    """Source positions (-1: none), and a function that takes raw chunks and
    fills the raw query rows."""
    rng = np.random.default_rng(seed + 17)
    B, n = case["B"], traffic.n
    src = rng.integers(0, n, B)
    src[rng.random(B) < p_random] = -1
    dev = _dev()
    z = torch.randn((B, case["d"]), generator=_gen(seed * 31 + 5, dev), device=dev)
    q = z.clone()

    def take(s, raw):
        here = np.nonzero((src >= s) & (src < s + raw.shape[0]))[0]
        if here.size:
            at = torch.from_numpy(here).to(dev)
            r = raw[torch.from_numpy(src[here] - s).to(dev)].float()
            q[at] = r + z[at] * (0.05 * r.norm(dim=1, keepdim=True) / math.sqrt(case["d"]))

    return src, q, take


def _fill(pool, traffic, take):
    tok, tr = traffic.labels()
    for s, raw in traffic.rows():
        e = s + raw.shape[0]
        pool.append(raw, tok[s:e], tr[s:e], tr[s:e])
        if take is not None:
            take(s, raw)
    traffic.drop_tables()


def _fresh_call(traffic, src):
    """The request behind a query: a new call of its source's kind, up to the
    token after the source position."""
    call, at = src // CALL, src % CALL
    t = (traffic.templates[traffic.cluster[call]] if traffic.clusters else traffic.tokens[call * CALL:][:CALL]).copy()
    t[traffic.rng.integers(0, len(t), MINTED)] = traffic.rng.integers(0, traffic.vocab, MINTED)
    return t[: min(at + 2, len(t))]


def _requests(case, traffic, src):
    """Anchors, lexical contexts and each request's own committed tokens."""
    B, H = case["B"], case["hist"]
    anchor = np.empty(B, np.int32)
    ctx, ctx_len = np.full((B, CTX), -1, np.int32), np.zeros(B, np.int32)
    excl = np.full(B, -1, np.int32)
    hist, hist_len = np.full((B, max(H, 1)), -1, np.int32), np.zeros(B, np.int32)
    calls = max(1, traffic.n // CALL)
    for b in range(B):
        mine = _fresh_call(traffic, int(src[b])) if src[b] >= 0 else traffic.rng.integers(0, traffic.vocab, 1)
        anchor[b] = mine[-1]
        if src[b] >= 0:
            c = mine[-CTX:]
            ctx[b, CTX - len(c):] = c
            ctx_len[b] = len(c)
            excl[b] = traffic.traces[src[b]]
        if H:
            want = int(traffic.rng.integers(max(1, H // 2), H + 1))
            old = traffic.rng.integers(0, calls, want // CALL + 1)
            row = traffic.tokens[(old[:, None] * CALL + np.arange(CALL)).reshape(-1) % traffic.n].copy()
            at = traffic.rng.integers(0, len(row), len(row) // 16)
            row[at] = traffic.rng.integers(0, traffic.vocab, len(at))
            row = np.concatenate([row, mine])[-want:]
            hist[b, : len(row)] = row
            hist_len[b] = len(row)
    to = lambda a: torch.from_numpy(a).to(_dev())  # noqa: E731
    return to(anchor), to(ctx), to(ctx_len), to(excl), to(hist), to(hist_len)


def _rule(case):
    return oil.DepthRule.paper(THETA) if case["bands"] else oil.DepthRule.fixed(case["L"], THETA)


def _i32(*shape):
    return torch.empty(shape, dtype=torch.int32, device=_dev())


def _store_buffers(case, rows):
    """The zeroed buffers of a store of `rows` positions, laid out once."""
    pool = oil.Pool(case["d"], rows, key_format=case["fmt"])
    for t in _buffers(pool).values():
        t.zero_()
    return pool


def _round(raw, tok, tr, case, t):
    """Round t's committed positions in tensors of their own, as a step has them."""
    a = case["n"] + t * case["add"]
    return tuple(x[a: a + case["add"]].clone() for x in (raw, tok, tr))


def prepare(case, seed):
    kind, dev = case["kind"], _dev()
    traffic = _Traffic(case, seed, case["n"] + (case["rounds"] * case["add"] if kind == "grow" else 0))
    s = dict(case=case)
    B = case.get("B", 0)
    if kind in ("step", "query"):
        src, q, take = _queries(case, seed, traffic, 0.0 if B == 1 else 0.25)
        pool = oil.Pool(case["d"], traffic.n, key_format=case["fmt"])
        _fill(pool, traffic, take)
        s.update(pool=pool, q=q.to(traffic.dtype).contiguous(),
                 top=(torch.empty((B, case["k"]), dtype=torch.float32, device=dev), _i32(B, case["k"])))
        if kind == "query":
            excl = np.where(src >= 0, traffic.traces[src], -1).astype(np.int32)
            s["excl"] = torch.from_numpy(excl).to(dev)
        else:
            k, L, slots = case["k"], case["L"], 1 + case["lex_budget"] + case["sem_budget"]
            names = ("anchor", "ctx", "ctx_len", "excl", "hist", "hist_len")
            s.update(zip(names, _requests(case, traffic, src)))
            s.update(rule=_rule(case), chains=(_i32(B, k, L), _i32(B, k)),
                     tree=(_i32(B, slots), _i32(B, slots), torch.empty((B, slots), dtype=torch.int8, device=dev),
                           _i32(B)))
            if case["lex"]:
                s.update(drafts=(_i32(B, case["lex"], case["lex_len"]), _i32(B, case["lex"])),
                         side=torch.cuda.Stream())
    elif kind in ("ingest", "grow"):
        pool = _store_buffers(case, traffic.n)
        tok, tr = traffic.labels()
        src, q, take = _queries(case, seed, traffic, 0.25) if kind == "grow" else (None, None, None)
        raw = torch.empty((traffic.n, case["d"]), dtype=traffic.dtype, device=dev)
        for at, x in traffic.rows():
            raw[at: at + x.shape[0]] = x
            if take is not None:
                take(at, x)
        traffic.drop_tables()
        s.update(pool=pool, raw=raw, tok=tok, tr=tr)
        if kind == "grow":
            s.update(q=q.to(traffic.dtype).contiguous(),
                     workspace=pool.workspace(B, case["k"]), more=[_round(raw, tok, tr, case, t)
                                                                   for t in range(case["rounds"])],
                     top=[(torch.empty((B, case["k"]), dtype=torch.float32, device=dev), _i32(B, case["k"]))
                          for _ in range(case["rounds"])])
    else:
        s.update(_verified(case, seed, traffic))
    return s


def _verified(case, seed, traffic, inserted=None):
    """Trees as a step leaves them, the verifier's predictions and states, and
    a standing ring that earlier steps filled (`inserted`, a list, receives
    what those steps put in)."""
    dev, B, k, L, d = _dev(), case["B"], case["k"], case["L"], case["d"]
    slots = 1 + case["sem_budget"]
    rng, g = traffic.rng, _gen(seed * 13 + 3, dev)
    ring = oil.RecyclePool(d, case["n"])
    out, held = {}, 0
    while held < case["n"] or not out:
        # continuations of one place of one kind of call, as retrieval returns them
        cl, at = rng.integers(0, case["clusters"], B), rng.integers(0, CALL - L - 1, B)
        chains = traffic.templates[cl[:, None], at[:, None] + 1 + np.arange(L)][:, None, :].repeat(k, 1)
        new = rng.random(chains.shape) < 0.08
        chains[new] = rng.integers(0, traffic.vocab, int(new.sum()))
        anchor = torch.from_numpy(traffic.templates[cl, at]).to(dev)
        ln = torch.full((B, k), L, dtype=torch.int32, device=dev)
        tree = oil.merge_trees(anchor, None, None, 0, torch.from_numpy(chains).to(dev), ln, case["sem_budget"], slots)
        tok, par, _, nn = (t.clone() for t in tree)
        live = torch.arange(slots, device=dev)[None, :] < nn[:, None]
        tok, par = torch.where(live, tok, -1), torch.where(live, par, -1)
        # the verifier agrees with one of a node's children three times in four
        target = torch.randint(0, traffic.vocab, (B, slots), generator=g, device=dev, dtype=torch.int32)
        agree = (torch.rand((B, slots), generator=g, device=dev) < 0.75) & live
        tok_h, par_h, agree_h, target_h = (t.cpu().numpy() for t in (tok, par, agree, target))
        for j in range(slots - 1, 0, -1):  # the earliest child wins
            b = np.nonzero((par_h[:, j] >= 0) & agree_h[np.arange(B), np.maximum(par_h[:, j], 0)])[0]
            target_h[b, par_h[b, j]] = tok_h[b, j]
        target = torch.from_numpy(target_h).to(dev)
        walk = oil.accept_walk(tok, par, nn, target)
        states = torch.randn((B, slots, d), generator=g, device=dev).to(traffic.dtype)
        ring.insert(tok, par, nn, target, walk[0], walk[1], states)
        held += max(1, int((nn - 1 - walk[0]).sum()))
        out = dict(tok=tok, par=par, nn=nn, target=target, states=states)
        if inserted is not None:
            inserted.append(_rejected(out))
    # lookups near the parents of nodes just drafted, and elsewhere
    node = np.minimum(rng.integers(1, slots, B), np.maximum(1, out["nn"].cpu().numpy() - 1))
    b = np.arange(B)
    up = np.maximum(out["par"].cpu().numpy()[b, node], 0)
    q = out["states"][torch.from_numpy(b).to(dev), torch.from_numpy(up).to(dev)].float()
    q = q + 0.3 * torch.randn(q.shape, generator=g, device=dev)
    anchor = torch.from_numpy(out["tok"].cpu().numpy()[b, node]).to(dev)
    words = (slots + 31) // 32
    session = oil.RecyclePool(d, 2 * B * case["sem_budget"])  # it turns over every few passes
    for t in (session.keys, session.tokens, session.rollouts):
        t.zero_()
    out.update(ring=ring, session=session, q=q.to(traffic.dtype).contiguous(), anchor=anchor, mask=_i32(B, slots, words),
               walk=(_i32(B), _i32(B, slots), _i32(B)),
               found=(torch.empty((B, 4), dtype=torch.float32, device=dev), _i32(B, 4, oil.REC_DEPTH), _i32(B, 4)))
    return out


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    return {"step": _run_step, "query": _run_query, "ingest": _run_ingest, "grow": _run_grow,
            "verify": _run_verify}[case["kind"]](case, s)


def _run_step(case, s):
    pool, side, drafts = s["pool"], s.get("side"), s.get("drafts")
    if side is not None:
        here = torch.cuda.current_stream()
        side.wait_stream(here)
        with torch.cuda.stream(side):
            pool.lexical(s["ctx"], s["ctx_len"], case["lex"], case["lex_len"], exclude_prompt=s["excl"], out=drafts,
                         hist=s["hist"], hist_len=s["hist_len"])
    scores, idx = pool.query_topk(s["q"], case["k"], out=s["top"])
    chains, lens = pool.gather(idx, scores, s["rule"], case["L"], out=s["chains"])
    if side is not None:
        here.wait_stream(side)
    lt, ll = drafts if drafts is not None else (None, None)
    slots = 1 + case["lex_budget"] + case["sem_budget"]
    tree = oil.merge_trees(s["anchor"], lt, ll, case["lex_budget"], chains, lens, case["sem_budget"], slots,
                           out=s["tree"])
    out = dict(scores=scores, idx=idx, chains=chains, lens=lens, tree=tree)
    if drafts is not None:
        out["drafts"] = drafts
    return out


def _run_query(case, s):
    scores, idx = s["pool"].query_topk(s["q"], case["k"], exclude_prompt=s["excl"], out=s["top"])
    return dict(scores=scores, idx=idx)


def _new_store(case, pool):
    """A new, empty store over the buffers that the server holds."""
    if case["fmt"] == "bf16":
        return oil.pool_create(case["d"], pool.capacity, pool.keys, pool.tokens, pool.traces, pool.prompts)
    store, at = ctypes.c_void_p(), lambda t: ctypes.c_void_p(t.data_ptr())
    status = oil.lib().oil_pool_create_fp8(case["d"], pool.capacity, at(pool.keys), at(pool.scales), at(pool.tokens),
                                           at(pool.traces), at(pool.prompts), ctypes.byref(store))
    if status:
        raise oil.OilError("oil_pool_create_fp8", status)
    return store


def _buffers(pool):
    out = dict(keys=pool.keys, tokens=pool.tokens, traces=pool.traces, prompts=pool.prompts)
    if pool.scales is not None:
        out["scales"] = pool.scales
    return out


def _run_ingest(case, s):
    store = _new_store(case, s["pool"])
    oil.pool_append(store, s["raw"], s["tok"], s["tr"], s["tr"])
    oil.pool_destroy(store)
    return _buffers(s["pool"])


def _run_grow(case, s):
    store, n = _new_store(case, s["pool"]), case["n"]
    oil.pool_append(store, s["raw"][:n], s["tok"][:n], s["tr"][:n], s["tr"][:n])
    for t in range(case["rounds"]):
        x, tok, tr = s["more"][t]
        oil.pool_append(store, x, tok, tr, tr)
        oil.pool_query_topk(store, s["q"], case["k"], s["workspace"], *s["top"][t])
    oil.pool_destroy(store)
    return dict(_buffers(s["pool"]), top=s["top"])


def _run_verify(case, s):
    tok, par, nn = s["tok"], s["par"], s["nn"]
    mask = oil.tree_mask(par, nn, mask=s["mask"])
    length, path, bonus = oil.accept_walk(tok, par, nn, s["target"], out=s["walk"])
    session = s["session"]
    session.insert(tok, par, nn, s["target"], length, path, s["states"])
    found = s["ring"].query(s["q"], s["anchor"], THETA, out=s["found"])
    return dict(mask=mask, length=length, path=path, bonus=bonus, keys=session.keys, tokens=session.tokens,
                rollouts=session.rollouts, head=session.head, found=found)


# ------------------------------------------------------------------ what a pass cannot do without
def _row_bytes(case):
    return case["d"] * (1 if case.get("fmt") == "fp8" else 2)


def work(case):
    kind, n, d, B = case["kind"], case["n"], case["d"], case.get("B", 0)
    raw = d * (4 if case["raw"] == "f32" else 2)
    if kind in ("step", "query"):
        nbytes = n * _row_bytes(case) + B * raw + 8 * B * case["k"]
        if kind == "step":
            nbytes += 4 * B * case["k"] * case["L"] + 9 * B * (1 + case["lex_budget"] + case["sem_budget"])
            if case["lex"]:
                nbytes += 4 * n + 4 * B * (case["hist"] + case["lex"] * case["lex_len"])
        return dict(bytes=nbytes, flops=2 * n * d * B)
    if kind == "ingest":
        return dict(bytes=n * (raw + _row_bytes(case) + 24), flops=4 * n * d)
    if kind == "grow":
        rows = n + case["rounds"] * case["add"]
        scans = sum(n + (t + 1) * case["add"] for t in range(case["rounds"]))
        return dict(bytes=rows * (raw + _row_bytes(case) + 24) + scans * _row_bytes(case) + case["rounds"] * B * raw,
                    flops=4 * rows * d + 2 * scans * d * B)
    # verify: three quarters of the slots hold a rejected node; a lookup reads
    # the ring's tokens and the keys of a few records per request
    slots = 1 + case["sem_budget"]
    records = B * slots * 3 // 4
    return dict(bytes=records * (raw + 2 * d + 40) + 4 * n + B * (raw + 8 * 2 * d) + B * slots * 4 * 8,
                flops=4 * records * d + 2 * B * 8 * d)


def tolerance(case):
    kind = case["kind"]
    if kind == "ingest":
        return "exact"  # stored rows are rounded once from 64 bits: the same bits from every implementation
    # scores are 32-bit sums of exact products: up to 1.6e-6 from 64 bits with
    # bf16 keys, 5.7e-6 with fp8 ones (whose matrix unit adds less exactly);
    # positions whose scores lie closer than that may change places
    if kind == "verify":
        return dict(rel=5e-6, differ=0.001)
    return dict(rel=2.5e-5 if case["fmt"] == "fp8" else 5e-6, differ=0.01)


# ------------------------------------------------------------------ the same in 64 bits
def _unit(raw):
    x = raw.double()
    return x / x.norm(dim=1, keepdim=True)


def _stored(case, raw):
    """Rows as the store defines them, in 64 bits: unit rows rounded to bf16,
    or to E4M3 under a power-of-two scale (and the inverse scale)."""
    u = _unit(raw)
    if case["fmt"] == "bf16":
        return u.to(torch.bfloat16).double(), None
    shift = 7 - torch.floor(torch.log2(u.abs().amax(dim=1, keepdim=True)))
    v = (u * torch.exp2(shift)).float().to(torch.float8_e4m3fn).double()
    return v * torch.exp2(-shift), torch.exp2(-shift)[:, 0]


def _best(case, chunks, q, prompts, excl):
    """The k best scores of each query over chunks of raw rows."""
    qs, _ = _stored(case, q)
    best = torch.full((qs.shape[0], 0), -math.inf, dtype=torch.float64, device=q.device)
    for s, raw in chunks:
        sc = qs @ _stored(case, raw)[0].T
        if excl is not None:
            sc[excl[:, None] == prompts[None, s: s + raw.shape[0]]] = -math.inf
        best = torch.cat([best, sc], dim=1)
        best = best.topk(min(case["k"], best.shape[1]), dim=1).values
    pad = case["k"] - best.shape[1]
    return torch.nn.functional.pad(best, (0, pad), value=-math.inf) if pad else best


def _tiles(unit, rows):
    """Unit rows in the order of the key buffer: 32 x 64 tiles, window by window."""
    n, d = unit.shape
    ld = (d + 63) // 64 * 64
    x = torch.zeros((rows, ld), dtype=torch.float64, device=unit.device)
    x[:n, :d] = unit
    return x.view(rows // 32, 32, ld // 64, 2, 4, 8).permute(2, 0, 4, 3, 1, 5).reshape(-1)


def _rejected(step):
    """Tokens and parents' states of the nodes that verification rejected, tree by tree."""
    tok, par, nn, target = (step[x].cpu().numpy() for x in ("tok", "par", "nn", "target"))
    trees, rows, tokens = [], [], []
    for b in range(len(nn)):
        taken, cur = set(), 0
        while True:
            below = [c for c in range(1, nn[b]) if par[b, c] == cur and tok[b, c] == target[b, cur]]
            if not below:
                break
            cur = below[0]
            taken.add(cur)
        left = [j for j in range(1, nn[b]) if j not in taken]
        trees += [b] * len(left)
        rows += [par[b, j] for j in left]
        tokens += [tok[b, j] for j in left]
    dev = _dev()
    states = step["states"][torch.tensor(trees, dtype=torch.long, device=dev),
                            torch.tensor(rows, dtype=torch.long, device=dev)]
    return torch.tensor(tokens, dtype=torch.int32, device=dev), states


def _exact_verify(case, seed, traffic):
    bf16, inserted = dict(case, fmt="bf16"), []
    step = _verified(case, seed, traffic, inserted)
    _, last = inserted[-1]
    keys = torch.zeros(step["session"].keys.shape, dtype=torch.float64, device=_dev())
    if len(last) <= len(keys):
        keys[: len(last), : case["d"]] = _unit(last)
    tok = torch.cat([t for t, _ in inserted])[-case["n"]:]
    q, _ = _stored(bf16, step["q"])
    best = []
    for s in range(0, len(tok), CHUNK):
        raw = torch.cat([x for _, x in inserted])[-case["n"]:][s: s + CHUNK]
        sc = q @ _stored(bf16, raw)[0].T
        sc[(step["anchor"][:, None] != tok[None, s: s + CHUNK]) | (sc < THETA)] = -math.inf
        best.append(sc)
    best = torch.cat(best + [torch.full((len(q), 4), -math.inf, dtype=torch.float64, device=_dev())], dim=1)
    return dict(keys=keys, found=[best.topk(4, dim=1).values, None, None])


def exact(case, seed):
    kind = case["kind"]
    traffic = _Traffic(case, seed, case["n"] + (case["rounds"] * case["add"] if kind == "grow" else 0))
    if kind in ("step", "query"):
        src, q, take = _queries(case, seed, traffic, 0.0 if case["B"] == 1 else 0.25)
        for s, raw in traffic.rows():
            take(s, raw)
        q = q.to(traffic.dtype)
        prompts = torch.from_numpy(traffic.traces).to(_dev())
        excl = None
        if kind == "query":
            excl = torch.from_numpy(np.where(src >= 0, traffic.traces[src], -1).astype(np.int32)).to(_dev())
        return dict(scores=_best(case, traffic.rows(), q, prompts, excl))
    if kind == "verify":
        return _exact_verify(case, seed, traffic)
    raw = torch.cat([x for _, x in traffic.rows()])
    out = {}
    if case["fmt"] == "bf16":
        blocks = -(-traffic.n // 32)
        blocks = -(-blocks // 128) * 128 if blocks > 1024 else blocks  # as large stores are padded
        out["keys"] = _tiles(_unit(raw), blocks * 32)
    else:
        out["scales"] = _stored(case, raw)[1]
    if kind == "grow":
        _, q, take = _queries(case, seed, traffic, 0.25)
        for s, x in traffic.rows():
            take(s, x)
        q = q.to(traffic.dtype)
        out["top"] = [(_best(case, [(0, raw[: case["n"] + (t + 1) * case["add"]])], q, None, None), None)
                      for t in range(case["rounds"])]
    return out
