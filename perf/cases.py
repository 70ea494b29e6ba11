"""What users of the matcher have it do, as cases that can be timed and compared.

Each case is a dict of plain values.  ``listed()`` names twelve of them, ``draw(rng)`` makes more of the same
kinds over the same ranges, ``prepare(case, seed)`` makes what a user's program holds before the call (strings and
offsets on the GPU, compiled and uploaded programs, a running server), ``run(state)`` is one call through the
package's entry points, ``work(case)`` the bytes it cannot do without, and ``exact(case, seed)`` the results of the
one kind of case that the standard library's ``re`` can give by itself.

The expressions and texts are those of ``paper_1108_3126_amd.workloads``: random trees over lowercase or printable
bytes, Zipf(1.1) characters, log-normal line lengths, and strings of the expression's language planted in a part
of the texts, so that some match and most do not.  An expression is a program's own and stays the same while its
inputs change, so it depends on the case alone; the texts depend on the seed.
"""
from __future__ import annotations

import functools
import math
import re

import numpy as np
import torch

from paper_1108_3126_amd import rx
from paper_1108_3126_amd import workloads as W
from paper_1108_3126_amd.server import Server

# the expression of the README's example: a log filter
PATTERN = r"err(or)?[0-9]{3}|time[ -]?out"
# the trees over lowercase bytes that match few random texts (others match nearly every one within a few bytes)
RARE = (1, 5, 7)


def listed():
    return [
        # a unit test's or a validator's call: a few short strings, where the call itself is what counts
        dict(name="small_1000", kind="small", n=1000, max_len=32, prog=0),
        # filtering one file of log lines with the README's expression
        dict(name="lines_20k", kind="lines", n=20_000, mean=120, max_len=4096, nodes=0, jit=True, first=False, prog=0),
        # filtering a day's log with a large expression
        dict(name="lines_1m", kind="lines", n=1_000_000, mean=120, max_len=4096, nodes=200, jit=True, first=False,
             prog=1),
        # where the first match of each line ends, with an expression that has just been typed in (not compiled
        # to a circuit)
        dict(name="first_lines_100k", kind="lines", n=100_000, mean=120, max_len=4096, nodes=64, jit=False,
             first=True, prog=6),
        # fixed-length records: the benchmark's workload
        dict(name="fixed_1m_256", kind="fixed", n=1_000_000, length=256, jit=True, first=False, prog=1),
        # fixed-length records of an odd size
        dict(name="fixed_odd_200k_100", kind="fixed", n=200_003, length=100, jit=True, first=False, prog=7),
        # where the first match ends, in fixed-length records
        dict(name="first_fixed_250k_256", kind="fixed", n=250_000, length=256, jit=True, first=True, prog=1),
        # a rule set of sixteen prepared expressions over half a million lines
        dict(name="multi_planes_16x500k", kind="multi", progs=16, n=500_000, mean=120, max_len=4096, planes=True,
             prog=2),
        # a few new expressions over one file's lines, with the call's default form
        dict(name="multi_table_4x20k", kind="multi", progs=4, n=20_000, mean=120, max_len=4096, planes=False, prog=7),
        # eight long texts (whole files, each one string) searched in turn, with the expression compiled
        dict(name="long_8x8m", kind="long", files=8, length=8 << 20, jit=True, first=False, prog=1),
        # an expression of 4,096 nodes that makes a backtracking matcher run forever
        dict(name="nested_4096", kind="nested", family="nested", k=819, n=256, length=1000),
        # a burst of requests to the server, each with its own expression and host strings
        dict(name="serving_100", kind="serving", requests=100, max_strings=2000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["small", "lines", "lines", "lines", "fixed", "fixed", "multi", "long", "nested", "serving"])
    if kind == "small":
        return dict(kind=kind, n=_log_int(rng, 100, 10_000), max_len=rng.randint(8, 64), prog=rng.randint(0, 99))
    if kind == "lines":
        mean = _log_int(rng, 30, 500)
        return dict(kind=kind, n=_log_int(rng, 5_000, 100_000_000 // mean // 2), mean=mean,
                    max_len=rng.choice([1000, 4096, 8192]), nodes=rng.choice([0, _log_int(rng, 16, 300)]),
                    jit=rng.random() < 0.5, first=rng.random() < 0.3, prog=rng.randint(0, 99))
    if kind == "fixed":
        length = rng.choice([16 * rng.randint(1, 64), rng.randint(10, 1000)])
        return dict(kind=kind, n=_log_int(rng, 5_000, 200_000_000 // length), length=length, jit=rng.random() < 0.7,
                    first=rng.random() < 0.3, prog=rng.choice(RARE))
    if kind == "multi":
        planes = rng.random() < 0.5
        return dict(kind=kind, progs=rng.randint(2, 16), n=_log_int(rng, 5_000, 400_000 if planes else 40_000),
                    mean=_log_int(rng, 60, 200), max_len=rng.choice([2000, 4096]), planes=planes,
                    prog=rng.randint(0, 99))
    if kind == "long":
        return dict(kind=kind, files=8, length=_log_int(rng, 100_000, 4 << 20), jit=rng.random() < 0.5,
                    first=rng.random() < 0.4, prog=rng.choice(RARE))
    if kind == "nested":
        return dict(kind=kind, family=rng.choice(["nested", "altstar"]), k=rng.randint(100, 585),
                    n=rng.randint(64, 512), length=_log_int(rng, 200, 1500))
    return dict(kind=kind, requests=rng.randint(20, 100), max_strings=_log_int(rng, 200, 2000))


# -- programs (the case's own; a user compiles an expression once and feeds it texts) --------------------------
@functools.lru_cache(maxsize=64)
def _tree(seed, nodes, lower):
    """A random searched expression of about `nodes` nodes over lowercase or printable bytes, and members of its
    language (padded rows and their lengths)."""
    if lower:
        p = W.single_program(seed)
    else:
        p = W.multi_programs(seed=1000 + seed, count=1, lo=nodes, hi=nodes)[0]
    return p, _members(p, seed)


def _members(p, seed, count=512, max_len=64):
    u = W._Uniforms(np.random.default_rng([seed, 77]), 4096)
    rows, lens, cache = np.zeros((count, max_len), np.uint8), np.zeros(count, np.int64), {}
    for i in range(count):
        w = None
        for _ in range(20):
            w = W.sample_member(p, u, max_len=max_len, _cache=cache)
            if w:
                break
        w = w or b""
        rows[i, :len(w)] = np.frombuffer(w, np.uint8)
        lens[i] = len(w)
    return rows, lens


def _pattern_members(count=512, max_len=64):
    words = [b"err404", b"error500", b"timeout", b"time-out", b"time out", b"err123"]
    rows, lens = np.zeros((count, max_len), np.uint8), np.zeros(count, np.int64)
    for i in range(count):
        w = words[i % len(words)]
        rows[i, :len(w)] = np.frombuffer(w, np.uint8)
        lens[i] = len(w)
    return rows, lens


@functools.lru_cache(maxsize=64)
def _program(nodes, seed, lower, jit):
    """An uploaded program (a circuit too, if the user asked for one) and members of its language."""
    if nodes == 0 and not lower:
        p, members = rx.compile_regex(PATTERN.encode(), search=True), _pattern_members()
    else:
        t, members = _tree(seed, nodes, lower)
        p = rx.compile(t.ast, t.root, t.classes, search=True)
    p.upload(torch.device("cuda", torch.cuda.current_device()))
    if jit:
        try:
            p.jit()
        except rx.RxError:   # a circuit too large for its kernel: the program is matched without
            pass
    return p, members


@functools.lru_cache(maxsize=16)
def _rule_set(count, seed, planes):
    trees = W.multi_programs(seed=seed, count=count)
    progs = [rx.compile(t.ast, t.root, t.classes, search=True).upload() for t in trees]
    if planes:
        rx.prepare_multi(progs)
    return progs


# -- texts ----------------------------------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1_000_003 + salt)
    return g


def _zipf(size, g):
    cdf = torch.from_numpy(W.zipf_cdf()).float().cuda()
    out = torch.empty(size, dtype=torch.uint8, device="cuda")
    step = 1 << 26
    for a in range(0, size, step):
        e = min(size, a + step)
        u = torch.rand(e - a, device="cuda", generator=g)
        out[a:e] = (torch.searchsorted(cdf, u, right=True).clamp_(max=94) + 0x20).to(torch.uint8)
    return out


def _plant(data, starts, lens, members, part, g):
    """Writes a random member into a random place of `part` of the strings that have room for one."""
    rows, ml = torch.from_numpy(members[0]).cuda(), torch.from_numpy(members[1]).cuda()
    n = starts.numel()
    pick = torch.nonzero(torch.rand(n, device="cuda", generator=g) < part).flatten()
    which = torch.randint(0, rows.shape[0], (pick.numel(),), device="cuda", generator=g)
    room = lens[pick] - ml[which]
    ok = (room >= 0) & (ml[which] > 0)
    pick, which, room = pick[ok], which[ok], room[ok]
    at = starts[pick] + (torch.rand(pick.numel(), device="cuda", generator=g) * (room + 1)).long().clamp(max=room)
    k = torch.arange(rows.shape[1], device="cuda")
    inside = k[None, :] < ml[which][:, None]
    data[(at[:, None] + k[None, :])[inside]] = rows[which][inside]


def _lines(n, mean, max_len, seed):
    g = _gen(seed, 1)
    z = torch.randn(n, device="cuda", generator=g, dtype=torch.float64)
    lens = torch.exp(z + (math.log(mean) - 0.5)).round().long().clamp(1, max_len)
    offsets = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    offsets[1:] = torch.cumsum(lens, 0)
    return _zipf(int(offsets[-1]), g), offsets, lens, g


def _quiet(p, g):
    """Pieces of 256 random lowercase bytes that the program rejects, also one after another, so that a text put
    together from them holds no match of its own and is read to its end."""
    k = 48
    x = torch.randint(97, 123, (4 * k, 256), dtype=torch.uint8, device="cuda", generator=g)
    x = x[rx.match_fixed(p, x.flatten(), 256, len(x)) == 0][:k]
    pairs = torch.cat([x[:, None].expand(-1, len(x), -1), x[None].expand(len(x), -1, -1)], 2).contiguous()
    bad = rx.match_fixed(p, pairs.flatten(), 512, len(x) * len(x)).view(len(x), len(x)).bool()
    return x[~(bad.any(0) | bad.any(1))]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "small":
        s = W.small_strings(seed, n=case["n"], max_len=case["max_len"])
        t = W.small_program(case["prog"])
        p = rx.compile(t.ast, t.root, t.classes, search=False).upload()
        return dict(kind=kind, p=p, data=torch.from_numpy(s.data).cuda(), offsets=torch.from_numpy(s.offsets).cuda())
    if kind == "lines":
        p, members = _program(case["nodes"], case["prog"], False, case["jit"])
        data, offsets, lens, g = _lines(case["n"], case["mean"], case["max_len"], seed)
        _plant(data, offsets[:-1], lens, members, 0.05, g)
        return dict(kind=kind, p=p, data=data, offsets=offsets, first=case["first"])
    if kind == "fixed":
        p, members = _program(0, case["prog"], True, case["jit"])
        n, length = case["n"], case["length"]
        g = _gen(seed, 2)
        data = torch.randint(97, 123, (n * length,), dtype=torch.uint8, device="cuda", generator=g)
        starts = torch.arange(n, device="cuda") * length
        _plant(data, starts, torch.full_like(starts, length), members, 0.1, g)
        return dict(kind=kind, p=p, data=data, length=length, n=n, first=case["first"])
    if kind == "multi":
        progs = _rule_set(case["progs"], case["prog"], case["planes"])
        data, offsets, _, _ = _lines(case["n"], case["mean"], case["max_len"], seed)
        cfg = rx.multi_config(form=rx.FORM_PLANES if case["planes"] else rx.FORM_TABLE)
        return dict(kind=kind, progs=progs, data=data, offsets=offsets, cfg=cfg)
    if kind == "long":
        p, members = _program(0, case["prog"], True, case["jit"])
        length, g = case["length"], _gen(seed, 3)
        pieces = _quiet(p, g)
        files = []
        for _ in range(case["files"]):   # half of the files hold a member, in their last 256 bytes
            data = pieces[torch.randint(0, len(pieces), (-(-length // 256),), device="cuda", generator=g)]
            data = data.flatten()[:length].contiguous()
            at = torch.full((1,), length - 256, dtype=torch.int64, device="cuda")
            _plant(data, at, torch.full_like(at, 256), members, 0.5, g)
            files.append(data)
        return dict(kind=kind, p=p, files=files, first=case["first"])
    if kind == "nested":
        t = W.pathological_program(case["family"], case["k"])
        s = W.pathological_strings(case["family"], case["length"], case["n"])
        flip = np.random.default_rng([seed, 5]).random(case["n"]) < 0.1   # a foreign byte somewhere: rejected there
        for i in np.nonzero(flip)[0]:
            s.data[s.offsets[i] + int(i * 37 + seed) % case["length"]] = 120
        p = _nested(case["family"], case["k"], t)
        return dict(kind="lines", p=p, data=torch.from_numpy(s.data).cuda(), offsets=torch.from_numpy(s.offsets).cuda(),
                    first=False)
    if kind == "serving":
        reqs = []
        for i in range(case["requests"]):   # a request's expression and string count are the case's, its texts the seed's
            tree, n = _request(i, case["max_strings"])
            rng = np.random.default_rng([seed, 6, i])
            offsets = np.zeros(n + 1, np.int64)
            np.cumsum(W.lognormal_lengths(rng, n, 256.0, 1.0, 16, 8192, arithmetic_mean=False), out=offsets[1:])
            reqs.append((tree, W.zipf_bytes(rng, int(offsets[-1])), offsets))
        return dict(kind=kind, server=Server(), reqs=reqs)
    raise ValueError(kind)


@functools.lru_cache(maxsize=512)
def _request(i, max_strings):
    tree, _ = W.serving_request(8, i, 2)   # the expression alone
    return tree, int(round(math.exp(np.random.default_rng([i, 7]).uniform(0.0, math.log(max_strings)))))


_nested_cache = {}


def _nested(family, k, tree):
    if (family, k) not in _nested_cache:
        if len(_nested_cache) >= 8:
            _nested_cache.clear()
        _nested_cache[family, k] = rx.compile(tree.ast, tree.root, tree.classes, search=False).upload()
    return _nested_cache[family, k]


def run(state):
    kind = state["kind"]
    if kind == "small":
        return rx.match(state["p"], state["data"], state["offsets"])
    if kind == "lines":
        f = rx.match_first if state["first"] else rx.match
        return f(state["p"], state["data"], state["offsets"])
    if kind == "fixed":
        f = rx.match_first_fixed if state["first"] else rx.match_fixed
        return f(state["p"], state["data"], state["length"], state["n"])
    if kind == "multi":
        return rx.match_multi(state["progs"], state["data"], state["offsets"], config=state["cfg"])
    if kind == "long":
        f = rx.match_first_long if state["first"] else rx.match_long
        return torch.cat([f(state["p"], data) for data in state["files"]])
    ids = [state["server"].submit(t, data, offsets) for t, data, offsets in state["reqs"]]
    return np.concatenate([state["server"].wait(i) for i in ids])


def work(case):
    """Every input byte read once and every result written once (matching is boolean: no floating point)."""
    kind = case["kind"]
    res = 8 if case.get("first") else 1
    if kind == "small":
        b = case["n"] * (case["max_len"] // 2 + 9)
    elif kind == "lines":
        b = case["n"] * (case["mean"] + 8 + res)
    elif kind in ("fixed", "nested"):
        b = case["n"] * (case["length"] + res)
    elif kind == "multi":
        b = case["n"] * (case["mean"] + 8 + case["progs"])
    elif kind == "long":
        b = case["files"] * (case["length"] + res)
    else:   # strings go to the device and bits come back: log-uniform counts, log-normal lengths of median 256
        strings = case["requests"] * (case["max_strings"] - 1) / math.log(case["max_strings"])
        b = strings * (256 * math.exp(0.5) + 9)
    return {"bytes": int(b), "flops": 0}


def exact(case, seed):
    """The README's expression has a form that the standard library matches; the random trees have none."""
    if case["kind"] != "lines" or case["nodes"] != 0 or case["n"] > 200_000:
        return None
    state = prepare(case, seed)
    data, offs = state["data"].cpu().numpy().tobytes(), state["offsets"].tolist()
    rexp = re.compile(PATTERN.encode(), re.DOTALL)
    if not case["first"]:
        return torch.tensor([rexp.search(data, a, b) is not None for a, b in zip(offs, offs[1:])], dtype=torch.uint8)
    out = []
    for a, b in zip(offs, offs[1:]):   # the earliest end over all starts
        ends = [m.end() for m in rexp.finditer(data[a:b])]
        out.append(min(ends) if ends else -1)
    return torch.tensor(out, dtype=torch.int64)
