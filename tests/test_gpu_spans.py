"""GPU: searched programs over equal spans of bytes (rx_match, rx_match_first and their fixed-length forms) against
the oracle and the one-lane-per-string kernel: every set width, strings that begin and end anywhere in a span, empty
strings, buffers at any alignment, threads that live on past a span and past the staged text."""
import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _compile(pattern_or_prog):
    from paper_1108_3126_amd import rx

    if isinstance(pattern_or_prog, bytes):
        ast, root, classes = rx.parse(pattern_or_prog)
    else:
        ast, root, classes = pattern_or_prog.ast, pattern_or_prog.root, pattern_or_prog.classes
    return rx.compile(ast, root, classes, search=True).upload(), (ast, root, classes)


def _earliest(tree, data, offs):
    """The oracle's earliest accepting prefix of every string: acceptance of a searched program is monotone in the
    prefix, so a binary search over prefix lengths (each step one oracle batch)."""
    n = len(offs) - 1
    lens = np.diff(offs)
    full = oracle.match(*tree, True, data, offs)
    lo, hi = np.zeros(n, np.int64), lens.copy()   # the answer lies in [lo, hi] where full is 1
    while (lo < hi).any():
        mid = (lo + hi) // 2
        po = np.zeros(n + 1, np.int64)
        np.cumsum(mid, out=po[1:])
        pd = np.concatenate([data[offs[i]:offs[i] + mid[i]] for i in range(n)] + [np.zeros(1, np.uint8)])
        m = oracle.match(*tree, True, pd, po).astype(bool)
        hi = np.where(m, mid, hi)
        lo = np.where(m, lo, np.minimum(mid + 1, hi))
    return np.where(full == 1, lo, -1), full


def _ragged(rng, alphabet, lens, skew):
    """Strings of the given lengths in a buffer whose first string begins `skew` bytes after an aligned address."""
    offs = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    offs += skew
    data = np.frombuffer(alphabet, np.uint8)[rng.integers(0, len(alphabet), size=int(offs[-1]) + 5)]
    return data, offs


def _check(dev, p, tree, data, offs, what):
    from paper_1108_3126_amd import rx

    want_first, want = _earliest(tree, data, offs)
    d, o = torch.from_numpy(np.ascontiguousarray(data)).to(dev), torch.from_numpy(offs).to(dev)
    print(what, len(offs) - 1, int(offs[-1]), flush=True)
    np.testing.assert_array_equal(rx.match(p, d, o).cpu().numpy(), want, err_msg=what)
    np.testing.assert_array_equal(rx.match_first(p, d, o).cpu().numpy(), want_first, err_msg=what)


# lengths around a span (16, 32, 64 bytes), around a region and around the staged tail
LENS = [0, 1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 0, 0, 95, 96, 97, 128, 300, 1000, 5000, 0]


@pytest.mark.parametrize("skew", [0, 1, 7, 16])
@pytest.mark.parametrize("pattern", [b"ab|ba+c", b"a.*b.*c.*d", b"(a|b)*cd", b"a{20}[bc]{30}d"])
def test_spans_against_the_oracle(dev, pattern, skew):
    p, tree = _compile(pattern)
    rng = np.random.default_rng([len(pattern), skew])
    lens = np.concatenate([rng.permutation(LENS) for _ in range(6)] + [rng.integers(0, 80, 300)])
    # rare letters: threads of the second pattern live on for many spans
    data, offs = _ragged(rng, b"xxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxxaaabcd" if b".*" in pattern else b"abcd", lens, skew)
    _check(dev, p, tree, data, offs, f"{pattern} skew {skew}")


@pytest.mark.parametrize("nodes", [30, 60, 120, 180, 240, 300, 420, 500, 600, 700, 800, 900])
def test_spans_every_set_width(dev, nodes):
    t = W.multi_programs(seed=300 + nodes, count=1, lo=nodes, hi=nodes)[0]
    p, tree = _compile(t)
    rng = np.random.default_rng(nodes)
    lens = np.concatenate([rng.integers(0, 200, 700), [3000, 0, 1]])
    offs = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    _check(dev, p, tree, W.zipf_bytes(rng, int(offs[-1])), offs, f"nodes {nodes} words {p.info.words}")


def test_spans_many_and_few_strings(dev):
    """More regions than workgroups, regions with more starts than their list holds, one string of many regions,
    and no bytes at all."""
    from paper_1108_3126_amd import rx

    p, tree = _compile(b"ab{3}c|ca{4}b")
    rng = np.random.default_rng(3)
    for lens, what in ((np.full(200_000, 3), "short"), (rng.integers(0, 2, 400_000), "bytes and empties"),
                       (np.full(30_000, 4096), "long")):
        data, offs = _ragged(rng, b"abc", lens, 3)
        d, o = torch.from_numpy(data).to(dev), torch.from_numpy(offs).to(dev)
        print(what, flush=True)
        want = rx.match(p, d, o, launch=(rx.VARIANT_LANE, 0, 0, 0)).cpu().numpy()
        np.testing.assert_array_equal(rx.match(p, d, o).cpu().numpy(), want, err_msg=what)
        sub = np.arange(0, len(lens), max(1, len(lens) // 500))
        np.testing.assert_array_equal(want[sub], oracle.match(*tree, True, data, offs, index=sub))
    empty = torch.zeros(5, dtype=torch.int64, device=dev)
    assert rx.match(p, torch.zeros(0, dtype=torch.uint8, device=dev), empty).cpu().tolist() == [0] * 4
    assert rx.match_first(p, torch.zeros(0, dtype=torch.uint8, device=dev), empty).cpu().tolist() == [-1] * 4


@pytest.mark.parametrize("length,n,shift", [(1, 1000, 0), (7, 3000, 0), (100, 2001, 0), (48, 500, 1), (333, 700, 3),
                                            (70_001, 3, 0)])
def test_spans_fixed_lengths(dev, length, n, shift):
    from paper_1108_3126_amd import rx

    p, tree = _compile(b"ab{2}c|c.a.b{4}")
    rng = np.random.default_rng(length)
    data = np.frombuffer(b"abc", np.uint8)[rng.integers(0, 3, n * length)]
    buf = torch.zeros(n * length + 16, dtype=torch.uint8, device=dev)
    d = buf[shift:shift + n * length]
    d.copy_(torch.from_numpy(data))
    offs = np.arange(n + 1, dtype=np.int64) * length
    want_first, want = _earliest(tree, data, offs)
    np.testing.assert_array_equal(rx.match_fixed(p, d, length, n).cpu().numpy(), want)
    np.testing.assert_array_equal(rx.match_first_fixed(p, d, length, n).cpu().numpy(), want_first)


def _mixed_programs():
    """Searched (over spans), anchored, nullable and searched-nullable programs, narrow and wide sets."""
    from paper_1108_3126_amd import rx

    out = [(*rx.parse(p), search) for p, search in ((b"ab+c", True), (b"a.*b.*c", False), (b"(ab)*", True), (b"[^q]*z", False),
                                                    (b"q.{40}z", True))]
    for seed, nodes in ((5, 40), (6, 500), (7, 900)):
        t = W.multi_programs(seed=seed, count=1, lo=nodes, hi=nodes)[0]
        out.append((t.ast, t.root, t.classes, True))
    return out


@pytest.mark.parametrize("n,mean,hi", [(1, 50, 50), (700, 100, 5000), (30_000, 60, 2000)])
@pytest.mark.parametrize("graph", [False, True])
def test_spans_in_batched_matching(dev, n, mean, hi, graph):
    """rx_match_multi's table form with lists that mix programs over spans and over buckets, and lists of one kind."""
    from paper_1108_3126_amd import rx

    progs = _mixed_programs()
    ps = [rx.compile(a, r, c, search=s).upload() for a, r, c, s in progs]
    rng = np.random.default_rng(n)
    lens = W.lognormal_lengths(rng, n, mean, 1.0, 0, hi)
    offs = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    data = W.zipf_bytes(rng, int(offs[-1]))
    d, o = torch.from_numpy(data).to(dev), torch.from_numpy(offs).to(dev)
    sub = np.arange(n) if n < 1000 else np.arange(0, n, 37)
    want = np.stack([oracle.match(a, r, c, s, data, offs, index=sub) for a, r, c, s in progs])
    for pick in (range(len(ps)), [1, 3], [0, 5, 7], [4]):
        pick = list(pick)
        print(n, pick, graph, flush=True)
        for _ in range(3 if graph else 1):
            got = rx.match_multi([ps[k] for k in pick], d, o, config=rx.multi_config(graph=graph)).cpu().numpy()
            np.testing.assert_array_equal(got[:, sub], want[pick])


@pytest.mark.parametrize("graph", [False, True])
def test_spans_in_the_server(dev, graph):
    """Requests of every kind in shared steps; a server whose steps hold few work items (several regions each)."""
    from paper_1108_3126_amd.server import Server

    progs = _mixed_programs()
    rng = np.random.default_rng(11)
    for cfg in (dict(), dict(step_bytes=1 << 20, step_strings=512, step_requests=8, block=256)):
        reqs, ids = [], []
        with Server(use_graph=graph, **cfg) as srv:
            for i in range(40):
                a, r, c, s = progs[i % len(progs)]
                n = int(rng.integers(0, 60))
                lens = W.lognormal_lengths(rng, n, 300, 1.5, 0, 8192)
                offs = np.zeros(n + 1, np.int64)
                np.cumsum(lens, out=offs[1:])
                data = W.zipf_bytes(rng, int(offs[-1]))
                ids.append(srv.submit(W.Program(a, r, c, s), data, offs))
                reqs.append((a, r, c, s, data, offs))
            for rid, (a, r, c, s, data, offs) in zip(ids, reqs):
                np.testing.assert_array_equal(srv.wait(rid), oracle.match(a, r, c, s, data, offs))


# -- the same over the compiled circuit (regions of 2,016 slots of 16 bytes) ----------------------------------------
CIRCUIT_LENS = [0, 1, 15, 16, 17, 31, 33, 0, 0, 511, 512, 513, 700, 40_000, 5, 0, 32_255, 32_256, 32_257, 100]


@pytest.mark.parametrize("pattern", [b"ab|ba+c", b"a.*b.*c.*d", b"(a|b)*cd", b"a{20}[bc]{30}d", b"a[^q]{600}b"])
def test_circuit_spans_against_the_oracle(dev, pattern):
    p, tree = _compile(pattern)
    try:
        p.jit()
    except Exception as e:   # more state words than the circuit holds: the tables run
        assert "state words" in str(e)
    for skew in (0, 3, 16):
        rng = np.random.default_rng([len(pattern), skew])
        lens = np.concatenate([rng.permutation(CIRCUIT_LENS), rng.integers(0, 80, 3000), rng.permutation(CIRCUIT_LENS)])
        rare = b".*" in pattern or b"^q" in pattern
        data, offs = _ragged(rng, b"x" * 150 + b"aabcd" if rare else b"abcd", lens, skew)
        _check(dev, p, tree, data, offs, f"circuit {pattern} skew {skew}")


@pytest.mark.parametrize("seed,nodes", [(4, 40), (5, 120), (6, 200), (8, 300)])
def test_circuit_spans_trees(dev, seed, nodes):
    t = W.multi_programs(seed=700 + seed, count=1, lo=nodes, hi=nodes)[0]
    p, tree = _compile(t)
    p.jit()
    rng = np.random.default_rng(nodes)
    lens = np.concatenate([rng.integers(0, 200, 2500), [9000, 0, 1]])
    offs = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    _check(dev, p, tree, W.zipf_bytes(rng, int(offs[-1])), offs, f"circuit nodes {nodes} {p.jit_stats()}")


def test_circuit_spans_many_strings(dev):
    """More regions than wavefronts; strings of one byte and empty ones (several begin at one byte)."""
    from paper_1108_3126_amd import rx

    p, tree = _compile(b"ab{3}c|ca{4}b")
    q, _ = _compile(b"ab{3}c|ca{4}b")
    p.jit()
    rng = np.random.default_rng(3)
    for lens, what in ((np.full(200_000, 3), "short"), (rng.integers(0, 2, 400_000), "bytes and empties"),
                       (rng.integers(1, 2000, 60_000), "mixed")):
        data, offs = _ragged(rng, b"abc", lens, 3)
        d, o = torch.from_numpy(data).to(dev), torch.from_numpy(offs).to(dev)
        print(what, flush=True)
        np.testing.assert_array_equal(rx.match(p, d, o).cpu().numpy(), rx.match(q, d, o).cpu().numpy(), err_msg=what)
        np.testing.assert_array_equal(rx.match_first(p, d, o).cpu().numpy(), rx.match_first(q, d, o).cpu().numpy(),
                                      err_msg=what)


@pytest.mark.parametrize("length,n,shift", [(1, 1000, 0), (100, 2001, 0), (48, 500, 1), (333, 700, 3), (70_001, 3, 0)])
def test_circuit_spans_fixed_lengths(dev, length, n, shift):
    from paper_1108_3126_amd import rx

    p, tree = _compile(b"ab{2}c|c.a.b{4}")
    p.jit()
    rng = np.random.default_rng(length)
    data = np.frombuffer(b"abc", np.uint8)[rng.integers(0, 3, n * length)]
    buf = torch.zeros(n * length + 16, dtype=torch.uint8, device=dev)
    d = buf[shift:shift + n * length]
    d.copy_(torch.from_numpy(data))
    want_first, want = _earliest(tree, data, np.arange(n + 1, dtype=np.int64) * length)
    np.testing.assert_array_equal(rx.match_fixed(p, d, length, n).cpu().numpy(), want)
    np.testing.assert_array_equal(rx.match_first_fixed(p, d, length, n).cpu().numpy(), want_first)


@pytest.mark.parametrize("jit", [False, True])
def test_long_string_with_a_thread_that_outlives_its_span(dev, jit):
    """One long string: a thread begun near the start that lives to the end (the span kernels leave it to the
    chunk-parallel ones), one that dies within the limit, and none; with and without an accept."""
    from paper_1108_3126_amd import rx

    p, tree = _compile(b"a[^q]*b|cde")
    if jit:
        p.jit()
    base = np.full(200_000, ord("x"), np.uint8)
    for edits in ((), ((100, b"a"),), ((100, b"a"), (199_999, b"b")), ((100, b"a"), (2_000, b"q"), (150_000, b"b")),
                  ((100, b"a"), (50_000, b"q"), (150_000, b"cde")), ((5, b"b"), (31_998, b"cde")), ((65_533, b"a"), (65_600, b"b"))):
        text = base.copy()
        for at, w in edits:
            text[at:at + len(w)] = np.frombuffer(w, np.uint8)
        d = torch.from_numpy(text).to(dev)
        want_first, want = _earliest(tree, text, np.array([0, text.size]))
        print(jit, edits, flush=True)
        assert int(rx.match_long(p, d).item()) == want[0]
        assert int(rx.match_first_long(p, d).item()) == want_first[0]
        assert int(rx.match_long(p, d, text.size, 50).item()) == want[0]
