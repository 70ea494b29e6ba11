"""GPU: the compiled circuit over spans, on batches large enough for it (a few thousand distinct strings over and over,
so the oracle's part stays small and every copy lies differently in the kernel's regions), with matches: uneven and
empty strings, equal lengths without offsets, unaligned starts, long texts, threads that outlive slot, lane and region,
both kinds of result.  Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import rx
from test_spans_cpu import PATTERNS, _program, _text, earliest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


ALL = [*PATTERNS, (4, 40), (6, 200), (8, 300)]


def _jitted(pattern):
    p, tree = _program(pattern)
    p.upload().jit()
    check = p.jit_selfcheck()
    assert p.jit_spans_source() and check["ran"] == 1 and not check["dropped"] & 256   # the circuit over spans is there
    return p, tree


def _strings(pattern, rng, lens):
    offs = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    return _text(rng, pattern, offs), offs


def _tiled(data, offs, times, skew):
    """The strings `times` times over, the first one `skew` bytes into the buffer."""
    n, size = len(offs) - 1, int(offs[-1])
    o = (offs[:-1][None] + np.arange(times, dtype=np.int64)[:, None] * size).ravel()
    d = np.concatenate([np.zeros(skew, np.uint8), np.tile(data[:size], times)])
    return d, np.concatenate([o, [n and times * size]]).astype(np.int64) + skew


def _compare(got, want, times, what):
    got = got.cpu().numpy().reshape(times, -1)
    bad = np.nonzero((got != want[None]).any(axis=1))[0]
    assert bad.size == 0, (what, bad[:5], np.nonzero(got[bad[0]] != want)[0][:10])


@pytest.mark.parametrize("skew", [0, 5])
@pytest.mark.parametrize("pattern", ALL, ids=str)
def test_uneven_strings(pattern, skew):
    p, tree = _jitted(pattern)
    rng = np.random.default_rng([len(str(pattern)), skew])
    lens = np.concatenate([rng.permutation([0, 1, 15, 16, 17, 31, 33, 0, 0, 511, 512, 513, 700, 5, 0, 100, 0, 40_000, 32_255]),
                           rng.integers(0, 200, 2500)])
    data, offs = _strings(pattern, rng, lens)
    want_first, want = earliest(tree, data, offs)
    assert 0 < want.sum() < len(want)
    times = -(-101_000 // len(lens))   # from 100,000 strings on (40,000 above two words)
    d, o = _tiled(data, offs, times, skew)
    d, o = torch.from_numpy(d).cuda(), torch.from_numpy(o).cuda()
    print(pattern, skew, o.numel() - 1, d.numel(), p.jit_stats(), flush=True)
    _compare(rx.match(p, d, o), want, times, "match")
    _compare(rx.match_first(p, d, o), want_first, times, "first")


@pytest.mark.parametrize("length,base,shift", [(100, 3000, 0), (333, 900, 3), (48, 6000, 1), (20, 9000, 0), (70_001, 5, 2)])
@pytest.mark.parametrize("pattern", [b"ab|ba+c", b"a{20}[bc]{30}d", (6, 200)], ids=str)
def test_equal_lengths(pattern, length, base, shift):
    p, tree = _jitted(pattern)
    rng = np.random.default_rng(length)
    data, offs = _strings(pattern, rng, np.full(base, length))
    want_first, want = earliest(tree, data, offs)
    if length <= 100:
        assert want.sum() < len(want)
    times = -(-12_500_000 // data.size)   # from 12 MB on (5 MB above two words)
    d = torch.zeros(data.size * times + 32, dtype=torch.uint8, device="cuda")[shift:shift + data.size * times]
    d.copy_(torch.from_numpy(np.tile(data, times)))
    print(pattern, length, base * times, flush=True)
    _compare(rx.match_fixed(p, d, length, base * times), want, times, "fixed")
    _compare(rx.match_first_fixed(p, d, length, base * times), want_first, times, "first fixed")


@pytest.mark.parametrize("edits", [(), ((100, b"a"),), ((100, b"a"), (12_999_999, b"b")), ((100, b"a"), (2_000, b"q"), (9_000_000, b"cde")),
                                   ((32_250, b"a"), (32_262, b"b")), ((12_999_997, b"cde"),), ((5_000_000, b"cde"), (77, b"a"))])
@pytest.mark.parametrize("pattern", [b"a[r-z]*b|cde|fghijklm"], ids=str)
def test_one_long_string(pattern, edits):
    p, tree = _program(pattern)
    p.upload().jit()
    text = np.full(13_000_000, ord("x"), np.uint8)
    for at, w in edits:
        text[at:at + len(w)] = np.frombuffer(w, np.uint8)
    # the oracle on the text with its middle runs of x cut short (what the pattern does there does not depend on them)
    keep = np.zeros(text.size, bool)
    for at in [0, text.size - 64] + [at for at, _ in edits]:
        keep[max(0, at - 64):at + 128] = True
    short, where = text[keep], np.nonzero(keep)[0]
    first, want = earliest(tree, short, np.array([0, short.size]))
    end = int(where[first[0] - 1]) + 1 if want[0] else -1
    d = torch.from_numpy(text).cuda()
    print(pattern, edits, end, flush=True)
    assert int(rx.match_long(p, d).item()) == want[0]
    assert int(rx.match_first_long(p, d).item()) == end


@pytest.mark.parametrize("jit", [False, True])
@pytest.mark.parametrize("length,base", [(64, 4000), (256, 2000), (100, 3000), (511, 1000), (512, 1000), (1040, 500)])
def test_programs_whose_threads_may_live_on(length, base, jit):
    """err.*timeout and the like: equal lengths stay with the kernels that one such thread does not slow down."""
    tree = rx.parse(b"a[^q]*b|cde")
    p = rx.compile(*tree, search=True).upload()
    if jit:
        p.jit()
    rng = np.random.default_rng(length)
    data, offs = _strings(b"a[^q]*b|cde", rng, np.full(base, length))
    want_first, want = earliest(tree, data, offs)
    assert 0 < want.sum() < base
    times = -(-20_000 // base)
    d, o = _tiled(data, offs, times, 0)
    d, o = torch.from_numpy(d).cuda(), torch.from_numpy(o).cuda()
    print(length, base * times, jit, flush=True)
    _compare(rx.match(p, d, o), want, times, "match")
    _compare(rx.match_first(p, d, o), want_first, times, "first")
    _compare(rx.match_fixed(p, d, length, base * times), want, times, "fixed")
    _compare(rx.match_first_fixed(p, d, length, base * times), want_first, times, "first fixed")
