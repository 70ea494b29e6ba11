"""The span kernels (a searched program over equal spans of bytes) on the CPU: the circuit's generated source
(rx_spans, the text that hiprtc compiles) and the table form (span_regions) run by tests/lockstep.h, every thread a
fiber, against the oracle.  Strings that begin and end anywhere, empty ones, unaligned starts, threads that outlive
their span, the region's last lane and the staged text; several workgroups; both kinds of result.  The text lies
against an unreadable page, and words past the kernel's LDS are checked."""
import ctypes
import functools
import os
import subprocess
import tempfile

import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import rx
from paper_1108_3126_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(rx.__file__), "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

PREAMBLE = '#include "lockstep.h"\n#include <sys/mman.h>\n#include <cstring>\n'

# the text's bytes, the last 16-byte block that holds any of them against an unreadable page
TEXT = r"""
struct Guarded {
    unsigned char *map, *bytes;
    size_t size;
    Guarded(const unsigned char* data, size_t n, size_t skew) {
        const size_t body = (n + skew + 15) / 16 * 16;
        size = (body + 4095) / 4096 * 4096 + 4096;
        map = (unsigned char*)mmap(nullptr, size, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
        bytes = map + size - 4096 - body + skew;
        memcpy(bytes, data, n);
        mprotect(map + size - 4096, 4096, PROT_NONE);
    }
    ~Guarded() { munmap(map, size); }
};
"""

CIRCUIT_DRIVER = r"""
extern "C" int run_spans(const unsigned char* data, long long nbytes, int skew, const long long* offsets, long long stride,
                         long long n, unsigned char* out, long long* first, const u32* first_row, const u32* follow,
                         const u32* bytemask, int prefix, int grid, long long* undone, long long limit) {
    Guarded text(data, nbytes, skew);
    rx_span_text X = {};
    X.bytes = text.bytes;
    X.offsets = offsets;
    X.stride = stride;
    X.n = n;
    X.out = out;
    X.first = first;
    X.first_row = first_row;
    X.follow = follow;
    X.bytemask = bytemask;
    X.prefix = prefix;
    X.undone = undone;
    lockstep::grid = grid;
    for (lockstep::block = 0; lockstep::block < grid; ++lockstep::block) {
        for (u32& x : rx_sp) x = 0x5a5a5a5au;
        lockstep::run(64, [&] { rx_spans(X); });
        for (int i = RX_LDS; i < RX_LDS + 64; ++i)
            if (rx_sp[i] != 0x5a5a5a5au) return 1;
    }
    return 0;
}
"""

TABLE_DRIVER = r"""
#include "rx_spans.h"
alignas(16) static uint32_t lds[rx::span_lds_words(RX_W, 32 * RX_W, RX_T) + 64];
extern "C" int run_spans(const unsigned char* data, long long nbytes, int skew, const int64_t* offsets, long long stride,
                         long long n, unsigned char* out, int64_t* first, const uint32_t* first_row,
                         const uint32_t* follow, const uint32_t* bytemask, int L, int prefix, int B, int grid,
                         int64_t* undone, long long limit) {
    Guarded text(data, nbytes, skew);
    rx::SpanProg P = {first_row, follow, bytemask, L, prefix};
    rx::SpanText X = {text.bytes, offsets, stride, n};
    rx::SpanOut O = {out, first, undone, limit};
    const int64_t o0 = offsets ? offsets[0] : 0, oN = offsets ? offsets[n] : n * stride;
    if (oN <= o0) return 0;
    const int64_t regions = (oN - o0 + 15 + RX_T * B - 1) / (RX_T * B), per = (regions + grid - 1) / grid;
    constexpr int WP = rx::span_row_words(RX_W);
    const int words = rx::span_lds_words(RX_W, L, RX_T);
    for (int64_t r0 = 0; r0 < regions; r0 += per) {
        for (uint32_t& x : lds) x = 0x5a5a5a5au;
        const int64_t r1 = r0 + per < regions ? r0 + per : regions;
        uint32_t *M = lds, *N = M + 256 * WP, *F = N + 257 * WP;
        lockstep::run(RX_T, [&] {
            rx::span_tables<RX_W, RX_T>(P, M, N, F);
            if (first)
                rx::span_regions<RX_W, RX_T, true>(P, X, O, o0, oN, B, r0, r1, M, N, F, F + L * WP);
            else
                rx::span_regions<RX_W, RX_T, false>(P, X, O, o0, oN, B, r0, r1, M, N, F, F + L * WP);
        });
        for (int i = words; i < words + 64; ++i)
            if (lds[i] != 0x5a5a5a5au) return 1;
    }
    return 0;
}
"""


def _build(code):
    d = tempfile.mkdtemp(prefix="rxspans")
    cpp, so = os.path.join(d, "c.cpp"), os.path.join(d, "c.so")
    open(cpp, "w").write(code)
    subprocess.check_call([CLANG, "-O1", "-std=c++17", "-shared", "-fPIC", "-w", f"-I{HERE}", f"-I{CSRC}", "-o", so, cpp])
    return ctypes.CDLL(so)


def _prefix(first, follow, mask, L):
    """The rank of the search prefix's any-byte leaf: every byte keeps it, its image is First."""
    for r in range(L):
        if np.array_equal(follow[r], first) and all((mask[c][r >> 5] >> (r & 31)) & 1 for c in range(256)):
            return r
    raise AssertionError("no prefix leaf")


@functools.lru_cache(maxsize=None)
def _lib(kind, key):
    if kind == "circuit":
        return _build(PREAMBLE + "#define RX_LDS 10240\n" + key.replace("extern __shared__ u32 rx_sp[];", "")
                      .replace("__attribute__((amdgpu_waves_per_eu(1, 1)))", "")
                      .replace("typedef unsigned int u32;", "typedef unsigned int u32;\nalignas(16) static u32 rx_sp[RX_LDS + 64];", 1)
                      + TEXT + CIRCUIT_DRIVER)
    return _build(PREAMBLE + f"#define RX_W {key}\n#define RX_T 128\n" + TEXT + TABLE_DRIVER)


_ptr = lambda a: None if a is None else ctypes.c_void_p(a.ctypes.data)


def run(kind, p, data, offs=None, stride=0, n=None, first=False, skew=0, grid=1, B=16, limit=None):
    """(results, undone) of a kind of span kernel on strings data[offs[i]:offs[i + 1]] or of one length."""
    frow, follow, mask, _ = p.sets()
    L = p.info.n_leaves
    n = len(offs) - 1 if offs is not None else n
    res = np.full(n, -1, np.int64) if first else np.zeros(n, np.uint8)
    undone = np.zeros(1, np.int64)
    src = p.jit_spans_source() if kind == "circuit" else p.info.words
    assert src
    f = _lib(kind, src).run_spans
    ll = ctypes.c_longlong
    frow, follow, mask = (np.ascontiguousarray(x, np.uint32) for x in (frow, follow, mask))
    u = _ptr(undone) if limit is not None else None
    head = [_ptr(data), ll(data.size), skew, _ptr(offs), ll(stride), ll(n), None if first else _ptr(res), _ptr(res) if first else None,
            _ptr(frow), _ptr(follow), _ptr(mask)]
    prefix = _prefix(frow, follow, mask, L)
    rc = f(*head, prefix, grid, u, ll(limit or 0)) if kind == "circuit" else f(*head, L, prefix, B, grid, u, ll(limit or 0))
    assert rc == 0, "words past the LDS were written"
    return res, int(undone[0])


def earliest(tree, data, offs):
    """The oracle's earliest accepting prefix of every string (see test_gpu_spans.py) and its results."""
    n = len(offs) - 1
    full = oracle.match(*tree, True, data, offs)
    lo, hi = np.zeros(n, np.int64), np.diff(offs)
    while (lo < hi).any():
        mid = (lo + hi) // 2
        po = np.zeros(n + 1, np.int64)
        np.cumsum(mid, out=po[1:])
        pd = np.concatenate([data[offs[i]:offs[i] + mid[i]] for i in range(n)] + [np.zeros(1, np.uint8)])
        m = oracle.match(*tree, True, pd, po).astype(bool)
        hi = np.where(m, mid, hi)
        lo = np.where(m, lo, np.minimum(mid + 1, hi))
    return np.where(full == 1, lo, -1), full


def _program(pattern):
    if isinstance(pattern, bytes):
        tree = rx.parse(pattern)
    else:
        t = W.multi_programs(seed=700 + pattern[0], count=1, lo=pattern[1], hi=pattern[1])[0]
        tree = (t.ast, t.root, t.classes)
    return rx.compile(*tree, search=True), tree


def _text(rng, pattern, offs):
    """Random text, members of the pattern's language in a part of the strings that have room for one."""
    size, lens = int(offs[-1]), np.diff(offs)
    if not isinstance(pattern, bytes):
        return W.zipf_bytes(rng, size)
    rare, member = PATTERNS[pattern]
    alpha = np.frombuffer(b"x" * 300 + b"aabcd" if rare else b"abcd", np.uint8)
    data = alpha[rng.integers(0, len(alpha), size)].copy()
    for i in np.nonzero((lens >= len(member)) & (rng.random(len(lens)) < 0.2))[0]:
        at = offs[i] + rng.integers(0, lens[i] - len(member) + 1)
        data[at:at + len(member)] = np.frombuffer(member, np.uint8)
    return data


# threads that end soon, that live to the string's end, that live on for hundreds of bytes; one, two and more words
# (letters of the pattern are rare in its text, a member)
PATTERNS = {b"ab|ba+c": (False, b"ab"), b"a.*b.*c.*d": (True, b"axbxxcxd"), b"(a|b)*cd": (False, b"cd"),
            b"a{20}[bc]{30}d": (False, b"a" * 20 + b"bc" * 15 + b"d"), b"a[^q]*b|cde": (True, b"cde"),
            b"a.{30}b.{20}c": (True, b"a" + b"x" * 30 + b"b" + b"x" * 20 + b"c"), b"a[g-z]*b|cde": (True, b"cde"),
            b"a[g-z]{2,50}b": (True, b"a" + b"x" * 48 + b"b")}
LENS = [0, 1, 15, 16, 17, 31, 33, 0, 0, 511, 512, 513, 700, 40_000, 5, 0, 32_255, 100, 0]


def _kinds(p):
    return ["table"] + (["circuit"] if p.jit_spans_source() else [])


def test_which_programs_have_a_circuit():
    assert [p for p in PATTERNS if "circuit" not in _kinds(_program(p)[0])] == []
    assert not rx.compile_regex(b"ab", search=False).jit_spans_source()    # anchored
    assert not rx.compile_regex(b"(ab)*", search=True).jit_spans_source()  # matches the empty string


@pytest.mark.parametrize("pattern", [*PATTERNS, (4, 40), (6, 200)], ids=str)
def test_uneven_strings(pattern):
    p, tree = _program(pattern)
    rng = np.random.default_rng(len(str(pattern)))
    for skew, grid in ((0, 1), (3, 2), (13, 3)):
        lens = np.concatenate([rng.permutation(LENS), rng.integers(0, 80, 300), rng.integers(0, 3, 600)])
        offs = np.zeros(len(lens) + 1, np.int64)
        np.cumsum(lens, out=offs[1:])
        data = _text(rng, pattern, offs)
        want_first, want = earliest(tree, data, offs)
        assert 0 < want.sum() < len(want)
        for kind in _kinds(p):
            for B in (16, 32, 64) if kind == "table" else (16,):
                for first, expect in ((False, want), (True, want_first)):
                    got, _ = run(kind, p, data, offs, first=first, skew=skew, grid=grid, B=B)
                    np.testing.assert_array_equal(got, expect, err_msg=f"{kind} skew {skew} B {B} first {first}")


@pytest.mark.parametrize("length,n,skew", [(1, 3000, 0), (7, 3000, 5), (100, 701, 0), (48, 1500, 1), (333, 300, 3), (70_001, 2, 0)])
def test_equal_lengths_without_offsets(length, n, skew):
    p, tree = _program(b"ab{2}c|c.a.b{4}")
    rng = np.random.default_rng(length)
    data = np.frombuffer(b"abcxxx", np.uint8)[rng.integers(0, 6, n * length)]
    want_first, want = earliest(tree, data, np.arange(n + 1, dtype=np.int64) * length)
    for kind in _kinds(p):
        for first, expect in ((False, want), (True, want_first)):
            got, _ = run(kind, p, data, stride=length, n=n, first=first, skew=skew, grid=2, B=32)
            np.testing.assert_array_equal(got, expect, err_msg=kind)


@pytest.mark.parametrize("edits", [(), ((100, b"a"),), ((100, b"a"), (69_999, b"b")), ((100, b"a"), (2_000, b"q"), (50_000, b"b")),
                                   ((5, b"b"), (31_998, b"cde")), ((65_533, b"a"), (65_550, b"b")), ((32_250, b"a"), (32_270, b"b"))])
def test_one_long_string(edits):
    """What a thread that outlives its span by more than the limit does to one string: it is followed, or reported."""
    p, tree = _program(b"a[^q]*b|cde")
    text = np.full(70_000, ord("x"), np.uint8)
    for at, w in edits:
        text[at:at + len(w)] = np.frombuffer(w, np.uint8)
    want_first, want = earliest(tree, text, np.array([0, text.size]))
    lives = any(w == b"a" for _, w in edits) and not (len(edits) == 2 and edits[1][0] - edits[0][0] < 30)
    for kind in _kinds(p):
        for first, expect in ((False, want), (True, want_first)):
            got, _ = run(kind, p, text, stride=text.size, n=1, first=first, B=64)
            np.testing.assert_array_equal(got, expect, err_msg=kind)
            got, undone = run(kind, p, text, stride=text.size, n=1, first=first, B=64, limit=256)
            assert bool(undone) == lives
            if not undone:
                np.testing.assert_array_equal(got, expect, err_msg=kind)


def test_one_long_string_is_given_up_early():
    """The kernels that follow are the faster ones where threads live on: the circuit does not run its whole region."""
    p, tree = _program(b"a[^q]*b|cde")
    for gap, gives_up in ((20, False), (100, True)):
        text = np.full(40_000, ord("x"), np.uint8)
        text[20_000], text[20_000 + gap] = ord("a"), ord("q")
        got, undone = run("circuit", p, text, stride=text.size, n=1, limit=128)
        assert bool(undone) == gives_up and got[0] == 0


@pytest.mark.parametrize("share", [0.0, 0.02, 0.2, 1.0])
@pytest.mark.parametrize("pattern", [b"a[^q]*b", b"a.*b.*c.*d", b"a{2}[^q]{70}[^q]*b", b"a[^q]{40}[^q]*b.{60}c"], ids=str)
def test_few_and_many_threads_that_live_on(pattern, share):
    """Threads that live to their string's end: none, fewer than a workgroup's list holds over its regions, more; sets
    of one to four words and of five (those that are not looked at for standing still)."""
    p, tree = _program(pattern)
    rng = np.random.default_rng([len(pattern), int(100 * share)])
    lens = np.concatenate([rng.integers(100, 400, 60), [5000, 0, 3, 2000]])
    offs = np.zeros(len(lens) + 1, np.int64)
    np.cumsum(lens, out=offs[1:])
    data = np.frombuffer(b"xyzxyzbcdd", np.uint8)[rng.integers(0, 10, int(offs[-1]))].copy()
    data[data == ord("b")] = np.where(rng.random(int((data == ord("b")).sum())) < 0.05, ord("b"), ord("x"))
    for i in np.nonzero(rng.random(len(lens)) < share)[0]:
        if lens[i] > 20:
            data[offs[i] + 10:offs[i] + 12] = ord("a")
    want_first, want = earliest(tree, data, offs)
    for B, grid in ((16, 1), (16, 3), (64, 1)):
        for first, expect in ((False, want), (True, want_first)):
            got, _ = run("table", p, data, offs, first=first, skew=5, grid=grid, B=B)
            np.testing.assert_array_equal(got, expect, err_msg=f"B {B} grid {grid} first {first}")


def test_programs_whose_threads_may_live_on():
    """Five-word sets among them; the oracle on a handful of strings."""
    p, tree = _program(b"a[^q]{150}[^q]*b|cde")
    assert p.info.words >= 5
    rng = np.random.default_rng(5)
    data = np.frombuffer(b"xyzab", np.uint8)[rng.integers(0, 5, 6000)].copy()
    offs = np.array([0, 3000, 3000, 3100, 5900, 6000], np.int64)
    want_first, want = earliest(tree, data, offs)
    for first, expect in ((False, want), (True, want_first)):
        got, _ = run("table", p, data, offs, first=first, B=16)
        np.testing.assert_array_equal(got, expect)
