"""GPU: runs of one byte in the wavefront kernels (a set that a byte maps to itself is left alone to the run's end): runs
that begin and end at every offset of a 16-byte block and of a wavefront's 1,024 bytes, at any buffer alignment, in
strings with and without an accept, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("ws", [0, 1, 2, 16])
@pytest.mark.parametrize("pattern,search", [(b"(((a*)*)*)b", False), (b"((a|aa)*)c", False), (b"x*(ab|ba|a{3})*c?", False),
                                            (b"a.*b.*c", True)])
def test_runs_of_one_byte(pattern, search, ws):
    from paper_1108_3126_amd import rx

    ast, root, classes = rx.parse(pattern)
    p = rx.compile(ast, root, classes, search=search).upload()
    rng = np.random.default_rng(len(pattern))
    strings = []
    for n in (0, 1, 2, 3, 15, 16, 17, 31, 1022, 1023, 1024, 1025, 1040, 2049, 4100):
        for tail in (b"", b"b", b"c", b"ab", b"bc"):
            strings.append(b"a" * n + tail)
            strings.append(b"a" * int(rng.integers(0, 20)) + b"b" * (n // 2) + b"a" * (n - n // 2) + tail)
    s = W.pack(strings)
    want = oracle.match(ast, root, classes, search, s.data, s.offsets)
    buf = torch.zeros(s.data.size + 32, dtype=torch.uint8, device="cuda")
    for shift in (0, 1, 7, 15):
        d = buf[shift:shift + s.data.size]
        d.copy_(torch.from_numpy(s.data))
        got = rx.match(p, d, torch.from_numpy(s.offsets).cuda(), launch=(rx.VARIANT_WAVE, 0, 0, ws)).cpu().numpy()
        np.testing.assert_array_equal(got, want, err_msg=f"{pattern} ws {ws} shift {shift}")


def test_runs_earliest_accepts():
    """The earliest accept in a run, of a program of the wavefront kernels (its set stops changing before the run ends)."""
    from paper_1108_3126_amd import rx

    prog = W.pathological_program("nested", 120)   # 601 nodes, anchored: a^n b
    p = rx.compile(prog.ast, prog.root, prog.classes, False).upload()
    big = W.pathological_program("nested", 600)
    q = rx.compile(big.ast, big.root, big.classes, False).upload()
    strings = [b"a" * n + t for n in (0, 1, 5, 63, 1000, 1025) for t in (b"", b"b", b"ba", b"xb")]
    s = W.pack(strings)
    want = [x.index(b"b") + 1 if b"b" in x and b"x" not in x else -1 for x in strings]
    for r in (p, q):
        got = rx.match_first(r, torch.from_numpy(s.data).cuda(), torch.from_numpy(s.offsets).cuda()).cpu().tolist()
        assert got == want
