"""One long string runs over spans before the chunk-parallel kernels, which do nothing where the spans have the result.
What the spans found is kept in the call's own workspace, behind the rows or maps: no other call can write it between
the two chunk-parallel kernels (kept in an array that calls share, the second could compose what the first, which saw
the result there, never wrote)."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import rx

def _need(p, length, chunks=0):
    n = ctypes.c_size_t()
    assert rx.lib().rx_match_long_workspace(p.handle, length, chunks, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.gpu
@pytest.mark.parametrize("jit", [False, True])
@pytest.mark.parametrize("length", [5_000, 200_000])
def test_finding_stays_in_the_workspace(jit, length):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = rx.compile_regex(b"a[g-z]*b|cdecdec", search=True).upload()
    tree = rx.parse(b"a[g-z]*b|cdecdec")
    if jit:
        p.jit()
    need, s = _need(p, length), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    for edits, lives in (((), False), (((100, b"a"),), True), (((100, b"a"), (length - 1, b"b")), True), (((length - 7, b"cdecdec"),), False)):
        text = np.full(length, ord("x"), np.uint8)
        for at, w in edits:
            text[at:at + len(w)] = np.frombuffer(w, np.uint8)
        want = int(oracle.match(*tree, True, text, np.array([0, length]))[0])
        end = {0: -1, 1: length}[want]
        d = torch.from_numpy(text).cuda()
        for first in (False, True):
            print(jit, length, edits, first, flush=True)
            work = torch.full((need + 64,), 0x5a, dtype=torch.uint8, device="cuda")
            out = torch.zeros(1, dtype=torch.int64 if first else torch.uint8, device="cuda")
            f = rx.lib().rx_match_first_long if first else rx.lib().rx_match_long
            assert f(p.handle, ctypes.c_void_p(d.data_ptr()), length, 0, ctypes.c_void_p(work.data_ptr()), need,
                     ctypes.c_void_p(out.data_ptr()), s) == 0
            assert int(out.item()) == (end if first else want)
            w = work.cpu().numpy()
            assert (w[need:] == 0x5a).all()
            if not lives:   # one word, and the chunk-parallel kernels wrote nothing
                at = np.nonzero(w[:need] != 0x5a)[0]
                assert at.size == 8 and at[0] % 8 == 0 and w[at].tobytes() == b"\2" + b"\0" * 7
