"""rx_match's layout check: id and finding are one word of the slot that calls share (as separate words, a reader could
take one from one call and one from another), and everything else comes from the call's own offsets.  Batches large
enough for the check, of a program that runs over spans and of one that does not, with the circuit compiled."""
import re

import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import rx
from paper_1108_3126_amd import workloads as W


def test_twin_reads_one_word_of_the_slot():
    t = W.single_program(1)
    src = rx.compile(t.ast, t.root, t.classes, True).jit_source()
    for name in ("rx_sliced_offsets_skew", "rx_sliced_offsets_skew_w"):
        body = src[src.index(f"void {name}("):]
        body = body[:body.index("\n}")]
        assert not re.search(r"\bslot\s*\[", body)
        assert len(re.findall(r"__hip_atomic_load\(slot,", body)) == 1


@pytest.fixture(scope="module")
def progs():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    t = W.single_program(1)
    out = {}
    for search in (True, False):
        p = rx.compile(t.ast, t.root, t.classes, search).upload()
        out[search] = (p.jit(), (t.ast, t.root, t.classes, search), t)
    # anchored: whole strings of lower-case letters but one, where random strings often match
    ast, root, classes = rx.parse(b"[a-y]*z?[a-y]*")
    out["anchored"] = (rx.compile(ast, root, classes, False).upload().jit(), (ast, root, classes, False), None)
    return out


BASE = 4096


def _batch(t, n, length, flaw, shift):
    """n strings: BASE distinct ones over and over.  flaw: a string one byte longer in the middle."""
    if t is None:
        rng = np.random.default_rng(length)
        base = rng.integers(97, 123, BASE * length).astype(np.uint8)
        base[base == 122] = np.where(rng.random(int((base == 122).sum())) < 0.3, 122, 97)
    else:
        base = W.single_strings(t, seed=length, n=BASE, length=length, plant_frac=0.1)[0].data
    data = np.tile(base, -(-n // BASE))[:n * length]
    offs = np.arange(n + 1, dtype=np.int64) * length
    if flaw:
        k = n // 2 + 5
        data = np.insert(data, offs[k + 1], 0x7a)
        offs[k + 1:] += 1
    return np.concatenate([np.full(shift, 0x7a, np.uint8), data]), offs + shift


@pytest.mark.gpu
@pytest.mark.parametrize("which,n", [(True, 524_288), (True, 600_001), (False, 16_384), ("anchored", 16_384), ("anchored", 100_001)])
@pytest.mark.parametrize("length,flaw,shift", [(16, False, 0), (64, False, 0), (64, True, 0), (64, False, 256), (64, False, 1), (48, False, 0)])
def test_equal_lengths_and_flaws(progs, which, n, length, flaw, shift):
    import torch

    p, (ast, root, classes, search), t = progs[which]
    data, offs = _batch(t, n, length, flaw, shift)
    print(which, n, length, flaw, shift, flush=True)
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda()
    got = rx.match(p, d, o).cpu().numpy()
    idx = np.unique(np.concatenate([np.arange(BASE), np.arange(n // 2 - 50, n // 2 + 50), np.arange(n - 100, n)])).astype(np.int64)
    want = oracle.match(ast, root, classes, search, data, offs, index=idx)
    if which is not False:
        assert 0 < want.sum() < len(want)
    np.testing.assert_array_equal(got[idx], want)
    np.testing.assert_array_equal(got, rx.match(p, d, o, launch=(rx.VARIANT_LANE, 0, 0, 0)).cpu().numpy())


@pytest.mark.gpu
def test_slots_wrap_for_a_program_without_spans(progs):
    """More calls than slots, equal-length and uneven batches in turn, and a captured call (its id stays the same)
    replayed among them."""
    import torch

    p, (ast, root, classes, search), _ = progs["anchored"]
    n = 16_384
    a, oa = _batch(None, n, 16, False, 0)
    b, ob = _batch(None, n, 16, True, 0)
    want = [oracle.match(ast, root, classes, search, x, o) for x, o in ((a, oa), (b, ob))]
    dev = [(torch.from_numpy(x).cuda(), torch.from_numpy(o).cuda()) for x, o in ((a, oa), (b, ob))]
    side = torch.cuda.Stream()
    rec = torch.zeros(n, dtype=torch.uint8, device="cuda")
    rx.match(p, *dev[0], out=rec)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        rx.match(p, *dev[0], out=rec)
    calls = 4200
    out = torch.empty((calls, n), dtype=torch.uint8, device="cuda")
    seen = []
    for k in range(calls):
        rx.match(p, *dev[k % 2], out=out[k])
        if k % 500 == 0:
            rec.fill_(7)
            torch.cuda.synchronize()
            with torch.cuda.stream(side):
                g.replay()
            rx.match(p, *dev[0], out=out[k if k % 2 == 0 else k - 1])
            torch.cuda.synchronize()
            seen.append(rec.cpu().numpy())
    got = out.cpu().numpy()
    for r in seen:
        np.testing.assert_array_equal(r, want[0])
    assert (got[0::2] == want[0]).all() and (got[1::2] == want[1]).all()
    assert 0 < want[0].sum() < n
