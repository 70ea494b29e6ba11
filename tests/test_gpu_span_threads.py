"""GPU: programs with sets of one width and tables of different sizes, each matched from a thread of its own: the kernel's
LDS limit, which belongs to the process, is the same for all of them."""
import threading

import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import rx

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_sizes_from_several_threads():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    jobs, failed = [], []
    for k in (475, 485, 495, 503):   # sets of sixteen words, all above 64 KiB of tables and text
        pat = b"a[b-d]{%d}e|xyz" % k
        p = rx.compile_regex(pat, search=True).upload()
        rng = np.random.default_rng(k)
        lens = rng.integers(0, 60, 400)
        offs = np.zeros(401, np.int64)
        np.cumsum(lens, out=offs[1:])
        data = np.frombuffer(b"abcdexyz", np.uint8)[rng.integers(0, 8, int(offs[-1]))].copy()
        want = oracle.match(*rx.parse(pat), True, data, offs)
        assert p.info.words == 16 and 0 < want.sum() < 400
        jobs.append((p, torch.from_numpy(data).cuda(), torch.from_numpy(offs).cuda(), want))

    def work(p, d, o, want):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(50):
                    got = rx.match(p, d, o)
                    multi = rx.match_multi([p], d, o)
                s.synchronize()
            assert (got.cpu().numpy() == want).all() and (multi.cpu().numpy()[0] == want).all()
        except Exception as e:   # noqa: BLE001
            failed.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=j) for j in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed
