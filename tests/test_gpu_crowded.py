"""GPU: earliest accepts where nearly every lane of a long string has one (the lanes' minimum is taken without an
atomic for each: those that cannot lower it are left out).  Against the closed form."""
import numpy as np
import pytest

from paper_1108_3126_amd import rx

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("jit", [False, True])
@pytest.mark.parametrize("length,n", [(16_000_000, 1), (2_000_000, 8), (500, 32_768), (191, 70_000), (192, 70_000)])
def test_an_accept_in_every_span(length, n, jit):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    p = rx.compile_regex(b"[0-9]b|ccc", search=True).upload()
    if jit:
        p.jit()
    rng = np.random.default_rng(length)
    text = np.full((n, length), ord("x"), np.uint8)
    text[:, 1::2] = ord("7")
    text[:, 2::2] = ord("b")        # from byte 3 on every other one ends an accept
    lead = rng.integers(0, length // 2, n)
    for i in range(n):
        text[i, :lead[i]] = ord("x")
    want = np.where(lead % 2 == 0, lead + 3, lead + 2)
    want[lead == 0] = 3
    late = rng.random(n) < 0.3     # and strings without one
    text[late] = ord("x")
    want[late] = -1
    d, o = torch.from_numpy(text.ravel()).cuda(), torch.arange(n + 1, dtype=torch.int64, device="cuda") * length
    print(length, n, jit, flush=True)
    np.testing.assert_array_equal(rx.match_first(p, d, o).cpu().numpy(), want)
    np.testing.assert_array_equal(rx.match_first_fixed(p, d, length, n).cpu().numpy(), want)
    if n <= 8:
        for i in range(n):
            assert int(rx.match_first_long(p, d[i * length:(i + 1) * length]).item()) == want[i]
