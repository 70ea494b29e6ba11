"""The circuit's new state words are all computed from the old ones: an update that is another word as it was (after a
leaf that every byte moves on) must not see that word's new value.  The generated step on the CPU against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1108_3126_amd import rx
from test_jit_cpu import cpu_circuit


@pytest.mark.parametrize("search", [True, False])
@pytest.mark.parametrize("pattern", [b"ab{2}c|c.a.b{4}", b"a..b|c...a", b"(a.|.b)*..c", b"a.{5}b.{3}"])
def test_words_that_any_byte_moves(pattern, search):
    ast, root, classes = rx.parse(pattern)
    p = rx.compile(ast, root, classes, search=search)
    rng = np.random.default_rng(len(pattern))
    for length in (4, 11, 64):
        data = np.frombuffer(b"abc", np.uint8)[rng.integers(0, 3, 512 * length)]
        want = oracle.match(ast, root, classes, search, data, np.arange(513, dtype=np.int64) * length)
        np.testing.assert_array_equal(cpu_circuit(p)(data, length, 512), want)
