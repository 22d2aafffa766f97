"""Short sorts where their way changes: keys staged as 32 or 64 bits (ranges of
32 and 33 bits), one pass of one workgroup for ranges of 8 bits beyond 1024
keys, list lengths that are no multiple of four."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


@pytest.mark.parametrize("n", [3, 61, 66, 1023, 1024, 1025, 2047, 4093, 4096])
def test_widths(ctx, n):
    import torch
    rng = np.random.default_rng(n)
    print("case sort widths", n, flush=True)
    for words, begin, width in ((1, 0, 8), (1, 5, 9), (1, 0, 32), (1, 32, 32), (1, 31, 33), (2, 60, 8), (2, 50, 32),
                                (2, 50, 33), (2, 96, 32)):
        keys = rng.integers(0, 1 << 63, size=(n, words), dtype=np.int64).astype(np.uint64) * np.uint64(2)
        keys[rng.integers(0, n, n // 3)] = np.uint64(2 ** 64 - 1)   # the largest value, many times
        big = [int(k[0]) + (int(k[1]) << 64 if words == 2 else 0) for k in keys]
        want = keys[sorted(range(n), key=lambda i: (big[i] >> begin) & ((1 << width) - 1))]
        t = torch.from_numpy((keys if words == 2 else keys[:, 0]).copy().view(np.int64)).cuda()
        assert ctx.keys_sort(t, begin_bit=begin, end_bit=begin + width) == n
        got = t.cpu().numpy().view(np.uint64).reshape(n, words)
        assert np.array_equal(got, want), (words, begin, width)
