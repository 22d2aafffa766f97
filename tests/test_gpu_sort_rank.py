"""Short sorts by counting: list lengths around a workgroup's 64 keys, an
eighth of the list and the longest list, bit ranges inside a word, across two
words and of a whole word, with few and many equal keys (which keep their
order)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


@pytest.mark.parametrize("n", [2, 7, 8, 9, 63, 64, 65, 127, 511, 512, 513, 1908, 4095, 4096, 4097])
def test_ranges_and_stability(ctx, n):
    import torch
    rng = np.random.default_rng(n)
    print("case rank sort", n, flush=True)
    for words, begin, end in ((1, 0, 64), (1, 32, 52), (1, 22, 46), (1, 63, 64), (2, 0, 64), (2, 64, 127), (2, 64, 128),
                              (2, 60, 100), (2, 107, 120), (2, 40, 104), (2, 0, 105)):
        for spread in (3, 1 << 62):
            keys = rng.integers(0, 1 << 62, size=(n, words), dtype=np.int64).astype(np.uint64) * np.uint64(4)
            keys += rng.integers(0, 4, size=(n, words)).astype(np.uint64)
            big = [int(k[0]) + (int(k[1]) << 64 if words == 2 else 0) for k in keys]
            mask = (1 << (end - begin)) - 1
            if spread == 3:   # few different values of the bits that decide
                pick = [int(x) * (mask // 3) for x in rng.integers(0, 4, n)]
                big = [(b & ~(mask << begin)) | ((p & mask) << begin) for b, p in zip(big, pick)]
                keys = np.array([[(b >> (64 * w)) & (2 ** 64 - 1) for w in range(words)] for b in big], np.uint64)
            want = keys[sorted(range(n), key=lambda i: (big[i] >> begin) & mask)]
            t = torch.from_numpy((keys if words == 2 else keys[:, 0]).copy().view(np.int64)).cuda()
            assert ctx.keys_sort(t, begin_bit=begin, end_bit=end) == n
            got = t.cpu().numpy().view(np.uint64).reshape(n, words)
            assert np.array_equal(got, want), (words, begin, end, spread)
