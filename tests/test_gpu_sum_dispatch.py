"""The coherent sum's large tiles against its small ones, with the rule that
chooses them asked in the test: a receiver's result is the same bits from a
channel of thousands of receivers (large tiles) and from one of its own few
(small tiles), also where a contraction is longer than 512."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
BIG = 16384


@pytest.fixture(scope="module")
def ctx():
    from paper_2402_13034_amd import risrt
    with risrt.Context(0) as c:
        yield c


@pytest.fixture(scope="module")
def small_tiles(tmp_path_factory):
    """The library's own rule, compiled for the host."""
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rule.cpp", d / "rule.so"
    src.write_text('#include "%s"\nextern "C" int small(long long R, long long C, long long k, int three, int cus) '
                   '{ return rt::small_tiles(R, C, k, three != 0, cus); }\n'
                   % os.path.join(HERE, "..", "paper_2402_13034_amd", "csrc", "rt_rules.hpp"))
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", str(so), str(src)])
    f = ctypes.CDLL(str(so)).small
    f.argtypes = [ctypes.c_longlong] * 3 + [ctypes.c_int] * 2
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return lambda R, C, k, three: bool(f(R, C, k, three, cus))


def _bits(x):
    b = np.ascontiguousarray(x).view(np.uint32).copy()
    b[np.isnan(x.view(np.float32))] = 0x7fc00000
    return b


def _sum(ctx, ch, G, real, prec):
    import torch
    E, P = ctx.ris_sum(ch, torch.from_numpy(np.ascontiguousarray(G)).cuda(), scale=0.7, gamma_is_real=real,
                       precision=prec, want_E=True, want_P=True)
    torch.cuda.synchronize()
    return E.cpu().numpy(), P.cpu().numpy()


# contractions of one element to several chunks of 64 and a rest, below and above 512 (331 and 600 elements)
@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("R,M", [(1, 1), (64, 9), (63, 31), (129, 64), (70, 100), (65, 331), (64, 600)])
def test_large_equals_small(ctx, small_tiles, R, M, real):
    rng = np.random.default_rng(R * 1000 + M)
    C = 600
    H = rng.normal(size=(BIG, 2 * M)).astype(np.float32).view(np.complex64)
    H *= (10 ** rng.uniform(-7, -5, (BIG, 1))).astype(np.float32)
    E_env = (rng.normal(size=(BIG, 2)) * 1e-6).astype(np.float32).view(np.complex64)[:, 0]
    G = (rng.normal(size=(M, C)) + (0 if real else 1j) * rng.normal(size=(M, C))).astype(np.complex64)
    wild = G[:, 200:300]
    wild[rng.integers(0, M, 40), rng.integers(0, 100, 40)] = rng.choice(
        np.array([1e-40, -3e-42, 3.39e38, -0.0, np.inf, np.nan, 65520.0, 1e-7, 1 + 2.0 ** -9], np.float32), 40)
    big, few = ctx.channel_create(E_env, H), ctx.channel_create(E_env[:R], H[:R])
    print("case sum dispatch", R, M, real, flush=True)
    k = M if real else 2 * M
    for prec in (1, 2, 3):
        assert not small_tiles(BIG, C, k, prec == 2)
        E, P = _sum(ctx, big, G, real, prec)
        for c0, n in ((0, 1), (3, 31), (0, 32), (7, 33), (1, 64), (0, 65), (200, 100)):
            assert small_tiles(R, n, k, prec == 2)
            e, p = _sum(ctx, few, G[:, c0:c0 + n], real, prec)
            assert np.array_equal(_bits(e), _bits(E[:R, c0:c0 + n])), (prec, c0, n)
            assert np.array_equal(_bits(p), _bits(P[:R, c0:c0 + n])), (prec, c0, n)
    ctx.destroy(big)
    ctx.destroy(few)
