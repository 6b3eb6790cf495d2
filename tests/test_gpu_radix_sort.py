"""The radix sort's three forms (two launches a pass with digits of up to 11
bits; three with up to 8, 1024 or 4096 keys to a block), called directly,
against torch's stable sort: counts around blocks of 1024, 2048 and 4096 keys
and around the forms' bounds, the count on the device below the bound, key bits
from 1 to 32 and not from bit 0, keys that are random, all equal, or few."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2511_16144_amd import binding as B
    h = C.CDLL(B.LIB_PATH)
    sort = h._ZN3lgs14radix_sort_u32EPjS0_S0_S0_PKjlliiPvP12ihipStream_tPb
    sort.argtypes = [C.c_void_p] * 5 + [C.c_int64, C.c_int64, C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p]
    sort.restype = None
    temp = h._ZN3lgs16radix_temp_bytesEll
    temp.argtypes, temp.restype = [C.c_int64, C.c_int64], C.c_size_t
    return sort, temp


def run(lib, n, n_max, small_max, lo, hi, kind, seed):
    sort, temp = lib
    rng = np.random.default_rng(seed)
    k = {"random": lambda: rng.integers(0, 2**32, n_max, dtype=np.uint32),
         "equal": lambda: np.full(n_max, 0x5a5a5a5a, np.uint32),
         "few": lambda: rng.choice(np.uint32([0, 1, 7, 0x80000000, 0xffffffff, 0x7f]), n_max)}[kind]()
    keys = torch.from_numpy(k.view(np.int32)).cuda()
    guard = 64
    bufs = [torch.full((n_max + guard,), -7, dtype=torch.int32, device="cuda") for _ in range(4)]
    bufs[0][:n_max] = keys
    bufs[1][:n_max] = torch.arange(n_max, dtype=torch.int32, device="cuda")
    tmp = torch.empty(temp(n_max, small_max) + 4 * guard, dtype=torch.uint8, device="cuda").fill_(0xee)
    n_dev = torch.tensor([n], dtype=torch.int32, device="cuda")
    alt = C.c_bool(False)
    sort(bufs[0].data_ptr(), bufs[1].data_ptr(), bufs[2].data_ptr(), bufs[3].data_ptr(),
         None if n == n_max else n_dev.data_ptr(), n_max, small_max, lo, hi, tmp.data_ptr(),
         torch.cuda.current_stream().cuda_stream, C.byref(alt))
    torch.cuda.synchronize()
    ok, ov = (bufs[2], bufs[3]) if alt.value else (bufs[0], bufs[1])
    d = (k[:n].astype(np.int64) >> lo) & ((1 << (hi - lo)) - 1)
    order = np.argsort(d, kind="stable")
    assert np.array_equal(ov[:n].cpu().numpy(), order.astype(np.int32))
    assert np.array_equal(ok[:n].cpu().numpy().view(np.uint32), k[:n][order])
    for b in bufs:
        assert bool((b[n_max:] == -7).all())
    assert bool((tmp[-4 * guard:] == 0xee).all())


SMALL, ROWS = 1 << 30, 0   # every count takes the small form / none does


@pytest.mark.parametrize("small_max", [SMALL, ROWS])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 20001])
def test_counts(lib, n, small_max):
    for kind in ("random", "equal", "few"):
        run(lib, n, n, small_max, 0, 32, kind, n)
        run(lib, n, 3 * n + 5000, small_max, 0, 32, kind, n)   # the count on the device, below the bound


@pytest.mark.parametrize("small_max", [SMALL, ROWS])
@pytest.mark.parametrize("lo,hi", [(0, 1), (0, 2), (0, 3), (0, 6), (0, 8), (0, 9), (0, 11), (0, 12), (0, 17), (0, 23),
                                   (3, 9), (5, 32)])
def test_bits(lib, lo, hi, small_max):
    for kind in ("random", "few"):
        run(lib, 9001, 9001, small_max, lo, hi, kind, hi)


@pytest.mark.parametrize("n", [(1 << 17) - 1, 1 << 17, (1 << 17) + 1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 3000001])
def test_bounds(lib, n):
    run(lib, n, n, 1 << 17, 0, 32, "random", 1)
    run(lib, n, n, 1 << 17, 0, 11, "few", 2)
    run(lib, n // 9, n, 1 << 19, 0, 32, "random", 3)


def test_none(lib):
    run(lib, 0, 5000, SMALL, 0, 32, "random", 1)
    run(lib, 0, 5000, ROWS, 0, 32, "random", 1)
