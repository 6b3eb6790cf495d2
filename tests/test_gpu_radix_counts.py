"""The radix sort where the count, which only the device knows, decides how a pass
runs: threads that share a digit's rows (past 16 tiles of 2048 keys, digits of up
to 9 bits), histograms of groups of tiles (past 48 and 128 rows to a thread),
blocks of one, two and four rows of keys (bounds above 2^20).  And the time that
it takes where most of the bound is there, or little."""
import ctypes as C

import pytest
import torch

from test_gpu_radix_sort import SMALL, lib, run  # noqa: F401 (lib: the fixture)

pytestmark = pytest.mark.gpu
TILE = 2048


@pytest.mark.parametrize("lo,hi", [(0, 32), (0, 11), (3, 13), (0, 9), (0, 7), (0, 2)])
@pytest.mark.parametrize("tiles", [16, 17, 48, 49, 64, 128, 129, 200])
def test_tiles(lib, tiles, lo, hi):  # noqa: F811
    for n in (TILE * tiles - 1, TILE * tiles, TILE * tiles + 1):
        run(lib, n, n, SMALL, lo, hi, "random", n)
    run(lib, TILE * tiles - 777, 1 << 19, SMALL, lo, hi, "few", tiles)   # the count below the bound


@pytest.mark.parametrize("n", [1, 1000, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 19) - 1, 1 << 19, (1 << 19) + 1,
                               (1 << 20) + 7])
def test_rows(lib, n):  # noqa: F811
    run(lib, n, (1 << 20) + 7, 0, 0, 32, "random", n)
    run(lib, n, (1 << 20) + 7, 0, 5, 16, "few", n)


def best_us(lib, n, n_max, small_max):  # noqa: F811
    sort, temp = lib
    bufs = [torch.randint(0, 1 << 30, (n_max,), dtype=torch.int32, device="cuda") for _ in range(4)]
    tmp = torch.empty(temp(n_max, small_max), dtype=torch.uint8, device="cuda")
    n_dev, alt = torch.tensor([n], dtype=torch.int32, device="cuda"), C.c_bool(False)
    stream = torch.cuda.current_stream().cuda_stream
    best = 1e9
    for _ in range(12):
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        for _ in range(20):
            sort(*[b.data_ptr() for b in bufs], n_dev.data_ptr(), n_max, small_max, 0, 32, tmp.data_ptr(), stream,
                 C.byref(alt))
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, e[0].elapsed_time(e[1]) * 50.0)
    return best


def test_the_form_of_fewest_launches_holds_for_any_count(lib):  # noqa: F811
    # all of 2^19 ids: 71 us against the next form's 68; 122 where every block
    # of the scatter reads the histograms of all
    small, rows = best_us(lib, 1 << 19, 1 << 19, SMALL), best_us(lib, 1 << 19, 1 << 19, 0)
    print(f"  2^19 of 2^19: {small:.1f} us, {rows:.1f} in the next form", flush=True)
    assert small < 1.4 * rows


def test_a_large_bound_with_few_keys(lib):  # noqa: F811
    # 84k of 2^22 ids: 47 us, as with a bound of 2^20 (45); 61 with blocks of 4096 keys
    large, middle = best_us(lib, 84000, 1 << 22, 0), best_us(lib, 84000, 1 << 20, 0)
    print(f"  84k of 2^22: {large:.1f} us, of 2^20 {middle:.1f}", flush=True)
    assert large < 1.2 * middle
