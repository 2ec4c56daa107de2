"""What the library does once for every device (csrc/device_once.h), on the host: by several threads, after failures, for devices that it
has no place for."""
from concurrent.futures import ThreadPoolExecutor

from tests.host_plan import host_library

SOURCE = r"""
#include "device_once.h"
static std::atomic<uint64_t> done{0};
static std::atomic<int> calls[64];
extern "C" int once(int device, int succeed) {
    return metok::once_per_device(done, device, [&] { calls[device].fetch_add(1); return succeed != 0; });
}
extern "C" int calls_of(int device) { return calls[device]; }
"""


def test_once_for_every_device():
    lib = host_library(SOURCE)
    assert not lib.once(5, 0) and not lib.once(5, 0) and lib.calls_of(5) == 2          # a failure is tried again
    assert lib.once(5, 1) and lib.once(5, 0) and lib.calls_of(5) == 3                  # a success is not
    assert not lib.once(-1, 1) and not lib.once(64, 1)
    with ThreadPoolExecutor(8) as pool:
        assert all(pool.map(lambda i: lib.once(i % 5 if i % 2 else 63 - i % 50, 1), range(4000)))
    before = [lib.calls_of(d) for d in range(64)]
    assert all(lib.once(d, 0) for d in (0, 1, 2, 3, 4, 63, 15)) and before == [lib.calls_of(d) for d in range(64)]
    assert max(before) <= 8
