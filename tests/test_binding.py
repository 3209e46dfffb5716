"""The binding's two marshalling paths: the native module and ctypes."""

import os
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_library_alone_is_enough():
    """Without the native module the binding loads, with a warning, and every call takes the ctypes path."""
    code = """
import sys, warnings
sys.modules["paper_2309_04909_amd._fastcall"] = None
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2309_04909_amd import bicop as B
assert any("_fastcall" in str(w.message) for w in seen), seen
import torch
x, prm, sd = torch.zeros(4, dtype=torch.int64), B.Params(64, 7, 11), B.Seeds(1, 2, 3)
for call in (lambda: B.drelu(x, x, prm, sd), lambda: B.trunc_det(x, x, 64, 13), lambda: B.drelu_send(0, x, prm, sd),
             lambda: B.rss_relu((x, x, x), prm, B.RssSeeds(1, 2, 3, 4, 5))):
    try:
        call()
    except TypeError:
        continue
    raise AssertionError("host tensors were not refused")
print("loaded", B.version())
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "loaded bicop" in r.stdout, r.stderr[-2000:]


SLOW_ALLOCATOR = r"""
#include <stddef.h>
#include <sys/types.h>
#include <unistd.h>
static int (*device_malloc)(void**, size_t);
static int (*device_free)(void*);
extern "C" void slow_setup(void* m, void* f) { device_malloc = (int (*)(void**, size_t))m; device_free = (int (*)(void*))f; }
extern "C" void* slow_alloc(ssize_t size, int, void*) {
    void* p = nullptr;
    usleep(300000);
    return device_malloc(&p, (size_t)size) == 0 ? p : nullptr;
}
extern "C" void slow_free(void* p, ssize_t, int, void*) { device_free(p); }
"""


@pytest.mark.gpu
def test_other_threads_run_while_outputs_are_allocated(tmp_path):
    """Allocating the outputs can wait for the device: the interpreter lock is free meanwhile."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import ctypes
    import threading
    import time
    from graph_kernels import _runtime
    from paper_2309_04909_amd import bicop as B
    src, lib = tmp_path / "slow.cpp", str(tmp_path / "slow.so")
    src.write_text(SLOW_ALLOCATOR)
    subprocess.run(["g++", "-O1", "-fPIC", "-shared", str(src), "-o", lib], check=True, timeout=60)
    x, prm, sd = torch.zeros(1 << 20, dtype=torch.int64, device="cuda"), B.Params(64, 7, 11), B.Seeds(1, 2, 3)
    want = B.drelu(x, x, prm, sd)
    torch.cuda.synchronize()
    hip = _runtime()
    ctypes.CDLL(lib).slow_setup(ctypes.cast(hip.hipMalloc, ctypes.c_void_p), ctypes.cast(hip.hipFree, ctypes.c_void_p))
    allocator = torch.cuda.memory.CUDAPluggableAllocator(lib, "slow_alloc", "slow_free")
    pool = torch.cuda.MemPool(allocator.allocator())
    ticks, stop = [], threading.Event()

    def tick():
        while not stop.is_set():
            ticks.append(time.perf_counter())
            time.sleep(0.002)
    thread = threading.Thread(target=tick)
    with torch.cuda.use_mem_pool(pool):
        thread.start()
        t0 = time.perf_counter()
        got = B.drelu(x, x, prm, sd)
        t1 = time.perf_counter()
        stop.set()
        thread.join()
    assert t1 - t0 > 0.25, "the call did not allocate from the slow pool"
    during = sum(t0 < t < t1 - 0.02 for t in ticks)
    assert during > 20, f"{during} steps of another thread in {t1 - t0:.2f} s"
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    torch.cuda.synchronize()
    # the pool gives its memory back through the allocator: it goes first, while the allocator is alive
    del got
    del pool
    del allocator
