"""condense_layer's library calls as Python makes them.  A process of its own loads a library in front of libsrigl that forwards them: it can report an error
behind a launch, and notes what stands in the pinned memory when the call comes back and whether the interpreter's lock was held."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

FRONT_OF_THE_LIBRARY = r"""
#include <dlfcn.h>
#include "srigl.h"
static void* lib;
static int (*lock_held)();   // PyGILState_Check
static int calls_with_lock, calls;
static int fail_count, fail_write;
static const void* words;
static size_t n_words;
static const srigl_report* report;
extern "C" void forward_to(const char* path) { lib = dlopen(path, RTLD_NOW); lock_held = (int (*)())dlsym(RTLD_DEFAULT, "PyGILState_Check"); }
extern "C" int with_lock() { return lock_held ? calls_with_lock : -1; }
extern "C" int made() { return calls; }
extern "C" void fail_behind(int count, int write) { fail_count = count; fail_write = write; }
// words of the last call's counts that are still missing; the last report's status
extern "C" int missing() { int n = 0; for (size_t i = 0; i < n_words; ++i) n += (__atomic_load_n((const unsigned long long*)words + i, __ATOMIC_ACQUIRE) >> 63) == 0; return n; }
extern "C" int status() { return report ? __atomic_load_n(&report->status, __ATOMIC_ACQUIRE) : -1; }
extern "C" srigl_status srigl_condense_count(const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, void* ws, size_t ws_bytes, void* counts, size_t bytes, void* st) {
    ++calls; calls_with_lock += lock_held();
    words = counts; n_words = counts ? bytes / 8 : 0;
    const srigl_status rc = ((decltype(&srigl_condense_count))dlsym(lib, "srigl_condense_count"))(mask, d_out, d_in, K, ws, ws_bytes, counts, bytes, st);
    return rc == SRIGL_OK && fail_count ? SRIGL_ERR_HIP : rc;
}
#define WRITES(NAME) \
extern "C" srigl_status NAME(const void* W, srigl_dtype t, const uint8_t* mask, int32_t d_out, int32_t d_in, int32_t K, int32_t cap, void* W_c, int32_t* idx, int32_t* active, \
                             uint16_t* seg, void* packed, size_t bytes, void* ws, size_t ws_bytes, srigl_report* rep, void* st) { \
    ++calls; calls_with_lock += lock_held(); \
    report = rep; \
    const srigl_status rc = ((decltype(&NAME))dlsym(lib, #NAME))(W, t, mask, d_out, d_in, K, cap, W_c, idx, active, seg, packed, bytes, ws, ws_bytes, rep, st); \
    return rc == SRIGL_OK && fail_write ? SRIGL_ERR_HIP : rc; \
}
WRITES(srigl_condense_write)
WRITES(srigl_condense)
"""

PROGRAM = r"""
import ctypes, os, sys
import torch                                                   # (the library takes the HIP runtime that torch has loaded)
front = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the package, whose calls then come here
front.forward_to(os.path.join(sys.argv[2], "paper_2305_02299_amd", "libsrigl.so").encode())
sys.path[:0] = [sys.argv[2], os.path.join(sys.argv[2], "tests")]
import synth_inputs as si
from gpu_util import dev
from paper_2305_02299_amd import binding as B_, condense_layer

def layer(d_out, d_in, K):
    L = si.make_layer(d_in, d_out, K, 1, ablate_frac=0.25, seed=d_out)
    return dev(L.W), dev(L.mask), K

def behind_work(*args):
    torch.cuda._sleep(50_000_000)                               # some 20 ms of work ahead in the stream
    try:
        return condense_layer(*args).n_active
    except B_.SriglError as e:
        return e.status
"""


def run(tmp_path, body):
    src, lib = tmp_path / "front.cpp", tmp_path / "front.so"
    src.write_text(FRONT_OF_THE_LIBRARY)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-o", str(lib), str(src), "-ldl"], check=True)
    r = subprocess.run([sys.executable, "-c", PROGRAM + body + "\nprint('calls ok', flush=True)", str(lib), ROOT], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "calls ok" in r.stdout, (r.stdout + r.stderr)[-1500:]


def test_an_error_behind_a_launch_does_not_give_the_memory_back(tmp_path):
    """A small layer, whose counts the first launch writes, and one whose report the second writes."""
    run(tmp_path, """
small, large = layer(700, 96, 9), layer(2100, 4096, 40)
assert behind_work(*small) == 525 and front.missing() == 0 and behind_work(*large) == 1575 and front.status() == B_.OK
for args, count, write in ((small, 1, 0), (small, 0, 1), (large, 0, 1)):
    front.fail_behind(count, write)
    assert behind_work(*args) == B_.ERR_HIP
    assert front.missing() == 0 and (args is small or front.status() == B_.OK), (count, write, front.missing(), front.status())
    torch.cuda.synchronize()
    front.fail_behind(0, 0)
    assert behind_work(*args) == args[1].shape[0] * 3 // 4
""")


def test_the_library_is_called_without_the_interpreters_lock(tmp_path):
    """All launches: on a stream whose queue is full a launch takes as long as the queue."""
    run(tmp_path, """
for d_out, d_in in ((700, 96), (2100, 4096)):
    assert behind_work(*layer(d_out, d_in, 9)) == d_out * 3 // 4
assert front.made() == 3 and front.with_lock() == 0, (front.made(), front.with_lock())
""")


def test_threads_on_streams_of_their_own():
    """Calls that wait on the host while others launch: every thread's layers are its own, with work ahead in its stream."""
    import threading

    import numpy as np
    import torch

    import oracle
    import synth_inputs as si
    from gpu_util import dev, host
    from paper_2305_02299_amd import condense_layer
    sizes = [(70, 33, 4), (700, 96, 9), (3072, 64, 6), (2100, 4096, 20)]      # (the last one's report comes from the second launch)
    layers = [si.make_layer(d_in, d_out, K, 1, ablate_frac=0.3, seed=d_out) for d_out, d_in, K in sizes]
    wanted = [oracle.condense(L.W, L.mask, L.K) for L in layers]
    inputs = [(dev(L.W), dev(L.mask), L.K) for L in layers]
    torch.cuda.synchronize()
    wrong = []

    def work(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(8):
                which = (t + i) % len(sizes)
                torch.cuda._sleep(2_000_000)
                got = condense_layer(*inputs[which])
                W_c, idx, active = wanted[which]
                if not (np.array_equal(host(got.active), active) and np.array_equal(host(got.idx), idx) and np.array_equal(host(got.W_c), W_c)):
                    wrong.append((t, i, which))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join(100)
    assert not any(th.is_alive() for th in threads) and not wrong, wrong
