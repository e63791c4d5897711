"""The unit tables of a batch fit the buffer that shtn_batch_device_bytes sizes.

Synthesis units lie in one queue per XCD, all padded to the longest, so the size
of a batch's device image depends on how evenly its orders are dealt.  No tiling,
algorithm or polar threshold may make it larger than the size that the caller was
told.  Runs without a GPU: in a process of its own, where a small library stands
in for the HIP calls of an upload and records the bytes of every copy.
"""
import ctypes
import itertools
import os
import random
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HIP_STUB = r"""
#include <stddef.h>
size_t copied;
static int handle;
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream)
{
    if (n > copied) copied = n;
    return 0;
}
int hipLaunchKernel(const void* f, ...) { return 0; }
int hipFuncSetAttribute(const void* f, ...) { return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 1; }
int hipStreamSynchronize(void* s) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = &handle; return 0; }
int hipStreamDestroy(void* s) { return 0; }
int hipStreamBeginCapture(void* s, int mode) { return 0; }
int hipStreamEndCapture(void* s, void** g) { *g = &handle; return 0; }
int hipGraphInstantiate(void** e, void* g, void* a, void* b, size_t n) { *e = &handle; return 0; }
int hipGraphDestroy(void* g) { return 0; }
int hipGraphExecDestroy(void* e) { return 0; }
int hipGraphLaunch(void* e, void* s) { return 0; }
int hipEventCreate(void** e) { *e = &handle; return 0; }
int hipEventDestroy(void* e) { return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipEventSynchronize(void* e) { return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { static int k; *ms = 1.0f + k++ % 7; return 0; }
"""

# plans (lmax, mmax, nlat, nphi) and how many fields each has
BATCHES = [
    # few long orders of many latitudes and many short ones
    [((1023, 2, 1024, 8), 9), ((7, 7, 8, 16), 400)],
    [((2047, 0, 2048, 2), 8)] + [((n, n, n + 1, 256), 1) for n in range(20, 70)],
    # orders that no latitude takes part in once the threshold is raised
    [((300, 300, 4, 1024), 3), ((31, 31, 32, 64), 40)],
    [((63, 63, 64, 128), 1)],
    [((0, 0, 1, 2), 1)],
    [((n, n, n + 1, 256), 2) for n in (15, 31, 63, 100)],
]


def random_batch(rng):
    out = []
    for _ in range(rng.randint(1, 6)):
        lmax = int(2 ** rng.uniform(0, 9))
        mmax = rng.choice([0, lmax, rng.randint(0, lmax)])
        nlat = max(1, rng.choice([lmax + 1, rng.randint(1, 700), 2 * lmax]))
        out.append(((lmax, mmax, nlat, 2 << (2 * mmax).bit_length()), rng.choice([1, 2, 7, 60, 300])))
    return out


def main(stub_path):
    stub = ctypes.CDLL(stub_path, mode=ctypes.RTLD_GLOBAL)  # before the library that calls HIP
    copied = ctypes.c_size_t.in_dll(stub, "copied")
    sys.path.insert(0, ROOT)
    from paper_1202_6522_amd import shtn as S
    rng = random.Random(5)
    tilings = [t for t in itertools.product((1, 2, 4), (1, 2, 4), (0, 1), (0, 1)) if t[0] * t[1] < 16]
    worst = 0.0
    for fields in BATCHES + [random_batch(rng) for _ in range(8)]:
        plans = [S.shtn_plan(*shape) for shape, _ in fields]
        at = itertools.count(1 << 40, 1 << 32)  # addresses of buffers that are never touched
        batch = S.shtn_batch([p for p, (_, n) in zip(plans, fields) for _ in range(n)])
        size = S.shtn_batch_device_bytes(batch)
        for polar in (None, -60, -3):
            for p in plans:
                if polar is not None:
                    S.shtn_plan_set_polar(p, polar)
                S.shtn_plan_upload(p, next(at), None)
            for k, stored in enumerate((0, 1)):
                if stored:
                    S.shtn_ptable_build(plans[0], next(at), S.shtn_ptable_bytes(plans[0]), None)
                    S.check(S.load_library().shtn_batch_set_algorithm(batch, S.SHTN_ALGO_STORED), "set_algorithm")
                for t in (tilings if not stored else rng.sample(tilings, 4)) + [None]:
                    if t:
                        S.shtn_batch_set_tiling(batch, *t)
                    copied.value = 0
                    S.shtn_batch_upload(batch, next(at), None)
                    assert 0 < copied.value <= size, (fields, polar, stored, t, copied.value, size)
                    worst = max(worst, copied.value / size)
                if stored:
                    S.check(S.load_library().shtn_batch_set_algorithm(batch, S.SHTN_ALGO_ONTHEFLY), "set_algorithm")
        S.shtn_batch_destroy(batch)
        for p in plans:
            S.shtn_plan_destroy(p)
    print("largest image over reported size %.3f" % worst)
    lib = S.load_library()

    def tune(batch, size, at):
        # the tuner uploads every candidate
        copied.value = 0
        us = ctypes.c_float()
        rc = lib.shtn_batch_tune(batch, *(ctypes.c_void_p(next(at)) for _ in range(4)), None, 1, None, ctypes.byref(us))
        assert rc == S.SHTN_OK and 0 < copied.value <= size, (rc, copied.value, size)

    for fields in BATCHES:
        plans = [S.shtn_plan(*shape) for shape, _ in fields]
        at = itertools.count(1 << 40, 1 << 36)
        for p in plans:
            S.shtn_plan_upload(p, next(at), None)
        batch = S.shtn_batch([p for p, (_, n) in zip(plans, fields) for _ in range(n)])
        S.shtn_batch_upload(batch, next(at), None)
        tune(batch, S.shtn_batch_device_bytes(batch), at)
        S.shtn_batch_destroy(batch)
    # a plan whose tables grew after the batch was made: refused, whatever else changed since
    plan = S.shtn_plan(300, 300, 301, 1024)
    batch = S.shtn_batch([plan] * 40)
    size = S.shtn_batch_device_bytes(batch)
    S.shtn_plan_set_tiling(plan, 1, 4, 1, 1, 0, 32, 1)
    S.shtn_plan_upload(plan, 1 << 40, None)
    S.shtn_batch_set_tiling(batch, 1, 1, 1, 0)  # the most units
    copied.value = 0
    rc = lib.shtn_batch_upload(batch, ctypes.c_void_p(1 << 41), None)
    assert rc == S.SHTN_ESTATE and copied.value == 0, (rc, copied.value, size)
    # fits with fewer units; the tuner leaves out the tilings that do not
    S.shtn_batch_set_tiling(batch, 2, 4, 0, 0)
    S.shtn_batch_upload(batch, 1 << 41, None)
    tune(batch, size, itertools.count(1 << 42, 1 << 36))
    # after a refused upload, calls are refused too: the tables are not those of the buffer
    S.shtn_batch_upload(batch, 1 << 41, None)
    S.shtn_plan_set_tiling(plan, 1, 4, 1, 1, 0, 32, 1)
    S.shtn_plan_upload(plan, 1 << 40, None)
    S.shtn_batch_set_tiling(batch, 1, 1, 1, 0)
    q, g, w = (ctypes.c_void_p(k << 43) for k in (1, 2, 3))
    assert lib.shtn_batch_upload(batch, ctypes.c_void_p(1 << 41), None) == S.SHTN_ESTATE
    assert lib.shtn_batch_synth(batch, q, g, w, None) == S.SHTN_ESTATE


def test_images_fit_the_reported_size(tmp_path):
    src, lib = tmp_path / "hip_stub.c", tmp_path / "libhip_stub.so"
    src.write_text(HIP_STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(lib)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    main(sys.argv[1])
