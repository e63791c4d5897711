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
int hipMemcpyAsync(void* dst, const void* src, size_t n, int kind, void* stream) { copied = n; return 0; }
int hipStreamSynchronize(void* stream) { return 0; }
int hipLaunchKernel(const void* f, ...) { return 0; }
int hipGetLastError(void) { return 0; }
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
    # a plan whose tables grew after the batch was made: refused, whatever else changed since
    plan = S.shtn_plan(300, 300, 301, 1024)
    batch = S.shtn_batch([plan] * 40)
    size = S.shtn_batch_device_bytes(batch)
    S.shtn_plan_set_tiling(plan, 1, 4, 1, 1, 0, 32, 1)
    S.shtn_plan_upload(plan, 1 << 40, None)
    S.shtn_batch_set_tiling(batch, 1, 1, 1, 0)  # the most units
    copied.value = 0
    rc = S.load_library().shtn_batch_upload(batch, ctypes.c_void_p(1 << 41), None)
    assert rc == S.SHTN_ESTATE and copied.value == 0, (rc, copied.value, size)


def test_images_fit_the_reported_size(tmp_path):
    src, lib = tmp_path / "hip_stub.c", tmp_path / "libhip_stub.so"
    src.write_text(HIP_STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), str(lib)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr


if __name__ == "__main__":
    main(sys.argv[1])
