"""Plans where device memory is short (CPU): the library's plan code on a stand-in for the device's
memory (tests/native/fake_memory.cpp).  Several radii a launch are only for speed, so every call that
a plan of one radius a launch finds memory for has to succeed, whatever the plan took for more, and the
launches must be given slots inside the blocks that were allocated."""

import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1305_1505_amd", "csrc")
GIB = 1 << 30


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_1305_1505_amd import binding as B

    out = str(tmp_path_factory.mktemp("fake") / "libpin_fake_memory.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-shared", "-fPIC", "-pthread", "-Wl,-Bsymbolic", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "native", "fake_memory.cpp"), *[os.path.join(CSRC, f) for f in
                    ("plan.cpp", "capi.cpp", "host_math.cpp")], "-o", out], check=True, capture_output=True)
    lib = ctypes.CDLL(out)
    lib.fake_memory.argtypes = [ctypes.c_size_t]
    lib.fake_used.restype = ctypes.c_size_t
    lib.fake_buffer.argtypes, lib.fake_buffer.restype = [ctypes.c_size_t], ctypes.c_void_p
    for name in ("fake_batch", "fake_batch_v"):
        getattr(lib, name).argtypes = [ctypes.c_void_p]
    lib.hipFree.argtypes = [ctypes.c_void_p]
    for name, (res, args) in B._sig.items():
        if hasattr(lib, name):
            getattr(lib, name).restype, getattr(lib, name).argtypes = res, args
    return B, lib


def _sizes(n, n_radii, fp64):
    rb = 8 if fp64 else 4
    slot, vol, spectrum = n ** 3 * rb, n ** 3, n * n * (n // 2 + 1) * 2 * rb
    plan = 11 * slot + 2 * n * rb + n * (n_radii + 1) * rb + (3 * (n // 2) ** 2 + 1) * 8
    # one radius a launch: the plan, the caller's buffers, V, L
    return slot, [plan, spectrum, vol * rb, vol, 3 * vol * rb, 4 * slot, 10 * slot]


def _session(B, lib, n, n_radii, fp64, total, leave=None):
    """A program's calls in turn on a device of `total` bytes; how many of them found their memory.
    leave: the caller takes all but these bytes before its first call with v_max."""
    lib.fake_memory(total)
    desc = B.make_desc(n, 2.0 * n, [float(n_radii - i) for i in range(n_radii)], prec=B.PIN_FP64 if fp64 else B.PIN_FP32)
    plan, held, done = ctypes.c_void_p(), [], 0
    batches = None
    if lib.pin_plan_create(ctypes.byref(desc), ctypes.byref(plan)) == B.PIN_OK:
        done = 1
        for size in _sizes(n, n_radii, fp64)[1][1:5]:
            b = lib.fake_buffer(size)
            if b is None:
                break
            held.append(b)
            done += 1
        if done == 5:
            dk, F, ridx, v = held
            assert lib.pin_collapse_times(plan, dk, F, ridx, None) == B.PIN_OK
            if leave is not None:
                held.append(lib.fake_buffer(total - lib.fake_used() - leave))
            for call in (lambda: lib.pin_collapse_times_v(plan, dk, F, ridx, v, None),
                         lambda: lib.pin_lpt3_displacement(plan, dk, v, None)):
                status = call()
                if status != B.PIN_OK:
                    assert status == B.PIN_ERR_OUT_OF_MEMORY
                    break
                done += 1
            for _ in range(2):      # again, on what is there now
                assert lib.pin_collapse_times_range(plan, dk, F, ridx, 0, n_radii, None) == B.PIN_OK
                if done > 5:
                    assert lib.pin_collapse_times_range_v(plan, dk, F, ridx, v, 0, n_radii, None) == B.PIN_OK
        batches = (lib.fake_batch(plan), lib.fake_batch_v(plan))
        assert lib.pin_plan_destroy(plan) == B.PIN_OK
    for b in held:
        assert lib.hipFree(b) == 0
    assert lib.fake_used() == 0 and lib.fake_bad() == 0
    return done, batches


@pytest.mark.parametrize("n,n_radii,fp64", [(32, 8, False), (64, 16, True), (96, 3, True), (128, 32, False), (256, 4, False)])
def test_calls_that_fit_one_radius_succeed(fake, n, n_radii, fp64):
    B, lib = fake
    slot, need = _sizes(n, n_radii, fp64)
    ends = [sum(need[:k + 1]) for k in range(len(need))]
    totals = sorted({e + d for e in ends for d in (-1, 0, 1, slot)} | {ends[0] + k * 3 * slot for k in range(60)} |
                    {ends[-1] * k for k in (2, 4, 8, 16, 32)} | {64 * GIB})
    for total in totals:
        done, batches = _session(B, lib, n, n_radii, fp64, total)
        assert done >= sum(e <= total for e in ends), (total, batches)
    assert batches[0] == min(n_radii, B_most(n, fp64, 9)), batches      # the largest device: as many as share a launch
    assert batches[1] == min(batches[0], B_most(n, fp64, 13)), batches


def B_most(n, fp64, slots):
    fit = (256 << 20) // (slots * n ** 3 * (8 if fp64 else 4))
    return max(1, min(16, fit))


@pytest.mark.parametrize("n,n_radii,fp64", [(32, 8, False), (64, 16, True), (128, 32, False)])
def test_vmax_falls_back_to_one_radius(fake, n, n_radii, fp64):
    """A plan with room for several radii, whose program then leaves memory for one radius's gradient
    slots only."""
    B, lib = fake
    slot, _ = _sizes(n, n_radii, fp64)
    done, batches = _session(B, lib, n, n_radii, fp64, 64 * GIB, leave=4 * slot)
    assert done == 6 and batches[0] > 1 and batches[1] == 1
    done, batches = _session(B, lib, n, n_radii, fp64, 64 * GIB, leave=4 * slot - 1)
    assert done == 5
