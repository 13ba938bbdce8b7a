"""What cdgrab_herding_bound launches and allocates, seen from the host without a GPU: the calls into
the HIP runtime are answered by a stand-in, in a process of its own, that launches nothing."""
import os
import subprocess
import sys

import pytest

STAND_IN = r"""
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
typedef struct { uint32_t x, y, z; } dim3;
size_t most_bytes = (size_t)1 << 60;  /* a larger allocation fails */
int capturing = 0, last = 0, mallocs = 0;
static uintptr_t next = 1 << 20;
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { return 101; }  /* the library then assumes 256 CUs */
int hipMalloc(void **p, size_t bytes) {
    if (bytes > most_bytes) return 2;
    ++mallocs;
    *p = (void *)next;
    next += (bytes + 255) & ~(size_t)255;
    return 0;
}
int hipFree(void *p) { return 0; }
int hipStreamSynchronize(void *s) { return 0; }
int hipStreamIsCapturing(void *s, int *status) { *status = capturing; return 0; }
int hipGetLastError(void) { int e = last; last = 0; return e; }
const char *hipGetErrorString(int e) { return "refused"; }
static struct { dim3 grid, block; size_t lds; void *stream; } config;  /* of the launch in between */
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    config.grid = grid; config.block = block; config.lds = lds; config.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
    Dl_info info;
    /* a grid holds fewer than 2^32 threads in each direction */
    const int fits = (uint64_t)grid.x * block.x < ((uint64_t)1 << 32) && grid.y <= 65535;
    printf("%s %u %u\n", dladdr(f, &info) && info.dli_sname ? info.dli_sname : "?", grid.x, block.x);
    fflush(stdout);
    if (!fits) last = 9;
    return fits ? 0 : 9;
}
"""

CALLER = r"""
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
lib.cdgrab_last_error.restype = ctypes.c_char_p
i64, ptr = ctypes.c_int64, ctypes.c_void_p
h = ptr()
assert lib.cdgrab_create(ctypes.byref(h), None) == 0
def bound(m, n, d):
    return lib.cdgrab_herding_bound(h, i64(m), i64(n), i64(d), ptr(4096), ptr(8192), ptr(512))
def mallocs():
    return ctypes.c_int.in_dll(hip, "mallocs").value
def text():
    return lib.cdgrab_last_error(h).decode()
def capture(on):
    ctypes.c_int.in_dll(hip, "capturing").value = on
def room(nbytes):
    ctypes.c_size_t.in_dll(hip, "most_bytes").value = nbytes
def mark(name):
    print("#", name, flush=True)
"""


@pytest.fixture(scope="module")
def call(tmp_path_factory):
    import paper_2302_00845_amd as pkg
    if not os.path.exists(pkg.library_path()):
        from paper_2302_00845_amd import build
        build.build_library(verbose=False)
    where = tmp_path_factory.mktemp("hip")
    src, so = where / "hip.c", where / "hip.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-D_GNU_SOURCE", "-o", str(so), str(src), "-ldl"], check=True)

    def run(code):
        """Launches (name, workgroups, threads) of every part of `code` that a mark() opens."""
        p = subprocess.run([sys.executable, "-c", CALLER + code, str(so), pkg.library_path()], text=True,
                           capture_output=True, timeout=120)
        assert p.returncode == 0, p.stderr
        parts, now = {}, None
        for line in p.stdout.splitlines():
            if line.startswith("# "):
                now = parts.setdefault(line[2:], [])
            elif now is not None:
                name, groups, threads = line.split()
                now.append((name, int(groups), int(threads)))
        return parts
    return run


@pytest.mark.parametrize("d", [(1 << 29) - 1, (1 << 29) + 5, (1 << 32) - 257])
def test_longest_rows_are_not_refused(call, d):
    """A thread per element in the prefix over the segments, of which rows this long have one."""
    launches = call("mark('call')\nrc = bound(1, 2, %d)\nassert rc == 0, text()\n" % d)["call"]
    assert len(launches) == 4


def test_steps_sums_stay_out_of_a_capture(call):
    """The sums kept from the first pass lie in a buffer that a later call with more steps replaces, so a launch that
    is recorded must not hold its address, whether the handle has the buffer or not."""
    parts = call("bound(5, 4000, 600)\n"           # room for the segments of everything that follows
                 "mark('eager')\nassert bound(6, 300, 600) == 0\n"
                 "capture(1)\nbefore = mallocs()\n"
                 "mark('captured')\nassert bound(6, 300, 600) == 0 and bound(6, 600, 600) == 0\n"
                 "assert mallocs() == before\n")
    kept = lambda part: [name for name, _, _ in parts[part] if "ELb1E" in name]  # the kernels' STEPS form
    assert len(kept("eager")) == 2 and not kept("captured")


def test_no_error_text_after_a_call_that_succeeds(call):
    """Where the steps' sums do not fit, the rows are read again: the call succeeds and says nothing."""
    call("assert bound(5, 4000, 600) == 0 and bound(6, 300, 600) == 0\n"
         "assert bound(0, 1, 1) != 0\nbefore = text()\nassert before\n"
         "room(1 << 20)\nassert bound(6, 2000, 600) == 0, text()\nassert text() == before\n"
         "assert bound(6, 2000, 700_000) != 0 and 'workspace' in text()\n")
