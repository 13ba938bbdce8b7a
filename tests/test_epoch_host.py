"""What the epochs allocate, free, launch and order, seen from the host without a GPU: the calls into the HIP runtime
are answered by a stand-in, in a process of its own, that launches nothing and prints every call that matters."""
import os
import re
import subprocess
import sys

import pytest

STAND_IN = r"""
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
typedef struct { uint32_t x, y, z; } dim3;
typedef unsigned long long u64;
size_t most_bytes = (size_t)1 << 60;  /* a larger allocation fails */
int capturing = 0;
int launches_left = 1 << 30;          /* the launch after these fails, and the following ones do not */
static int last = 0;
static uintptr_t next = 1 << 20, handles = 16;
#define SAY(...) (printf(__VA_ARGS__), fflush(stdout))
int hipGetDeviceCount(int *n) { *n = 1; return 0; }
int hipSetDevice(int d) { return 0; }
int hipGetDevicePropertiesR0600(void *p, int d) { return 101; }  /* the library then assumes 256 CUs */
int hipMalloc(void **p, size_t bytes) {
    if (bytes > most_bytes) return 2;
    *p = (void *)next;
    SAY("malloc %llx %llu\n", (u64)next, (u64)bytes);
    next += (bytes + 255) & ~(size_t)255;
    return 0;
}
int hipFree(void *p) { SAY("free %llx\n", (u64)(uintptr_t)p); return 0; }
int hipStreamSynchronize(void *s) { SAY("sync %llx\n", (u64)(uintptr_t)s); return 0; }
int hipStreamIsCapturing(void *s, int *status) { *status = capturing; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned flags) { *s = (void *)(handles += 16); return 0; }
int hipStreamDestroy(void *s) { return 0; }
int hipEventCreate(void **e) { *e = (void *)(handles += 16); return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { *e = (void *)(handles += 16); return 0; }
int hipEventDestroy(void *e) { return 0; }
int hipEventRecord(void *e, void *s) { SAY("record %llx %llx\n", (u64)(uintptr_t)e, (u64)(uintptr_t)s); return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned flags) {
    SAY("wait %llx %llx\n", (u64)(uintptr_t)e, (u64)(uintptr_t)s);
    return 0;
}
int hipMemcpyAsync(void *to, const void *from, size_t bytes, int kind, void *s) { return 0; }
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
    if (launches_left-- == 0) { last = 9; return 9; }
    SAY("launch %s %u %u %llx\n", dladdr(f, &info) && info.dli_sname ? info.dli_sname : "?", grid.x, grid.y,
        (u64)(uintptr_t)stream);
    return 0;
}
"""

CALLER = r"""
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
lib.cdgrab_last_error.restype = ctypes.c_char_p
i64, ptr, f32 = ctypes.c_int64, ctypes.c_void_p, ctypes.c_float
class Options(ctypes.Structure):
    _fields_ = [(k, ptr if k == "stream" else ctypes.c_int32) for k in
                ("device", "block_pairs", "stream", "timing", "pass1_groups", "apply_mode", "gram_mode", "apply_groups")]
def handle(**options):
    h = ptr()
    assert lib.cdgrab_create(ctypes.byref(h), ctypes.byref(Options(**options))) == 0
    return h
h = handle()
IN, SIGNS, PERM, DOTS, W, V, LABELS = (ptr((1 << 50) + (i << 44)) for i in range(7))  # (no kernel runs)
def epoch(m, n, d, h=h):
    return lib.cdgrab_balance_epoch(h, i64(m), i64(n), i64(d), IN, None, None, None, SIGNS, PERM, None, None, DOTS)
def train(m, n, in_dim, classes, h=h):
    return lib.cdgrab_train_epoch_softmax(h, i64(m), i64(n), i64(in_dim), i64(classes), IN, LABELS, None, W, None,
                                          f32(0.1), f32(0), SIGNS, PERM, None, None)
def text(h=h):
    return lib.cdgrab_last_error(h).decode()
def capture(on):
    ctypes.c_int.in_dll(hip, "capturing").value = on
def room(nbytes):
    ctypes.c_size_t.in_dll(hip, "most_bytes").value = nbytes
def fail_launch(after):
    ctypes.c_int.in_dll(hip, "launches_left").value = after
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
        """The calls (what, arguments ..) of every part of `code` that a mark() opens."""
        p = subprocess.run([sys.executable, "-c", CALLER + code, str(so), pkg.library_path()], text=True,
                           capture_output=True, timeout=120)
        assert p.returncode == 0, p.stderr
        parts, now = {}, None
        for line in p.stdout.splitlines():
            if line.startswith("# "):
                now = parts.setdefault(line[2:], [])
            elif now is not None:
                now.append(tuple(line.split()))
        return parts
    return run


def of(calls, what):
    return [c[1:] for c in calls if c[0] == what]


def kernels(calls):
    return [c[0] for c in of(calls, "launch")]


def walks_of(calls):
    """Per launch that walks rows of at most 64 elements: are its Gram results beforehand (its last template argument)?"""
    return [re.search(r"narrow_walkI(?:L[ib]\d+E)*Lb([01])EEE", k).group(1) == "1" for k in kernels(calls) if "narrow_walk" in k]


def test_long_narrow_epochs_leave_a_recorded_chain_its_buffers(call):
    """Rows of at most 64 elements have a workspace of their own: a chain of steps that was recorded holds the addresses
    of its Gram tiles, which an epoch of such rows must neither free nor replace."""
    parts = call("mark('warm')\nassert epoch(4, 64, 1024) == 0\n"
                 "capture(1)\nmark('recorded')\nassert epoch(4, 64, 1024) == 0\ncapture(0)\n"
                 "mark('narrow')\nassert epoch(1, 100_000, 16) == 0\n"
                 "mark('again')\nassert epoch(4, 64, 1024) == 0\n")
    assert any("gram_tiles" in k for k in kernels(parts["recorded"])) and not of(parts["recorded"], "malloc")
    assert walks_of(parts["narrow"]) == [True]
    had = {address for address, _ in of(parts["warm"], "malloc")}
    assert had and not had & {address for address, in of(parts["narrow"], "free")}
    assert not of(parts["again"], "malloc") and not of(parts["again"], "free")


def test_recorded_narrow_epochs_are_those_that_run_eagerly(call):
    """Same launches, so the same sums in the same order; nothing is allocated, and no buffer that a recorded call was
    given is freed by a longer epoch, however often those follow."""
    parts = call("mark('eager')\nassert epoch(2, 1200, 20) == 0\n"
                 "capture(1)\nmark('recorded')\nassert epoch(2, 1200, 20) == 0\ncapture(0)\n"
                 "mark('longer')\nassert epoch(2, 4800, 20) == 0\n"
                 "capture(1)\nmark('recorded longer')\nassert epoch(2, 4800, 20) == 0\ncapture(0)\n"
                 "mark('longest')\nassert epoch(3, 100_000, 64) == 0 and epoch(1, 400_000, 16) == 0\n"
                 "mark('destroyed')\nlib.cdgrab_destroy(h)\n")
    assert kernels(parts["eager"]) == kernels(parts["recorded"])
    assert kernels(parts["longer"]) == kernels(parts["recorded longer"])
    assert all(walks_of(parts[p]) and all(walks_of(parts[p])) for p in ("recorded", "recorded longer", "longest"))
    assert not of(parts["recorded"], "malloc") and not of(parts["recorded longer"], "malloc")
    had = {address for p in ("eager", "longer") for address, _ in of(parts[p], "malloc")}
    freed = {address for p in ("longer", "recorded longer", "longest") for address, in of(parts[p], "free")}
    assert had and not had & freed
    # two buffers at most: the first, and one that holds what any epoch takes
    big = [int(size) for p in ("longer", "longest") for _, size in of(parts[p], "malloc") if int(size) > 1 << 20]
    assert len(big) == 1 and big[0] < 68 << 20
    assert had <= {address for address, in of(parts["destroyed"], "free")}


def test_narrow_epochs_where_there_is_no_room(call):
    """Recorded before the handle has run such a shape, or with no memory for the Gram results: the form without workspace,
    and no error text."""
    parts = call("assert epoch(4, 64, 16) == 0\nassert epoch(1, 3, 16) != 0\nbefore = text()\nassert before\n"
                 "capture(1)\nmark('recorded')\nassert epoch(1, 4000, 16) == 0\ncapture(0)\n"
                 "room(1 << 20)\nmark('no room')\nassert epoch(1, 4000, 16) == 0\nassert text() == before\n"
                 "room(1 << 40)\nmark('room')\nassert epoch(1, 4000, 16) == 0\n"
                 "room(1 << 20)\nmark('no more room')\nassert epoch(1, 40_000, 16) == 0\nassert text() == before\n")
    for p in ("recorded", "no room", "no more room"):
        assert walks_of(parts[p]) == [False] and not any("narrow_bands" in k for k in kernels(parts[p]))
    assert not of(parts["recorded"], "malloc")
    assert walks_of(parts["room"]) == [True] and sum("narrow_bands" in k for k in kernels(parts["room"])) == 1


@pytest.mark.parametrize("m,n,d,beside", [
    (16, 300, 7850, True), (1, 600, 32_768, True), (1, 600, 40_959, True), (1, 600, 40_960, False),
    (1, 4096, 20_000, True), (1, 600, 49_152, False),
    (1, 4096, 65_536, False), (1, 600, 65_540, False), (1, 600, 131_072, False), (1, 600, 900, False),
])
def test_rows_read_beside_a_walk(call, m, n, d, beside):
    """The next step's rows are read beside a walk where they fit the L2s; the last step has none after it."""
    part = call("h = handle(gram_mode=2)\nmark('epoch')\nassert epoch(%d, %d, %d, h) == 0\n" % (m, n, d))["epoch"]
    grids = [int(y) for name, _, y, _ in of(part, "launch") if "chain_walk" in name]
    assert len(grids) > 1 and grids[-1] == 1
    assert all((y > 8) == beside for y in grids[:-1])


TRAIN = [(8, 900, 30, 4), (4, 1100, 7, 4), (4, 1500, 783, 3), (16, 260, 12, 5), (16, 1000, 784, 10)]


def streams_of(calls):
    return {s for name, _, _, s in of(calls, "launch")}


def joined(calls, side):
    """Does the first stream wait for an event behind the last launch on stream `side`?"""
    last = max(i for i, c in enumerate(calls) if c[0] == "launch" and c[4] == side)
    ends = [c[1] for c in calls[last:] if c[0] == "record" and c[2] == side]
    return any(c[0] == "wait" and c[1] in ends and c[2] == "0" for c in calls[last:])


@pytest.mark.parametrize("m,n,in_dim,classes", TRAIN)
def test_training_chunks_go_to_a_second_stream(call, m, n, in_dim, classes):
    """Several chunks, each balanced on the second stream behind its rows, its buffer filled again only behind that, and all
    of it before what follows; with timing, or while launches are recorded, everything on the one stream."""
    shape = "%d, %d, %d, %d" % (m, n, in_dim, classes)
    parts = call("mark('beside')\nassert train(%s) == 0\n"
                 "capture(1)\nmark('recorded')\nassert train(%s) == 0\ncapture(0)\n"
                 "t = handle(timing=1)\nmark('timed')\nassert train(%s, t) == 0\n" % (shape, shape, shape))
    assert streams_of(parts["recorded"]) == streams_of(parts["timed"]) == {"0"}
    calls = parts["beside"]
    side, = streams_of(calls) - {"0"}
    walk = [c for c in calls if c[0] == "launch" and ("chain_walk" in c[1] or "narrow_walk" in c[1])]
    assert all(c[4] == side for c in walk)
    to_side, to_main = (sum(c[0] == "wait" and c[2] == s for c in calls) for s in (side, "0"))
    assert to_side >= 2 and to_main == to_side - 2 + 1  # a wait per chunk; from the third chunk on for its buffer, and the end
    assert joined(calls, side)


@pytest.mark.parametrize("m,n,in_dim,classes", [(4, 1100, 7, 4), (16, 1000, 784, 10)])
def test_streams_meet_again_where_a_launch_fails(call, m, n, in_dim, classes):
    """Whichever launch fails: what has gone to the second stream is ordered before what follows the call on the first, and
    the next call begins on the first."""
    shape = "%d, %d, %d, %d" % (m, n, in_dim, classes)
    total = sum(c[0] == "launch" for c in call("mark('all')\nassert train(%s) == 0\n" % shape)["all"])
    tries = sorted({0, 1, total - 1, *range(0, total, max(1, total // 40))})
    parts = call("".join("h%d = handle()\nmark('%d')\nfail_launch(%d)\nassert train(%s, h%d) in (-3, -4)\nmark('%d after')\n"
                         "fail_launch(1 << 30)\nassert epoch(4, 64, 1024, h%d) == 0\n" % (k, k, k, shape, k, k, k) for k in tries))
    on_side = 0
    for k in tries:
        calls = parts[str(k)]
        for side in streams_of(calls) - {"0"}:
            on_side += 1
            assert joined(calls, side)
        assert streams_of(parts["%d after" % k]) == {"0"}
    assert on_side > 3
