"""The pinned buffer that reduction kernels write their results to: when a
tree may hand it on.

A destroyed tree returns the buffer to a pool that serves every tree of the
process, and a tree bound anew to another stream keeps it.  Calls such as
mg_nn_inputs enqueue writes to it without a host wait, so both must wait for
the bound stream first, whatever its handle (the null stream is one) and
device.  These tests run the library against a stand-in for the HIP runtime
(host memory, no device, no kernel runs) that lists the calls it gets, in a
child process that loads the stand-in before the library."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_;
static int dev = 0;
static size_t shmem;
static void *stream;
static dim3_ grid, block;
static int fail_sync = 0;
void stand_in_fail_sync(int f) { fail_sync = f; }
#define SAY(...) (printf(__VA_ARGS__), fflush(stdout), 0)
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t sh, void *s) { grid = g; block = b; shmem = sh; stream = s; return 0; }
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *sh, void **s) { *g = grid; *b = block; *sh = shmem; *s = stream; return 0; }
int hipLaunchKernel(const void *f, dim3_ g, dim3_ b, void **a, size_t sh, void *s) { return SAY("launch %zx on %d\n", (size_t)s, dev); }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) { memcpy(d, s, n); return SAY("copy %zx on %d\n", (size_t)st, dev); }
int hipStreamSynchronize(void *s) { SAY("wait %zx on %d\n", (size_t)s, dev); return fail_sync ? 400 : 0; }
int hipHostMalloc(void **p, size_t n, unsigned flags) { *p = calloc(1, n); return SAY("pinned %zx flags %x\n", (size_t)*p, flags); }
int hipHostFree(void *p) { return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { *d = h; return SAY("result %zx\n", (size_t)h); }
int hipGetDevice(int *d) { *d = dev; return 0; }
int hipSetDevice(int d) { dev = d; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { *s = malloc(8); return 0; }
int hipGetLastError(void) { return 0; }
"""

PRELUDE = """
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
from paper_1708_08434_amd import mg as M
from paper_1708_08434_amd import nn as NN
from workloads import uniform_boxes

def tree():
    b = uniform_boxes(2)
    return M.mg_tree_create(M.make_domain(), b.level, b.ijk, b.tree)

def bind(h, stream):
    need = int(M.mg_tree_info(h).workspace_bytes)
    ws = np.zeros(need + 256, dtype=np.uint8)
    M.mg_tree_bind(h, (ws.ctypes.data + 255) // 256 * 256, need, stream)
    return ws

def norms(h):  # enqueues a write of the results and returns
    NN.mg_nn_inputs(h, 4096, 4096)

def mark(what):
    print(what, flush=True)

"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    d = tmp_path_factory.mktemp("hip")
    src, so = d / "hip.c", d / "hip.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    return str(so)


def calls(stand_in, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, stand_in], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr
    return r.stdout.split("\n")


def between(log, a, b):
    return log[log.index(a) + 1:log.index(b)]


@pytest.mark.parametrize("stream", [0, 0x1000])
def test_destroy_waits_for_the_bound_stream(stand_in, stream):
    log = calls(stand_in, f"""
h = tree()
ws = bind(h, {stream})
norms(h)
mark("destroy")
M.mg_tree_destroy(h)
mark("end")
""")
    assert "launch %x on 0" % stream in log
    assert between(log, "destroy", "end") == ["wait %x on 0" % stream]


def test_destroy_waits_on_the_device_of_the_tree(stand_in):
    """The null stream is the current device's: a tree of device 1 destroyed
    while device 0 is current waits on device 1, and device 0 stays current."""
    log = calls(stand_in, """
hip.hipSetDevice(1)
h = tree()
ws = bind(h, 0)
norms(h)
hip.hipSetDevice(0)
mark("destroy")
M.mg_tree_destroy(h)
mark("end")
d = ctypes.c_int()
hip.hipGetDevice(ctypes.byref(d))
print("current", d.value)
""")
    assert between(log, "destroy", "end") == ["wait 0 on 1"]
    assert "current 0" in log


@pytest.mark.parametrize("old,new", [(0, 0x1000), (0x1000, 0x2000), (0x1000, 0)])
def test_rebind_waits_for_the_old_stream(stand_in, old, new):
    log = calls(stand_in, f"""
h = tree()
ws = bind(h, {old})
norms(h)
mark("rebind")
ws2 = bind(h, {new})
mark("end")
M.mg_tree_destroy(h)
""")
    assert between(log, "rebind", "end")[0] == "wait %x on 0" % old


def test_a_tree_that_was_never_bound_waits_for_nothing(stand_in):
    log = calls(stand_in, """
h = tree()
mark("destroy")
M.mg_tree_destroy(h)
mark("end")
""")
    assert between(log, "destroy", "end") == []


def test_a_buffer_whose_stream_cannot_be_waited_for_is_not_handed_on(stand_in):
    """Destroy and rebind when the wait fails (the caller has destroyed the
    stream): writes may still be under way, so the next bind takes another
    buffer."""
    log = calls(stand_in, """
h = tree()
ws = bind(h, 0x1000)
norms(h)
hip.stand_in_fail_sync(1)
try:
    bind(h, 0x2000)
except M.MGError:
    pass
M.mg_tree_destroy(h)
h = tree()
ws = bind(h, 0x1000) if not hip.stand_in_fail_sync(0) else None
norms(h)
hip.stand_in_fail_sync(1)
M.mg_tree_destroy(h)
hip.stand_in_fail_sync(0)
h = tree()
ws = bind(h, 0x3000)
M.mg_tree_destroy(h)
h = tree()
ws = bind(h, 0)
""")
    used = [s for s in log if s.startswith("result")]
    assert len(used) == 5
    assert used[0] not in used[1:]      # the rebind's failed wait
    assert used[2] not in used[3:]      # the destroy's failed wait
    assert used[3] == used[4]           # waited for: handed on


def test_result_buffers_are_mapped_on_every_device(stand_in):
    """Kernels of any device write to a pooled buffer, whichever device was
    current when it was allocated: hipHostMallocPortable (1) and
    hipHostMallocMapped (2)."""
    log = calls(stand_in, """
h = tree()
ws = bind(h, 0)
M.mg_tree_destroy(h)
hip.hipSetDevice(1)
h = tree()
ws = bind(h, 0)
""")
    used = [s.split()[1] for s in log if s.startswith("result")]
    assert len(used) == 2 and used[0] == used[1]
    flags = [int(s.split()[3], 16) for s in log if s.startswith("pinned " + used[0])]
    assert len(flags) == 1 and flags[0] & 3 == 3
