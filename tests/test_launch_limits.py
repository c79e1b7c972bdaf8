"""Grids of accepted batches stay launchable (CPU test, no GPU call is made).

HIP refuses a launch of 2^32 or more work-items in one dimension. A process
of its own loads a stand-in for the few HIP runtime calls the library makes
before the library itself, so its launches resolve to the stand-in, which
refuses such grids as HIP does and records the others: kernel, workgroups,
workgroup size and the first pointer of the kernel's argument block (the
input a launch starts from). The pointers passed in are never read.
"""

import json
import subprocess
import sys

import pytest

from paper_2307_12607_amd import _capi

STAND_IN = r"""
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
static dim3 g_grid, g_block;
static size_t g_shmem;
static void *g_stream;
static int g_err;
static int n_launches;
static struct { const void *fn; unsigned long long grid, block; const void *first; } launches[4096];
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, void *stream) {
    g_grid = grid; g_block = block; g_shmem = shmem; g_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, void **stream) {
    *grid = g_grid; *block = g_block; *shmem = g_shmem; *stream = g_stream;
    return 0;
}
int hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t shmem, void *stream) {
    unsigned long long threads = (unsigned long long)block.x * block.y * block.z;
    if ((unsigned long long)grid.x * block.x >= 1ull << 32 || grid.y != 1 || grid.z != 1 ||
        threads == 0 || threads > 1024 || grid.x == 0)
        return g_err = 9;
    if (n_launches < 4096) {
        launches[n_launches].fn = fn;
        launches[n_launches].grid = grid.x;
        launches[n_launches].block = threads;
        launches[n_launches].first = *(const void **)args[0];
        ++n_launches;
    }
    return 0;
}
int hipGetLastError(void) { int e = g_err; g_err = 0; return e; }
int launch_count(void) { return n_launches; }
void launch_at(int i, unsigned long long *out) {
    out[0] = (unsigned long long)launches[i].fn;
    out[1] = launches[i].grid;
    out[2] = launches[i].block;
    out[3] = (unsigned long long)launches[i].first;
}
"""

CHILD = r"""
import ctypes, json, sys
stand_in, lib, name, calls = json.loads(sys.argv[1])
s = ctypes.CDLL(stand_in, mode=ctypes.RTLD_GLOBAL)
fn = getattr(ctypes.CDLL(lib), name)
conv = {"i": ctypes.c_int32, "p": ctypes.c_void_p, "z": ctypes.c_size_t, "d": ctypes.c_double,
        "f": lambda v: (ctypes.c_float * len(v))(*v)}
results = []
for args in calls:
    first = s.launch_count()
    status = fn(*[conv[t](v) for t, v in args])
    out, rec = [], (ctypes.c_ulonglong * 4)()
    for i in range(first, s.launch_count()):
        s.launch_at(i, rec)
        out.append(list(rec))
    results.append([status, out])
print(json.dumps(results))
"""

# Addresses far apart (1 TB), never read.
SRC, MV, GOUT, GSRC, GMV, WS = (("p", (i + 1) << 40) for i in range(6))


@pytest.fixture(scope="module")
def launches_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("stand_in")
    (d / "hip.c").write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", str(d / "hip.c"), "-o",
                    str(d / "hip.so")], check=True)

    def run(name, *calls):
        job = json.dumps([str(d / "hip.so"), _capi.LIB_PATH, name, calls])
        r = subprocess.run([sys.executable, "-c", CHILD, job], capture_output=True, text=True,
                           check=True)
        return json.loads(r.stdout)

    return run


def covered(launches, base, stride, per_item):
    """The launches that start from an input at ``base`` as (first item, items),
    each item (frame or plane) taking ``per_item`` workgroups."""
    spans = []
    for _, grid, _, first in launches:
        assert grid % per_item == 0 and (first - base) % stride == 0
        spans.append(((first - base) // stride, grid // per_item))
    return spans


def assert_consecutive(spans, total):
    at = 0
    for first, items in spans:
        assert first == at
        at += items
    assert at == total


@pytest.mark.parametrize("n", [1, (1 << 23) - 1, 1 << 23, (1 << 24) + 5])
@pytest.mark.parametrize("recorded", [False, True])
def test_adjoint_of_many_tiny_frames(launches_of, n, recorded):
    """Frames of one pixel, one tile each: past 2^23 of them one launch of
    512-thread tiles would reach 2^32 work-items."""
    phases = [1.0]
    name = "exw_warp_backward_batched" + ("_recorded" if recorded else "")
    [[status, launches]] = launches_of(name, [
        SRC, ("i", 0), ("i", n), ("i", 1), ("i", 1), ("i", 1), MV, ("f", phases), ("i", 1), GOUT,
        GSRC, GMV, WS, ("z", 1 << 40), ("p", 0)])
    assert status == 0
    tiles = [r for r in launches if r[2] == 512]  # the tile kernel's workgroups
    assert_consecutive(covered(tiles, SRC[1], 4, 1), n)


@pytest.mark.parametrize("c,hw", [(64, 1), (64, 128 * 128), (1, 30000 * 30000), (3, 1080 * 1920)])
@pytest.mark.parametrize("n", [1, 1 << 16, (1 << 18) - 1])
@pytest.mark.parametrize("dtype", [0, 1])
def test_emd_of_many_planes(launches_of, c, hw, n, dtype):
    """Up to 2^24 - 64 planes, as long as the batch is within 2^40 values."""
    if n * c * hw > 1 << 40 or n * c >= 1 << 24:
        pytest.skip("not accepted")
    esize = 2 if dtype else 4
    [[status, launches]] = launches_of("exw_buffer_emd", [
        ("p", 1 << 42), ("p", 1 << 43), ("i", dtype), ("i", n), ("i", c), ("i", 1), ("i", hw),
        ("d", -1.0), ("d", 1.0), ("i", 64), ("p", 1 << 40), ("p", 1 << 41), ("z", 1 << 40), ("p", 0)])
    assert status == 0
    # the histogram kernel starts from cur, the clearing one from the workspace
    hist = [r for r in launches if r[3] >= 1 << 42]
    parts = hist[0][1] // covered_planes(hist, n * c, hw * esize)
    assert_consecutive(covered(hist, 1 << 42, hw * esize, parts), n * c)


def covered_planes(hist, planes, plane_bytes):
    """Planes of the first histogram launch: up to where the second one starts."""
    return planes if len(hist) == 1 else (hist[1][3] - hist[0][3]) // plane_bytes


@pytest.mark.parametrize("b,c,h,w", [(1, 1, 11, 11), (1 << 25, 1, 11, 65), (5, 1 << 23, 11, 65),
                                     (1 << 24, 2, 11, 64), ((1 << 24) + 1, 1, 11, 139),
                                     (24, 4, 1080, 1920)])
@pytest.mark.parametrize("dtype", [0, 2])
def test_quality_of_many_planes(launches_of, b, c, h, w, dtype):
    esize = 2 if dtype else 4
    [[status, launches]] = launches_of("exw_frame_quality", quality_call(b, c, h, w, dtype))
    assert status == 0
    # the strip kernel starts from pred, the fold of the frames from the workspace
    strips = [r for r in launches if r[3] >= 1 << 43]
    per_plane = strips[0][1] // covered_planes(strips, b * c, h * w * esize)
    assert_consecutive(covered(strips, 1 << 43, h * w * esize, per_plane), b * c)


def quality_call(b, c, h, w, dtype):
    return [("p", 1 << 43), ("p", 1 << 42), ("i", dtype), ("i", b), ("i", c), ("i", h), ("i", w),
            ("d", 1.0), ("p", 1 << 40), ("p", 1 << 41), ("z", 1 << 40), ("p", 0)]


def test_quality_strips_fit_the_workspace(launches_of):
    """One pair of partial sums per strip: the strips of a plane never
    outnumber the 64 x 66 blocks of positions the workspace is sized by."""
    shapes = [(b, c, h, w) for b, c in ((1, 1), (3, 4), (700, 3))
              for h in (11, 19, 76, 77, 150, 270, 1080, 4000)
              for w in (11, 64, 65, 74, 75, 128, 129, 138, 139, 256, 257, 266, 333, 1000, 1920)]
    results = launches_of("exw_frame_quality", *[quality_call(*s, 0) for s in shapes])
    for (b, c, h, w), (status, launches) in zip(shapes, results):
        assert status == 0
        strips = [r for r in launches if r[3] >= 1 << 43]
        room = _capi.lib().exw_frame_quality_workspace_bytes(b, c, h, w) // 16
        assert 0 < sum(r[1] for r in strips) <= room, (b, c, h, w)


@pytest.mark.parametrize("n,h,w", [(1, 1080, 1920), (1 << 23, 1, 1), ((1 << 24) + 7, 3, 5), (1, 1 << 28, 1),
                                   (1, 1 << 30, 1), (3, (1 << 28) + 40, 2)])
def test_dynamic_objects_of_many_tiles(launches_of, n, h, w):
    [[status, launches]] = launches_of("exw_dynamic_objects", [
        ("p", 1 << 42), ("i", n), ("i", h), ("i", w), ("i", 8), ("p", 1 << 40), ("p", 1 << 43),
        ("z", 1 << 45), ("p", 0)])
    assert status == 0
    tiles = n * -(-h // 32) * -(-w // 64)
    passes = [r for r in launches if r[3] == 1 << 42]  # both passes start from the stencil
    kernels = list(dict.fromkeys(r[0] for r in passes))
    grids = [sum(r[1] for r in passes if r[0] == k) for k in kernels]
    assert grids == [tiles, -(-tiles // 2)]  # one tile, and two tiles, per workgroup
