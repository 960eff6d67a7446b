"""The plan of the work queues (size_launch and queue_entry of
sbr_forward.hip) hands out every index once.  Their own text is compiled for
the host and called here, with 4 or 256 compute units: on small calls every
entry is taken, on the largest that the entry points accept (2^40 rays,
4096 transmitters of 2^40) samples of them."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_21719_amd", "csrc")

HARNESS = r"""
static int g_cu = 256;
static int64_t g_chunk = 1;
int rt_persistent_blocks(int block, int) { return g_cu * std::max(1, 16 * 64 / block); }
int64_t rt_order_chunk(const LaunchOrder&) { return g_chunk; }
rt_status rt_fail(rt_status st, const std::string&) { return st; }
static FwdArgs g_args;
struct Call {       // what a launch passes to size_launch, and what it gets
    int64_t n_work, lattice, begin, chunk, n_wide, cells;
    int32_t cu, block, n_tx, deposit, refill, brute;
    int64_t blocks, once, width, nq, claim, n_units, n_claim, per_queue, n_first, first_width, spread;
};
extern "C" int plan(Call* c) {
    g_cu = c->cu;
    g_chunk = c->chunk;
    rt_scene s;
    s.n_wide = c->n_wide;
    s.n_tri = 2 * c->n_wide;
    FwdArgs& a = g_args;
    memset(&a, 0, sizeof(a));
    a.n_work = c->n_work;
    a.n_tx = c->n_tx;
    a.tx.n_rays = c->lattice;
    a.ray_begin = c->begin;
    a.deposit = c->deposit;
    a.refill = c->refill;
    a.tape_groups = 4;
    a.map_stride = c->cells;
    LaunchOrder order{0, c->chunk > 1 ? 10 : 0, 0};
    int blocks = 0;
    const int st = SIZE_LAUNCH;
    c->blocks = blocks;
    c->once = a.once;
    c->width = a.width;
    c->nq = a.nq;
    c->claim = a.claim;
    c->n_units = a.n_units;
    c->n_claim = a.n_claim;
    c->per_queue = (int64_t)a.per_queue;
    c->n_first = a.n_first;
    c->first_width = a.first_width;
    c->spread = a.by_r == 1 && a.by_k == a.nq * a.by_q ? a.run : 0;
    return st;
}
// work of entry i of queue q, of the last plan
extern "C" void entry(unsigned i, int q, int64_t* r) { queue_entry(g_args, i, q, r, r + 1); }
// times each index is handed out
extern "C" void hand_out(unsigned char* seen) {
    for (int q = 0; q < g_args.nq; q++)
        for (unsigned i = 0; i < g_args.per_queue; i++) {
            int64_t b, e;
            queue_entry(g_args, i, q, &b, &e);
            for (int64_t n = b; n < e; n++) seen[n]++;
        }
}
"""


class Call(C.Structure):
    _fields_ = ([(n, C.c_int64) for n in ("n_work", "lattice", "begin", "chunk", "n_wide", "cells")] +
                [(n, C.c_int32) for n in ("cu", "block", "n_tx", "deposit", "refill", "brute")] +
                [(n, C.c_int64) for n in ("blocks", "once", "width", "nq", "claim", "n_units", "n_claim", "per_queue",
                                          "n_first", "first_width", "spread")])


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    with open(os.path.join(CSRC, "sbr_forward.hip")) as f:
        src = f.read()
    parts = [re.search(p, src, re.S).group(0) for p in
             (r"struct FwdArgs \{.*?\n\};\n", r"__device__ __forceinline__ void queue_entry\(.*?\n\}\n",
              r"static constexpr int64_t kLargeTree[^\n]*;\n", r"static rt_status size_launch\(.*?\n\}\n")]
    call = "size_launch(a, &s, c->block, order, c->brute != 0, &blocks)"
    d = tmp_path_factory.mktemp("queues")
    cpp, so = str(d / "q.cpp"), str(d / "q.so")
    head, harness = HARNESS.split("static FwdArgs g_args;")
    with open(cpp, "w") as f:
        f.write('#include <algorithm>\n#include <cstdlib>\n#include <cstring>\n#include "rt_internal.h"\n'
                "using std::min;\n" + head + "".join(parts) + "static FwdArgs g_args;" +
                harness.replace("SIZE_LAUNCH", call))
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                           "-shared", "-fPIC", "-Wl,-z,lazy", cpp, "-o", so])
    L = C.CDLL(so, mode=os.RTLD_LAZY)
    L.entry.argtypes = [C.c_uint, C.c_int, C.c_void_p]
    L.hand_out.argtypes = [C.c_void_p]
    return L


def _plan(lib, n_work, cu=256, block=256, n_tx=0, chunk=987, n_wide=100, begin=0, lattice=None, deposit=2, refill=64,
          brute=0, cells=10_000):
    c = Call(n_work=n_work, lattice=lattice or n_work, begin=begin, chunk=chunk, n_wide=n_wide, cu=cu, block=block,
             n_tx=n_tx, deposit=deposit, refill=refill, brute=brute, cells=cells)
    assert lib.plan(C.byref(c)) == 0
    return c


def _every_index_once(lib, c):
    if c.once:
        return                     # no queues: one unit per wavefront
    seen = np.zeros(c.n_work, np.uint8)
    lib.hand_out(seen.ctypes.data)
    assert np.all(seen == 1)


LANES = 4 * 16 * 64                # of 4 compute units


@pytest.mark.parametrize("n", [1, LANES - 447, LANES + 1, 4 * LANES + 77, 33 * LANES + 17, 70 * LANES + 5])
@pytest.mark.parametrize("n_tx", [0, 1, 3])
@pytest.mark.parametrize("queues,claim", [(None, None), ("1", "64"), ("7", "192"), ("32", "4096")])
def test_every_index_once(lib, monkeypatch, n, n_tx, queues, claim):
    if queues:
        monkeypatch.setenv("RTMAP_QUEUES", queues)
        monkeypatch.setenv("RTMAP_CLAIM", claim)
    for n_wide in (100, 40_000):
        for chunk in (1, 987):
            for begin, lattice in ((0, n), (n // 3, 2 * n)):
                _every_index_once(lib, _plan(lib, n, 4, n_tx=n_tx, chunk=chunk, n_wide=n_wide, begin=begin,
                                             lattice=lattice))


@pytest.mark.parametrize("n,n_tx,queues,claim", [(2 ** 40, 0, "1", "64"), (2 ** 40, 0, "1", "256"),
                                                 (2 ** 40 - 12345, 0, None, None), (2 ** 38 + 1, 0, "1", "64"),
                                                 (2 ** 44 + 999, 4096, None, None), (2 ** 52, 4096, None, None),
                                                 (2 ** 52, 4096, "1", "64")])
def test_largest_calls(lib, monkeypatch, n, n_tx, queues, claim):
    """Entries are counted in 32 bits: the units grow until they suffice."""
    if queues:
        monkeypatch.setenv("RTMAP_QUEUES", queues)
        monkeypatch.setenv("RTMAP_CLAIM", claim)
    c = _plan(lib, n, n_tx=n_tx)
    assert c.per_queue < 2 ** 32 and c.n_claim * c.nq < 2 ** 32
    assert c.n_claim * c.nq >= c.n_units
    rest = n - c.n_claim * c.nq * c.claim
    assert (c.per_queue - c.n_claim) * c.nq * c.width >= rest
    # entries far apart and next to each other: no index twice
    rng = np.random.default_rng(3)
    pick = np.unique(np.concatenate([np.arange(2000), c.n_claim - np.arange(1, 2000), c.per_queue - np.arange(1, 2000),
                                     rng.integers(0, c.per_queue, 5000)]))
    got = []
    r = (C.c_int64 * 2)()
    for i in pick:
        for q in {0, int(c.nq) // 2, int(c.nq) - 1}:
            lib.entry(int(i), q, r)
            if r[0] < r[1]:
                got.append((r[0], r[1]))
    got = np.array(sorted(got))
    assert len(got) > 5000 and got[0, 0] >= 0 and got[-1, 1] <= n
    assert np.all(got[1:, 0] >= got[:-1, 1])


@pytest.mark.parametrize("n", [1, 100, 20_000, 100_000])
def test_brute_force_keeps_whole_wavefronts(lib, n):
    """Each narrow wavefront would test all triangles for its few rays."""
    assert _plan(lib, n, brute=1).width == 64
    assert _plan(lib, n).width < 64


@pytest.mark.parametrize("n_tx", [0, 1, 3])
@pytest.mark.parametrize("queues,claim", [(None, None), ("1", "64"), ("7", "192"), ("32", "4096")])
def test_stretches(lib, monkeypatch, n_tx, queues, claim):
    """Calls of many units whose deposits are not summed (atomic strategy, or
    lattice order) go through stretches in turn, the others along one front."""
    if queues:
        monkeypatch.setenv("RTMAP_QUEUES", queues)
        monkeypatch.setenv("RTMAP_CLAIM", claim)
    for n in (4 * LANES - 64, 4 * LANES - 63, 5 * LANES + 1, 9 * LANES + 77, 33 * LANES + 17, 70 * LANES + 5):
        for deposit, chunk in ((1, 987), (2, 1), (1, 1), (2, 987)):
            for begin, lattice in ((0, n), (n // 3, 2 * n)):
                for n_wide in (100, 40_000):
                    c = _plan(lib, n, 4, n_tx=n_tx, chunk=chunk, n_wide=n_wide, begin=begin, lattice=lattice,
                              deposit=deposit)
                    if not queues and n_wide == 100:
                        assert bool(c.spread) == (n > 4 * LANES - 64 and (deposit, chunk) != (2, 987))
                    _every_index_once(lib, c)
    if not queues:
        c = _plan(lib, 2 ** 40, n_tx=n_tx, deposit=1)
        assert c.spread == 16 and c.per_queue < 2 ** 32 and c.n_claim * c.nq >= c.n_units


@pytest.mark.parametrize("n_tx", [2, 3, 4, 16, 64])
def test_horizons_of_several_transmitters(lib, n_tx):
    """On a large tree the transmitters of middling calls go through stretches."""
    for units in (1, 2, 3, 4, 7, 15, 17, 30, 33, 63, 65):
        n = units * LANES + 77
        c = _plan(lib, n, 4, n_tx=n_tx, n_wide=40_000)
        few = 1 if n_tx >= 4 else 0
        assert c.spread == (few if units < 4 else 4 if units < min(64, 8 * n_tx) else 0)
        _every_index_once(lib, c)
        assert not _plan(lib, n, 4, n_tx=n_tx, n_wide=30_000).spread


@pytest.mark.parametrize("n_tx", [0, 1, 3])
def test_maps_of_few_cells(lib, n_tx):
    """Wavefronts that add to the same cells: whole ones in small calls on a small
    scene, stretches in large calls."""
    for cells in (1, 31, 32, 256, 257):
        for n in (1, 900, LANES // 4 + 3):
            for n_wide in (5, 31, 32, 300):
                c = _plan(lib, n, 4, n_tx=n_tx, n_wide=n_wide, cells=cells)
                assert (c.width == 64) == (cells <= 256 and n_wide < 32)
                _every_index_once(lib, c)
        n = 9 * LANES + 77
        for n_wide in (5, 300, 40_000):
            c = _plan(lib, n, 4, n_tx=n_tx, n_wide=n_wide, cells=cells)
            if n_wide < 32_768:
                assert (c.spread == 4) == (cells < 32)
            _every_index_once(lib, c)
