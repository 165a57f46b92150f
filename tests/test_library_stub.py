"""The library's host code on the CPU, against a runtime without a device (hip_stub.c): what it does
when device memory runs out or a launch fails, and what it launches.  Each scenario in a process of
its own, the stub loaded before the library."""
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2107_13952_amd", "libeprl.so")
OK, ENOMEM, EHIP = 0, -2, -3


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("stub") / "hip_stub.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-o", out,
                    os.path.join(HERE, "hip_stub.c")], check=True)
    return out


class Library:
    """The library over the stub: one context, calls with buffers of the stub's memory."""

    def __init__(self, path):
        self.stub = ctypes.CDLL(path, mode=ctypes.RTLD_GLOBAL)
        for name in ("stub_live", "stub_peak"):
            getattr(self.stub, name).restype = ctypes.c_size_t
        self.stub.stub_grid.restype = ctypes.c_long
        self.stub.stub_limit.argtypes = [ctypes.c_size_t]
        self.lib = ctypes.CDLL(LIB)
        self.ctx = self.context()
        self.buf = ctypes.c_void_p()
        assert self.stub.hipMalloc(ctypes.byref(self.buf), ctypes.c_size_t(1 << 20)) == 0
        self.stub.stub_peak()

    def context(self):
        ctx = ctypes.c_void_p()
        assert self.lib.eprl_create(ctypes.byref(ctx), 0, None) == 0
        return ctx

    def launches(self, name):
        return self.stub.stub_launches(name.encode())

    def vertex(self, two_j, dl, ctx=None):
        return self.lib.eprl_vertex_tensor(ctx or self.ctx, (ctypes.c_int * 10)(*two_j), dl, ctypes.c_double(1.2),
                                           self.buf, self.buf)

    def batch(self, configs, ctx=None):
        n = len(configs)
        js = (ctypes.c_int * (10 * n))(*[s for two_j, _ in configs for s in two_j])
        dls = (ctypes.c_int * n)(*[dl for _, dl in configs])
        ptrs = (ctypes.c_void_p * n)(*[self.buf.value] * n)
        return self.lib.eprl_vertex_tensor_batched(ctx or self.ctx, n, js, dls, ctypes.c_double(1.2), ptrs, ptrs)

    def sixj(self, two_j):
        return self.lib.eprl_sixj_batch(self.ctx, 1, (ctypes.c_int * 6)(*[two_j] * 6), self.buf)


SMALL = [([2] * 10, 2), ([4, 4, 5, 3, 5, 5, 6, 4, 3, 6], 1)]


# A table of factorials that cannot grow leaves the old one in place: the batch laid out with it runs
# on, and never with the address of freed memory.
def factorial_table_stays_when_it_cannot_grow(lib):
    for how in ("memory", "launch"):
        assert lib.batch(SMALL) == OK
        if how == "memory":
            lib.stub.stub_limit(lib.stub.stub_live())
            assert lib.sixj(200) == ENOMEM
            lib.stub.stub_limit(1 << 40)
        else:
            lib.stub.stub_fail(b"fact_kernel")
            assert lib.sixj(200) == EHIP
            lib.stub.stub_fail(None)
        assert lib.batch(SMALL) == OK
        assert lib.vertex(*SMALL[1]) == OK
        assert lib.stub.stub_stale() == 0
    assert lib.sixj(200) == OK
    assert lib.batch(SMALL) == OK
    assert lib.stub.stub_stale() == 0


RING_VALU = 3
# Spins, dl: 8-wide tiles, 16-wide tiles.
LARGE = [([6] * 10, 8), ([13, 10, 11, 12, 10, 14, 11, 13, 13, 10], 6)]


def needed(lib, call, algorithm):
    """Device memory that `call` takes on a fresh context."""
    ctx = lib.context()
    assert lib.lib.eprl_set_algorithm(ctx, algorithm) == OK
    before = lib.stub.stub_live()
    lib.stub.stub_peak()
    assert call(ctx) == OK
    need = lib.stub.stub_peak() - before
    lib.lib.eprl_destroy(ctx)
    return need


# Memory for the kernels without derived tables, and no more, is enough for a vertex tensor and for a
# core range; with memory the x-outer kernel takes over again.
def vertex_runs_without_memory_for_derived_tables(lib):
    for two_j, dl in LARGE:
        def cores(ctx):
            return lib.lib.eprl_vertex_tensor_cores(ctx, (ctypes.c_int * 10)(*two_j), dl, ctypes.c_double(1.2), lib.buf,
                                                    ctypes.c_int64(0), ctypes.c_int64((dl + 1) ** 3), 0, lib.buf)
        for call in (lambda ctx: lib.vertex(two_j, dl, ctx), cores):
            need = needed(lib, call, RING_VALU)
            assert needed(lib, call, 0) > need
            ctx = lib.context()
            lib.stub.stub_limit(lib.stub.stub_live() + need)
            for _ in range(2):
                lib.stub.stub_clear()
                assert call(ctx) == OK
                assert lib.launches("chain_kernel") == 0 and lib.launches("ring_kernel") == 1
            lib.stub.stub_limit(1 << 40)
            lib.stub.stub_clear()
            assert call(ctx) == OK
            assert lib.launches("chain_kernel") == 1 and lib.launches("ring_kernel") == 0
            lib.lib.eprl_destroy(ctx)


# A batch that does not fit takes its derived tables in several passes, then one configuration to a
# pass, then the kernels without them; the last it does not keep.
def batch_runs_with_less_memory(lib):
    configs = [([6] * 10, 5), ([13, 10, 11, 12, 10, 14, 11, 13, 13, 10], 4), ([8] * 10, 4)] + SMALL
    call = lambda ctx: lib.batch(configs, ctx)
    most, least = needed(lib, call, 0), needed(lib, call, RING_VALU)
    assert most > least
    for need, passes in ((most - (1 << 20), True), (least, False)):
        ctx = lib.context()
        base = lib.stub.stub_live()
        lib.stub.stub_limit(base + need)
        for _ in range(2):
            lib.stub.stub_clear()
            assert call(ctx) == OK
            assert lib.stub.stub_stale() == 0
            assert (lib.launches("chain_prep_batch_kernel") > 1) == passes
            assert (lib.launches("ring_batch_kernel") > 0) == (not passes)
        lib.stub.stub_limit(1 << 40)
        lib.stub.stub_clear()
        assert call(ctx) == OK
        assert (lib.launches("chain_prep_batch_kernel") > 1) == passes
        assert lib.launches("ring_batch_kernel") == 0
        lib.lib.eprl_destroy(ctx)


# The autotuner tries the default split too: where that is the fastest, it stays.
def autotune_tries_the_default(lib):
    lib.stub.stub_watch(b"chain_kernel")
    for two_j, dl in LARGE:
        ctx = lib.context()
        assert lib.vertex(two_j, dl, ctx) == OK
        default = lib.stub.stub_grid()
        lib.stub.stub_fastest(ctypes.c_long(default))
        out = (ctypes.c_int * 3)()
        assert lib.lib.eprl_autotune(ctx, (ctypes.c_int * 10)(*two_j), dl, lib.buf, lib.buf, out) == OK
        assert lib.vertex(two_j, dl, ctx) == OK
        assert lib.stub.stub_grid() == default
        lib.lib.eprl_destroy(ctx)


# A core range makes the derived tables of its own (l24, l25) only: for one core T2 of one pair and T5 of
# one l25, instead of those of all (dl + 1)^2 pairs and dl + 1 values.
def core_range_makes_its_own_derived_tables(lib):
    lib.stub.stub_watch(b"chain_prep_kernel")
    for two_j, dl in LARGE:
        js, nd = (ctypes.c_int * 10)(*two_j), dl + 1
        grid = []
        for lo, hi in ((0, nd ** 4), (nd ** 4 // 2, nd ** 4 // 2 + 1), (nd ** 2 - 1, nd ** 2 + 1), (5, 5)):
            assert lib.lib.eprl_vertex_tensor_cores(lib.ctx, js, dl, ctypes.c_double(1.2), lib.buf, ctypes.c_int64(lo),
                                                    ctypes.c_int64(hi), 0, lib.buf) == OK
            grid.append(lib.stub.stub_grid())
        whole, one, two, none = grid
        # T5 blocks nd (x, l35) per l25, T2 blocks x per pair; the rest is the same for every range
        assert two - one == one - none > 0
        assert whole - none == (nd * nd + nd * nd) * (one - none) // (nd + 1)


# The booster builder loads its lists and 4jm tables again whenever a refinement replaces the workspace,
# also by one at the same address.
def boosters_follow_the_workspace(lib):
    lib.stub.stub_read(ctypes.c_double(1.0))   # an error above the tolerance: n = 16, 32, ..., 512, each with a larger workspace
    for reuse in (0, 1):
        ctx = lib.context()
        assert lib.lib.eprl_sixj_batch(ctx, 1, (ctypes.c_int * 6)(*[200] * 6), lib.buf) == OK
        lib.stub.stub_reuse(reuse)
        lib.stub.stub_clear()
        info = (ctypes.c_double * 3)()
        assert lib.lib.eprl_boosters(ctx, (ctypes.c_int * 10)(*[2] * 10), 1, ctypes.c_double(1.2), ctypes.c_double(0.5),
                                     lib.buf, info) == OK
        assert info[2] == 512 and lib.launches("integrals_kernel") == 6
        assert lib.launches("fourjm_table_kernel") == 6
        lib.lib.eprl_destroy(ctx)


# Edges of few blocks (one at dl = 0, eight at dl = 1) take their r integrals block by block, not by tiles of
# 16 x 16 blocks; edges of many by tiles, a remainder of fewer than sixteen blocks too.
def boosters_of_few_blocks(lib):
    lib.stub.stub_read(ctypes.c_double(0.0))
    lib.stub.stub_watch(b"booster_block_integrals_kernel")
    for two_j, dl, tiles, blocks in ((14, 0, 0, 4), (2, 1, 0, 32), (2, 3, 1, 0), (1, 6, 1, 0)):
        lib.stub.stub_clear()
        assert lib.lib.eprl_boosters(lib.ctx, (ctypes.c_int * 10)(*[two_j] * 10), dl, ctypes.c_double(1.2),
                                     ctypes.c_double(0.5), lib.buf, None) == OK
        assert lib.launches("booster_integrals_kernel") == tiles
        assert lib.launches("booster_block_integrals_kernel") == (1 if blocks else 0)
        if blocks:
            m = sum(abs(a + b + c) <= two_j for a in range(-two_j, two_j + 1, 2) for b in range(-two_j, two_j + 1, 2)
                    for c in range(-two_j, two_j + 1, 2))
            assert lib.stub.stub_grid() == blocks * ((m + 3) // 4)


# Few shells at large spins: no more workgroups than their partial sums are worth (one to two rounds of the
# chip, down to a multiple of the i1 values); many shells: the full number (11 x 208 where the partial sums
# reach their 256 MB).
def small_sums_are_split_less(lib):
    lib.stub.stub_watch(b"chain_kernel")
    for two_j, dl, lo, hi in (([12] * 10, 1, 200, 512), ([10] * 10, 1, 200, 768), ([14] * 10, 0, 200, 512),
                              ([6] * 10, 3, 1000, 3072), ([6] * 10, 8, 8000, 8192), (LARGE[1][0], 6, 2288, 2288)):
        assert lib.vertex(two_j, dl) == OK
        assert lo <= lib.stub.stub_grid() <= hi, (two_j, dl, lib.stub.stub_grid())


SCENARIOS = [factorial_table_stays_when_it_cannot_grow,
             vertex_runs_without_memory_for_derived_tables,
             batch_runs_with_less_memory,
             autotune_tries_the_default,
             core_range_makes_its_own_derived_tables,
             boosters_follow_the_workspace,
             boosters_of_few_blocks,
             small_sums_are_split_less]


@pytest.mark.parametrize("scenario", [f.__name__ for f in SCENARIOS])
def test_library(stub, scenario):
    res = subprocess.run([sys.executable, os.path.abspath(__file__), stub, scenario], capture_output=True, text=True,
                         timeout=300)
    assert res.returncode == 0, res.stdout + res.stderr


if __name__ == "__main__":
    globals()[sys.argv[2]](Library(sys.argv[1]))
