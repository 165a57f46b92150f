"""The x-outer kernel of the factorised order at the edges of its tiles, against the CPU oracle.

Workloads over its row tiles (one and two per wavefront) and column tiles (one to eleven, in one or
two column blocks), for one to fourteen shells per link (one to four groups of four spin values) and
k windows of at most and of more than sixteen positions; the ones with many shells over a few cores,
on the oracle's shells.  Tolerance: an output entry is a sum of at most
16^2 shells of a core times 16 k3, k4 and x values each, every product rounded a few times:
about 16^3 units of 2^-53 relative to the largest entry, 5e-13.
"""
import ctypes
import sys

import numpy as np
import pytest

import workloads
from oracle import ranges as R
from oracle import vertex as V

pytestmark = pytest.mark.gpu

TOL = 5e-13


@pytest.fixture(scope="module")
def lib():
    import paper_2107_13952_amd as lib
    return lib


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


# Twice the spins, dl, cores (None: all), dimensions
CASES = [([2, 6, 3, 1, 7, 6, 5, 7, 8, 8], 0, None, (1, 3, 7, 4, 2)),
         ([8, 10, 4, 6, 9, 4, 7, 10, 7, 4], 1, None, (5, 5, 8, 2, 5)),
         ([9, 15, 4, 6, 0, 7, 16, 12, 15, 15], 0, None, (3, 1, 1, 5, 7)),
         ([4, 4, 5, 3, 5, 5, 6, 4, 3, 6], 2, None, (4, 5, 4, 5, 4)),
         ([10, 3, 2, 13, 9, 9, 12, 7, 13, 10], 1, None, (2, 9, 4, 3, 11)),
         ([9, 9, 7, 7, 9, 9, 7, 8, 10, 8], 0, None, (8, 8, 9, 8, 7)),
         ([13, 12, 8, 11, 14, 11, 14, 14, 8, 7], 0, None, (9, 12, 9, 7, 7)),
         ([10, 13, 11, 12, 12, 16, 14, 14, 11, 13], 0, None, (11, 11, 12, 12, 12)),
         ([15, 12, 15, 16, 13, 15, 13, 14, 13, 14], 0, None, (13, 14, 13, 15, 13)),
         ([15] * 10, 0, None, (16, 16, 16, 16, 16)),
         ([14, 5, 14, 1, 3, 14, 9, 5, 9, 7], 9, (4321, 4326), (2, 4, 3, 6, 2)),
         ([8, 8, 6, 2, 15, 7, 8, 8, 13, 13], 9, (777, 779), (3, 5, 8, 5, 3)),
         ([1, 6, 9, 8, 10, 7, 8, 9, 9, 5], 9, (9990, 10000), (2, 2, 7, 6, 6)),
         ([7, 7, 8, 10, 6, 8, 9, 10, 9, 6], 9, (0, 1), (7, 7, 7, 7, 7)),
         ([3, 2, 3, 2, 4, 3, 4, 3, 3, 3], 13, (20000, 20004), (3, 4, 3, 4, 3))]


@pytest.mark.parametrize("two_j,dl,cores,dims", CASES)
def test_tile_edges(lib, torch, two_j, dl, cores, dims):
    assert tuple(lib.layout(two_j, dl)[0]) == dims
    b = workloads.synthetic_boosters(400 + dl, R.block_shapes(two_j, dl))
    bd = torch.from_numpy(b).cuda()
    print(f"tile edges {two_j} dl={dl} cores={cores}", flush=True)
    sys.stdout.flush()
    if cores is None:
        a, ref = lib.vertex_tensor(two_j, dl, 1.2, bd), V.vertex_tensor(two_j, dl, b)
    else:
        nd = dl + 1
        lo, hi = cores
        shells = []
        for core in range(lo, hi):
            o24, o25, o34, o35 = core // nd ** 3, core // nd ** 2 % nd, core // nd % nd, core % nd
            shells += [(o23, o24, o25, o34, o35, o45) for o23 in range(nd) for o45 in range(nd)]
        a = lib.vertex_tensor_cores(two_j, dl, 1.2, bd, lo, hi)
        ref = V.vertex_tensor(two_j, dl, b, shells=shells)
    scale = np.abs(ref).max()
    assert scale > 0
    assert np.abs(a.cpu().numpy() - ref).max() <= TOL * scale


# The widest tiles at many shells: two row tiles by seven to eleven column tiles (two T row groups in
# flight, and two columns of H from nine tiles on), one and two column blocks (thirteen tiles: the last of
# the second block is padding), two to four groups of four spin values, an odd last group among them, and
# windows of more than sixteen positions.  Each on the oracle's shells of the core with the widest window.
# Tolerance: as above; an entry is a sum over at most 14^2 shells, and no sum of the chain (x, k3, k4, k5,
# k2, l45, l23) is longer than 40.
MANY = [([11, 14, 11, 10, 15, 15, 13, 15, 12, 15], 8, 2957, (10, 12, 13, 12, 11)),
        ([13, 13, 13, 15, 12, 15, 16, 13, 12, 17], 9, 4067, (13, 13, 13, 13, 13)),
        ([13, 13, 8, 8, 15, 15, 13, 15, 13, 8], 10, 5384, (9, 14, 14, 9, 9)),
        ([13, 12, 8, 15, 9, 12, 12, 13, 14, 9], 8, 2216, (9, 10, 10, 9, 10)),
        ([13, 12, 9, 8, 11, 10, 16, 14, 15, 9], 8, 3674, (9, 10, 12, 8, 9)),
        ([15, 12, 15, 14, 16, 12, 9, 14, 16, 9], 8, 2945, (13, 10, 13, 10, 9)),
        ([13, 8, 13, 8, 10, 16, 15, 9, 11, 8], 12, 6688, (9, 11, 9, 8, 7)),
        ([14, 13, 15, 14, 12, 9, 13, 15, 12, 13], 13, 24788, (14, 10, 12, 10, 13)),
        ([11, 15, 12, 12, 16, 10, 13, 13, 12, 11], 13, 24816, (11, 10, 13, 11, 12)),
        ([15, 14, 15, 8, 12, 13, 16, 12, 12, 12], 13, 19313, (9, 13, 12, 12, 9)),
        ([14, 14, 14, 10, 13, 12, 15, 13, 16, 13], 13, 19311, (11, 13, 13, 13, 11)),
        ([13, 15, 10, 14, 18, 12, 17, 16, 15, 12], 12, 17673, (11, 13, 15, 10, 13)),
        ([15, 12, 12, 13, 17, 17, 15, 16, 15, 15], 5, 14, (12, 16, 13, 13, 14))]


@pytest.mark.parametrize("two_j,dl,core,dims", MANY)
def test_widest_tiles_many_shells(lib, torch, two_j, dl, core, dims):
    assert tuple(lib.layout(two_j, dl)[0]) == dims
    nd = dl + 1
    b = workloads.synthetic_boosters(600 + dl, R.block_shapes(two_j, dl))
    print(f"widest tiles {two_j} dl={dl} core={core}", flush=True)
    a = lib.vertex_tensor_cores(two_j, dl, 1.2, torch.from_numpy(b).cuda(), core, core + 1)
    o24, o25, o34, o35 = core // nd ** 3, core // nd ** 2 % nd, core // nd % nd, core % nd
    ref = V.vertex_tensor(two_j, dl, b, shells=[(o23, o24, o25, o34, o35, o45)
                                                for o23 in range(nd) for o45 in range(nd)])
    scale = np.abs(ref).max()
    assert scale > 0
    assert np.abs(a.cpu().numpy() - ref).max() <= TOL * scale


# A tensor entry A(i1..i5) depends on the booster entries of its own i2..i5 only: with one infinite or NaN
# booster entry every other entry has the bits of the call without it (zeros that pad the tables meet no
# infinity of another edge).
@pytest.mark.parametrize("two_j,dl", [([9, 8, 12, 9, 5, 11, 3, 10, 7, 7], 3), ([4] * 10, 2), ([3, 2, 3, 2, 4, 3, 4, 3, 3, 3], 4),
                                      ([13, 10, 11, 12, 10, 14, 11, 13, 13, 10], 2), ([2, 3, 2, 1, 3, 2, 3, 1, 1, 3], 2)])
def test_infinities_stay_in_their_entries(lib, torch, two_j, dl):
    dims, _, offs = lib.layout(two_j, dl)
    n3 = (dl + 1) ** 3
    b = workloads.synthetic_boosters(800 + dl, R.block_shapes(two_j, dl))
    clean = lib.vertex_tensor(two_j, dl, 1.2, torch.from_numpy(b).cuda())
    rng = np.random.default_rng(800 + dl)
    for trial in range(24):
        at = int(rng.integers(len(b)))
        block = int(np.searchsorted(offs, at, side="right")) - 1
        edge, columns = block // n3, int(offs[block + 1] - offs[block]) // dims[block // n3 + 1]
        row = (at - int(offs[block])) // columns
        print(f"infinities {two_j} dl={dl} entry {at} edge {edge + 2} row {row}", flush=True)
        c = b.copy()
        c[at] = (np.nan, np.inf, -np.inf)[trial % 3]
        a = lib.vertex_tensor(two_j, dl, 1.2, torch.from_numpy(c).cuda())
        rest = [q for q in range(dims[edge + 1]) if q != row]
        assert torch.equal(a.index_select(edge + 1, torch.tensor(rest, dtype=torch.int64, device="cuda")),
                           clean.index_select(edge + 1, torch.tensor(rest, dtype=torch.int64, device="cuda")))


# A layout kept from call to call must follow the buffers of each call: two batches of one shape
# (factorised configurations of both kinds of tables and a per-shell one), called in turn with other
# boosters and outputs, on the default and on a side stream, equal the plain calls bit by bit.
@pytest.mark.parametrize("shape", [[([2] * 10, 2), ([4, 4, 5, 3, 5, 5, 6, 4, 3, 6], 1), ([1] * 10, 16)],
                                   [([3, 2, 3, 2, 4, 3, 4, 3, 3, 3], 3), ([2] * 10, 2)]])
def test_batch_follows_its_buffers(lib, torch, shape):
    sets = [[torch.from_numpy(workloads.synthetic_boosters(500 + 10 * k + q, R.block_shapes(j, d))).cuda()
             for q, (j, d) in enumerate(shape)] for k in range(3)]
    plain = [[lib.vertex_tensor(j, d, 1.2, b) for (j, d), b in zip(shape, s)] for s in sets]
    side = torch.cuda.Stream()
    for k in (0, 1, 2, 1, 0):
        print("batch buffers", k, flush=True)
        if k == 2:
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                out = lib.vertex_tensor_batched(shape, 1.2, sets[k])
            torch.cuda.current_stream().wait_stream(side)
        else:
            out = lib.vertex_tensor_batched(shape, 1.2, sets[k])
        for a, p in zip(out, plain[k]):
            assert torch.equal(a, p)


# A batch whose derived tables are taken in several passes (configurations of several kernel variants, one
# to three of a variant) on the same memory, first in two or three passes, then one configuration to a
# pass, equals the plain calls bit by bit, also where a layout is kept and the buffers change.
def test_batch_in_passes(lib, torch):
    shape = [([2] * 10, 3), ([4, 4, 5, 3, 5, 5, 6, 4, 3, 6], 2), ([9, 9, 7, 7, 9, 9, 7, 8, 10, 8], 1), ([2] * 10, 2),
             ([13, 12, 8, 11, 14, 11, 14, 14, 8, 7], 0), ([1] * 10, 16), ([4, 4, 5, 3, 5, 5, 6, 4, 3, 6], 1)]
    sets = [[torch.from_numpy(workloads.synthetic_boosters(700 + 10 * k + q, R.block_shapes(j, d))).cuda()
             for q, (j, d) in enumerate(shape)] for k in range(2)]
    plain = [[lib.vertex_tensor(j, d, 1.2, b) for (j, d), b in zip(shape, s)] for s in sets]
    handle, bound = lib._ctx("cuda").handle, lib._lib.eprl_internal_batch_pass
    bound.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
    try:
        for limit in (3 << 19, 1 << 19, 0):
            assert bound(handle, limit) == 0
            for k in (0, 1, 0):
                print("batch in passes", limit, k, flush=True)
                for a, p in zip(lib.vertex_tensor_batched(shape, 1.2, sets[k]), plain[k]):
                    assert torch.equal(a, p)
    finally:
        bound(handle, 8 << 30)


# Index arithmetic of the contractions at its edges: dimensions of one, powers of two, primes, and one
# past 2^16.  A complex product is within sqrt(8) 2^-53, so either side's sum of N products of up to six
# factors is within (N + 15) 2^-53 of the sum of their moduli.
@pytest.mark.parametrize("dims", [(1, 1, 1, 1, 1), (3, 5, 7, 2, 11), (16, 8, 1, 4, 32), (1, 2, 65537, 1, 3), (13, 1, 1, 17, 1)])
def test_contraction_indices(lib, torch, dims):
    gen = torch.Generator().manual_seed(sum(dims))
    a = torch.randn(dims, dtype=torch.float64, generator=gen)
    psi = [torch.randn(n, dtype=torch.complex128, generator=gen) for n in dims]
    print("contraction", dims, flush=True)
    ad, pd = a.cuda(), [p.cuda() for p in psi]
    for m in range(1, 6):
        got = lib.contract_trailing(ad, pd[5 - m:]) if m < 5 else lib.contract_boundary(ad, pd)
        ref, mod = a.to(torch.complex128), a.abs()
        for p in reversed(psi[5 - m:]):
            ref, mod = ref @ p, mod @ p.abs()
        bound = (2 * int(np.prod(dims[5 - m:])) + 30) * 2.0 ** -53 * mod
        assert ((got.cpu().reshape(ref.shape) - ref).abs() <= bound).all()
