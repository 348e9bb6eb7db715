"""Allocations that fail. A lattice that has no memory for its blur groups is
built without them, and an adjoint without memory for its wide blocks filters
narrower ones; any other failure is reported and leaves the library usable."""
import gc

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


class Allocator:
    """Device memory from torch; the failing hook returns no memory for the
    allocations that `refuse(index, bytes)` names."""

    def __init__(self):
        import torch
        self.torch, self.dev = torch, torch.cuda.current_device()
        self.sizes, self.refuse = [], lambda i, n: False

    def alloc(self, nbytes, stream):
        self.sizes.append(nbytes)
        if self.refuse(len(self.sizes) - 1, nbytes):
            return 0
        return self.torch.cuda.caching_allocator_alloc(nbytes, self.dev, stream)

    def free(self, ptr, stream):
        self.torch.cuda.caching_allocator_delete(ptr)


@pytest.fixture()
def mem():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import paper_2106_06695_amd as sgp
    a = Allocator()
    gc.collect()
    sgp.set_allocator(a.alloc, a.free)
    try:
        yield sgp, a
    finally:
        gc.collect()
        sgp.set_allocator(None, None)


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def _blur_launches(sgp, lat, V):
    import torch
    with sgp.profile() as prof:
        sgp.lattice_mvm(lat, V)
        torch.cuda.synchronize()
    return prof.results["blur"][0]


@pytest.mark.parametrize("order", [1, 2])
def test_build_with_an_allocation_refused(mem, order):
    """Each allocation of a build refused in turn: an error, or a lattice
    without groups (the fused pairs, or a launch per direction of the wider
    stencil) whose products are the same bit for bit."""
    sgp, a = mem
    d, n = 11, 17000
    w = workloads.small_case(500, n, d, channels=3, kind="mixture")
    X, V = _cuda(w.X), _cuda(w.values)
    lat = sgp.lattice_build(X, w.lengthscales, order=order)
    count = len(a.sizes)
    assert lat.m >= 8192 and _blur_launches(sgp, lat, V) == 4  # three groups
    ref = sgp.lattice_mvm(lat, V).cpu().numpy()
    lat.free()
    without = 0
    for i in range(count):
        print(f"build order={order}: allocation {i} of {count} refused", flush=True)
        a.sizes.clear()
        a.refuse = lambda k, nbytes: k == i
        try:
            lat = sgp.lattice_build(X, w.lengthscales, order=order)
        except sgp.SGPError as e:
            assert e.code == -2
            continue
        finally:
            a.refuse = lambda k, nbytes: False
        without += 1
        assert _blur_launches(sgp, lat, V) == ((d + 2) // 2 if order == 1 else d + 1)
        np.testing.assert_array_equal(sgp.lattice_mvm(lat, V).cpu().numpy(), ref)
        lat.free()
    assert without == 2  # the groups' rows, and their counts
    lat = sgp.lattice_build(X, w.lengthscales, order=order)
    np.testing.assert_array_equal(sgp.lattice_mvm(lat, V).cpu().numpy(), ref)
    lat.free()


def test_adjoint_narrows_its_blocks(mem):
    """A lattice with groups whose work arrays for 16 channels find no memory:
    the adjoint filters narrower blocks, with the same bits; with no memory for
    those either, an error, and the next call is served."""
    sgp, a = mem
    n, d = 200000, 16
    rng = np.random.default_rng(d)
    X = _cuda(rng.standard_normal((n, d)))
    V, G = _cuda(rng.standard_normal((n, 2))), _cuda(rng.standard_normal((n, 2)))
    lat = sgp.lattice_build(X, np.full(d, 0.5))
    print(f"adjoint blocks: m={lat.m}", flush=True)
    assert 2 * lat.m * 16 * 4 > 320 << 20  # the fused pairs would take 8 channels
    a.sizes.clear()
    dX, dl = sgp.lattice_mvm_grad(lat, X, V, G)
    ref, wide = dX.cpu().numpy(), max(a.sizes)
    assert wide >= 4 * 16 * 4 * lat.m  # a block of 16
    lat.free()
    lat = sgp.lattice_build(X, np.full(d, 0.5))
    a.refuse = lambda i, nbytes: nbytes >= wide
    dX2, dl2 = sgp.lattice_mvm_grad(lat, X, V, G)
    np.testing.assert_array_equal(dX2.cpu().numpy(), ref)
    np.testing.assert_array_equal(np.asarray(dl2), np.asarray(dl))
    a.refuse = lambda i, nbytes: False
    lat.free()
    lat = sgp.lattice_build(X, np.full(d, 0.5))
    m = lat.m
    a.refuse = lambda i, nbytes: nbytes >= 4 * 8 * 4 * m  # a block of 8
    with pytest.raises(sgp.SGPError) as e:
        sgp.lattice_mvm_grad(lat, X, V, G)
    assert e.value.code == -2
    a.refuse = lambda i, nbytes: False
    dX2, _ = sgp.lattice_mvm_grad(lat, X, V, G)
    np.testing.assert_array_equal(dX2.cpu().numpy(), ref)
    lat.free()


# seed, n, d, ell: m = 16,474 (CG's vectors per point); m = 9,992 of 50,001 points (on the lattice)
@pytest.mark.parametrize("seed,n,d,ell,on_lattice", [(500, 17000, 11, (0.5, 2.0), False),
                                                      (205, 50001, 11, (0.7, 2.0), True)])
def test_work_memory_of_the_blur(mem, seed, n, d, ell, on_lattice):
    """The blur by groups works in two lattice arrays in place; steps and pairs
    take three (four inside CG), and the buffer grows when the switch turns to
    them. Results do not depend on it."""
    sgp, a = mem
    C = 3
    w = workloads.small_case(seed, n, d, channels=C, kind="mixture", ell_range=ell)
    X, V = _cuda(w.X), _cuda(w.values)

    def largest(call):
        a.sizes.clear()
        out = call().cpu().numpy()
        return out, max(a.sizes, default=0)

    def solve(lat):
        return lambda: sgp.cg_solve(lat, V, 0.1, 0.0, max_iter=11)[0]

    got = {}
    for fuse in (True, False):
        prev = sgp.blur_fuse_enable(fuse)
        try:
            for name in ("mvm", "cg"):
                lat = sgp.lattice_build(X, w.lengthscales)
                m = lat.m
                assert m >= 8192 and (3 * m <= 2 * n) == on_lattice
                got[name, fuse] = largest((lambda: sgp.lattice_mvm(lat, V)) if name == "mvm" else solve(lat))
                if fuse:  # the same lattice, then without groups and with them again
                    sgp.blur_fuse_enable(False)
                    again, _ = largest((lambda: sgp.lattice_mvm(lat, V)) if name == "mvm" else solve(lat))
                    sgp.blur_fuse_enable(True)
                    back, grown = largest((lambda: sgp.lattice_mvm(lat, V)) if name == "mvm" else solve(lat))
                    np.testing.assert_array_equal(again, got[name, True][0])
                    np.testing.assert_array_equal(back, got[name, True][0])
                    assert grown == 0
                lat.free()
        finally:
            sgp.blur_fuse_enable(prev)
    print(f"work memory m={m} on_lattice={on_lattice} {[(k, v[1]) for k, v in got.items()]}", flush=True)
    for name, extra in (("mvm", 1 * 4), ("cg", 2 * 8)):
        np.testing.assert_array_equal(got[name, True][0], got[name, False][0])
        assert got[name, False][1] - got[name, True][1] == extra * m * C
