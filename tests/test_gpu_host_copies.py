"""Fields between pageable host arrays and the device: every node arrives at its own place.

The density is random per node, so a chunk that lands elsewhere shows. The initial populations are
equilibria: their sum gives the density back within the rounding of at most 27 terms,
27 * 2**-52 < 1e-14; the bar is 1e-13.
"""
import threading

import numpy as np
import pytest

from tests.gpu_cases import Case

pytestmark = pytest.mark.gpu


# the largest field copied directly and one plane more, ragged rows (repacked on the device) with a
# ragged last chunk, more chunks than workers' buffers, a small field, and a 2D box
@pytest.mark.parametrize("dims", [(128, 64, 64), (128, 64, 65), (141, 100, 67), (96, 80, 300), (67, 33, 29), (1000, 703, 1)])
def test_fields_of_several_threads_match_the_direct_copy(dims):
    import torch
    import paper_2112_01975_amd as P
    nx, ny, nz = dims
    D, N = (2 if nz == 1 else 3), nx * ny * nz
    nc = 3 if D == 2 else 6
    case = Case(D, nx, ny, nz, a=0.02, T_reduced=0.8)
    rv, rl = case.coexistence()
    failed = []

    def work(seed):
        try:
            rng = np.random.default_rng(seed)
            rho0 = rng.uniform(rv, rl, N)
            u0 = rng.uniform(-0.01, 0.01, (D, N))
            with P.Simulation(case.params()) as s:
                s.init(rho0, u0)
                rho, U, _ = s.moments()
                pt = P.lbm_pressure_tensor(s.ctx, N, case.params().lattice)
                buf = torch.zeros((1 + D + nc) * N, dtype=torch.float64, pin_memory=True)   # copied directly
                at = buf.data_ptr()
                tot = np.empty(4)
                assert P.lib().lbm_moments(s.ctx, at, at + 8 * N, tot.ctypes.data) == 0
                assert P.lib().lbm_pressure_tensor(s.ctx, at + 8 * (1 + D) * N) == 0
                ref = buf.numpy()
                assert np.abs(rho / rho0 - 1.0).max() <= 1e-13
                assert np.array_equal(rho, ref[:N])
                assert np.array_equal(U.ravel(), ref[N:(1 + D) * N])
                assert np.array_equal(pt.ravel(), ref[(1 + D) * N:])
                # the velocity is u plus half the force over the density: taken from zero velocity,
                # what is left is u (densities and velocities of order 1 and 0.01, 27 terms)
                s.init(rho0)
                U0 = s.moments()[1]
                assert np.abs(U - U0 - u0).max() <= 1e-13
                # an unfit density is refused wherever it is, as before
                for bad in (0.0, -1.0, np.inf, np.nan):
                    r = rho0.copy()
                    r[N - 1] = bad
                    with pytest.raises(P.LbmError):
                        s.init(r)
        except BaseException as e:
            failed.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


# 256 x 192 with both fields is more than the pinned megabyte, its density alone and 64 x 48 less
def test_batch_moments_of_small_and_large_cases():
    import ctypes as C
    import paper_2112_01975_amd as P
    cases = [Case(2, 64, 48, a=0.02, T_reduced=0.8), Case(2, 256, 192, a=0.02, T_reduced=0.8)]
    rv, rl = cases[0].coexistence()
    rng = np.random.default_rng(11)
    b = P.lbm_batch_create([c.params() for c in cases])
    try:
        rho0 = [rng.uniform(rv, rl, c.N) for c in cases]
        for k in range(2):
            P.lbm_batch_init_fields(b, k, rho0[k])
        for k, c in enumerate(cases):
            got = []
            for want_rho, want_u in ((1, 1), (1, 0), (0, 1), (0, 0)):
                rho, U, tot = np.full(c.N, -7.0), np.full((2, c.N), -7.0), np.empty(4)
                rc = P.lib().lbm_batch_moments(b, k, rho.ctypes.data_as(C.c_void_p) if want_rho else None,
                                               U.ctypes.data_as(C.c_void_p) if want_u else None, tot.ctypes.data_as(C.c_void_p))
                assert rc == 0
                got.append((rho, U, tot))
            with P.Simulation(c.params()) as s:
                s.init(rho0[k])
                r1, U1, t1 = s.moments()
            rho, U, tot = got[0]
            assert np.abs(rho / rho0[k] - 1.0).max() <= 1e-13
            assert np.abs(U - U1).max() <= 1e-10
            assert abs(tot[0] - t1[0]) <= 1e-12 * t1[0]
            assert np.array_equal(got[1][0], rho) and np.all(got[1][1] == -7.0)
            assert np.array_equal(got[2][1], U) and np.all(got[2][0] == -7.0)
            assert all(np.array_equal(g[2], tot) for g in got[1:])
    finally:
        P.lbm_batch_destroy(b)


# the copies are ordered with what the caller queued on its per-thread stream: populations read with
# steps still queued, and populations set with steps still queued, fields of more than 4 MiB
def test_copies_are_ordered_on_the_per_thread_stream():
    import paper_2112_01975_amd as P
    case = Case(3, 128, 128, 96, a=0.02, T_reduced=0.8)
    rv, rl = case.coexistence()
    rho0 = np.random.default_rng(3).uniform(rv, rl, case.N)
    got = []
    for handle in (None, 2):   # the context's own stream, hipStreamPerThread
        with P.Simulation(case.params(check_every=-1)) as s:
            P.lbm_set_stream(s.ctx, handle)
            s.init(rho0)
            first = P.lbm_get_populations(s.ctx)
            s.step(25)
            after = P.lbm_get_populations(s.ctx)
            s.step(25)
            P.lbm_set_populations(s.ctx, first)
            s.step(25)
            got.append((after, P.lbm_get_populations(s.ctx)))
    assert np.array_equal(got[0][0], got[0][1])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


# device and pinned arrays get the same values as pageable ones, for small cases and large
def test_batch_moments_into_device_and_pinned_arrays():
    import ctypes as C
    import torch
    import paper_2112_01975_amd as P
    cases = [Case(2, 64, 48, a=0.02, T_reduced=0.8), Case(2, 256, 192, a=0.02, T_reduced=0.8)]
    rv, rl = cases[0].coexistence()
    rng = np.random.default_rng(12)
    b = P.lbm_batch_create([c.params() for c in cases])
    try:
        for k, c in enumerate(cases):
            P.lbm_batch_init_fields(b, k, rng.uniform(rv, rl, c.N))
        for k, c in enumerate(cases):
            rho, U, tot = np.empty(c.N), np.empty((2, c.N)), np.empty(4)
            ptr = [x.ctypes.data_as(C.c_void_p) for x in (rho, U, tot)]
            assert P.lib().lbm_batch_moments(b, k, *ptr) == 0
            for mem in (torch.zeros(3 * c.N, dtype=torch.float64, device="cuda"),
                        torch.zeros(3 * c.N, dtype=torch.float64, pin_memory=True)):
                torch.cuda.synchronize()
                at, t = mem.data_ptr(), np.empty(4)
                assert P.lib().lbm_batch_moments(b, k, C.c_void_p(at), C.c_void_p(at + 8 * c.N), t.ctypes.data_as(C.c_void_p)) == 0
                got = mem.cpu().numpy()
                assert np.array_equal(got[:c.N], rho) and np.array_equal(got[c.N:], U.ravel()) and np.array_equal(t, tot)
    finally:
        P.lbm_batch_destroy(b)


# fields and populations of more than 20 MiB each, which go up through the workers too; padded rows
@pytest.mark.parametrize("dims,prec", [((192, 176, 170), 0), ((250, 240, 190), 1)])
def test_large_uploads(dims, prec):
    import paper_2112_01975_amd as P
    case = Case(3, *dims, a=0.02, T_reduced=0.8)
    rv, rl = case.coexistence()
    rng = np.random.default_rng(61)
    rho0, u0 = rng.uniform(rv, rl, case.N), rng.uniform(-0.01, 0.01, (3, case.N))
    with P.Simulation(case.params(prec, rv if prec else 0.0)) as s:
        s.init(rho0, u0)
        rho, U, _ = s.moments()
        assert np.abs(rho / rho0 - 1.0).max() <= (1e-13 if prec == 0 else 2e-6)   # 27 terms of 2**-52 or 2**-24
        pops = P.lbm_get_populations(s.ctx)
        s.step(1)
        P.lbm_set_populations(s.ctx, pops)
        assert np.array_equal(P.lbm_get_populations(s.ctx), pops)
        r2, U2, _ = s.moments()
        assert np.array_equal(r2, rho) and np.array_equal(U2, U)
