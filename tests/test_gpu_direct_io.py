"""Initial fields taken from device memory and read-out fields written into it
without staging (needs a device): the same bits as through host memory, in
every layout, into destinations of any 4-byte alignment, with nothing written
beside the fields asked for; both lattices."""

import ctypes as C

import numpy as np
import pytest

from paper_2510_18688_amd import workloads as W, workloads3 as W3

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbf_mod():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2510_18688_amd import lbf
    lbf.load()
    return lbf


CASES = {
    "walls_131x67": lambda: W.porous_medium(nx=131, ny=67, seed=5, rmin=6.0, rmax=10.0, porosity=0.8),
    "drop_70x45": lambda: W.slab_drop(70, 45, 12.0, 75.0, -1.0),
    "one_node": lambda: W.slab_drop(1, 1, 0.3, 75.0, -1.0),
}


@pytest.mark.parametrize("mdot", [0, 1])
@pytest.mark.parametrize("rb", [0, 4])
@pytest.mark.parametrize("name", sorted(CASES))
def test_fields_2d(lbf_mod, name, rb, mdot):
    import torch
    L = lbf_mod.load()
    case = CASES[name]()
    case.mat.phi_src_mdot = mdot
    a = lbf_mod.Sim(case, row_block=rb)
    b = lbf_mod.Sim(case, row_block=rb)
    b.workspace.fill_(0xff)   # nothing of the old workspace may show
    b.set_geometry(case.phi0, case.cos_theta)
    for w in range(4):
        b.set_wall_temperature(w, case.wall_profile(w))
    b.init_fields(torch.as_tensor(case.phi, dtype=torch.float32, device="cuda").contiguous(),
                  torch.as_tensor(case.T, dtype=torch.float32, device="cuda").contiguous())
    sa = torch.empty(a.state_bytes(), dtype=torch.uint8, device="cuda")
    sb = torch.empty_like(sa)
    for steps in (0, 7):
        a.step(steps)
        b.step(steps)
        a.save_state(sa)
        b.save_state(sb)
        assert torch.equal(sa, sb), steps
        want = a.fields()
        n = case.nodes
        for shift in (0, 1):
            buf = torch.full((13 * n + 9,), -7.0, dtype=torch.float32, device="cuda")
            lbf_mod.check(L.lbf_read_fields(b.h, C.c_void_p(buf.data_ptr() + 4 * (4 + shift)), 1))
            got = buf.cpu().numpy()
            assert (got[:4 + shift] == -7.0).all() and (got[4 + shift + 13 * n:] == -7.0).all()
            got = got[4 + shift:4 + shift + 13 * n].reshape(13, case.ny, case.nx)
            for i, k in enumerate(lbf_mod.FIELDS):
                assert np.array_equal(got[i], want[k]), (k, shift)
        for k in ("phi", "p", "phihat"):
            one = torch.full((n + 2,), -7.0, dtype=torch.float32, device="cuda")
            lbf_mod.check(L.lbf_read_field(b.h, lbf_mod.FIELDS.index(k), C.c_void_p(one.data_ptr() + 4), 1))
            got = one.cpu().numpy()
            assert got[0] == -7.0 and got[-1] == -7.0
            assert np.array_equal(got[1:-1].reshape(case.ny, case.nx), want[k]), k
            assert np.array_equal(b.field(k), want[k]), k


@pytest.mark.parametrize("mdot", [0, 1])
@pytest.mark.parametrize("rb", [0, 8])
def test_fields_3d(lbf_mod, rb, mdot):
    import torch
    L = lbf_mod.load()
    case = W3.fracture(40, 22, 17, aperture=9.0)
    case.mat.phi_src_mdot = mdot
    a, b = lbf_mod.Sim3(case, row_block=rb), lbf_mod.Sim3(case, row_block=rb)
    b.workspace.fill_(0xff)
    p0, ct = (np.ascontiguousarray(v, dtype=np.float32) for v in (case.phi0, case.cos_theta))
    lbf_mod.check(L.lbf3_set_geometry(b.h, C.c_void_p(p0.ctypes.data), C.c_void_p(ct.ctypes.data), 0))
    phi, T = (torch.as_tensor(v, dtype=torch.float32, device="cuda").contiguous() for v in (case.phi, case.T))
    lbf_mod.check(L.lbf3_init_fields(b.h, C.c_void_p(phi.data_ptr()), C.c_void_p(T.data_ptr()), 1))
    sa = torch.empty(a.state_bytes(), dtype=torch.uint8, device="cuda")
    sb = torch.empty_like(sa)
    n = case.nodes
    for steps in (0, 3):
        a.step(steps)
        b.step(steps)
        a.save_state(sa)
        b.save_state(sb)
        assert torch.equal(sa, sb), steps
        buf = torch.full((14 * n + 2,), -7.0, dtype=torch.float32, device="cuda")
        lbf_mod.check(L.lbf3_read_fields(b.h, C.c_void_p(buf.data_ptr() + 4), 1))
        got = buf.cpu().numpy()
        assert got[0] == -7.0 and got[-1] == -7.0
        want = a.fields()
        for i, k in enumerate(lbf_mod.FIELDS3):
            assert np.array_equal(got[1 + i * n:1 + (i + 1) * n], want[k].ravel()), k
        assert a.reduce() == b.reduce()
