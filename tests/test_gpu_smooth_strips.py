"""The marching passes of the Cahn-Hilliard smoothing at the sizes where they
can go wrong (needs a device): images a node wider, narrower and as wide as
the strips' 48 (2D, four steps a pass) or 60 columns, rows and slabs around the
strip heights, images narrower than a strip's overlap, every remainder of the
steps against four, and buffers that overlap the working planes.

Bar: one Euler step from |c| <= 1 rounds by a few units of 6e-8, and the scheme
inside its stability bound does not amplify them, so ten steps stay within
2e-6 of the FP64 oracle."""

import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TOL = 2e-6


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2510_18688_amd import lbf, porous
    lbf.load()
    return porous


CASES = [((8, 47), 4), ((9, 48), 5), ((7, 49), 6), ((45, 97), 7), ((3, 145), 9), ((64, 5), 4), ((2, 2), 8),
         ((4, 14, 60), 1), ((5, 15, 59), 2), ((3, 13, 61), 3), ((9, 29, 121), 2), ((2, 1, 7), 3), ((17, 3, 2), 4)]


@pytest.mark.parametrize("wrap", [False, True])
@pytest.mark.parametrize("shape, iters", CASES)
def test_strip_edges_match_oracle(P, shape, iters, wrap):
    from oracle import ch_oracle
    rng = np.random.default_rng(sum(shape) + iters)
    img = (rng.random(shape) < 0.5).astype(np.uint8)
    per = (wrap, not wrap, wrap)[:len(shape)]
    g = P.ch_smooth(img, per, iters)
    o = ch_oracle.smooth(img, per, iters)
    err = float(np.abs(g.astype(np.float64) - o).max())
    assert err <= TOL, (shape, iters, wrap, err)


@pytest.mark.parametrize("shape, iters", [((40, 100), 3), ((40, 100), 10), ((6, 20, 70), 1), ((6, 20, 70), 4)])
def test_result_inside_the_workspace(P, shape, iters):
    """phi0 may lie in the caller's workspace: the same values as elsewhere."""
    import torch
    from paper_2510_18688_amd import lbf
    L = lbf.load()
    P._declare(L)
    rng = np.random.default_rng(iters)
    img = torch.as_tensor((rng.random(shape) < 0.5).astype(np.uint8), device="cuda")
    per = (False, True, False)[:len(shape)]
    want = P.ch_smooth(img, per, iters)
    p = P.ch_params(shape, per)
    need = L.lbf_ch_workspace_bytes(p.nx, p.ny, p.nz)
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    for off in (0, need // 2):
        ws = torch.empty(need, dtype=torch.uint8, device="cuda")
        lbf.check(L.lbf_ch_smooth(C.byref(p), C.c_void_p(img.data_ptr()), 1, C.c_void_p(ws.data_ptr() + off), 1,
                                  iters, st, C.c_void_p(ws.data_ptr()), need))
        got = ws[off:off + 4 * img.numel()].view(torch.float32).reshape(shape)
        assert torch.equal(got, want), off


@pytest.mark.parametrize("tail, iters", [((1,), 4), ((1, 1), 1)])
def test_longest_columns(P, tail, iters):
    """One column of close to 2^31 nodes: strips of the last rows and slabs end where the
    image does.  The image repeats every 4099 nodes, so the result does, away from the
    walls; near them it is that of the image's first and last nodes alone."""
    import torch
    from paper_2510_18688_amd import lbf
    L = lbf.load()
    P._declare(L)
    p, n = 4099, 2 ** 31 - 20000
    need = L.lbf_ch_workspace_bytes(n, 1, 1)
    if torch.cuda.mem_get_info()[0] < 1.3 * (need + 7 * n):
        pytest.skip("needs 41 GB of device memory")
    g = torch.Generator().manual_seed(3)
    tile = (torch.rand(p, generator=g) < 0.5).to(torch.uint8).cuda()
    img = tile.repeat(n // p + 1)[:n]

    def smooth(a):
        out = torch.empty(a.numel(), dtype=torch.float32, device="cuda")
        q = P.ch_params((a.numel(),) + tail, (False,) * (1 + len(tail)))
        size = L.lbf_ch_workspace_bytes(q.nx, q.ny, q.nz)
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        lbf.check(L.lbf_ch_smooth(C.byref(q), C.c_void_p(a.data_ptr()), 1, C.c_void_p(out.data_ptr()), 1, iters,
                                  C.c_void_p(torch.cuda.current_stream().cuda_stream), C.c_void_p(ws.data_ptr()), size))
        return out

    got = smooth(img)
    first, last = smooth(img[:3 * p].clone()), smooth(img[-3 * p:].clone())
    m = n // p
    assert bool((got[p:(m - 1) * p].view(m - 2, p) == first[p:2 * p]).all())
    assert torch.equal(got[:p], first[:p]) and torch.equal(got[-2 * p:], last[-2 * p:])


@pytest.mark.parametrize("wrap", [False, True])
@pytest.mark.parametrize("ny", [1, 2, 3, 4, 6, 7, 10, 11, 13, 14, 15, 17])
def test_columns_of_few_rows(P, ny, wrap):
    """3D images whose last strip leaves some of a workgroup's wavefronts (four rows each,
    the first from -1) without rows."""
    from oracle import ch_oracle
    shape = (9, ny, 7)
    img = (np.random.default_rng(ny).random(shape) < 0.5).astype(np.uint8)
    per = (wrap, wrap, not wrap)
    err = float(np.abs(P.ch_smooth(img, per, 3).astype(np.float64) - ch_oracle.smooth(img, per, 3)).max())
    assert err <= TOL, (ny, wrap, err)
