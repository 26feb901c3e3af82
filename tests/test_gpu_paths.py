"""The paths that a size picks, at the sizes where they change: each against
the path next to it on the same input, or against the oracle."""
import numpy as np
import pytest

from gpu_common import announce, host, require_gpu, to_dev, torch
from oracle import opt as oopt

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return require_gpu()


@pytest.mark.parametrize("nx,ny", [(1, 1), (63, 64), (65, 2047), (2048, 2049), (5000, 32767), (32768, 32768)])
@pytest.mark.parametrize("kind", ["uniform", "clustered"])
def test_small_cloud_sort_equals_the_general_one(dev, nx, ny, kind):
    """Clouds of up to 32768 points are sorted in two launches, larger ones in
    five. The search is exact either way, so a target made longer by points too
    far away to be anyone's neighbour gives the same neighbours and distances,
    bit for bit. Clustered: cells that hold most of the points (one cell across
    many workgroups' shares), a NaN and an infinite point."""
    from paper_2106_03452_amd import optimize as O
    announce(f"chamfer sort {nx} x {ny} {kind}")
    rng = np.random.default_rng(nx + 3 * ny)
    x, y = rng.random((nx, 3)).astype(np.float32), rng.random((ny, 3)).astype(np.float32)
    if kind == "clustered":
        for c in (x, y):
            k = len(c) * 3 // 4
            c[:k] = 0.41 + 0.01 * c[:k]
            if len(c) > 100:
                c[7, 1], c[11, 2] = np.nan, np.inf
                c[20:40] = c[50:70]  # equal distances: the lower index
    far = np.full((32769 - ny, 3), 1e6, np.float32)
    small = O.chamfer_raw(to_dev(x, dev), to_dev(y, dev))
    general = O.chamfer_raw(to_dev(x, dev), to_dev(np.concatenate([y, far]), dev))
    # a point at infinity is as far from every finite one: the added ones do not change its neighbour either
    for s, g in zip(small[1:3], general[1:3]):
        assert torch.equal(s, g)
    for s, g in zip(small[3:], general[3:]):
        assert torch.equal(s, g[:ny])


@pytest.mark.parametrize("nx,ny", [(2, 1023), (1024, 1025), (2048, 3071), (3072, 3072), (3073, 100), (100, 3073)])
@pytest.mark.parametrize("kind", ["uniform", "clustered"])
def test_one_workgroup_sort_equals_the_general_one(dev, nx, ny, kind):
    """Clouds of up to 3072 points are sorted in one launch."""
    test_small_cloud_sort_equals_the_general_one(dev, nx, ny, kind)


@pytest.mark.parametrize("nf", [1, 1023, 1024, 1025, 65537, (1 << 20) + 1025])
def test_sampling_across_scan_blocks(dev, nf):
    """Running areas are kept per block of 1024 faces; above 1024 blocks the
    block sums are scanned in a launch of their own."""
    from paper_2106_03452_amd import optimize as O
    announce(f"sampling of {nf} faces")
    rng = np.random.default_rng(nf)
    v = rng.random((nf + 2, 3)).astype(np.float32)
    f = (np.arange(nf)[:, None] + np.arange(3)).astype(np.int32)
    w = (np.arange(nf) % 5 != 1).astype(np.float32)
    u = rng.random((777, 3)).astype(np.float32)
    u[0], u[1] = 0.0, np.nextafter(np.float32(1), np.float32(0))
    pts, _, face, bary = O.sample_raw(to_dev(v, dev), torch.from_numpy(f).to(dev), to_dev(u, dev),
                                      face_weight=to_dev(w, dev))
    ref = oopt.sample_mesh(v, f, u, None, w)
    assert np.array_equal(host(face), ref["face"])
    assert np.abs(host(pts) - ref["points"]).max() <= 1e-6
    assert np.abs(host(bary) - ref["bary"]).max() <= 1e-6


def test_chamfer_gradient_takes_the_factor_in_or_out(dev):
    """The kernel multiplies by the loss' gradient; a graph of the backward and
    batched gradients get the product as an operation of its own."""
    from paper_2106_03452_amd import optimize as O
    announce("chamfer gradient times a factor")
    rng = np.random.default_rng(4)
    x = to_dev(rng.random((3000, 3)).astype(np.float32), dev).requires_grad_(True)
    y = to_dev(rng.random((2000, 3)).astype(np.float32), dev)
    c = torch.tensor([0.5, 3.0], device=dev, requires_grad=True)
    ref = oopt.chamfer(host(x), host(y))["grad"]
    plain, = torch.autograd.grad(O.ChamferFunction.apply(x, y) * c[1], x)
    graph, = torch.autograd.grad(O.ChamferFunction.apply(x, y) * c[1], x, create_graph=True)
    batch, = torch.autograd.grad(O.ChamferFunction.apply(x, y), x, c.detach(), is_grads_batched=True)
    dc, = torch.autograd.grad(graph.sum(), c)
    tol = 1e-5 * 3 * np.abs(ref).max()
    for got, k in ((plain, 3.0), (graph, 3.0), (batch[0], 0.5), (batch[1], 3.0)):
        assert np.abs(host(got) - k * ref).max() <= tol
    # d(sum(c x grad)) / dc; 9000 terms summed in float32
    assert dc[0] == 0 and abs(float(dc[1]) - ref.sum()) <= 9000 * tol


@pytest.mark.parametrize("nf", [12, 1025, (1 << 20) + 1025])
def test_many_samples_equal_few(dev, nf):
    """Above 65536 samples four wavefronts are a workgroup; a sample depends on
    its own random numbers only, so the two kernels give the same ones, bit for bit."""
    from paper_2106_03452_amd import optimize as O
    announce(f"many samples of {nf} faces")
    rng = np.random.default_rng(nf)
    v, n = (to_dev(rng.random((nf + 2, 3)), dev) for _ in range(2))
    f = torch.from_numpy((np.arange(nf)[:, None] + np.arange(3)).astype(np.int32)).to(dev)
    u = to_dev(rng.random((65536 + 257, 3)), dev)
    many = O.sample_raw(v, f, u, n)
    for part in (slice(0, 65536), slice(65536 - 64, None)):
        for a, b in zip(many, O.sample_raw(v, f, u[part], n)):
            assert torch.equal(a[part], b)


def test_strided_arguments_give_the_contiguous_results(dev):
    """Equally sized strided clouds, and faces that are columns of a wider array."""
    from paper_2106_03452_amd import optimize as O
    announce("strided arguments of sampling and chamfer")
    rng = np.random.default_rng(8)
    x, y = (to_dev(rng.random((3000, 3)), dev) for _ in range(2))
    v, u = (to_dev(rng.random((3000, 3)), dev) for _ in range(2))
    f = torch.from_numpy(rng.integers(0, 3000, (5000, 3)).astype(np.int32)).to(dev)
    wide = torch.cat([f, torch.full_like(f, 2999)], 1)
    strided = lambda t: t.t().contiguous().t()
    for a, b in zip(O.chamfer_raw(strided(x), strided(y)), O.chamfer_raw(x, y)):
        assert torch.equal(a, b)
    for a, b in zip(O.sample_raw(strided(v), wide[:, :3], strided(u), strided(y)), O.sample_raw(v, f, u, y)):
        assert torch.equal(a, b)
    grads = []
    for faces, g in ((f, y), (wide[:, :3], strided(y)), (strided(f), y)):
        w = v.clone().requires_grad_(True)
        grads.append(torch.autograd.grad(O.SampleFunction.apply(w, faces, u), w, g)[0])
    # a vertex gets about five terms of up to 1 by float atomics, in any order
    for g in grads[1:]:
        assert float((g - grads[0]).abs().max()) <= 1e-5


def _cloud(kind, points, seed=0):
    """Clouds that reach few planes and row tiles, or all of them."""
    rng = np.random.default_rng(seed)
    p = rng.random((points, 3))
    if kind == "sheet":  # two neighbouring planes, at the domain's edge
        p[:, 0] = 0.999 + 0.002 * p[:, 0]
    elif kind == "rod":  # a few rows of every plane
        p[:, 1] = 0.49 + 0.004 * p[:, 1]
    elif kind == "ball":
        p = 0.5 + 0.2 * (p - 0.5)
    n = rng.standard_normal((points, 3))
    return p.astype(np.float32), n.astype(np.float32)


@pytest.mark.parametrize("res", [32, 64, 128])
@pytest.mark.parametrize("points", [1, 1023, 1024, 1025, 32768, 32769, 131072])
def test_two_launch_sort_equals_three(dev, res, points):
    """Up to 131072 points are sorted in two launches. The splat is an exact sum,
    so points with zero normals, as many as take the cloud to the other path,
    leave the raster as it is, bit for bit. One point is not finite."""
    from paper_2106_03452_amd import function as F
    announce(f"sort {res}^3, {points} points")
    p, n = _cloud("ball", points, points)
    if points > 1:
        p[points // 2, 1] = np.nan
    more = 131073 - points
    two = F.debug_splat(to_dev(p, dev), to_dev(n, dev), res)
    three = F.debug_splat(to_dev(np.concatenate([p, _cloud("all", more)[0]]), dev),
                          to_dev(np.concatenate([n, np.zeros((more, 3))]), dev), res)
    assert torch.equal(two, three)
    assert float(two.abs().max()) > 0


@pytest.mark.parametrize("res", [8, 16, 32, 64, 128, 256, 512])
@pytest.mark.parametrize("kind", ["one", "sheet", "rod", "ball", "all"])
def test_nothing_unwritten_is_read(dev, res, kind):
    """Planes and row tiles without a point are neither written nor read: the
    solve and its gradients must not depend on what the buffers held before
    (zeros, or bytes that read as NaN)."""
    from paper_2106_03452_amd import _lib, function as F
    announce(f"stale scratch {res}^3 {kind}")
    p, n = (to_dev(a, dev) for a in _cloud(kind, 1 if kind == "one" else 3000, res))
    P = p.shape[0]
    g = torch.randn((res,) * 3, generator=torch.Generator(device=dev).manual_seed(res), device=dev)
    out = []
    for byte in (0, 255):
        ws = torch.full((_lib.workspace_bytes(res, P),), byte, dtype=torch.uint8, device=dev)
        stale = torch.full((_lib.saved_bytes(res, P),), byte, dtype=torch.uint8, device=dev)
        del stale  # the allocator hands it out again as the saved state
        chi, saved = F.forward(p, n, res, workspace=ws)
        ws.fill_(byte)
        out.append((chi, *F.backward(chi, saved, g, P, res, workspace=ws)))
    for a, b in zip(*out):
        assert bool(torch.isfinite(a).all()) and torch.equal(a, b)


@pytest.mark.parametrize("res,slabs", [(16, 16), (64, 1), (64, 8), (256, 4)])
@pytest.mark.parametrize("kind", ["one", "sheet", "rod", "all"])
def test_slab_solve_reads_nothing_unwritten(dev, res, slabs, kind):
    from paper_2106_03452_amd import slab as S
    announce(f"slab stale scratch {res}^3 / {slabs} {kind}")
    p, n = (to_dev(a, dev) for a in _cloud(kind, 1 if kind == "one" else 3000, res))
    out = []
    for byte in (0, 255):
        ws = torch.full((S.workspace_bytes(res, p.shape[0], slabs),), byte, dtype=torch.uint8, device=dev)
        out.append(S.forward(p, n, res, slabs=slabs, workspace=ws)[0])
    assert bool(torch.isfinite(out[0]).all()) and torch.equal(*out)


@pytest.mark.parametrize("res,slabs", [(256, (1, 2, 64)), (512, (2, 8, 16, 64)), (1024, (1, 8, 64))])
@pytest.mark.parametrize("kind", ["one", "rod", "all"])
def test_large_slab_solves_do_not_depend_on_the_slabs(dev, res, slabs, kind):
    """Few slabs share out lists of live row tiles, many take a tile per workgroup;
    the largest grids have 8-column tiles and planes of 16 or 64 row tiles, up to
    all of them live and up to 96 items on a workgroup's list. The same grid bit
    for bit, whatever the workspace held."""
    from paper_2106_03452_amd import slab as S
    announce(f"slab counts {res}^3 {slabs} {kind}")
    p, n = (to_dev(a, dev) for a in _cloud(kind, {"one": 1, "rod": 3000, "all": 300000}[kind], res))
    out = []
    for k, g in enumerate(slabs):
        ws = torch.full((S.workspace_bytes(res, p.shape[0], g),), 255 * (k % 2), dtype=torch.uint8, device=dev)
        out.append(S.forward(p, n, res, slabs=g, workspace=ws)[0])
        del ws
        assert bool(torch.isfinite(out[0]).all()) and torch.equal(out[0], out[-1])
        del out[1:]


@pytest.mark.parametrize("res", [32, 64, 128])
@pytest.mark.parametrize("kind", ["sheet", "ball", "all"])
def test_single_and_batched_solves_agree(dev, res, kind):
    """A single solve up to 128^3 transforms s G and W apart and adds them in the
    j0 pass, a batch transforms their sum: the same in exact arithmetic; both
    round to float32 (the oracle tests' bound on either is 1e-5)."""
    from paper_2106_03452_amd import batch as B, function as F
    announce(f"single against batch {res}^3 {kind}")
    jobs = []
    for seed in (1, 2):
        p, n = (to_dev(a, dev) for a in _cloud(kind, 2000 * seed, seed))
        g = torch.randn((res,) * 3, generator=torch.Generator(device=dev).manual_seed(seed), device=dev)
        jobs.append(B.Job(p, n, res, 2.0, g))
    plan = B.BatchPlan(jobs)
    for ws in plan.ws:
        ws.fill_(255)
    plan.run()
    for j, (chi, dp, dn) in zip(jobs, plan.results()):
        p, n = j.points.clone().requires_grad_(True), j.normals.clone().requires_grad_(True)
        one = F.solve(p, n, res)
        grads = torch.autograd.grad(one, (p, n), j.dchi)
        for a, b in zip((chi, dp, dn), (one.detach(), *grads)):
            assert float((a - b).norm()) <= 2e-5 * float(b.norm())


@pytest.mark.parametrize("res", [8, 64, 128, 256])
@pytest.mark.parametrize("kind", ["blobs", "empty", "full"])
def test_sized_marching_cubes_equals_the_plain_call(dev, res, kind):
    """The totals arrive before the mesh is written; capacities that are too small
    give the same totals."""
    import ctypes
    from paper_2106_03452_amd import _lib, mesh as M
    announce(f"sized marching cubes {res}^3 {kind}")
    g = torch.Generator(device=dev).manual_seed(res)
    x = torch.nn.functional.interpolate(torch.randn((1, 1, 4, 4, 4), generator=g, device=dev), size=(res,) * 3,
                                        mode="trilinear")[0, 0].contiguous()
    chi = {"blobs": x, "empty": torch.ones_like(x), "full": torch.randn((res,) * 3, generator=g, device=dev)}[kind]
    L, ctx, dv = _lib.lib(), _lib.context(0), torch.device(dev)
    stream = torch.cuda.current_stream(dv).cuda_stream
    cap_v, cap_t = (3 * res ** 3, 5 * res ** 3) if kind == "full" else (64 * res * res, 128 * res * res)
    got = []
    for sized, vcap, tcap in ((False, cap_v, cap_t), (True, cap_v, cap_t), (True, 1, 1)):
        state = torch.empty(M.state_bytes(res), dtype=torch.uint8, device=dv)
        v, vn = torch.zeros((vcap, 3), device=dv), torch.zeros((vcap, 3), device=dv)
        e = torch.zeros((vcap,), dtype=torch.int32, device=dv)
        t = torch.zeros((tcap, 3), dtype=torch.int32, device=dv)
        nv, nt, st = ctypes.c_int64(-1), ctypes.c_int64(-1), ctypes.c_int(-1)
        tot = (ctypes.byref(nv), ctypes.byref(nt), ctypes.byref(st))
        args = (ctx.handle, chi.data_ptr(), res, 0.0, v.data_ptr(), vn.data_ptr(), e.data_ptr(), vcap, t.data_ptr(), tcap,
                state.data_ptr())
        if sized:
            _lib.check(L.psr_marching_cubes_sized(*args, *tot, stream), "sized")
        else:
            _lib.check(L.psr_marching_cubes(*args, stream), "plain")
            _lib.check(L.psr_mc_counts(state.data_ptr(), stream, *tot), "counts")
        got.append(((nv.value, nt.value, st.value), (v, vn, e, t)))
    assert got[0][0] == got[1][0] == got[2][0] and got[0][0][2] == 0
    assert (got[0][0][0] == 0) == (kind == "empty")
    for a, b in zip(got[0][1], got[1][1]):
        assert torch.equal(a, b)
