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
