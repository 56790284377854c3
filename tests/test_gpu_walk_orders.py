"""GPU: a walk's result does not depend on how its points' blocks and records are taken: a large batch, whose blocks go in
chunks per XCD and whose records come through LDS in the wavefronts whose points lie in order, against the same points in
batches small enough (at most 64 blocks) to be walked in order of id and straight from memory: host, path, status and
interpolant bit for bit.  Points in order, in none, and in order in every other run of 64; starts that are no element,
points outside the mesh, walks cut off by max_iter; from given, CNN and overlay starts, on both sides of the batch
sizes at which the order changes."""
import gc

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_18379_amd import cnnsns
    cnnsns.lib()
    yield cnnsns
    gc.collect()


@pytest.fixture(scope="module")
def mesh2(C, wl):
    xy, tri = wl.mesh(200, 5)
    mesh = C.Mesh(xy, tri)
    yield mesh, xy, tri
    mesh.close()


@pytest.fixture(scope="module")
def mesh3(C, wl):
    xyz, tet = wl.kuhn_mesh(40, 5)
    mesh = C.Mesh3D(xyz, tet)
    yield mesh, tet
    mesh.close()


def _points(n, dim, cells, order):
    """n points, some outside the mesh: row by row of `cells` to a side, in no order, or both in turn by runs of 64."""
    x = np.random.default_rng(n + dim).uniform(-0.01, 1.01, (n, dim))
    if order == "none":
        return x
    key = [x[:, 0]] + [np.floor(x[:, d] * cells) for d in range(1, dim)]
    y = x[np.lexsort(key)]
    if order == "both":
        scattered = (np.arange(n) // 64) % 2 == 1
        y[scattered] = np.random.default_rng(1).permutation(y[scattered])
    return y


def _near_starts(x, step, lookup_of):
    """For each point the element under a point a little off it; a few that are none."""
    start = lookup_of(np.clip(x + step, 0.0, 1.0 - 1e-9))
    start[::1000] = np.random.default_rng(3).choice([-1, 2**31 - 1, -2**31], len(start[::1000]))
    return start


def _equal(whole, run, n, batch):
    parts = [run(slice(k, min(k + batch, n))) for k in range(0, n, batch)]
    for k, t in enumerate(whole):
        assert torch.equal(t.view(torch.uint8), torch.cat([p[k] for p in parts]).view(torch.uint8))


@pytest.mark.parametrize("order", ["rows", "none", "both"])
@pytest.mark.parametrize("n, max_iter", [(16_385, 0), (163_840 - 256, 0), (163_840 - 192, 11), (163_841, 0), (180_007, 11)])
def test_given_starts(C, mesh2, n, max_iter, order):
    mesh, xy, tri = mesh2
    x = _points(n, 2, 256, order)
    # the two triangles of a cell of the 199 x 199 have consecutive ids
    cell = lambda p: (2 * (np.floor(p[:, 1] * 199) * 199 + np.floor(p[:, 0] * 199))).astype(np.int32)  # noqa: E731
    start = torch.from_numpy(_near_starts(x, 0.05, cell)).cuda()
    xp = torch.from_numpy(x).cuda()
    nodal = torch.from_numpy(np.random.default_rng(2).standard_normal((len(xy), 2))).cuda()
    one = lambda c: C.locate(mesh, xp[c], start=start[c], max_iter=max_iter)  # noqa: E731
    _equal(one(slice(0, n)), one, n, 16_384)
    one = lambda c: C.locate_interpolate(mesh, xp[c], nodal, start=start[c], max_iter=max_iter)  # noqa: E731
    _equal(one(slice(0, n)), one, n, 16_384)


@pytest.mark.parametrize("order", ["rows", "none", "both"])
@pytest.mark.parametrize("n, max_iter", [(98_048, 0), (98_049, 0), (131_071, 11)])
def test_given_starts_3d(C, mesh3, n, max_iter, order):
    mesh, tet = mesh3
    x = _points(n, 3, 46, order)
    cell = lambda p: (6 * ((np.floor(p[:, 2] * 39) * 39 + np.floor(p[:, 1] * 39)) * 39 + np.floor(p[:, 0] * 39))).astype(np.int32)  # noqa: E731
    start = torch.from_numpy(_near_starts(x, 0.05, cell)).cuda()
    xp = torch.from_numpy(x).cuda()
    one = lambda c: C.locate3d(mesh, xp[c], start=start[c], max_iter=max_iter)  # noqa: E731
    _equal(one(slice(0, n)), one, n, 16_384)


@pytest.mark.parametrize("mode", ["cnn", "asg"])
@pytest.mark.parametrize("n", [32_768, 32_769, 100_003, 6_144 * 512, 6_144 * 512 + 1])
def test_looked_up_starts(C, mesh2, n, mode):
    mesh, xy, tri = mesh2
    xp = torch.from_numpy(_points(n, 2, 256, "both")).cuda()
    origin = (xp + 0.02).clamp_(0.0, 1.0)
    disp = torch.full((2, mesh.G, mesh.G), -0.015, dtype=torch.float32, device="cuda") if mode == "cnn" else None
    nodal = torch.from_numpy(np.random.default_rng(2).standard_normal((len(xy), 2))).cuda()
    kw = lambda c: dict(origin=origin[c], disp=disp) if mode == "cnn" else {}  # noqa: E731
    one = lambda c: C.locate(mesh, xp[c], **kw(c))  # noqa: E731
    _equal(one(slice(0, n)), one, n, 32_768)
    one = lambda c: C.locate_interpolate(mesh, xp[c], nodal, **kw(c))  # noqa: E731
    _equal(one(slice(0, n)), one, n, 32_768)
