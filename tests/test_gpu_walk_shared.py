"""GPU: the walk of a large batch from given starts, whose records come through LDS and whose blocks go in chunks per XCD,
against the same points in small batches, which take neither: host, path and status (and the interpolant) bit for bit.
The counts are ragged in blocks, rounds of chunks and wavefronts; among the points are starts that are no element, points
outside the mesh and, in one run each, walks cut off by max_iter."""
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


def _points(rng, n, dim, n_el):
    xp = rng.uniform(-0.02, 1.02, (n, dim))
    start = rng.integers(0, n_el, n).astype(np.int32)
    start[::1000] = rng.choice([-1, n_el, -2**31, 2**31 - 1], len(start[::1000]))
    return torch.from_numpy(xp).cuda(), torch.from_numpy(start).cuda()


def _equal(whole, parts):
    for k, t in enumerate(whole):
        assert torch.equal(t.view(torch.uint8), torch.cat([p[k] for p in parts]).view(torch.uint8))


@pytest.mark.parametrize("n", [393_217 - 64, 393_217, 401_003])
@pytest.mark.parametrize("max_iter", [0, 19])
def test_locate_shared_equals_small_batches(C, wl, n, max_iter):
    w = wl.build(n_side=60, seed=1, field="fourier", field_seed=9, U=1.0, k=3.0, origins="nodes", G=32)
    mesh = C.Mesh(w.xy, w.tri, overlay_side=32)
    xp, start = _points(np.random.default_rng(n + max_iter), n, 2, len(w.tri))
    nodal = torch.from_numpy(np.random.default_rng(2).standard_normal((len(w.xy), 2))).cuda()
    cuts = [slice(k, min(k + 131_072, n)) for k in range(0, n, 131_072)]
    _equal(C.locate(mesh, xp, start=start, max_iter=max_iter),
           [C.locate(mesh, xp[c], start=start[c], max_iter=max_iter) for c in cuts])
    _equal(C.locate_interpolate(mesh, xp, nodal, start=start, max_iter=max_iter),
           [C.locate_interpolate(mesh, xp[c], nodal, start=start[c], max_iter=max_iter) for c in cuts])
    mesh.close()


@pytest.mark.parametrize("n", [98_049 - 1, 98_049, 131_071])
@pytest.mark.parametrize("max_iter", [0, 19])
def test_locate3d_shared_equals_small_batches(C, wl, n, max_iter):
    w = wl.build_3d("t1")
    mesh = C.Mesh3D(w.xyz, w.tet, overlay_side=w.G)
    xp, start = _points(np.random.default_rng(n + max_iter), n, 3, w.n_tet)
    cuts = [slice(k, min(k + 50_000, n)) for k in range(0, n, 50_000)]
    _equal(C.locate3d(mesh, xp, start=start, max_iter=max_iter),
           [C.locate3d(mesh, xp[c], start=start[c], max_iter=max_iter) for c in cuts])
    mesh.close()
