"""GPU: the forward passes at the ends of the number range.  Velocities up to FP32's largest finite value give the displacements
of the FP64 oracle (the FP32 pass; both its forms); and a velocity that is not a number, or infinite, reaches no cell that
the network's four layers do not connect with it."""
import gc

import numpy as np
import pytest
import torch

from test_gpu_cnn import _dev, _square_mesh, _within

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_18379_amd import cnnsns
    cnnsns.lib()
    yield cnnsns
    gc.collect()


@pytest.mark.parametrize("G", [33, 128, 200, 600])
@pytest.mark.parametrize("top", [3.389e38, 3.39e38, 3.4e38, np.finfo(np.float32).max])
def test_largest_velocities(C, oracle_mod, wl, G, top):
    """The FP32 bar of test_gpu_cnn.py, 1e-5 relative plus 1e-5 of the channel's maximum; the first layer's weights are small, so
    that no later layer leaves the range."""
    rng = np.random.default_rng(G)
    vel = (rng.uniform(-1.0, 1.0, (2, G, G)) * top).astype(np.float32)
    vel[0, ::7, ::5] = top
    vel[1, ::5, ::7] = -top
    ws, bs = wl.random_weights(G)
    ws[0] = (ws[0] * 1e-3).astype(np.float32)
    mesh = _square_mesh(C, G)
    disp = C.predict(mesh, _dev(vel), C.Weights(ws, bs), "f32").cpu().numpy()
    mesh.close()
    assert np.isfinite(disp).all()
    assert _within(disp, oracle_mod.cnn_forward(vel, ws, bs)) <= 1.0


def _far(at, shape):
    """The cells more than four from `at` in some direction."""
    d = np.zeros(shape, dtype=int)
    for axis, (a, n) in enumerate(zip(at, shape)):
        d = np.maximum(d, np.abs(np.arange(n) - a).reshape([-1 if k == axis else 1 for k in range(len(shape))]))
    return d > 4


@pytest.mark.parametrize("G", [40, 200, 600])
@pytest.mark.parametrize("precision, value", [("f32", np.nan), ("f32", np.inf), ("f32", -np.inf), ("bf16", np.nan), ("bf16", np.inf),
                                              ("fp8", np.nan)])
def test_not_finite_stays_near(C, wl, G, precision, value):
    rng = np.random.default_rng(G)
    vel = rng.standard_normal((2, G, G)).astype(np.float32)
    W = C.Weights(*wl.random_weights(G))
    mesh = _square_mesh(C, G)
    for at in ((G // 2, G // 3), (0, G - 1), (G - 1, min(255, G - 2))):
        vel[(0,) + at] = 0.0
        clean = C.predict(mesh, _dev(vel), W, precision).cpu().numpy()
        vel[(0,) + at] = value
        disp = C.predict(mesh, _dev(vel), W, precision).cpu().numpy()
        vel[(0,) + at] = 0.0
        far = _far(at, (G, G))
        assert np.array_equal(disp[:, far], clean[:, far])
    mesh.close()


@pytest.mark.parametrize("G", [12, 35])
@pytest.mark.parametrize("precision", ["f32", "bf16"])
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_not_finite_stays_near_3d(C, wl, G, precision, value):
    rng = np.random.default_rng(G)
    vel = rng.standard_normal((3, G, G, G)).astype(np.float32)
    ch = (3, 32, 32, 32, 3)
    W = C.Weights3D([(rng.standard_normal((ch[k + 1], ch[k], 3, 3, 3)) * np.sqrt(2.0 / (27 * ch[k]))).astype(np.float32) for k in range(4)],
                    [(0.1 * rng.standard_normal(c)).astype(np.float32) for c in ch[1:]])
    mesh = C.Mesh3D(*wl.kuhn_mesh(2, 1), overlay_side=G)
    for at in ((G // 2, G // 3, G // 4), (0, G - 1, min(31, G - 1))):
        vel[(0,) + at] = 0.0
        clean = C.predict3d(mesh, torch.from_numpy(vel).cuda(), W, precision).cpu().numpy()
        vel[(0,) + at] = value
        disp = C.predict3d(mesh, torch.from_numpy(vel).cuda(), W, precision).cpu().numpy()
        vel[(0,) + at] = 0.0
        far = _far(at, (G, G, G))
        assert np.array_equal(disp[:, far], clean[:, far])
    mesh.close()
