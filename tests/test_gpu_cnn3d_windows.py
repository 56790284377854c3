"""GPU: the 3D forward passes give a cell the same bits wherever it lies in a block: the pass over a window of the grid equals
the pass over the whole of it, off the window's four-cell border.  Window sides beside the 8 x 32 cells of a block, the
pairs of planes that the BF16 layers take (odd and even segments) and the planes of a block."""
import gc

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def whole():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_18379_amd import cnnsns as C
    from paper_2412_18379_amd import workload as W
    C.lib()
    G = 66
    vel = np.random.default_rng(3).standard_normal((3, G, G, G)).astype(np.float32)
    w = W.build_3d("t1")
    net = C.Weights3D(*_weights(4))

    def predict(v, precision):
        mesh = C.Mesh3D(w.xyz, w.tet, overlay_side=v.shape[1])
        out = C.predict3d(mesh, torch.from_numpy(np.ascontiguousarray(v)).cuda(), net, precision).cpu().numpy()
        mesh.close()
        return out

    yield vel, predict, {p: predict(vel, p) for p in ("bf16", "f32")}
    gc.collect()


def _weights(seed):
    rng = np.random.default_rng(seed)
    shapes = [(32, 3, 3, 3, 3), (32, 32, 3, 3, 3), (32, 32, 3, 3, 3), (3, 32, 3, 3, 3)]
    return ([(rng.standard_normal(s) * np.sqrt(2.0 / np.prod(s[1:]))).astype(np.float32) for s in shapes],
            [(0.1 * rng.standard_normal(s[0])).astype(np.float32) for s in shapes])


@pytest.mark.parametrize("n", [9, 16, 17, 31, 32, 33, 40, 65])
@pytest.mark.parametrize("precision", ["bf16", "f32"])
def test_window_equals_whole(whole, precision, n):
    vel, predict, full = whole
    G = vel.shape[1]
    for z, y, x in ((0, 0, 0), (G - n, 1, (G - n) // 2)):
        part = predict(vel[:, z:z + n, y:y + n, x:x + n], precision)
        inner = full[precision][:, z + 4:z + n - 4, y + 4:y + n - 4, x + 4:x + n - 4]
        assert np.array_equal(part[:, 4:-4, 4:-4, 4:-4], inner)
