"""GPU: the BF16 and FP8 forward passes, which walk down strips of 122 output columns, where their tiling has edges: a few
rows and columns, one strip less, exactly and more than full, a strip of one column, and strips laid end to end with blocks
that cross from one to the next (G = 2320).  Bars of test_gpu_cnn.py, and the same bits wherever a pixel lies in a
strip: the pass over a window of the grid equals the pass over the whole of it, off the window's four-pixel border (for
FP8 with the same largest velocity in both, from which its scales follow; its accuracy is tested elsewhere).
"""
import gc

import numpy as np
import pytest
import torch

from test_gpu_cnn import BF16_MAX, BF16_MEAN, _bf16_errors, _dev, _square_mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_18379_amd import cnnsns
    cnnsns.lib()
    yield cnnsns
    gc.collect()


@pytest.mark.parametrize("G", [2, 3, 121, 122, 123, 125, 244, 245, 2320])
@pytest.mark.parametrize("precision", ["bf16", "fp8"])
def test_strip_edges(C, oracle_mod, wl, precision, G):
    rng = np.random.default_rng(G)
    vel = np.clip(rng.standard_normal((2, G, G)), -4.0, 4.0).astype(np.float32)
    vel[:, ::25, ::25] = 4.0
    ws, bs = wl.random_weights(G)
    W = C.Weights(ws, bs)

    def predict(v):
        mesh = _square_mesh(C, v.shape[1])
        out = C.predict(mesh, _dev(v), W, precision).cpu().numpy()
        mesh.close()
        return out

    disp = predict(vel)
    if G <= 245 and precision == "bf16":
        emax, emean = _bf16_errors(disp, oracle_mod.cnn_forward(vel, ws, bs))
        assert emax <= BF16_MAX and emean <= BF16_MEAN, (emax, emean)
    n = min(G - 37, 300)
    for y, x in ((37, 5), (G - n, G - n), (11, (G - n) // 2)) if n > 8 else ():
        part = predict(np.ascontiguousarray(vel[:, y:y + n, x:x + n]))
        assert np.array_equal(part[:, 4:-4, 4:-4], disp[:, y + 4:y + n - 4, x + 4:x + n - 4])


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("at", [0, -1])
def test_fp8_velocity_scale_at_any_alignment(C, wl, offset, at):
    """The grid's maximum is found where it is the first or last value, at every alignment of the velocity (its scale
    is what differs by a factor of 64 if it is not): the same bits as from an aligned copy with that maximum inside."""
    G = 33
    rng = np.random.default_rng(7)
    vel = rng.uniform(-1.0, 1.0, 2 * G * G).astype(np.float32)
    ws, bs = wl.random_weights(7)
    W = C.Weights(ws, bs)
    mesh = _square_mesh(C, G)
    vel[at] = 64.0
    buf = torch.zeros(2 * G * G + 3, dtype=torch.float32, device="cuda")
    view = buf[offset:offset + 2 * G * G].view(2, G, G)
    view.copy_(_dev(vel.reshape(2, G, G)))
    got = C.predict(mesh, view, W, "fp8").cpu().numpy()
    vel[G * G + G // 2 * G + G // 2] = 64.0  # 16 rows and columns from either corner: not in its pixel's window
    ref = C.predict(mesh, _dev(vel.reshape(2, G, G)), W, "fp8").cpu().numpy()
    mesh.close()
    corner = (slice(None), slice(0, 8), slice(0, 8)) if at == 0 else (slice(None), slice(-8, None), slice(-8, None))
    assert np.array_equal(got[corner], ref[corner])
