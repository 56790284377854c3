"""GPU: the row-streaming form of the FP32 forward pass against the FP64 oracle where its tiling has edges:
a strip of one column and of exactly half the wavefronts, segments of one row, and the largest overlay of
its small range."""
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
    gc.collect()  # meshes kept by reference cycles (their release synchronises the device) go now, not in a later capture


@pytest.mark.parametrize("G", [32, 127, 128, 513, 640, 832, 896, 1025])
def test_rows_form_full_grid(C, oracle_mod, wl, G):
    """The FP32 bar of test_gpu_cnn.py: 1e-5 relative plus 1e-5 of the channel's maximum."""
    rng = np.random.default_rng(G)
    vel = rng.standard_normal((2, G, G)).astype(np.float32)
    ws, bs = wl.random_weights(G)
    mesh = _square_mesh(C, G)
    disp = C.predict(mesh, _dev(vel), C.Weights(ws, bs), "f32").cpu().numpy()
    mesh.close()
    assert _within(disp, oracle_mod.cnn_forward(vel, ws, bs)) <= 1.0
