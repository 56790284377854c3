"""GPU: the FP8 forward pass against the FP64 oracle where its strips of 122 columns have edges, the whole grid up to its
sides: exact on a net whose values FP8 holds, for one strip less, exactly and more than full, and a strip of a column."""
import gc

import numpy as np
import pytest
import torch

from test_gpu_cnn_fp8 import _activations, _dev, _square_mesh, exact_net

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def C():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_18379_amd import cnnsns
    cnnsns.lib()
    yield cnnsns
    gc.collect()


@pytest.mark.parametrize("G", [1, 2, 3, 8, 121, 122, 123, 125, 244, 245, 367])
def test_fp8_exact_at_strip_edges(C, oracle_mod, G):
    rng = np.random.default_rng(G)
    vel = rng.integers(-3, 4, size=(2, G, G)).astype(np.float32)
    ws, bs = exact_net(G)
    assert max(a.max() for a in _activations(vel, ws, bs)) <= 16  # every value e4m3 holds
    mesh = _square_mesh(C, G)
    disp = C.predict(mesh, _dev(vel), C.Weights(ws, bs), "fp8").cpu().numpy()
    mesh.close()
    assert np.array_equal(disp.astype(np.float64), oracle_mod.cnn_forward(vel, ws, bs))
