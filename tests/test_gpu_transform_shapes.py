"""The dense update where its kernels change shape: input and output widths on either side of 128, row counts at the
edges of their tiles and of a second turn, and one of the two gradients asked for alone."""
import numpy as np
import pytest
import torch

from parity import assert_close, to_device, to_f64
from test_gpu_transform import bits, dev, test_transform_fwd_bwd as check  # noqa: F401
from workloads import make_features

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [63, 64, 65, 127, 129])
@pytest.mark.parametrize("Fin,Fout", [(256, 128), (224, 96), (160, 32), (128, 256), (32, 224), (192, 224)])
def test_tile_edges(dev, oracle, n, Fin, Fout):  # noqa: F811
    check(dev, oracle, n, Fin, Fout, True)


@pytest.mark.parametrize("n", [32 * 256 + 1, 64 * 256 + 1, 2 * 128 * 256 + 77])
@pytest.mark.parametrize("Fin,Fout", [(256, 128), (128, 128), (256, 256)])
def test_second_turn(dev, oracle, n, Fin, Fout):  # noqa: F811
    check(dev, oracle, n, Fin, Fout, False)


@pytest.mark.parametrize("Fin,Fout", [(128, 128), (96, 64), (256, 160)])
def test_one_gradient_alone(dev, Fin, Fout):  # noqa: F811
    B, n = dev.B, 777
    P = to_device(make_features(n, Fin, 0.5, 1, "bf16"), "bf16")
    W = to_device(make_features(Fin, Fout, Fin ** -0.5, 2, "bf16"), "bf16")
    gH = to_device(make_features(n, Fout, 1.0, 3, "bf16"), "bf16")
    H = dev.layer_transform_fwd(P, W, True)
    gP, gW = dev.layer_transform_bwd(P, W, H, gH, True)
    ws = torch.empty(B.e2eg_layer_transform_workspace_bytes(1, n, Fin, Fout, B.E2EG_BF16), dtype=torch.uint8, device="cuda")
    gP1, gW1 = torch.zeros_like(gP), torch.zeros_like(gW)
    stream = torch.cuda.current_stream().cuda_stream
    B.e2eg_layer_transform(1, n, Fin, Fout, B.E2EG_BF16, 1, P, W, H, gH, gP1, None, ws, None, stream)
    B.e2eg_layer_transform(1, n, Fin, Fout, B.E2EG_BF16, 1, P, W, H, gH, None, gW1, ws, None, stream)
    assert torch.equal(gP, gP1) and torch.equal(gW, gW1)
