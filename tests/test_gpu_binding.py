"""What the binding hands back on the GPU: new outputs are plain tensors, whatever
kind of tensor the activations are."""
import sys

import pytest

from test_gpu_prompt import make_layer
from test_gpu_parity import grid_f32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Tagged(torch.Tensor):
    pass


@pytest.mark.parametrize("batch", [1, 80])
def test_outputs_of_tensor_subclasses_are_plain(batch):
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] binding subclass batch={batch}", file=sys.stderr, flush=True)
    p, n, g, out, inp = 2, 256, 256, 96, 512
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    codes, scales, _ = make_layer(p, n, out, inp, g, 5)
    plain = torch.randn((batch, inp), device="cuda")
    x = plain.as_subclass(Tagged)
    assert type(x.new_empty((1,))) is Tagged
    x_rot = H.rht_activations(x, g, 3)
    ys = [x_rot, H.qmatmul(x_rot.as_subclass(Tagged), codes, scales, grid, g, out),
          H.qmatmul_fused(x, codes, scales, grid, g, 3, out),
          H.qmatmul_fused_noalloc(x, codes, scales, grid, g, 3, out),
          *H.qmatmul_fused_multi(x, [(codes, scales, 3, out)] * 2, grid, g)]
    want = H.qmatmul_fused(plain, codes, scales, grid, g, 3, out)
    for y in ys:
        assert type(y) is torch.Tensor
    for y in ys[2:]:
        assert torch.equal(y, want)
