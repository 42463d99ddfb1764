"""GPU parity of the quantization error at sizes where a wavefront takes several
groups in turn, for every code width, with codes at any byte alignment."""
import sys

import numpy as np
import pytest

from oracle import higgs_oracle as O
from paper_2411_17525_amd import synth
from test_gpu_parity import grid_f32, weight_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,g,out,inp,dtype,offset", [
    (2, 64, 1024, 2101, 4096, "bf16", 1),   # 8404 groups on 8192 wavefronts
    (2, 256, 1024, 2101, 4096, "f32", 0),
    (2, 1024, 1024, 2101, 4096, "bf16", 2),
    (1, 16, 1024, 2101, 4096, "f32", 3),
    (1, 256, 1024, 2101, 4096, "bf16", 0),
    (2, 64, 512, 1050, 4096, "f32", 2),     # rotated across lanes instead of through LDS
    (1, 16, 64, 261, 2048, "bf16", 1),
])
def test_layer_error_many_groups(p, n, g, out, inp, dtype, offset):
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] layer error p={p} n={n} g={g} {out}x{inp} {dtype} +{offset}",
          file=sys.stderr, flush=True)
    grid = grid_f32(p, n)
    gd = torch.from_numpy(grid).cuda()
    wt = synth.student_t_weight(out, inp, seed=out + g, dtype=dtype)
    w = weight_dev(wt)
    codes, scales = H.quantize(w, gd, g, 21)
    moved = torch.empty(codes.numel() + offset, dtype=torch.uint8, device="cuda")[offset:]
    moved.copy_(codes.reshape(-1))
    t2, ge = H.layer_error(w, moved, scales, gd, g, 21)
    ge = ge.cpu().numpy().reshape(out, inp // g, 2)
    rows = np.r_[0:3, out // 2, out - 3:out]
    vals = wt.values[rows].astype(np.float64)
    w_hat = O.dequantize(O.unpack_codes(codes.cpu().numpy()[rows], n, inp // p),
                         scales.cpu().numpy()[rows], grid.astype(np.float64), g, 21)
    shape = (len(rows), inp // g, g)
    # fp64 sums: log2(g) butterfly roundings and g terms, far below 1e-9
    assert np.allclose(ge[rows, :, 0], ((vals - w_hat) ** 2).reshape(shape).sum(axis=2),
                       rtol=1e-9, atol=0)
    assert np.allclose(ge[rows, :, 1], (vals ** 2).reshape(shape).sum(axis=2), rtol=1e-12, atol=0)
    assert abs(t2 - ge[..., 0].sum() / ge[..., 1].sum()) <= 1e-12 * t2
