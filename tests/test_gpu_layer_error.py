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


@pytest.mark.parametrize("p,n,g,out,inp,dtype", [
    (2, 64, 2048, 1050, 16384, "bf16"),     # 8400 groups on 8192 wavefronts
    (1, 256, 2048, 1050, 16384, "f32"),
    (2, 256, 4096, 2101, 16384, "f32"),
    (1, 16, 4096, 2101, 16384, "bf16"),
])
def test_layer_error_groups_above_1024(p, n, g, out, inp, dtype):
    """Wavefronts of 32 or 64 weights per lane that take a second group."""
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] layer error p={p} n={n} g={g} {out}x{inp} {dtype}", file=sys.stderr,
          flush=True)
    grid = grid_f32(p, n)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(g + n)
    w = 0.02 * torch.randn((out, inp), generator=gen, device="cuda")
    w = w if dtype == "f32" else w.to(torch.bfloat16)
    gen.manual_seed(g)
    # codes of another layer: the error is any size, and every code occurs
    codes = torch.randint(0, 256, (out, H.codes_row_bytes(inp, p, n)), generator=gen,
                          device="cuda", dtype=torch.uint8)
    scales = (0.02 * torch.rand((out, inp // g), generator=gen, device="cuda")).half()
    t2, ge = H.layer_error(w, codes, scales, torch.from_numpy(grid).cuda(), g, 21)
    ge = ge.cpu().numpy().reshape(out, inp // g, 2)
    rows = np.r_[0:2, out // 2, out - 3:out]
    vals = w[rows].double().cpu().numpy()
    w_hat = O.dequantize(O.unpack_codes(codes.cpu().numpy()[rows], n, inp // p),
                         scales.cpu().numpy()[rows], grid.astype(np.float64), g, 21)
    shape = (len(rows), inp // g, g)
    # fp64 sums: log2(g) butterfly roundings and g terms, far below 1e-9
    assert np.allclose(ge[rows, :, 0], ((vals - w_hat) ** 2).reshape(shape).sum(axis=2),
                       rtol=1e-9, atol=0)
    assert np.allclose(ge[rows, :, 1], (vals ** 2).reshape(shape).sum(axis=2), rtol=1e-12, atol=0)
    # 1024 partial sums of about eight, then a tree
    assert abs(t2 - ge[..., 0].sum() / ge[..., 1].sum()) <= 1e-12 * t2
