"""GPU parity of the product at prompt-sized batches (more than 64 rows) against
a plain PyTorch fp64 product of the same rotated activations, codes and scales.

The sizes reach every block shape that a code width has (256 x 128 in waves of
64 x 128 or 64 x 64, 128 x 128 with two K-groups, 128 x 64 with four), with and
without a K-split (test_wide_plan.py holds them to that): one row past a tile,
ragged rows, rows of an odd number of 64-weight blocks (g = 64)."""
import sys

import numpy as np
import pytest

from paper_2411_17525_amd import synth
from test_gpu_parity import check_qmm, grid_f32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FORMATS = ((2, 64), (2, 256), (2, 1024), (1, 16), (1, 256))
# batch, out, in, g
SIZES = [
    (1000, 8200, 512, 128),
    (129, 17000, 2048, 256),
    (129, 17000, 512, 512),
    (129, 4200, 2560, 512),   # splits of two or more stages each
    (129, 4200, 5120, 256),
    (129, 9000, 5120, 128),
    (300, 9000, 4096, 1024),
    (385, 1000, 1024, 1024),
    (65, 100, 512, 128),
    (65, 100, 640, 128),      # three splits, the last one short
    (257, 513, 4096, 4096),   # one group per row
]
SIZES_G64 = [
    (129, 17000, 512, 64),
    (65, 12000, 1088, 64),
    (129, 9000, 4160, 64),
    (128, 129, 576, 64),    # three splits, the last one stage
    (65, 100, 1088, 64),    # five splits, the last one stage
    (257, 2000, 576, 64),
    (64, 1500, 1088, 64),
    (17, 129, 576, 64),
    (33, 12000, 640, 64),   # K-groups of four and two stages, one of none
    (49, 200, 6208, 64),    # long rows start at 49 rows (16 points)
]
CASES = [(p, n) + s for p, n in FORMATS for s in SIZES]
CASES += [(p, n) + s for p, n in FORMATS if p == 1 for s in SIZES_G64]
# scalar 256-point grid: 128 x 64 blocks from 33 rows (g = 128) or 9 (g = 64)
CASES += [(1, 256, 33, 300, 640, 128), (1, 256, 64, 12000, 2048, 128), (1, 256, 9, 131, 512, 64),
          (1, 256, 33, 300, 8192, 128), (1, 256, 33, 200, 6208, 64)]
# partial sums of 12, 20 or more and 28 splits
CASES += [(2, 256, 65, 100, 9216, 1024), (1, 16, 70, 33, 20480, 1024), (1, 256, 33, 300, 28672, 128)]
# activations converted by blocks of 16 waves (from 4096 groups): a last block
# of four waves; waves with two groups, the second pass partial
CASES += [(2, 256, 1025, 129, 4096, 1024), (1, 16, 137, 131, 4160, 64), (2, 64, 300, 100, 4096, 128)]
# by a block per group (g = 4096, and 2048 up to 1400 groups)
CASES += [(2, 256, 70, 100, 4096, 2048), (1, 16, 1401, 33, 2048, 2048), (2, 64, 131, 70, 12288, 4096)]


def make_layer(p, n, out, inp, g, seed):
    from oracle import higgs_oracle as O
    idx = synth.random_codes(out, inp // p, n, seed)
    scales = synth.random_scales_f16(out, inp // g, seed + 1)
    codes = torch.from_numpy(O.pack_codes(idx, n)).cuda()
    return (codes, torch.from_numpy(scales.view(np.int16)).cuda().view(torch.float16),
            torch.from_numpy(idx.astype(np.int64)).cuda())


def reference(x_rot, idx, scales, grid, g):
    """fp64 product and the sum of its terms' magnitudes."""
    out, inp = idx.shape[0], x_rot.shape[1]
    w = grid.double()[idx].reshape(out, inp // g, g) * scales.double()[:, :, None]
    w = w.reshape(out, inp)
    return x_rot.double() @ w.t(), x_rot.double().abs() @ w.abs().t()


@pytest.mark.parametrize("p,n,batch,out,inp,g", CASES)
def test_prompt_product(p, n, batch, out, inp, g):
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] prompt p={p} n={n} batch={batch} {out}x{inp} g={g}", file=sys.stderr,
          flush=True)
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    codes, scales, idx = make_layer(p, n, out, inp, g, 7)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    x = torch.randn((batch, inp), generator=gen, device="cuda")
    x_rot = H.rht_activations(x, g, 3)
    y = H.qmatmul(x_rot, codes, scales, grid, g, out)
    fused = H.qmatmul_fused(x, codes, scales, grid, g, 3, out)
    ref, _ = reference(x_rot, idx, scales, grid, g)
    assert torch.equal(y, fused)
    check_qmm(y.cpu().numpy(), ref.cpu().numpy())


@pytest.mark.parametrize("p,n,batch,out,inp,g", [
    (2, 256, 1000, 8200, 512, 128), (2, 1024, 129, 17000, 2048, 256), (1, 256, 129, 17000, 512, 64),
    (2, 64, 65, 100, 1024, 128), (1, 16, 65, 100, 1088, 64)])
def test_prompt_product_unit_changes(p, n, batch, out, inp, g):
    """Scale groups whose magnitudes, and scales, differ by up to 2^90, zero
    scales and zero activation groups: every group's sums are added to totals
    of another magnitude."""
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] prompt units p={p} n={n} batch={batch} {out}x{inp} g={g}",
          file=sys.stderr, flush=True)
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    codes, scales, idx = make_layer(p, n, out, inp, g, 9)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(6)
    groups = inp // g
    x = torch.randn((batch, groups, g), generator=gen, device="cuda")
    x *= torch.exp2(torch.randint(-45, 46, (batch, groups, 1), generator=gen,
                                  device="cuda").float())
    x[:, 0] *= torch.rand((batch, 1), generator=gen, device="cuda") > 0.3
    x[::5, 1] = 0
    x = x.reshape(batch, inp).contiguous()
    scales[torch.rand(scales.shape, generator=gen, device="cuda") < 0.02] = 0
    scales[3] = 0
    scales[:, groups // 2] *= 2.0 ** -9
    y = H.qmatmul(x, codes, scales, grid, g, out)
    ref, terms = reference(x, idx, scales, grid, g)
    # each term's two factors are rounded to fp16 once: (1 + 2^-11)^2 - 1 of
    # its magnitude, and a little for the fp32 sums
    assert bool(torch.isfinite(y).all())
    assert bool(((y.double() - ref).abs() <= 1.02 * 2.0 ** -10 * terms).all())
    assert bool((y[:, 3] == 0).all())


@pytest.mark.parametrize("p,n,batch,out,inp,g", CASES)
def test_prompt_product_whole_numbers(p, n, batch, out, inp, g):
    """Whole grid points, activations (times powers of two that differ by row
    and group) and scales whose sums of magnitudes stay below 2^24: every
    operand is exact in fp16 and every sum in fp32, in any order, so a product
    whose sums are kept per group and added to totals once per group is exact.
    A sum carried over groups in units of the last one's scale is not."""
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] prompt whole p={p} n={n} batch={batch} {out}x{inp} g={g}", file=sys.stderr,
          flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(8)

    def ints(lo, hi, shape):
        return torch.randint(lo, hi + 1, shape, generator=gen, device="cuda").float()

    grid = ints(-3, 3, (n, p))
    codes, _, idx = make_layer(p, n, out, inp, g, 11)
    scales = (2 * ints(0, 3, (out, inp // g)) + 1).half()  # 1, 3, 5, 7
    x = ints(-3, 3, (batch, inp // g, g)) * torch.exp2(ints(0, 3, (batch, inp // g, 1)))
    x = x.reshape(batch, inp)
    y = H.qmatmul(x, codes, scales, grid, g, out)
    ref, terms = reference(x, idx, scales, grid, g)
    assert float(terms.max()) < 2 ** 24
    assert torch.equal(y.double(), ref)


@pytest.mark.parametrize("p,n", FORMATS)
@pytest.mark.parametrize("batch", [40, 130])
def test_values_far_below_the_largest_keep_their_bits(p, n, batch):
    """One value of every group is 2^24 times the others, which have 11
    significant bits; its grid point is the origin, so the product is that of the
    others. In units that put the largest value just below 2^15 they are normal
    fp16 numbers: every operand is exact and only the fp32 sums round."""
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] small values p={p} n={n} batch={batch}", file=sys.stderr, flush=True)
    out, inp, g = 300, 2048, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(10)

    def ints(lo, hi, shape):
        return torch.randint(lo, hi + 1, shape, generator=gen, device="cuda").float()

    grid = ints(1, 40, (n, p)) * (2 * ints(0, 1, (n, p)) - 1)
    grid[0] = 0
    from oracle import higgs_oracle as O
    idx = np.maximum(synth.random_codes(out, inp // p, n, 13), 1)
    idx.reshape(out, inp // g, g // p)[:, :, 5] = 0
    codes = torch.from_numpy(O.pack_codes(idx, n)).cuda()
    idx = torch.from_numpy(idx.astype(np.int64)).cuda()
    scales = torch.exp2(ints(-9, -5, (out, inp // g))).half()
    # largest value in [2^k, 2^(k+1)) for k over a run of exponents
    x = ints(1024, 2047, (batch, inp // g, g)) * 2.0 ** -34  # [2^-24, 2^-23)
    x *= 2 * ints(0, 1, x.shape) - 1
    x[:, :, 5 * p] = 1.5
    x *= torch.exp2(ints(0, 20, (batch, inp // g, 1)))
    x = x.reshape(batch, inp)
    y = H.qmatmul(x, codes, scales, grid, g, out)
    ref, terms = reference(x, idx, scales, grid, g)
    # products exact (11 + 6 bits); each term passes at most in + in / g fp32
    # additions, each within 2^-24 of a partial sum of magnitudes
    assert bool(((y.double() - ref).abs() <= (inp + inp // g) * 2.0 ** -24 * terms).all())
    # which 2^-8, what a value that lost four bits would show, is far above
    assert (inp + inp // g) * 2.0 ** -24 < 2.0 ** -12


def test_prompt_group_and_noalloc_match_single_calls():
    from paper_2411_17525_amd import higgs as H
    p, n, g, batch, inp = 2, 256, 256, 300, 1024
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    x = torch.randn((batch, inp), device="cuda").to(torch.bfloat16)
    layers = []
    for k, out in enumerate((8200, 129, 1000)):
        codes, scales, _ = make_layer(p, n, out, inp, g, 20 + k)
        layers.append((codes, scales, 40 + k, out))
    ys = H.qmatmul_fused_multi(x, layers, grid, g)
    for (codes, scales, seed, out), y in zip(layers, ys):
        assert torch.equal(y, H.qmatmul_fused(x, codes, scales, grid, g, seed, out))
        assert torch.equal(y, H.qmatmul_fused_noalloc(x, codes, scales, grid, g, seed, out))


# layers of one call: K-splits of several lengths in one launch, with numbers of
# work items that are no multiple of eight; equal layers; one split layer among
# unsplit ones; one group per row
GROUPS = [
    (2, 1024, 128, 257, 8192, (8192, 260, 130)),
    (2, 256, 1024, 65, 4096, (4096, 1024, 1000)),
    (1, 16, 64, 33, 1024, (512, 512, 512, 512)),
    (1, 256, 128, 130, 2048, (17000, 129, 900)),
    (2, 64, 4096, 65, 4096, (300, 100, 200)),
    (2, 256, 2048, 66, 6144, (300, 100)),
]


@pytest.mark.parametrize("p,n,g,batch,inp,outs", GROUPS)
def test_prompt_groups_match_single_calls(p, n, g, batch, inp, outs):
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] prompt group p={p} n={n} batch={batch} {outs}x{inp} g={g}",
          file=sys.stderr, flush=True)
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    x = torch.randn((batch, inp), device="cuda").to(torch.bfloat16)
    layers = []
    for k, out in enumerate(outs):
        codes, scales, _ = make_layer(p, n, out, inp, g, 20 + k)
        layers.append((codes, scales, 40 + k, out))
    for call in (layers, [(c, sc, 9, out) for c, sc, _, out in layers]):  # own and shared seeds
        ys = H.qmatmul_fused_multi(x, call, grid, g)
        for (codes, scales, seed, out), y in zip(call, ys):
            assert torch.equal(y, H.qmatmul_fused(x, codes, scales, grid, g, seed, out))
            x_rot = H.rht_activations(x, g, seed)
            assert torch.equal(y, H.qmatmul(x_rot, codes, scales, grid, g, out))


@pytest.mark.parametrize("p,n,g,out,inp,small,large", [
    (2, 256, 1024, 4096, 4096, 160, 257), (2, 1024, 1024, 14336, 4096, 80, 129),
    (1, 16, 64, 14336, 4096, 32, 129), (1, 256, 64, 1024, 1024, 160, 768)])
def test_workspace_of_a_larger_batch(p, n, g, out, inp, small, large):
    """A workspace kept for a larger batch, smaller than the small batch's plan
    takes: the call computes the same product; a byte less than the least is
    refused."""
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] kept workspace p={p} n={n} {out}x{inp} g={g} {small} of {large}",
          file=sys.stderr, flush=True)
    kept = H.qmatmul_fused_workspace_bytes(large, out, inp, p, n, g)
    assert kept < H.qmatmul_fused_workspace_bytes(small, out, inp, p, n, g)
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    codes, scales, idx = make_layer(p, n, out, inp, g, 31)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    x = torch.randn((small, inp), generator=gen, device="cuda")
    x_rot = H.rht_activations(x, g, 3)
    ws = torch.empty(kept, dtype=torch.uint8, device="cuda")
    ref, _ = reference(x_rot, idx, scales, grid, g)
    y = H.qmatmul(x_rot, codes, scales, grid, g, out, workspace=ws)
    check_qmm(y.cpu().numpy(), ref.cpu().numpy())
    assert torch.equal(y, H.qmatmul_fused(x, codes, scales, grid, g, 3, out, workspace=ws))
    multi = H.qmatmul_fused_multi_workspace_bytes(large, (out, out), inp, p, n, g)
    ws = torch.empty(multi, dtype=torch.uint8, device="cuda")
    ys = H.qmatmul_fused_multi(x, [(codes, scales, 3, out)] * 2, grid, g, workspace=ws)
    for y in ys:
        check_qmm(y.cpu().numpy(), ref.cpu().numpy())
    with pytest.raises(H.HiggsError):
        H.qmatmul(x_rot, codes, scales, grid, g, out, workspace=ws[:small * inp * 2])
