"""GPU parity of the encoder where a wavefront takes several groups at once and
the last one it takes is not full, over several turns, for every code width and
group size, with vectors outside the search index's buckets."""
import sys

import numpy as np
import pytest

from oracle import higgs_oracle as O
from paper_2411_17525_amd import synth
from test_gpu_parity import check_codes, grid_f32

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,g,out,inp,dtype", [
    (2, 64, 128, 3, 640, "bf16"),      # 15 groups, 8 at once
    (2, 256, 128, 3, 384, "f32"),      # 9
    (2, 256, 512, 5, 1536, "bf16"),    # 15 groups, 2 at once
    (2, 1024, 256, 7, 768, "f32"),     # 21 groups, 4 at once
    (2, 1024, 512, 3, 512, "bf16"),
    (1, 16, 64, 7, 704, "bf16"),       # 77 groups, 16 at once
    (1, 16, 512, 3, 1536, "f32"),
    (1, 256, 64, 5, 192, "f32"),       # 15 groups, one wavefront not full
    (1, 256, 256, 9, 768, "bf16"),
    (1, 16, 128, 1, 128, "f32"),       # one group
    (2, 256, 256, 3301, 1024, "bf16"),  # 13204 groups: more than one turn
    (2, 64, 1024, 9001, 1024, "bf16"),
])
def test_encode_ragged_groups(p, n, g, out, inp, dtype):
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] encode groups p={p} n={n} g={g} {out}x{inp} {dtype}", file=sys.stderr,
          flush=True)
    grid = grid_f32(p, n)
    wt = synth.student_t_weight(out, inp, seed=3 * out + g, dtype=dtype)
    vals = wt.values.copy()
    # rows whose rotated groups reach beyond four standard deviations: a few
    # rotated values carry most of the group's energy
    signs = O.rht_signs(31, g).astype(np.float64)
    rng = np.random.default_rng(5)
    for r in range(0, out, max(1, out // 7)):
        rot = rng.standard_normal(g) * 0.05
        rot[rng.choice(g, size=3, replace=False)] = np.sqrt(g / 3.0) * rng.choice((-1, 1), 3)
        h = rot.copy()
        step = 1
        while step < g:  # the inverse rotation: sigma * H / sqrt(g)
            h = h.reshape(-1, 2, step)
            h = np.stack((h[:, 0] + h[:, 1], h[:, 0] - h[:, 1]), axis=1).reshape(-1)
            step *= 2
        vals[r, :g] = (h * signs / np.sqrt(g) * 0.02).astype(np.float32)
    if dtype == "bf16":
        bits = synth.f32_to_bf16_bits(vals)
        vals = synth.bf16_bits_to_f32(bits)
        w = torch.from_numpy(bits.view(np.int16)).cuda().view(torch.bfloat16)
    else:
        w = torch.from_numpy(vals).cuda()
    gd = torch.from_numpy(grid).cuda()
    # one spare row behind the outputs: nothing past the last group is written
    codes = torch.full((out + 1, H.codes_row_bytes(inp, p, n)), 0xA5, dtype=torch.uint8,
                       device="cuda")
    scales = torch.full((out + 1, inp // g), 7.0, dtype=torch.float16, device="cuda")
    H.quantize(w, gd, g, 31, codes=codes, scales=scales)
    full, full_scales = H.quantize(w, gd, g, 31, index=False)
    assert torch.equal(codes[:out], full) and torch.equal(scales[:out], full_scales)
    assert bool((codes[out] == 0xA5).all()) and bool((scales[out] == 7.0).all())
    rows = np.unique(np.r_[0:3, out // 7, out // 2, out - 2, out - 1])
    rows = rows[(rows >= 0) & (rows < out)]
    ref = O.quantize(vals[rows].astype(np.float64), grid.astype(np.float64), g, 31)
    check_codes(codes, scales, ref, n, rows=rows, grid=grid)


@pytest.mark.parametrize("p,n", [(1, 16), (1, 256), (2, 64), (2, 256), (2, 1024)])
@pytest.mark.parametrize("g", [128, 1024])
def test_encode_at_the_last_bucket_edge(p, n, g):
    """Rotated values of exactly the largest double below 4 (and its negative),
    the edge of the square that the search index covers, on either or both axes:
    the codes are those of the full scan."""
    from paper_2411_17525_amd import higgs as H
    print(f"[gpu-case] encode edge p={p} n={n} g={g}", file=sys.stderr, flush=True)
    # 16 equal weights: norm 4 * 49, each normalised to 49 * fl(1 / 196), which
    # is the largest double below 1/4, and 16 of them add up without rounding
    below = np.nextafter(4.0, 0.0)
    assert 16 * (49.0 * (1.0 / 196.0)) == below
    signs = O.rht_signs(31, g).astype(np.float64)
    j = np.arange(g)
    rows, want = [], []
    for at in (j[:16], j[1:33:2], j[:32:2], j[g - 16:]):  # both parities, even only
        for alternate in (0, 1):
            for s in (1.0, -1.0):
                x = np.zeros(g)
                x[at] = s * 49.0 * (1 - 2 * (alternate * (at & 1)))
                rows.append(x * signs)
                h, step = x * (1.0 / 196.0), 1
                while step < g:
                    h = h.reshape(-1, 2, step)
                    h = np.stack((h[:, 0] + h[:, 1], h[:, 0] - h[:, 1]), axis=1).reshape(-1)
                    step *= 2
                want.append(np.abs(h).reshape(-1, p))
    want = np.concatenate(want)
    assert bool((want == below).any(axis=0).all())
    if p == 2:
        assert bool((want == below).all(axis=1).any()) and bool((want == (below, 0)).all(1).any())
    w = torch.from_numpy(np.stack(rows).astype(np.float32)).cuda()
    gd = torch.from_numpy(grid_f32(p, n)).cuda()
    codes, scales = H.quantize(w, gd, g, 31)
    full, full_scales = H.quantize(w, gd, g, 31, index=False)
    assert torch.equal(codes, full) and torch.equal(scales, full_scales)


# 1024-weight turns below, at and above the line where a block's waves share
# their weights (512, 1024 and 1536 turns of blocks of 4, 8 and 12 waves), a last
# turn that is not full, and more turns than blocks
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("p,n,line", [(1, 16, 1024), (1, 256, 1024), (2, 64, 512), (2, 256, 1536),
                                      (2, 1024, 1536)])
def test_few_rows_without_an_index(p, n, line, dtype):
    from paper_2411_17525_amd import higgs as H
    grid = torch.from_numpy(grid_f32(p, n)).cuda()
    index = H.search_index(grid)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    for g in (64 * p, 256, 1024):
        for out, inp in ((1, 1024), (3, 3072), (5, 1024 + g % 1024), (line, 1024),
                         (line + 1, 1024), (300, 1024)):
            print(f"[gpu-case] no index p={p} n={n} g={g} {out}x{inp} {dtype}", file=sys.stderr,
                  flush=True)
            w = torch.randn((out, inp), generator=gen, device="cuda")
            w[0, :g] = 0  # a group of zeros
            w = w if dtype == "f32" else w.to(torch.bfloat16)
            codes, scales = H.quantize(w, grid, g, 5, index=False)[:2]
            want, ws = H.quantize(w, grid, g, 5, index=index)[:2]
            assert torch.equal(codes, want)
            assert torch.equal(scales.view(torch.int16), ws.view(torch.int16))
