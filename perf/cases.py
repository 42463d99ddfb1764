"""Workloads whose speed is tracked: the calls that a program serving or
quantizing HIGGS layers makes, over the sizes, formats and types it makes them
with.

A case names a path ("kind") and its sizes:
  linear       one layer from raw activations (QuantizedLinear.forward)
  two_step     the same layer through the separate rotation and product calls
  group        layers that read the same activations (q/k/v, gate/up), one call
  block        the seven linear layers of a transformer block, four calls
  block_graph  the same four calls captured once in a HIP graph and replayed
  encode       quantization of a weight matrix (search index at hand)
  error        the quantization error of an encoded layer
  gptq         quantization with GPTQ rounding (factor at hand)
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2411_17525_amd import higgs as H
from paper_2411_17525_amd import synth

DEV = "cuda"
POOL = 1 << 16  # rotated weight vectors that a layer's codes are drawn from
ROTATION_SEED = 11

# The linear layers of a Llama-3.1-8B block in calls: layers of one call read
# the same activations.
BLOCK = (((4096, 1024, 1024), 4096), ((4096,), 4096), ((14336, 14336), 4096), ((4096,), 14336))


def listed():
    return [
        # one projection of a chat turn's decode step, called eagerly: the
        # smallest call there is
        dict(name="token_linear", kind="linear", batch=1, outs="4096", inp=4096, p=2, n=256,
             g=1024, x="bf16"),
        # a whole block's layers for one token, as a serving loop replays them
        dict(name="token_block", kind="block_graph", batch=1, p=2, n=256, g=1024, x="bf16"),
        # four sequences (or four speculated tokens) through an 8-bit layer
        # with long rows
        dict(name="decode4_ch8_down", kind="linear", batch=4, outs="4096", inp=14336, p=1, n=256,
             g=512, x="f32"),
        # a decode step of 16 sequences
        dict(name="decode16_block", kind="block", batch=16, p=2, n=256, g=1024, x="bf16"),
        # a decode step of 64 sequences
        dict(name="decode64_gate_up", kind="group", batch=64, outs="14336,14336", inp=4096, p=2,
             n=256, g=1024, x="bf16"),
        # prompt of a ragged length, fp32 activations, layer of a size that is
        # no multiple of anything, rotation and product called separately
        dict(name="prefill300_ragged", kind="two_step", batch=300, outs="11003", inp=5120, p=1,
             n=16, g=128, x="f32"),
        # a chunk of a chunked prefill, 5-bit codes
        dict(name="prefill512_down", kind="linear", batch=512, outs="4096", inp=14336, p=2,
             n=1024, g=1024, x="bf16"),
        # a whole prompt, the largest call
        dict(name="prefill2048_gate_up", kind="group", batch=2048, outs="14336,14336", inp=4096,
             p=2, n=256, g=1024, x="bf16"),
        # quantizing a checkpoint's MLP layer
        dict(name="encode_gate", kind="encode", outs="14336", inp=4096, p=2, n=256, g=1024,
             x="bf16"),
        # quantizing an fp32 layer at 5 bits with smaller groups
        dict(name="encode_f32_n1024", kind="encode", outs="4096", inp=4096, p=2, n=1024, g=256,
             x="f32"),
        # one entry of the error table that the bitwidth allocation reads
        dict(name="error_down_n64", kind="error", outs="4096", inp=14336, p=2, n=64, g=1024,
             x="bf16"),
        # GPTQ rounding of an attention projection
        dict(name="gptq_q", kind="gptq", outs="4096", inp=4096, p=2, n=256, g=1024, x="bf16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(("linear", "two_step", "group", "encode", "error", "gptq"),
                       (40, 12, 18, 14, 8, 8))[0]
    p, n = rng.choice(((1, 16), (2, 64), (2, 256), (2, 256), (2, 1024), (1, 256)))
    g = rng.choice([v for v in (64, 128, 256, 512, 1024, 1024, 1024, 2048) if v >= 64 * p])
    case = dict(kind=kind, p=p, n=n, g=g, x=rng.choice(("bf16", "bf16", "f32")))
    if kind == "gptq":
        case.update(inp=max(1, _log_int(rng, 512, 4096) // g) * g,
                    outs=str(_log_int(rng, 256, 4096)))
        return case
    if kind in ("encode", "error"):
        if g > 1024:
            case["g"] = g = 1024
        case.update(inp=max(1, _log_int(rng, 1024, 14336) // g) * g,
                    outs=str(_log_int(rng, 128, 4096)))
        return case
    inp = max(1, _log_int(rng, 1024, 14336) // g) * g
    outs = [_log_int(rng, 256, 14336) for _ in range(rng.randint(2, 4) if kind == "group" else 1)]
    batch = _log_int(rng, 1, 2048)
    case.update(batch=min(batch, max(1, 2048 * 14336 * 4096 // (sum(outs) * inp))), inp=inp,
                outs=",".join(map(str, outs)))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _grid_np(p, n):
    if (p, n) == (1, 256):
        return H.make_uniform_grid(n)[0]
    return H.make_grid(p, n, 0, 1 << 14, 50)[0]


def _grid(case):
    return torch.from_numpy(_grid_np(case["p"], case["n"])).to(DEV)


@functools.lru_cache(maxsize=None)
def _pool(p, n):
    """POOL rotated p-vectors, N(0, I), and their nearest grid points: what a
    layer's rotated weights and codes are distributed like."""
    v = torch.from_numpy(np.random.default_rng(77).standard_normal((POOL, p)).astype(np.float32))
    d = torch.cdist(v.double(), torch.from_numpy(_grid_np(p, n)).double())
    return v.to(DEV), d.argmin(dim=1).to(torch.int32).to(DEV)


def _gen(seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    return gen


def _pack(idx, n):
    """LSB-first bit stream of each row's indices."""
    bits = int(math.log2(n))
    if bits == 8:
        return idx.to(torch.uint8).contiguous()
    per, nbytes = {4: (2, 1), 6: (4, 3), 10: (4, 5)}[bits]
    v = idx.reshape(idx.shape[0], -1, per).to(torch.int64)
    word = sum(v[:, :, k] << (bits * k) for k in range(per))
    out = torch.stack([(word >> (8 * k)) & 255 for k in range(nbytes)], dim=-1)
    return out.to(torch.uint8).reshape(idx.shape[0], -1).contiguous()


def _layer_parts(case, out, inp, gen):
    """Indices [out, in/p] and fp16 scales [out, in/g] of one encoded layer."""
    _, near = _pool(case["p"], case["n"])
    pick = torch.randint(0, POOL, (out, inp // case["p"]), generator=gen, device=DEV)
    sc = 0.02 * (0.8 + 0.4 * torch.rand((out, inp // case["g"]), generator=gen, device=DEV))
    return near[pick], sc.to(torch.float16), pick


def _activations(case, inp, gen):
    """N(0, 1) with a few outlier channels, as an LLM's hidden states have."""
    x = torch.randn((case["batch"], inp), generator=gen, device=DEV)
    cols = torch.randperm(inp, generator=gen, device=DEV)[:max(1, inp // 1000)]
    x[:, cols] *= 20.0
    return x.to(torch.bfloat16) if case["x"] == "bf16" else x


def _calls(case):
    """(outs, in) of each call of the case's product."""
    if case["kind"] in ("block", "block_graph"):
        return BLOCK
    return ((tuple(int(o) for o in case["outs"].split(",")), case["inp"]),)


def _weight(case, seed):
    out, inp = int(case["outs"]), case["inp"]
    w, _ = synth.student_t_weight_device(out, inp, seed, DEV)
    # fp32 weights use more than bf16's bits
    return w if case["x"] == "bf16" else w.float() * 1.0009765625


def _signs(g, seed):
    with np.errstate(over="ignore"):
        j = np.arange(1, g + 1, dtype=np.uint64)
        z = np.uint64(seed) + j * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return torch.from_numpy(1.0 - 2.0 * (z >> np.uint64(63)).astype(np.float64)).to(DEV)


def _hadamard(v, g):
    """H v / sqrt(g) over blocks of g along the last axis, in 64 bits."""
    shape = v.shape
    v = v.double().reshape(-1, g)
    h = 1
    while h < g:
        v = v.reshape(-1, g // (2 * h), 2, h)
        v = torch.stack((v[:, :, 0] + v[:, :, 1], v[:, :, 0] - v[:, :, 1]), dim=2).reshape(-1, g)
        h *= 2
    return (v / math.sqrt(g)).reshape(shape)


def _rotate(v, g, seed):
    shape = v.shape
    s = _signs(g, seed)
    return _hadamard((v.double().reshape(-1, g) * s).reshape(shape), g)


def _error_parts(case, seed):
    """A weight matrix whose rotated p-vectors are pool vectors, rounded to its
    type, with the codes and scales that encode it."""
    out, inp, g = int(case["outs"]), case["inp"], case["g"]
    gen = _gen(seed)
    idx, _, pick = _layer_parts(case, out, inp, gen)
    rot = _pool(case["p"], case["n"])[0][pick].reshape(out, inp)
    w = torch.empty((out, inp), device=DEV, dtype=torch.float32)
    for r in range(0, out, 512):  # the inverse rotation: sigma * H / sqrt(g)
        w[r:r + 512] = (_hadamard(rot[r:r + 512], g).reshape(-1, g) *
                        _signs(g, ROTATION_SEED)).reshape(-1, inp).float() * 0.02
    if case["x"] == "bf16":
        w = w.to(torch.bfloat16)
    sc = (w.double().reshape(out, -1, g).norm(dim=2) / math.sqrt(g)).to(torch.float16)
    return w, idx, sc


def prepare(case, seed):
    kind = case["kind"]
    if kind == "encode":
        grid = _grid(case)
        return dict(case=case, w=_weight(case, seed), grid=grid, index=H.search_index(grid))
    if kind == "error":
        w, idx, sc = _error_parts(case, seed)
        return dict(case=case, w=w, codes=_pack(idx, case["n"]), scales=sc, grid=_grid(case))
    if kind == "gptq":
        inp = case["inp"]
        gen = _gen(seed + 1)
        # calibration activations with correlated channels
        x = torch.randn((2048, inp), generator=gen, device=DEV)
        x = x + 0.5 * x.roll(1, dims=1) + torch.randn((2048, 1), generator=gen, device=DEV)
        factor = H.gptq_factor(H.rht_activations(x, case["g"], ROTATION_SEED))
        return dict(case=case, w=_weight(case, seed), grid=_grid(case), factor=factor)
    gen = _gen(seed)
    grid, calls = _grid(case), []
    for outs, inp in _calls(case):
        layers = []
        for k, out in enumerate(outs):
            idx, sc, _ = _layer_parts(case, out, inp, gen)
            layers.append(H.QuantizedLinear(_pack(idx, case["n"]), sc, grid, case["g"],
                                            ROTATION_SEED + k, out, inp))
        calls.append((_activations(case, inp, gen), layers))
    state = dict(case=case, calls=calls)
    if kind == "block_graph":
        _products(state)  # loads the kernels before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            state["outputs"] = _products(state)
        state["graph"] = graph
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def _products(state):
    ys = []
    for x, layers in state["calls"]:
        if len(layers) == 1:
            ys.append(layers[0].forward(x))
        else:
            ys += H.qmatmul_fused_multi(
                x, [(q.codes, q.scales, q.seed, q.out_features) for q in layers],
                layers[0].grid, layers[0].g)
    return ys


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "block_graph":
        state["graph"].replay()
        return state["outputs"]
    if kind == "two_step":
        x, layers = state["calls"][0]
        return [layers[0].forward_two_step(x)]
    if kind == "encode":
        return list(H.quantize(state["w"], state["grid"], case["g"], ROTATION_SEED,
                               index=state["index"]))
    if kind == "error":
        return list(H.layer_error(state["w"], state["codes"], state["scales"], state["grid"],
                                  case["g"], ROTATION_SEED))
    if kind == "gptq":
        return list(H.quantize_gptq(state["w"], state["grid"], case["g"], ROTATION_SEED,
                                    state["factor"]))
    return _products(state)


def work(case):
    """Codes, scales, weights, activations and outputs once; two operations
    per multiply-add (the rotation and the search are not counted)."""
    code_bits = math.log2(case["n"]) / case["p"]
    g, xb = case["g"], 2 if case["x"] == "bf16" else 4
    if case["kind"] in ("encode", "error", "gptq"):
        out, inp = int(case["outs"]), case["inp"]
        nbytes = out * inp * (xb + code_bits / 8 + 2 / g)
        if case["kind"] == "error":
            return {"bytes": nbytes + 16 * out * inp / g, "flops": 2.0 * out * inp}
        if case["kind"] == "gptq":  # upper triangle of the factor; rounding feeds later columns
            return {"bytes": nbytes + 4.0 * inp * inp, "flops": 1.0 * out * inp * inp}
        return {"bytes": nbytes, "flops": 2.0 * out * inp}
    nbytes = flops = 0.0
    for outs, inp in _calls(case):
        nbytes += case["batch"] * inp * xb
        for out in outs:
            nbytes += out * inp * (code_bits / 8 + 2 / g) + 4 * case["batch"] * out
            flops += 2.0 * case["batch"] * out * inp
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "encode":
        return "exact"  # codes of a 64-bit search, scales with one rounding
    if case["kind"] == "gptq":
        # 64-bit sums: a code may differ where another order of the sums meets
        # a tie, and then the later codes of that row
        return {"rel": 0.0, "differ": 1e-4}
    if case["kind"] == "error":
        return {"rel": 1e-12}  # 64-bit sums
    # fp16 grid points and activations, 32-bit sums: about 3e-4 against 64 bits
    return {"rel": 1.2e-3, "max": 1e-2}


def exact(case, seed):
    kind, g, p = case["kind"], case["g"], case["p"]
    if kind in ("encode", "gptq"):
        w = _weight(case, seed).double()
        return [None, w.reshape(w.shape[0], -1, g).norm(dim=2) / math.sqrt(g)]
    grid = _grid(case).double()
    if kind == "error":
        w, idx, sc = _error_parts(case, seed)
        err, norm = [], []
        for r in range(0, w.shape[0], 512):
            rot = _rotate(w[r:r + 512], g, ROTATION_SEED)
            hat = grid[idx[r:r + 512].long()].reshape(rot.shape[0], -1, g)
            hat = hat * sc[r:r + 512].double()[:, :, None]
            err.append(((rot.reshape(hat.shape) - hat) ** 2).sum(dim=2))
            norm.append((w[r:r + 512].double().reshape(hat.shape) ** 2).sum(dim=2))
        err, norm = torch.cat(err).reshape(-1), torch.cat(norm).reshape(-1)
        return [float(err.sum() / norm.sum()), torch.stack((err, norm), dim=1)]
    gen, ys = _gen(seed), []
    for outs, inp in _calls(case):
        parts = [_layer_parts(case, out, inp, gen)[:2] for out in outs]
        x = _activations(case, inp, gen)
        for k, (idx, sc) in enumerate(parts):
            xr = _rotate(x, g, ROTATION_SEED + k)
            y = torch.empty((x.shape[0], idx.shape[0]), device=DEV, dtype=torch.float64)
            for r in range(0, idx.shape[0], 2048):
                hat = grid[idx[r:r + 2048].long()].reshape(-1, inp // g, g)
                hat = (hat * sc[r:r + 2048].double()[:, :, None]).reshape(-1, inp)
                y[:, r:r + 2048] = xr @ hat.t()
            ys.append(y)
    return ys
