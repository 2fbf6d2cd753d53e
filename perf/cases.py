"""What a user of this library has it do, as cases that can be timed.

A case is one pruned convolution layer (or, with "net", the layers of a bundled workload one after the other, each
output the next layer's input), run the way the library is used: the CSR is packed, planned and uploaded once, and every
pass is one forward call per layer on a batch that is already on the GPU.

  path "tiled"   the fused form: escoin_sconv_forward_tiled on the unpadded input
  path "direct"  the two-kernel form: escoin_pad_in, then escoin_sconv_forward on the padded array
  flags          0, or the fused epilogue: 1 = bias, 2 = ReLU, 3 = both

Shapes are the bundled workloads' and the test suite's (pruned AlexNet-, GoogLeNet- and ResNet-style layers, a first
layer of a network); sparsities run from 50 % to 95 %, as pruning leaves them.
"""
import math

import numpy as np
import torch

from paper_1802_10280_amd import workloads as wl
from paper_1802_10280_amd.runner import LayerRunner


def _layer(name, N, C, HW, M, RS, stride, pad, sparsity, flags=0, path="tiled", skew=False):
    return dict(name=name, N=N, C=C, H=HW, W=HW, M=M, R=RS, S=RS, stride=stride, pad=pad, sparsity=sparsity,
                flags=flags, path=path, skew=skew)


def listed():
    return [
        # the smallest call: one small image, where launch and call overheads are most of it
        _layer("tiny", 1, 16, 14, 32, 3, 1, 1, 0.80),
        # latency of a single image through a middle layer of an AlexNet-style network, epilogue fused
        _layer("alexnet_b1", 1, 384, 13, 384, 3, 1, 1, 0.65, flags=3),
        # the same layer in a serving batch: odd maps (13x13), moderate sparsity
        _layer("alexnet_b64", 64, 384, 13, 384, 3, 1, 1, 0.65, flags=3),
        # inception-style 1x1 reduction (a sparse matrix product): little arithmetic per byte
        _layer("googlenet_1x1", 32, 192, 28, 64, 1, 1, 0, 0.70),
        # inception-style 5x5 with few channels
        _layer("googlenet_5x5", 32, 16, 28, 32, 5, 1, 2, 0.70),
        # residual-network 3x3 layers: large maps with few channels, tiny maps with many
        _layer("resnet_56", 32, 64, 56, 64, 3, 1, 1, 0.80),
        _layer("resnet_7", 32, 512, 7, 512, 3, 1, 1, 0.80),
        # first layer of a network: three input channels, 7x7 stride 2, a ragged batch
        _layer("first_7x7s2", 5, 3, 224, 64, 7, 2, 3, 0.50, flags=3),
        # a large layer at the two ends of what pruning reaches
        _layer("large_s50", 64, 256, 28, 256, 3, 1, 1, 0.50),
        _layer("large_s95", 64, 256, 28, 256, 3, 1, 1, 0.95),
        # three layers back to back on the device (the middle one of stride 2), bias + ReLU fused
        dict(name="chain", net="chain", flags=3, path="tiled"),
        # the general kernel and its padding pass: any CSR order, no plan
        _layer("two_kernel_28", 32, 128, 28, 128, 3, 1, 1, 0.80, path="direct"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One layer of the same ranges: any batch, channel counts and map sizes (odd ones among them), the filters, strides
    and sparsities above, sometimes rows of very unequal length, sometimes the two-kernel form."""
    while True:
        R = rng.choice([1, 3, 3, 3, 3, 5])
        stride = 2 if R > 1 and rng.random() < 0.2 else 1
        HW = _log_int(rng, 7, 64)
        case = _layer("drawn", _log_int(rng, 1, 64), _log_int(rng, 16, 512), HW, _log_int(rng, 32, 512), R, stride, R // 2,
                      round(rng.uniform(0.5, 0.95), 3), flags=rng.choice([0, 1, 2, 3]),
                      path="direct" if rng.random() < 0.15 else "tiled", skew=rng.random() < 0.15)
        if rng.random() < 0.3:
            case["W"] = _log_int(rng, 7, 64)
        s = _specs(case)[0]
        dense = 2.0 * s.N * s.M * s.E * s.F * s.C * s.R * s.S
        words = s.N * (s.C * s.H * s.W + s.M * s.E * s.F)
        # no more than the largest listed layer (the two-kernel form, several times slower: a tenth of it)
        if dense <= (6e9 if case["path"] == "direct" else 5.9e10) and words <= 64 * 2 * 256 * 784:
            del case["name"]
            return case


def _specs(case):
    if "net" in case:
        return [wl.LAYERS[n] for n in wl.CONFIG_LAYERS[case["net"]]]
    return [wl.LayerSpec("case", 9, 0, case["N"], case["C"], case["H"], case["W"], case["M"], case["R"], case["S"],
                         case["stride"], case["pad"], case["sparsity"], skew=case["skew"], permute_rows=case["skew"])]


def _weights(spec, rng):
    """A pruned filter bank as CSR: every weight kept with probability 1 - sparsity (or, skewed, rows of power-law
    length in random order), the kept ones N(0, 0.05)."""
    cols = spec.C * spec.R * spec.S
    noise = rng.random((spec.M, cols), dtype=np.float32)
    if spec.skew:
        keep = wl.skewed_row_nnz(spec.M, cols, int(round(spec.M * cols * (1.0 - spec.sparsity))))[rng.permutation(spec.M)]
        limit = np.take_along_axis(np.sort(noise, axis=1), keep[:, None] - 1, axis=1)
        mask = noise <= limit
    else:
        mask = noise >= np.float32(spec.sparsity)
    w = np.zeros((spec.M, cols), dtype=np.float32)
    w[mask] = rng.standard_normal(int(mask.sum()), dtype=np.float32) * np.float32(0.05)
    return w.reshape(spec.M, spec.C, spec.R, spec.S)


def _input(spec, gen):
    """An activation map as it leaves a ReLU (half of it zeros), or image data for a first layer."""
    shape = (spec.N, spec.C, spec.H, spec.W)
    if spec.C <= 3:
        return torch.randn(shape, device="cuda", generator=gen)
    x = torch.rand(shape, device="cuda", generator=gen)
    return x.mul_(torch.rand(shape, device="cuda", generator=gen) >= 0.5)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = np.random.Generator(np.random.PCG64(seed))
    runners = []
    for spec in _specs(case):
        w = _weights(spec, rng)
        rowptr, colidx, value = wl.dense_to_csr(w)
        bias = rng.standard_normal(spec.M, dtype=np.float32) * np.float32(0.1)
        layer = wl.Layer(spec, w, rowptr, colidx, value, None, bias)
        d_in = runners[-1].d_out if runners else _input(spec, gen)
        runners.append(LayerRunner(layer, path=case["path"], flags=case["flags"], d_in=d_in))
    return runners


def run(state):
    return [r.run() for r in state]


def work(case):
    """Every input and output word once, the CSR (values, column indices, row pointers) once; a multiply and an add per
    nonzero and output position."""
    total_bytes, flops = 0.0, 0.0
    for s in _specs(case):
        nnz = s.M * s.C * s.R * s.S * (1.0 - s.sparsity)
        total_bytes += 4.0 * s.N * (s.C * s.H * s.W + s.M * s.E * s.F) + 4.0 * (2 * nnz + s.M + 1)
        flops += 2.0 * nnz * s.N * s.E * s.F
    return {"bytes": total_bytes, "flops": flops}


def tolerance(case):
    """Sums of up to some thousand fp32 products, whose order is free."""
    return {"rel": 1e-5}
