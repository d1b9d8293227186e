"""Kernel variants and dispatch branches at the sizes where they can go
wrong, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2606_08469_amd import binding

from _gpu import report, to_np

pytestmark = pytest.mark.gpu


def random_mlp(widths, dtype, seed, off=0):
    """FP32 weights, and a device MLP whose weights start `off` elements into
    their buffers (off = 1: aligned for single elements only)."""
    g = np.random.default_rng(seed)
    W = [(g.uniform(-1, 1, (o, i)) * np.sqrt(6.0 / (i + o))).astype(np.float32) for i, o in zip(widths, widths[1:])]
    b = [(0.1 * g.normal(size=o)).astype(np.float32) for o in widths[1:]]
    dev = []
    for w in W:
        buf = torch.zeros(w.size + off, dtype=dtype, device="cuda")
        buf[off:] = torch.from_numpy(w.reshape(-1)).to(dtype)
        dev.append(buf[off:].view(w.shape))
    ref = [to_np(w).astype(np.float32) for w in dev]  # the rounded weights
    return binding.MLP(dev, [torch.from_numpy(v).cuda() for v in b]), oracle.MLP(ref, b)


@pytest.mark.parametrize("widths", [(20, 64, 3), (64, 64, 64, 64, 3), (76, 128, 128, 3), (128, 128, 128, 128, 128, 3)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("B,off", [(1, 0), (15, 1), (33, 0), (64, 0), (65, 1), (130, 0), (8 * 256 * 64 + 17, 0)])
def test_decoder_shapes(widths, dtype, B, off):
    """One to four input chunks, ragged row counts, weights aligned for whole
    fragments or not, weights in LDS or (FP32, four 128-wide layers) not.
    FP32: products and sums of at most 128 terms per layer, 1e-5. 16 bit:
    each layer rounds its activations to 2^-11 (2^-8 for BF16) relative, at
    most four roundings deep: 4 * 2^-8 < 0.02 of a row's scale."""
    if B > 1000 and (dtype == torch.bfloat16 or widths[0] == 20):
        pytest.skip("the persistent loop is covered by the other shapes")
    print(f"[case] decoder {widths} {dtype} B={B} off={off}", flush=True)
    mlp, omlp = random_mlp(widths, dtype, 7, off)
    h = (0.5 * torch.randn(B, widths[0], generator=torch.Generator().manual_seed(B))).to(dtype).cuda()
    rgb = to_np(binding.mlp_fwd(mlp, h))
    rows = np.arange(B) if B < 1000 else np.concatenate([np.arange(64), np.arange(B - 200, B)])
    want = oracle.mlp_fwd(omlp, to_np(h)[rows].astype(np.float64))
    rms = float(np.sqrt(np.mean(want ** 2)))
    worst = float(np.max(np.abs(rgb[rows] - want) / (np.abs(want) + rms)))
    report(f"decoder {widths} {dtype} B={B}", worst=worst)
    assert worst <= (1e-5 if dtype == torch.float32 else 0.02)
