"""The bound of the GPU test of the fp32 gate GEMM's six products of bf16
parts, checked against an emulation: the six together stay below it, and
leaving any one out exceeds it."""

import numpy as np
import pytest
import torch

from oracle import dynamics as OD
from tests.gpu_util import THREE_PART_RMS, rms, three_part_rows

PRODUCTS = [(2, 0), (0, 2), (1, 0), (1, 1), (0, 1), (0, 0)]   # (audio part, visual part), in order


def _parts(x):
    out = []
    for _ in range(3):
        h = torch.from_numpy(x).bfloat16().float().numpy()
        out.append(h)
        x = x - h
    return out


def _scores(xv, xa, left_out):
    """1 - d_hat from fp32 sums over 32 elements and a product at a time, the
    small products by themselves."""
    dim = xv.shape[1]
    pad = ((0, 0), (0, -dim % 32))
    V, A = ([np.pad(p, pad).astype(np.float64) for p in _parts(x)] for x in (xv, xa))
    acc = [np.zeros((xv.shape[0], xa.shape[0]), np.float32) for _ in range(2)]
    for k in range(0, V[0].shape[1], 32):
        for i, (a, v) in enumerate(PRODUCTS):
            if i != left_out:
                into = int(a + v == 0)
                acc[into] = (acc[into] + V[v][:, k:k + 32] @ A[a][:, k:k + 32].T).astype(np.float32)
    inv = (1.0 / np.linalg.norm(xa.astype(np.float64), axis=1)).astype(np.float32)
    cos = ((acc[1] + acc[0]) * inv).max(axis=1) / np.linalg.norm(xv.astype(np.float64), axis=1)
    return 1.0 - OD.minmax(1.0 - cos)


@pytest.mark.parametrize("dim", [8, 40, 264, 1288, 3584])
def test_bound_separates_six_products_from_five(dim):
    for seed in range(3):
        xv, xa = three_part_rows(np.random.default_rng(seed), 200, 40, dim)
        d, _ = OD.direct_distance(xv.astype(np.float64), xa.astype(np.float64), xv.shape[0], 1)
        want = 1.0 - OD.minmax(d)
        assert rms(_scores(xv, xa, None), want) < THREE_PART_RMS / 2
        for i in range(len(PRODUCTS)):
            assert rms(_scores(xv, xa, i), want) > 2 * THREE_PART_RMS, PRODUCTS[i]
