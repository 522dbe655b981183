"""Helpers shared by the GPU parity tests: move generator bits to the device
and back as raw bit patterns (no arithmetic on either side)."""

import sys

import numpy as np


def log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def to_dev(x, dtype):
    """Raw generator array -> CUDA tensor of the same bits."""
    import torch
    if dtype == "bf16":
        t = torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16)
    else:
        t = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32))
    return t.cuda()


def bits(t):
    """CUDA tensor -> numpy array of its raw bits."""
    import torch
    t = t.detach().contiguous().cpu()
    if t.dtype == torch.bfloat16:
        return t.view(torch.int16).numpy().view(np.uint16)
    if t.dtype == torch.float32:
        return t.view(torch.int32).numpy().view(np.uint32)
    return t.numpy()


def raw_bits(x, dtype):
    x = np.ascontiguousarray(x)
    return x.view(np.uint16) if dtype == "bf16" else x.astype(np.float32).view(np.uint32)


def score_tol(dtype):
    return 2e-3 if dtype == "bf16" else 1e-5


def three_part_rows(rng, visual, audio, dim):
    """fp32 rows whose three bf16 parts all count: five elements a row, spread
    over the K steps, each 1 with a second part of about 2^-9 and a third of
    about 2^-18 of random signs.  So few terms keep the rounding of the sums
    (rms under 8e-8 of a cosine) below what any of the six products of the
    parts that are summed contributes (rms over 7e-7).  Three audio rows, the
    first, the middle and the last, have them; the others have one element
    elsewhere and a cosine of 0 to every visual row."""
    pos = np.linspace(0, dim - 1, 5).astype(int)

    def rows(n):
        sign = lambda: rng.choice([-1.0, 1.0], (n, 5))
        x = np.zeros((n, dim))
        x[:, pos] = sign() * (1 + sign() * rng.uniform(0.6, 0.98, (n, 5)) * 2.0 ** -9
                              + sign() * rng.uniform(1.2, 1.9, (n, 5)) * 2.0 ** -18)
        return x.astype(np.float32)

    xa = np.zeros((audio, dim), np.float32)
    xa[:, np.setdiff1d(np.arange(dim), pos)[0]] = 1.0
    xa[[0, audio // 2, audio - 1]] = rows(3)
    return rows(visual), xa


THREE_PART_RMS = 2.5e-7   # bound on the rms error of 1 - d_hat over such rows


def rms(got, want):
    return float(np.sqrt(np.mean((np.asarray(got, np.float64) - want) ** 2)))
