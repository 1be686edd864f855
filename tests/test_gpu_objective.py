"""qe_objective (Sec. 2.1 problem (1)) against fp64 sums of the same numbers, at
the edges of its tiles (128 and 256) and of its runs over K.  Bound: every
product is good to 2^-23 of itself and is added into an fp32 sum of at most n = p and at
most 32 * 256 products (the longest run of tiles).  Its roundings, each below 2^-24 of
the sum so far and random in sign, come to about sqrt(n) 2^-24 <= 2^-17.5 of its sum of
magnitudes, and the q p running sums of a form, whose errors are independent, to
sqrt(n / (q p)) 2^-24 <= 2^-24 / sqrt(q) of the form's: 2^-20 of the sum of magnitudes
covers both with room."""
import numpy as np
import pytest
import torch

import synth
from parity import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("outliers", [False, True])
@pytest.mark.parametrize("q,p", [(1, 1), (3, 127), (130, 129), (127, 301), (300, 640), (512, 512),
                                 (2048, 2048), (2100, 1056), (700, 2085)])
def test_objective_matches_fp64(qe, q, p, outliers):
    W = synth.gaussian((q, p), seed=61, std=0.02)
    Wh = (W + synth.gaussian((q, p), seed=62, std=0.004)).astype(np.float32)
    H = np.where(np.arange(q * p).reshape(q, p) % 97 == 5, synth.gaussian((q, p), seed=63, std=0.1),
                 0.0).astype(np.float32)
    X = synth.gaussian((p, 64), seed=64)
    X[::50] *= 30.0
    S = (X @ X.T).astype(np.float64)
    S = ((S + S.T) / 2 + 0.1 * np.eye(p) * np.trace(S) / p).astype(np.float32)
    out = host(qe.objective(dev(W), dev(Wh), dev(S), H=dev(H) if outliers else None))
    # the fp32 values the kernel forms, then 64 bits
    D = (Wh + H if outliers else Wh) - W
    for got, A in zip(out, (D, W)):
        A, S64 = A.astype(np.float64), S.astype(np.float64)
        ref = np.sum(A * (A @ S64))
        mag = np.sum(np.abs(A) * (np.abs(A) @ np.abs(S64)))
        assert abs(got - ref) <= 2.0 ** -20 * mag, (got, ref, mag)


def test_objective_long_runs(qe):
    """2048 x 8448: column tiles of up to 33 tiles of K in runs of 32 (8192 products in
    an fp32 sum) and a second run of one tile, against fp64 products on the device."""
    q, p = 2048, 8448
    W, Wh = dev(synth.gaussian((q, p), seed=68)), dev(synth.gaussian((q, p), seed=69))
    a = torch.arange(p, device="cuda")
    S = torch.where((a[:, None] // 7 + a[None, :] // 7) % 3 == 0, 1.0, -0.5) * (
        0.999 ** (a[:, None] - a[None, :]).abs().float())
    out = host(qe.objective(W, Wh, S))
    S64 = S.double()
    for got, A in zip(out, ((Wh - W).double(), W.double())):
        ref = float((A * (A @ S64)).sum())
        mag = float((A.abs() * (A.abs() @ S64.abs())).sum())
        assert abs(got - ref) <= 2.0 ** -20 * mag, (got, ref, mag)


def test_objective_unaligned(qe):
    """Rows of 4 k + 1 floats from a base 4 bytes off: no 16-byte alignment."""
    q, p = 260, 513
    W, Wh = synth.gaussian((q, p), seed=65), synth.gaussian((q, p), seed=66)
    A = synth.gaussian((p, p), seed=67)
    S = (A + A.T).astype(np.float32)

    def off(a):
        buf = torch.full((a.size + 65,), float("nan"), device="cuda")
        v = buf[1:1 + a.size].view(*a.shape)
        v.copy_(dev(a))
        return v
    out = host(qe.objective(off(W), off(Wh), off(S)))
    for got, A in zip(out, (Wh - W, W)):
        A, S64 = A.astype(np.float64), S.astype(np.float64)
        mag = np.sum(np.abs(A) * (np.abs(A) @ np.abs(S64)))
        assert abs(got - np.sum(A * (A @ S64))) <= 2.0 ** -20 * mag
