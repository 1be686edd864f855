"""Sweeps from valid codes run row by row (Sec. 3.2: rows are independent; a
kept coordinate changes nothing), against the fp64 oracle through the parity
protocol of tests/parity.py, at the edges of the kernel's column groups (256),
of one wave's columns (1024) and of its range (16384), and where the choice
between this form and the blocked one is made on the device."""
import numpy as np
import pytest
import torch

import synth
from parity import dev, host, teacher_forced
from test_gpu_cd import check_parity, gpu_cd, layer

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,p,bits", [(3, 1, 4), (7, 3, 3), (5, 255, 4), (5, 256, 8), (5, 257, 3),
                                      (6, 512, 2), (6, 513, 4), (4, 1023, 3), (4, 1025, 4),
                                      (3, 2048, 1), (3, 4099, 3), (2, 16384, 4)])
def test_rows_match_oracle(qe, oracle, q, p, bits):
    W, X = layer(q, p, 64 if p > 8192 else 2 * p + 64, 51 + p, corr=0.5)
    # few tokens: more damping keeps the conditioning of the longer runs
    S32 = oracle.damp(oracle.gram(X), 4.0 if p > 8192 else 0.01).astype(np.float32)
    scale, zero = oracle.grid_minmax(W, bits)
    g = gpu_cd(qe, W, S32, bits, scale, zero, 3)
    check_parity(oracle, W, S32, bits, scale, zero, g, f"rows {q}x{p} b={bits}")
    one = gpu_cd(qe, W, S32, bits, scale, zero, 3, per_sweep=False)
    for k in ("What", "codes", "R"):
        assert np.array_equal(one[k], g[k])
    assert one["obj"] == g["obj"]


def test_choice_on_the_device(qe, oracle):
    """2048 x 2048 with few tokens: more coordinates would move in sweep 2 than
    the row form is given (blocked sweep), fewer in the later ones (rows)."""
    q = p = 2048
    W, X = layer(q, p, 1024, 52)
    S32 = oracle.damp(oracle.gram(X), 0.01).astype(np.float32)
    scale, zero = oracle.grid_minmax(W, 4)
    g = gpu_cd(qe, W, S32, 4, scale, zero, 5)
    one = gpu_cd(qe, W, S32, 4, scale, zero, 5, per_sweep=False)
    for k in ("What", "codes", "R"):
        assert np.array_equal(one[k], g[k])
    assert one["obj"] == g["obj"]
    # R rounds as in the blocked form exactly while the blocked form ran
    dense = gpu_cd(qe, W, S32, 4, scale, zero, 5, extra=qe.QE_CD_DENSE)
    same = [np.array_equal(a, b) for a, b in zip(g["Rs"], dense["Rs"])]

    def would_move(k):
        t = np.rint(g["whats"][k] / scale[:, None] + zero[:, None])
        u = t - g["Rs"][k] / np.diag(S32) / scale[:, None]
        return float(np.mean(np.clip(np.rint(u), 0, 15) != t))

    assert would_move(0) > 0.13 and would_move(1) < 0.1      # the line lies at 0.118 here
    assert same[0] and same[1] and not same[4], same
    rows = synth.row_sample(q, 48, 2)
    cut = lambda hist: [h[rows] for h in hist]
    teacher_forced(oracle, W[rows], S32.astype(np.float64), 4, scale[rows], zero[rows], cut(g["hist"]),
                   cut(g["whats"]), cut(g["Rs"]), label="choice 2048x2048")


def ar1(p, rho):
    """Sigma of AR(1) channels, exactly symmetric, with 1% damping."""
    a = np.arange(p)
    return (rho ** np.abs(a[:, None] - a[None, :]) + 0.01 * np.eye(p)).astype(np.float32)


@pytest.mark.parametrize("q,p", [(512, 512), (70, 1501), (2048, 2048)])
def test_warm_start_that_keeps_moving(qe, oracle, q, p):
    """From codes far off, most coordinates move in every one of seven sweeps (above
    the line of any shape): all of them run in the blocked form, also those past the
    first few of a call and in layers that What = W always leaves to the row form.
    (QE_RELAX_PERIOD keeps a call in the blocked form, here without a relaxed sweep.)"""
    W, S32 = synth.gaussian((q, p), seed=55, std=0.02), ar1(p, 0.9)
    scale, zero = oracle.grid_minmax(W, 4)
    c0 = synth.integers((q, p), seed=56, lo=0, hi=16)
    W0 = oracle.dequant(c0, scale, zero).astype(np.float32)
    start = dict(W0=W0, codes0=c0)
    want = gpu_cd(qe, W, S32, 4, scale, zero, 7, extra=qe.QE_RELAX_PERIOD(255), **start)
    moved = [np.mean(a != b) for a, b in zip([c0] + want["hist"], want["hist"])]
    assert min(moved) > 0.3, moved
    g = gpu_cd(qe, W, S32, 4, scale, zero, 7, **start)
    one = gpu_cd(qe, W, S32, 4, scale, zero, 7, per_sweep=False, **start)
    for k in range(7):
        assert np.array_equal(g["Rs"][k], want["Rs"][k]), f"sweep {k + 1}"
    for k in ("What", "codes", "R"):
        assert np.array_equal(one[k], want[k])
    assert one["obj"] == g["obj"] == want["obj"]


def few_tokens(p, n, seed, out=0):
    """Damped Gram matrix of n random tokens, exactly symmetric (on the device), the first
    `out` channels 30 times as large: the fewer tokens per channel and the more such
    channels, the more codes a sweep moves."""
    X = dev(synth.gaussian((p, n), seed=seed))
    X[:out] *= 30
    S = X @ X.T / n
    S = (S + S.T) / 2
    S.diagonal().add_(0.01 * S.diagonal().mean())
    return S.contiguous()


@pytest.mark.parametrize("q,p", [(2060, 1101), (1290, 2304), (1030, 3075), (520, 4100)])
def test_few_rows_round_as_many(qe, q, p):
    """Rows are independent: those of a layer small enough to apply another wave's moves
    several at a time end bit for bit as within a layer that applies them one by one."""
    W, S = dev(synth.gaussian((q, p), seed=59, std=0.02)), few_tokens(p, 4 * p, 60)
    scale, zero = qe.grid_minmax(W, 4)
    Wh, R, codes = torch.empty_like(W), torch.empty_like(W), torch.zeros((q, p), dtype=torch.uint8, device="cuda")
    qe.cd_sweep(W, S, 4, scale, zero, Wh, codes, R, 2, flags=qe.QE_INIT_FROM_W)
    n = q - 20
    few = [t[:n].clone() for t in (Wh, codes, R)]
    flags = qe.QE_R_VALID | qe.QE_CODES_VALID
    before = codes.clone()
    qe.cd_sweep(W, S, 4, scale, zero, Wh, codes, R, 2, flags=flags)
    qe.cd_sweep(W[:n], S, 4, scale[:n], zero[:n], few[0], few[1], few[2], 2, flags=flags)
    moves = float((codes != before)[:n].float().sum(1).mean())
    assert 16 < moves < 0.1 * p, moves               # lists of many moves, below the line
    for a, b in zip(few, (Wh, codes, R)):
        assert torch.equal(a, b[:n])


@pytest.mark.parametrize("q,p", [(70, 1501), (384, 1792)])
def test_few_rows_choose_their_second_sweep(qe, q, p):
    """As many tokens as channels, some of them large: the second sweep from What = W moves far more codes than
    the row form is given, also in a layer of few rows.  It runs in the blocked form, the
    third one row by row.  (QE_RELAX_PERIOD keeps a call in the blocked form.)"""
    W, S = dev(synth.gaussian((q, p), seed=61, std=0.02)), few_tokens(p, p, 62, out=p // 50)
    scale, zero = qe.grid_minmax(W, 4)

    def run(sweeps, extra=0):
        Wh, R, codes = torch.empty_like(W), torch.empty_like(W), torch.zeros((q, p), dtype=torch.uint8, device="cuda")
        qe.cd_sweep(W, S, 4, scale, zero, Wh, codes, R, sweeps, flags=qe.QE_INIT_FROM_W | extra)
        return codes, R
    one, two = run(1), run(2)
    assert float((one[0] != two[0]).float().mean()) > 0.2
    assert torch.equal(two[1], run(2, qe.QE_RELAX_PERIOD(255))[1])
    assert not torch.equal(run(3)[1], run(3, qe.QE_RELAX_PERIOD(255))[1])


def test_fixed_point_and_no_objective(qe, oracle):
    """Rows that stop moving leave the later sweeps early: the objective stays,
    and a call without one gives the same state."""
    W, X = layer(40, 300, 2048, 53, corr=0.5)
    S32 = oracle.damp(oracle.gram(X), 0.01).astype(np.float32)
    scale, zero = oracle.grid_minmax(W, 4)
    g = gpu_cd(qe, W, S32, 4, scale, zero, 60, per_sweep=False)
    assert g["obj"][-1] == g["obj"][-2] == g["obj"][40]
    assert all(a >= b for a, b in zip(g["obj"], g["obj"][1:]))
    Wd, Sd, sc, ze = dev(W), dev(S32), dev(scale), dev(zero)
    Wh, R, codes = dev(W), dev(W), dev(np.zeros(W.shape, np.uint8))
    qe.cd_sweep(Wd, Sd, 4, sc, ze, Wh, codes, R, 60)
    assert np.array_equal(host(Wh), g["What"]) and np.array_equal(host(R), g["R"])
    assert np.array_equal(host(codes), g["codes"])
    before = host(R).copy()
    qe.cd_sweep(Wd, Sd, 4, sc, ze, Wh, codes, R, 2, flags=qe.QE_R_VALID | qe.QE_CODES_VALID)
    assert np.array_equal(host(R), before) and np.array_equal(host(codes), g["codes"])


def test_more_sweeps_than_one_launch(qe, oracle):
    """With an objective a launch of the row form takes 128 sweeps; the next one starts
    from the state and the objective that it left.  Slowly settling rows (8 bits, from
    codes far off, rho = 0.995): still moving behind the 128th sweep and behind the
    256th.  The same state without an objective (one launch), and in two calls.  (Fewer
    than 16 rows: the row form from the first sweep on.)"""
    q, p, sweeps = 8, 1100, 300
    W, S32 = synth.gaussian((q, p), seed=57, std=0.02), ar1(p, 0.995)
    scale, zero = oracle.grid_minmax(W, 8)
    c0 = synth.integers((q, p), seed=58, lo=0, hi=256)
    W0 = oracle.dequant(c0, scale, zero).astype(np.float32)
    Wd, Sd, sc, ze = dev(W), dev(S32), dev(scale), dev(zero)

    def run(*calls, with_obj=True, extra=0):
        Wh, codes = dev(W0), dev(c0.astype(np.uint8))
        R, out, flags = torch.empty_like(Wd), [], qe.QE_CODES_VALID
        for k in calls:
            obj = torch.zeros(k, dtype=torch.float64, device="cuda")
            if out:
                obj[0] = out[-1]
                flags |= qe.QE_OBJ_IN
            qe.cd_sweep(Wd, Sd, 8, sc, ze, Wh, codes, R, k, flags=flags | extra,
                        obj=obj if with_obj else None)
            flags = qe.QE_R_VALID | qe.QE_CODES_VALID
            out += host(obj).tolist()
        return host(codes), host(Wh), host(R), out
    codes, Wh, R, f = run(sweeps)
    assert all(a >= b for a, b in zip(f, f[1:]))
    assert f[126] > f[127] > f[128] > f[130] and f[255] > f[256] > f[260]
    for got in (run(sweeps, with_obj=False), run(100, 200)):
        assert np.array_equal(got[0], codes) and np.array_equal(got[1], Wh) and np.array_equal(got[2], R)
    assert got[3] == f
    assert not np.array_equal(run(sweeps, extra=qe.QE_RELAX_PERIOD(255))[2], R)     # the blocked form's
    assert f[-1] == pytest.approx(oracle.objective(W, Wh, S32), rel=1e-4)


@pytest.mark.parametrize("dense", [False, True])
@pytest.mark.parametrize("q,p", [(17, 257), (150, 301), (129, 640), (260, 1027)])
def test_alignment_changes_nothing(qe, oracle, q, p, dense):
    """Arrays whose rows are not 16-byte aligned (an odd p, bases 4 bytes off), with
    NaN around them that any read past their ends would pick up: bitwise the
    results of aligned bases, in the blocked form and row by row."""
    W, X = layer(q, p, 2 * p, 54, corr=0.5)
    S32 = oracle.damp(oracle.gram(X), 0.01).astype(np.float32)
    scale, zero = oracle.grid_minmax(W, 4)
    flag = qe.QE_CD_DENSE if dense else 0
    want = gpu_cd(qe, W, S32, 4, scale, zero, 3, per_sweep=False, extra=flag)

    def off(a):
        buf = torch.full((a.size + 67,), float("nan"), device="cuda")
        v = buf[1:1 + a.size].view(*a.shape)
        v.copy_(dev(a))
        return v
    Wh, R = off(np.zeros_like(W)), off(np.zeros_like(W))
    cbuf = torch.zeros(q * p + 8, dtype=torch.uint8, device="cuda")
    codes = cbuf[1:1 + q * p].view(q, p)
    qe.cd_sweep(off(W), off(S32), 4, dev(scale), dev(zero), Wh, codes, R, 3, flags=qe.QE_INIT_FROM_W | flag)
    assert np.array_equal(host(Wh), want["What"]) and np.array_equal(host(R), want["R"])
    assert np.array_equal(host(codes).astype(np.int32), want["codes"])
