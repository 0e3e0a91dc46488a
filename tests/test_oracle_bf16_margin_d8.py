"""The margin of the d = 8 tiles (rows as two BF16 parts, queries as one, the
norm and the threshold as three parts each in the accumulator's start value),
checked on the CPU against FP64 with the arithmetic of the matrix unit spelled
out: BF16 operands rounded to nearest even, exact products, FP32 sums in any
order.  The margin is 1.25 times the proven bound; the error has to stay below
the bound itself."""
import itertools
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_1304_4327_amd", "csrc", "bf16_tile.hpp")


def _constants():
    """C1 and C2 of bf16_margin_d8 as the kernel has them."""
    body = re.search(r"bf16_margin_d8\(float qlen, float rlen\) \{(.*?)\n\}", open(SRC).read(), re.S).group(1)
    out = []
    for name in ("C1", "C2"):
        expr = re.search(name + r" = ([^,;]*)[,;]", body).group(1)
        expr = re.sub(r"0x1p-(\d+)f", r"(2.0 ** -\1)", expr)
        out.append(float(eval(re.sub(r"(\d)f\b", r"\1", expr), {"__builtins__": {}})))
    return out


def _bf16(x):
    """Round float32 to BF16 (nearest, ties to even), as float32."""
    u = np.asarray(x, np.float32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & np.uint32(0xFFFF0000)).view(np.float32)


def _parts(x, n):
    out, rest = [], np.asarray(x, np.float32)
    for _ in range(n):
        h = _bf16(rest)
        out.append(h)
        rest = (rest - h).astype(np.float32)
    return out


def _fp32_norm(x):
    """fmaf chain over the dimensions: one rounding a step."""
    s = np.zeros(x.shape[0], np.float32)
    for j in range(x.shape[1]):
        s = (x[:, j].astype(np.float64) ** 2 + s).astype(np.float32)
    return s


def _cases(rng, n, d):
    scale = 10.0 ** rng.uniform(-6, 6, (n, 1))
    q, r = rng.standard_normal((n, d)), rng.standard_normal((n, d))
    kind = rng.integers(0, 5, n)
    # operands half way between two BF16 numbers, where rounding costs most
    mid = (1.0 + 2.0 ** -8) * np.sign(q)
    q = np.where(kind[:, None] == 1, mid, q)
    r = np.where(kind[:, None] == 2, (1.0 + 2.0 ** -8 + 2.0 ** -16) * np.sign(r), r)
    # near each other and far from the centre; along each other
    r = np.where(kind[:, None] == 3, q * (1 + 1e-3 * rng.standard_normal((n, 1))), r)
    r = np.where(kind[:, None] == 4, mid * np.abs(r[:, :1]), r)
    q = np.where(kind[:, None] == 4, mid, q)
    return (q * scale).astype(np.float32), (r * scale * 10.0 ** rng.uniform(-2, 2, (n, 1))).astype(np.float32)


@pytest.mark.parametrize("d", [5, 6, 7, 8])
def test_error_stays_below_the_bound(d):
    c1, c2 = (c / 1.25 for c in _constants())
    rng = np.random.default_rng(d)
    q, r = _cases(rng, 60_000, d)  # already centred: the centre's rounding is inside C2
    exact = ((q.astype(np.float64) - r.astype(np.float64)) ** 2).sum(1)
    qn, rn = _fp32_norm(q), _fp32_norm(r)
    thr = (qn * rng.uniform(-1, 3, len(qn))).astype(np.float32)
    qb = _bf16(-2.0 * q)
    rh, rl = _parts(r, 2)
    terms = [rh[:, j] * qb[:, j].astype(np.float64) for j in range(d)]
    terms += [rl[:, j] * qb[:, j].astype(np.float64) for j in range(d)]
    start = _parts(rn, 3) + [-p for p in _parts(thr, 3)]
    # the three parts are the whole number
    for whole, parts in ((rn, start[:3]), (thr, [-p for p in start[3:]])):
        assert np.array_equal(sum(p.astype(np.float64) for p in parts), whole.astype(np.float64))
    ql, rl_ = np.sqrt(qn.astype(np.float64)), np.sqrt(rn.astype(np.float64))
    bound = c1 * ql * rl_ + c2 * (ql + rl_) ** 2
    # the value that is compared: D - thr, against |q - r|^2 - |q|^2 - thr; its
    # terms are no larger than (|q| + |r|)^2 but for the threshold's, which the
    # kernel keeps within a margin of the values it decides about
    near = np.abs(thr.astype(np.float64)) <= 2 * (ql + rl_) ** 2
    assert near.mean() > 0.5
    want = exact - qn.astype(np.float64) - thr
    qn_err = np.abs(qn.astype(np.float64) - (q.astype(np.float64) ** 2).sum(1))
    for order in itertools.islice(itertools.permutations(range(3)), 6):
        groups = [start, terms[:d], terms[d:]]
        acc = np.zeros(len(q), np.float32)
        for g in order:
            for t in groups[g]:
                acc = (acc.astype(np.float64) + t).astype(np.float32)
        err = np.abs(acc.astype(np.float64) - want) + qn_err
        assert np.all(err[near] <= bound[near]), float((err / bound)[near].max())


def test_the_operand_term_is_needed():
    """The C2 terms alone do not cover the operands' rounding (a margin without
    C1 would lose rows), so the check above has teeth."""
    _, c2 = _constants()
    q, r = _cases(np.random.default_rng(1), 20_000, 8)
    est = (_fp32_norm(r).astype(np.float64) + (_bf16(-2.0 * q).astype(np.float64) * r).sum(1)
           + _fp32_norm(q).astype(np.float64))
    exact = ((q.astype(np.float64) - r.astype(np.float64)) ** 2).sum(1)
    ql, rl = np.linalg.norm(q.astype(np.float64), axis=1), np.linalg.norm(r.astype(np.float64), axis=1)
    assert np.any(np.abs(est - exact) > c2 * (ql + rl) ** 2)
