"""fp64 attention over operands that are already rounded to bf16, with a bound on
what rounding the weights can still change.

The bf16 kernels round a row's weights once, each by a factor within 1 +- 2^-9,
and divide by the sum of the rounded ones.  So with A the weighted mean of |v|,
|out - ref| <= 2^-9 (A + |ref|) / (1 - 2^-9), and the log of the sum is off by
2^-9 / (1 - 2^-9) at most."""
import numpy as np

import workload as W

EPS = 2.0 ** -9 / (1 - 2.0 ** -9)


def rotate(x, pos, base=10000.0):
    """Rotate-half embedding of x [n, heads, d] at pos [n], in fp64."""
    h = x.shape[-1] // 2
    ang = np.asarray(pos, np.float64)[:, None] * base ** (-np.arange(h) / h)
    c, s = np.cos(ang)[:, None], np.sin(ang)[:, None]
    x = x.astype(np.float64)
    return np.concatenate([x[..., :h] * c - x[..., h:] * s, x[..., h:] * c + x[..., :h] * s], -1)


def bf16(x):
    return W.round_to_bf16(x.astype(np.float32)).astype(np.float64)


def attend(logits, v, see=None):
    """logits [m, n] (natural), v [n, d], see [m, n] or None (all): (out, bound on
    out's rounding error, lse)."""
    x = logits if see is None else np.where(see, logits, -np.inf)
    top = x.max(-1, keepdims=True)
    p = np.exp(x - top)
    total = p.sum(-1, keepdims=True)
    out = p @ v / total
    return out, EPS * (p @ np.abs(v) / total + np.abs(out)), (top + np.log(total))[:, 0]


def beyond(got, out, bound):
    """Share of elements off by more than the bound (and fp32's own rounding), and the largest error over it."""
    r = np.abs(got - out) / (1.01 * bound + 2e-6)
    return float((r > 1).mean()), float(r.max())
