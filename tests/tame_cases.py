"""Hyper-parameters and scales around the ends of the range in which the update pass takes its short root and division, and the
conditions of that range one by one (adam.hpp: tame_range), so that a test can say which of them its cases meet."""
from __future__ import annotations

import math

import numpy as np

from paper_2310_18313_amd import binding as B

# lr is large where the update is to show: an fp32 master weight then resolves single ulps of the quotient
HPS = {
    "plain": dict(lr=3e-4, step=100),
    "first step": dict(lr=3e-4, step=1, beta2=0.999),
    "no momentum": dict(lr=1e-2, step=7, beta1=0.0, beta2=0.0, weight_decay=0.0),
    "small eps, late": dict(lr=1.0, step=100000, eps=2.0 ** -36, beta1=0.999, beta2=0.9999),
    "large eps, full decay": dict(lr=1.0, step=3, eps=1024.0, weight_decay=1.0),
    "huge eps": dict(lr=1024.0, step=3, eps=2.0 ** 70, weight_decay=0.0),
    "small beta1": dict(lr=1.0, step=2, beta1=2.0 ** -9, weight_decay=0.0),
    "small beta2": dict(lr=1.0, step=2, beta2=2.0 ** -9, weight_decay=0.0),
    "betas near one": dict(lr=1.0, step=2, beta1=1.0 - 2.0 ** -23, beta2=1.0 - 2.0 ** -23, weight_decay=0.0),
}
N_TENSORS = 700


def scales(hp: str, master: int) -> dict:
    """Per buffer the tensors' scales: a third as a run has them, the others anywhere between well past the ends; a few
    gradients carry the scale of an FP8 sum over three ranks."""
    nt = N_TENSORS
    rng = np.random.default_rng(1000 + 10 * list(HPS).index(hp) + master)
    usual = rng.random(nt) < 0.3

    def some(inside, anywhere):
        return np.ldexp(1.0, np.where(usual, rng.integers(*inside, nt), rng.integers(*anywhere, nt))).astype(np.float32)

    out = {"g_meta": some((16, 32), (-30, 60)), "m_meta": some((14, 26), (-34, 66)), "v_meta": some((30, 45), (-64, 100)),
           "w_meta": some((10, 18), (-62, 48)) if master == B.STATE_F16 else np.ones(nt, np.float32)}
    out["g_meta"][rng.random(nt) < 0.04] *= np.float32(3.0)
    return out


def host_constants(h: B.AdamHparams) -> list:
    """b1, 1 - b1, 1 / (1 - b1^t), b2, 1 - b2, 1 / (1 - b2^t), eps as the library hands them to its kernels, and the decay."""
    f = np.float32
    out = []
    for b in (h.beta1, h.beta2):
        out += [f(b), f(1.0 - b), f(1.0 / (1.0 - math.pow(b, h.step)))]
    return [float(x) for x in out] + [float(f(h.eps)), float(f(1.0 - h.lr * h.weight_decay))]


def missed(const: list, inverse) -> set:
    """The conditions that a tensor with these inverse scales (gradient, moments, weight) does not meet."""
    b1, omb1, rbc1, b2, omb2, rbc2, eps, decay = const
    e = lambda x: math.frexp(x)[1] - 1
    isg, ism, isv, isw = (float(x) for x in inverse)
    eg, em, ev, ew, e1, e2, r1, r2 = (e(x) for x in (isg, ism, isv, isw, omb1, omb2, rbc1, rbc2))
    vhi = max(16 + ev, e2 + 1 + 2 * (eg + 16)) + 1 + r2 + 1
    vlo = min(1000 if b2 == 0 else e(b2) - 24 + ev, e2 + 2 * eg - 32) + r2
    j = min((60 - vhi) >> 1, 50)
    mlo = min(e1 + eg - 39, 1000 if b1 == 0 else e(b1) - 32 + em)
    mhi = max(9 + em, e1 + 1 + eg + 16) + 1
    met = {"gradient scale a power of two": math.frexp(isg)[0] == 0.5, "beta1": b1 == 0 or b1 >= 2.0 ** -8,
           "beta2": b2 == 0 or b2 >= 2.0 ** -8, "decay": decay == 0 or abs(decay) >= 2.0 ** -60,
           "gradient scale not too small": eg <= 24, "first moment, low": em >= -60, "first moment, high": em <= 31,
           "second moment, low": ev >= -90, "second moment, high": ev <= 60, "weight, low": ew >= -40, "weight, high": ew <= 60,
           "smallest gradient": e1 + eg - 16 >= -100, "smallest square": e2 + 2 * eg - 32 >= -120, "common factor": j >= -50,
           "smallest root": vlo + 2 * j >= -80, "eps, low": e(eps) + j >= -20, "eps, high": e(eps) + j <= 60,
           "smallest dividend": mlo + r1 + j >= -60, "largest dividend": mhi + r1 + 1 + j <= 60}
    return {k for k, ok in met.items() if not ok}


# conditions that no call can miss alone: 1 - lr * weight_decay is 0 or at least 2^-48 in double arithmetic of fp32 factors; a
# gradient small enough has too small a square first; v' / bc2 < 2^110 whatever the scales within the other conditions
IMPLIED = {"decay", "smallest gradient", "common factor"}
CONDITIONS = {"gradient scale a power of two", "beta1", "beta2", "gradient scale not too small", "first moment, low", "first moment, high",
              "second moment, low", "second moment, high", "weight, low", "weight, high", "smallest square", "smallest root",
              "eps, low", "eps, high", "smallest dividend", "largest dividend"}
