"""The steps at the edges of the ranges in which they take a shorter route, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_23349_amd as fo
from helpers import bits16, download, to_dev_u16, upload_state

pytestmark = pytest.mark.gpu


def _step(kind, bufs, states, grads, t, hp, nthreads=16):
    """One exact step of the list on the GPU and of every tensor on the oracle."""
    tl = fo.TensorList(bufs)
    if kind == "adamw":
        fo.adamw_step_exact(tl, hp["beta1"], hp["beta2"], hp["eps"], t)
    elif kind == "sgd":
        fo.sgd_step(tl, hp["momentum"])
    else:
        fo.lion_step(tl, hp["beta1"], hp["beta2"])
    for b, st, g in zip(bufs, states, grads):
        lr, wd = np.float32(b.lr), np.float32(b.weight_decay)
        if kind == "adamw":
            oracle.adamw_step(st, g, lr, wd, hp["beta1"], hp["beta2"], hp["eps"], t, nthreads)
        elif kind == "sgd":
            oracle.sgd_step(st, g, lr, wd, hp["momentum"], nthreads)
        else:
            oracle.lion_step(st, g, lr, wd, hp["beta1"], hp["beta2"], nthreads)


def _same(b, st, where):
    got = download(b)
    nan = (st.thp & 0x7fff) > 0x7f80          # the sign of a NaN weight and the correction beside it are unspecified
    for k in got:
        want, have = getattr(st, k), got[k]
        if k in ("thp", "rho"):
            want, have = want[~nan], have[~nan]
        bad = np.flatnonzero(want != have)
        assert bad.size == 0, f"{where}: {bad.size} of {want.size} {k}, first at {bad[:1]}: {have[bad[:1]]} for {want[bad[:1]]}"
    assert np.array_equal(nan, (got["thp"] & 0x7fff) > 0x7f80), where


HP = dict(beta1=0.9, beta2=0.999, eps=1e-8, momentum=0.9)


def _state(rng, n, kind, thp):
    """A state with the given BF16 weights, any corrections and codes, and scales around 1e-4."""
    st = oracle.TensorState(np.zeros(n, np.float32), kind)
    ng = (n + 31) // 32
    st.thp = thp.astype(np.uint16)
    st.rho = rng.integers(-127, 128, n).astype(np.int8)
    st.mq = rng.integers(-127, 128, n).astype(np.int8)
    st.ms = rng.integers(0x0400, 0x1400, ng).astype(np.uint16)
    if kind == "adamw":
        st.vq = rng.integers(1, 256, n).astype(np.uint8)
        st.vs = rng.integers(0x0400, 0x1400, ng).astype(np.uint16)
    return st


@pytest.mark.parametrize("kind", ["adamw", "sgd", "lion"])
@pytest.mark.parametrize("n", [70001, (1 << 20) + 5])
@pytest.mark.parametrize("weights", ["exponents 0 to 24", "zeros among ordinary ones", "infinities among ordinary ones",
                                     "large", "shrinking out of the range"])
def test_weights_around_the_range_of_the_short_split(kind, n, weights):
    # the short forms of Algorithm 1 hold for magnitudes from 2^-110 on (exponent field 16 of theta'), before and after the
    # update; whole wavefronts of one kind, and wavefronts in which a single weight is outside
    rng = np.random.default_rng(n)
    sign = rng.integers(0, 2, n) << 15
    thp = (rng.normal(0, 0.02, n).astype(np.float32).view(np.uint32) >> 16).astype(np.int64)
    lr, wd = 1e-3, 0.01
    if weights == "exponents 0 to 24":
        thp = sign | rng.integers(0, 25 * 128, n)
        thp[n // 2:] = (sign | (rng.integers(15 * 128, 18 * 128, n)))[n // 2:]
        lr, wd = 1e-37, 0.0
    elif weights == "zeros among ordinary ones":
        thp[rng.random(n) < 2e-3] = 0
        thp[rng.random(n) < 2e-3] = 0x8000
        thp[:4096] = 0
    elif weights == "infinities among ordinary ones":
        thp[rng.random(n) < 1e-3] = 0x7f80
        thp[rng.random(n) < 1e-3] = 0xff80
        wd = 0.0
    elif weights == "large":
        thp = sign | rng.integers(250 * 128, 255 * 128, n)
        wd = 0.0
    else:
        wd = 0.0 if kind == "adamw" else 1000.0          # with lr 1e-3: theta - lr * wd * theta is next to nothing
    st = _state(rng, n, kind, thp)
    if weights == "infinities among ordinary ones":
        st.rho[((st.thp & 0x7fff) == 0x7f80) & (rng.random(n) < 0.5)] = 0
    b = upload_state(st)
    b.lr, b.weight_decay = lr, wd
    for t in (1, 2):
        g = (rng.normal(0, 1e-4, n).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
        if weights == "shrinking out of the range":
            g[rng.random(n) < 0.5] = 0
        b.grad.copy_(to_dev_u16(g, torch.bfloat16))
        _step(kind, [b], [st], [g], t, HP)
        _same(b, st, f"{kind} {weights} step {t}")


@pytest.mark.parametrize("beta1,steps", [(0.9, (163, 164, 165, 166)), (0.5, (24, 25, 26)), (0.0, (1, 2))])
def test_steps_around_the_one_from_which_the_momentum_needs_no_correction(beta1, steps):
    # 1 - beta1^t rounds to 1 in FP32 from t = 165 on for 0.9, from 25 on for 0.5 and always for 0
    rng = np.random.default_rng(7)
    states, bufs = [], []
    for n in (33, 5000, (1 << 20) + 100):
        thp = rng.normal(0, 0.02, n).astype(np.float32).view(np.uint32) >> 16
        states.append(_state(rng, n, "adamw", thp))
        bufs.append(upload_state(states[-1]))
        bufs[-1].lr, bufs[-1].weight_decay = 1e-3, 0.01
    for t in steps:
        grads = []
        for b in bufs:
            g = (rng.normal(0, 1e-4, b.numel).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
            b.grad.copy_(to_dev_u16(g, torch.bfloat16))
            grads.append(g)
        _step("adamw", bufs, states, grads, t, dict(HP, beta1=beta1))
        for b, st in zip(bufs, states):
            _same(b, st, f"beta1 {beta1} step {t} numel {st.n}")
