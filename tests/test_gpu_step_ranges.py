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


# The first sizes whose stores go through to memory (176160768 bytes of arrays at 7, 6 and 14 bytes an element), and the
# limits up to which a launch's workgroups are not held back; from 2^27 elements on SGD and Lion take 512 lanes, here with a ragged
# last tile.
@pytest.mark.parametrize("kind,n", [("adamw", 25165824), ("adamw", 25165823), ("sgd", 29360128), ("lion", 29360127),
                                    ("adamw", 1 << 22), ("sgd", (1 << 22) - 1), ("lion", 1 << 22), ("sgd", (1 << 22) + 1),
                                    ("sgd", (1 << 27) + 77), ("lion", (1 << 27) + 4095), ("lion", (1 << 27) - 1)])
def test_launch_rules_on_both_sides_of_their_limits(kind, n):
    rng = np.random.default_rng(n)
    small = 1000
    thp = rng.normal(0, 0.02, n).astype(np.float32).view(np.uint32) >> 16
    g = (rng.normal(0, 1e-4, n).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    for sizes in ((n,), (small, n - small)):             # one tensor (no table), and a list
        cut = np.cumsum((0,) + sizes)
        states = [_state(rng, k, kind, thp[a:a + k]) for a, k in zip(cut, sizes)]
        grads = [g[a:a + k] for a, k in zip(cut, sizes)]
        bufs = [upload_state(st) for st in states]
        for b, x in zip(bufs, grads):
            b.lr, b.weight_decay = 1e-3, 0.01
            b.grad.copy_(to_dev_u16(x, torch.bfloat16))
        _step(kind, bufs, states, grads, 1, HP)
        for b, st in zip(bufs, states):
            _same(b, st, f"{kind} {sizes}")


# Tensors of whole groups of tiles and of a tile or an element more or less, beside one that makes the launch large enough for
# them to be dealt out (32 tiles of 2048 elements).
@pytest.mark.parametrize("kind", ["sgd", "lion"])
def test_tiles_around_a_group_that_is_dealt_out(kind):
    rng = np.random.default_rng(11)
    sizes = [32 * 2048 * k + d for k in (1, 2) for d in (-2048, -1, 0, 1, 2048, 2049)] + [29360128 + 31 * 2048 + 7]
    bufs, states, grads = [], [], []
    for n in sizes:
        thp = rng.normal(0, 0.02, n).astype(np.float32).view(np.uint32) >> 16
        states.append(_state(rng, n, kind, thp))
        bufs.append(upload_state(states[-1]))
        bufs[-1].lr, bufs[-1].weight_decay = 1e-3, 0.01
        grads.append((rng.normal(0, 1e-4, n).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16))
        bufs[-1].grad.copy_(to_dev_u16(grads[-1], torch.bfloat16))
    _step(kind, bufs, states, grads, 1, HP)
    for b, st in zip(bufs, states):
        _same(b, st, f"{kind} numel {st.n}")


# A launch holds 2^28 elements; the second one of this list is far below the size from which stores go through, and a group of tiles
# that are dealt out lies across the cut.  Every element of every array.
@pytest.mark.parametrize("kind,split,quant", [("sgd", True, True), ("lion", True, True), ("adamw", True, False), ("sgd", False, True)])
def test_tiles_that_are_dealt_out_across_two_launches(kind, split, quant):
    arrays = [("param", "thp"), ("rho", "rho"), ("theta", "theta32"), ("m_q", "mq"), ("m_scale", "ms"), ("v_q", "vq"), ("v_scale", "vs"),
              ("m", "m32"), ("v", "v32")]
    rng = np.random.default_rng(28)
    theta = rng.normal(0, 0.02, 1000003).astype(np.float32)
    grad = (rng.normal(0, 1e-4, 1000003).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    bufs, states, grads = [], [], []
    for n in (17 * 4096, (1 << 28) + 200000):
        st = oracle.TensorState(np.resize(theta, n), kind, split_weights=split, quantize_states=quant)
        b = fo.ParamBuffers(n, kind, split_weights=split, quantize_states=quant)
        for x, y in arrays:
            if getattr(b, x) is not None:
                getattr(b, x).view(torch.uint8).copy_(torch.from_numpy(getattr(st, y).view(np.uint8)))
        grads.append(np.resize(grad, n))
        b.grad.copy_(to_dev_u16(grads[-1], torch.bfloat16))
        b.lr, b.weight_decay = 1e-3, 0.01
        bufs.append(b)
        states.append(st)
    lr, wd = np.float32(1e-3), np.float32(0.01)
    if kind == "adamw":
        fo.adamw_step_ex(bufs, HP["beta1"], HP["beta2"], HP["eps"], 1)
    elif kind == "sgd":
        (fo.sgd_step if split else fo.sgd_step_ex)(bufs, HP["momentum"])
    else:
        fo.lion_step(bufs, HP["beta1"], HP["beta2"])
    for b, st, g in zip(bufs, states, grads):
        if kind == "adamw":
            oracle.adamw_step(st, g, lr, wd, HP["beta1"], HP["beta2"], HP["eps"], 1, 16)
        elif kind == "sgd":
            oracle.sgd_step(st, g, lr, wd, HP["momentum"], 16)
        else:
            oracle.lion_step(st, g, lr, wd, HP["beta1"], HP["beta2"], 16)
        for x, y in arrays:
            if getattr(b, x) is not None:
                got, want = getattr(b, x).view(torch.uint8).cpu().numpy(), getattr(st, y).view(np.uint8)
                assert np.array_equal(got, want), f"{x}: {int((got != want).sum())} bytes of {want.size}, numel {st.n}"


@pytest.mark.parametrize("kind,split,quant,n", [("adamw", False, False, 12582912), ("sgd", False, False, 17616077),
                                                ("adamw", True, False, 13550829), ("lion", True, False, 19573419),
                                                ("adamw", False, True, 22020096), ("sgd", False, True, 25165824)])
def test_ablation_launch_rules_on_both_sides_of_their_limits(kind, split, quant, n):
    # (the first sizes whose stores go through: 14, 10, 13, 9, 8 and 7 bytes an element)
    f32 = lambda t: t.cpu().numpy().view(np.uint32)
    for k in (n, n - 1):
        rng = np.random.default_rng(k)
        st = oracle.TensorState(rng.normal(0, 0.02, k).astype(np.float32), kind, split_weights=split, quantize_states=quant)
        b = fo.ParamBuffers(k, kind, split_weights=split, quantize_states=quant)
        if split:
            b.param.copy_(to_dev_u16(st.thp, torch.bfloat16)); b.rho.copy_(torch.from_numpy(st.rho))
        else:
            b.theta.copy_(torch.from_numpy(st.theta32))
        g = (rng.normal(0, 1e-4, k).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
        b.grad.copy_(to_dev_u16(g, torch.bfloat16))
        b.lr, b.weight_decay = 1e-3, 0.01
        lr, wd = np.float32(b.lr), np.float32(b.weight_decay)
        if kind == "adamw":
            fo.adamw_step_ex([b], HP["beta1"], HP["beta2"], HP["eps"], 1)
            oracle.adamw_step(st, g, lr, wd, HP["beta1"], HP["beta2"], HP["eps"], 1, 16)
        elif kind == "sgd":
            fo.sgd_step_ex([b], HP["momentum"])
            oracle.sgd_step(st, g, lr, wd, HP["momentum"], 16)
        else:
            fo.lion_step_ex([b], HP["beta1"], HP["beta2"])
            oracle.lion_step(st, g, lr, wd, HP["beta1"], HP["beta2"], 16)
        if split:
            assert np.array_equal(bits16(b.param), st.thp) and np.array_equal(b.rho.cpu().numpy(), st.rho)
        else:
            assert np.array_equal(f32(b.theta), st.theta32.view(np.uint32))
        if quant:
            assert np.array_equal(b.m_q.cpu().numpy(), st.mq) and np.array_equal(bits16(b.m_scale), st.ms)
        else:
            assert np.array_equal(f32(b.m), st.m32.view(np.uint32))
        if kind == "adamw" and quant:
            assert np.array_equal(b.v_q.cpu().numpy(), st.vq) and np.array_equal(bits16(b.v_scale), st.vs)
        elif kind == "adamw":
            assert np.array_equal(f32(b.v), st.v32.view(np.uint32))


@pytest.mark.parametrize("n", [(1 << 23) - 1, (1 << 23) + 1])
def test_codecs_on_both_sides_of_the_limit_of_their_stores(n):
    rng = np.random.default_rng(n)
    x = rng.normal(0, 1e-3, n).astype(np.float32)
    d, ng = torch.from_numpy(x).cuda(), (n + 31) // 32
    e = lambda k, dt: torch.zeros(k, dtype=dt, device="cuda")
    p, r, mq, ms, back = e(n, torch.bfloat16), e(n, torch.int8), e(n, torch.int8), e(ng, torch.float16), e(n, torch.float32)
    fo.split_weights(d, p, r)
    thp, rho = oracle.split(x)
    assert np.array_equal(bits16(p), thp) and np.array_equal(r.cpu().numpy(), rho)
    fo.reconstruct_weights(p, r, back)
    assert np.array_equal(back.cpu().numpy().view(np.uint32), oracle.reconstruct(thp, rho).view(np.uint32))
    fo.quantize_momentum(d, mq, ms)
    q, s = oracle.quantize_momentum(x)
    assert np.array_equal(mq.cpu().numpy(), q) and np.array_equal(bits16(ms), s)
    fo.dequantize_momentum(mq, ms, back)
    assert np.array_equal(back.cpu().numpy().view(np.uint32), oracle.dequantize_momentum(q, s).view(np.uint32))
    v, vq, vs = d * d, e(n, torch.uint8), e(ng, torch.float16)
    fo.quantize_variance(v, vq, vs)
    q, s = oracle.quantize_variance(v.cpu().numpy())
    assert np.array_equal(vq.cpu().numpy(), q) and np.array_equal(bits16(vs), s)
    fo.dequantize_variance(vq, vs, back)
    assert np.array_equal(back.cpu().numpy().view(np.uint32), oracle.dequantize_variance(q, s).view(np.uint32))


@pytest.mark.parametrize("n", [(1 << 25) + 1, (1 << 25) - 1, 1 << 22, (1 << 22) - 1])
def test_conversions_on_both_sides_of_their_limits(n):
    g = torch.Generator(device="cuda").manual_seed(n)
    f = fo.ParamBuffers(n, "sgd", with_grad=False, split_weights=False, quantize_states=False)
    f.theta.normal_(0, 0.02, generator=g)
    f.m.normal_(0, 1e-4, generator=g)
    c = fo.ParamBuffers(n, "sgd", with_grad=False)
    c.theta, c.m = f.theta, f.m
    theta, m = f.theta.cpu().numpy(), f.m.cpu().numpy()
    fo.compress_state("sgd", [c])
    thp, rho = oracle.split(theta)
    q, s = oracle.quantize_momentum(m)
    got = download(c)
    assert np.array_equal(got["thp"], thp) and np.array_equal(got["rho"], rho)
    assert np.array_equal(got["mq"], q) and np.array_equal(got["ms"], s)
    fo.decompress_state("sgd", [c])
    assert np.array_equal(f.theta.cpu().numpy().view(np.uint32), oracle.reconstruct(thp, rho).view(np.uint32))
    assert np.array_equal(f.m.cpu().numpy().view(np.uint32), oracle.dequantize_momentum(q, s).view(np.uint32))


# To FP32, tensors of whole groups of tiles and of a tile or an element more or less, beside one that makes the call large enough for
# them to be dealt out (32 tiles of 1024 elements).
@pytest.mark.parametrize("kind", ["adamw", "sgd"])
def test_decompressing_around_a_group_that_is_dealt_out(kind):
    g = torch.Generator(device="cuda").manual_seed(5)
    bufs = []
    for n in [32 * 1024 * k + d for k in (1, 2) for d in (-1024, -1, 0, 1, 1024, 1025)] + [(1 << 25) + 31 * 1024 + 7]:
        f = fo.ParamBuffers(n, kind, with_grad=False, split_weights=False, quantize_states=False)
        c = fo.ParamBuffers(n, kind, with_grad=False)
        c.param.normal_(0, 0.02, generator=g)
        for q, lo, hi in ((c.rho, -127, 128), (c.m_q, -127, 128), (c.v_q, 0, 256)):
            if q is not None:
                q.random_(lo, hi, generator=g)
        for s in (c.m_scale, c.v_scale):
            if s is not None:
                s.uniform_(1e-5, 1e-3, generator=g)
        c.theta, c.m, c.v = f.theta, f.m, f.v
        bufs.append(c)
    fo.decompress_state(kind, bufs)
    bits = lambda t: t.cpu().numpy().view(np.uint32)
    for c in bufs:
        got = download(c)
        assert np.array_equal(bits(c.theta), oracle.reconstruct(got["thp"], got["rho"]).view(np.uint32)), c.numel
        assert np.array_equal(bits(c.m), oracle.dequantize_momentum(got["mq"], got["ms"]).view(np.uint32)), c.numel
        if kind == "adamw":
            assert np.array_equal(bits(c.v), oracle.dequantize_variance(got["vq"], got["vs"]).view(np.uint32)), c.numel


@pytest.mark.parametrize("n", [1 << 25, (1 << 25) - 1])       # single wavefronts, and 256 lanes
def test_compressing_a_list_on_both_sides_of_its_limit(n):
    sizes = [1, 31, 255, 256, 257, 1023, 1025, 4097]
    sizes.append(n - sum(sizes))
    g = torch.Generator(device="cuda").manual_seed(n)
    bufs = []
    for k in sizes:
        f = fo.ParamBuffers(k, "adamw", with_grad=False, split_weights=False, quantize_states=False)
        f.theta.normal_(0, 0.02, generator=g)
        f.m.normal_(0, 1e-4, generator=g)
        f.v.normal_(0, 1e-4, generator=g).square_()
        c = fo.ParamBuffers(k, "adamw", with_grad=False)
        c.theta, c.m, c.v = f.theta, f.m, f.v
        bufs.append(c)
    fo.compress_state("adamw", bufs)
    for c in bufs:
        thp, rho = oracle.split(c.theta.cpu().numpy())
        mq, ms = oracle.quantize_momentum(c.m.cpu().numpy())
        vq, vs = oracle.quantize_variance(c.v.cpu().numpy())
        for k, want in dict(thp=thp, rho=rho, mq=mq, ms=ms, vq=vq, vs=vs).items():
            assert np.array_equal(download(c)[k], want), (c.numel, k)


# Whatever differs, unpacking has to leave every buffer as it was: any word of the header and of the table, in a table that
# ends inside a workgroup's first pass and in longer ones.
@pytest.mark.parametrize("n_tensors", [1, 5, 600, 5000])
def test_unpacking_checks_every_word_of_the_table(n_tensors):
    bufs = [fo.ParamBuffers(1 + i % 67, "sgd", with_grad=False) for i in range(n_tensors)]
    for i, b in enumerate(bufs):
        b.rho.fill_(i % 50 + 1)
    blob = torch.zeros(fo.checkpoint_size("sgd", [b.numel for b in bufs]), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("sgd", bufs, 5, blob)
    table = 64 + 16 * n_tensors
    for b in bufs:
        b.rho.zero_()
    for at in sorted({0, 4, 8, 12, 24, 32, 40, 48, 56, 63, 64, table // 2 // 4 * 4, table - 16, table - 5, table - 1}):
        blob[at] ^= 0x10
        with pytest.raises(fo.FlashOptimError) as err:
            fo.checkpoint_unpack("sgd", blob, bufs)
        assert err.value.status == -5, at
        blob[at] ^= 0x10
    assert not any(b.rho.any() for b in bufs[::97])
    for step in (0, 1 << 40, 2**63 - 1):                # the step is the caller's
        blob[16:24] = torch.from_numpy(np.frombuffer(np.int64(step).tobytes(), np.uint8).copy()).cuda()
        assert fo.checkpoint_unpack("sgd", blob, bufs) == step
    assert all((b.rho == i * 97 % 50 + 1).all() for i, b in enumerate(bufs[::97]))


# Blobs of 24 to 256 MB whose header and table are 4 KB or less (252 tensors) are checked by every workgroup of the copy: both sides of these
# limits, and words all over a long and a short table.
@pytest.mark.parametrize("n_tensors,n", [(252, 110_000), (253, 110_000), (1020, 26_000), (1021, 26_000), (3, 9_000_000), (3, 1_900_000), (3, 2_200_000)])
def test_unpacking_checks_every_word_within_the_copy(n_tensors, n):
    sizes = [n + i % 7 for i in range(n_tensors)]
    off = np.cumsum([0] + [(k + 255) // 256 * 256 for k in sizes])
    arena = fo.ParamBuffers(int(off[-1]), "sgd", with_grad=False)
    bufs = fo.TensorList([arena.shard(int(o), k) for o, k in zip(off, sizes)])
    blob = torch.zeros(fo.checkpoint_size("sgd", sizes), dtype=torch.uint8, device="cuda")
    arena.rho.fill_(3)
    fo.checkpoint_pack("sgd", bufs, 5, blob)
    arena.rho.zero_()
    table = 64 + 16 * n_tensors
    for at in sorted({0, 4, 8, 12, 24, 32, 40, 48, 56, 63, 64, table // 2 // 4 * 4, table - 16, table - 5, table - 1}):
        blob[at] ^= 0x10
        with pytest.raises(fo.FlashOptimError) as err:
            fo.checkpoint_unpack("sgd", blob, bufs)
        assert err.value.status == -5, at
        blob[at] ^= 0x10
    assert not arena.rho.any()
    for step in (0, 1 << 40, 2**63 - 1):                # the step is the caller's
        blob[16:24] = torch.from_numpy(np.frombuffer(np.int64(step).tobytes(), np.uint8).copy()).cuda()
        assert fo.checkpoint_unpack("sgd", blob, bufs) == step
    assert all((arena.rho[int(o):int(o) + k] == 3).all() for o, k in zip(off, sizes))


@pytest.mark.parametrize("n", [65_000_000, 67_000_000])      # blobs of 264 and 272 MB: checked in the copy, and ahead of it
def test_unpacking_on_both_sides_of_the_limit_of_its_blob(n):
    b = fo.ParamBuffers(n, "lion", with_grad=False)
    for x, lo, hi in ((b.rho, -127, 128), (b.m_q, -127, 128), (b.param.view(torch.int16), -32768, 32768), (b.m_scale.view(torch.int16), 0, 31744)):
        x.random_(lo, hi)
    arrays = lambda t: [t.param.view(torch.int16), t.rho, t.m_q, t.m_scale.view(torch.int16)]
    blob = torch.zeros(fo.checkpoint_size("lion", [n]), dtype=torch.uint8, device="cuda")
    fo.checkpoint_pack("lion", [b], 12, blob)
    f = fo.ParamBuffers(n, "lion", with_grad=False)
    blob[24] ^= 1
    with pytest.raises(fo.FlashOptimError):
        fo.checkpoint_unpack("lion", blob, [f])
    assert not any(x.any() for x in arrays(f))
    blob[24] ^= 1
    assert fo.checkpoint_unpack("lion", blob, [f]) == 12
    assert all(torch.equal(x, y) for x, y in zip(arrays(f), arrays(b)))


# Lists whose coarse table spans several tiles and tensors with one entry: the tensor of a tile is searched for.
@pytest.mark.parametrize("order", ["small first", "large first", "large among small"])
def test_tiles_of_long_lists(order):
    rng = np.random.default_rng(3)
    sizes = [1 + i * 37 % 3000 for i in range(3000)]
    sizes.insert({"small first": 3000, "large first": 0, "large among small": 1234}[order], 40000001)
    total = sum(sizes)
    cut = np.cumsum([0] + sizes)
    x = np.resize(rng.normal(0, 0.02, 1000003).astype(np.float32), total)
    m = np.resize(rng.normal(0, 1e-4, 1000033).astype(np.float32), total)
    g = np.resize((rng.normal(0, 1e-4, 1000037).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16), total)
    bufs, states = [], []
    for a, k in zip(cut, sizes):
        b = fo.ParamBuffers(k, "sgd")
        b.theta, b.m = torch.from_numpy(x[a:a + k]).cuda(), torch.from_numpy(m[a:a + k]).cuda()
        b.grad.copy_(to_dev_u16(g[a:a + k], torch.bfloat16))
        b.lr, b.weight_decay = 1e-3, 0.01
        st = oracle.TensorState(np.zeros(k, np.float32), "sgd")
        st.thp, st.rho = oracle.split(x[a:a + k])
        st.mq, st.ms = oracle.quantize_momentum(m[a:a + k])
        bufs.append(b)
        states.append(st)
    fo.compress_state("sgd", bufs)
    for i, (b, st) in enumerate(zip(bufs, states)):
        _same(b, st, f"compress, tensor {i}")
        b.theta, b.m = torch.zeros_like(b.theta), torch.zeros_like(b.m)
    fo.decompress_state("sgd", bufs)
    for i, (b, st) in enumerate(zip(bufs, states)):
        assert np.array_equal(b.theta.cpu().numpy().view(np.uint32), oracle.reconstruct(st.thp, st.rho).view(np.uint32)), i
        assert np.array_equal(b.m.cpu().numpy().view(np.uint32), oracle.dequantize_momentum(st.mq, st.ms).view(np.uint32)), i
    _step("sgd", bufs, states, [g[a:a + k] for a, k in zip(cut, sizes)], 1, HP)
    for i, (b, st) in enumerate(zip(bufs, states)):
        _same(b, st, f"step, tensor {i}")
