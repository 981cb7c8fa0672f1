"""The decoders' factors, which the kernels form in fewer operations than the divisions that define them: every code byte."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_23349_amd as fo
from helpers import bits16, download, to_dev_u16, upload_state

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("state", ["momentum", "variance"])
def test_every_code_of_every_kind_of_scale(state, linear):
    # 256 codes in eight groups, for zero, the smallest and largest subnormals, powers of two, odd mantissas and 65504
    scales = np.array([0, 1, 2, 0x3ff, 0x400, 0x401, 0x1234, 0x2c00, 0x2d55, 0x3c00, 0x3fff, 0x7bff], np.uint16)
    q = np.tile(np.arange(256, dtype=np.uint8), scales.size)
    s = np.repeat(scales, 8)
    code = q.view(np.int8) if state == "momentum" else q
    want = (oracle.dequantize_momentum if state == "momentum" else oracle.dequantize_variance)(code, s, linear)
    out = torch.empty(q.size, dtype=torch.float32, device="cuda")
    fo.dequantize_state(state, linear, torch.from_numpy(code.copy()).cuda(), to_dev_u16(s, torch.float16), out)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))


def test_every_correction_of_every_exponent():
    thp = np.repeat((np.arange(0, 256) << 7).astype(np.uint16), 256)
    thp[::3] |= 0x805d                                  # some negative, some with a mantissa (NaN where the exponent is 255)
    rho = np.tile(np.arange(256, dtype=np.uint8), 256).view(np.int8)
    out = torch.empty(thp.size, dtype=torch.float32, device="cuda")
    fo.reconstruct_weights(to_dev_u16(thp, torch.bfloat16), torch.from_numpy(rho.copy()).cuda(), out)
    got, want = out.cpu().numpy(), oracle.reconstruct(thp, rho)
    nan = np.isnan(want)
    assert np.array_equal(got.view(np.uint32)[~nan], want.view(np.uint32)[~nan]) and np.isnan(got[nan]).all()


@pytest.mark.parametrize("n", [1, 3, 4, 63, 64, 255, 256, 257, 511, 1023, 2049])
def test_sizes_around_a_wavefront(n):
    rng = np.random.default_rng(n)
    x = rng.normal(0, 0.02, n).astype(np.float32)
    p, r = torch.zeros(n, dtype=torch.bfloat16, device="cuda"), torch.zeros(n, dtype=torch.int8, device="cuda")
    p16, r16 = torch.zeros_like(p), torch.zeros(n, dtype=torch.int16, device="cuda")
    back, back16 = torch.zeros(n, device="cuda"), torch.zeros(n, device="cuda")
    d = torch.from_numpy(x).cuda()
    fo.split_weights(d, p, r)
    fo.reconstruct_weights(p, r, back)
    fo.split_weights_i16(d, p16, r16)
    fo.reconstruct_weights_i16(p16, r16, back16)
    for N, pp, rr, bb in ((127, p, r, back), (32767, p16, r16, back16)):
        thp, rho = oracle.split(x, N)
        assert np.array_equal(pp.view(torch.int16).cpu().numpy().view(np.uint16), thp) and np.array_equal(rr.cpu().numpy(), rho)
        assert np.array_equal(bb.cpu().numpy().view(np.uint32), oracle.reconstruct(thp, rho, N).view(np.uint32))


# Group maxima around every border of the momentum codes' estimate: no scale, subnormal scales (where the largest element can be
# half as large again as the scale), the largest one, and magnitudes on both sides of 2^100, from which the exact form is used.
MAXIMA = np.float32([0, 1e-45, 2.9e-8, 2.99e-8, 5e-8, 8.9e-8, 1.4e-6, 6.1e-5, 1e-3, 1, 1.0004, 65504, 65520, 1e5, 1e20, 1.2676e30,
                     1.2677e30, 1e36, 3.3e38])


def _momenta():
    rng = np.random.default_rng(11)
    x = rng.uniform(-1, 1, (MAXIMA.size * 8, 32)).astype(np.float32)
    x[1::8] **= 9                                        # most of the group far below its maximum
    x[2::8] *= np.float32(1e-6)
    x[3::8, 5:] = 0
    # ... and elements right at the ties between two codes: f(x) = x / (1 + x) = (k + 1/2) / 254
    tie = (np.arange(32) * 4 + 0.5) / 254
    x[4::8], x[5::8] = tie / (1 - tie), -np.nextafter((tie / (1 - tie)).astype(np.float32), np.float32(1))
    x[:, 0] = np.where(rng.integers(0, 2, x.shape[0]), 1, -1)
    with np.errstate(under="ignore"):
        return (x * np.repeat(MAXIMA, 8)[:, None]).astype(np.float32).reshape(-1)


def test_momentum_codes_of_every_kind_of_group():
    x = _momenta()
    q, s = torch.empty(x.size, dtype=torch.int8, device="cuda"), torch.empty(x.size // 32, dtype=torch.float16, device="cuda")
    fo.quantize_momentum(torch.from_numpy(x).cuda(), q, s)
    want_q, want_s = oracle.quantize_momentum(x)
    assert np.array_equal(bits16(s), want_s) and np.array_equal(q.cpu().numpy(), want_q)


@pytest.mark.parametrize("numel", [152 * 32, 1 << 20])       # four and eight elements to a lane
def test_step_with_momenta_of_every_kind_of_group(numel):
    g = np.resize((_momenta().view(np.uint32) >> 16).astype(np.uint16), numel)
    st = oracle.TensorState(np.full(numel, 0.02, np.float32), "sgd")
    b = upload_state(st)
    b.lr, b.weight_decay = 1e-30, 0.0
    b.grad.copy_(to_dev_u16(g, torch.bfloat16))
    fo.sgd_step([b], 0.9)
    oracle.sgd_step(st, g, np.float32(1e-30), np.float32(0), 0.9, 8)
    got = download(b)
    for k in ("mq", "ms", "thp", "rho"):
        assert np.array_equal(got[k], getattr(st, k)), k
