"""The decoders' factors, which the kernels form in fewer operations than the divisions that define them: every code byte."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_23349_amd as fo
from helpers import to_dev_u16

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
