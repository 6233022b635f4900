"""The encoder's f32 products run on v_mfma_f32_16x16x4_f32; with one or two
lanes a workgroup the fused decoder runs the same chains as fmaf in increasing
k.  Their tables agree only if the two give the same bits, over all values."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, K = 96, 32


def _signs(rng, shape):
    return rng.choice(np.float32([-1, 1]), shape)


def _operands(kind, rng):
    shape = (N, 16, K)
    a, b = (rng.standard_normal(shape).astype(np.float32) for _ in range(2))
    if kind == "exponents":                       # products over 240 binades
        a *= np.exp2(rng.integers(-60, 61, shape)).astype(np.float32)
        b *= np.exp2(rng.integers(-60, 61, shape)).astype(np.float32)
    elif kind == "denormal inputs":
        a = (_signs(rng, shape) * rng.integers(0, 1 << 23, shape).astype(np.int32).view(np.float32)).astype(np.float32)
        b *= np.exp2(rng.integers(0, 24, shape)).astype(np.float32)
    elif kind == "denormal products":             # products and sums around 2^-149 .. 2^-120
        a *= np.exp2(rng.integers(-75, -60, shape)).astype(np.float32)
        b *= np.exp2(rng.integers(-75, -60, shape)).astype(np.float32)
    elif kind == "near overflow":                 # some sums pass the largest float on their way
        a *= np.exp2(rng.integers(60, 65, shape)).astype(np.float32)
        b *= np.exp2(rng.integers(60, 63, shape)).astype(np.float32)
    elif kind == "signed zeros":
        a = np.where(rng.random(shape) < 0.7, np.float32(0) * _signs(rng, shape), a).astype(np.float32)
        b = np.where(rng.random(shape) < 0.7, np.float32(0) * _signs(rng, shape), b).astype(np.float32)
        a[:N // 3] = np.float32(-0.0)
    elif kind == "cancellation":                  # pairs that cancel to the last bits
        a[..., 1::2] = -a[..., 0::2]
        b[..., 1::2] = np.nextafter(b[..., 0::2], np.float32(np.inf))
        b *= np.exp2(rng.integers(-20, 21, shape[:2] + (1,))).astype(np.float32)
    elif kind == "infinities and NaN":
        for x in (a, b):
            x[rng.random(shape) < 0.01] = np.inf
            x[rng.random(shape) < 0.01] = -np.inf
            x[rng.random(shape) < 0.003] = np.nan
    return a, b


@pytest.mark.parametrize("kind", ["plain", "exponents", "denormal inputs", "denormal products", "near overflow",
                                  "signed zeros", "cancellation", "infinities and NaN"])
def test_mfma_chain_is_the_fmaf_chain(kind):
    from paper_2511_11337_amd import _lib
    fn = _lib.load().boa_test_f32_chain
    fn.restype = C.c_int
    fn.argtypes = [C.c_void_p, C.c_void_p, C.c_uint32, C.c_uint32, C.c_void_p, C.c_void_p, C.c_void_p]
    a, b = _operands(kind, np.random.default_rng(len(kind)))
    da, db = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    out = [torch.empty((N, 16, 16), dtype=torch.float32, device="cuda") for _ in range(2)]
    print(f"[gpu] f32 chains: {kind}", flush=True)
    assert fn(da.data_ptr(), db.data_ptr(), N, K, out[0].data_ptr(), out[1].data_ptr(), None) == 0
    m, f = (t.cpu().numpy() for t in out)
    nan = np.isnan(m)
    assert np.array_equal(nan, np.isnan(f))
    assert np.array_equal(m.view(np.uint32)[~nan], f.view(np.uint32)[~nan])
    if kind == "plain":                           # and both are the product
        ref = np.matmul(a.astype(np.float64), b.astype(np.float64).transpose(0, 2, 1))
        mag = np.matmul(np.abs(a).astype(np.float64), np.abs(b).astype(np.float64).transpose(0, 2, 1))
        assert np.all(np.abs(m - ref) <= K * 2.0 ** -24 * mag)
