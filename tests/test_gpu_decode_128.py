"""d_model 128 in the fused decoder, at every number of lanes per workgroup: the
f32 products of two lanes run on a shorter ring of weights there than at the
other widths.  The bytes have to come back exactly."""
import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_decode_d128(dtype):
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(128, 2)
    m = boa.Model(cfg, init_weights(cfg, 21))
    lens = np.array([1, 2, 3, 4, 5, 6, 7, 8, 9, 40, 2, 3, 70, 1, 4, 5, 64, 65, 33, 2, 6, 20, 3], dtype=np.uint64)
    data = records_f32_mix(int(lens.sum()), 128)
    first = data[np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int64)]
    pay, off, plen, _ = boa.encode_dev(m, torch.from_numpy(data).cuda(), lens, dtype=dtype, ideal=False)
    plen = plen.cpu().numpy().astype(np.uint32).astype(np.uint64)
    for g in (1, 2, 4, 8, 16):
        print(f"[gpu] decode d128 {dtype} lanes/wg {g}", flush=True)
        out = boa.decode_dev(m, pay, off, plen, first, lens, dtype=dtype, decode_kernel="fused", fused_lanes=g, max_lanes=17)
        assert np.array_equal(out.cpu().numpy(), data)
