"""The fused decoder where its phases can go wrong: chunks around the period of
the conv window on several chunks per lane, lanes that end early, and the lane
counts at which the automatic number of lanes per workgroup changes.  The
decoder must rebuild the encoder's integer tables, so the bytes have to come
back exactly."""
import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu


def _round_trip(m, data, lens, dtype, **kw):
    import paper_2511_11337_amd as boa
    first = data[np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int64)]
    pay, off, plen, _ = boa.encode_dev(m, torch.from_numpy(data).cuda(), lens, dtype=dtype, ideal=False)
    plen = plen.cpu().numpy().astype(np.uint32).astype(np.uint64)
    return boa.decode_dev(m, pay, off, plen, first, lens, dtype=dtype, **kw).cpu().numpy()


@pytest.mark.parametrize("D,groups", [(64, (1, 2, 4, 16)), (256, (1, 2, 8, 16)), (512, (1, 2, 4, 8))])
@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_decode_around_the_conv_window(D, groups, dtype):
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(D, 2)
    m = boa.Model(cfg, init_weights(cfg, 11 + D))
    lens = np.array([1, 2, 3, 4, 5, 6, 7, 8, 9, 40, 2, 3, 70, 1, 4, 5, 64, 65, 33, 2, 6, 20, 3], dtype=np.uint64)
    data = records_f32_mix(int(lens.sum()), D)
    for g in groups:
        print(f"[gpu] decode shapes d{D} {dtype} lanes/wg {g}", flush=True)
        assert np.array_equal(_round_trip(m, data, lens, dtype, decode_kernel="fused", fused_lanes=g, max_lanes=7), data)


@pytest.mark.parametrize("lanes", [256, 257, 513])
def test_decode_lanes_around_a_full_chip(lanes):
    """One lane per workgroup up to 256 lanes, two from 257, four from 513."""
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(64, 2)
    m = boa.Model(cfg, init_weights(cfg, 3))
    lens = np.full(lanes, 9, dtype=np.uint64)
    data = records_f32_mix(int(lens.sum()), lanes)
    print(f"[gpu] decode of {lanes} lanes", flush=True)
    assert np.array_equal(_round_trip(m, data, lens, "bf16"), data)


def test_small_region_takes_one_lane_per_workgroup():
    """300 lanes choose two lanes per workgroup and state in device memory; a region that holds only the one-lane
    form (state in LDS) still decodes, one byte less is refused."""
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(64, 2)
    m = boa.Model(cfg, init_weights(cfg, 5))
    lens = np.full(300, 11, dtype=np.uint64)
    data = records_f32_mix(int(lens.sum()), 9)
    small = boa.workspace_size(m, lens, "decode", dtype="bf16", fused_lanes=1)
    assert small < boa.workspace_size(m, lens, "decode", dtype="bf16")
    print(f"[gpu] decode of 300 lanes in {small} bytes", flush=True)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    assert np.array_equal(_round_trip(m, data, lens, "bf16", workspace=ws), data)
    with pytest.raises(boa.BoaError):
        _round_trip(m, data, lens, "bf16", workspace=ws[:small - 1])
