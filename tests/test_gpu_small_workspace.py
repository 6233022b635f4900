"""An encode call in a workspace smaller than its preferred size: a region sized
for a batch of many chunks also takes one of few, with shorter tiles and the
same bytes."""
import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu


def _payloads(m, data, lens, dtype, **kw):
    import paper_2511_11337_amd as boa
    pay, off, plen, _ = boa.encode_dev(m, data, lens, dtype=dtype, ideal=False, **kw)
    host, plen = pay.cpu().numpy(), plen.cpu().numpy().astype(np.uint32)
    return [host[int(o):int(o) + int(n)].tobytes() for o, n in zip(off, plen)]


@pytest.mark.parametrize("D,dtype", [(64, "f32"), (256, "bf16"), (512, "fp8")])
def test_region_of_a_batch_of_more_lanes(D, dtype):
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(D, 2)
    m = boa.Model(cfg, init_weights(cfg, 9))
    many = 65536 // (2 * D)                              # lanes that fill the scan per channel
    few = np.full(many // 4, 4 * 48, dtype=np.uint64)
    region = boa.workspace_size(m, np.full(many, 48, dtype=np.uint64), "encode", dtype=dtype)
    full = boa.workspace_size(m, few, "encode", dtype=dtype)
    assert region < full
    data = torch.from_numpy(records_f32_mix(int(few.sum()), D)).cuda()
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    ref = _payloads(m, data, few, dtype)
    for size in (full, full - 1, region):
        print(f"[gpu] encode d{D} {dtype} in {size} of {full} bytes", flush=True)
        assert _payloads(m, data, few, dtype, workspace=ws[:size]) == ref
    assert _payloads(m, data, few, dtype, workspace=ws[:region], tile_t=64) == ref
    with pytest.raises(boa.BoaError) as e:
        boa.encode_dev(m, data, few, dtype=dtype, ideal=False, workspace=ws[:full // 5])
    assert e.value.name == "BOA_E_ARG"
