"""The integer pipeline's word-sized arithmetic where it can go wrong: states and
activations at their saturation limits, decays from none to underflow and near
constant rows, against the integer oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import intpipe as ip
from synth import ModelConfig, init_weights, param_layout, records_f32_mix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale,decay,d_model", [(40.0, 4.0, 64), (6.0, -6.0, 64), (1e-4, 0.0, 64), (12.0, 8.0, 128)])
def test_tables_at_the_limits(scale, decay, d_model):
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(d_model, 2)
    w = init_weights(cfg, 77).copy()
    at = 0
    for name, shape in param_layout(cfg):
        n = int(np.prod(shape))
        if name.endswith("A_log"):
            w[at:at + n] += decay
        elif not name.endswith("norm_w"):
            w[at:at + n] *= scale
        at += n
    seqs = np.stack([records_f32_mix(48, 3), np.zeros(48, dtype=np.uint8)])
    print(f"[gpu] integer ranges scale={scale} decay={decay} d{d_model}", flush=True)
    q = boa.QModel(boa.Model(cfg, w))
    tb, lg = boa.int_tables(q, torch.from_numpy(seqs).cuda())
    ref_l, ref_t = ip.stream_tables(ip.convert(cfg, w), seqs)
    assert np.array_equal(tb.cpu().numpy().view(np.uint16).astype(np.int64), ref_t)
    assert np.array_equal(lg.cpu().numpy().astype(np.int64), ref_l)
