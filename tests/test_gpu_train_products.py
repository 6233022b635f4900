"""Training products at the sizes where their launch shapes change: enough rows
for the 64-row workgroups with a ragged last one, few rows with the reduction
in spans, d_model 512 (a reduction of 2048), and a feed-forward width no row
product is built for.  Gradients against the FP64 oracle, held to the bounds of
the model gradient tests: FP32 2e-3 relative + 2e-4 of the tensor's largest
magnitude; BF16 operands 3e-2 and 3e-2 (three products of operands rounded to
2^-9)."""
import numpy as np
import pytest
import torch

from oracle.grad import loss_and_grad as oracle_loss_grad
from synth import ModelConfig, init_weights, records_f32_mix
from synth.weights import param_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,n_layers,ffn_mult,B,T,dtype", [
    (64, 1, 0, 65, 254, "f32"), (64, 1, 0, 65, 254, "bf16"), (128, 1, 0, 3, 60, "bf16"), (512, 1, 0, 1, 9, "f32"),
    (512, 1, 0, 1, 9, "bf16"), (64, 1, 3, 2, 33, "f32")])
def test_gradients_at_launch_shape_edges(d_model, n_layers, ffn_mult, B, T, dtype):
    import paper_2511_11337_amd as boa
    import paper_2511_11337_amd.train as tr
    print(f"[gpu] gradient d_model={d_model} ffn={ffn_mult} {B}x{T} {dtype}", flush=True)
    cfg = ModelConfig(d_model=d_model, n_layers=n_layers, ffn_mult=ffn_mult)
    flat = init_weights(cfg, 17)
    flat = (flat + np.random.default_rng(3).normal(0, 0.02, flat.size)).astype(np.float32)
    seqs = np.stack([records_f32_mix(T, 900 + b) for b in range(B)])
    loss, grad = tr.loss_and_grad(boa.Model(cfg, flat), torch.from_numpy(seqs).cuda(), chunk_t=64, dtype=dtype)
    ref_loss, ref = oracle_loss_grad(cfg, flat, seqs, Tc=64)
    rtol, frac = (2e-3, 2e-4) if dtype == "f32" else (3e-2, 3e-2)
    assert abs(loss - ref_loss) <= (1e-5 if dtype == "f32" else 1e-3) * abs(ref_loss)
    g, at = grad.cpu().numpy().astype(np.float64), 0
    for name, shape in param_layout(cfg):
        n = int(np.prod(shape))
        a, b = g[at:at + n], ref[at:at + n]
        at += n
        err = np.abs(a - b)
        assert (err <= frac * np.abs(b).max() + rtol * np.abs(b)).all(), (name, float(err.max()), float(np.abs(b).max()))
