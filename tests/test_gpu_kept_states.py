"""chunk_t of a training call: from four layers on it trades the memory of the
kept scan states for making them again, without changing a bit of the gradient."""
import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu


def _model(D, L):
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(D, L)
    return boa.Model(cfg, init_weights(cfg, 17))


def _tokens(B, T):
    return torch.from_numpy(records_f32_mix(B * T, 23).reshape(B, T)).cuda()


@pytest.mark.parametrize("D,L,B,T,dtype", [(64, 4, 3, 130, "f32"), (64, 5, 2, 601, "bf16"), (128, 4, 2, 257, "f32")])
def test_gradient_does_not_depend_on_chunk_t(D, L, B, T, dtype):
    from paper_2511_11337_amd import train
    m, tok = _model(D, L), _tokens(B, T)
    ref = None
    for chunk_t in (8, 1, 12, 64, 128, 256, 100000):
        print(f"[gpu] kept states d{D} x {L} {dtype} chunk_t={chunk_t}", flush=True)
        loss, grad = train.loss_and_grad(m, tok, chunk_t=chunk_t, dtype=dtype)
        if ref is None:
            ref = loss, grad
        assert loss == ref[0] and torch.equal(grad, ref[1]), chunk_t


def test_chunk_t_bounds_the_memory():
    from paper_2511_11337_amd import train
    D, L, B, T = 256, 8, 8, 2049
    tok = _tokens(B, T)
    used = {}
    for chunk_t in (8, 256):
        m = _model(D, L)
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        before = torch.cuda.mem_get_info()[0]
        print(f"[gpu] training memory at chunk_t={chunk_t}", flush=True)
        train.loss_and_grad(m, tok, chunk_t=chunk_t, dtype="bf16")
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        used[chunk_t] = before - torch.cuda.mem_get_info()[0]
        m.close()
    unit = B * (T - 1) * 2 * D * 4                       # one d_inner float a row: 2 a layer kept, L + 3 at most
    assert used[8] - used[256] > 0.8 * (2 * L - (L + 3)) * unit
