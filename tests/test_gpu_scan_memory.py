"""The backward scan's scratch memory: at most one chunk's states of every
sequence and the partial sums of every row (or 256 MiB), by taking sequences and
chunks a part at a time, with the same gradients."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(Bt, T, Di, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return rnd(Bt, T, Di), rnd(Bt, T, Di).abs() * 0.1, rnd(Di, 16) * 0.3, rnd(Bt, T, 32), rnd(Di), rnd(Bt, T, Di)


def _grads(ins, chunk_t):
    """dx, ddt, dbc, dA_log, dD by the library's entry points (every tensor allocated before the backward call)."""
    from paper_2511_11337_amd import _lib
    x, dt, A, bc, D, dy = ins
    Bt, T, Di = x.shape
    s = torch.cuda.current_stream().cuda_stream
    y = torch.empty_like(x)
    hs = torch.empty((Bt, -(-T // chunk_t), 16, Di), device="cuda")
    _lib.check(_lib.load().boa_scan_fwd_dev(x.data_ptr(), dt.data_ptr(), A.data_ptr(), bc.data_ptr(), D.data_ptr(), Bt, T, Di,
                                            chunk_t, y.data_ptr(), hs.data_ptr(), s))
    out = torch.empty_like(x), torch.empty_like(x), torch.empty_like(bc), torch.zeros_like(A), torch.zeros_like(D)

    def backward():
        _lib.check(_lib.load().boa_scan_bwd_dev(x.data_ptr(), dt.data_ptr(), A.data_ptr(), bc.data_ptr(), D.data_ptr(),
                                                dy.data_ptr(), Bt, T, Di, chunk_t, hs.data_ptr(),
                                                *(t.data_ptr() for t in out), s))
        return out
    return backward


@pytest.mark.parametrize("Bt,T,Di,chunk_t,whole_t", [
    (6, 6001, 1024, 64, 6001),          # groups of sequences
    (1, 40003, 1024, 64, 40003),        # chunks of one sequence at a time
    (1, 40003, 1024, 100, 40003),       # the same, chunk ends off the groups of eight steps
    (3, 500, 128, 1, 500), (2, 700, 72, 7, 700), (2, 1000, 64, 63, 1000)])   # short chunks taken together
def test_parts_give_the_same_gradients(Bt, T, Di, chunk_t, whole_t):
    print(f"[gpu] scan parts B={Bt} T={T} Di={Di} chunk_t={chunk_t}", flush=True)
    ins = _inputs(Bt, T, Di, T)
    got = _grads(ins, chunk_t)()
    ref = _grads(ins, whole_t)()
    for a, b in zip(got[:3], ref[:3]):                   # chained values: the same operations in the same order
        assert torch.equal(a, b)
    for a, b in zip(got[3:], ref[3:]):                   # sums over time and sequences: grouped by part
        mag = b.abs().max().item()
        assert (a - b).abs().max().item() <= 2 * Bt * T * 2.0 ** -24 * max(mag, 1.0)


def test_scratch_stays_within_a_chunk_of_states():
    Bt, T, Di, chunk_t = 32, 4096, 512, 256
    ins = _inputs(Bt, T, Di, 1)
    backward = _grads(ins, chunk_t)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    bound = 4 * (Bt * chunk_t * 16 * Di + Di // 64 * Bt * T * 32)
    free = torch.cuda.mem_get_info()[0]
    print(f"[gpu] scan backward with {bound * 5 // 4 >> 20} MiB free", flush=True)
    hold = torch.empty(free - bound * 5 // 4, dtype=torch.uint8, device="cuda")
    try:
        out = backward()
    finally:
        del hold
        torch.cuda.empty_cache()
    assert all(torch.isfinite(t).all() for t in out)
