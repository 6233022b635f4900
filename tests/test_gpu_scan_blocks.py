"""The time-blocked selective scan at the sizes where its cuts can go wrong:
one step, a partial last block, chunk lengths that are and are not multiples
of the sub-block, states so far apart that the call makes its own, and both
state splits (one and four states per thread), against the FP64 oracle.

Tolerance: float32 sums of T terms in any order are within T 2^-24 of the sum
of magnitudes, on top of the 1e-5 of a tensor's scale and 1e-4 relative that
the elementwise operations (hardware exp2) are held to elsewhere."""
import numpy as np
import pytest
import torch

from oracle.grad import scan_forward, scan_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bt,T,Di,chunk_t", [
    (1, 1, 64, 256), (2, 64, 72, 8), (2, 65, 72, 12), (1, 300, 128, 257), (2, 330, 64, 32), (2, 41, 1024, 5),
    (16, 70, 1024, 64)])
def test_scan_blocks_match_oracle(Bt, T, Di, chunk_t):
    import paper_2511_11337_amd.train as tr
    print(f"[gpu] scan blocks B={Bt} T={T} Di={Di} chunk_t={chunk_t}", flush=True)
    rng = np.random.default_rng(T + chunk_t)
    N = 16
    x = rng.normal(size=(Bt, T, Di))
    dt = np.exp(rng.normal(-1.5, 0.5, (Bt, T, Di)))
    A_log = rng.normal(0, 0.5, (Di, N))
    Bm, Cm = rng.normal(size=(Bt, T, N)), rng.normal(size=(Bt, T, N))
    Dv = rng.normal(size=Di)
    dy = rng.normal(size=(Bt, T, Di))
    A = -np.exp(A_log)
    y_ref, saved = scan_forward(x, dt, A, Bm, Cm, Dv, save_every=chunk_t)
    gx, gdt, gA, gB, gC, gD = scan_backward(dy, x, dt, A, Bm, Cm, Dv, saved, chunk_t)
    leaves = [torch.tensor(a, dtype=torch.float32, device="cuda", requires_grad=True) for a in (x, dt, A_log, Bm, Cm, Dv)]
    y = tr.selective_scan(*leaves, chunk_t=chunk_t)
    y.backward(torch.tensor(dy, dtype=torch.float32, device="cuda"))
    got = [y] + [t.grad for t in leaves]
    for what, a, b in zip(("y", "dx", "ddt", "dA_log", "dB", "dC", "dD"), got, (y_ref, gx, gdt, gA * A, gB, gC, gD)):
        a = a.detach().cpu().numpy().astype(np.float64)
        atol = (1e-5 + T * 2.0 ** -24) * np.abs(b).max()
        err = np.abs(a - b)
        assert (err <= atol + 1e-4 * np.abs(b)).all(), (what, float(err.max()), atol)
