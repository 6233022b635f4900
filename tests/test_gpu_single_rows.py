"""d_model 512 a row at a time: the kernels of a one-row tile (also those of the
per-step decoder, and of calls whose chunks have two bytes) build the tables of
the tiled encoder and of the fused decoder, so payloads are equal byte for byte
and every byte comes back."""
import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu


def _model():
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(512, 2)
    return boa.Model(cfg, init_weights(cfg, 543))


def _encode(m, data, lens, dtype, **kw):
    import paper_2511_11337_amd as boa
    pay, off, plen, _ = boa.encode_dev(m, torch.from_numpy(data).cuda(), lens, dtype=dtype, ideal=False, **kw)
    plen = plen.cpu().numpy().astype(np.uint32).astype(np.uint64)
    host = pay.cpu().numpy()
    return pay, off, plen, [host[int(o):int(o) + int(n)].tobytes() for o, n in zip(off, plen)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
def test_one_row_tiles(dtype):
    m = _model()
    rng = np.random.default_rng(6)
    lens = rng.integers(1, 60, 40).astype(np.uint64)
    lens[:4] = (1, 2, 3, 90)
    data = records_f32_mix(int(lens.sum()), 77)
    ref = None
    for max_lanes, tile in [(5, 64), (5, 1), (0, 1), (0, 16)]:
        print(f"[gpu] one-row tiles d512 {dtype} max_lanes={max_lanes} tile={tile}", flush=True)
        got = _encode(m, data, lens, dtype, max_lanes=max_lanes, tile_t=tile)[3]
        ref = got if ref is None else ref
        assert got == ref, (max_lanes, tile)


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("kernel", ["fused", "steps"])
def test_two_byte_chunks(dtype, kernel):
    import paper_2511_11337_amd as boa
    m = _model()
    lens = np.full(70, 2, dtype=np.uint64)
    data = records_f32_mix(140, 5)
    print(f"[gpu] two-byte chunks d512 {dtype} {kernel}", flush=True)
    pay, off, plen, _ = _encode(m, data, lens, dtype)
    out = boa.decode_dev(m, pay, off, plen, data[::2].copy(), lens, dtype=dtype, decode_kernel=kernel)
    assert np.array_equal(out.cpu().numpy(), data)
