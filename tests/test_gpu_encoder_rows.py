"""The encoder's tables do not depend on which kernels a tile's shape selects:
one row per launch, the scan over states and blocks of rows (few lanes), the
scan per channel (many lanes), column-tiled and row-block products with 16 rows
a workgroup or more, ragged last tiles, chunks that start inside a tile and
lanes that end early.  The payloads have to be equal byte for byte."""
import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16", "fp8"])
@pytest.mark.parametrize("D,lanes", [(64, 600), (128, 300), (256, 150), (512, 80)])
def test_payloads_do_not_depend_on_the_kernels(D, lanes, dtype):
    import paper_2511_11337_amd as boa
    cfg = ModelConfig(D, 2)
    m = boa.Model(cfg, init_weights(cfg, 31 + D))
    rng = np.random.default_rng(D)
    lens = rng.integers(1, 140, lanes).astype(np.uint64)
    lens[:5] = (1, 2, 3, 17, 300)
    data = records_f32_mix(int(lens.sum()), D)
    d = torch.from_numpy(data).cuda()
    ref = None
    # (lanes, tile): few lanes at tiles around the blocks of 16 rows and stages of 64; all lanes, rows
    # around 2048 and 16 x 256; a row at a time
    for max_lanes, tile in [(3, 16), (3, 63), (3, 65), (7, 130), (40, 64), (0, 3), (0, 17), (0, 64), (0, 256), (5, 1)]:
        print(f"[gpu] encoder rows d{D} {dtype} max_lanes={max_lanes} tile={tile}", flush=True)
        if tile == 1 and D == 512:
            continue
        pay, off, plen, _ = boa.encode_dev(m, d, lens, dtype=dtype, max_lanes=max_lanes, tile_t=tile, ideal=False)
        plen = plen.cpu().numpy().astype(np.uint32)
        pay = pay.cpu().numpy()
        got = [pay[int(o):int(o) + int(n)].tobytes() for o, n in zip(off, plen)]
        if ref is None:
            ref = got
        assert got == ref, (max_lanes, tile)
