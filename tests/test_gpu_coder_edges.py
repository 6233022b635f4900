"""The encoder's coder and the chunk CRC at the edges of their batches: payloads
do not depend on how the rows are tiled, on the lanes a wave holds (one, or up
to sixteen from 512 lanes on) or on the chunks a lane runs one after another,
and the stored CRC is zlib's for every remainder of the pieces a wave takes.
Exact comparisons throughout."""
import struct
import zlib

import numpy as np
import pytest
import torch

from synth import ModelConfig, init_weights, records_f32_mix

pytestmark = pytest.mark.gpu
CFG = ModelConfig(64, 2)


@pytest.fixture(scope="module")
def model():
    import paper_2511_11337_amd as boa
    return boa.Model(CFG, init_weights(CFG, 21))


def _payloads(m, data, lens, **kw):
    import paper_2511_11337_amd as boa
    pay, off, plen, ideal = boa.encode_dev(m, torch.from_numpy(data).cuda(), lens, **kw)
    plen = plen.cpu().numpy().astype(np.uint32)
    pay = pay.cpu().numpy()
    return [pay[int(o):int(o) + int(n)].tobytes() for o, n in zip(off, plen)], ideal.cpu().numpy()


@pytest.mark.parametrize("lanes,tile", [(1, 63), (1, 64), (1, 65), (3, 7), (511, 32), (512, 31), (512, 33),
                                        (1030, 32), (4100, 64)])
def test_payloads_do_not_depend_on_lanes_or_tiles(model, lanes, tile):
    print(f"[gpu] coder edges lanes={lanes} tile={tile}", flush=True)
    rng = np.random.default_rng(lanes + tile)
    n = max(lanes, 9)
    lens = rng.integers(1, 70 if lanes > 3 else 300, n).astype(np.uint64)
    lens[:4] = (1, 2, 3, 65)
    data = records_f32_mix(int(lens.sum()), lanes)
    got, gi = _payloads(model, data, lens, max_lanes=lanes, tile_t=tile)
    ref, ri = _payloads(model, data, lens, max_lanes=200, tile_t=128)
    assert got == ref
    assert np.array_equal(gi, ri)


def test_crc_of_every_remainder(model):
    import paper_2511_11337_amd as boa
    print("[gpu] chunk CRCs", flush=True)
    lens = np.array([1, 2, 3, 4, 5, 63, 64, 65, 127, 255, 256, 257, 259, 1000, 2047, 2049, 4099, 8195], dtype=np.uint64)
    data = records_f32_mix(int(lens.sum()), 8)
    blob = boa.compress(model, data, chunk_lens=lens)
    off = 0
    for i, n in enumerate(lens):
        length, _, _, crc, _, _ = struct.unpack_from("<QQIIBB", blob, 64 + 32 * i)
        assert length == n
        assert crc == zlib.crc32(data[off:off + int(n)].tobytes()), int(n)
        off += int(n)
    assert boa.decompress(model, blob) == data.tobytes()
