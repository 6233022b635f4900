"""The tuned launch-shape table shipped with the package: every entry is a
shape the library accepts, keyed as the autotuner keys its sweeps."""
import json
import re
from types import SimpleNamespace

import pytest

from paper_2511_11337_amd import autotune


def test_tuned_table_entries_are_valid_shapes():
    with open(autotune.TABLE) as fh:
        table = json.load(fh)
    assert table
    for key, shape in table.items():
        m = re.fullmatch(r"v3\|gfx\d+x\d+\|d(\d+)\|l(\d+)\|(f32|bf16|fp8)\|lanes(\d+)", key)
        assert m, key
        lanes = int(m.group(4))
        assert lanes & (lanes - 1) == 0, key                     # lane counts are rounded up to powers of two
        assert shape["tile_t"] in autotune.TILES, key
        assert shape["decode_kernel"] in ("fused", "steps"), key
        if shape["decode_kernel"] == "fused":
            assert shape["fused_lanes"] in autotune.FUSED_LANES, key
        assert isinstance(shape["use_graph"], bool), key


class _Swept(Exception):
    pass


class _Data:
    @property
    def is_cuda(self):                                           # the first thing a sweep asks of its data
        raise _Swept


class _Asked(dict):
    """A cache that holds nothing and records what it was asked for."""

    def __init__(self):
        self.keys_asked = []

    def __contains__(self, key):
        self.keys_asked.append(key)
        return False


def test_cached_shapes_are_for_one_library_and_one_lane_count(tmp_path, monkeypatch):
    import torch
    from paper_2511_11337_amd import _lib
    dev = SimpleNamespace(name="card", gcnArchName="gfx950:sramecc+", multi_processor_count=256)
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda i: dev)
    asked = _Asked()
    monkeypatch.setattr(autotune, "_load", lambda path=None: {} if path else asked)
    model = SimpleNamespace(cfg=SimpleNamespace(d_model=256, n_layers=3))

    def key(lens):
        with pytest.raises(_Swept):
            autotune.tune(model, _Data(), lens, dtype="bf16")
        return asked.keys_asked[-1]

    a = key([4096] * 300)
    assert key([4096] * 300) == a
    assert key([4096] * 512) != a                                # one rounded-up count, other decoder shapes
    _lib.load()
    other = tmp_path / "libboa.so"
    other.write_bytes(b"another build")
    monkeypatch.setattr(_lib, "LIB_PATH", str(other))
    assert key([4096] * 300) != a


def test_table_lanes_are_for_the_entrys_own_count(monkeypatch):
    import torch
    dev = SimpleNamespace(name="card", gcnArchName="gfx950", multi_processor_count=256)
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda i: dev)
    model = SimpleNamespace(cfg=SimpleNamespace(d_model=256, n_layers=3))
    entry = autotune._load(autotune.TABLE)["v3|gfx950x256|d256|l3|bf16|lanes8192"]
    assert autotune.tune(model, _Data(), [4096] * 8192, dtype="bf16") == entry
    # 5000 lanes in workgroups of 16 leave most of a second round of the chip empty
    assert autotune.tune(model, _Data(), [4096] * 5000, dtype="bf16") == {**entry, "fused_lanes": 0}
