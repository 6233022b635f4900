"""The encoder mixer's form (blocks of rows, or the scan per channel) by lanes and
rows: where each is taken, seen in the workspace, and equal payloads from both."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _model(D):
    import paper_2511_11337_amd as boa
    from synth import ModelConfig, init_weights
    cfg = ModelConfig(d_model=D, n_layers=2)
    return boa, boa.Model(cfg, init_weights(cfg, 4200 + D))


@pytest.mark.parametrize("D,lanes,short,long", [(64, 6, 34, 38), (64, 128, 66, 70), (128, 16, 40, 44), (256, 1, 46, 50),
                                                (512, 4, 64, 68)])
def test_rows_from_the_shortest_tile_that_pays(D, lanes, short, long):
    """Blocks of rows keep the conv output, Delta and states: 12 d_inner bytes a row."""
    boa, m = _model(D)

    def size(rows):
        return boa.workspace_size(m, np.full(lanes, rows + 1, dtype=np.uint64), "encode", dtype="bf16", tile_t=rows)

    per_row = lambda a, b: (size(b) - size(a)) / lanes / (b - a)
    plain = per_row(short - 8, short)
    assert size(long) - size(short) > (long - short) * lanes * plain + 0.8 * lanes * long * 10 * 2 * D


@pytest.mark.parametrize("D,lanes,rows", [(64, 128, 130), (128, 64, 128), (512, 16, 190)])
def test_own_allocation_and_workspace_give_equal_payloads(D, lanes, rows):
    """Past 64 MiB a call that allocates for itself takes the scan per channel."""
    from synth import records_f32_mix
    boa, m = _model(D)
    lens = np.full(lanes, rows + 1, dtype=np.uint64)
    d = torch.from_numpy(records_f32_mix(int(lens.sum()), D)).cuda()
    n = boa.workspace_size(m, lens, "encode", dtype="bf16", tile_t=rows)
    assert n > 64 << 20
    w = torch.empty(n, dtype=torch.uint8, device="cuda")
    a = boa.encode_dev(m, d, lens, dtype="bf16", tile_t=rows, ideal=False, max_lanes=lanes)
    b = boa.encode_dev(m, d, lens, dtype="bf16", tile_t=rows, ideal=False, max_lanes=lanes, workspace=w)
    la, lb = (x[2].cpu().numpy() for x in (a, b))
    assert np.array_equal(la, lb)
    pa, pb = a[0].cpu().numpy(), b[0].cpu().numpy()
    for i in range(lanes):
        assert np.array_equal(pa[int(a[1][i]):][:int(la[i])], pb[int(b[1][i]):][:int(lb[i])])
