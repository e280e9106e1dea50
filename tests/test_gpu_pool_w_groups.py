"""The fused pool and W at row counts where a wave takes fewer than 32 rows per turn
(1 and 3 rows, several turns, a ragged last group): the rows' bits are those of the
same rows in a larger call."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pool", ["importance", "mean"])
def test_bits_do_not_depend_on_the_row_count(pool):
    import paper_1806_01973_amd as ps
    g = torch.Generator(device="cuda").manual_seed(4)
    n, T, rows = 5000, 50, 140_001
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda") * 0.06
    layer = ps.DeviceLayer(rnd(512, 256), rnd(512), rnd(256, 768), rnd(256), dtype=torch.bfloat16,
                           dataflow="dense_then_pool", pool=pool)
    h = torch.randn((rows, 256), generator=g, device="cuda").bfloat16()
    nbr = ps.Neighborhoods.empty(rows, T)
    nbr.idx.copy_(torch.randint(-1, n, (rows, T), generator=g, device="cuda"))
    nbr.counts.fill_(1), nbr.weights.fill_(1.0 / T)
    full = ps.convolve_layer(layer, h, n, nbr)
    for k in (1, 33, 2048, 2049, 6143, 65_536, 70_001, 131_073):
        print(f"[case] pool and W {pool} rows={k}", flush=True)
        part = ps.Neighborhoods(nbr.idx[:k], nbr.counts[:k], nbr.weights[:k])
        assert torch.equal(ps.convolve_layer(layer, h, n, part), full[:k])
