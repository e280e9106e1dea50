"""Products whose launches take another tile shape (few rows, narrow outputs).

A row of ReLU(h G1^T + g) has the same bits whatever the number of rows beside it,
i.e. whichever tile shape the row count selects, and the row-norm layers of few rows
agree with 64 bits: per element (K + 8) 2^-24 of the summed magnitudes before the norm
in fp32; bf16 storage adds half a unit in the last place (2^-9) of each rounded value.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d,hidden", [(48, 64), (96, 176), (256, 320)])
def test_row_bits_do_not_depend_on_the_tile_shape(dtype, d, hidden):
    import paper_1806_01973_amd as ps
    print(f"[case] tile shapes {dtype} {d} -> {hidden}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(d)
    mlp = ps.DeviceMLP(torch.randn((hidden, d), generator=gen) * d ** -0.5,
                       torch.randn(hidden, generator=gen), torch.eye(hidden), dtype=dt)
    h = torch.randn((70001, d), generator=gen).to(dt).cuda()
    full = ps.output_mlp(mlp, h)
    for rows in (1, 63, 65, 8191, 16384, 33000):
        assert torch.equal(ps.output_mlp(mlp, h[:rows]), full[:rows]), rows


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,d,m,dout", [(1, 16, 16, 16), (33, 64, 48, 64), (200, 80, 96, 80),
                                           (999, 96, 64, 256), (257, 48, 32, 272), (70, 64, 64, 512)])
def test_row_norm_layers_of_few_rows(dtype, rows, d, m, dout):
    import paper_1806_01973_amd as ps
    print(f"[case] few rows {dtype} {rows} x {d}/{m}/{dout}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(rows)
    W = torch.randn((dout, d + m), generator=gen) * (d + m) ** -0.5
    w = torch.rand(dout, generator=gen) * 0.2
    layer = ps.DeviceLayer(torch.zeros((m, d)), torch.ones(m), W, w, dtype=dt)
    h = torch.randn((rows, d), generator=gen).to(dt).cuda()
    nbr = ps.Neighborhoods.empty(rows, 1)  # one neighbour each: the pooled row is all ones
    nbr.idx.zero_(), nbr.counts.fill_(1), nbr.weights.fill_(1.0)
    out = ps.convolve_layer(layer, h, 1, nbr).double().cpu()
    Wd, wd = layer.W.double().cpu(), layer.w.double().cpu()
    x = torch.cat([h.double().cpu(), torch.ones((rows, m), dtype=torch.float64)], 1)
    z = torch.relu(x @ Wd.t() + wd)
    norm = z.norm(dim=1, keepdim=True)
    bound = (d + m + 8) * 2.0 ** -24 * (x.abs() @ Wd.abs().t() + wd.abs())
    # The norm moves by at most the bound's own norm; the sum of dout squares rounds too.
    ref = z / norm
    tol = (bound + ref * bound.norm(dim=1, keepdim=True)) / norm + ref * (dout + 8) * 2.0 ** -24
    if dtype == "bf16":
        tol = tol + ref * 2.0 ** -8
    assert ((out - ref).abs() <= tol).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("dataflow", ["pool_then_dense", "dense_then_pool"])
@pytest.mark.parametrize("d,m,dout", [(64, 48, 64), (96, 64, 128), (288, 336, 176), (160, 512, 256),
                                      (256, 64, 512)])
def test_layer_row_bits_do_not_depend_on_the_row_count(dtype, dataflow, d, m, dout):
    """A layer's rows, behind row maps on both sides and with one neighbour each, have the
    same bits whatever the number of rows beside them: transform, neighbour half and
    row-norm product change tile shapes in between (8,192, 16,384 and 32,768 rows, and
    below one large tile per CU), and with them the K sweep's start in bf16."""
    import paper_1806_01973_amd as ps
    print(f"[case] layer row bits {dtype} {dataflow} {d}/{m}/{dout}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(d + m)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    layer = ps.DeviceLayer(rnd(m, d) * d ** -0.5, rnd(m) * 0.1, rnd(dout, d + m) * (d + m) ** -0.5,
                           rnd(dout) * 0.1, dtype=dt, dataflow=dataflow)
    N = 70_001
    h = rnd(N, d).to(dt)
    nbr = ps.Neighborhoods.empty(N, 1)
    nbr.idx.copy_(torch.arange(N)[:, None])
    nbr.counts.fill_(1), nbr.weights.fill_(1.0)
    maps = [torch.randperm(N, generator=g, device="cuda").to(torch.int32) for _ in range(2)]

    def rows(k):
        part = ps.Neighborhoods(nbr.idx[:k], nbr.counts[:k], nbr.weights[:k])
        return ps.convolve_layer(layer, h, k, part, self_rows=maps[0][:k], transform_rows=maps[1][:k])

    full = rows(N)
    for k in (1, 500, 8192, 8193, 12_788, 16_384, 16_385, 32_000, 33_000, 60_000):
        assert torch.equal(rows(k), full[:k]), k
