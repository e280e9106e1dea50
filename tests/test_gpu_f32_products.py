"""fp32 products on the bf16 matrix cores (operands split into bf16 triples).

z = G2 ReLU(G1 h + g) with G2 the identity leaves the first product as it is
(x * 1 splits and sums back exactly), so output_mlp shows it element by element.
Bound per element against 64 bits: K products of exactly split operands, at most
K fp32 roundings each of 2^-24 of the running sum of magnitudes, and the left-out
parts' 3 * 2^-25: (K + 8) 2^-24 (|h| |G1|^T + |g|).
"""

import pytest
import torch

pytestmark = pytest.mark.gpu


def _mlp(rows, d, hidden, seed):
    import paper_1806_01973_amd as ps
    g = torch.Generator().manual_seed(seed)
    G1 = torch.randn((hidden, d), generator=g) * d ** -0.5
    bias = torch.randn(hidden, generator=g) * 0.1
    h = torch.randn((rows, d), generator=g)
    return ps.DeviceMLP(G1, bias, torch.eye(hidden)), h


def _check(z, mlp, h):
    G1, g = mlp.G1.double().cpu(), mlp.g.double().cpu()
    ref = torch.relu(h.double() @ G1.t() + g)
    bound = (h.shape[1] + 8) * 2.0 ** -24 * (h.double().abs() @ G1.abs().t() + g.abs())
    bad = (z.double().cpu() - ref).abs() > bound
    assert not bad.any(), f"{int(bad.sum())} of {bad.numel()} outside the bound"


# Tile edges (128 rows, 128 columns, chunks of 16), one chunk, odd chunk counts, and the
# row count from which the weights are split once (16,384).
@pytest.mark.parametrize("rows,d,hidden", [
    (1, 16, 16), (31, 32, 48), (127, 48, 128), (129, 272, 144), (16383, 64, 64),
    (16384, 16, 16), (16385, 80, 272), (20001, 256, 512),
])
def test_products_within_the_fp32_bound(rows, d, hidden):
    import paper_1806_01973_amd as ps
    print(f"[case] f32 product {rows} x {d} -> {hidden}", flush=True)
    mlp, h = _mlp(rows, d, hidden, rows + d)
    _check(ps.output_mlp(mlp, h.cuda()), mlp, h)


def test_same_bits_without_room_for_the_split_weights():
    import paper_1806_01973_amd as ps
    rows, d, hidden = 17000, 96, 160
    mlp, h = _mlp(rows, d, hidden, 3)
    h = h.cuda()
    base = (rows * hidden * 4 + 255) // 256 * 256  # the hidden rows alone
    small = torch.empty(base, dtype=torch.uint8, device="cuda")
    assert torch.equal(ps.output_mlp(mlp, h), ps.output_mlp(mlp, h, workspace=small))


def _transform(mlp, h):
    """ReLU(h G1^T + g) as a layer's projected rows: with no output rows the call stops
    there, and they are the first region of its workspace."""
    import paper_1806_01973_amd as ps
    m, d = mlp.G1.shape
    layer = ps.DeviceLayer(mlp.G1, mlp.g, torch.zeros((16, d + m)), torch.zeros(16))
    ws = torch.empty(ps.convolve_workspace_size(layer, len(h), 0), dtype=torch.uint8, device="cuda")
    ps.convolve_layer(layer, h.cuda(), len(h), ps.Neighborhoods.empty(0, 1), workspace=ws)
    return ws[:len(h) * m * 4].view(torch.float32).view(len(h), m).cpu()


@pytest.mark.parametrize("rows", [300, 16500])
def test_infinities_nan_and_extreme_magnitudes(rows):
    import paper_1806_01973_amd as ps
    mlp, h = _mlp(rows, 64, 96, 9)
    h[3, 5] = float("inf")
    h[7, 1] = -float("inf")
    h[11, 2] = float("nan")
    h[40] *= 1e38 / h[40].abs().max()
    h[40, 0] = 3.4e38  # rounds to infinity in bf16
    h[131] *= 1e-36
    h[132] = 0.0
    z = _transform(mlp, h)
    for r in (3, 7):  # +-infinity by the sign of the weight, then ReLU
        ref = torch.relu(h[r].double() @ mlp.G1.double().cpu().t() + mlp.g.double().cpu())
        assert torch.equal(z[r].double(), ref)
    assert not z[11].any()  # ReLU of NaN is 0
    ok = torch.tensor([r for r in range(rows) if r not in (3, 7, 11)])
    _check(z[ok], mlp, h[ok])
    # Without the bias the tiny row's own digits show.
    tiny = ps.DeviceMLP(mlp.G1, torch.zeros(96), torch.eye(96))
    _check(_transform(tiny, h[100:200]), tiny, h[100:200])


# Operands at the ends of the range, which bf16 parts do not hold: 2^-130 beside ordinary
# values, 2^-125 * 2^110, 2^-140 * 2^120, 1e-36 * 1e20, one tiny weight row beside others.
# Per element (K + 8) 2^-24 of the summed magnitudes and K roundings at fp32's last place.
def _odd(rows, d, hidden, seed):
    g = torch.Generator().manual_seed(seed)
    h = torch.randn((rows, d), generator=g)
    G1 = torch.randn((hidden, d), generator=g) * d ** -0.5
    G1[0] = 0.0
    G1[0, 0] = 1.0               # picks h[:, 0] alone
    G1[1] = 0.0
    G1[1, 1] = 2.0 ** 110
    G1[2] = 0.0
    G1[2, 2] = 2.0 ** 120
    G1[3] = 0.0
    G1[3, 3] = 1e20
    G1[4] *= 2.0 ** -118
    h[5, 0] = 1.2345 * 2.0 ** -130
    h[6, 1] = 1.2345 * 2.0 ** -125
    h[7, 2] = 1.2345 * 2.0 ** -140
    h[rows - 1, 3] = 1.2345e-36
    h[8] *= 2.0 ** 100           # beside the tiny weight row
    h[8, 1:4] = 0.0              # (2^210 is beyond fp32)
    return h, G1


def _check_odd(z, h, G1):
    K = h.shape[1]
    ref = torch.relu(h.double() @ G1.double().t())
    bound = (K + 8) * (2.0 ** -24 * (h.double().abs() @ G1.double().abs().t()) + 2.0 ** -149)
    bad = (z.double() - ref).abs() > bound
    assert not bad.any(), (int(bad.sum()), torch.nonzero(bad)[:8].tolist())


# (Weights are split beforehand from 3 G multiply-adds on.)
@pytest.mark.parametrize("rows,d,hidden", [(300, 64, 96), (300, 272, 16), (16500, 64, 96),
                                           (16500, 80, 272), (70_001, 272, 176)])
def test_operands_at_the_ends_of_the_range(rows, d, hidden):
    import paper_1806_01973_amd as ps
    print(f"[case] ends of the range {rows} x {d} -> {hidden}", flush=True)
    h, G1 = _odd(rows, d, hidden, rows + d)
    _check_odd(_transform(ps.DeviceMLP(G1, torch.zeros(hidden), torch.eye(hidden)), h), h, G1)


def test_a_lone_product_is_rounded_once():
    # Diagonal weights: fp32 rounds each product once, so half a unit in the last place
    # (2^-24 of it); the parts' sums add below 2^-31.
    import paper_1806_01973_amd as ps
    for rows in (4000, 20000):
        g = torch.Generator().manual_seed(rows)
        diag = (1.0 + torch.rand(64, generator=g)) * 2.0 ** torch.randint(-9, 9, (64,), generator=g)
        h = torch.randn((rows, 64), generator=g).abs()
        z = _transform(ps.DeviceMLP(torch.diag(diag), torch.zeros(64), torch.eye(64)), h)
        ref = h.double() * diag.double()
        assert float(((z.double() - ref).abs() / ref).max()) <= 2.0 ** -24 * (1 + 2.0 ** -6)


def _norm_layer(h, x, W, self_rows, m):
    """A layer whose pooled rows n are x's (x >= 0: one neighbour each, Q the identity):
    z / ||z||, z = ReLU(W [h_self | n])."""
    import paper_1806_01973_amd as ps
    layer = ps.DeviceLayer(torch.eye(m), torch.zeros(m), W, torch.zeros(len(W)))
    nbr = ps.Neighborhoods.empty(len(x), 1)
    nbr.idx.copy_(torch.arange(len(x))[:, None])
    nbr.counts.fill_(1), nbr.weights.fill_(1.0)
    rows_in = torch.cat([h, x]).cuda()
    tr = torch.arange(len(h), len(h) + len(x), dtype=torch.int32, device="cuda")
    return ps.convolve_layer(layer, rows_in, len(x), nbr, self_rows=self_rows.cuda(),
                             transform_rows=tr).cpu()


@pytest.mark.parametrize("dout,rows,d", [(dout, rows, 32) for dout in (16, 64, 128, 256, 512)
                                         for rows in (300, 16500)] +
                         [(dout, (3 << 30) // (288 * dout) + 77, 144) for dout in (64, 128, 256, 512)])
def test_row_norm_tiles_with_odd_rows(rows, dout, d):
    """Infinities and tiny values in either source of a row-norm tile, behind a row map;
    the last ones with the weights split beforehand."""
    print(f"[case] row-norm tiles with odd rows {rows} x {d} -> {dout}", flush=True)
    m = d
    g = torch.Generator().manual_seed(rows + dout)
    h, x = torch.randn((rows, d), generator=g), torch.rand((rows, m), generator=g)
    W = torch.randn((dout, d + m), generator=g) * 0.1
    W[2] = 0.0
    W[2, 1], W[2, d + 1] = 2.0 ** 110, 2.0 ** 110
    perm = torch.randperm(rows, generator=g).to(torch.int32)
    # A row whose other columns are small beside the lone large weight's.
    h[:, 1], x[:, 1] = 0.0, 0.0
    h[perm[5], 1] = 1.2345 * 2.0 ** -125      # self half of row 5
    x[9, 1] = 1.2345 * 2.0 ** -125            # pooled half of row 9
    clean = _norm_layer(h, x, W, perm, m)
    a = torch.cat([h[perm.long()], x], 1).double()
    z = torch.relu(a @ W.double().t())
    mag = a.abs() @ W.double().abs().t()
    norm = z.norm(dim=1, keepdim=True)
    bound = (d + m + 8) * 2.0 ** -24 * mag
    tol = (bound + (z / norm) * bound.norm(dim=1, keepdim=True)) / norm + (z / norm) * (dout + 8) * 2.0 ** -24
    live = norm[:, 0] > 0
    assert (((clean.double() - z / norm).abs() <= tol) | ~live[:, None]).all()
    # Odd rows leave the bits of the others alone, whichever half they sit in.
    h2, x2 = h.clone(), x.clone()
    h2[perm[20], 3] = float("inf")
    x2[21, 4] = float("inf")
    h2[perm[22], 7] = float("nan")
    h2[perm[23]] *= 2.0 ** -120
    got = _norm_layer(h2, x2, W, perm, m)
    same = torch.ones(rows, dtype=torch.bool)
    same[20:24] = False
    assert torch.equal(got[same], clean[same])


def test_bits_at_the_ends_of_the_range_do_not_depend_on_the_row_count():
    # Few rows split the weights in their tiles, many beforehand, in other tile shapes.
    import paper_1806_01973_amd as ps
    h, G1 = _odd(70_001, 272, 176, 5)
    mlp = ps.DeviceMLP(G1, torch.zeros(176), torch.eye(176))
    many = _transform(mlp, h)
    for k in (9, 70, 300, 16500):
        assert torch.equal(_transform(mlp, h[:k]), many[:k]), k


@pytest.mark.parametrize("rows,d,hidden", [(20_001, 512, 400), (70_001, 272, 176)])
def test_products_with_weights_split_beforehand(rows, d, hidden):
    """The fp32 bound, and the same bits from a workspace without room for the split
    weights; both of the output layers' products split, and the first alone."""
    import paper_1806_01973_amd as ps
    print(f"[case] split weights {rows} x {d} -> {hidden}", flush=True)
    mlp, h = _mlp(rows, d, hidden, rows)
    z = ps.output_mlp(mlp, h.cuda())
    _check(z, mlp, h)
    small = torch.empty((rows * hidden * 4 + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
    assert torch.equal(ps.output_mlp(mlp, h.cuda(), workspace=small), z)
