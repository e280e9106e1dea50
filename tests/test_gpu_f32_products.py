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
