"""The pool over column slabs (tables of 48 MB and more, rows of 1 KB and more, 8 GB of
them gathered, deep neighbourhoods that share popular rows) and its turn to whole rows where the probe finds
them short or evenly spread, in layers whose W passes the pooled
rows through: W = [0 | I], so the layer's output is the pooled row, ReLU'd and normalised.

Rows beyond the table's end, 256- and 128-byte slabs, absent and out-of-range slots,
weights given and derived from counts, mean and max. Against 64 bits on sampled rows:
(T + 8) 2^-24 per element of the summed magnitudes (and of the norm's own error), plus the
storage's half unit in the last place (2^-9, twice) in bf16.
"""

import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(dt, n, m, T, rows, pool, weights, short, popular, seed=1):
    import paper_1806_01973_amd as ps
    g = torch.Generator(device="cuda").manual_seed(seed)
    eye = torch.eye(m, device="cuda")
    # P = ReLU(h I + 0) = h for h >= 0; W's self half is zero.
    dout = min(m, 512)  # the widest output; the last columns of wider rows
    W = torch.cat([torch.zeros((dout, m), device="cuda"), eye[m - dout:]], 1)
    layer = ps.DeviceLayer(eye, torch.zeros(m), W, torch.zeros(dout), dtype=dt, pool=pool)
    h = torch.rand((n, m), generator=g, device="cuda").to(dt)
    nbr = ps.Neighborhoods.empty(rows, T, weights)
    idx = torch.randint(0, n, (rows, T), generator=g, device="cuda")
    if popular:  # half of the slots among 500 rows
        hot = torch.randint(0, 500, (rows, T), generator=g, device="cuda")
        idx = torch.where(torch.rand((rows, T), generator=g, device="cuda") < 0.5, hot, idx)
    idx = idx.to(torch.int32)
    live = torch.randint(0, 4 if short else T + 1, (rows, 1), generator=g, device="cuda")
    if not short:
        live[::2] = T  # most rows are full
    pos = torch.arange(T, device="cuda")
    idx[pos >= live] = -1
    idx[7::50, 0] = n + 3  # outside the table: skipped
    nbr.idx.copy_(idx)
    cnt = torch.randint(1, 9, (rows, T), generator=g, device="cuda") * (pos < live)
    nbr.counts.copy_(cnt.to(torch.uint16))
    w = cnt / cnt.sum(1, keepdim=True).clamp(min=1)
    if weights:
        nbr.weights.copy_(w.float())
    out = ps.convolve_layer(layer, h, n, nbr, self_rows=torch.zeros(rows, dtype=torch.int32, device="cuda"))
    pick = torch.cat([torch.arange(40, device="cuda"), torch.arange(rows - 40, rows, device="cuda"),
                      torch.randint(0, rows, (300,), generator=g, device="cuda")])
    i = idx[pick].long()
    ok = (i >= 0) & (i < n)
    x = h[i.clamp(0, n - 1)].double()
    if pool == "max":
        z = torch.where(ok.any(1)[:, None], x.masked_fill(~ok[..., None], -1.0).amax(1), 0.0)
    else:
        a = w[pick].double() if pool == "importance" else ok / ok.sum(1, keepdim=True).clamp(min=1).double()
        z = (x * torch.where(ok, a, 0.0)[..., None]).sum(1)
    z = z[:, m - dout:]
    norm = z.norm(dim=1, keepdim=True)
    ref = torch.where(norm > 0, z / norm, 0.0)
    tol = ref * 2 * (T + m ** 0.5 + 8) * 2.0 ** -24
    if dt == torch.bfloat16:
        tol = tol + ref * 2 * 2.0 ** -8
    assert ((out[pick].double() - ref).abs() <= tol).all()
    return layer, h, nbr, out


@pytest.mark.parametrize("pool", ["importance", "mean", "max"])
@pytest.mark.parametrize("dt,n,m,T,weights,short,popular", [
    (torch.float32, 50_003, 256, 50, True, False, True),    # 51 MB, 256-byte slabs
    (torch.float32, 30_000, 432, 37, False, False, True),   # a last slab that is not whole
    (torch.float32, 530_001, 256, 64, True, False, True),   # 543 MB, 128-byte slabs
    (torch.bfloat16, 60_000, 512, 50, True, False, True),
    (torch.bfloat16, 530_000, 512, 61, False, False, True),
    (torch.float32, 530_000, 256, 50, True, False, False),  # evenly spread: whole rows
    (torch.float32, 60_000, 256, 50, True, True, True),     # short rows: whole rows
    (torch.bfloat16, 60_000, 512, 64, False, True, True),
])
def test_slabs_and_whole_rows(pool, dt, n, m, T, weights, short, popular):
    print(f"[case] pool slabs {pool} {dt} n={n} m={m} T={T} short={short} popular={popular}",
          flush=True)
    _run(dt, n, m, T, 16_384 + 77, pool, weights, short, popular)


# At 8 GB of gathered rows and more the probe runs and the choice shows: a call with few
# of the same rows always takes whole rows, whose sums have another order (an element in
# a few hundred thousand then rounds otherwise at the least, also in bf16).
@pytest.mark.parametrize("pool", ["importance", "mean", "max"])
@pytest.mark.parametrize("dt,n,m,T,rows,weights,short,popular,slabs", [
    (torch.float32, 50_003, 256, 50, 175_003, True, False, True, True),     # 256-byte slabs
    (torch.float32, 60_000, 272, 64, 140_001, False, False, True, True),    # last slab not whole
    (torch.float32, 530_001, 256, 64, 140_001, True, False, True, True),    # 128-byte slabs
    (torch.bfloat16, 60_000, 512, 64, 140_001, True, False, True, True),    # 256-byte slabs
    (torch.bfloat16, 60_000, 528, 62, 140_001, False, False, True, True),   # last slab not whole
    (torch.bfloat16, 530_000, 528, 64, 140_001, True, False, True, True),   # 128-byte slabs
    (torch.float32, 530_000, 256, 64, 140_001, True, False, False, False),  # evenly spread
    (torch.float32, 60_000, 256, 64, 140_001, True, True, True, False),     # short rows
    (torch.bfloat16, 60_000, 512, 64, 140_001, False, True, True, False),
])
def test_the_choice_between_slabs_and_whole_rows(pool, dt, n, m, T, rows, weights, short, popular,
                                                 slabs):
    import paper_1806_01973_amd as ps
    print(f"[case] pool choice {pool} {dt} n={n} m={m} T={T} short={short} popular={popular}",
          flush=True)
    layer, h, nbr, out = _run(dt, n, m, T, rows, pool, weights, short, popular)
    k = 100_000
    part = ps.Neighborhoods(nbr.idx[:k], nbr.counts[:k], nbr.weights[:k] if weights else None)
    self_rows = torch.zeros(k, dtype=torch.int32, device="cuda")
    whole = ps.convolve_layer(layer, h, n, part, self_rows=self_rows)
    if pool == "max":  # the same bits either way
        assert torch.equal(whole, out[:k])
    else:
        assert torch.equal(whole, out[:k]) != slabs


def test_the_choice_does_not_depend_on_the_workspace():
    """A workspace with no room for the split weights gives the same bits, slabs or not."""
    import paper_1806_01973_amd as ps
    n, m, T, rows = 60_000, 256, 64, 140_001
    layer, h, nbr, out = _run(torch.float32, n, m, T, rows, "importance", True, False, True)
    rows_of = lambda r: (r * m * 4 + 255) // 256 * 256
    small = torch.empty(rows_of(n) + rows_of(rows), dtype=torch.uint8, device="cuda")
    assert small.numel() < ps.convolve_workspace_size(layer, n, rows)
    self_rows = torch.zeros(rows, dtype=torch.int32, device="cuda")
    assert torch.equal(ps.convolve_layer(layer, h, n, nbr, self_rows=self_rows, workspace=small), out)


def test_output_over_the_self_rows():
    """A layer that writes its rows over the self rows it reads: the choice must not lie
    there, so the pool takes whole rows (the bits of a call of few rows)."""
    import paper_1806_01973_amd as ps
    n, m, T, rows = 60_000, 256, 64, 140_001
    layer, _, nbr, _ = _run(torch.float32, n, m, T, rows, "importance", True, False, True)
    g = torch.Generator(device="cuda").manual_seed(3)
    W = torch.randn((m, 2 * m), generator=g, device="cuda") * 0.05
    layer = ps.DeviceLayer(torch.eye(m, device="cuda"), torch.zeros(m), W, torch.zeros(m))
    h = torch.rand((rows, m), generator=g, device="cuda")
    k = 5_000
    part = ps.Neighborhoods(nbr.idx[:k], nbr.counts[:k], nbr.weights[:k])
    want = ps.convolve_layer(layer, h, n, part)
    apart = ps.convolve_layer(layer, h, n, nbr)
    assert not torch.equal(apart[:k], want)  # slabs
    ps.convolve_layer(layer, h, n, nbr, out=h)
    assert torch.equal(h[:k], want)
    # Entries of unit rows: another order of T weighted values moves them by under 2 T 2^-24.
    assert (h - apart).abs().max() <= 2 * T * 2.0 ** -24
