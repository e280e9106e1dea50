"""Max-margin loss at the edges of its tiles: 16 queries per block, 16 negatives per wave,
k-steps of 32 columns in groups, rows that are not whole 16-byte vectors.

Against 64 bits: a hinge term moves by at most the errors of its two scores, each
(d + 8) 2^-24 of the summed magnitudes (fp32 accumulation, exact operands)."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,n,k,d", [(1, 1, 0, 1), (16, 16, 1, 32), (17, 15, 3, 33), (15, 129, 0, 31),
                                     (33, 17, 2, 136), (40, 130, 1, 257), (18, 40, 1, 512),
                                     (3, 300, 33, 520), (19, 31, 2, 1000)])
def test_loss_at_tile_edges(dtype, B, n, k, d):
    import paper_1806_01973_amd as ps
    print(f"[case] loss {dtype} B={B} n={n} k={k} d={d}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(B + d)
    rows = lambda *s: torch.randn(s, generator=gen).mul_(d ** -0.5).to(dt)
    q, p, ng = rows(B, d), rows(B, d), rows(n, d)
    h = rows(B, k, d) if k else None
    loss, per = ps.max_margin_loss(q.cuda(), p.cuda(), ng.cuda(), 0.1,
                                   h.cuda() if k else None)
    Q, P, N = q.double(), p.double(), ng.double()
    s = torch.cat([Q @ N.t()] + ([(Q[:, None] * h.double()).sum(2)] if k else []), 1)
    mag = torch.cat([Q.abs() @ N.abs().t()] + ([(Q.abs()[:, None] * h.double().abs()).sum(2)] if k else []), 1)
    pos, pmag = (Q * P).sum(1, keepdim=True), (Q.abs() * P.abs()).sum(1, keepdim=True)
    ref = torch.relu(s - pos + 0.1).mean(1)
    tol = (d + 8) * 2.0 ** -24 * (mag + pmag).mean(1) + (n + k + 8) * 2.0 ** -24 * (ref + 0.1)
    assert ((per.double().cpu() - ref).abs() <= tol).all()
    assert abs(float(loss) - float(ref.mean())) <= float(tol.mean()) + 2e-6 * float(ref.mean())


def test_loss_with_infinite_and_huge_rows():
    import paper_1806_01973_amd as ps
    gen = torch.Generator().manual_seed(2)
    q, p, ng = (torch.randn((20, 64), generator=gen) for _ in range(3))
    q[:, 5] = q[:, 5].abs() + 0.1
    ng[3, 5] = -3.4e38  # a score far below every margin
    ng[4, 5] = 3.4e38   # rounds to infinity in bf16; a huge finite hinge
    ng[4, 6:] = 0.0
    loss, per = ps.max_margin_loss(q.cuda(), p.cuda(), ng.cuda(), 0.1)
    s = q.double() @ ng.double().t() - (q.double() * p.double()).sum(1, keepdim=True) + 0.1
    ref = torch.relu(s).mean(1)
    fine = s.amax(1) < 3e38  # the scores themselves fit fp32
    assert fine.any()
    assert torch.allclose(per.double().cpu()[fine], ref[fine], rtol=1e-5)
    ng[4, 5] = float("inf")
    _, per = ps.max_margin_loss(q.cuda(), p.cuda(), ng.cuda(), 0.1)
    assert torch.isinf(per).all()


def test_scores_of_values_at_the_ends_of_the_range():
    """Tiny queries against huge negatives and the other way round, tiny values beside
    ordinary ones, an infinite and a NaN row among others; also in rows that are not whole
    vectors. Each score has fp32's error, (d + 8) 2^-24 of the summed magnitudes."""
    import paper_1806_01973_amd as ps
    for d in (64, 65):
        gen = torch.Generator().manual_seed(d)
        q, p, ng = (torch.randn((n, d), generator=gen) for n in (20, 20, 40))
        p *= 0.0
        ng[:, :4] = 0.0
        q[3] *= 2.0 ** -120
        ng[5] = 0.0
        ng[5, 0] = 2.0 ** 115
        q[4, 0] = 1.2345 * 2.0 ** -130  # against ng[5]: the lone product 1.2e-5
        q[:, 0] = torch.where(torch.arange(20) == 4, q[:, 0], 0.0)
        q[:, 1] = torch.where(torch.arange(20) == 7, 2.0 ** 120, 0.0)
        ng[6, 1] = 1.2345 * 2.0 ** -125
        s = q.double() @ ng.double().t()  # (the positives are zero rows)
        mag = q.double().abs() @ ng.double().abs().t()
        _, per = ps.max_margin_loss(q.cuda(), p.cuda(), ng.cuda(), 0.1)
        ref = torch.relu(s + 0.1).mean(1)
        tol = (d + 8) * 2.0 ** -24 * mag.mean(1) + 48 * 2.0 ** -24 * (ref + 0.1)
        assert ((per.double().cpu() - ref).abs() <= tol).all()
        # One negative at a time, so that no other term hides its score.
        for n in (5, 6):
            _, one = ps.max_margin_loss(q.cuda(), p.cuda(), ng[n:n + 1].cuda(), 0.0)
            tol1 = (d + 8) * 2.0 ** -24 * mag[:, n] + 2.0 ** -149
            assert ((one.double().cpu() - torch.relu(s[:, n])).abs() <= tol1).all(), n
        # An infinite negative moves every pair to infinity or leaves its term at 0; a NaN
        # query has only zero terms; the others keep their bits.
        q2 = q.clone()
        q2[11, 9] = float("nan")
        _, per2 = ps.max_margin_loss(q2.cuda(), p.cuda(), ng.cuda(), 0.1)
        assert float(per2[11]) == 0.0
        keep = torch.arange(20) != 11
        assert torch.equal(per2.cpu()[keep], per.cpu()[keep])
        ng2 = ng.clone()
        ng2[30, 20] = float("inf")
        _, per3 = ps.max_margin_loss(q.cuda(), p.cuda(), ng2.cuda(), 0.1)
        up = q[:, 20] > 0
        assert torch.isinf(per3.cpu()[up]).all() and torch.isfinite(per3.cpu()[~up]).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,d", [(1, 8), (4, 64), (5, 264), (15, 72), (16, 130), (17, 1024), (70, 96)])
def test_hard_negatives_at_the_edges_of_their_groups(dtype, k, d):
    """4 or 16 rows of a pair at a time, 8 threads each; tables that start on a whole
    vector and one element past it give the same sums up to their order."""
    import paper_1806_01973_amd as ps
    print(f"[case] hard negatives {dtype} k={k} d={d}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(k + d)
    B = 21
    rows = lambda *s: torch.randn(s, generator=gen).mul_(d ** -0.5).to(dt)
    q, p, ng, h = rows(B, d), rows(B, d), rows(3, d), rows(B, k, d)
    Q = q.double()
    dots = lambda t: torch.cat([Q @ ng.double().t(), (Q[:, None] * t).sum(2)], 1)
    pos = (Q * p.double()).sum(1, keepdim=True)
    ref = torch.relu(dots(h.double()) - pos + 0.1).mean(1)
    mag = (torch.cat([Q.abs() @ ng.double().abs().t(), (Q.abs()[:, None] * h.double().abs()).sum(2)], 1)
           + (Q.abs() * p.double().abs()).sum(1, keepdim=True)).mean(1)
    tol = (d + 8) * 2.0 ** -24 * mag + (k + 11) * 2.0 ** -24 * (ref + 0.1)
    base = torch.zeros(B * k * d + 8, dtype=dt, device="cuda")
    for shift in (0, 1):
        hd = base[shift:shift + B * k * d].view(B, k, d)
        hd.copy_(h)
        _, per = ps.max_margin_loss(q.cuda(), p.cuda(), ng.cuda(), 0.1, hd)
        assert ((per.double().cpu() - ref).abs() <= tol).all(), shift
