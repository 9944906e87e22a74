"""fp32 attention against fp64 softmax over the same rows, at the edges of its tiles: 16 queries to a
workgroup, 16 slots to a tile, eight waves and up to 16 slot ranges that share the tiles."""
import numpy as np
import pytest

from paper_2603_05959_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_old,H,layers", [
    (1, 1, 1, 1), (1, 14, 3, 1), (8, 8, 5, 3), (1, 15, 2, 2), (1, 16, 1, 2),   # one tile, ragged and full; one slot of the next
    (15, 113, 2, 1), (16, 112, 2, 1), (17, 112, 2, 2),  # eight tiles: one a wave; one query of the next block
    (2, 254, 1, 1), (3, 254, 1, 1),                     # sixteen tiles, two for each wave; one more
    (1, 495, 1, 1), (1, 496, 1, 1), (33, 1000, 1, 1),   # the last size in one range, the first in two; four ranges
    (16, 4080, 1, 1), (40, 4057, 3, 2),                 # the most ranges; ranges of unequal length
    (272, 1300, 16, 1), (97, 2048, 4, 24),              # more blocks than CUs: two or more ranges each, and one
])
def test_matches_fp64_softmax(M, n_old, H, layers):
    import torch
    gen = torch.Generator().manual_seed(M * 1000 + n_old)
    cache = B.Cache(layers, H, 64, M, 64, max(n_old, M), "f32")
    n_old = min(n_old, max(n_old, M))
    rnd = lambda *s: torch.randn(s, generator=gen, dtype=torch.float32)
    old = [(rnd(n_old, H, 64), rnd(n_old, H, 64)) for _ in range(layers)]
    # three frames seen, so that a later frame's ids stay unique
    for l, (k, v) in enumerate(old):
        cache.import_(l, 3 + n_old // M, np.arange(n_old, dtype=np.uint32), k.numpy(), v.numpy(),
                      np.ones(n_old, np.float32), np.zeros(n_old, np.uint8))
    out = cache.new_output()
    for rep in range(2):                                # the arrival counters are back at zero for the second frame
        q, k, v = (rnd(layers, M, H, 64) for _ in range(3))
        q[:, 0] *= 12.0                                 # one dominant key, and a reference that is passed by far
        cache.step(q.cuda(), k.cuda(), v.cuda(), torch.ones(layers, M, 64, device="cuda"), None, out)
        got = out.cpu().double()
        for l in range(layers):
            kk, vv = torch.cat([old[l][0], k[l]]).double(), torch.cat([old[l][1], v[l]]).double()
            p = torch.softmax(torch.einsum("mhd,nhd->hmn", q[l].double(), kk) / 8.0, dim=-1)
            ref = torch.einsum("hmn,nhd->mhd", p, vv)
            # a score carries at most about 64 roundings of 2^-24 times its terms' size (|s| up to about 60 in the
            # scaled rows): relative errors of weights and outputs near 1e-5 at worst, 1e-6 in the mean
            assert (got[l] - ref).norm() / ref.norm() < 5e-6, (rep, l)
        e = [cache.export(l) for l in range(layers)]
        old = [(torch.from_numpy(x["k"]), torch.from_numpy(x["v"])) for x in e]
    cache.close()


@pytest.mark.parametrize("n_old", [3, 10, 17])           # one tile for one wave; the second tile of two, ragged and nearly full
def test_rows_behind_the_last_slot_are_not_read(n_old):
    """Evicted entries stay in memory behind the resident ones, infinities and NaN among them."""
    import torch
    M, H, Bq = 5, 2, 40
    gen = torch.Generator().manual_seed(2)
    cache = B.Cache(1, H, 64, M, 64, Bq, "f32")
    ids, ones, zeros = np.arange(Bq, dtype=np.uint32), np.ones(Bq, np.float32), np.zeros(Bq, np.uint8)
    for l, poison in enumerate((float("inf"), float("nan"))):
        fill = np.full((Bq, H, 64), poison, np.float32)
        cache.import_(0, 8, ids, fill, fill, ones, zeros)            # every slot, before the few that stay resident
        ko, vo = (torch.randn(n_old, H, 64, generator=gen) for _ in range(2))
        cache.import_(0, 8, ids[:n_old], ko.numpy(), vo.numpy(), ones[:n_old], zeros[:n_old])
        q, k, v = (torch.randn(1, M, H, 64, generator=gen) for _ in range(3))
        out = cache.new_output()
        cache.step(q.cuda(), k.cuda(), v.cuda(), torch.ones(1, M, 64).cuda(), None, out)
        kk, vv = torch.cat([ko, k[0]]).double(), torch.cat([vo, v[0]]).double()
        ref = torch.einsum("hmn,nhd->mhd", torch.softmax(torch.einsum("mhd,nhd->hmn", q[0].double(), kk) / 8.0, dim=-1), vv)
        assert (out[0].cpu().double() - ref).norm() / ref.norm() < 5e-6, poison
    cache.close()


@pytest.mark.parametrize("n_old,H,layers", [(700, 1, 1), (4000, 2, 1), (300, 16, 24)])   # split into ranges, and not
def test_values_near_the_ends_of_the_fp32_range(n_old, H, layers):
    """Logits that rise slowly enough for the softmax reference to stay behind, and many slots of almost no
    weight, over values of V near the largest fp32 number: the result is a mean of them and finite.  And values
    near the smallest one."""
    import torch
    M = 3
    for size in (1e38, 1e-36):
        cache = B.Cache(layers, H, 64, M, 64, n_old, "f32")
        gen = torch.Generator().manual_seed(n_old)
        n = n_old + M
        # every 32nd slot is one of the rising ones (from e^-6 to 1); between them the weights are e^-60 and less
        logit = torch.full((n,), -60.0)
        logit[::32] = torch.linspace(-6.0, 0.0, len(logit[::32]))
        k = torch.zeros(layers, n, H, 64)
        k[..., 0] = logit[None, :, None] * 8.0
        v = (0.5 + torch.rand(layers, n, H, 64, generator=gen)) * size * torch.where(torch.rand(64, generator=gen) < 0.5, -1.0, 1.0)
        v /= torch.softmax(logit.double(), 0).max().reciprocal().float()      # sums of weighted values stay finite, too
        for l in range(layers):
            cache.import_(l, 3 + n_old // M, np.arange(n_old, dtype=np.uint32), k[l, :n_old].numpy(), v[l, :n_old].numpy(),
                          np.ones(n_old, np.float32), np.zeros(n_old, np.uint8))
        q = torch.zeros(layers, M, H, 64)
        q[..., 0] = 1.0
        out = cache.new_output()
        cache.step(q.cuda(), k[:, n_old:].contiguous().cuda(), v[:, n_old:].contiguous().cuda(), torch.ones(layers, M, 64, device="cuda"), None, out)
        got = out.cpu().double()
        p = torch.softmax(logit.double(), 0)
        ref = torch.matmul(p, v.double().permute(0, 2, 1, 3)).unsqueeze(1)
        assert torch.isfinite(got).all()
        # sixty-four roundings of 2^-24 in a score of size 60, as above; few of them where the weight is
        assert (got - ref).norm() / (ref.norm() * M ** 0.5) < 5e-6, size
        cache.close()


@pytest.mark.parametrize("scale,q0,k0", [(3e38, 0.0, 1.0), (2.5e38, 4e-19, 4e-19), (1.0, 1.2e19, 2e19), (0.5, 1.2e19, 2e19), (0.0, 3e5, 7e5),
                                         (2.0, 1.0, 3.0)])
@pytest.mark.parametrize("M,n_old", [(5, 90), (17, 3000)])       # one range of the slots, and several
def test_scores_up_to_the_end_of_the_fp32_range(scale, q0, k0, M, n_old):
    """Every finite softmax scale is accepted, and every score counts that is finite once scaled."""
    import torch
    H, n = 2, n_old + M
    cache = B.Cache(1, H, 64, M, 64, n_old, "f32", softmax_scale=scale)
    gen = torch.Generator().manual_seed(M)
    k, v = torch.zeros(n, H, 64), torch.randn(n, H, 64, generator=gen)
    k[:, :, 3] = k0 * torch.randint(0, 4, (n, 1), generator=gen) / 3.0        # four sizes of score: ties at the top
    q = torch.zeros(1, M, H, 64)
    q[..., 3] = q0
    cache.import_(0, 3 + n_old // M, np.arange(n_old, dtype=np.uint32), k[:n_old].numpy(), v[:n_old].numpy(),
                  np.ones(n_old, np.float32), np.zeros(n_old, np.uint8))
    out = cache.new_output()
    cache.step(q.cuda(), k[None, n_old:].contiguous().cuda(), v[None, n_old:].contiguous().cuda(),
               torch.ones(1, M, 64, device="cuda"), None, out)
    s = q[0, 0, 0, 3].double() * k[:, 0, 3].double() * float(np.float32(scale or 0.125))
    assert s.abs().max() < 3.4e38
    ref = torch.einsum("n,nhd->hd", torch.softmax(s, 0), v.double())
    got = out[0].cpu().double()
    # scores are equal, too far apart for more than one group to count, or at most 40 with errors of a few 2^-24 of that
    assert ((got - ref).norm(dim=(1, 2)) / ref.norm() < 5e-6).all(), (got - ref).abs().max()
    cache.close()
