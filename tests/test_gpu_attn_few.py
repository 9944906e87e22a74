"""Small launches of bf16 handles against fp64 softmax over the same rows, at the edges of the kernel they
take: 16 queries to a group, one, two or four groups to a workgroup, 32 slots to a tile, eight waves and up
to 16 slot ranges; and sizes on both sides of the line to the kernel for large ones."""
import numpy as np
import pytest

from paper_2603_05959_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,n_old,H,layers,out", [
    (1, 1, 1, 1, "f32"), (1, 30, 3, 1, "bf16"), (1, 31, 1, 2, "f32"), (1, 32, 1, 1, "f32"),   # one tile, ragged and full; two
    (15, 241, 2, 1, "f32"), (16, 240, 2, 1, "bf16"), (17, 240, 2, 2, "f32"),   # eight tiles: one a wave; one query of the next block
    (1, 479, 1, 1, "f32"), (1, 480, 1, 1, "f32"),                   # the last size in one range, the first in two
    (1, 4095, 1, 1, "f32"), (5, 4200, 3, 1, "bf16"),                # the most ranges; ranges of unequal length
    (33, 16000, 16, 1, "f32"), (64, 8000, 16, 1, "bf16"),           # two groups, the last one of padding; two full ones
    (128, 16384, 16, 1, "f32"), (97, 4096, 16, 12, "bf16"),         # four groups, split and not
    (1041, 4096, 1, 1, "f32"), (513, 2048, 4, 1, "f32"),            # many blocks of few heads
    (300, 4096, 16, 1, "f32"), (400, 4096, 16, 1, "f32"), (700, 4096, 16, 1, "f32"),   # here, and the large kernel
])
def test_matches_fp64_softmax(M, n_old, H, layers, out):
    import torch
    gen = torch.Generator().manual_seed(M * 1000 + n_old)
    cache = B.Cache(layers, H, 64, M, 64, max(n_old, M), "bf16", out_dtype=out)
    kernel = B.ovggt_attn_route(cache.cfg, layers, n_old + M)["kernel"]
    assert kernel == ("items" if M in (400, 700) else "few")
    rnd = lambda *s: torch.randn(s, generator=gen, dtype=torch.float32).bfloat16()
    old = [(rnd(n_old, H, 64), rnd(n_old, H, 64)) for _ in range(layers)]
    for l, (k, v) in enumerate(old):
        cache.import_(l, 3 + n_old // M, np.arange(n_old, dtype=np.uint32), k.view(torch.int16).numpy().view(np.uint16),
                      v.view(torch.int16).numpy().view(np.uint16), np.ones(n_old, np.float32), np.zeros(n_old, np.uint8))
    o = cache.new_output()
    for rep in range(2):                                # the arrival counters are back at zero for the second frame
        q, k, v = (rnd(layers, M, H, 64) for _ in range(3))
        q[:, 0] *= 6.0                                  # one dominant key, and a reference that is passed by far
        cache.step(q.cuda(), k.cuda(), v.cuda(), torch.ones(layers, M, 64, device="cuda").bfloat16(), None, o)
        got = o.double()
        for l in sorted({0, layers - 1}):
            # the cache holds half(bf16): exact for all but values below 2^-14
            kk, vv = (torch.cat([a, b]).half().double().cuda() for a, b in ((old[l][0], k[l]), (old[l][1], v[l])))
            for h in sorted({0, H // 2, H - 1}):
                p = torch.softmax(torch.mm(q[l, :, h].double().cuda(), kk[:, h].t().contiguous()) / 8.0, dim=-1)
                ref = torch.mm(p, vv[:, h])
                err = ((got[l, :, h] - ref).norm() / ref.norm()).item()
                # weights rounded to 11 bits (relative errors of 2^-11 / sqrt(3) at most in the mean, as random signs add up);
                # the kernel for large launches rounds the scaled queries to 11 bits too; a bf16 output has 8 bits
                assert err < 2.0 ** -11 + (2.0 ** -11 if kernel == "items" else 0.0) + (2.0 ** -9 if out == "bf16" else 0.0), (rep, l, h, err)
        e = [cache.export(l) for l in range(layers)]
        old = [tuple(torch.from_numpy(x[n]).bfloat16() for n in "kv") for x in e]
    cache.close()


@pytest.mark.parametrize("n_old", [3, 17, 40])           # one tile; its last rows; the second tile of two
def test_rows_behind_the_last_slot_carry_no_weight(n_old):
    """Evicted entries stay in memory behind the resident ones, NaN among them."""
    import torch
    M, H, Bq = 5, 2, 70
    gen = torch.Generator().manual_seed(2)
    cache = B.Cache(1, H, 64, M, 64, Bq, "bf16")
    assert B.ovggt_attn_route(cache.cfg, 1, n_old + M)["kernel"] == "few"
    ids, ones, zeros = np.arange(Bq, dtype=np.uint32), np.ones(Bq, np.float32), np.zeros(Bq, np.uint8)
    fill = np.full((Bq, H, 64), 0x7FC0, np.uint16)                   # NaN in every slot, before the few that stay resident
    cache.import_(0, 14, ids, fill, fill, ones, zeros)
    ko, vo = (torch.randn(n_old, H, 64, generator=gen).bfloat16() for _ in range(2))
    bits = lambda x: x.view(torch.int16).numpy().view(np.uint16)
    cache.import_(0, 14, ids[:n_old], bits(ko), bits(vo), ones[:n_old], zeros[:n_old])
    q, k, v = (torch.randn(1, M, H, 64, generator=gen).bfloat16() for _ in range(3))
    o = cache.new_output()
    cache.step(q.cuda(), k.cuda(), v.cuda(), torch.ones(1, M, 64).bfloat16().cuda(), None, o)
    kk, vv = torch.cat([ko, k[0]]).half().double(), torch.cat([vo, v[0]]).half().double()
    ref = torch.einsum("hmn,nhd->mhd", torch.softmax(torch.einsum("mhd,nhd->hmn", q[0].double(), kk) / 8.0, dim=-1), vv)
    assert (o[0].cpu().double() - ref).norm() / ref.norm() < 2.0 ** -11          # as above
    cache.close()


@pytest.mark.parametrize("dtype,M,H,budget,kernel", [("bf16", 1, 4, 40, "few"), ("bf16", 700, 16, 4096, "items"), ("f32", 40, 2, 100, "f32")])
def test_timing_counts_the_launches_there_are(dtype, M, H, budget, kernel):
    """Bracketed launches per kernel class: a merge pass only where there is one."""
    import torch
    cache = B.Cache(1, H, 64, M, 64, budget, dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, r = torch.randn(1, M, H, 64, device="cuda").to(dt), torch.ones(1, M, 64, device="cuda").to(dt)
    out = cache.new_output()
    for level in (1, 2):
        while cache.size(0) < budget:                   # the last frames are on a full cache
            cache.step(x, x, x, r, None, out)
        B.ovggt_profile_read(cache.h, cache.stream)
        B.ovggt_profile_enable(cache.h, level, 1)
        for _ in range(5):
            cache.step(x, x, x, r, None, out)
        assert B.ovggt_attn_route(cache.cfg, 1, budget + M)["kernel"] == kernel
        got = B.ovggt_profile_read(cache.h, cache.stream)
        assert got["attn"][1] == 5 and got["combine"][1] == (5 if kernel == "items" else 0)
        assert got["append"][1] == got["score_select"][1] == (5 if level == 2 else 0)
        assert got["attn"][0] > 0
    cache.close()
