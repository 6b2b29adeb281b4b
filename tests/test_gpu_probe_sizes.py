"""Probe classes at the sizes where the selection changes its width and the scan its last block, against the classes
that a plain sort of the same weights in 64 bits gives."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(batch, hkv, G, cap, lengths, sample):
    import torch
    from paper_2601_16986_amd import ckv
    units, n_max = batch * hkv, int(max(lengths))
    g = ckv.CrystalKV(1, batch, hkv * G, hkv, 128, cap, np.full((1, batch, hkv), cap - 1, np.int32), t0=n_max, budget_min=1, budget_max=cap - 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(3)
    rnd = lambda *shape: torch.randn(shape, generator=gen, device=g.device).to(torch.bfloat16)
    k, v, q = rnd(batch, hkv, n_max, 128), rnd(batch, hkv, n_max, 128), rnd(batch, hkv * G, 128)
    pos = torch.stack([torch.randperm(n_max, generator=gen, device=g.device) for _ in range(units)]).reshape(batch, hkv, n_max).int().contiguous()
    # equal keys tie exactly (which of them belongs to which class is pinned in test_ties_alone_decide)
    k[:, :, n_max // 2:] = k[:, :, :n_max - n_max // 2]
    z = torch.zeros((batch, hkv, n_max), dtype=torch.int32, device=g.device)
    g.load_cache(0, k, v, torch.tensor(np.asarray(lengths, np.int32).reshape(batch, hkv), device=g.device), z.float(), z, pos)
    for noalloc in (False, True):
        cls = torch.full((batch, hkv, cap), 255, dtype=torch.uint8, device=g.device)
        cls = g.probe_noalloc(0, q, cls) if noalloc else g.probe(0, q)
        got = cls.cpu().numpy().reshape(units, cap)
        for u in sample:
            n, b, h = int(lengths[u]), u // hkv, u % hkv
            s = q[b, h * G:(h + 1) * G].double() @ k[b, h, :n].double().t().contiguous() / np.sqrt(128.0)
            a = torch.softmax(s, dim=-1).mean(0).cpu().numpy()
            p = pos[b, h, :n].cpu().numpy()
            # equal keys have equal weights on the device; make the 64-bit ones equal too before ties go to the position
            a = np.where(np.arange(n) >= n_max // 2, a[np.arange(n) % (n_max // 2)] if n_max % 2 == 0 else a, a)
            order, kq = np.lexsort((-p, a)), (3 * n) // 10
            want = np.ones(n, np.uint8)
            want[order[:kq]] = 0
            want[order[n - kq:]] = 2
            assert np.all(got[u, n:] == 255) and (got[u, :n] == 0).sum() == kq and (got[u, :n] == 2).sum() == kq
            wrong = np.flatnonzero(got[u, :n] != want)
            if kq:
                edges = a[order[[kq - 1, kq, n - kq - 1, n - kq]]]
                # fp32 sums and the hardware exponential carry a few 1e-6: only weights that close to a boundary may differ
                assert all(np.min(np.abs(a[i] - edges) / edges) < 1e-5 for i in wrong), (u, n, len(wrong))
            else:
                assert len(wrong) == 0
    g.close()


@pytest.mark.parametrize("G,cap,lengths", [
    (1, 64, [1, 2, 3, 33]), (8, 160, [127, 128, 129, 160 - 2]), (5, 4128, [4096, 4095, 4097, 100]), (3, 16416, [16384, 8193, 16385, 8192]),
    (4, 32768, [32766, 9350, 255, 257]),
])
def test_wide_classes(G, cap, lengths):
    _check(2, 2, G, cap, lengths, range(4))


def test_many_small_units():
    """Enough units for workgroups of 256 threads; lengths at the edges of 4, 8 and 16 entries per thread."""
    edge = [1, 10, 31, 129, 1024, 1025, 2048, 2050]
    _check(528, 2, 2, 2080, [edge[i % 8] for i in range(1056)], range(0, 1056, 67))


@pytest.mark.parametrize("batch,cap,n,distinct", [
    (2, 4096, 4000, 1), (2, 8192, 8100, 3), (2, 16384, 16000, 1), (2, 32768, 32000, 5),           # 4, 8, 16, 32 entries per thread of 1024
    (528, 1024, 1000, 3), (528, 2048, 2011, 1), (528, 4096, 3900, 4), (528, 8192, 4200, 2),       # ... and of 256
    (2, 96, 70, 1), (2, 64, 33, 2),
])
def test_ties_alone_decide(batch, cap, n, distinct):
    """A unit of a few distinct keys: every entry ties with a large part of the unit, across both boundaries, and the classes follow
    the positions exactly (within a group of equal weights the lower position ranks higher)."""
    import torch
    from paper_2601_16986_amd import ckv
    hkv, G = 2, 2
    g = ckv.CrystalKV(1, batch, hkv * G, hkv, 128, cap, np.full((1, batch, hkv), cap - 1, np.int32), t0=4 * n, budget_min=1, budget_max=cap - 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(11)
    # keys far enough apart that the groups' order does not hang on rounding: group i lies i / 2 further along every query's mean
    base = torch.randn(128, generator=gen, device=g.device)
    q = (base + 0.05 * torch.randn((batch, hkv * G, 128), generator=gen, device=g.device)).to(torch.bfloat16)
    rows = (base[None] * (0.05 * torch.arange(distinct, device=g.device)[:, None])).to(torch.bfloat16)
    which = torch.randint(0, distinct, (batch, hkv, n), generator=gen, device=g.device)
    k = rows[which].contiguous()
    pos = torch.rand((batch, hkv, 4 * n), generator=gen, device=g.device).argsort(-1)[..., :n].int().contiguous()
    z = torch.zeros((batch, hkv, n), dtype=torch.int32, device=g.device)
    g.load_cache(0, k, k, torch.full((batch, hkv), n, dtype=torch.int32, device=g.device), z.float(), z, pos)
    got = g.probe(0, q)[..., :n]
    kq = (3 * n) // 10
    # rank: heavier group first, then lower position
    order = (which.long() * (8 * n) + (4 * n - pos.long())).argsort(-1, descending=True)
    want = torch.ones_like(got)
    want.scatter_(-1, order[..., :kq], 2)
    want.scatter_(-1, order[..., n - kq:], 0)
    assert torch.equal(got, want)
    assert torch.equal(g.probe_noalloc(0, q, torch.zeros((batch, hkv, cap), dtype=torch.uint8, device=g.device))[..., :n], want)
    g.close()
