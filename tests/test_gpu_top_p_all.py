"""top_p of 1 and above marks every entry, however the weights' sum rounds: in the step's two implementations, deferred, and in the
prompt replay with its rows in registers and in LDS. (Queries four times as long as usual: the smallest weights lie far below the sum's last bit.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("how", ["split", "fused", "defer"])
@pytest.mark.parametrize("n", [40, 2000, 5000, 9000])
@pytest.mark.parametrize("p", [1.0, 1.5, float("inf")])
def test_step(p, n, how):
    import torch
    from paper_2601_16986_amd import ckv
    B, H, G, cap = 8, 4, 3, (n + 64) // 32 * 32
    g = ckv.CrystalKV(1, B, H * G, H, 128, cap, np.full((1, B, H), cap - 1, np.int32), t0=n, top_p=p)
    g.set_path(2 if how == "fused" else 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(n)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    k = rnd(B, H, n, 128)
    g.load_prompt(0, k, k)
    g.decode_step(4 * rnd(B, H * G, 128), rnd(B, H, 128), rnd(B, H, 128), layer=0, defer=how == "defer")
    g.join()
    for b in range(B):
        for h in range(H):
            e = g.export_unit(0, b, h, with_kv=False)
            assert e["n"] == n + 1 and np.all(e["tau"] == n) and np.all(e["flags"] & 1)
    assert g.status() == 0
    g.close()


@pytest.mark.parametrize("P", [600, 9000, 16500])
def test_replay(P):
    import torch
    from paper_2601_16986_amd import ckv
    B, H, G, W = 2, 4, 5, 3
    g = ckv.CrystalKV(1, B, H * G, H, 128, (P + 64) // 32 * 32, np.full((1, B, H), P, np.int32), t0=P, top_p=1.0)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(P)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    k = rnd(B, H, P, 128)
    g.load_prompt(0, k, k)
    g.seed_prompt(0, 4 * rnd(W, B, H * G, 128))
    for b in range(B):
        for h in range(H):
            assert np.all(g.export_unit(0, b, h, with_kv=False)["tau"] == P - 1)
    g.close()
