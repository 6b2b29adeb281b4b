"""Loaded layers on either side of the size from which values go past the caches: entries as given, the rest of a last block zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [8191, 8192, 8193])        # of 64 units: keys and values of 256 MiB at 8192
@pytest.mark.parametrize("ragged", [False, True])
def test_entries_as_given(P, ragged):
    import torch
    from paper_2601_16986_amd import ckv
    Bz, Hkv, cap = 8, 8, 8224
    g = ckv.CrystalKV(1, Bz, Hkv, Hkv, 128, cap, np.full((1, Bz, Hkv), P, np.int32), t0=P, budget_min=1, budget_max=cap - 1)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(P)
    k = torch.randn((Bz, Hkv, P, 128), generator=gen, device=g.device, dtype=torch.bfloat16)
    v = torch.randn((Bz, Hkv, P, 128), generator=gen, device=g.device, dtype=torch.bfloat16)
    lengths = np.full((Bz, Hkv), P)
    if ragged:
        lengths.reshape(-1)[:8] = [0, 1, 31, 32, 33, 257, P - 1, P]
        pos = torch.arange(P, dtype=torch.int32, device=g.device).expand(Bz, Hkv, P).contiguous()
        g.load_cache(0, k, v, torch.from_numpy(lengths.astype(np.int32)).to(g.device), torch.full((Bz, Hkv, P), 2.0, device=g.device), pos, pos)
    else:
        g.load_prompt(0, k, v)
    assert np.array_equal(g.lengths()[0], lengths)
    for u in [0, 1, 2, 3, 4, 5, 6, 7, 40, 63]:
        b, h = divmod(u, Hkv)
        n = lengths[b, h]
        e = g.export_unit(0, b, h)
        assert np.array_equal(e["pos"], np.arange(n))
        assert np.array_equal(e["K"], k[b, h, :n].float().cpu().numpy()) and np.array_equal(e["V"], v[b, h, :n].float().cpu().numpy())
    # a unit has 33 segments of 256 slots of its own, in order; the slots of a last block that hold nothing are read and multiplied by 0
    slots = 33 * 256
    for u in range(64):
        n = int(lengths.reshape(-1)[u])
        end = (n + 31) // 32 * 32
        block = g.v_pool[u * slots * 128:(u + 1) * slots * 128].view(-1, 32 * 128)
        if n % 32:                                        # 16-byte pieces of eight entries each
            assert int((block[end // 32 - 1] != 0).sum()) == int((v.view(64, P, 128)[u, end - 32:n] != 0).sum())
    assert g.status() == 0
    g.close()
