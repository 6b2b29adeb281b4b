"""What a new context's buffers hold before anything is loaded: budgets, segments, spare list, time, zeros, on memory that held
something else; and its decay table, short and long (the long one does not fit the place through which the rest is staged)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("headroom", [0, 1, 40])
@pytest.mark.parametrize("L,batch,hkv,cap", [(1, 1, 1, 32), (3, 1, 1, 288), (2, 3, 5, 800), (7, 16, 8, 2080), (256, 1, 2, 512)])
def test_state(L, batch, hkv, cap, headroom):
    import torch
    from paper_2601_16986_amd import ckv
    rng = np.random.default_rng(L + cap)
    headroom = min(headroom, cap - 1)
    budgets = rng.integers(1, cap - headroom, (L, batch, hkv)).astype(np.int32) if cap - headroom > 1 else np.ones((L, batch, hkv), np.int32)
    args, more = (L, batch, hkv * 2, hkv, 128, cap, budgets), dict(t0=77, headroom=headroom, budget_max=cap - 1, prompt_len=300 if headroom else 0)
    arena = torch.full((ckv.arena_bytes(*args, **more),), 0xA7, dtype=torch.uint8, device="cuda:0")
    g = ckv.CrystalKV(*args, arena=arena, **more)
    assert np.array_equal(g.budgets(), budgets) and not g.lengths().any() and g.time() == 77 and g.status() == 0
    mseg, pool = (cap + 255) // 256, g.pool_slots // 256
    need = np.full(budgets.size, mseg) if headroom == 0 else np.minimum(mseg, (budgets.reshape(-1) + headroom + 255) // 256)
    first = np.concatenate([[0], np.cumsum(need)[:-1]])
    t = g.segment_table()
    assert np.array_equal(t["owned"], need)
    want = np.where(np.arange(mseg) < need[:, None], first[:, None] + np.arange(mseg), 0)
    assert np.array_equal(t["rows"], want)
    assert np.array_equal(t["spare"], np.arange(pool - 1, need.sum() - 1, -1))
    for x in (g.k_pool, g.v_pool, g.crf, g.tau, g.pos, g.flags):
        assert not bool(x.view(torch.uint8).any())
    e = g.export_unit(L - 1, batch - 1, hkv - 1)
    assert e["n"] == 0 and e["n_evicted"] == 0
    g.rebudget()                                             # no steps yet: nothing changes
    assert np.array_equal(g.budgets(), budgets)
    g.close()


@pytest.mark.parametrize("offset", [0, 4, 8, 12, 16])
def test_flags_anywhere(offset):
    """The flags need not lie at a multiple of 16 bytes; nothing around them is written."""
    import ctypes as C
    import torch
    from paper_2601_16986_amd import ckv
    g = ckv.CrystalKV(2, 2, 3, 3, 128, 288, np.full((2, 2, 3), 200, np.int32))
    S = g.pool_slots
    mem = torch.full((S + 64,), 0xA7, dtype=torch.uint8, device=g.device)
    buffers, budgets, ctx = ckv.Buffers.from_buffer_copy(g.buffers), g.budgets(), C.c_void_p()
    buffers.flags = mem.data_ptr() + offset
    g.close()
    rc = g.lib.ckv_init(C.byref(ctx), C.byref(g.layout), budgets.ctypes.data_as(C.c_void_p), C.byref(g.params), C.byref(buffers), g._stream())
    assert rc == ckv.OK
    torch.cuda.synchronize()
    g.lib.ckv_destroy(ctx)
    assert not bool(mem[offset:offset + S].any()) and bool((mem[:offset] == 0xA7).all()) and bool((mem[offset + S:] == 0xA7).all())


@pytest.mark.parametrize("lam,delta", [(0.5, 3), (0.9, 700), (0.9999, 60000), (1.0, 60000)])
@pytest.mark.parametrize("batch,hkv", [(1, 1), (4, 8)])
def test_decay_table(batch, hkv, lam, delta):
    import torch
    from paper_2601_16986_amd import ckv
    P = 40
    g = ckv.CrystalKV(1, batch, hkv, hkv, 128, 64, np.full((1, batch, hkv), 60, np.int32), lam=lam, top_p=1.0, t0=P - 1 + delta)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(2)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    g.load_prompt(0, rnd(batch, hkv, P, 128), rnd(batch, hkv, P, 128))
    g.decode_step(rnd(1, batch, hkv, 128), rnd(1, batch, hkv, 128), rnd(1, batch, hkv, 128), evict=False)
    want = np.float32(np.float32(np.power(np.float64(np.float32(lam)), float(delta))) + np.float32(1.0))
    for b in range(batch):
        e = g.export_unit(0, b, hkv - 1, with_kv=False)
        assert np.array_equal(e["crf"], np.append(np.full(P, want, np.float32), np.float32(1.0)))       # every entry is hit
    g.close()
