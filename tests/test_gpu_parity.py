"""GPU parity of the HIP path against the CPU oracle on small workloads: geometries,
call shapes (all layers / per layer), eviction on its own, re-budgeting, probe classes,
the attention-weighted variant, bf16 output, edge cases, determinism, graph replay."""
import numpy as np
import pytest

from tests import parity

pytestmark = pytest.mark.gpu


def _mods():
    from oracle import crystal_kv as ok
    from paper_2601_16986_amd import ckv, workloads as wl
    return ok, ckv, wl


def _pair(cfg, cap, budgets=None, stream=None, n_steps=None, load=True, path=0, **kw):
    ok, ckv, wl = _mods()
    st = stream if stream is not None else wl.make_stream(cfg, n_steps)
    budgets = wl.draw_budgets(cfg) if budgets is None else budgets
    okw = {k: v for k, v in kw.items() if k not in ("out_dtype", "headroom", "pool_slots", "prompt_len")}   # the rest is the GPU side's own business
    o = ok.CrystalKVOracle(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, budgets,
                           lam=cfg.lam, top_p=cfg.top_p, t0=cfg.prompt, budget_min=cfg.budget_min,
                           budget_max=cfg.budget_max, **okw)
    g = ckv.CrystalKV(cfg.n_layers, cfg.batch, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cap, budgets,
                      lam=cfg.lam, top_p=cfg.top_p, t0=cfg.prompt, budget_min=cfg.budget_min,
                      budget_max=cfg.budget_max, **kw)
    g.set_path(path)          # 1 = separate scan/finish kernels, 2 = fused per-unit kernel (3, 4: its two variants)
    if load and cfg.prompt > 0:
        for l in range(cfg.n_layers):
            o.load_prompt(l, st.prompt_k[l], st.prompt_v[l])
            g.load_prompt(l, st.prompt_k[l], st.prompt_v[l])
    return st, o, g


def _small(name, **kw):
    _, _, wl = _mods()
    base = dict(n_layers=2, batch=2, prompt=45, decode_steps=40, budget=56, budget_min=1, budget_max=95,
                adaptive=False, rebudget_interval=0)
    base.update(kw)
    return wl.scaled(wl.CONFIGS[name], **base)


PATHS = [1, 3, 4]  # separate kernels; fused kernel with 4 and with 2 wavefronts per unit


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("hq,hkv", [(2, 2), (8, 2), (10, 2), (14, 2), (16, 2), (6, 2)])
def test_lockstep_every_group_size(hq, hkv, path):
    """G = 1, 4, 5, 7, 8, 3 query heads per KV head; prompt length not a multiple of the 32-entry block;
    two layers and two sequences through the all-layers call; K/V rows checked after compaction."""
    cfg = _small("tiny", n_q_heads=hq, n_kv_heads=hkv, seed=77 + hq)
    st, o, g = _pair(cfg, cap=96, path=path)
    stats = parity.lockstep(g, o, st, cfg.decode_steps, check_kv_every=10)
    assert stats.resynced <= 2, stats.notes
    assert g.status() == 0 and g.time() == cfg.prompt + cfg.decode_steps
    g.close()


@pytest.mark.parametrize("path", PATHS)
def test_units_longer_than_a_chunk_and_ragged_tails(path):
    """Budgets 300..700 so units span several 256-entry chunks with ragged last blocks, and the
    scan's runs start in the middle of chunks; 7B-like group size 7."""
    _, _, wl = _mods()
    cfg = _small("qwen7b", n_layers=1, batch=3, n_q_heads=14, n_kv_heads=2, prompt=333, decode_steps=24,
                 budget=500, budget_min=300, budget_max=735, seed=5)
    budgets = np.array([[[300, 700], [513, 333], [641, 352]]], dtype=np.int32)
    st, o, g = _pair(cfg, cap=736, budgets=budgets, path=path)
    stats = parity.lockstep(g, o, st, cfg.decode_steps, check_kv_every=8)
    assert stats.resynced <= 2, stats.notes
    assert np.array_equal(g.lengths(), o.lengths())
    g.close()


@pytest.mark.parametrize("path", [3, 4])
def test_fused_kernel_with_logits_spilling_out_of_lds(path):
    """A unit of ~3000 entries with 8 query heads per KV head needs 96 KB of logits: more than the fused
    kernel's LDS tile, so the logits of its last blocks take the global-memory route; a second, small
    unit in the same call stays resident.  Also exercises several blocks per wavefront."""
    _, _, wl = _mods()
    cfg = _small("qwen7b", n_layers=1, batch=1, n_q_heads=16, n_kv_heads=2, prompt=2890, decode_steps=6,
                 budget=1800, budget_min=600, budget_max=3071, seed=15)
    budgets = np.array([[[2900, 700]]], dtype=np.int32)
    st, o, g = _pair(cfg, cap=3072, budgets=budgets, path=path)
    avail, lds_main = g.path_info()
    assert avail and 3000 * 8 * 4 > lds_main
    stats = parity.lockstep(g, o, st, cfg.decode_steps, check_kv_every=3)
    assert stats.resynced <= 1, stats.notes
    g.close()


@pytest.mark.parametrize("path", [3, 4])
@pytest.mark.parametrize("hq", [2, 10, 16])
def test_new_entry_alone_in_its_block(path, hq):
    """Budgets that are multiples of 32: in the steady state every unit holds B + 1 entries while it attends, the
    new one alone in the last block.  The fused kernel then does not stream that block: the entry joins the
    merge as a state of its own (logits and value row from the step's inputs).  From an empty
    cache (the first entry is alone too) through growth over block boundaries into the steady state."""
    cfg = _small("qwen14b", n_layers=2, batch=2, n_q_heads=hq, n_kv_heads=2, prompt=0, decode_steps=150,
                 budget=64, budget_min=1, budget_max=128, seed=37)
    budgets = np.array([[[64, 96], [32, 128]], [[64, 64], [96, 32]]], dtype=np.int32)
    st, o, g = _pair(cfg, cap=160, budgets=budgets, path=path, load=False)
    stats = parity.lockstep(g, o, st, cfg.decode_steps, check_kv_every=25)
    assert stats.resynced <= 2, stats.notes
    assert np.array_equal(g.lengths(), budgets) and g.status() == 0
    g.close()


@pytest.mark.parametrize("path", [3, 4])
def test_new_entry_alone_in_a_block_whose_logits_live_in_global_memory(path):
    """As above for a unit too long for the LDS tile: the lone entry's logits take the global-memory route."""
    cfg = _small("qwen7b", n_layers=1, batch=1, n_q_heads=16, n_kv_heads=2, prompt=2890, decode_steps=6,
                 budget=1800, budget_min=600, budget_max=3071, seed=15)
    budgets = np.array([[[2880, 704]]], dtype=np.int32)
    st, o, g = _pair(cfg, cap=3072, budgets=budgets, path=path)
    _, lds_main = g.path_info()
    assert 2881 * 8 * 4 > lds_main
    stats = parity.lockstep(g, o, st, cfg.decode_steps, check_kv_every=3)
    assert stats.resynced <= 1, stats.notes
    assert g.lengths().tolist() == [[[2880, 704]]]
    g.close()


@pytest.mark.parametrize("path,n_big", [(3, 4500), (3, 8300), (4, 2500), (4, 4400)])
def test_fused_kernel_large_units(path, n_big):
    """Units beyond 16 entries per thread: 17..32 per thread keep the weights in registers with the per-entry
    state loaded in chunks, more than 32 per thread go through the LDS-resident generic path.  (Path 3 has 256
    threads per unit, path 4 has 128.)  A small unit shares the call."""
    cfg = _small("qwen7b", n_layers=1, batch=1, n_q_heads=4, n_kv_heads=2, prompt=n_big - 10, decode_steps=4,
                 budget=n_big // 2, budget_min=200, budget_max=n_big + 60, seed=23)
    budgets = np.array([[[n_big, 300]]], dtype=np.int32)
    cap = (n_big + 64 + 31) // 32 * 32
    st, o, g = _pair(cfg, cap=cap, budgets=budgets, path=path)
    waves, _ = g.path_info()
    assert waves == (2 if path == 4 else 4)
    stats = parity.lockstep(g, o, st, cfg.decode_steps, check_kv_every=2)
    assert stats.resynced <= 1, stats.notes
    assert np.array_equal(g.lengths(), o.lengths())
    g.close()


@pytest.mark.parametrize("defer", [False, True])
def test_units_at_the_maximum_capacity(defer):
    """cap = 32768 slots, the most the layout admits: one unit stays full (one entry evicted per step once
    its budget is reached), the other is cut from 32700 entries to a budget of 16000 in its first step (the
    general select and compaction at full size) and then scanned as 63 chunks.  Single-layer calls, plain
    and with deferred bookkeeping (the scan then merges up to 129 runs per unit)."""
    cfg = _small("qwen7b", n_layers=1, batch=1, n_q_heads=4, n_kv_heads=2, prompt=32700, decode_steps=8,
                 budget=32704, budget_min=200, budget_max=32767, seed=29)
    budgets = np.array([[[32704, 16000]]], dtype=np.int32)
    st, o, g = _pair(cfg, cap=32768, budgets=budgets)
    stats = parity.LockstepStats()
    for s in range(cfg.decode_steps):
        ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
        out = g.decode_step(st.q[s, 0], st.k_new[s, 0], st.v_new[s, 0], layer=0, defer=defer).cpu().numpy()[None]
        assert parity.out_error(out, ref) <= parity.OUT_TOL
        for key, rec in recs.items():
            parity.compare_unit(g, o, key, rec, stats, check_kv=(s in (0, 7)))
    assert stats.resynced <= 1, stats.notes
    assert g.status() == 0 and np.array_equal(g.lengths(), o.lengths())
    assert g.lengths().tolist() == [[[32704, 16000]]]
    g.close()


@pytest.mark.parametrize("path", PATHS)
def test_attention_only_steps(path):
    """CKV_ATTENTION_ONLY (the FullKV baseline): outputs as the oracle's attention over the growing cache;
    scores and taus of the old entries stay as loaded, the new entries arrive with CRF 0 and tau = pos = t,
    nothing is evicted; combining it with eviction is refused."""
    _, ckv, _ = _mods()
    # prompt 60: the caches grow across a block boundary (64), where the new entry is alone in its block
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, prompt=60, decode_steps=12, budget=60, seed=31)
    st, o, g = _pair(cfg, cap=128, path=path)
    before = {key: g.export_unit(*key, with_kv=False) for key in o.units}
    for s in range(cfg.decode_steps):
        ref, _ = o.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False)
        out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s], attention_only=True).cpu().numpy()
        assert parity.out_error(out, ref) <= parity.OUT_TOL
    assert g.status() == 0 and g.time() == cfg.prompt + cfg.decode_steps
    for key, b in before.items():
        e = g.export_unit(*key, with_kv=False)
        n0 = b["n"]
        assert e["n"] == n0 + cfg.decode_steps
        assert np.array_equal(e["crf"][:n0], b["crf"]) and np.array_equal(e["tau"][:n0], b["tau"])
        assert np.array_equal(e["pos"][:n0], b["pos"])
        new_t = np.arange(cfg.prompt, cfg.prompt + cfg.decode_steps)
        assert np.array_equal(e["pos"][n0:], new_t) and np.array_equal(e["tau"][n0:], new_t)
        assert np.all(e["crf"][n0:] == 0)
    with pytest.raises(ckv.CkvError) as err:
        # both flags at once: refused during argument validation, before any pointer is looked at
        g._check(g.lib.ckv_decode_step(g.ctx, -1, 1, 1, 1, 1, ckv.FUSE_EVICT | ckv.ATTENTION_ONLY, None))
    assert err.value.code == ckv.EINVAL
    g.close()


def test_path_selection_api():
    """Mode 0 picks the fused kernel only for enough units; 1 forces the separate kernels; 2-4 the fused
    variants; other values are refused."""
    _, ckv, _ = _mods()
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, seed=2)
    st, o, g = _pair(cfg, cap=96)
    assert g.path_info()[0] == 0                       # 4 units: separate kernels by default
    for mode, waves in ((1, 0), (2, 4), (3, 4), (4, 2)):
        g.set_path(mode)
        assert g.path_info()[0] == waves
    for bad in (-1, 5):
        with pytest.raises(ckv.CkvError) as e:
            g.set_path(bad)
        assert e.value.code == ckv.EINVAL
    g.close()


@pytest.mark.parametrize("hq,hkv,P,W,lam,L", [(8, 2, 45, 9, 0.5, 2), (10, 2, 70, 32, 0.7, 2), (2, 2, 33, 1, 0.5, 2), (14, 2, 300, 17, 0.97, 2),
                                               (16, 2, 64, 64, 0.0, 2), (8, 2, 610, 40, 1.0, 2), (10, 2, 4105, 20, 0.7, 2),
                                               (8, 2, 9000, 6, 0.5, 2), (2, 2, 16390, 21, 0.5, 2),
                                               (10, 2, 300, 40, 0.7, 24), (8, 2, 8300, 10, 0.5, 12), (4, 2, 530, 64, 0.9, 36)])
def test_seed_prompt_matches_oracle_then_decodes(hq, hkv, P, W, lam, L):
    """Scores of a loaded prompt from its last W queries (all of it for W = P, one query for W = 1; prompts
    shorter and longer than a 256-entry chunk, not multiples of the 32-entry block; windows that are and are not
    multiples of the number of queries a pass over the keys takes, floor(16 / G) = 4, 3, 16, 2, 2; windows across
    the prompt lengths at which the replay's bookkeeping changes its code path, 8, 16 and 32 entries per thread
    of a 512-thread workgroup; contexts of two layers, whose replay takes one tile of queries at a time in its own
    buffers, and of more, whose replay takes batches of 6, 2 and 3 tiles in the decode workspace): CRF bits and
    tau of every entry equal the oracle's; the time and the Alg. 2
    window are untouched (the decode steps and the re-allocation that follow match the oracle as after any load)."""
    cfg = _small("tiny", n_layers=L, batch=2 if P < 4000 else 1, n_q_heads=hq, n_kv_heads=hkv, prompt=P, decode_steps=max(W, 10),
                 lam=lam, budget=P + 5, budget_min=8, budget_max=P + 30, seed=300 + W)
    st, o, g = _pair(cfg, cap=(P + 64) // 32 * 32)
    total0 = o.budgets().sum(axis=(0, 2))
    resync = 0
    for l in range(cfg.n_layers):
        q_obs = st.q[:W, l]
        decs = o.seed_prompt(l, q_obs)
        g.seed_prompt(l, q_obs)
        for key, dl in decs.items():
            u, e = o.units[key], g.export_unit(*key)
            assert e["n"] == P and np.array_equal(e["pos"], u.pos)
            if np.array_equal(e["crf"].view(np.uint32), u.crf.view(np.uint32)) and np.array_equal(e["tau"], u.tau):
                continue
            # only entries at the edge of a sub-margin decision of the window may carry other scores
            sub = [d for d in dl if min(d.sum_margin, d.edge_gap) < parity.MARGIN_TOL]
            may = set(i for d in sub for i in parity.edge_entries(d))
            differ = set(np.nonzero((e["crf"].view(np.uint32) != u.crf.view(np.uint32)) | (e["tau"] != u.tau))[0].tolist())
            assert sub and differ <= may, (key, sorted(differ), sorted(may))
            parity.sync_unit_to_gpu(g, o, key)
            resync += 1
    assert resync <= 1 + len(o.units) * W // 4000          # sub-margin decisions are rare, not absent
    assert g.time() == P and g.status() == 0
    stats = parity.lockstep(g, o, st, 10, check_kv_every=5)
    assert stats.resynced <= 1, stats.notes
    if resync == 0 and stats.resynced == 0:
        nb = o.rebudget()
        g.rebudget()
        assert np.array_equal(g.budgets(), nb) and np.array_equal(nb.sum(axis=(0, 2)), total0)
    g.close()


@pytest.mark.parametrize("L,P,W", [(1, 77, 12), (24, 300, 20)])
def test_seed_prompt_with_the_attention_weighted_reward(L, P, W):
    """The labelled reward variant through the prompt replay (one tile of queries at a time in a context of one
    layer, a batch of several tiles in one of 24): every entry's score accumulates its mean weights (within
    1e-5 relative of the oracle's, as for decode steps), tau = P - 1 for every entry."""
    ok, _, _ = _mods()
    cfg = _small("tiny", n_layers=L, n_q_heads=10, n_kv_heads=2, prompt=P, decode_steps=W, budget=P + 5, budget_min=8,
                 budget_max=P + 30, seed=91)
    st, o, g = _pair(cfg, cap=(P + 64) // 32 * 32, reward_mode=ok.REWARD_ATTN_WEIGHTED)
    o.seed_prompt(0, st.q[:W, 0])
    g.seed_prompt(0, st.q[:W, 0])
    for key, u in o.units.items():
        e = g.export_unit(*key, with_kv=False)
        assert np.array_equal(e["pos"], u.pos) and np.array_equal(e["tau"], u.tau)
        assert np.allclose(e["crf"], u.crf, rtol=1e-5, atol=1e-30)
        assert np.all(u.tau == P - 1)
    g.close()


def test_seed_prompt_argument_and_state_errors():
    _, ckv, _ = _mods()
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, seed=5)
    st, o, g = _pair(cfg, cap=96)
    P = cfg.prompt
    with pytest.raises(ckv.CkvError) as e:
        g.seed_prompt(0, st.q[:P + 1, 0].repeat(2, axis=0)[:P + 1])       # W > P
    assert e.value.code == ckv.EINVAL
    with pytest.raises(ckv.CkvError) as e:
        g.seed_prompt(7, st.q[:4, 0])
    assert e.value.code == ckv.EINVAL
    g.seed_prompt(0, st.q[:4, 0])                                          # twice is allowed: same result
    g.seed_prompt(0, st.q[:4, 0])
    g.decode_step(st.q[0], st.k_new[0], st.v_new[0])
    with pytest.raises(ckv.CkvError) as e:
        g.seed_prompt(0, st.q[:4, 0])                                      # the layer has been stepped
    assert e.value.code == ckv.ESTATE
    g.close()


def test_lambda_top_p_sweep_script_runs(capsys, monkeypatch):
    """The hyper-parameter sweep (a user-facing script on top of the binding) at a toy size: recalls are
    fractions, and the recommended setting keeps more of the heavy positions than a sliding window."""
    import json
    import sys
    from paper_2601_16986_amd import sweep
    monkeypatch.setattr(sys, "argv", ["sweep", "--tokens", "224", "--prompt", "32", "--budget", "40"])
    sweep.main()
    res = json.loads(capsys.readouterr().out.strip().splitlines()[-1])["results"]
    assert len(res) == 27 and all(0.0 <= r["heavy_recall"] <= 1.0 and 0.0 <= r["crystal_recall"] <= 1.0 for r in res)
    rec = next(r for r in res if r["name"] == "recent")
    best = next(r for r in res if r["name"] is None and r["lambda"] == 0.5 and r["top_p"] == 0.9)
    sink = next(r for r in res if r["name"] == "sink + recent")
    assert best["heavy_recall"] >= rec["heavy_recall"] and best["heavy_recall"] >= sink["heavy_recall"]


def test_per_layer_calls():
    """The shape a real model imposes: one call per layer, t advancing after the last layer."""
    cfg = _small("llama8b", n_layers=3, n_q_heads=8, n_kv_heads=2, seed=11)
    st, o, g = _pair(cfg, cap=96)
    stats = parity.LockstepStats()
    import torch
    for s in range(20):
        ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
        outs = [g.decode_step(st.q[s, l], st.k_new[s, l], st.v_new[s, l], layer=l) for l in range(cfg.n_layers)]
        assert g.time() == cfg.prompt + s + 1
        out = torch.stack(outs).cpu().numpy()
        assert parity.out_error(out, ref) <= parity.OUT_TOL
        for key, rec in recs.items():
            parity.compare_unit(g, o, key, rec, stats)
    assert stats.resynced <= 2
    # layers out of order are refused, and so is a second prompt for a layer that holds entries
    _, ckv, _ = _mods()
    with pytest.raises(ckv.CkvError) as e1:
        g.decode_step(st.q[20, 1], st.k_new[20, 1], st.v_new[20, 1], layer=1)
    assert e1.value.code == ckv.ESTATE
    with pytest.raises(ckv.CkvError) as e2:
        g.load_prompt(0, st.prompt_k[0], st.prompt_v[0])
    assert e2.value.code == ckv.ESTATE
    g.close()


@pytest.mark.parametrize("path", [0, 3])
def test_per_layer_calls_of_layers_with_a_unit_per_workgroup_take_the_fused_kernel(path):
    """A layer of 512 units (batch 64 x 8 KV heads) fills the fused kernel's grid, so single-layer steps run
    it on the layer's part of the schedule, with inputs and output addressed relative to the layer; all-layers
    steps in between use the budget-ordered schedule again.  Lock-step with the oracle throughout."""
    import torch
    cfg = _small("llama8b", n_layers=2, batch=64, n_q_heads=16, n_kv_heads=8, prompt=20, decode_steps=14,
                 budget=24, budget_min=1, budget_max=63, seed=43)
    st, o, g = _pair(cfg, cap=64, path=path)
    waves, _ = g.path_info()
    assert waves == 4
    stats = parity.LockstepStats()
    for s in range(cfg.decode_steps):
        ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
        if s % 5 == 3:
            out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s]).cpu().numpy()
        else:
            out = torch.stack([g.decode_step(st.q[s, l], st.k_new[s, l], st.v_new[s, l], layer=l)
                               for l in range(cfg.n_layers)]).cpu().numpy()
        assert parity.out_error(out, ref) <= parity.OUT_TOL
        assert g.time() == cfg.prompt + s + 1
        for key, rec in recs.items():
            parity.compare_unit(g, o, key, rec, stats)
    assert stats.resynced <= 3, stats.notes
    assert g.status() == 0 and np.array_equal(g.lengths(), o.lengths())
    g.close()


@pytest.mark.parametrize("prompt,bf16", [(8, False), (333, False), (2100, False), (333, True)])
def test_scan_that_merges_its_own_partials_gives_the_bits_of_the_finish_kernel(prompt, bf16):
    """Attention-only steps get their output from the scan itself (the wavefront that publishes a unit's last
    run merges the unit); plain steps get it from the finish kernel.  Same cache, same queries: the same bits,
    and the oracle's values, for units of one block (several units per wavefront), of two or three runs, and of
    more runs than one batch of the merge holds.  Steps with deferred bookkeeping come from the single-layer
    scan, which cuts the units differently (other rounding): the oracle's values, and the plain step's scores."""
    import torch
    cfg = _small("qwen14b", n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, prompt=prompt, decode_steps=10,
                 budget=prompt + 20, budget_min=1, budget_max=prompt + 20, seed=17)
    cap = (prompt + 21 + 31) // 32 * 32
    _, ckv, wl = _mods()
    kw = dict(out_dtype=ckv.BF16) if bf16 else {}
    st, o, g_plain = _pair(cfg, cap=cap, path=1, **kw)
    _, _, g_attn = _pair(cfg, cap=cap, stream=st, path=1, **kw)
    _, _, g_defer = _pair(cfg, cap=cap, stream=st, path=1, **kw)
    _, _, g_all = _pair(cfg, cap=cap, stream=st, path=1, **kw)
    for s in range(cfg.decode_steps):
        ref, _ = o.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False)
        layers = range(cfg.n_layers)
        a = torch.stack([g_plain.decode_step(st.q[s, l], st.k_new[s, l], st.v_new[s, l], layer=l, evict=False) for l in layers])
        b = torch.stack([g_attn.decode_step(st.q[s, l], st.k_new[s, l], st.v_new[s, l], layer=l, attention_only=True)
                         for l in layers])
        c = torch.stack([g_defer.decode_step(st.q[s, l], st.k_new[s, l], st.v_new[s, l], layer=l, evict=False, defer=True)
                         for l in layers])
        d = g_all.decode_step(st.q[s], st.k_new[s], st.v_new[s], attention_only=True)
        if bf16:                                                             # within one bf16 ulp of the rounded reference
            ref16 = wl.bf16_round(ref.astype(np.float32))
            ulp = np.maximum(np.abs(ref16), 2.0 ** -126) * 2.0 ** -7
            for x in (a, c, d):
                assert np.all(np.abs(x.float().cpu().numpy() - ref16) <= ulp + parity.OUT_TOL * 1e-2 * np.abs(ref).max())
        else:
            assert parity.out_error(a.cpu().numpy(), ref) <= parity.OUT_TOL
            assert parity.out_error(c.cpu().numpy(), ref) <= parity.OUT_TOL  # other shares, other rounding
            assert parity.out_error(d.cpu().numpy(), ref) <= parity.OUT_TOL
        assert torch.equal(a, b), ("attention only", s, float((a.float() - b.float()).abs().max()))
        for g in (g_plain, g_attn, g_defer, g_all):
            assert g.time() == cfg.prompt + s + 1
    g_defer.join()
    # the deferred bookkeeping took the same decisions as the plain step's: the same scores, bit for bit
    for key in o.units:
        e1, e2 = g_plain.export_unit(*key, with_kv=False), g_defer.export_unit(*key, with_kv=False)
        assert np.array_equal(e1["crf"], e2["crf"]) and np.array_equal(e1["tau"], e2["tau"])
    for g in (g_plain, g_attn, g_defer, g_all):
        assert g.status() == 0
        g.close()


@pytest.mark.parametrize("hq,hkv,cap", [(8, 2, 96), (10, 2, 416)])
def test_per_layer_calls_with_deferred_bookkeeping(hq, hkv, cap):
    """Single-layer steps whose scores and evictions run on the context's own stream (CKV_DEFER_BOOKKEEPING):
    the attention output is on the caller's stream at once, the state equals the oracle's after every step,
    through evictions, a re-allocation of the budgets (which has to order itself after the bookkeeping in
    flight) and all-layers steps mixed in."""
    big = cap > 96
    cfg = _small("llama8b", n_layers=4, n_q_heads=hq, n_kv_heads=hkv, seed=13, **(dict(prompt=330, budget=340, budget_min=64,
                                                                                budget_max=400) if big else {}))
    st, o, g = _pair(cfg, cap=cap)
    stats = parity.LockstepStats()
    import torch
    for s in range(24):
        ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
        if s % 8 == 5:                               # an all-layers step in between: it waits for what is in flight
            out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s]).cpu().numpy()
        else:
            outs = [g.decode_step(st.q[s, l], st.k_new[s, l], st.v_new[s, l], layer=l, defer=True) for l in range(cfg.n_layers)]
            out = torch.stack(outs).cpu().numpy()
        assert parity.out_error(out, ref) <= parity.OUT_TOL
        assert g.time() == cfg.prompt + s + 1
        for key, rec in recs.items():
            parity.compare_unit(g, o, key, rec, stats)
        if s == 11 and stats.resynced == 0:
            nb = o.rebudget()
            g.rebudget()
            assert np.array_equal(g.budgets(), nb)
    assert stats.resynced <= 2, stats.notes
    _, ckv, _ = _mods()
    for bad in dict(layer=-1, defer=True), dict(layer=0, defer=True, attention_only=True, evict=False):
        with pytest.raises(ckv.CkvError) as e:
            g.decode_step(st.q[24] if bad["layer"] == -1 else st.q[24, 0], st.k_new[24] if bad["layer"] == -1 else st.k_new[24, 0],
                          st.v_new[24] if bad["layer"] == -1 else st.v_new[24, 0], **bad)
        assert e.value.code == ckv.EINVAL
    g.close()


def test_hip_graph_of_deferred_per_layer_steps_matches_eager():
    """Two decode steps of three single-layer calls each, with deferred bookkeeping, captured into one HIP graph
    (the context's stream takes part in the capture and rejoins it through join()) and replayed three times
    with eager work in between: outputs and final state equal those of the same calls made eagerly on another context."""
    import torch
    cfg = _small("tiny", n_layers=3, n_q_heads=8, n_kv_heads=2, decode_steps=8, seed=72)
    st, o, g = _pair(cfg, cap=96)
    _, _, g2 = _pair(cfg, cap=96)
    dev = g.device
    as_dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev).to(torch.bfloat16)
    q, k, v = as_dev(st.q), as_dev(st.k_new), as_dev(st.v_new)
    eager = [torch.stack([g2.decode_step(q[s, l], k[s, l], v[s, l], layer=l, defer=True) for l in range(3)]).clone() for s in range(6)]
    g2.join()
    torch.cuda.synchronize()
    sq, sk, sv = q[:2].clone(), k[:2].clone(), v[:2].clone()
    outs = [[torch.empty_like(eager[0][0]) for _ in range(3)] for _ in range(2)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for i in range(2):
            for l in range(3):
                g.decode_step(sq[i, l], sk[i, l], sv[i, l], layer=l, out=outs[i][l], defer=True)
        g.join()
    for rep in range(3):
        sq.copy_(q[2 * rep:2 * rep + 2]); sk.copy_(k[2 * rep:2 * rep + 2]); sv.copy_(v[2 * rep:2 * rep + 2])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.isfinite((torch.randn(1 << 16, device=dev) * 2).sum().item())
        for i in range(2):
            for l in range(3):
                assert torch.equal(outs[i][l], eager[2 * rep + i][l]), (rep, i, l)
    assert g.time() == cfg.prompt + 6
    for key in o.units:
        a, b = g.export_unit(*key), g2.export_unit(*key)
        for f in ("pos", "crf", "tau", "flags"):
            assert np.array_equal(a[f], b[f])
    g.close(); g2.close()


@pytest.mark.parametrize("path", PATHS)
def test_eviction_on_its_own_and_after_a_budget_cut(path):
    """Steps without eviction let caches grow past their budgets; ckv_evict then removes many entries
    at once (the general select + compaction path), also after budgets were cut."""
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, prompt=40, decode_steps=60, budget=50, seed=3)
    st, o, g = _pair(cfg, cap=128, path=path)
    stats = parity.LockstepStats()
    s = 0
    for rnd in range(3):
        for _ in range(12):
            ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False)
            out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False).cpu().numpy()
            assert parity.out_error(out, ref) <= parity.OUT_TOL
            for key, rec in recs.items():
                parity.compare_unit(g, o, key, rec, stats, evicting=False)
            s += 1
        if rnd == 1:                      # cut budgets: k becomes large
            newb = np.full((cfg.n_layers, cfg.batch, cfg.n_kv_heads), 23, dtype=np.int32)
            newb[0, 0, 0] = 7
            g.set_budgets(newb)
            for key, u in o.units.items():
                u.budget = int(newb[key])
        ev = o.evict()
        g.evict()
        for key in o.units:
            e = g.export_unit(*key)
            u = o.units[key]
            assert e["n"] == u.n == u.budget
            assert np.array_equal(e["evicted_pos"], ev[key])
            assert np.all(e["evicted_flags"] == 2)
            og, oo = np.argsort(e["pos"]), np.argsort(u.pos)
            assert np.array_equal(e["pos"][og], u.pos[oo])
            assert np.array_equal(e["crf"][og], u.crf[oo]) and np.array_equal(e["tau"][og], u.tau[oo])
            assert np.array_equal(e["K"][og], u.K[oo].astype(np.float32))
            assert np.array_equal(e["V"][og], u.V[oo].astype(np.float32))
    assert stats.resynced <= 2
    g.close()


@pytest.mark.parametrize("every,n_sink", [(1, 4), (7, 4), (5, 0), (9, 30)])
def test_sink_plus_recent_window_policy_matches_oracle(every, n_sink):
    """The comparison policy of Sec. 2.3 (initial + most recent tokens) on the same caches: steps without
    eviction, then ckv_evict_window every few steps.  Evicted positions, survivors with their scores, taus,
    keys and values as the oracle's; with n_sink above the budget of one unit the lowest sinks stay."""
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, prompt=40, decode_steps=36, budget=26, seed=23)
    budgets = np.full((cfg.n_layers, cfg.batch, cfg.n_kv_heads), 26, dtype=np.int32)
    budgets[1, 0, 1] = 9
    st, o, g = _pair(cfg, cap=96, budgets=budgets)
    stats = parity.LockstepStats()

    def evict_and_compare():
        ev = o.evict_window(n_sink)
        g.evict_window(n_sink)
        for key in o.units:
            e = g.export_unit(*key)
            u = o.units[key]
            assert e["n"] == u.n == u.budget
            assert np.array_equal(e["evicted_pos"], ev[key])
            assert np.all(e["evicted_flags"] == 2)
            og, oo = np.argsort(e["pos"]), np.argsort(u.pos)
            assert np.array_equal(e["pos"][og], u.pos[oo])
            assert np.array_equal(e["crf"][og], u.crf[oo]) and np.array_equal(e["tau"][og], u.tau[oo])
            assert np.array_equal(e["K"][og], u.K[oo].astype(np.float32))
            assert np.array_equal(e["V"][og], u.V[oo].astype(np.float32))

    evict_and_compare()                                # the prompt (40 entries) down to the budgets
    for s in range(cfg.decode_steps):
        ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False)
        out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False).cpu().numpy()
        assert parity.out_error(out, ref) <= parity.OUT_TOL
        for key, rec in recs.items():
            parity.compare_unit(g, o, key, rec, stats, evicting=False)
        if (s + 1) % every == 0:
            evict_and_compare()
    assert stats.resynced <= 2, stats.notes
    if every == 1 and n_sink == 4:                     # the sliding window itself
        t = cfg.prompt + cfg.decode_steps - 1
        e = g.export_unit(0, 0, 0, with_kv=False)
        assert sorted(e["pos"].tolist()) == list(range(4)) + list(range(t - 21, t + 1))
    _, ckv, _ = _mods()
    with pytest.raises(ckv.CkvError) as err:
        g.evict_window(-1)
    assert err.value.code == ckv.EINVAL
    g.close()


@pytest.mark.parametrize("path", PATHS)
def test_rebudget_matches_alg2_oracle(path):
    """Alg. 2 on the device: budgets bit-identical to the oracle's, totals conserved, bounds kept;
    the next fused eviction brings the caches down to the new budgets."""
    _, _, wl = _mods()
    cfg = wl.scaled(wl.CONFIGS["qwen14b"], n_layers=3, batch=2, n_q_heads=10, n_kv_heads=2, prompt=70,
                    decode_steps=48, budget=64, budget_min=16, budget_max=120, seed=9)
    st, o, g = _pair(cfg, cap=160, path=path)
    total0 = o.budgets().sum(axis=(0, 2))
    stats = parity.LockstepStats()
    s = 0
    for rnd in range(3):
        for _ in range(12):
            ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
            g.decode_step(st.q[s], st.k_new[s], st.v_new[s])
            for key, rec in recs.items():
                parity.compare_unit(g, o, key, rec, stats)
            s += 1
        assert stats.resynced == 0, "window sums are only comparable without re-synchronised units"
        nb = o.rebudget()
        g.rebudget()
        gb = g.budgets()
        assert np.array_equal(gb, nb), (gb - nb)
        assert np.array_equal(gb.sum(axis=(0, 2)), total0)
        assert gb.min() >= cfg.budget_min and gb.max() <= cfg.budget_max
        assert not np.array_equal(gb, wl.draw_budgets(cfg)) or rnd > 0
    g.close()


def test_probe_classes():
    """Sec. 3 classes under the answer-probe query: counts floor(0.3 n) and the same entries as the oracle."""
    _, _, wl = _mods()
    cfg = wl.scaled(wl.CONFIGS["tiny"], decode_steps=100)
    st, o, g = _pair(cfg, cap=160)
    parity.lockstep(g, o, st, 100)
    cls = g.probe(0, st.probe_q[0]).cpu().numpy()
    t_before = g.time()
    for (l, b, h), u in o.units.items():
        ref, abar = o.probe((l, b, h), st.probe_q[l, b, h * o.G:(h + 1) * o.G])
        e = g.export_unit(l, b, h, with_kv=False)
        got = cls[b, h, :e["n"]]
        by_pos_g = dict(zip(e["pos"].tolist(), got.tolist()))
        by_pos_o = dict(zip(u.pos.tolist(), ref.tolist()))
        # entries whose weight is within rounding of a class boundary may fall either way
        srt = np.sort(abar)
        k = (3 * u.n) // 10
        edges = [srt[k - 1], srt[k], srt[u.n - k - 1], srt[u.n - k]]
        for p_, a in zip(u.pos.tolist(), abar.tolist()):
            if by_pos_g[p_] != by_pos_o[p_]:
                assert min(abs(a - x) / x for x in edges) < 1e-5, (p_, a)
        assert (got == 2).sum() == k and (got == 0).sum() == k
    assert g.time() == t_before and np.array_equal(g.lengths(), o.lengths())
    g.close()


@pytest.mark.parametrize("path", PATHS)
def test_attention_weighted_reward_variant(path):
    """reward = mean attention weight (labelled variant): scores within 1e-5 relative of the oracle's,
    same evictions unless the last kept and first evicted scores are closer than that."""
    ok, ckv, _ = _mods()
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, decode_steps=30, seed=21)
    st, o, g = _pair(cfg, cap=96, reward_mode=ok.REWARD_ATTN_WEIGHTED, path=path)
    for s in range(cfg.decode_steps):
        ref, recs = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
        out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s]).cpu().numpy()
        assert parity.out_error(out, ref) <= parity.OUT_TOL
        for key, rec in recs.items():
            u = o.units[key]
            e = g.export_unit(*key, with_kv=False)
            if set(e["pos"].tolist()) != set(u.pos.tolist()):
                assert rec.evict_gap < 1e-5, (key, s, rec.evict_gap)
                parity.sync_unit_to_gpu(g, o, key)
                continue
            og, oo = np.argsort(e["pos"]), np.argsort(u.pos)
            assert np.allclose(e["crf"][og], u.crf[oo], rtol=1e-5, atol=1e-30)
            assert np.array_equal(e["tau"][og], u.tau[oo])
            parity.sync_unit_to_gpu(g, o, key)        # keep both sides on the oracle's exact scores
    g.close()


@pytest.mark.parametrize("path", PATHS)
def test_bf16_output(path):
    """out_dtype bf16: within one bf16 ulp of the oracle's output rounded to bf16."""
    _, ckv, wl = _mods()
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, decode_steps=8, seed=31)
    st, o, g = _pair(cfg, cap=96, out_dtype=ckv.BF16, path=path)
    for s in range(cfg.decode_steps):
        ref, _ = o.decode_step(st.q[s], st.k_new[s], st.v_new[s])
        out = g.decode_step(st.q[s], st.k_new[s], st.v_new[s]).float().cpu().numpy()
        ref16 = wl.bf16_round(ref.astype(np.float32))
        ulp = np.maximum(np.abs(ref16), 2.0 ** -126) * 2.0 ** -7
        assert np.all(np.abs(out - ref16) <= ulp + parity.OUT_TOL * 1e-2 * np.abs(ref).max())
    g.close()


@pytest.mark.parametrize("path", PATHS)
@pytest.mark.parametrize("lam,top_p", [(0.0, 0.9), (1.0, 0.9), (0.7, 1.0), (0.5, 0.5), (0.99, 0.9)])
def test_parameter_corners(lam, top_p, path):
    """lambda = 0 (LRU) and 1 (LFU), p >= 1 (every entry hit), a low p, and a decay table of ~9000 entries."""
    _, _, wl = _mods()
    cfg = wl.scaled(_small("tiny", n_q_heads=8, n_kv_heads=2, decode_steps=30, seed=41), lam=lam, top_p=top_p)
    st, o, g = _pair(cfg, cap=96, path=path)
    stats = parity.lockstep(g, o, st, cfg.decode_steps)
    assert stats.resynced <= 2, stats.notes
    if top_p >= 1.0:
        for key in o.units:
            assert np.all(g.export_unit(*key, with_kv=False)["flags"] & 1)
    g.close()


def test_empty_start_capacity_and_argument_errors():
    ok, ckv, wl = _mods()
    cfg = _small("tiny", n_layers=1, batch=1, n_q_heads=8, n_kv_heads=2, prompt=0, decode_steps=40, budget=20,
                 budget_max=31, seed=51)
    st, o, g = _pair(cfg, cap=32, load=False)
    # no prompt: the first step attends over the new entry alone
    stats = parity.lockstep(g, o, st, 10)
    assert np.array_equal(g.lengths(), o.lengths()) and o.lengths().max() == 10
    # without eviction the caches fill; an append to a full unit is reported, nothing is written out of bounds
    for s in range(10, 36):
        g.decode_step(st.q[s], st.k_new[s], st.v_new[s], evict=False)
    assert g.status() == ckv.ECAPACITY and g.status() == 0      # reported once, then cleared
    assert g.lengths().max() == 32
    # argument errors
    with pytest.raises(ckv.CkvError) as e1:
        g.decode_step(st.q[0, 0], st.k_new[0, 0], st.v_new[0, 0], layer=5)
    assert e1.value.code == ckv.EINVAL
    with pytest.raises(ckv.CkvError) as e2:
        g.load_prompt(0, np.zeros((1, 2, 4, 128), np.float32), np.zeros((1, 2, 4, 128), np.float32))
    assert e2.value.code == ckv.EINVAL                          # a prompt longer than t0
    with pytest.raises(ckv.CkvError):
        g.set_budgets(np.full((1, 1, 2), 32))                   # budget must stay below cap
    with pytest.raises(ckv.CkvError):
        ckv.CrystalKV(1, 1, 8, 2, 64, 32, np.full((1, 1, 2), 8))   # head_dim 64
    g.close()


@pytest.mark.parametrize("path", PATHS)
def test_runs_are_deterministic(path):
    """Same inputs twice: outputs and state bit-identical (no atomics on floating-point data)."""
    cfg = _small("qwen14b", n_layers=2, batch=2, n_q_heads=10, n_kv_heads=2, prompt=300, decode_steps=12,
                 budget=320, budget_max=351, seed=61)
    res = []
    for _ in range(2):
        st, o, g = _pair(cfg, cap=352, path=path)
        outs = [g.decode_step(st.q[s], st.k_new[s], st.v_new[s]).cpu().numpy().copy() for s in range(cfg.decode_steps)]
        state = [g.export_unit(*key) for key in o.units]
        res.append((outs, state))
        g.close()
    for a, b in zip(res[0][0], res[1][0]):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    for a, b in zip(res[0][1], res[1][1]):
        for f in ("pos", "crf", "tau", "flags", "K", "V"):
            assert np.array_equal(a[f], b[f]), f


@pytest.mark.parametrize("path", PATHS)
def test_hip_graph_replay_matches_eager(path):
    """Four decode steps captured into one HIP graph (time lives in device memory) and replayed three
    times, with eager work between the replays; every replay must equal the eager run."""
    import torch
    cfg = _small("tiny", n_q_heads=8, n_kv_heads=2, decode_steps=12, seed=71)
    st, o, g = _pair(cfg, cap=96, path=path)
    _, _, g2 = _pair(cfg, cap=96, path=path)
    dev = g.device
    as_dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev).to(torch.bfloat16)
    q, k, v = as_dev(st.q), as_dev(st.k_new), as_dev(st.v_new)
    eager = [g2.decode_step(q[s], k[s], v[s]).clone() for s in range(12)]
    torch.cuda.synchronize()
    sq, sk, sv = q[:4].clone(), k[:4].clone(), v[:4].clone()          # static input buffers of the graph
    outs = [torch.empty_like(eager[0]) for _ in range(4)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for i in range(4):
            g.decode_step(sq[i], sk[i], sv[i], out=outs[i])
    for rep in range(3):
        sq.copy_(q[4 * rep:4 * rep + 4]); sk.copy_(k[4 * rep:4 * rep + 4]); sv.copy_(v[4 * rep:4 * rep + 4])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        scratch = (torch.randn(1 << 16, device=dev) * 2).sum().item()   # unrelated eager work between replays
        assert np.isfinite(scratch)
        for i in range(4):
            assert torch.equal(outs[i], eager[4 * rep + i]), (rep, i)
    assert g.time() == cfg.prompt + 12
    for key in o.units:
        a, b = g.export_unit(*key), g2.export_unit(*key)
        for f in ("pos", "crf", "tau", "flags"):
            assert np.array_equal(a[f], b[f])
    g.close(); g2.close()


@pytest.mark.parametrize("path", [3, 4])
def test_probe_classes_on_multi_chunk_units_of_a_fused_path_context(path):
    """Sec. 3 classes on units of 300..700 entries (several 256-entry chunks, ragged last blocks, 7 query
    heads per KV head) in a context whose decode steps run the fused kernel: the probe shares the context's
    workspace (partials, logits buffer) with those steps, leaves the caches untouched, and the
    decode steps that follow still match the oracle."""
    cfg = _small("qwen7b", n_layers=1, batch=3, n_q_heads=14, n_kv_heads=2, prompt=333, decode_steps=16,
                 budget=500, budget_min=300, budget_max=735, seed=5)
    budgets = np.array([[[300, 700], [513, 333], [641, 352]]], dtype=np.int32)
    st, o, g = _pair(cfg, cap=736, budgets=budgets, path=path)
    stats = parity.lockstep(g, o, parity_slice(st, 0, 8), 8)
    cls = g.probe(0, st.probe_q[0]).cpu().numpy()
    for (l, b, h), u in o.units.items():
        ref, abar = o.probe((l, b, h), st.probe_q[l, b, h * o.G:(h + 1) * o.G])
        e = g.export_unit(l, b, h, with_kv=False)
        got = cls[b, h, :e["n"]]
        by_pos_g = dict(zip(e["pos"].tolist(), got.tolist()))
        by_pos_o = dict(zip(u.pos.tolist(), ref.tolist()))
        srt = np.sort(abar)
        k = (3 * u.n) // 10
        assert k >= 90
        edges = [srt[k - 1], srt[k], srt[u.n - k - 1], srt[u.n - k]]
        for p_, a in zip(u.pos.tolist(), abar.tolist()):
            if by_pos_g[p_] != by_pos_o[p_]:
                assert min(abs(a - x) / x for x in edges) < 1e-5, (p_, a)
        assert (got == 2).sum() == k and (got == 0).sum() == k and (cls[b, h, e["n"]:] == 255).all()
    stats2 = parity.lockstep(g, o, parity_slice(st, 8, 8), 8, check_kv_every=8)
    assert stats.resynced + stats2.resynced <= 2 and g.status() == 0
    g.close()


def parity_slice(st, first, count):
    from dataclasses import replace
    return replace(st, q=st.q[first:first + count], k_new=st.k_new[first:first + count], v_new=st.v_new[first:first + count])
