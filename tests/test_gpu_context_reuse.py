"""Contexts made and closed one after another, and several at once from several threads, with deferred bookkeeping on the
streams they take over from each other: the same results as a context of its own."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(seed, steps=6):
    import torch
    from paper_2601_16986_amd import ckv
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=gen, device=dev).to(torch.bfloat16)
    with torch.cuda.stream(torch.cuda.Stream(dev)):
        L, P, B = 3, 70, 48
        g = ckv.CrystalKV(L, 2, 8, 2, 128, 96, np.full((L, 2, 2), B, np.int32), t0=P, budget_min=1, budget_max=95, headroom=1, prompt_len=P)
        for l in range(L):
            k = rnd(2, 2, P, 128)
            g.load_prompt(l, k, rnd(2, 2, P, 128))
            g.evict(l)
        outs = [g.decode_step(rnd(2, 8, 128), rnd(2, 2, 128), rnd(2, 2, 128), layer=l, defer=True).clone() for _ in range(steps) for l in range(L)]
        g.join()
        torch.cuda.current_stream().synchronize()
        state = [g.export_unit(l, b, h, with_kv=False) for l in range(L) for b in range(2) for h in range(2)]
        g.close()
    return torch.stack(outs).cpu().numpy(), state


def test_contexts_hand_their_streams_on():
    want = {seed: _run(seed) for seed in range(3)}
    got, errors = {seed: [] for seed in range(3)}, []

    def work(seed):
        try:
            for _ in range(4):
                got[seed].append(_run(seed))
        except Exception as e:                 # reported by the main thread
            errors.append(e)

    threads = [threading.Thread(target=work, args=(s,), daemon=True) for s in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=100)
        assert not t.is_alive()
    assert not errors, errors
    for seed, (outs, state) in want.items():
        assert len(got[seed]) == 4
        for run_outs, run_state in got[seed]:
            assert np.array_equal(outs, run_outs)
            for a, b in zip(state, run_state):
                assert a["n"] == b["n"] and all(np.array_equal(a[k], b[k]) for k in ("pos", "crf", "tau", "flags"))
