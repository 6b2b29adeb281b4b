"""The scan of few units in both of its shapes (chosen by the entries the budgets allow) at the edges of its blocks, chunks
and workgroups, against attention in 64 bits; the step's records behind it, in a launch of their own at this capacity (deferred, plain, or
without bookkeeping)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 31, 32, 33, 255, 256, 257, 511, 2047, 2048, 2049, 4100, 6000, 63, 1023]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("G", [1, 5, 8])
@pytest.mark.parametrize("budget", [6100, 20000])            # 16 units: 97600 entries (a block per wavefront), 320000 (a chunk)
@pytest.mark.parametrize("mode", ["attention", "plain", "defer"])
def test_edges(mode, budget, G, bf16):
    import torch
    from paper_2601_16986_amd import ckv
    batch, hkv, cap, n_max, t = 8, 2, 20032, max(LENGTHS), 7000
    g = ckv.CrystalKV(1, batch, hkv * G, hkv, 128, cap, np.full((1, batch, hkv), budget, np.int32), t0=t, budget_min=1, budget_max=cap - 1,
                      headroom=1, prompt_len=0, out_dtype=ckv.BF16 if bf16 else ckv.F32)
    gen = torch.Generator(device=g.device)
    gen.manual_seed(11)
    rnd = lambda *s: torch.randn(s, generator=gen, device=g.device).to(torch.bfloat16)
    k, v = rnd(batch, hkv, n_max, 128), rnd(batch, hkv, n_max, 128)
    q, kn, vn = rnd(batch, hkv * G, 128), rnd(batch, hkv, 128), rnd(batch, hkv, 128)
    pos = torch.arange(n_max, device=g.device, dtype=torch.int32).expand(batch, hkv, n_max).contiguous()
    lengths = torch.tensor(LENGTHS, dtype=torch.int32, device=g.device).reshape(batch, hkv)
    g.load_cache(0, k, v, lengths, torch.ones_like(pos, dtype=torch.float32), pos, pos)
    if mode == "attention":
        out = g.decode_step(q, kn, vn, layer=0, attention_only=True)
    else:
        out = g.decode_step(q, kn, vn, layer=0, defer=mode == "defer")
    g.join()
    out = out.double().cpu().numpy().reshape(batch, hkv, G, 128)
    for u, n in enumerate(LENGTHS):
        b, h = divmod(u, hkv)
        kk, vv = torch.cat([k[b, h, :n], kn[b, h, None]]).double().cpu(), torch.cat([v[b, h, :n], vn[b, h, None]]).double().cpu()
        s = q[b, h * G:(h + 1) * G].double().cpu() @ kk.t() / np.sqrt(128.0)
        ref = (torch.softmax(s, dim=-1) @ vv).numpy()
        # fp32 accumulation, probabilities to 16 bits and more: 2e-5 of the row; a bf16 output is rounded to 2^-8
        bound = (2.0 ** -8 if bf16 else 2e-5) * np.abs(ref).max(-1, keepdims=True)
        assert np.all(np.abs(out[b, h] - ref) <= bound), (u, n, float(np.abs(out[b, h] - ref).max()))
        e = g.export_unit(0, b, h)
        assert e["n"] == n + 1 and e["pos"][n] == t and e["tau"][n] == t and e["crf"][n] == (0.0 if mode == "attention" else 1.0)
        assert np.array_equal(e["K"][n], kn[b, h].float().cpu().numpy()) and np.array_equal(e["V"][n], vn[b, h].float().cpu().numpy())
    assert g.status() == 0 and g.time() == t + 1
    g.close()
