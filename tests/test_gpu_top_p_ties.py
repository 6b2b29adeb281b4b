"""Equal weights at the top-p threshold, about as many as the bookkeeping's list holds and more: the lowest positions are hit, exactly as many as p asks
for, in the step's one kernel and in both kernels that follow a scan."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap,defer", [(320, False), (320, True), (8224, False)])
@pytest.mark.parametrize("n", [3, 64, 255, 256, 257, 300])
def test_lowest_positions(n, cap, defer):
    import torch
    from paper_2601_16986_amd import ckv
    B, t = 3, 5000
    asked = max(1, int(0.37 * n))
    p = (asked - 0.5) / n                    # half an entry's weight from the next count; fp32 weights are off by 2^-22 of that at most
    g = ckv.CrystalKV(1, B, 2, 1, 128, cap, np.full((1, B, 1), n, np.int32), t0=t, top_p=p, budget_min=1, budget_max=cap - 1)
    dev = g.device
    rng = np.random.default_rng(n)
    pos = torch.from_numpy(np.stack([rng.permutation(4000)[:n - 1] for _ in range(B)]).astype(np.int32)).reshape(B, 1, n - 1).to(dev)
    k = torch.zeros((B, 1, n - 1, 128), dtype=torch.bfloat16, device=dev)
    g.load_cache(0, k, k, torch.full((B, 1), n - 1, dtype=torch.int32, device=dev), torch.ones((B, 1, n - 1), device=dev), pos, pos)
    new = torch.zeros((B, 1, 128), dtype=torch.bfloat16, device=dev)
    g.decode_step(torch.ones((B, 2, 128), dtype=torch.bfloat16, device=dev), new, new, layer=0, evict=False, defer=defer)
    if defer:
        g.join()
    for b in range(B):
        e = g.export_unit(0, b, 0, with_kv=False)
        want = e["pos"] <= np.sort(e["pos"])[asked - 1]
        want[-1] = True                      # the entry that arrived
        assert e["n"] == n and e["pos"][-1] == t and np.array_equal(e["tau"] == t, want)
    assert g.status() == 0
    g.close()
