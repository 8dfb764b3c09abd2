"""The split of the dense-tile launches: experts whose routed rows sit at the
edges of the streaming / dense threshold, of the 32-row groups and of the 128- and
256-row items, one expert that holds nearly every row, so that the ranges of tiles
per XCD are as uneven as they get, and few experts with large items, whose tiles
the XCDs share by number. At hidden 1024 and above the small tiles ride in the
streaming launches (up to 512 routes per expert on average).

k = 1 makes every gate 1 and every expert's rows exactly the tokens sent to
it. Every output row is checked against the oracle in float64; the bound is
the bf16 bound of the layer outputs, per expert, so that one missing or
misplaced item (at least a tenth of an expert's rows, each off by about its
own norm) fails it. Each pass has activations of its own and starts from outputs
that are not numbers: the intermediate rows that the pass before left at the same
places are wrong for it, so a tile dropped in the second pass, where the retained
experts are hits, fails too.
"""
import numpy as np
import pytest
import torch

from oracle import oled_oracle as O
from paper_2609_33385_amd import harness as HN
from paper_2609_33385_amd import workload as W

pytestmark = pytest.mark.gpu

SPLITS = {
    "edges": [64, 65, 96, 97, 128, 255, 256, 257, 511, 512, 513, 1, 0, 33],
    "one-holds-most": [2305, 65, 64, 2],
    "few-large": [1300, 700, 520, 1793, 64, 900, 1025, 513],   # tiles counted, not priced
    "many-large": [577 + 5 * e for e in range(17)],            # one expert more than that takes
    "many-small": [65 + e % 3 for e in range(40)],
}


@pytest.mark.parametrize("H,I", [(256, 256), (768, 512), (1024, 256), (1024, 2048)])
@pytest.mark.parametrize("name", SPLITS)
def test_dense_split(name, H, I):
    rows = SPLITS[name]
    E, T = len(rows), sum(rows)
    w = W.WORKLOADS[1].replace(wid=500, name=f"split-{name}", dtype="bf16", batch=1, block=T,
                               n_experts=E, top_k=1, hidden=H, inter=I, n_layers=1, n_iters=1,
                               capacity=E // 2)
    P = 5
    rng = np.random.default_rng(H + I)
    expert = rng.permutation(np.repeat(np.arange(E), rows))
    lg = np.zeros((T, E), np.float32)
    lg[np.arange(T), expert] = 4.0
    raw = W.expert_blocks(w, 3, range(P))
    pool = HN.fill_pool(w, 3, P, raw=raw)
    ctx = HN.make_context(w, pool, max_tokens=T)
    y = torch.empty((T, H), dtype=torch.bfloat16, device="cuda")
    conf = torch.rand(T, device="cuda")
    try:
        for i in range(2):   # the second pass runs the retained experts as hits
            print(f"[split] {name} H={H} I={I} pass {i}", flush=True)
            xh = W.activations(w, 3, 0, 0, i)
            y.fill_(float("nan"))
            HN.layer_step(ctx, 0, torch.from_numpy(lg).cuda(), conf, HN.to_device(xh), y)
            st = ctx.read_layer_state(0, T)
            assert st["counts"].tolist() == rows
            if i:   # dense tiles of hits are among them
                assert np.any((np.asarray(rows) >= 65) & st["resident_before"])
            got = O.decode(HN.from_device(y))
            x = O.decode(xh)
            for e in range(E):
                t = np.flatnonzero(expert == e)
                if not len(t):
                    continue
                w13, w2 = W.split_expert(w, O.decode(raw[e % P]))
                a = x[t] @ w13.T
                ref = (a[:, :I] / (1 + np.exp(-a[:, :I])) * a[:, I:]) @ w2.T
                err = np.linalg.norm(got[t] - ref) / np.linalg.norm(ref)
                assert err <= 2e-2, f"{name}: expert {e} with {rows[e]} rows: rel L2 {err:.3e}"
    finally:
        ctx.close()
        pool.free()
