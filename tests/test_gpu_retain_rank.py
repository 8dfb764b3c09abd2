"""The retention's ranking where its forms meet: every candidate fits (nothing
is ranked), exactly one too many, and far too many, at expert counts around
the ranking's groups of 8 and its quarters of the experts, with many equal
keys (confidence 0 and 1 only, few tokens). The retained sets are integers and
must be the oracle's."""
import numpy as np
import pytest
import torch

from oracle import oled_oracle as O
from paper_2609_33385_amd import harness as HN
from paper_2609_33385_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", ["fits", "one_over", "half"])
@pytest.mark.parametrize("E", [1, 7, 9, 31, 33, 64, 129, 255, 256])
def test_retained_set(E, over):
    T, k = max(2, E // 3), 1 if E < 3 else 2
    rng = np.random.default_rng(E)
    logits = [rng.standard_normal((T, E)).astype(np.float32) for _ in range(3)]
    active = len(np.unique(O.route(logits[0], k)[0]))
    C = {"fits": active, "one_over": active - 1, "half": active // 2}[over]
    w = W.WORKLOADS[1].replace(wid=600, name=f"rank-E{E}", batch=1, block=T, n_experts=E, top_k=k,
                               hidden=128, inter=128, n_layers=1, n_iters=3, capacity=C)
    pool = HN.fill_pool(w, 0, 1)
    ctx = HN.make_context(w, pool, max_tokens=T)
    res = np.zeros(E, bool)
    try:
        for i, lg in enumerate(logits):
            print(f"[rank] E={E} C={C} iteration {i}", flush=True)
            conf = rng.integers(0, 2, T).astype(np.float32)
            HN.layer_step(ctx, 0, torch.from_numpy(lg).cuda(), torch.from_numpy(conf).cuda())
            st = ctx.read_layer_state(0, T)
            ref = O.layer_step(lg, conf, res, k, C)
            res = ref["resident_after"]
            assert np.array_equal(st["resident_after"], res), f"E={E} C={C} iteration {i}"
    finally:
        ctx.close()
        pool.free()
