"""CPU: the GPU test of the wide batches' decode attention sees a lost key. The oracle loses one at an edge of a block, of a
wavefront round or of a split, or a whole block or split, and the measure of that test has to exceed its bound."""
import numpy as np
import pytest

import wide_attention
from oracle import from_torch
from oracle import ladder_oracle as lo
from paper_2501_06589_amd import inputs


def _steps(w, tensors, cached, lose=None):
    cfg = from_torch.config_from_workload(w)
    state = lo.State.empty(cfg, 1, w.batch, cached + wide_attention.STEPS)
    from_torch.load_kv(state, 0, 0, *inputs.kv_cache(w, 0, 0, w.batch, cached))
    state.pos = cached
    right = lo.causal_gqa_attention

    def attention(q, k, v, s0):
        gone = [p for p in lose(s0) if 0 <= p <= s0]
        k, v = (np.delete(t[:, :, :s0 + 1], gone, axis=2) for t in (k, v))
        return right(q, k, v, k.shape[2] - 1)

    if lose:
        lo.causal_gqa_attention = attention
    try:
        layers = [from_torch.layer_from_tensors(t) for t in tensors]
        return [lo.forward_eq2(from_torch.to_f64(inputs.embeddings(w, w.batch, 1, inputs.SEED_DECODE0 + i)), layers, cfg, state)
                for i in range(wide_attention.STEPS)]
    finally:
        lo.causal_gqa_attention = right


@pytest.mark.parametrize("nq,nkv,d", wide_attention.HEADS)
@pytest.mark.parametrize("cached", wide_attention.CACHED)
def test_a_lost_key_exceeds_the_bound(nq, nkv, d, cached):
    w, tensors = wide_attention.case(nq, nkv, d, cached)
    want = _steps(w, tensors, cached)
    lost = {"first": lambda s0: [0], "new": lambda s0: [s0], "last cached": lambda s0: [s0 - 1]}
    for p in (31, 32, 127, 128, 255, 256, 1023, 1024):
        if p < cached:
            lost["key %d" % p] = lambda s0, p=p: [p]
    if cached >= 64:
        lost["block"] = lambda s0: range(32, 64)
    if cached >= 256:
        lost["split"] = lambda s0: range(128, 256)
    for name, lose in lost.items():
        got = _steps(w, tensors, cached, lose)
        errs = [wide_attention.error(w, i, g, r) for i, (g, r) in enumerate(zip(got, want))]
        assert min(errs) > 3 * wide_attention.TOL, (name, errs)
