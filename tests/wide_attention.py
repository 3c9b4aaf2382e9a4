"""One layer whose steps show the decode attention of a wide batch by itself: the GPU test and the CPU test of what it can see
share the inputs, the measure and the bound."""
import numpy as np

from oracle import from_torch
from paper_2501_06589_amd import inputs

HEADS = [(2, 2, 64), (4, 2, 128), (4, 1, 64), (8, 1, 128)]      # q heads, kv heads, head size
CACHED = [1, 31, 127, 128, 300, 1025]
STEPS = 3
TOL = 0.0029 * 5.8      # the bound of one module: 0.29 % of RMS, its maximum 5.8 times that


def case(nq, nkv, d, cached):
    w = inputs.WORKLOADS["8b"].with_(name="wide_attn", n_layers=1, hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, inter=352,
                                     batch=17, prefill=0, kv_preload=cached, decode_steps=STEPS)
    tensors = [[inputs.layer_weights(w, 0, 0)]]
    tensors[0][0]["w_down"].zero_()
    tensors[0][0]["wv"].mul_(3)      # (new entries of the cache about as large as the ones that are handed over)
    return w, tensors


def error(w, step, got, want):
    """Largest error of what the attention module adds to the stream, over the RMS of that (17 rows at once)."""
    x = from_torch.to_f64(inputs.embeddings(w, w.batch, 1, inputs.SEED_DECODE0 + step)).reshape(want.shape)
    return float(np.max(np.abs(got - want)) / np.sqrt(np.mean((want - x) ** 2)))
