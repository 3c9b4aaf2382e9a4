"""The attention of a prompt by itself, row by row: every order in which its workgroups are dealt out."""
import numpy as np
import pytest
import torch

from oracle import from_torch
from oracle import ladder_oracle as lo
from paper_2501_06589_amd import inputs

pytestmark = pytest.mark.gpu
# Operands that are rounded to bf16 on the way, each to 2^-9 of itself: the normed rows, q, k, v, the softmax weights, the attention output; twice that
# for what they are multiplied with.
TOL = 6 * 2.0 ** -8


@pytest.fixture(scope="module")
def harness():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("batch,nq,nkv,d,T", [
    (1, 4, 1, 128, 65),       # five workgroups of one query tile
    (1, 16, 4, 128, 1024),    # 256: one row of CUs, full
    (1, 16, 4, 64, 1025),     # 260: a second row of four, in reverse
    (3, 8, 4, 128, 400),      # 156 of 32 queries (two heads each)
    (5, 16, 4, 128, 250),     # 320: pairs that are no multiple of 8
    (37, 4, 4, 64, 90),       # 296 of 64 queries (a head each)
    (13, 32, 8, 64, 190),     # 1248: five rows of CUs, the last one ragged
    (20, 16, 4, 128, 256),    # 1280: the most of one tile
    (27, 16, 4, 64, 177),     # 1296: two tiles (648)
    (43, 8, 4, 128, 250),     # two tiles, two heads per workgroup
])
def test_every_row_of_a_prompt(harness, batch, nq, nkv, d, T):
    w = inputs.WORKLOADS["8b"].with_(name="prompt_attn", n_layers=1, hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, inter=64,
                                     batch=batch, prefill=T, decode_steps=0)
    tensors = [[inputs.layer_weights(w, 0, 0)]]
    tensors[0][0]["w_down"].zero_()     # (what the call adds to the stream is the attention module's output)
    harness.say(f"[case] batch {batch} heads {nq}/{nkv} of {d} tokens {T}")
    emb = inputs.embeddings(w, batch, T, inputs.SEED_PREFILL)
    hand = [emb.float().to("cuda:0"), torch.zeros(batch, T, w.hidden, device="cuda:0"), torch.zeros(batch, T, w.hidden, device="cuda:0")]
    ctx = harness.build_gpu(w, tensors)
    got = ctx.prefill_stage(hand)[1].cpu().double().numpy()     # the attention module's output, all rows
    ctx.free()
    cfg = from_torch.config_from_workload(w)
    state = lo.State.empty(cfg, 1, batch, T)
    x = from_torch.to_f64(emb)
    want = lo.forward_eq2(x, [from_torch.layer_from_tensors(tensors[0])], cfg, state, None, wiring="ladder") - x
    err = np.linalg.norm(got - want, axis=-1) / np.linalg.norm(want, axis=-1)
    worst = np.unravel_index(np.argmax(err), err.shape)
    assert err.max() < TOL, (worst, err.max())
