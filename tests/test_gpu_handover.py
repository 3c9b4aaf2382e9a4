"""GPU: the handed-over cache (ladder_load_kv) and the greedy token at the edges of their kernels: 16-byte and element-wise
accesses give the same bits, whatever the length, head size and alignment; the first arg max whatever the row length."""
import numpy as np
import pytest
import torch

from paper_2501_06589_amd import inputs, ladder

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TINY = inputs.WORKLOADS["tiny"]


@pytest.fixture(scope="module")
def harness():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("bf16", 20), ("fp32", 64), ("fp32", 30)])
@pytest.mark.parametrize("S", [1, 63, 64, 65, 130])
def test_load_kv_alignment_and_ragged_lengths(harness, dtype, d, S):
    w = TINY.with_(name="kv", dtype=dtype, n_layers=1, n_q_heads=4, n_kv_heads=2, head_dim=d, batch=3, prefill=0, kv_preload=S,
                   decode_steps=1, tp_degree=1, n_real_shards=1)
    res = harness.run_case(w, kv_preload=S, decode_steps=1)          # against the oracle
    assert max(res.errs) < (1e-4 if dtype == "fp32" else 2e-2), res.errs
    ctx = harness.build_gpu(w, harness.make_tensors(w))
    k, v = (t.to(DEV) for t in inputs.kv_cache(w, 0, 0, w.batch, S))
    x = inputs.embeddings(w, w.batch, 1, inputs.SEED_DECODE0)[:, 0].contiguous().to(DEV)
    outs = []
    for off in (0, 1):      # (off 1: contiguous tensors whose storage starts off a 16-byte boundary)
        shifted = []
        for t in (k, v):
            buf = torch.empty(t.numel() + off, dtype=t.dtype, device=DEV)
            buf[off:].copy_(t.flatten())
            shifted.append(buf[off:].view(t.shape))
        ctx.load_kv(0, 0, *shifted)
        outs.append(ctx.decode_step(x).cpu())
    assert torch.equal(outs[0], outs[1])
    ctx.free()


@pytest.mark.parametrize("V", [1, 3, 1023, 4096, 4100, 16389, 20000])
def test_first_argmax_of_any_row_length(harness, V):
    w = TINY.with_(name="head", n_layers=1, tp_degree=1, n_real_shards=1, batch=3)
    hw = inputs.head_weights(w, max(V, 2), V, device=DEV)
    x = torch.randn(3, w.hidden, generator=torch.Generator().manual_seed(V)).to(DEV)
    for kind in ("random", "ties", "equal"):
        ctx = ladder.Ladder(ladder.config_for(w))
        w_lm = hw["w_lm"].clone()
        if kind == "equal":
            w_lm.zero_()
        elif kind == "ties":      # every column twice, a stretch apart
            w_lm[:, V // 2:2 * (V // 2)] = w_lm[:, :V // 2].clone()
        ctx.load_head(hw["table"], hw["final_norm"], w_lm)
        logits, toks = ctx.head(x)
        assert np.array_equal(toks.cpu().numpy(), np.argmax(logits.cpu().numpy(), axis=-1)), (kind, V)
        ctx.free()


@pytest.mark.parametrize("rows", [1, 16, 17, 64, 65])
@pytest.mark.parametrize("hidden,V", [(256, 48), (256, 64), (256, 1056), (4096, 4000), (4096, 16)])
def test_head_rows(harness, hidden, V, rows):
    """The packed head's two products: the skinny GEMM for up to 16 rows where it takes the width, the tiled one for more rows,
    an odd number of column tiles, and widths so narrow that the skinny one would split K."""
    w = TINY.with_(name="head_rows", dtype="bf16", hidden=hidden, inter=352, n_layers=1, tp_degree=1, n_real_shards=1, batch=rows)
    hw = inputs.head_weights(w, V, V, device=DEV)
    ctx = ladder.Ladder(ladder.config_for(w))
    ctx.load_head(hw["table"], hw["final_norm"], hw["w_lm"])
    x = torch.randn(rows, w.hidden, generator=torch.Generator().manual_seed(V)).to(DEV)
    logits, toks = ctx.head(x)
    y = x.double() / torch.sqrt((x.double() ** 2).mean(-1, keepdim=True) + w.rms_eps) * hw["final_norm"].double()
    want = y @ hw["w_lm"].double()
    # (the normed rows are rounded to bf16 once: 2^-9 of each term at most)
    assert float((logits.double() - want).abs().max() / want.square().mean().sqrt()) < 2e-2
    assert np.array_equal(toks.cpu().numpy(), np.argmax(logits.cpu().numpy(), axis=-1))
    if rows <= 16:      # (LADDER_HEAD_STATIC_MAX_ROWS)
        got = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
        ctx.head_static(x, got)
        assert torch.equal(got, toks)
    ctx.free()
