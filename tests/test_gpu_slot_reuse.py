"""GPU: a cache slot that held a longer sequence full of infinities and NaN gives the next sequence the bits of a fresh context, in
every kernel that reads the cache: prefill of few and of more tokens, fused, chained, captured and per-operation steps, wide
batches, the plain path; while the position moves over block borders."""
import pytest
import torch

from paper_2501_06589_amd import inputs, ladder

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
STEPS = 68      # more than 64 positions
TINY = inputs.WORKLOADS["tiny"].with_(name="slot", n_layers=2, dtype="bf16", inter=352, tp_degree=1, n_real_shards=1)


@pytest.fixture(scope="module")
def harness():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


def _poison(ctx, w):
    bad = torch.tensor([float("nan"), float("inf"), -float("inf"), 1.0]).repeat(64)[:, None].expand(256, w.head_dim)
    bad = bad.expand(w.batch, w.n_kv_heads, 256, w.head_dim).to(w.torch_dtype).contiguous().to(DEV)
    for i in range(w.n_layers):
        ctx.load_kv(i, 0, bad, bad)


def _same(harness, w, start, steps=STEPS, **cfg):
    tensors = harness.make_tensors(w)
    xs = [inputs.embeddings(w, w.batch, 1, inputs.SEED_DECODE0 + i)[:, 0].contiguous().to(DEV) for i in range(steps)]
    outs = []
    for used in (False, True):
        ctx = harness.build_gpu(w, tensors, max_seq=256, **cfg)
        if used:
            _poison(ctx, w)
        outs.append([start(ctx).cpu()] + [ctx.decode_step(x).cpu() for x in xs])
        ctx.free()
    for i, (a, b) in enumerate(zip(*outs)):
        assert torch.isfinite(a).all() and torch.equal(a, b), i


@pytest.mark.parametrize("nq,nkv,d", [(2, 2, 64), (8, 1, 128)])
@pytest.mark.parametrize("cached", [1, 32, 63, 64, 129, 188])      # (the last one: up to the end of the cache)
@pytest.mark.parametrize("batch,cfg", [(2, dict()), (2, dict(decode_fused=1)), (2, dict(decode_fused=2)), (2, dict(decode_fused=0)),
                                       (2, dict(decode_graph=1)), (17, dict()), (17, dict(decode_graph=1)),
                                       (2, dict(kernel_path=ladder.LADDER_PATH_GENERIC))])
def test_steps_behind_a_handed_over_cache(harness, nq, nkv, d, cached, batch, cfg):
    w = TINY.with_(n_q_heads=nq, n_kv_heads=nkv, head_dim=d, batch=batch, prefill=0, kv_preload=cached)

    def start(ctx):
        for i in range(w.n_layers):
            k, v = (t.to(DEV) for t in inputs.kv_cache(w, i, 0, batch, cached))
            if i:       # off a 16-byte boundary: the element-wise kernel
                k, v = (torch.cat([t.flatten()[:1], t.flatten()])[1:].view(t.shape) for t in (k, v))
            ctx.load_kv(i, 0, k, v)
        return torch.zeros(1)

    _same(harness, w, start, **cfg)


@pytest.mark.parametrize("tokens,batch", [(1, 2), (3, 2), (33, 2), (63, 1), (64, 1), (65, 1), (100, 3), (130, 2), (160, 8), (1, 17), (5, 17)])
@pytest.mark.parametrize("nq,nkv,d", [(2, 2, 64), (8, 1, 128)])
def test_prompt_and_steps(harness, nq, nkv, d, tokens, batch):
    """(160 tokens of 8 sequences: more than 1024 rows, whose appends are an epilogue)"""
    w = TINY.with_(n_q_heads=nq, n_kv_heads=nkv, head_dim=d, batch=batch, prefill=tokens, kv_preload=0)
    x = inputs.embeddings(w, batch, tokens, inputs.SEED_PREFILL).to(DEV)
    _same(harness, w, lambda ctx: ctx.prefill(x))
