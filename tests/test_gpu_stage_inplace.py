"""GPU: a pipeline stage may leave its three tensors in the buffers they came in; every schedule gives the same bits as with
buffers of their own (the stream is copied out by the residual updates while the stage still runs)."""
import pytest
import torch

from paper_2501_06589_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("n_layers", [1, 2])
@pytest.mark.parametrize("dtype,rows", [("fp32", 5), ("bf16", 12), ("bf16", 70), ("bf16", 1100)])
def test_outputs_in_the_input_buffers(n_layers, dtype, rows):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    w = inputs.WORKLOADS["tiny"].with_(name="inplace", dtype=dtype, n_layers=n_layers, tp_degree=2, n_real_shards=1, batch=1,
                                       prefill=rows, decode_steps=1, peer_pool=1)
    ctx = gpu_harness.build_gpu(w, gpu_harness.make_tensors(w), inputs.peer_partials(w, rows))
    g = torch.Generator().manual_seed(rows)
    hand = [torch.randn(1, rows, w.hidden, generator=g).to(DEV) for _ in range(3)]
    want = ctx.prefill_stage(hand)
    for perm in ((0, 1, 2), (2, 0, 1), (1, 2, 0)):
        bufs = [t.clone() for t in hand]
        outs = [bufs[i] for i in perm]
        ctx._check(ctx._lib.ladder_prefill_stage(ctx._h, *[t.data_ptr() for t in bufs], 1, rows, *[t.data_ptr() for t in outs]))
        for a, b in zip(want, outs):
            assert torch.equal(a, b), perm
    ctx.free()
