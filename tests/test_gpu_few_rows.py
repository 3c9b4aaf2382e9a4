"""GPU: the projections of calls of few and medium rows (ring GEMM, split K, partial products added up by the next kernel) at
the edges of their tiles, splits and row ranges, against the CPU oracle."""
import numpy as np
import pytest
import torch

import wide_attention
from paper_2501_06589_amd import inputs, ladder

pytestmark = pytest.mark.gpu

# one layer; hidden 2080 = 65 k tiles (an odd number: the last stage of 64 k is half filled), N no multiple of a tile
WIDE = inputs.WORKLOADS["8b"].with_(name="few_rows", n_layers=1, hidden=2080, n_q_heads=16, n_kv_heads=2, inter=2080,
                                    batch=1, kv_preload=0, decode_steps=2)
# the bound of a prefill of one layer: 0.29 % of RMS per module and sqrt(modules), its maximum 5.8 times that
TOL = 0.0029 * 2 ** 0.5 * 5.8


@pytest.fixture(scope="module")
def harness():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


@pytest.mark.parametrize("rows", [16, 17, 33, 64, 65, 129, 300, 513, 1024, 1025])
def test_prefill_rows(harness, rows):
    """16 rows and fewer: the skinny GEMM; up to 1024: partial products; beyond: the residual epilogue."""
    res = harness.run_case(WIDE.with_(prefill=rows), decode_steps=1)
    assert max(res.errs) < TOL, res.errs


@pytest.mark.parametrize("batch,prefill", [(3, 43), (17, 3), (40, 1)])
def test_several_sequences_and_wide_decode(harness, batch, prefill):
    res = harness.run_case(WIDE.with_(batch=batch, prefill=prefill), decode_steps=2)
    assert max(res.errs) < TOL, res.errs


def test_two_computed_shards_and_peers(harness):
    """Several shards share the partial-product buffer, slot after slot; peers are added behind them."""
    w = WIDE.with_(tp_degree=3, n_real_shards=2, prefill=100, peer_pool=2)
    res = harness.run_case(w, decode_steps=1)
    assert max(res.errs) < TOL, res.errs


@pytest.mark.parametrize("nq,nkv,d", wide_attention.HEADS)
@pytest.mark.parametrize("cached", wide_attention.CACHED)
def test_wide_decode_attention(harness, nq, nkv, d, cached):
    """Batches above 16: one and several splits, at the edges of a 32-key block, of a wavefront round and of a split, while
    the position moves over them; every number of q heads per kv head. What is compared is what attention adds to the stream
    (the MLP adds nothing): a single lost key shows (test_wide_attention_sensitivity.py)."""
    w, tensors = wide_attention.case(nq, nkv, d, cached)
    res = harness.run_case(w, kv_preload=cached, max_tokens=1, tensors=tensors)
    assert max(res.errs) < TOL, res.errs
    errs = [wide_attention.error(w, i, g, r) for i, (g, r) in enumerate(zip(res.gpu, res.ref))]
    assert max(errs) < wide_attention.TOL, errs


def test_residual_epilogue_of_the_wide_ring_tile(harness):
    """128 x 256 tiles with the residual update as epilogue, ragged in both directions, more peers than are requested at once;
    the second layer reads the rows and the sums of squares that the epilogue left."""
    w = WIDE.with_(name="wide_tile", n_layers=2, hidden=4128, prefill=1101, tp_degree=5, peer_pool=2)
    res = harness.run_case(w, decode_steps=0, gen_device="cuda:0")
    assert max(res.errs) < TOL * 2 ** 0.5, res.errs


@pytest.mark.parametrize("batch,prefill,hidden,inter,n_q,peers", [
    (1, 257, 4160, 4160, 8, 0),     # the first row count that takes them: 128 columns, SwiGLU (32.5 row blocks of 8, 65 column blocks)
    (1, 513, 2112, 8256, 8, 0),     # 128 columns, K of 129 stages in 3 splits: the rows' partial products
    (1, 700, 576, 8256, 8, 2),      # 256 columns, SwiGLU, K of 9 stages (an odd number)
    (1, 1025, 4160, 1088, 8, 9),    # 192 columns, residual update with more peers than are requested at once; 17 stages
    (3, 700, 1088, 416, 16, 0),     # 192 columns, rotary + append over three sequences; 4.25 column blocks elsewhere
    (3, 1000, 2112, 2112, 16, 2)])  # 256 columns in every projection, the last column block a quarter full
def test_two_workgroups_per_cu(harness, batch, prefill, hidden, inter, n_q, peers):
    """The tiles of 128 rows x 128 / 192 / 256 columns that share a CU in pairs, ragged in both directions, with every epilogue; the
    second layer reads what the residual update left."""
    w = WIDE.with_(name="pairs", n_layers=2, hidden=hidden, inter=inter, n_q_heads=n_q, batch=batch, prefill=prefill,
                   tp_degree=1 + peers, peer_pool=2 if peers else 0)
    res = harness.run_case(w, decode_steps=0, gen_device="cuda:0")
    assert max(res.errs) < TOL * 2 ** 0.5, res.errs


def test_residual_epilogue_of_the_largest_tile(harness):
    """256 x 256 tiles with the residual update as epilogue (taken without peers only), ragged in both directions: 4 rows and 64 columns
    in the last tiles; the second layer reads what the epilogue left."""
    w = WIDE.with_(name="large_tile", n_layers=2, hidden=2112, inter=512, n_q_heads=4, batch=2, prefill=2050, tp_degree=1, peer_pool=0)
    res = harness.run_case(w, decode_steps=0, gen_device="cuda:0")
    assert max(res.errs) < TOL * 2 ** 0.5, res.errs


@pytest.mark.parametrize("rows", [385, 400, 500])
def test_swiglu_epilogue_of_the_largest_tile(harness, rows):
    """256 x 256 tiles with SwiGLU as epilogue (taken up to 1024 rows), ragged in both directions: 129, 144 and 244 rows and three
    quarters of the columns in the last tiles."""
    w = WIDE.with_(name="large_tile_swiglu", hidden=2112, inter=14304, n_q_heads=4, prefill=rows)
    res = harness.run_case(w, decode_steps=0, gen_device="cuda:0")
    assert max(res.errs) < TOL, res.errs


@pytest.mark.parametrize("rows", [100, 1100])
def test_embeddings_off_a_16_byte_boundary(harness, rows):
    """The same bits wherever the call's input lies (the residual update of module 1 reads it 16 bytes at a time beyond 1024 rows)."""
    w = WIDE.with_(name="offset_input", hidden=512, inter=416, n_q_heads=4, prefill=rows)
    ctx = harness.build_gpu(w, harness.make_tensors(w))
    x = inputs.embeddings(w, 1, rows, inputs.SEED_PREFILL, "cuda:0")
    want = ctx.prefill(x)
    held = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
    for shift in (4, 8):     # elements: 8 and 16 bytes
        at = held[shift:shift + x.numel()].view(x.shape)
        at.copy_(x)
        assert torch.equal(want, ctx.prefill(at)), shift
    ctx.free()


@pytest.mark.parametrize("n_layers", [3, 4])
def test_module_streams_leave_the_same_bits(harness, n_layers):
    """Calls that run attention and MLP modules on two streams (65 - 256 and 513 - 1024 rows of four layers of 190 MB, 256 and 513 - 1024 of three) against the
    same calls in order, with calls of other row counts in between and decode steps behind them."""
    w = WIDE.with_(name="streams", n_layers=n_layers, hidden=4096, inter=6144, prefill=1024)
    tensors = harness.make_tensors(w, "cuda:0")
    side, order = (harness.build_gpu(w, tensors, overlap_modules=v) for v in (1, 0))
    x = inputs.embeddings(w, 1, 1024, inputs.SEED_PREFILL, "cuda:0")
    for rows in (100, 256, 257, 513, 1024, 65, 100):
        calls = []
        for ctx in (side, order):
            out = [ctx.prefill(x[:, :rows].contiguous())]
            out += [ctx.decode_step(x[:, i].contiguous()) for i in range(2)]
            calls.append(out)
        for a, b in zip(*calls):
            assert torch.equal(a, b), rows
    side.free()
    order.free()


def test_wide_decode_replayed_from_a_graph(harness):
    """Every replay of a captured wide step against the eager steps, with eager work and a synchronisation between them."""
    import numpy as np
    w = WIDE.with_(name="wide_graph", hidden=256, inter=352, n_q_heads=4, batch=17, prefill=0, kv_preload=126, decode_steps=5)
    eager = harness.run_case(w, kv_preload=126, decode_steps=5, gpu_only=True, max_tokens=1, decode_graph=0)
    graph = harness.run_case(w, kv_preload=126, decode_steps=5, gpu_only=True, max_tokens=1, decode_graph=1)
    for a, b in zip(eager.gpu, graph.gpu):      # (run_case copies every step's result to the host)
        assert np.array_equal(a, b)


@pytest.mark.parametrize("batch", [64, 65, 100, 257])
def test_decode_of_many_sequences_under_every_schedule(harness, batch):
    """Steps of a layer that prompts of as many rows run on two streams: with module streams and in order, launched eagerly and replayed from a
    captured graph, the same bits; and the right ones (one layer's bound for each of the four)."""
    import numpy as np
    w = WIDE.with_(name="many_sequences", n_layers=4, hidden=2112, inter=9152, n_q_heads=8, batch=batch, prefill=0, kv_preload=70, decode_steps=3)
    tensors = harness.make_tensors(w, "cuda:0")
    runs = [harness.run_case(w, kv_preload=70, decode_steps=3, tensors=tensors, gen_device="cuda:0", gpu_only=i > 0, max_tokens=1, overlap_modules=overlap,
                             decode_graph=graph) for i, (overlap, graph) in enumerate(((1, 0), (1, 1), (0, 0), (0, 1)))]
    assert max(runs[0].errs) < TOL * 4 ** 0.5, runs[0].errs
    for r in runs[1:]:
        for a, b in zip(runs[0].gpu, r.gpu):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("rows", [17, 100, 300])
@pytest.mark.parametrize("hidden,inter", [(448, 32), (448, 416), (32, 64)])
def test_products_of_a_single_stage(harness, hidden, inter, rows):
    """K of 64 and less (one 64-wide q head, 32 hidden or SwiGLU columns) and splits of K whose last one is a single stage
    of 64 (448 in 3 and 416 in 3): the ring's start requests more stages than there are."""
    w = WIDE.with_(name="one_stage", hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=64, inter=inter, batch=1, prefill=rows)
    res = harness.run_case(w, decode_steps=0)
    assert max(res.errs) < TOL, res.errs


@pytest.mark.parametrize("shape", [dict(hidden=1024, n_q_heads=8, n_kv_heads=2, head_dim=128, inter=8192),
                                   dict(hidden=8192, n_q_heads=8, n_kv_heads=1, head_dim=128, inter=3584)])
def test_same_bits_in_contexts_of_any_capacity(harness, shape):
    """What a context was sized for does not change how a call's products are split (700 and 1000 rows: the number of partial
    products that would pay is larger than what the buffers of a small context hold)."""
    w = WIDE.with_(name="capacity", prefill=1024, **shape)
    tensors = harness.make_tensors(w, "cuda:0")
    big = harness.build_gpu(w, tensors, max_tokens=4096, max_batch=4, max_seq=4096)
    x = inputs.embeddings(w, 1, 1024, inputs.SEED_PREFILL, "cuda:0")
    for rows in (17, 100, 250, 300, 337, 700, 1000):
        own = harness.build_gpu(w, tensors, max_tokens=rows, max_seq=rows)
        want, got = big.prefill(x[:, :rows].contiguous()), own.prefill(x[:, :rows].contiguous())
        own.free()
        assert torch.equal(want, got), rows
    big.free()


# (rows, prompt or step, wiring): pairs of small tiles, small and tall, tall and large ones, SwiGLU from partial products, one token for each of many sequences
@pytest.mark.parametrize("batch,prefill", [(1, 17), (2, 32), (1, 65), (1, 128), (3, 67), (1, 256), (1, 257), (17, 1), (40, 1), (200, 1)])
@pytest.mark.parametrize("wiring", [ladder.LADDER_WIRING_LADDER, ladder.LADDER_WIRING_PARALLEL])
@pytest.mark.parametrize("hidden,inter", [(512, 1056), (4160, 416)])
def test_modules_that_share_launches_leave_the_same_bits(harness, batch, prefill, wiring, hidden, inter):
    """17 to 256 rows: the two modules' products in a launch each time and both residual updates in one, against one after the other on one stream:
    the same bits, and the right ones."""
    w = WIDE.with_(name="beside", n_layers=2, hidden=hidden, inter=inter, n_q_heads=4, n_kv_heads=2, head_dim=64, batch=batch, prefill=prefill,
                   tp_degree=3, n_real_shards=1, peer_pool=2)
    tensors = harness.make_tensors(w)
    runs = [harness.run_case(w, tensors=tensors, gpu_only=not on, decode_steps=1, wiring=wiring, overlap_modules=on, reduce_on_side_stream=0) for on in (1, 0)]
    assert max(runs[0].errs) < TOL, runs[0].errs
    for a, b in zip(*(r.gpu for r in runs)):
        assert np.array_equal(a, b)
