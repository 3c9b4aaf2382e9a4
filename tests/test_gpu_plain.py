"""GPU: the plain kernels (fp32 storage, odd sizes, bf16 on request) at the edges of their tiles, passes and chunks, against
the CPU oracle; all computed shards share a launch."""
import numpy as np
import pytest
import torch

from paper_2501_06589_amd import inputs, ladder

pytestmark = pytest.mark.gpu

BASE = inputs.WORKLOADS["tiny"].with_(name="plain", n_layers=1, tp_degree=3, n_real_shards=3, decode_steps=2)


@pytest.fixture(scope="module")
def harness():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import gpu_harness
    return gpu_harness


# K of one pass and less, a pass more, ragged; N inside one column block, a multiple of 4 and not
@pytest.mark.parametrize("hidden,nq,nkv,d,inter", [(8, 1, 1, 2, 1), (256, 3, 3, 30, 345), (264, 4, 2, 64, 63), (520, 2, 1, 250, 257)])
@pytest.mark.parametrize("rows", [1, 4, 5, 64, 65])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_sizes(harness, hidden, nq, nkv, d, inter, rows, dtype):
    w = BASE.with_(hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, inter=inter, prefill=rows, dtype=dtype)
    res = harness.run_case(w, kernel_path=ladder.LADDER_PATH_GENERIC)
    # (one layer of bf16 roundings between the modules: the prefill bound of the other tests)
    assert max(res.errs) < (1e-4 if dtype == "fp32" else 0.0029 * 2 ** 0.5 * 5.8), res.errs


@pytest.mark.parametrize("wiring,n_std", [(ladder.LADDER_WIRING_LADDER, 0), (ladder.LADDER_WIRING_LADDER, 1), (ladder.LADDER_WIRING_LADDER, 2),
                                          (ladder.LADDER_WIRING_STANDARD, 0), (ladder.LADDER_WIRING_PARALLEL, 0)])
@pytest.mark.parametrize("n_layers,rows,shards", [(1, 5, 2), (3, 1, 2), (3, 64, 2), (3, 65, 2), (3, 1, 9), (3, 3, 9)])
def test_rows_made_where_they_are_multiplied(harness, wiring, n_std, n_layers, rows, shards):
    """Up to 64 rows the stream is summed and normed by the projections that read it: one or two module outputs behind a stored
    stream, peers among them, more partial sums than are requested at once; 65 rows and too many pieces take the reduce kernel."""
    if n_std > n_layers:
        pytest.skip("more standard layers than layers")
    w = BASE.with_(name="made", n_layers=n_layers, prefill=rows, hidden=264, inter=96, tp_degree=shards + 1, n_real_shards=shards, peer_pool=2)
    res = harness.run_case(w, wiring=wiring, n_standard_layers=n_std)
    assert max(res.errs) < 1e-4, res.errs


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("rows,shards", [(32, 1), (36, 1), (8, 4), (12, 4)])
def test_as_many_workgroups_as_the_chip_holds_and_more(harness, dtype, rows, shards):
    """512 workgroups of four rows in the gate/up projection, and 576 and 768: one sweep over gate and up or two, rows made by the projections or not
    (bf16), with a row block that is not full behind them (the steps)."""
    w = BASE.with_(name="held", n_layers=2, prefill=rows, hidden=136, inter=4096, tp_degree=shards, n_real_shards=shards, dtype=dtype)
    res = harness.run_case(w, kernel_path=ladder.LADDER_PATH_GENERIC)
    assert max(res.errs) < (1e-4 if dtype == "fp32" else 0.0029 * 4 ** 0.5 * 5.8), res.errs


# (hidden: one, two and four pieces per thread, some of them behind the row's end, and rows too long for that; shards, peers: sums of 0 - 9 pieces)
@pytest.mark.parametrize("hidden,shards,peers", [(1024, 1, 1), (1032, 2, 2), (2056, 3, 0), (4088, 9, 1), (4104, 1, 7), (8200, 6, 1), (16384, 5, 3), (16392, 2, 6)])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_reduce_of_rows_of_any_length(harness, hidden, shards, peers, dtype):
    """65 rows take the reduce kernel: its pieces of a row in registers and its sums, four requested at a time."""
    if dtype == "bf16" and hidden > 8200:
        # (5.8 sigma of an average element bounds the errors of some 10^5 of them; the 65 x 16384 of longer rows, whose sigma differs by row, reach
        # 6.2 with a mean square as small as that of the others.  8200 columns take the same kernel)
        pytest.skip("more elements than the bound is made for")
    w = BASE.with_(name="reduce", hidden=hidden, n_q_heads=1, n_kv_heads=1, head_dim=32, inter=40, prefill=65, tp_degree=shards + peers,
                   n_real_shards=shards, dtype=dtype)
    res = harness.run_case(w, kernel_path=ladder.LADDER_PATH_GENERIC)
    assert max(res.errs) < (1e-4 if dtype == "fp32" else 0.0029 * 2 ** 0.5 * 5.8), res.errs


@pytest.mark.parametrize("cached", [63, 64, 255, 256, 700])
def test_attention_chunks(harness, cached):
    """One step behind a handed-over cache: part of a chunk, whole chunks, more chunks than wavefronts."""
    w = BASE.with_(batch=2, prefill=0, kv_preload=cached, n_q_heads=4, n_kv_heads=2)
    res = harness.run_case(w, kv_preload=cached)
    assert max(res.errs) < 1e-4, res.errs


@pytest.mark.parametrize("dtype,batch,nq,nkv,cached", [("fp32", 2, 2, 2, 300), ("fp32", 1, 4, 2, 700), ("bf16", 17, 2, 2, 300),
                                                       ("bf16", 17, 4, 1, 1025)])
def test_stretches_of_scores_of_minus_infinity(harness, dtype, batch, nq, nkv, cached):
    """Cached keys whose scores are -inf, whole chunks of them (64 positions in the plain kernel, 32 in the one of wide bf16
    batches, and whole splits of that): they weigh nothing, as keys with a huge negative score do; same bits."""
    w = BASE.with_(name="minus_inf", dtype=dtype, tp_degree=1, n_real_shards=1, hidden=256, inter=352, n_q_heads=nq, n_kv_heads=nkv,
                   head_dim=64, batch=batch, prefill=0, kv_preload=cached, decode_steps=1)
    tensors = harness.make_tensors(w)
    t = tensors[0][0]
    k, v = inputs.kv_cache(w, 0, 0, batch, cached)
    x = inputs.embeddings(w, batch, 1, inputs.SEED_DECODE0)[:, 0]
    # the step's rotated queries, and for each kv head a dim in which its q heads agree in sign
    xd = x.double()
    y = xd / torch.sqrt((xd * xd).mean(-1, keepdim=True) + w.rms_eps) * t["attn_norm"].double()
    q = (y @ t["wq"].double()).view(batch, nkv, nq // nkv, 32, 2)
    ang = cached * w.rope_theta ** (-torch.arange(0, 64, 2, dtype=torch.float64) / 64)
    q = torch.stack([q[..., 0] * ang.cos() - q[..., 1] * ang.sin(), q[..., 0] * ang.sin() + q[..., 1] * ang.cos()], -1).flatten(-2)
    agree = torch.maximum(q.amin(2), -q.amax(2))                    # [batch][kv head][dim]: positive where the signs agree
    dim = agree.argmax(-1, keepdim=True)
    assert float(agree.gather(-1, dim).min()) > 0.02
    sign = q[:, :, 0].gather(-1, dim).sign()
    outs = []
    for huge in (1e9, float("inf")):      # (1e9 x 0.02 / 8 = 2.5e6: the weight is exactly 0 as well)
        kk = k.clone()
        row = torch.zeros(batch, nkv, 64, dtype=k.dtype).scatter(-1, dim, (-huge * sign).to(k.dtype))
        for a, b in ((32, 64), (96, 256), (640, 700), (384, 1020)):
            kk[:, :, a:min(b, cached)] = row[:, :, None]
        ctx = harness.build_gpu(w, tensors, max_tokens=1)
        ctx.load_kv(0, 0, kk.cuda(), v.cuda())
        outs.append(ctx.decode_step(x.contiguous().cuda()).cpu())
        ctx.free()
    assert torch.isfinite(outs[0]).all() and torch.equal(*outs)


@pytest.mark.parametrize("rows", [30, 100, 1100])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_more_tiles_than_the_chip_holds(harness, dtype, rows):
    """The order in which blocks take the tiles of a large grid: one ragged group of row blocks and several (of 64 x 16 rows), tile
    counts that are no multiple of 8; fp32 tiles with the shorter pass over K, K no multiple of it."""
    w = BASE.with_(tp_degree=1, n_real_shards=1, hidden=264, n_q_heads=4, n_kv_heads=2, head_dim=66, inter=6500, prefill=rows, dtype=dtype)
    res = harness.run_case(w, kernel_path=ladder.LADDER_PATH_GENERIC, gen_device="cuda:0")
    assert max(res.errs) < (1e-4 if dtype == "fp32" else 0.0029 * 2 ** 0.5 * 5.8), res.errs


def test_overlapped_schedules_of_the_plain_path(harness):
    """Layers of 32 MB and more run their modules on two streams, or the reduces on a side stream, smaller ones in order: the
    schedules give the same bits, and the right ones."""
    w = BASE.with_(name="overlap", n_layers=3, hidden=1024, n_q_heads=8, n_kv_heads=4, head_dim=128, inter=1409, tp_degree=4,
                   n_real_shards=2, batch=2, prefill=9, decode_steps=3, peer_pool=2)
    assert w.params_per_layer() * w.n_real_shards * 4 >= 32 << 20
    tensors = harness.make_tensors(w, "cuda:0")
    runs = [harness.run_case(w, tensors=tensors, gen_device="cuda:0", gpu_only=i > 0, overlap_modules=overlap, reduce_on_side_stream=side)
            for i, (overlap, side) in enumerate(((0, 0), (1, 1), (0, 1)))]
    assert max(runs[0].errs) < 1e-4, runs[0].errs
    for r in runs[1:]:
        for a, b in zip(runs[0].gpu, r.gpu):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("dtype,inter", [("fp32", 96), ("bf16", 96), ("fp32", 2800), ("bf16", 5600)])
@pytest.mark.parametrize("wiring", [ladder.LADDER_WIRING_LADDER, ladder.LADDER_WIRING_STANDARD, ladder.LADDER_WIRING_PARALLEL])
def test_schedule_switches_leave_the_bits(harness, wiring, dtype, inter):
    """One computed shard, a row and a few: layers below 32 MB, whose projections sum and norm the rows themselves, and beyond, which run on
    two streams, with a side stream or in order as they are told, with and without an emulated latency: the same bits from all of them."""
    w = BASE.with_(name="switches", dtype=dtype, n_layers=3, hidden=1024, n_q_heads=4, n_kv_heads=2, head_dim=64, inter=inter, tp_degree=2,
                   n_real_shards=1, prefill=5, peer_pool=2)
    assert (w.params_per_layer() * (4 if dtype == "fp32" else 2) >= 32 << 20) == (inter > 96)
    tensors = harness.make_tensors(w, "cuda:0")
    runs = [harness.run_case(w, tensors=tensors, gen_device="cuda:0", gpu_only=i > 0, wiring=wiring, kernel_path=ladder.LADDER_PATH_GENERIC,
                             overlap_modules=overlap, reduce_on_side_stream=side, reduce_delay_us=delay)
            for i, (overlap, side, delay) in enumerate(((0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 20), (1, 1, 20)))]
    # (three layers of bf16 roundings between the modules)
    assert max(runs[0].errs) < (1e-4 if dtype == "fp32" else 0.0029 * 6 ** 0.5 * 5.8), runs[0].errs
    for r in runs[1:]:
        for a, b in zip(runs[0].gpu, r.gpu):
            assert np.array_equal(a, b)


def test_more_blocks_than_one_grid_dimension_takes(harness):
    """4 million rows, the most that 64-row tiles in the second grid dimension took: projections and attention have more than
    2^24 blocks of 256 threads each. The last sequences come out as in a call of their own."""
    w = BASE.with_(name="many_blocks", dtype="bf16", tp_degree=1, n_real_shards=1, hidden=8, n_q_heads=5, n_kv_heads=1, head_dim=2,
                   inter=4160, batch=32767, prefill=128, decode_steps=0)
    assert w.batch * w.prefill * w.n_q_heads > 1 << 24 and w.batch * w.prefill // 16 * (w.inter // 64) > 1 << 24
    tensors = harness.make_tensors(w)
    x = inputs.embeddings(w, w.batch, w.prefill, inputs.SEED_PREFILL, "cuda:0")
    ctx = harness.build_gpu(w, tensors, kernel_path=ladder.LADDER_PATH_GENERIC)
    got = ctx.prefill(x)
    ctx.free()
    few = harness.build_gpu(w.with_(batch=64), tensors, kernel_path=ladder.LADDER_PATH_GENERIC)
    for first in (0, 16384, w.batch - 64):
        assert torch.equal(got[first:first + 64], few.prefill(x[first:first + 64].contiguous())), first
    few.free()


@pytest.mark.parametrize("wiring", [ladder.LADDER_WIRING_LADDER, ladder.LADDER_WIRING_STANDARD, ladder.LADDER_WIRING_PARALLEL])
@pytest.mark.parametrize("dtype,n_layers,rows,path", [("fp32", 1, 64, ladder.LADDER_PATH_GENERIC), ("bf16", 1, 1, ladder.LADDER_PATH_GENERIC),
                                                      ("bf16", 1, 64, ladder.LADDER_PATH_GENERIC), ("bf16", 2, 64, ladder.LADDER_PATH_GENERIC),
                                                      ("bf16", 1, 10, ladder.LADDER_PATH_AUTO), ("bf16", 1, 1100, ladder.LADDER_PATH_AUTO)])
def test_input_and_output_in_the_same_memory(harness, wiring, dtype, n_layers, rows, path):
    """A prefill and a decode step whose input lies at the start, in the middle and at the end of their output's memory (fp32: a quarter
    before it, in it, a quarter behind): the same bits as with buffers of their own (what writes the output must not read the input)."""
    w = BASE.with_(name="same_memory", dtype=dtype, tp_degree=1, n_real_shards=1, n_layers=n_layers, hidden=1024, n_q_heads=4, n_kv_heads=2,
                   head_dim=64, inter=352, prefill=rows)
    ctx = harness.build_gpu(w, harness.make_tensors(w), wiring=wiring, kernel_path=path)
    x = inputs.embeddings(w, 1, rows, inputs.SEED_PREFILL, "cuda:0")
    e = inputs.embeddings(w, 1, 1, inputs.SEED_DECODE0, "cuda:0")[:, 0].contiguous()
    want = ctx.prefill(x), ctx.decode_step(e)
    for place in (0, 1, 2):
        got = []
        for call, given in ((ctx.prefill, x), (ctx.decode_step, e)):
            n = given.numel()
            held = torch.empty(2 * n, dtype=torch.float32, device=given.device)
            out = held[n // 2:n // 2 + n].view(given.shape)
            first = (n // 4, n // 2, 3 * n // 4) if dtype == "fp32" else (n, 3 * n // 2, 2 * n)     # in elements of the input
            at = held.view(x.dtype)[first[place]:first[place] + n].view(given.shape)
            at.copy_(given)
            got.append(call(at, out))
        for a, b in zip(want, got):
            assert torch.equal(a, b), place
    ctx.free()


@pytest.mark.parametrize("dtype,hidden,nq,nkv,d,inter,rows,shards,n_std,n_layers", [
    ("fp32", 264, 3, 3, 30, 345, 1, 2, 0, 3),      # weights and cache rows element by element
    ("fp32", 264, 4, 2, 30, 96, 5, 2, 1, 3),       # behind a standard layer
    ("fp32", 136, 2, 1, 64, 3840, 32, 1, 0, 2),    # QKV and gate/up: 512 workgroups together
    ("fp32", 136, 2, 1, 64, 3841, 32, 1, 0, 2),    # and more
    ("fp32", 136, 7, 7, 16, 64, 64, 1, 0, 2),      # attention and down: 496
    ("fp32", 136, 8, 8, 16, 64, 64, 1, 0, 2),      # 560
    ("bf16", 256, 4, 2, 64, 352, 1, 1, 0, 1),
    ("bf16", 264, 4, 2, 64, 345, 9, 2, 0, 2),      # (bf16 weights one by one: reduce kernel)
])
def test_modules_beside_each_other(harness, dtype, hidden, nq, nkv, d, inter, rows, shards, n_std, n_layers):
    """A layer's modules share launches where the MLP does not read the attention's output and two workgroups per CU hold them; with an emulated
    latency they run one after the other: the same bits, and the right ones."""
    w = BASE.with_(name="beside", dtype=dtype, n_layers=n_layers, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, inter=inter, prefill=rows,
                   tp_degree=shards + 1, n_real_shards=shards, peer_pool=2)
    tensors = harness.make_tensors(w)
    runs = [harness.run_case(w, tensors=tensors, gpu_only=delay > 0, n_standard_layers=n_std, kernel_path=ladder.LADDER_PATH_GENERIC,
                             reduce_delay_us=delay) for delay in (0, 5)]
    assert max(runs[0].errs) < (1e-4 if dtype == "fp32" else 0.0029 * (2 * n_layers) ** 0.5 * 5.8), runs[0].errs
    for a, b in zip(*(r.gpu for r in runs)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("nq,nkv,d", [(1, 1, 64), (2, 1, 64), (2, 2, 66), (4, 2, 64), (4, 4, 30), (2, 1, 130)])
@pytest.mark.parametrize("cached", [1, 62, 63, 126, 127, 200, 254, 255])
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_attention_with_its_output_projection(harness, nq, nkv, d, cached, dtype):
    """One row whose attention and output projection share a launch behind a short cache (256 positions times heads; heads of at most 256 elements
    together), at the edges of that and of a wavefront's chunk: the same bits as the launches by themselves."""
    w = BASE.with_(name="attn_out", dtype=dtype, hidden=264, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, inter=96, prefill=0, kv_preload=cached,
                   tp_degree=2, n_real_shards=2)
    tensors = harness.make_tensors(w)
    runs = [harness.run_case(w, tensors=tensors, kv_preload=cached, gpu_only=delay > 0, kernel_path=ladder.LADDER_PATH_GENERIC,
                             reduce_delay_us=delay) for delay in (0, 5)]
    assert max(runs[0].errs) < (1e-4 if dtype == "fp32" else 0.0029 * 2 ** 0.5 * 5.8), runs[0].errs
    for a, b in zip(*(r.gpu for r in runs)):
        assert np.array_equal(a, b)
