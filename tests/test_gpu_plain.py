"""GPU: the plain kernels (fp32 storage, odd sizes, bf16 on request) at the edges of their tiles, passes and chunks, against
the CPU oracle; all computed shards share a launch."""
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


@pytest.mark.parametrize("cached", [63, 64, 255, 256, 700])
def test_attention_chunks(harness, cached):
    """One step behind a handed-over cache: part of a chunk, whole chunks, more chunks than wavefronts."""
    w = BASE.with_(batch=2, prefill=0, kv_preload=cached, n_q_heads=4, n_kv_heads=2)
    res = harness.run_case(w, kv_preload=cached)
    assert max(res.errs) < 1e-4, res.errs
