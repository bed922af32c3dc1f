"""Attention output rows at the edges of the output store: row blocks that end
after 1, 15, 16, 17, 31 or 32 rows, consecutive and scattered, next to rows of
memory that must stay as they were."""
import pytest
import torch

import workloads
from gpu_harness import GpuRun, check_request

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2609_32999_amd as P
    P.lib()   # fail loudly if the library is missing


@pytest.mark.parametrize("tail", [1, 15, 16, 17, 31, 32])
@pytest.mark.parametrize("name,kernel,hit,hq", [
    ("small_bf16", 4, 0, 32), ("small_bf16", 3, 0, 32), ("small_bf16", 3, 1, 16),
    ("small_fp8", 4, 1, 32), ("small_fp8", 3, 0, 8), ("small_fp8", 3, 1, 64)])
def test_rows_of_a_block(name, kernel, hit, hq, tail):
    cfg = workloads.get_config(name)
    shape = cfg.model.__class__(**{**vars(cfg.model), "n_q_heads": hq})
    # 32 text rows, one unit (96 rows computed, or a window of 16), the tail
    wl = workloads.make_workload(cfg.with_(
        model=shape, n_requests=1, units_per_request=1, unit_tokens=96, pool_units=1,
        residency_pattern=(hit,), unit_order=((0,),), n_recompute=16, instruction_tokens=32,
        query_tokens=tail, extra={}))
    run = GpuRun(wl, attn_kernel=kernel)
    check_request(run, 0)
    # the same launch into the middle of a larger buffer
    T = run.plan.num_compute_tokens
    assert T == 32 + (16 if hit else 96) + tail
    big = torch.full((T + 64, *run.out.shape[1:]), 7.0, dtype=run.out.dtype, device="cuda")
    lse = torch.full((T + 64, hq), 7.0, device="cuda")
    run.sess.attn(run.plan, run.q, big[32:32 + T], lse[32:32 + T])
    torch.cuda.synchronize()
    assert torch.equal(big[32:32 + T].view(torch.int16), run.out.view(torch.int16))
    assert torch.equal(lse[32:32 + T].view(torch.int32), run.lse.view(torch.int32))
    for x in (big, lse):
        assert bool((x[:32] == 7.0).all()) and bool((x[32 + T:] == 7.0).all())
