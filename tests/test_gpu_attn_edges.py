"""bf16 attention where the last key tile ends: one to 32 keys in it, with
and without a whole 16-key block past the end, whose slots hold NaN.  The
staging waves take one 16-key block each and put another key's V in the
place of the missing ones."""
import pytest
import torch

import workloads
from gpu_harness import GpuRun, check_request, check_request_sentinels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2609_32999_amd as P
    P.lib()   # fail loudly if the library is missing


@pytest.mark.parametrize("last", [1, 15, 16, 17, 31, 32])
@pytest.mark.parametrize("kernel,page,alias_v", [(3, 16, False), (4, 16, False), (4, 32, False),
                                                 (3, 32, True), (4, 16, True)])
def test_last_tile(last, kernel, page, alias_v):
    cfg = workloads.get_config("small_bf16")
    shape = cfg.model.__class__(**{**vars(cfg.model), "page_size": page})
    # units of 64 tokens from position 32: the prompt ends `last` keys into a
    # tile; MISS, HIT, MISS, HIT
    wl = workloads.make_workload(cfg.with_(
        model=shape, n_requests=1, units_per_request=4, unit_tokens=64, pool_units=4,
        residency_pattern=(0, 1, 0, 1), unit_order=((0, 1, 2, 3),), instruction_tokens=32,
        query_tokens=last))
    assert (wl.requests[0].prompt_len - 1) % 32 + 1 == last
    run = GpuRun(wl, attn_kernel=kernel, alias_v=alias_v)
    check_request(run, 0, check_kv=not alias_v)
    if not alias_v:
        check_request_sentinels(run, 0)


@pytest.mark.parametrize("kernel", [3, 4])
@pytest.mark.parametrize("split,over", [
    (1, dict(unit_tokens=(250, 300), units_per_request=6, pool_units=8)),   # over 32 ranges
    (2, {}),
    (3, dict(n_recompute=1, instruction_tokens=0, query_tokens=1)),
    (5, dict(n_requests=1)),
])
def test_split_ranges_past_rows(kernel, split, over):
    """Every unit cached: an item's rows are recompute windows far apart, so
    most key ranges lie past some of its rows, which weigh nothing there."""
    wl = workloads.make_workload(workloads.get_config("small_bf16").with_(
        hit_prob=1.0, residency_pattern=None, **over))
    run = GpuRun(wl, attn_kernel=kernel, split_tiles=split)
    assert run.plan.num_attn_splits > 0
    for r in range(len(wl.requests)):
        check_request(run, r)
