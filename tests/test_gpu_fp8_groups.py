"""e4m3 attention with an item's key tiles dealt to three wave groups: tile
counts of every remainder, partial last tiles, unit-local items of fewer
tiles than groups, every GQA group size, against the oracle."""
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


@pytest.mark.parametrize("hq,scope,unit,tail", [
    (32, "global", 272, 1), (32, "global", 272, 17), (32, "global", 288, 32),
    (32, "local", 32, 20), (32, "local", 272, 40),
    (8, "global", 272, 13), (16, "local", 272, 13), (64, "global", 272, 13),
])
def test_wave_groups(hq, scope, unit, tail):
    cfg = workloads.get_config("small_fp8")
    shape = cfg.model.__class__(**{**vars(cfg.model), "n_q_heads": hq})
    n = 1100 // unit + 1 if unit < 100 else 4
    pattern = tuple(i % 2 for i in range(n))
    wl = workloads.make_workload(cfg.with_(
        model=shape, n_requests=1, units_per_request=n, unit_tokens=unit, pool_units=n,
        residency_pattern=pattern, unit_order=(tuple(range(n)),), miss_scope=scope,
        instruction_tokens=16, query_tokens=tail, extra={}))
    run = GpuRun(wl, attn_kernel=4)
    assert run.plan.attn_rows_per_item == 32 and run.plan.attn_wave_groups == 3
    check_request(run, 0)
