"""One plan on two streams at once: calls of plans without split items share
nothing, so each gives the bits of the call alone.  A prompt of 28 key tiles
(bf16: whole under the automatic rule) and of 36 (e4m3: three wave groups)."""
import pytest
import torch

import workloads
from paper_2609_32999_amd import staging
from paper_2609_32999_amd.session import Session

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2609_32999_amd as P
    P.lib()   # fail loudly if the library is missing


@pytest.mark.parametrize("name,unit,groups", [("small_bf16", 208, 1), ("small_fp8", 272, 3)])
def test_two_streams(name, unit, groups):
    wl = workloads.make_workload(workloads.get_config(name).with_(
        n_requests=1, units_per_request=4, unit_tokens=unit, pool_units=4,
        residency_pattern=(0, 1, 0, 1), unit_order=((0, 1, 2, 3),), instruction_tokens=32,
        query_tokens=17, extra={}))
    s = Session(wl.model, wl.n_pool_pages, wl.n_req_pages)
    staging.upload_pool(s, wl)
    plan = s.plan(wl.requests, attn_kernel=4)
    assert plan.num_attn_splits == 0 and plan.attn_wave_groups == groups
    q, k, v = staging.fresh_inputs(s, wl, plan)
    s.assemble(plan, k, v)
    qs = [q, q.flip(0).contiguous()]
    want = [s.new_outputs(plan) for _ in qs]
    got = [s.new_outputs(plan) for _ in qs]
    for x, (out, lse) in zip(qs, want):
        s.attn(plan, x, out, lse)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in qs]
    for _ in range(20):
        for st, x, (out, lse) in zip(streams, qs, got):
            s.attn(plan, x, out, lse, stream=st)
    torch.cuda.synchronize()
    for (a, b), (c, d) in zip(want, got):
        assert torch.equal(a.view(torch.int16), c.view(torch.int16)) and torch.equal(b, d)
