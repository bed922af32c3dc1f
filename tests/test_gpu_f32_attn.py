"""The fp32 attention kernel at its edges: every head dim, GQA groups, key
ranges around its 16-key tiles and 16-row blocks, and a V that is not finite
at a position later than the rows it shares a tile with."""
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


def _workload(d, hq, hkv, scope="global", **kw):
    cfg = workloads.get_config("small_f32")
    shape = cfg.model.__class__(**{**vars(cfg.model), "head_dim": d, "n_q_heads": hq,
                                   "n_kv_heads": hkv})
    return workloads.make_workload(cfg.with_(model=shape, miss_scope=scope, **kw))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("hq,hkv,scope,kw", [
    (4, 4, "global", dict(unit_tokens=(15, 17))),
    (8, 2, "local", {}),
    (3, 1, "global", dict(unit_tokens=(31, 33), query_tokens=1, instruction_tokens=0)),
    (4, 2, "global", dict(unit_tokens=(200, 300), n_recompute=1)),
])
def test_f32_shapes(d, hq, hkv, scope, kw):
    wl = _workload(d, hq, hkv, scope, **kw)
    run = GpuRun(wl)
    for r in range(len(wl.requests)):
        check_request(run, r)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_f32_later_v_does_not_reach_earlier_rows(d, bad):
    run = GpuRun(_workload(d, 4, 2))
    s, plan = run.sess, run.plan
    want = run.out.clone()
    last = run.rows_of(0)[-1]         # request 0's last prompt position
    v = run.v.clone()
    v[last, 0, 3] = bad
    s.append(plan, run.k, v)
    out, lse = s.new_outputs(plan, True)
    s.attn(plan, run.q, out, lse)
    torch.cuda.synchronize()
    # rows up to it sum the same keys; within its tile one row at a time, in
    # another order of the 64-bit sums: within one fp32 rounding
    hit = torch.zeros_like(out, dtype=torch.bool)
    hit[last, :2, 3] = True           # the query heads of KV head 0
    assert not torch.isfinite(out[hit]).any()
    assert torch.isfinite(out[~hit]).all()
    err = (out[~hit].double() - want[~hit].double()).norm() / want[~hit].double().norm()
    assert err <= 2.0 ** -24, float(err)
