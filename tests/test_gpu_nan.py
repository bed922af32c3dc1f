"""Scores that are not numbers, where partial softmaxes are merged: a NaN
query, and a run of keys that are all NaN for the rows that see them.  A
partial softmax whose scores are all NaN has no maximum; it must not pass for
one that saw no key, so outputs and log-sum-exps of such rows are NaN, as without a
merge, and those of other rows are numbers."""
import numpy as np
import pytest
import torch

import workloads
from gpu_harness import GpuRun

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2609_32999_amd as P
    P.lib()   # fail loudly if the library is missing


def _attn(run, q):
    out, lse = run.sess.new_outputs(run.plan, with_lse=True)
    run.sess.attn(run.plan, q, out, lse)
    torch.cuda.synchronize()
    return out, lse


def _pages(run, lo, hi):
    """Request pages of positions lo .. hi - 1 of request 0."""
    req, b = run.wl.requests[0], run.wl.model.page_size
    return torch.as_tensor(np.asarray(req.block_table)[lo // b:hi // b].astype(np.int64),
                           device="cuda")


def _check_nan(got, rows):
    for t in got:
        assert torch.isnan(t[rows].float()).all()


def _check_finite(got, rows):
    for t in got:
        assert torch.isfinite(t[rows].float()).all()


def _bf16(kernel, split):
    wl = workloads.make_workload(workloads.get_config("small_bf16"))
    run = GpuRun(wl, attn_kernel=kernel, split_tiles=split)
    assert (run.plan.num_attn_splits > 0) == (split > 0)
    return run


def _fp8():
    cfg = workloads.get_config("small_fp8")
    wl = workloads.make_workload(cfg.with_(
        n_requests=1, units_per_request=4, unit_tokens=272, pool_units=4,
        residency_pattern=(0, 1, 0, 1), unit_order=((0, 1, 2, 3),), instruction_tokens=16,
        query_tokens=17, extra={}))
    run = GpuRun(wl, attn_kernel=4)
    assert run.plan.attn_wave_groups == 3
    return run


_PLANS = [(4, -1), (3, -1), (4, 2), (3, 2), (4, 5)]


@pytest.mark.parametrize("kernel,split", _PLANS)
def test_bf16_nan_query(kernel, split):
    run = _bf16(kernel, split)
    row = int(run.rows_of(0)[-1])
    q = run.q.clone()
    q[row] = float("nan")
    got = _attn(run, q)
    _check_nan(got, [row])
    _check_finite(got, [r for r in range(len(run.pos)) if r != row])


@pytest.mark.parametrize("kernel,split", _PLANS)
def test_bf16_nan_keys(kernel, split):
    """Keys 32 .. 319 of request 0: at least one whole range of 2 or 5 tiles."""
    run = _bf16(kernel, split)
    assert run.wl.requests[0].prompt_len > 320
    run.sess.req_k[0][_pages(run, 32, 320)] = float("nan")
    got = _attn(run, run.q)
    rows = run.rows_of(0)
    _check_nan(got, rows[run.pos[rows] >= 32])
    _check_finite(got, np.setdiff1d(np.arange(len(run.pos)), rows[run.pos[rows] >= 32]))


@pytest.mark.parametrize("first", [0, 1, 2])
def test_e4m3_nan_keys(first):
    """Every third key tile from `first` on: the tiles of one wave group."""
    run = _fp8()
    req = run.wl.requests[0]
    for j in range(first, (req.prompt_len + 31) // 32, 3):
        run.sess.req_scale[0][_pages(run, 32 * j, min(32 * j + 32, len(req.block_table) * 16)),
                              0] = float("nan")
    got = _attn(run, run.q)
    rows = run.rows_of(0)
    _check_nan(got, rows[run.pos[rows] >= 32 * first])
