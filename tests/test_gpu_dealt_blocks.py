"""Decode launches whose wide prefix blocks and pieces take turns in the grid,
on the GPU against the oracle: block counts on, past and below whole runs,
fewer pieces than blocks, and few persistent workgroups."""

from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_25523_amd import binding as B  # noqa: E402
from paper_2608_25523_amd import runner as RN  # noqa: E402
from paper_2608_25523_amd import workloads as W  # noqa: E402
from test_gpu_parity import assert_untouched, run_and_check  # noqa: E402
import parity as PT  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    # (requests, prefix tokens, options, wide blocks)
    (40, 256, dict(piece_steps=1), 128),                        # one run of blocks
    (40, 300, dict(piece_steps=1), 160),                        # one run and a part
    (40, 220, dict(piece_steps=1), 112),                        # less than a run
    (20, 1024, dict(piece_steps=1), 256),                       # more steps in the blocks: they stay in front
    (40, 300, dict(piece_steps=1, decode_workers=140), 160),
]


@pytest.mark.parametrize("case", CASES, ids=[f"dealt{i}" for i in range(len(CASES))])
def test_dealt_blocks(case):
    reqs, plen, opts, wide = case
    b = W.make_batch(120 + reqs, num_q_heads=32, num_kv_heads=8, head_dim=128, num_pages=512, prefix_len=[plen],
                     agent=[0] * reqs, suffix_len=[20 + 3 * i % 40 for i in range(reqs)], n_rows=[1] * reqs)
    hv = W.host_values(b, 121)
    ds, _, _ = run_and_check(b, hv, f"dealt {reqs} requests over {plen}", **opts)
    assert ds.plan.stats().num_wide_blocks == wide


@pytest.mark.parametrize("case", [CASES[1], CASES[4]], ids=["dealt1", "dealt4"])
def test_dealt_step(case):
    """The same grids with the append folded in: outputs and pool equal append
    + attention bit for bit, other pages untouched."""
    reqs, plen, opts, wide = case
    b = W.make_batch(130 + reqs, num_q_heads=32, num_kv_heads=8, head_dim=128, num_pages=512, prefix_len=[plen],
                     agent=[0] * reqs, suffix_len=[20 + 3 * i % 40 for i in range(reqs)], n_rows=[1] * reqs)
    hv = W.host_values(b, 131)
    ds, o_ref, l_ref = run_and_check(b, hv, f"dealt step, {reqs} requests over {plen}", **opts)
    assert ds.plan.stats().num_wide_blocks == wide
    del ds
    ds = RN.DeviceStep(b, hv, **opts)
    B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse)
    B.pfx_sync_check()
    o, l = ds.outputs()
    assert np.array_equal(o, o_ref) and np.array_equal(l, l_ref)
    exp_k, exp_v = PT.expected_pools(b, hv)
    gk, gv = ds.read_pages(hv.pages)
    assert np.array_equal(gk, exp_k) and np.array_equal(gv, exp_v)
    assert_untouched(ds, hv.pages, "dealt step")
