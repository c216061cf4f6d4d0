"""Decode piece records of every length, on the GPU against the oracle: one row
and one step, whole and broken vectors of rows and of steps, the most of both,
fetched at a workgroup's start (one piece each) and by direct copies beside the
pieces before (three persistent workgroups)."""

from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_25523_amd import binding as B  # noqa: E402
from paper_2608_25523_amd import workloads as W  # noqa: E402
from test_gpu_parity import run_and_check  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [
    # (Hq, Hkv, d, rows of the agent, prefix, piece steps, most rows and steps of a piece)
    (32, 8, 128, 1, 0, 1, 1, 1),
    (16, 16, 64, 5, 96, 3, 5, 3),
    (8, 8, 128, 64, 2048, 64, 64, 64),
    (8, 8, 64, 63, 1810, 57, 63, 57),
    (8, 8, 128, 60, 1792, 56, 60, 56),
]


@pytest.mark.parametrize("engine", [B.PFX_DECODE_MFMA, B.PFX_DECODE_VALU])
@pytest.mark.parametrize("case", CASES, ids=[f"records{i}" for i in range(len(CASES))])
def test_record_lengths(case, engine):
    hq, hkv, d, rows, plen, piece, most_rows, most_steps = case
    b = W.make_batch(500 + rows, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=1024,
                     prefix_len=[plen], agent=[0] * rows, suffix_len=[17 + i % 15 for i in range(rows)],
                     n_rows=[1] * rows)
    hv = W.host_values(b, 501)
    ds, o, l = run_and_check(b, hv, "piece records", piece_steps=piece, decode_engine=engine)
    segs = ds.plan.export(3)
    assert int(segs[:, 2].max()) * hkv // hq == most_rows and int(segs[:, 3].max()) == most_steps
    _, o3, l3 = run_and_check(b, hv, "piece records, three workgroups", piece_steps=piece, decode_workers=3,
                              decode_engine=engine)
    assert np.array_equal(o, o3) and np.array_equal(l, l3)
