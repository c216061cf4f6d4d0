"""The merge launches at the edges of their part counts, on the GPU: rows of
1 and of 8 parts (one thread per unit), 9 (the first count that four waves
share), 32 and 33 (one and two batches of a wave's parts) and 66."""

from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2608_25523_amd import binding as B  # noqa: E402
from paper_2608_25523_amd import runner as RN  # noqa: E402
from paper_2608_25523_amd import workloads as W  # noqa: E402
from test_gpu_parity import announce, assert_untouched, run_and_check  # noqa: E402
import parity as PT  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,hq,hkv", [(128, 32, 8), (64, 6, 3)])
@pytest.mark.parametrize("parts", [1, 8, 9, 32, 33, 66])
def test_merge_part_counts(parts, d, hq, hkv):
    """One-step pieces: a request over parts - 1 prefix steps and one suffix
    step has `parts` parts, one without a prefix as many suffix steps, and a
    row of few parts sits beside them.  Against the oracle, and pfx_step
    (append folded into the merge) against append + attention bit for bit."""
    plen = 32 * (parts - 1)
    b = W.make_batch(300 + parts, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512,
                     prefix_len=[plen, 20], agent=[0, -1, 1, 0], suffix_len=[7, 32 * parts - 5, 3, 32],
                     n_rows=[1, 1, 2, 1])
    hv = W.host_values(b, 400 + parts)
    ds, o_ref, l_ref = run_and_check(b, hv, f"merge-parts-{parts}-d{d}", piece_steps=1)
    assert int(ds.plan.export(7)[:, 1].max()) == max(parts, 2)
    del ds
    ds = RN.DeviceStep(b, hv, piece_steps=1)
    B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse)
    B.pfx_sync_check()
    o, l = ds.outputs()
    assert np.array_equal(o, o_ref) and np.array_equal(l, l_ref)
    exp_k, exp_v = PT.expected_pools(b, hv)
    gk, gv = ds.read_pages(hv.pages)
    assert np.array_equal(gk, exp_k) and np.array_equal(gv, exp_v)
    assert_untouched(ds, hv.pages, "merge-parts step")
    announce(f"merge parts {parts} d={d}: step equals append + attention")


@pytest.mark.parametrize("d,hq,hkv", [(128, 32, 8), (64, 8, 2)])
def test_lone_short_items_round_once(d, hq, hkv):
    """Requests without a prefix, of 97 to 512 keys, in a small launch: the
    bits of 16-step pieces, which hold each row in one fp32 state."""
    lens = [97, 160, 288, 512]
    b = W.make_batch(310, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=[700],
                     agent=[-1] * 4 + [0], suffix_len=lens + [100], n_rows=[1] * 5)
    hv = W.host_values(b, 311)
    _, o16, l16 = run_and_check(b, hv, f"lone items, 16 steps, d={d}", piece_steps=16)
    _, o, l = run_and_check(b, hv, f"lone items, d={d}")
    assert np.array_equal(o[:4], o16[:4]) and np.array_equal(l[:4], l16[:4])


@pytest.mark.parametrize("d,hq,hkv", [(128, 32, 8), (64, 6, 3)])
def test_rows_do_not_depend_on_longer_ones(d, hq, hkv):
    """At a fixed piece length a request without a prefix has the same bits
    alone and beside one whose rows have more than eight parts."""
    for parts in (1, 4, 8, 9):
        lens = [32 * 4 * parts - 5, 32 * 4 * 10]
        b = W.make_batch(420, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=[],
                         agent=[-1, -1], suffix_len=lens, n_rows=[1, 1])
        hv = W.host_values(b, 420)
        ds, o2, l2 = run_and_check(b, hv, f"{parts} parts beside 10, d={d}", piece_steps=4)
        assert ds.plan.export(7)[:, 1].reshape(2, hkv)[:, 0].tolist() == [parts, 10]
        alone = B.pfx_plan_create(ds.pool, [0], [], [], [-1], [0, len(b.suffix_pages[0])], b.suffix_pages[0],
                                  lens[:1], [0, 1], hq, B.PFX_MODE_DECODE, piece_steps=4).upload()
        B.pfx_attention(ds.pool, alone, ds.q, ds.o, ds.lse)
        B.pfx_sync_check()
        o1, l1 = ds.outputs()
        assert np.array_equal(o1[0], o2[0]) and np.array_equal(l1[0], l2[0])


@pytest.mark.parametrize("d,hq,hkv", [(128, 32, 8), (64, 32, 8)])
def test_fixed_length_rows_of_an_agent(d, hq, hkv):
    """At a fixed piece length a request with a prefix has the same bits alone
    and among 16 of its agent (64 columns: no wide blocks), one of them with
    more than eight parts."""
    lens = [50, 1500] + [30 + 13 * i for i in range(14)]
    b = W.make_batch(430, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=[700],
                     agent=[0] * 16, suffix_len=lens, n_rows=[1] * 16)
    hv = W.host_values(b, 431)
    ds, o16, l16 = run_and_check(b, hv, f"16 requests of an agent, d={d}", piece_steps=4)
    assert ds.plan.stats().num_wide_blocks == 0
    pp, sp = b.prefix_pages[0], b.suffix_pages
    for r in (0, 1, 9):
        one = B.pfx_plan_create(ds.pool, [0, len(pp)], pp, [700], [0], [0, len(sp[r])], sp[r], lens[r:r + 1], [0, 1],
                                hq, B.PFX_MODE_DECODE, piece_steps=4).upload()
        o, l = torch.empty_like(ds.o[:1]), torch.empty_like(ds.lse[:1])
        B.pfx_attention(ds.pool, one, ds.q[r:r + 1], o, l)
        B.pfx_sync_check()
        assert np.array_equal(RN.to_host_bits(o)[0], o16[r]) and np.array_equal(l.cpu().numpy()[0], l16[r])
