"""Extend blocks of small launches, cut and whole, on the GPU against the oracle: pieces that start in the
prefix, in the suffix and on the step between them, rows that see nothing of a
piece, blocks with padding columns, several blocks and requests, head_dim 64
and 128, G from 1 to 16, beside decode rows, without LSE, through the
allocation-free entry point, and with the append folded in."""

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

CASES = [
    # (Hq, Hkv, d, prefixes, requests (agent, L, n))
    (32, 8, 128, [1500], [(0, 33, 33)]),
    (32, 8, 128, [1501], [(0, 300, 70), (0, 20, 1), (-1, 5, 1)]),
    (32, 8, 128, [], [(-1, 1300, 300)]),
    (16, 16, 128, [17, 1200], [(0, 40, 40), (1, 130, 130), (-1, 9, 9)]),
    (32, 2, 64, [2033], [(0, 513, 100), (0, 20, 20), (0, 9, 1)]),
    (8, 8, 64, [1999], [(0, 129, 129)]),
]


@pytest.mark.parametrize("case", CASES, ids=[f"chunks{i}" for i in range(len(CASES))])
def test_cut_blocks(case):
    hq, hkv, d, plen, reqs = case
    b = W.make_batch(90, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=plen,
                     agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
    hv = W.host_values(b, 91)
    ds, o_ref, l_ref = run_and_check(b, hv, f"chunks Hq={hq} Hkv={hkv} d={d} {plen} {reqs}")
    # A cut plan's workspace holds the pieces' states: 512 d bytes a piece at least.
    assert ds.plan.workspace_bytes() > 8 * 512 * d
    plan = ds.plan
    run_and_check(b, hv, "chunks, no LSE", with_lse=False)
    ds = RN.DeviceStep(b, hv)
    B.pfx_attention_noalloc(ds.pool, plan, ds.q, ds.o, ds.lse, k_new=ds.k_new, v_new=ds.v_new)
    B.pfx_sync_check()
    o, l = ds.outputs()
    assert np.array_equal(o, o_ref) and np.array_equal(l, l_ref)
    announce("chunks: the allocation-free call gives the same bits")


def test_peaked_scores_in_cut_blocks():
    """Rising and one-hot scores: the pieces' maxima lie far apart."""
    b = W.make_batch(92, num_q_heads=32, num_kv_heads=8, head_dim=128, num_pages=512, prefix_len=[2000],
                     agent=[0, 0], suffix_len=[150, 40], n_rows=[150, 40])
    hv = W.host_values_shaped(b, 93, key_gain=lambda p: 1.0 + p / 256.0, q_gain=4.0, v_gain=0.25)
    run_and_check(b, hv, "chunks, rising scores")
    run_and_check(b, W.plant_one_hot(b, W.host_values(b, 94), 95, alpha_log2=4), "chunks, one-hot")


# (Hq, Hkv, d, prefixes, requests): new tokens that start inside a page, on a
# page and on a step, end on each of those, and share a page with old ones.
# Every row sees 17 keys or more: over two or three N(0, 1) values |O| passes 2,
# where the rounding of O alone is half of 2^-6 and with P's (2^-9 of each
# term) goes past the stated 1e-2.
STEPS = [
    (32, 8, 128, [1500], [(0, 300, 70), (0, 48, 32), (0, 64, 32), (0, 50, 33), (-1, 40, 23), (0, 20, 1), (0, 9, 4)]),
    (8, 2, 64, [100], [(0, 32, 32), (0, 47, 16), (-1, 34, 17), (0, 33, 5), (0, 16, 1)]),
    (16, 16, 128, [40], [(0, 140, 130), (0, 31, 31), (0, 90, 17), (-1, 48, 32)]),
    (32, 2, 64, [1000], [(0, 700, 51), (0, 65, 64), (-1, 37, 3)]),
]


@pytest.mark.parametrize("engine", [B.PFX_DECODE_MFMA, B.PFX_DECODE_VALU])
@pytest.mark.parametrize("case", STEPS, ids=[f"step{i}" for i in range(len(STEPS))])
def test_step_with_extend_blocks(case, engine):
    """pfx_step with the append folded into the extend blocks: outputs and pool
    equal append + attention bit for bit, other pages untouched."""
    hq, hkv, d, plen, reqs = case
    b = W.make_batch(96, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=plen,
                     agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
    hv = W.host_values(b, 97)
    ds, o_ref, l_ref = run_and_check(b, hv, f"step over {plen} {reqs}", decode_engine=engine)
    del ds
    ds = RN.DeviceStep(b, hv, decode_engine=engine)
    B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse)
    B.pfx_sync_check()
    o, l = ds.outputs()
    assert np.array_equal(o, o_ref) and np.array_equal(l, l_ref)
    exp_k, exp_v = PT.expected_pools(b, hv)
    gk, gv = ds.read_pages(hv.pages)
    assert np.array_equal(gk, exp_k) and np.array_equal(gv, exp_v)
    assert_untouched(ds, hv.pages, "step with extend blocks")


@pytest.mark.parametrize("d", [64, 128])
def test_fixed_length_rows_do_not_depend_on_the_batch(d):
    """At a fixed piece length an extend request, short or long, has the same
    bits alone, among other prefills and beside decode rows."""
    lens, rows = [300, 40, 260, 700, 50], [90, 40, 33, 300, 1]
    def batch(k):
        return W.make_batch(99, num_q_heads=32, num_kv_heads=8, head_dim=d, num_pages=512, prefix_len=[1500],
                            agent=[0] * 5, suffix_len=lens, n_rows=[n if i in k else 0 for i, n in enumerate(rows)])
    hv = W.host_values(batch(range(5)), 100)
    row0 = np.concatenate([[0], np.cumsum(rows)])
    ds, o, l = run_and_check(batch(range(5)), hv, f"fixed length, all, d={d}", piece_steps=16)
    for k in ([0], [1], [2], [3], [1, 4]):
        plan = B.plan_from_batch(ds.pool, batch(k), piece_steps=16).upload()
        q = torch.cat([ds.q[row0[i]:row0[i + 1]] for i in k])
        ok, lk = torch.empty_like(q), torch.empty(q.shape[:2], dtype=torch.float32, device="cuda")
        B.pfx_attention(ds.pool, plan, q, ok, lk)
        B.pfx_sync_check()
        n = rows[k[0]]
        assert np.array_equal(RN.to_host_bits(ok[:n]), o[row0[k[0]]:row0[k[0] + 1]])
        assert np.array_equal(lk[:n].cpu().numpy(), l[row0[k[0]]:row0[k[0] + 1]])


@pytest.mark.parametrize("case", [CASES[0], CASES[1], CASES[4]], ids=["alone", "mixed", "d64"])
def test_smaller_workspace_keeps_blocks_whole(case):
    """A workspace without room for the pieces is taken: the bits are those of
    whole blocks, through append + attention and through the step, nothing past
    its end is written, and the allocation-free call still cuts.  One byte less
    is refused."""
    hq, hkv, d, plen, reqs = case
    b = W.make_batch(101, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=plen,
                     agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
    hv = W.host_values(b, 102)
    _, o_cut, l_cut = run_and_check(b, hv, f"cut {plen} {reqs}")
    whole, o_ref, l_ref = run_and_check(b, hv, f"whole {plen} {reqs}", piece_steps=16)
    least = whole.plan.workspace_bytes()
    del whole
    announce(f"workspace of {least} bytes for the same batch")
    for step in (False, True):
        ds = RN.DeviceStep(b, hv)
        assert ds.plan.workspace_bytes() > least
        ws = torch.full((least + 512,), 0x5A, dtype=torch.uint8, device="cuda")
        ws = ws[-ws.data_ptr() % 256:]
        with pytest.raises(B.PfxError) as e:
            ds.plan.upload(workspace=ws[:least - 1])
        assert e.value.code == B.PFX_ENOMEM
        ds.plan.upload(workspace=ws[:least])
        if step:
            B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse)
        else:
            ds.step()
        B.pfx_sync_check()
        o, l = ds.outputs()
        assert np.array_equal(o, o_ref) and np.array_equal(l, l_ref)
        exp_k, exp_v = PT.expected_pools(b, hv)
        gk, gv = ds.read_pages(hv.pages)
        assert np.array_equal(gk, exp_k) and np.array_equal(gv, exp_v)
        assert bool((ws[least:] == 0x5A).all())
        B.pfx_attention_noalloc(ds.pool, ds.plan, ds.q, ds.o, ds.lse, k_new=ds.k_new, v_new=ds.v_new)
        B.pfx_sync_check()
        o, l = ds.outputs()
        assert np.array_equal(o, o_cut) and np.array_equal(l, l_cut)


MORE = [
    # (Hq, Hkv, d, prefixes, requests, rows checked against the oracle)
    (16, 8, 128, [1500], [(0, 140, 140), (0, 20, 1)], None),     # G = 2
    (16, 2, 128, [1500], [(0, 70, 70), (0, 33, 33)], None),      # G = 8
    (6, 3, 64, [2100], [(0, 150, 90), (0, 9, 1)], None),         # 3 KV heads: no head keeps to one XCD
    (32, 8, 128, [4500], [(0, 1200, 1200)], 40),                 # pieces in two rounds
    (32, 2, 64, [16], [(0, 1100, 1100)], 60),                    # 276 whole blocks, the second 256 reversed
    (48, 3, 64, [16], [(0, 700, 700)], 60),                      # 264 whole blocks, not reversed
]


@pytest.mark.parametrize("case", MORE, ids=["g2", "g8", "kv3", "two-rounds", "reversed", "kv3-whole"])
def test_more_block_shapes(case):
    """Query groups, KV head counts and launch sizes past those of the cases
    above: against the oracle (on sampled rows where the batch is large), all
    rows against whole blocks within twice the rounding of P and O, and the
    step bit for bit against append + attention."""
    hq, hkv, d, plen, reqs, sample = case
    b = W.make_batch(110, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=plen,
                     agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
    hv = W.host_values_fast(b, 111)
    rows = None
    if sample:
        n = reqs[0][2]
        rows = {0: sorted({0, 1, 15, 16, 31, 32, n - 1} | set(np.random.default_rng(1).integers(0, n, sample).tolist()))}
    ds, o, l = run_and_check(b, hv, f"blocks Hq={hq} Hkv={hkv} d={d} {plen} {reqs}", rows=rows)
    states = ds.plan.workspace_bytes() // (512 * d + 1024)
    assert states > 512 if plen[0] == 4500 else states < 8 if plen[0] == 16 else 8 < states < 512
    whole = B.plan_from_batch(ds.pool, b, piece_steps=16).upload()
    o1, l1 = torch.empty_like(ds.o), torch.empty_like(ds.lse)
    B.pfx_attention(ds.pool, whole, ds.q, o1, l1)
    B.pfx_sync_check()
    # Cut and whole blocks round P (2^-9 of each term) against other maxima, and O: the outputs differ by less than
    # both roundings of both sides, 4 * 2^-9 of their 2-norm.
    x, y = ds.o.double(), o1.double()
    assert float((x - y).norm() / y.norm()) < 2 ** -7 and float((ds.lse - l1).abs().max()) < 1e-2
    del ds
    ds = RN.DeviceStep(b, hv)
    B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse)
    B.pfx_sync_check()
    os, ls = ds.outputs()
    assert np.array_equal(o, os) and np.array_equal(l, ls)
    exp_k, exp_v = PT.expected_pools(b, hv)
    gk, gv = ds.read_pages(hv.pages)
    assert np.array_equal(gk, exp_k) and np.array_equal(gv, exp_v)
    assert_untouched(ds, hv.pages, "block shapes")


@pytest.mark.parametrize("case", [CASES[1], STEPS[0]], ids=["cut", "mixed"])
def test_captured_step(case):
    """pfx_step over cut blocks and decode rows captured into a graph and
    replayed, other work and a fresh pool between the replays: each replay
    equals the eager step bit for bit."""
    hq, hkv, d, plen, reqs = case
    b = W.make_batch(120, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=512, prefix_len=plen,
                     agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
    hv = W.host_values(b, 121)
    ds = RN.DeviceStep(b, hv)
    first = ds.k_pool.clone(), ds.v_pool.clone()
    announce(f"captured step over {plen} {reqs}")
    B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse)
    B.pfx_sync_check()
    want = [t.clone() for t in (ds.o, ds.lse, ds.k_pool, ds.v_pool)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.pfx_step(ds.pool, ds.plan, ds.k_new, ds.v_new, ds.q, ds.o, ds.lse,
                   stream=torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        for t, f in ((ds.k_pool, first[0]), (ds.v_pool, first[1])):
            t.copy_(f)
        ds.o.zero_()
        ds.lse.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for t, w in zip((ds.o, ds.lse, ds.k_pool, ds.v_pool), want):
            assert torch.equal(t.view(torch.int16) if t.dtype == torch.bfloat16 else t,
                               w.view(torch.int16) if w.dtype == torch.bfloat16 else w)
