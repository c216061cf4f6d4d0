"""The default decode piece length (host only): 16 steps, 32 from 12288 steps
on, or the shortest from 3 on with which every workgroup of the launch is
resident at once, where that is shorter; and the piece records."""

import ctypes as C

import numpy as np
import pytest

pytest.importorskip("torch")

from paper_2608_25523_amd import binding as B  # noqa: E402
from paper_2608_25523_amd import workloads as W  # noqa: E402


def plan(b, **kw):
    return B.plan_from_batch(B.make_pool(b.num_pages, b.num_kv_heads, b.head_dim), b, B.PFX_MODE_MIXED, **kw)


def batch(d, reqs, plen, extend=0):
    a = np.arange(reqs + (extend > 0)) % len(plen)
    n = [1] * reqs + ([extend] if extend else [])
    s = [33 + 37 * i % 500 for i in range(reqs)] + ([extend] if extend else [])
    return W.make_batch(7, num_q_heads=32, num_kv_heads=8, head_dim=d, num_pages=65536, prefix_len=plen, agent=a,
                        suffix_len=s, n_rows=n)


@pytest.mark.parametrize("d,reqs,plen,extend", [
    (128, 1, [2048], 0), (128, 4, [2048], 0), (128, 16, [700, 3000, 1500], 0), (128, 32, [500, 3000], 0),
    (64, 32, [500, 3000], 0), (128, 64, [2048] * 4, 0), (128, 4, [2048], 600), (128, 4, [2048], 3000),
    (128, 1, [], 0)])
def test_shortest_length_that_is_resident(d, reqs, plen, extend):
    if not plen:
        b = W.make_batch(7, num_q_heads=32, num_kv_heads=8, head_dim=d, num_pages=64, prefix_len=[], agent=[-1],
                         suffix_len=[20], n_rows=[1])
    else:
        b = batch(d, reqs, plen, extend)
    s = plan(b).stats()
    assert s.num_decode_steps < 12288
    room = 0 if extend else 512 if d == 128 else 1024   # beside extend blocks the pieces stay long
    count = {l: plan(b, piece_steps=l).stats() for l in range(3, 17)}
    fits = [l for l in count if count[l].num_decode_pieces + count[l].num_wide_blocks <= room]
    want = count[min(fits) if fits else 16]
    assert (s.num_decode_pieces, s.num_wide_blocks) == (want.num_decode_pieces, want.num_wide_blocks)


def test_length_of_few_long_items():
    """One long request past 12288 steps: as many pieces as are resident, more
    than 32-step pieces would be."""
    b = W.make_batch(7, num_q_heads=32, num_kv_heads=8, head_dim=128, num_pages=4096, prefix_len=[49000], agent=[0],
                     suffix_len=[280], n_rows=[1])
    s = plan(b).stats()
    assert 12288 <= s.num_decode_steps < 16384
    assert plan(b, piece_steps=32).stats().num_decode_pieces < s.num_decode_pieces <= 512
    assert plan(b, piece_steps=24).stats().num_decode_pieces > 512


def test_length_of_larger_launches():
    b = batch(128, 160, [500, 4000, 2000, 1000])
    s = plan(b).stats()
    assert 12288 <= s.num_decode_steps < 32768
    assert s.num_decode_pieces == plan(b, piece_steps=32).stats().num_decode_pieces


@pytest.mark.parametrize("d,hq,hkv", [(128, 32, 8), (64, 8, 2), (128, 16, 16)])
@pytest.mark.parametrize("keys,parts", [(97, 1), (160, 1), (288, 1), (512, 1), (513, 0)])
def test_lone_short_items_stay_whole(d, hq, hkv, keys, parts):
    """A request whose only item fits one piece of 16 steps has one state, as
    with 16-step pieces, whatever else is in the launch; a longer one is cut."""
    def parts_of(reqs, plen, **kw):
        b = W.make_batch(8, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=1024, prefix_len=plen,
                         agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[1] * len(reqs))
        return plan(b, **kw).export(7)[:, 1].reshape(len(reqs), hkv)
    for reqs, plen in (([(-1, keys)], []), ([(-1, 20), (-1, keys), (-1, 40)], []), ([(0, keys)], [0]),
                       ([(0, 200), (-1, keys), (0, 300)], [2048])):
        got = parts_of(reqs, plen)
        lone = [i for i, r in enumerate(reqs) if r[1] == keys]
        assert np.array_equal(got[lone], parts_of(reqs, plen, piece_steps=16)[lone]) if parts else (got[lone] > 1).all()


@pytest.mark.parametrize("reqs,plen,most", [(1, [2048], 32), (4, [2048], 64), (16, [700, 3000, 1500], 128)])
def test_short_pieces_have_short_records(reqs, plen, most):
    """What a plan writes and an upload copies does not grow with the pieces of
    a small launch: no more than 16-step pieces in records of 1088 bytes."""
    b = batch(128, reqs, plen)
    s, long = plan(b).stats(), plan(b, piece_steps=16).stats()
    assert s.num_decode_pieces > long.num_decode_pieces
    tables = s.workspace_bytes - 264 * s.num_partial_rows
    assert tables < most << 10 and tables < 1088 * long.num_decode_pieces


@pytest.mark.parametrize("reqs,plen,engine,room", [
    (24, [8192], B.PFX_DECODE_MFMA, 768), (64, [2048], B.PFX_DECODE_MFMA, 768),
    (16, [8192], B.PFX_DECODE_MFMA, 1024), (16, [8192], B.PFX_DECODE_VALU, 768)])
def test_resident_workgroups_of_the_kernel_that_runs(reqs, plen, engine, room):
    """d = 64: three workgroups of the kernel with wide blocks, or of the
    vector-ALU engine, fit a compute unit, four of the other."""
    b = batch(64, reqs, plen)
    s = plan(b, decode_engine=engine).stats()
    assert (s.num_wide_blocks > 0) == (reqs > 16)
    count = {l: plan(b, piece_steps=l, decode_engine=engine).stats() for l in range(3, 17)}
    fits = [l for l in count if count[l].num_decode_pieces + count[l].num_wide_blocks <= room]
    want = count[min(fits)]
    assert (s.num_decode_pieces, s.num_wide_blocks) == (want.num_decode_pieces, want.num_wide_blocks)
    assert min(fits) > 3


def test_export_of_part_of_the_records():
    """pfx_plan_export writes min(cap, size) values of the piece records, also
    when the cut falls inside one."""
    p = plan(batch(128, 4, [2048]))
    full = p.export(3).reshape(-1)
    for cap in (0, 1, 271, 272, 273, len(full) - 1, len(full) + 5):
        out, n = np.full(len(full) + 8, -7, np.int32), C.c_int64()
        assert B.LIB.pfx_plan_export(p.h, 3, out.ctypes.data_as(C.c_void_p), cap, C.byref(n)) == 0
        m = min(cap, len(full))
        assert n.value == len(full) and np.array_equal(out[:m], full[:m]) and (out[m:] == -7).all()
