"""Extend blocks cut along their keys: which launches are cut, and that the
pieces cover every block once (host only, through the plan builder built with
g++ and tests/native/chunk_check.cpp)."""

from __future__ import annotations

import os
import shutil
import subprocess

import pytest

pytest.importorskip("torch")

from paper_2608_25523_amd import binding as B  # noqa: E402
from paper_2608_25523_amd import workloads as W  # noqa: E402

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def case_text(b):
    """A batch in the driver's format."""
    pind, pids, plen = b.prefix_csr()
    sind, sids = b.suffix_csr()
    rows = [[b.num_pages, b.num_kv_heads, b.head_dim, b.num_q_heads, 3, 0, 0], [len(plen)], plen, pind, pids,
            [len(b.agent)], b.agent, sind, sids, b.suffix_len, b.q_indptr()]
    return "\n".join(" ".join(str(int(x)) for x in r) for r in rows) + "\n"


# (Hq, Hkv, d, prefixes, requests (agent, L, n), cut?)
CASES = [
    (32, 8, 128, [4096], [(0, 300, 300)], True),
    (32, 8, 128, [4093], [(0, 32, 32)], True),               # the prefix ends inside a step, on a lone page
    (32, 8, 128, [], [(-1, 5000, 40)], True),                # no prefix
    (32, 8, 128, [17, 3000], [(0, 40, 40), (1, 40, 40), (-1, 9, 9)], True),   # long and short blocks together
    (16, 16, 128, [2049], [(0, 201, 201), (0, 30, 1)], True),
    (32, 2, 64, [2048], [(0, 513, 100), (0, 20, 20)], True),
    (32, 8, 128, [8000], [(0, 1200, 1200)], True),           # two rounds of pieces
    (32, 8, 128, [1000], [(0, 100, 100)] * 8, False),        # short blocks: a second launch costs more
    (32, 8, 128, [2048], [(0, 1999, 1999)], False),          # the chip is full already
    (8, 2, 64, [128], [(0, 32, 32)] * 4, False),
]


SOURCE = os.path.join(ROOT, "tests", "native", "chunk_check.cpp")


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(SOURCE), reason="needs g++ and the checker's source")
def test_pieces_cover_every_block(tmp_path):
    exe = tmp_path / "chunk_check"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"),
                    SOURCE,
                    os.path.join(ROOT, "paper_2608_25523_amd", "csrc", "pfx_plan.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    text = ""
    for hq, hkv, d, plen, reqs, _ in CASES:
        b = W.make_batch(31, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=2048, prefix_len=plen,
                         agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
        text += case_text(b)
    inp = tmp_path / "cases.txt"
    inp.write_text(text)
    res = subprocess.run([str(exe), str(inp)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
    lines = res.stdout.splitlines()
    assert len(lines) == len(CASES)
    for line, case in zip(lines, CASES):
        assert (not line.startswith("cut 0 ")) == case[-1], (case, line)
        if case[-1]:
            assert int(line.split(", ")[1].split()[0]) <= 1024


@pytest.mark.parametrize("case", [c for c in CASES if c[-1]], ids=lambda c: f"{c[0]}-{c[3]}-{c[4][0][2]}")
def test_fixed_length_keeps_blocks_whole(case):
    """With a piece length given, a plan holds no states of cut blocks."""
    hq, hkv, d, plen, reqs, _ = case
    b = W.make_batch(32, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_pages=2048, prefix_len=plen,
                     agent=[r[0] for r in reqs], suffix_len=[r[1] for r in reqs], n_rows=[r[2] for r in reqs])
    pool = B.make_pool(b.num_pages, hkv, d)
    states = 8 * 128 * 4 * d  # of one block in two, at the least
    assert B.plan_from_batch(pool, b).workspace_bytes() > states
    for steps in (16, 64):
        s = B.plan_from_batch(pool, b, piece_steps=steps).stats()
        assert s.workspace_bytes - s.num_partial_rows * (2 * d + 8) < 64 << 10


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc not available")
def test_no_scratch_in_the_piece_kernels(tmp_path):
    from paper_2608_25523_amd.build import FLAGS
    out = tmp_path / "k.s"
    subprocess.run(["/opt/rocm/bin/hipcc", *[f for f in FLAGS if f not in ("-shared", "-fPIC")], "-S",
                    "--cuda-device-only", "-I", os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "paper_2608_25523_amd", "csrc", "pfx_kernels.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    blocks = [b.split(".end_amdhsa_kernel")[0] for b in out.read_text().split(".amdhsa_kernel ")[1:]]
    mine = [b for b in blocks if any(n in b.split()[0] for n in ("chunk_kernel", "chunk_merge", "merge_parts"))]
    assert len(mine) == 14
    for b in mine:
        assert ".amdhsa_private_segment_fixed_size 0" in b, b.split()[0]
