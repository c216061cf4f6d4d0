"""pfx_page_copy on the GPU, bit for bit against the page-copy oracle: the
longest list that travels in the launch and the first that does not, pages that
are not whole workgroups, every direction between device and pinned host
memory, and a launch captured into a graph and replayed after its lists are
gone."""

from __future__ import annotations

import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
from paper_2608_25523_amd import binding as B  # noqa: E402

pytestmark = pytest.mark.gpu


def pool(pages, hkv, d, where, gen):
    t = torch.randint(-30000, 30000, (2, pages, hkv, 16, d), dtype=torch.int16, generator=gen)
    t = t.pin_memory() if where == "host" else t.cuda()
    return t, B.make_pool(pages, hkv, d, t[0], t[1])


def bits(t):
    return t.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("src_at,dst_at", [("host", "gpu"), ("gpu", "host"), ("gpu", "gpu"), ("host", "host")])
@pytest.mark.parametrize("n,hkv,d", [(1, 8, 128), (448, 1, 64), (449, 3, 64), (70, 3, 64), (33, 5, 128)])
def test_page_copy(n, hkv, d, src_at, dst_at):
    print(f"\n[gpu-case] page copy n={n} hkv={hkv} d={d} {src_at} -> {dst_at}", flush=True)
    gen = torch.Generator().manual_seed(n + hkv)
    rng = np.random.default_rng(n)
    src, sp = pool(n + 3, hkv, d, src_at, gen)
    dst, dp = pool(n + 9, hkv, d, dst_at, gen)
    d_ids = rng.permutation(n + 9)[:n].astype(np.int32)
    s_ids = rng.integers(0, n + 3, size=n).astype(np.int32)
    want = [oracle.page_copy(bits(dst[i]).copy(), bits(src[i]), d_ids, s_ids) for i in range(2)]
    ws = torch.empty(B.pfx_page_copy_workspace_bytes(n) + 256, dtype=torch.uint8, device="cuda")
    B.pfx_page_copy(dp, sp, d_ids, s_ids, ws)
    B.pfx_sync_check()
    assert all(np.array_equal(bits(dst[i]), want[i]) for i in range(2))


def test_captured_page_copy():
    gen = torch.Generator().manual_seed(3)
    src, sp = pool(40, 8, 64, "gpu", gen)
    dst, dp = pool(40, 8, 64, "gpu", gen)
    first = dst.clone()
    d_ids, s_ids = np.arange(40, dtype=np.int32)[::-1].copy(), np.arange(40, dtype=np.int32)
    want = [oracle.page_copy(bits(first[i]).copy(), bits(src[i]), d_ids, s_ids) for i in range(2)]
    ws = torch.empty(B.pfx_page_copy_workspace_bytes(40) + 256, dtype=torch.uint8, device="cuda")
    print("\n[gpu-case] captured page copy, 3 replays", flush=True)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.pfx_page_copy(dp, sp, d_ids, s_ids, ws, stream=torch.cuda.current_stream().cuda_stream)
    d_ids[:] = 0
    for _ in range(3):
        dst.copy_(first)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(np.array_equal(bits(dst[i]), want[i]) for i in range(2))
