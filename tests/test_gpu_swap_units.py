"""The block copy's units: a block is moved in passes of 64, 32, 16 or 8 KiB, whichever divides it, by as many workgroups
as put 512 KiB in flight.  Block sizes of every kind, lists of one block, of as many as there are workgroups and one more,
and a single workgroup that takes every unit in turn; bytes of both pools against the copy oracle."""
import numpy as np
import pytest
import torch

from oracle import blockcopy as C
from paper_2512_12928_amd import binding as B
from paper_2512_12928_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hkv", [1, 2, 3, 4, 5, 8, 12])          # 8, 16, 24, 32, 40, 64, 96 KiB
@pytest.mark.parametrize("n,wgs", [(1, 0), (8, 0), (9, 0), (65, 0), (7, 1)])
def test_blocks_of_every_size(Hkv, n, wgs):
    bb, M, Mh = W.LayerShape(Hkv, Hkv).block_bytes, 160, 150
    rng = np.random.default_rng(Hkv * 100 + n)
    dev_np, host_np = rng.integers(0, 256, (M, bb), dtype=np.uint8), rng.integers(0, 256, (Mh, bb), dtype=np.uint8)
    dev, host = torch.from_numpy(dev_np).to("cuda:0"), torch.from_numpy(host_np.copy()).pin_memory()
    ctx = B.ps_create(Hkv, Hkv, M, Mh, swap_workgroups=wgs)
    d, h = rng.permutation(M).astype(np.int32), rng.permutation(Mh).astype(np.int32)
    out, side = torch.cuda.Stream(), torch.cuda.Stream()
    n1, t1 = B.ps_swap_out(ctx, d[:n], h[:n], -1, dev, host, out)                       # both directions at once
    n2, t2 = B.ps_swap_in(ctx, h[n:2 * n], d[n:2 * n], -1, host, dev, side)
    assert n1 == n2 == n
    B.ps_ticket_wait(ctx, t1)
    B.ps_ticket_wait(ctx, t2)
    want_dev, want_host = dev_np.copy(), host_np.copy()
    C.swap_out(dev_np, want_host, d[:n], h[:n], -1)
    C.swap_in(host_np, want_dev, h[n:2 * n], d[n:2 * n], -1)
    assert np.array_equal(host.numpy(), want_host) and np.array_equal(dev.cpu().numpy(), want_dev)
    B.ps_destroy(ctx)
