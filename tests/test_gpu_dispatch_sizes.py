"""Slot assignment and copy on each of their launch shapes: one chunk of tokens
(a single launch), a few chunks without wave-uniform rows (no scan launch) and
more, in token order with a carry and in batch-prioritized order."""
from __future__ import annotations

import numpy as np
import pytest

from tests.gpu_harness import expert_host, host

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2404_19429_amd import lancet_moe
    return lancet_moe


def _walk(idx, order, carry, C, E):
    """Rows taken one assignment after another over the walk."""
    used = carry.copy()
    slot = np.full(idx.shape, -1, np.int32)
    for t in order:
        for r, e in enumerate(idx[t]):
            if used[e] < C:
                slot[t, r] = used[e]
                used[e] += 1
    return slot, used


# 1 / 255 / 256: one chunk, of d 4096 and 2056 with k = 8 wide enough for the
# general launches; 257 / 2048 with d 72 or 96 (rows are not whole waves): bases
# summed in the copy up to k = 3; k = 4, 2049: the scan launch; d 512: wave-uniform rows.
@pytest.mark.parametrize("T,d,E,k,dtype", [(1, 64, 4, 1, "bf16"), (255, 96, 5, 3, "f32"), (256, 512, 64, 2, "bf16"),
                                           (257, 72, 8, 2, "f32"), (2048, 96, 16, 2, "bf16"), (2049, 96, 3, 2, "bf16"),
                                           (2048, 96, 16, 3, "bf16"), (2048, 72, 16, 4, "f32"),
                                           (700, 512, 8, 2, "bf16"), (256, 4096, 64, 8, "bf16"),
                                           (255, 2056, 32, 8, "f32")])
def test_dispatch_launch_shapes(L, T, d, E, k, dtype):
    g = np.random.default_rng(T)
    C = max(1, T * k // (2 * E) + 3)     # below the demand of a skewed choice: some are dropped
    cfg = L.make_cfg(T, d, 64, E, k, C, dtype=dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.from_numpy(g.standard_normal((T, d)).astype(np.float32)).cuda().to(dt)
    logits = g.standard_normal((T, E)).astype(np.float32) + np.linspace(0, 2, E, dtype=np.float32)
    idx = np.argsort(-logits, axis=1, kind="stable")[:, :k].astype(np.int32)
    carry = g.integers(0, C, E).astype(np.int32)
    b = L.alloc_layer(cfg)
    di = torch.from_numpy(idx).cuda()
    L.moe_dispatch(cfg, x, di, torch.from_numpy(carry).cuda(), b.fill, b.slot, b.send_buf, b.ws_dispatch)
    _check(L, cfg, b, x, idx, *_walk(idx, range(T), carry, C, E))
    L.moe_dispatch_bpr(cfg, x, torch.from_numpy(logits).cuda(), di, b.fill, b.slot, b.send_buf, b.order, b.ws_bpr)
    order = host(b.order)[:T]
    np.testing.assert_array_equal(np.sort(order), np.arange(T))
    _check(L, cfg, b, x, idx, *_walk(idx, order, np.zeros(E, np.int32), C, E))


def _check(L, cfg, b, x, idx, slot, used):
    np.testing.assert_array_equal(host(b.slot), slot)
    np.testing.assert_array_equal(host(b.fill), np.minimum(used, cfg.C))
    send = expert_host(b.send_buf, cfg, cfg.d_model)
    t, r = np.nonzero(slot >= 0)
    np.testing.assert_array_equal(send[idx[t, r], slot[t, r]], host(x)[t])
