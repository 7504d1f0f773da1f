"""Gate on each of its launch shapes: list lengths (k rounded up to 1, 2, 4, 8),
expert tiles (16, 32, 48, 64) and 16- or 32-token blocks, with tied logits and
fewer experts than the four lanes of a token."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import moe_oracle as O
from tests.gpu_harness import host, log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2404_19429_amd import lancet_moe
    return lancet_moe


# More than 12288 tokens take 32-token blocks on 256 CUs; 16391 and 37 end inside a block.
@pytest.mark.parametrize("T", [1, 37, 16391])
@pytest.mark.parametrize("E,k,renorm,dtype", [(1, 1, 0, "f32"), (3, 1, 0, "bf16"), (3, 3, 1, "f32"), (16, 2, 1, "bf16"),
                                              (17, 4, 0, "bf16"), (33, 5, 1, "bf16"), (48, 3, 0, "f32"),
                                              (64, 8, 1, "bf16"), (9, 7, 1, "bf16"), (8, 8, 0, "f32")])
def test_gate_launch_shapes(L, T, E, k, renorm, dtype):
    """Logits within an ulp of the float64 ones; the choices are those of the
    kernel's own logits.  A weight is a quotient of float sums of at most E
    exponentials, each off by a few u plus u |l - max| from its rounded argument
    (u = 2^-24)."""
    log(f"[gate] T={T} E={E} k={k} renorm={renorm} {dtype}")
    d = 72
    g = np.random.default_rng(E * 100 + k)
    x = g.integers(-2, 3, (T, d)).astype(np.float32)           # small integers: exact products, many ties
    Wg = (g.integers(-2, 3, (E, d)) / 16).astype(np.float32)
    bias = (g.integers(-4, 5, E) / 16).astype(np.float32) if k > 1 else None
    cfg = L.make_cfg(T, d, 64, E, k, max(1, T), dtype=dtype, renorm=renorm)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dev = [torch.from_numpy(v).cuda().to(dt) for v in (x, Wg)]
    lg = torch.empty(T, E, device="cuda")
    idx = torch.empty(T, k, dtype=torch.int32, device="cuda")
    w = torch.empty(T, k, device="cuda")
    L.moe_gate_topk(cfg, *dev, None if bias is None else torch.from_numpy(bias).cuda(), lg, idx, w)
    got = host(lg)
    np.testing.assert_array_max_ulp(got, O.gate_logits(x, Wg, bias), maxulp=1)
    want = O.topk_route(got, k)
    np.testing.assert_array_equal(host(idx), want)
    ref = O.gate_weights(got, want, renorm)[1]
    span = float((got.max(axis=1) - got.min(axis=1)).max())
    assert np.all(np.abs(host(w) - ref) <= (E + 2 * span + 16) * 2.0 ** -24 * ref)
