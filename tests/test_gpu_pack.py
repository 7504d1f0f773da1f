"""moe_pack_weights at its edges: the float copy of a few elements and of a last
part-filled block, the bf16 blocks of matrices whose strips of 16 rows end with a
launch block's eight and inside them."""
from __future__ import annotations

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2404_19429_amd import lancet_moe
    return lancet_moe


def _packed(W, dtype):
    """[E][R][X] in the layout the expert products read: 16 x 32 blocks for bf16, plain for float."""
    E, R, X = W.shape
    return W if dtype == "f32" else W.view(E, R // 16, 16, X // 32, 32).transpose(2, 3).contiguous().view(E, R, X)


SHAPES = [("f32", 1, 8, 8), ("f32", 5, 72, 104), ("f32", 3, 512, 1024), ("bf16", 1, 64, 64), ("bf16", 3, 192, 320), ("bf16", 1, 192, 64),
          ("bf16", 2, 1024, 128), ("bf16", 3, 256, 768), ("bf16", 1, 4032, 4160), ("bf16", 1, 8128, 256)]


def _weights(L, dtype, E, d, f):
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cfg = L.make_cfg(1, d, f, E, 1, 1, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(E * d + f)
    W1, W2 = (torch.randn(E, *s, device="cuda", generator=g).to(dt) for s in ((f, d), (d, f)))
    return cfg, W1, W2


@pytest.mark.parametrize("dtype,E,d,f", SHAPES)
def test_pack_weights_layout(L, dtype, E, d, f):
    cfg, W1, W2 = _weights(L, dtype, E, d, f)
    # one buffer with a guard past each copy: nothing is written outside it
    n = W1.numel()
    buf = torch.full((2, n + 64), float("nan"), device="cuda", dtype=W1.dtype)
    L.moe_pack_weights(cfg, W1, W2, buf[0, :n], buf[1, :n])
    torch.cuda.synchronize()
    assert torch.equal(buf[0, :n].view(E, f, d), _packed(W1, dtype))
    assert torch.equal(buf[1, :n].view(E, d, f), _packed(W2, dtype))
    assert bool(buf[:, n:].isnan().all())


@pytest.mark.parametrize("dtype,E,d,f", SHAPES)
def test_copy_of_w2_may_take_the_memory_of_w1(L, dtype, E, d, f):
    cfg, W1, W2 = _weights(L, dtype, E, d, f)
    want1, want2 = _packed(W1, dtype).clone(), _packed(W2, dtype).clone()
    W1p = torch.empty_like(W1)
    L.moe_pack_weights(cfg, W1, W2, W1p, W1)
    torch.cuda.synchronize()
    assert torch.equal(W1p, want1)
    assert torch.equal(W1.view(E, d, f), want2)
