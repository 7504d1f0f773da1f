"""float32 expert products: tile and K remainders, empty and short experts, and
both tile sizes, against float64 products of the kernel's own inputs, and bit for
bit against chains of fused multiply-adds."""
from __future__ import annotations

import numpy as np
import pytest

from synth import LayerSpec, layer_inputs
from tests.gpu_harness import ebuf, host, run_layer, spec_C
from tests.tile_choice import PRODUCTS, expert_tile

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_2404_19429_amd import lancet_moe
    return lancet_moe


# d and f multiples of 8 that end inside a 16-K block, a stage and a tile; k = E
# fixes 130 and 33 rows per expert (one past a tile, one past a wave's rows);
# 2600 tokens over two wide experts take the larger tile.
@pytest.mark.parametrize("T,d,f,E,k", [(130, 72, 104, 4, 4), (33, 8, 40, 2, 2), (37, 64, 200, 16, 1),
                                       (2600, 136, 1032, 2, 2)],
                         ids=["rows_130", "rows_33_d8", "few_rows_empty_experts", "large_tile"])
def test_products_match_float64(L, T, d, f, E, k):
    """Each output is a float sum of K products in order: within (K + 2) u sum|a||b|
    of the exact value, u = 2^-24 (act and act' add at most a few u of a term)."""
    spec = LayerSpec(name="f32", T=T, d=d, f=f, E=E, k=k, cf_num=5, cf_den=4, dtype="f32", act="identity",
                     renorm=1 if k > 1 else 0, seed=91)
    inp = layer_inputs(spec)
    b, _ = run_layer(L, spec, inp, spec_C(spec))
    fill = host(b.fill)
    buf = {n: ebuf(b, n).astype(np.float64) for n in ("send_buf", "H", "A", "O", "dO", "dH", "dXe")}
    u = 2.0 ** -24
    for e in range(E):
        n = int(fill[e])
        W1, W2 = inp["W1"][e].astype(np.float64), inp["W2"][e].astype(np.float64)
        r = {q: v[e, :n] for q, v in buf.items()}
        for name, got, a, c in (("H", r["H"], r["send_buf"], W1.T), ("O", r["O"], r["A"], W2.T),
                                ("dH", r["dH"], r["dO"], W2), ("dXe", r["dXe"], r["dH"], W1),
                                ("dW2", host(b.dW2)[e], r["dO"].T, r["A"]),
                                ("dW1", host(b.dW1)[e], r["dH"].T, r["send_buf"])):
            bound = (a.shape[1] + 2) * u * (np.abs(a) @ np.abs(c))
            assert np.all(np.abs(got - a @ c) <= bound), f"{name} of expert {e} ({n} rows)"


def _fma(acc, a, b):
    """acc + a b of float32 arrays, rounded once.  The product is exact in double; the
    sum is rounded to odd there (its error, by a two-sum, makes an inexact even result
    step to its odd neighbour), after which rounding to float32 is the rounding of the
    exact value."""
    p = a.astype(np.float64) * b
    c = acc.astype(np.float64)
    s = c + p
    t = s - c
    e = (c - (s - t)) + (p - t)
    even = (s.view(np.int64) & 1) == 0
    s = np.where((e != 0) & even, np.nextafter(s, np.where(e > 0, np.inf, -np.inf)), s)
    return s.astype(np.float32)


def _in_order(A, B):
    """A B of float32 matrices, every element one chain of fused multiply-adds in K order."""
    acc = np.zeros((A.shape[0], B.shape[1]), np.float32)
    for k in range(A.shape[1]):
        acc = _fma(acc, A[:, k:k + 1], B[k:k + 1])
    return acc


# tiles of H and dH, of expert_out and dXe, of dW2 and dW1 (256 compute units): each
# kind of product is on both sizes.  tiny: x and W1 so small that H and the products
# and sums in it are subnormal.
@pytest.mark.parametrize("T,d,f,E,k,tiles,tiny", [(512, 40, 1792, 1, 1, (64, 32, 32), False),
                                                  (512, 1792, 40, 1, 1, (32, 64, 32), False),
                                                  (64, 448, 448, 4, 4, (32, 32, 64), False),
                                                  (37, 72, 104, 2, 2, (32, 32, 32), True),
                                                  (512, 24, 1792, 1, 1, (64, 32, 32), True)])
def test_products_are_the_bits_of_a_loop_of_fused_multiply_adds(L, T, d, f, E, k, tiles, tiny):
    spec = LayerSpec(name="f32", T=T, d=d, f=f, E=E, k=k, cf_num=1, cf_den=1, dtype="f32", act="identity",
                     renorm=1 if k > 1 else 0, seed=92)
    inp = layer_inputs(spec)
    if tiny:
        for n in ("x", "W1"):
            inp[n] = (inp[n] * np.float32(2.0 ** -66)).astype(np.float32)
    b, _ = run_layer(L, spec, inp, spec_C(spec))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for p, want in zip(PRODUCTS, (tiles[0], tiles[1], tiles[0], tiles[1], tiles[2], tiles[2])):
        assert expert_tile(b.cfg, p, cus=cus)[0] == want, p
    fill = host(b.fill)
    buf = {n: ebuf(b, n) for n in ("send_buf", "H", "A", "O", "dO", "dH", "dXe")}
    if tiny:
        small = np.abs(buf["H"][0, :int(fill[0])])
        assert (small > 0).mean() > 0.5 and small.max() < 2.0 ** -126, (small.max(), (small > 0).mean())
    for e in range(E):
        n = int(fill[e])
        r = {q: v[e, :n] for q, v in buf.items()}
        W1, W2 = inp["W1"][e].astype(np.float32), inp["W2"][e].astype(np.float32)
        for name, got, a, c in (("H", r["H"], r["send_buf"], W1.T), ("O", r["O"], r["A"], W2.T),
                                ("dH", r["dH"], r["dO"], W2), ("dXe", r["dXe"], r["dH"], W1),
                                ("dW2", host(b.dW2)[e], r["dO"].T, r["A"]),
                                ("dW1", host(b.dW1)[e], r["dH"].T, r["send_buf"])):
            np.testing.assert_array_equal(got, _in_order(a, c), err_msg=f"{name} of expert {e}")
