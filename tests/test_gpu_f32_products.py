"""float32 expert products: tile and K remainders, empty and short experts, and
both tile sizes, against float64 products of the kernel's own inputs."""
from __future__ import annotations

import numpy as np
import pytest

from synth import LayerSpec, layer_inputs
from tests.gpu_harness import ebuf, host, run_layer, spec_C

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
