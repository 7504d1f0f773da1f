"""The choice of a product's tile follows the device's compute units (host only)."""
import pytest

L = pytest.importorskip("paper_2404_19429_amd.lancet_moe", reason="library not built")
from tests.tile_choice import PRODUCTS, dense_tile, expert_tile  # noqa: E402

SIZES = [(1531, 768, 3072, 8, 1), (48, 1024, 4096, 16, 2), (2048, 768, 3072, 8, 2), (3108, 768, 3072, 8, 2),
         (4096, 1024, 4096, 16, 2), (4096, 2048, 8192, 16, 2), (6000, 1536, 6144, 32, 2), (16384, 2048, 8192, 8, 2),
         (20000, 512, 2048, 8, 1)]


@pytest.mark.parametrize("dtype,ksplit", [("bf16", 0), ("bf16", 1), ("f32", 0)])
@pytest.mark.parametrize("T,d,f,E,k", SIZES)
def test_half_the_experts_on_half_the_device_take_the_same_tiles(T, d, f, E, k, dtype, ksplit):
    """With the rows per expert and the widths the same, a device with half the
    compute units runs half the tiles in the same rounds."""
    whole = L.make_cfg(T, d, f, E, k, T, dtype=dtype, ksplit=ksplit)
    half = L.make_cfg(T // 2, d, f, E // 2, k, T, dtype=dtype, ksplit=ksplit)
    for p in PRODUCTS:
        assert expert_tile(whole, p, cus=256) == expert_tile(half, p, cus=128), p


def test_dense_products_take_smaller_tiles_on_a_larger_device():
    tiles = [dense_tile(2048, 2048, 2048, cus) for cus in (32, 64, 256)]
    assert tiles == [(256, 256), (256, 256), (128, 128)]
