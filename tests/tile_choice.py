"""Which tile shape the library gives a bf16 product: the choice of its launches,
asked of the library itself (it is not part of the C ABI, so by its C++ name)."""
import ctypes

from paper_2404_19429_amd import lancet_moe as L

PRODUCTS = L.PRODUCTS   # fwd1, fwd2, dA, dXe, dW2, dW1

_expert = L._lib["_ZN4lmoe11expert_tileERK7moe_cfgibi"]
_expert.restype, _expert.argtypes = ctypes.c_int, [ctypes.POINTER(L.moe_cfg), ctypes.c_int, ctypes.c_bool, ctypes.c_int]
_dense = L._lib["_ZN4lmoe10dense_tileEliii"]
_dense.restype, _dense.argtypes = ctypes.c_int, [ctypes.c_int64] + [ctypes.c_int] * 3


def _shape(v):
    return v >> 16, v & 0xffff


def expert_tile(cfg, product, later=False, cus=256):
    """(rows, columns) of the tile of one of PRODUCTS, (0, 0) where the device picks 128
    or 256 wide by the row counts; later: a batch partition after the first."""
    return _shape(_expert(ctypes.byref(cfg), PRODUCTS.index(product), later, cus))


def dense_tile(M, N, K, cus=256):
    return _shape(_dense(M, N, K, cus))
