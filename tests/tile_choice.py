"""Which tile shape the library gives a product: the choice of its launches, asked of
the library itself (it is not part of the C ABI, so by its C++ name)."""
import ctypes

PRODUCTS = ["fwd1", "fwd2", "dA", "dXe", "dW2", "dW1"]


def _ask(name, args, *values):
    from paper_2404_19429_amd import lancet_moe as L
    fn = L._lib[name]
    fn.restype, fn.argtypes = ctypes.c_int, args
    v = fn(*values)
    return v >> 16, v & 0xffff


def expert_tile(cfg, product, later=False, cus=256):
    """(rows, columns) of the tile of one of PRODUCTS, (0, 0) where the device picks 128
    or 256 wide by the row counts; later: a batch partition after the first."""
    return _ask("_ZN4lmoe11expert_tileERK7moe_cfgibi", [ctypes.c_void_p, ctypes.c_int, ctypes.c_bool, ctypes.c_int],
                ctypes.byref(cfg), PRODUCTS.index(product), later, cus)


def dense_tile(M, N, K, cus=256):
    return _ask("_ZN4lmoe10dense_tileEliii", [ctypes.c_int64] + [ctypes.c_int] * 3, M, N, K, cus)
