"""The GEMM forms the library picks, asked from its host code (no GPU needed):
the rows of a tile and the number of parts that a product's K range is cut into.
gemm_plan and gemm_max_splits of kernels.h, by their C++ names."""
import ctypes as C

import paper_2411_06465_amd as L

STORE_BF16, ACC_F32 = 0, 2        # EpiKind


class _Plan(C.Structure):
    _fields_ = [("tile", C.c_int32), ("splits", C.c_int32), ("stream_c", C.c_bool)]


def plan(M, N, K, kind, max_splits):
    """Of a product of the layer backward."""
    f = L.lib()._ZN3l4d9gemm_planElllNS_7EpiKindEib
    f.argtypes, f.restype = [C.c_int64] * 3 + [C.c_int, C.c_int, C.c_bool], _Plan
    p = f(M, N, K, kind, max_splits, True)
    return p.tile, p.splits


def layer_max_splits(M, N, K, kind):
    f = L.lib()._ZN3l4d15gemm_max_splitsElllb
    f.argtypes, f.restype = [C.c_int64] * 3 + [C.c_bool], C.c_int
    return f(M, N, K, kind == ACC_F32)


def layer_plans(w):
    """(tile, splits) of the products of a layer backward that may split."""
    d, tok = w.d_h, w.micro_batch * w.s_c
    nq, qkv = w.a_t * d, (w.a_t + 2 * w.k_t) * d
    shapes = dict(o_dx=(tok, nq, w.hidden, STORE_BF16), o_dw=(w.hidden, nq, tok, ACC_F32),
                  qkv_dw=(qkv, w.hidden, tok, ACC_F32), gate_up_dw=(2 * w.f_t, w.hidden, tok, ACC_F32),
                  down_dw=(w.hidden, w.f_t, tok, ACC_F32))
    return {n: plan(*s, layer_max_splits(*s)) for n, s in shapes.items()}
