"""The library's dispatch rules and its products, called directly (ctypes on the
C++ symbols that csrc/ops.h declares; test_plans.py checks the struct layouts)."""
import ctypes as C

from paper_2606_04484_amd import capi

AJ_OK = 0
vp, i32, i64 = C.c_void_p, C.c_int, C.c_int64


class GemmPlan(C.Structure):
    _fields_ = [("tile", i32), ("long_k", C.c_bool), ("tiles", i32), ("whole", i32), ("split", i32),
                ("k_piece", i32)]


class Gemm(C.Structure):
    _fields_ = [("M", i32), ("N", i32), ("K", i32), ("A", vp), ("lda", i64), ("a_kmajor", C.c_bool),
                ("B", vp), ("ldb", i64), ("b_kmajor", C.c_bool), ("C", vp), ("ldc", i64),
                ("c_f32", C.c_bool), ("out", i32), ("R", vp), ("partial", vp),
                ("partial_cap", C.c_size_t), ("swiglu_gu", vp), ("recompute", C.c_bool), ("A2", vp),
                ("lda2", i64), ("B2", vp), ("ldb2", i64), ("K2", i32)]


class AttnArgs(C.Structure):
    _fields_ = [("n_tok", i32), ("n_seg", i32), ("Hq", i32), ("Hkv", i32), ("hd", i32), ("base", i32),
                ("cu_seqlens", vp), ("qkv", vp), ("o", vp), ("lse", vp), ("scale", C.c_float)]


class AttnBwdArgs(C.Structure):
    _fields_ = [("n_tok", i32), ("n_seg", i32), ("Hq", i32), ("Hkv", i32), ("hd", i32), ("base", i32),
                ("cu_seqlens", vp), ("qkv", vp), ("o", vp), ("dout", vp), ("lse", vp), ("delta", vp),
                ("dqkv", vp), ("scale", C.c_float), ("part", vp), ("part_floats", C.c_size_t)]


STRUCTS = {"GemmPlan": GemmPlan, "Gemm": Gemm, "AttnArgs": AttnArgs, "AttnBwdArgs": AttnBwdArgs}


def _fn(name, restype, *argtypes):
    f = getattr(capi.lib(), name)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


def gemm_plan(M, N, K, cap, eight_wave=False):
    return _fn("_ZN2aj9gemm_planEiiimb", GemmPlan, i32, i32, i32, C.c_size_t, C.c_bool)(
        M, N, K, cap, eight_wave)


def partial_floats(M, N):
    """gemm_partial_floats: at most 512 blocks of 256 x 256, 16 a tile."""
    return min(16 * -(-M // 256) * -(-N // 256), 512) * 65536


def gemm_bf16(g, stream):
    rc = _fn("_ZN2aj4gemmItEEiRKNS_4GemmEP12ihipStream_t", i32, C.POINTER(Gemm), vp)(
        C.byref(g), stream)
    assert rc == AJ_OK, rc


def attn_row_waves(n_tok, n_seg, heads):
    return _fn("_ZN2aj14attn_row_wavesEiii", i32, i32, i32, i32)(n_tok, n_seg, heads)


def attn_dkv_parts(a):
    return _fn("_ZN2aj14attn_dkv_partsERKNS_11AttnBwdArgsE", i32, C.POINTER(AttnBwdArgs))(C.byref(a))


def attn_fwd_bf16(a, stream):
    rc = _fn("_ZN2aj8attn_fwdItEEiRKNS_8AttnArgsEP12ihipStream_t", i32, C.POINTER(AttnArgs), vp)(
        C.byref(a), stream)
    assert rc == AJ_OK, rc


def attn_bwd_bf16(a, stream):
    rc = _fn("_ZN2aj8attn_bwdItEEiRKNS_11AttnBwdArgsEP12ihipStream_t", i32, C.POINTER(AttnBwdArgs), vp)(
        C.byref(a), stream)
    assert rc == AJ_OK, rc
