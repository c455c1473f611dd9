"""Which kernel a dense FWD / BWI call runs, asked of the built library on the host.

The interface names the kernels of the zero-skipping forms only (st_conv_kernel_name).  The functions that choose among the dense ones are not
part of it, but the library exports them under their C++ names; the structure they take is st::Geom of st_common.hpp.
"""
import ctypes

import paper_1911_10175_amd as st


class _Geom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("N", "Ci", "Ko", "Hi", "Wi", "Ho", "Wo", "R", "S", "sw", "sh", "pw", "ph", "uw", "uh")] + [
        ("sel", ctypes.c_void_p), ("want", ctypes.c_int), ("thr", ctypes.c_uint), ("describe", ctypes.c_char_p), ("describe_len", ctypes.c_int),
        ("w", ctypes.c_void_p), ("wt", ctypes.c_int)]


def _ask(name, g):
    f = ctypes.CDLL(st.lib_path())[f"_ZN2st{len(name)}{name}ERKNS_4GeomE"]
    f.restype = ctypes.c_bool
    return f(ctypes.byref(g))


def _correlation(d, bwi):
    if bwi:
        return _Geom(N=d.N, Ci=d.K, Ko=d.C, Hi=d.OH, Wi=d.OW, Ho=d.H, Wo=d.W, R=d.R, S=d.S, sw=1, sh=1, pw=d.R - 1 - d.pad_w, ph=d.S - 1 - d.pad_h,
                     uw=d.stride_w, uh=d.stride_h, wt=1)
    return _Geom(N=d.N, Ci=d.C, Ko=d.K, Hi=d.H, Wi=d.W, Ho=d.OH, Wo=d.OW, R=d.R, S=d.S, sw=d.stride_w, sh=d.stride_h, pw=d.pad_w, ph=d.pad_h, uw=1, uh=1)


def f16_pieces(d, bwi=False):
    """Whether that kernel forms its products from two f16 pieces (else from three bf16 ones)."""
    return _ask("fwd_dense_half", _correlation(d, bwi))


def bww_f16_pieces(d):
    """Whether the dense BWW forms its products from two f16 pieces."""
    f = ctypes.CDLL(st.lib_path())["_ZN2st14bww_dense_halfERK12st_conv_desc"]
    f.restype = ctypes.c_bool
    return f(ctypes.byref(d._c()))


def bww_line(d):
    """Zero fraction, per mille, from which on the self-selecting BWW skips zeros."""
    f = ctypes.CDLL(st.lib_path())["_ZN2st20bww_sparse_thresholdERK12st_conv_desc"]
    f.restype = ctypes.c_uint
    return f(ctypes.byref(d._c()))


def dense_kernel(d, bwi=False):
    """ "32" or "16": channels that the kernel on bf16 pieces takes at a time; for 1x1 layers also "lds", whole filters in LDS, and "fp32",
    both on fp32 matrix instructions."""
    g = _correlation(d, bwi)
    if d.R == 3:
        return "32" if _ask("fwd_dense_wide", g) else "16"
    if _ask("pw_dense_direct_supported", g):
        return "lds"
    if _ask("pw_small", g):
        return "fp32"
    return "32" if _ask("pw_wide", g) else "16"
