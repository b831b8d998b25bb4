"""ctypes view of libkbl.so (include/kbl.h).  Argument marshalling only."""

from __future__ import annotations

import ctypes as C
import os
import re

HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(HERE, "libkbl.so")
HEADER = os.path.join(os.path.dirname(HERE), "include", "kbl.h")
HEADERS = (HEADER, os.path.join(os.path.dirname(HERE), "include", "kbl_fr1d.h"))

KBL_OK = 0
KBL_ERR_ARG = 1
KBL_ERR_GAMMA = 2
KBL_ERR_GRID = 3
KBL_ERR_UNSUPPORTED = 4
KBL_ERR_HIP = 5
KBL_ERR_WORKSPACE = 6
NOALLOC_WORKSPACE_BYTES = 256 << 20

GRID_GLOBAL = 0
GRID_STENCIL = 1

PREC_FP64 = 0
PREC_MIXED_BF16 = 1
PREC_MIXED_FP16 = 2
PREC_MIXED_FP32 = 3
# Launch configurations behind the tile indices of kbl_autotune_bounds
# (FP64 2D: threads BX x BY, nodes per thread TX x TY, table mode, where mode
# 3 is the culling kernel with one element per wave; mixed 2D:
# x tiles per wave, y k-steps, waves per workgroup).
FP64_TILES = {0: (16, 16, 1, 1, 0), 1: (16, 16, 2, 2, 0), 2: (16, 16, 3, 3, 0),
              3: (16, 16, 3, 3, 1), 4: (16, 8, 3, 6, 0), 5: (16, 16, 4, 4, 0),
              6: (16, 16, 4, 4, 1), 7: (32, 8, 2, 8, 1), 8: (16, 16, 2, 4, 0),
              9: (16, 16, 4, 2, 0), 10: (16, 16, 2, 2, 2), 11: (16, 16, 3, 3, 2),
              12: (16, 16, 4, 4, 2), 13: (16, 8, 3, 6, 2), 14: (16, 16, 4, 4, 3)}
# d = 3 tiles: (BX, BY, BZ, TX, TY, TZ) covers nx <= BX TX, ny <= BY TY, any nz
# (9 is the culling kernel)
FP64_TILES_3D = {0: (8, 8, 4, 2, 2, 2), 1: (8, 8, 4, 3, 3, 1), 2: (16, 16, 1, 2, 2, 2),
                 3: (16, 16, 1, 3, 3, 1), 4: (16, 16, 1, 4, 4, 1), 5: (8, 8, 4, 2, 2, 4),
                 6: (8, 8, 4, 3, 3, 2), 7: (8, 8, 4, 4, 4, 1), 8: (16, 16, 1, 3, 3, 2), 9: (8, 8, 4, 8, 8, 2)}
MIXED_TILES = {0: (1, 1, 1), 1: (2, 2, 1), 2: (1, 2, 2), 3: (3, 3, 1), 4: (1, 3, 3),
               5: (2, 4, 2), 6: (1, 4, 4)}
# launch shapes of kbl_autotune_bounds' result (8 * tile + shape)
AUTOTUNE_SHAPES = ({"elements_per_workgroup": 1}, {"workgroups_per_cu": 1},
                   {"workgroups_per_cu": 2}, {"workgroups_per_cu": 4},
                   {"workgroups_per_cu": 8}, {"elements_per_workgroup": 2},
                   {"elements_per_workgroup": 4})


def decode_autotune(c: int) -> dict:
    """Tile index and launch shape of a kbl_autotune_bounds result."""
    return {"tile": c // 8, **AUTOTUNE_SHAPES[c % 8]}


def launch_workgroups(shape: dict, n_elem: int, n_cu: int) -> int:
    """Workgroups of a launch shape (as decode_autotune gives it) for n_elem elements."""
    if "workgroups_per_cu" in shape:
        return min(n_elem, shape["workgroups_per_cu"] * n_cu)
    k = min(shape["elements_per_workgroup"], n_elem)
    if k <= 1:
        return n_elem
    return 8 * (((n_elem + 7) // 8 + k - 1) // k)   # k consecutive elements per workgroup


RS_BAD_INPUT = 1 << 16
FLAG_INDEPENDENT_ALPHA = 0x1
FLAG_ENERGY_PERSTATE = 0x2

ST_INADMISSIBLE = 0x1
ST_RHO_FLOOR = 0x2
ST_EPS_RULE = 0x4
ST_LIMITED = 0x8
ST_PSTEP = 0x10
ST_PMEAN_FLOOR = 0x20
ST_MEAN_OUTSIDE = 0x40
ST_BAD_BOUNDS = 0x80
ST_BAD_STENCIL = 0x100
ST_TOO_LARGE = 0x200
ST_ASYMMETRIC = 0x400


class VGrid(C.Structure):
    _fields_ = [("mode", C.c_int32), ("n", C.c_int32 * 3), ("lo", C.c_double * 3),
                ("hi", C.c_double * 3), ("k", C.c_double)]


class Params(C.Structure):
    _fields_ = [("gamma", C.c_double), ("r_fac", C.c_double), ("rho_floor", C.c_double),
                ("p_floor", C.c_double), ("eps_alpha", C.c_double), ("precision", C.c_int32),
                ("flags", C.c_int32)]


FR_PERIODIC = 0
FR_DIRICHLET = 1
FR_MAX_DEGREE = 7


class Fr1dCfg(C.Structure):
    _fields_ = [("p", C.c_int32), ("bc", C.c_int32), ("n_elem", C.c_int64), ("x0", C.c_double),
                ("x1", C.c_double), ("left", C.c_double * 3), ("right", C.c_double * 3),
                ("limit", C.c_int32), ("reserved", C.c_int32)]


class KblError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        msg = _load().kbl_status_string(code).decode() if _lib is not None else str(code)
        super().__init__(f"{where}: {msg} (status {code})")


_lib = None


def header_symbols():
    """Entry points declared in include/kbl.h and include/kbl_fr1d.h."""
    txt = "".join(open(h).read() for h in HEADERS)
    return sorted(set(re.findall(r"^\s*(?:[\w\s\*]+?)\b(kbl_\w+)\s*\(", txt, flags=re.M)))


def _load():
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                f"libkbl.so is not built ({LIB_PATH}); run `python -m paper_2407_20966_amd.build`")
        lib = C.CDLL(LIB_PATH)
        P = C.c_void_p
        lib.kbl_default_params.argtypes = [C.POINTER(Params), C.c_double]
        lib.kbl_default_params.restype = None
        lib.kbl_status_string.argtypes = [C.c_int]
        lib.kbl_status_string.restype = C.c_char_p
        lib.kbl_version.argtypes = []
        lib.kbl_version.restype = C.c_int32
        lib.kbl_compute_bounds.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64, C.c_int32,
                                           C.c_int64, P, P, P, C.POINTER(VGrid), P, P, P]
        lib.kbl_compute_bounds.restype = C.c_int
        lib.kbl_limit.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64, C.c_int32,
                                  P, P, P, P, P, P, P]
        lib.kbl_limit.restype = C.c_int
        lib.kbl_compute_bounds_nodes.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64,
                                                 C.c_int64, C.c_int64, P, P, P, C.POINTER(VGrid),
                                                 P, P, P]
        lib.kbl_compute_bounds_nodes.restype = C.c_int
        lib.kbl_riemann_states.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64, C.c_int64,
                                           P, P, P, P, P, P, P, C.c_int64, P, P, P]
        lib.kbl_riemann_states.restype = C.c_int
        lib.kbl_autotune_bounds.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64, C.c_int32,
                                            C.c_int64, P, P, P, C.POINTER(VGrid), P, P,
                                            C.c_int64, P]
        lib.kbl_autotune_bounds.restype = C.c_int32
        lib.kbl_autotune_clear.argtypes = []
        lib.kbl_autotune_clear.restype = None
        lib.kbl_bounds_launch.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64, C.c_int32,
                                          C.c_int64, C.POINTER(VGrid), C.POINTER(C.c_int32),
                                          C.POINTER(C.c_int64)]
        lib.kbl_bounds_launch.restype = C.c_int
        lib.kbl_backward_workspace_bytes.argtypes = [C.c_int32, C.c_int64, C.c_int32, C.c_int64]
        lib.kbl_backward_workspace_bytes.restype = C.c_size_t
        lib.kbl_bounds_limit_backward.argtypes = [C.POINTER(Params), C.c_int32, C.c_int64,
                                                  C.c_int32, C.c_int64, P, P, P,
                                                  C.POINTER(VGrid), P, P, P, P, P, P, P, P,
                                                  P, P, C.c_size_t, P]
        lib.kbl_bounds_limit_backward.restype = C.c_int
        lib.kbl_bounds_limit_backward_noalloc.argtypes = [C.POINTER(Params), C.c_int32,
                                                          C.c_int64, C.c_int32, C.c_int64, P, P,
                                                          P, C.POINTER(VGrid), P, P, P, P, P, P,
                                                          P, P, P, P]
        lib.kbl_bounds_limit_backward_noalloc.restype = C.c_int
        lib.kbl_status_summary.argtypes = [P, C.c_int64, P, P]
        lib.kbl_status_summary.restype = C.c_int
        F = C.POINTER(Fr1dCfg)
        lib.kbl_fr1d_columns.argtypes = [F]
        lib.kbl_fr1d_columns.restype = C.c_int64
        lib.kbl_fr1d_workspace_bytes.argtypes = [F]
        lib.kbl_fr1d_workspace_bytes.restype = C.c_size_t
        lib.kbl_fr1d_rhs.argtypes = [F, C.c_double, P, P, P]
        lib.kbl_fr1d_rhs.restype = C.c_int
        lib.kbl_fr1d_limit.argtypes = [F, C.POINTER(Params), C.POINTER(VGrid), P, P, C.c_size_t,
                                       P, P]
        lib.kbl_fr1d_limit.restype = C.c_int
        lib.kbl_fr1d_step.argtypes = [F, C.POINTER(Params), C.POINTER(VGrid), C.c_double, P, P,
                                      C.c_size_t, P, P]
        lib.kbl_fr1d_step.restype = C.c_int
        lib.kbl_fr1d_max_speed.argtypes = [F, C.c_double, P, P, P]
        lib.kbl_fr1d_max_speed.restype = C.c_int
        lib.kbl_fr1d_cfl_dt.argtypes = [F, C.c_double, P, C.c_double, C.c_double, P, P]
        lib.kbl_fr1d_cfl_dt.restype = C.c_int
        lib.kbl_fr1d_step_dev.argtypes = [F, C.POINTER(Params), C.POINTER(VGrid), P, P, P,
                                          C.c_size_t, P, P]
        lib.kbl_fr1d_step_dev.restype = C.c_int
        _lib = lib
    return _lib


def bounds_launch(params: Params, dim: int, n_elem: int, n_s: int, nnz: int, vgrid: VGrid):
    """(tile, blocks) that kbl_compute_bounds would choose now for such a call."""
    tile, blocks = C.c_int32(), C.c_int64()
    rc = lib().kbl_bounds_launch(C.byref(params), dim, n_elem, n_s, nnz, C.byref(vgrid),
                                 C.byref(tile), C.byref(blocks))
    if rc != KBL_OK:
        raise KblError(rc, "kbl_bounds_launch")
    return tile.value, blocks.value


def lib():
    return _lib if _lib is not None else _load()
