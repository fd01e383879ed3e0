"""Helpers shared by the GPU parity tests and those of the host-side plans."""
import ctypes

import numpy as np
import torch

from paper_2407_19775_amd import binding


def to_gpu(a: np.ndarray) -> torch.Tensor:
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def to_np(t: torch.Tensor) -> np.ndarray:
    return t.detach().cpu().numpy()


def assert_y_close(y_gpu: np.ndarray, y_ref: np.ndarray, rel: float = 1e-2):
    """The fp16 output bar: relative Frobenius error <= rel and, element by element,
    |delta| <= rel * |ref| + rel * rms(ref).  Returns the observed worst ratios."""
    g = y_gpu.astype(np.float64)
    r = y_ref.astype(np.float64)
    assert g.shape == r.shape
    assert np.all(np.isfinite(g))
    if r.size == 0:
        return 0.0, 0.0
    fro = np.linalg.norm(g - r) / max(np.linalg.norm(r), 1e-30)
    rms = np.sqrt(np.mean(r * r))
    bound = rel * np.abs(r) + rel * rms
    worst = float(np.max(np.abs(g - r) / np.maximum(bound, 1e-30)))
    assert fro <= rel, ("Frobenius", fro)
    assert worst <= 1.0, ("elementwise", worst)
    return fro, worst


def gemm_splits(M: int, K: int, N: int) -> int:
    """Ranges into which the tiled GEMM splits K, as the library plans it (a C++ function of it, outside its C ABI)."""
    f = binding.lib()._ZN4mmd816plan_gemm_splitsEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_int
    return f(M, K, N)


def ranges_on_small_tiles(M: int, K: int, N: int) -> bool:
    """Whether those ranges go on 128 x 128 tiles (a C++ function of the library)."""
    f = binding.lib()._ZN4mmd824one_round_of_small_tilesEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_bool
    s = gemm_splits(M, K, N)
    return s > 1 and f(M, N, s)


class CriticalPlan(ctypes.Structure):
    _fields_ = [("g_slabs", ctypes.c_int), ("dense_from", ctypes.c_int)]


def critical_column_plan(M: int, K: int, N: int, splits: int = None):
    """How many critical columns the tiled GEMM takes as fp16 slabs through its ring, and from how many on it makes
    its dense pass instead, by the library's own plan (a C++ function of it, outside its C ABI)."""
    f = binding.lib()._ZN4mmd821plan_critical_columnsEiiibi
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int], CriticalPlan
    p = f(M, (K + 127) // 128 * 2, N, True, splits or gemm_splits(M, K, N))
    return 32 * (8 + p.g_slabs), max(257, p.dense_from)          # (never for what the first eight slabs hold)


def lora_read_column(s: int, end: int, kq: int, K: int) -> int:
    """First of the 16 columns that a lane group of the adapter's down-projection reads (a C++ function of the library)."""
    f = binding.lib()._ZN4mmd816lora_read_columnEiiii
    f.argtypes, f.restype = [ctypes.c_int] * 4, ctypes.c_int
    return f(s, end, kq, K)


def lora_ranges_in(nbytes: int, M: int, K: int, N: int, r: int) -> int:
    """Ranges of K of an adapter's down-projection in a workspace of that many bytes, 0 where the call is refused (a C++
    function of the library)."""
    f = binding.lib()._ZN4mmd812plan_lora_inEmiiii
    f.argtypes, f.restype = [ctypes.c_size_t] + [ctypes.c_int] * 4, ctypes.c_int
    return f(nbytes, M, K, N, r)


def static_decode_plan(M: int, K: int, N: int):
    """Ranges of K and rows per pass of the decode kernels in the array of the entry point without a workspace (a C++ function
    of the library)."""
    class Plan(ctypes.Structure):
        _fields_ = [("splits", ctypes.c_int), ("pass_rows", ctypes.c_int)]
    f = binding.lib()._ZN4mmd818plan_static_decodeEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, Plan
    p = f(M, K, N)
    return p.splits, p.pass_rows


def prep_single_rows(M: int, K: int) -> bool:
    """Whether more than 128 rows are prepared with a row per workgroup (a C++ function of the library)."""
    f = binding.lib()._ZN4mmd816prep_single_rowsEii
    f.argtypes, f.restype = [ctypes.c_int] * 2, ctypes.c_bool
    return f(M, K)


def panel_plan(M: int, K: int, N: int):
    """Ranges of K of the kernel for a few rows that prepares its own operands and splits K, and the 64-column slabs of a range (a
    C++ function of the library); 0 ranges: not for this call."""
    class Plan(ctypes.Structure):
        _fields_ = [(name, ctypes.c_int) for name in ("n_slabs", "tiles_n", "splits", "slabs_per_split")]
    f = binding.lib()._ZN4mmd810plan_panelEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, Plan
    p = f(M, K, N)
    return p.splits, p.slabs_per_split


def rows_kernel_fits(M: int, K: int, N: int) -> bool:
    """Whether the layer is the single kernel for a few rows (a C++ function of the library)."""
    f = binding.lib()._ZN4mmd816rows_kernel_fitsEiii
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_bool
    return f(M, (K + 127) // 128 * 128, N)
