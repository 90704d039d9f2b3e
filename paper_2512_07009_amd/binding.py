"""Python binding of libflock (the C ABI in include/flock.h).

Argument marshalling only: torch tensors provide device memory and the
current HIP stream; every step of the computation runs in the library's HIP
kernels.  There is no CPU fallback: if libflock.so is missing or the device is
not a gfx950 GPU, calls raise.
"""

from __future__ import annotations

import ctypes
import os

import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "libflock.so")

FLOCK_OK = 0
FLOCK_EINVAL = -1
FLOCK_ENOMEM = -2
FLOCK_EDEVICE = -3
FLOCK_EUNSUPPORTED = -4

QUANTA_PER_PX = 16

_lib = None


class FlockError(RuntimeError):
    def __init__(self, status: int, message: str):
        super().__init__(f"flock status {status}: {message}")
        self.status = status


def lib() -> ctypes.CDLL:
    """The loaded libflock.so (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: build it with "
                               "`python -m paper_2512_07009_amd.build` (there is no fallback path)")
        L = ctypes.CDLL(LIB_PATH)
        p, i32, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
        L.cluster_frames.argtypes = [p, p, i32, i32, i32, i32, i32, p, p, p, p, sz, p]
        L.cluster_frames.restype = i32
        L.density_frames.argtypes = [p, p, i32, i32, i32, i32, i32, i32, i32, ctypes.c_float, p, p, sz, p]
        L.density_frames.restype = i32
        L.cluster_frames_workspace.argtypes = [i32, i32, i32]
        L.cluster_frames_workspace.restype = sz
        L.density_frames_noalloc.argtypes = [p, p, i32, i32, i32, i32, i32, i32, i32, ctypes.c_float, p, p]
        L.density_frames_noalloc.restype = i32
        L.density_frames_workspace.argtypes = [i32, i32, i32, i32]
        L.density_frames_workspace.restype = sz
        L.heatmap_frames.argtypes = [p, i32, i32, i32, ctypes.c_double, ctypes.c_float, i32,
                                     p, p, p, p, p, p, p, sz, p]
        L.heatmap_frames.restype = i32
        L.heatmap_frames_workspace.argtypes = [i32, i32, i32]
        L.heatmap_frames_workspace.restype = sz
        L.roi_filter_frames.argtypes = [p, p, i32, i32, p, i32, p, p, p, p, p, sz, p]
        L.roi_filter_frames.restype = i32
        L.roi_filter_frames_workspace.argtypes = [i32, i32]
        L.roi_filter_frames_workspace.restype = sz
        L.drinker_proximity_frames.argtypes = [p, p, i32, i32, p, i32, i32, p, p, p, p, sz, p]
        L.drinker_proximity_frames.restype = i32
        L.drinker_proximity_frames_workspace.argtypes = [i32, i32]
        L.drinker_proximity_frames_workspace.restype = sz
        L.mask_components_frames.argtypes = [p, i32, i32, i32, ctypes.c_float, i32, p, p, p, i32,
                                             p, p, p, p, p, p, p, sz, p]
        L.mask_components_frames.restype = i32
        L.mask_components_frames_workspace.argtypes = [i32, i32, i32, i32]
        L.mask_components_frames_workspace.restype = sz
        L.flock_last_error.argtypes = []
        L.flock_last_error.restype = ctypes.c_char_p
        L.flock_version.argtypes = []
        L.flock_version.restype = ctypes.c_char_p
        _lib = L
    return _lib


def _check(status: int):
    if status != FLOCK_OK:
        msg = lib().flock_last_error().decode()
        if status == FLOCK_EINVAL:
            raise ValueError(f"flock: {msg}")
        raise FlockError(status, msg)


def _ptr(t):
    return t.data_ptr() if t is not None else None


# The current device and a device's current stream, without the objects that
# torch.cuda.current_device() and current_stream() make (about 1 us each; a
# call with one small kernel takes about 10 us in all).
_current_device = getattr(torch._C, "_cuda_getDevice", None) or torch.cuda.current_device
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None) or \
    (lambda index: torch.cuda.current_stream(index).cuda_stream)


def _workspace(nbytes: int, dev, stream):
    """Scratch for one call, allocated on the stream the kernels run on.
    torch's caching allocator hands a freed block out again only to work
    ordered after it on that stream, so the block is not reused before the
    kernels finish, with no cross-stream bookkeeping (and none under graph
    capture, where the block comes from the graph's own pool)."""
    if not nbytes:
        return None
    if stream is None or stream.cuda_stream == _raw_stream(dev.index):
        return torch.empty(nbytes, dtype=torch.uint8, device=dev)  # on dev's current stream
    with torch.cuda.device(dev), torch.cuda.stream(stream):
        return torch.empty(nbytes, dtype=torch.uint8, device=dev)


def _call(fn, dev, stream, *args):
    """fn(*args, stream) with dev as the current device."""
    if _current_device() == dev.index:
        st = fn(*args, _raw_stream(dev.index) if stream is None else stream.cuda_stream)
    else:
        with torch.cuda.device(dev):
            st = fn(*args, _raw_stream(dev.index) if stream is None else stream.cuda_stream)
    _check(st)


def _batch(xy: torch.Tensor, offsets: torch.Tensor):
    if not (xy.is_cuda and offsets.is_cuda):
        raise ValueError("xy and offsets must be device tensors")
    if xy.dtype != torch.int32 or offsets.dtype != torch.int32:
        raise ValueError("xy and offsets must be int32")
    if xy.dim() != 2 or xy.shape[1] != 2 or not xy.is_contiguous():
        raise ValueError("xy must be a contiguous [T, 2] tensor")
    if offsets.dim() != 1 or offsets.numel() < 1 or not offsets.is_contiguous():
        raise ValueError("offsets must be a contiguous [F + 1] tensor")
    return offsets.numel() - 1, xy.shape[0]


def eps_to_quanta(eps_px: float) -> int:
    q = eps_px * QUANTA_PER_PX
    if abs(q - round(q)) > 1e-9:
        raise ValueError(f"eps_px = {eps_px} is not a multiple of 1/16 px")
    return int(round(q))


def cluster_frames(xy: torch.Tensor, offsets: torch.Tensor, eps_px: float, min_pts: int,
                   max_frame_points: int = 0, out=None, stream=None):
    """Cluster every frame; returns (labels int32[T], kind uint8[T], n_clusters int32[F]).

    max_frame_points: an upper bound on birds per frame (0 = unknown); it
    sizes on-chip storage and is not checked against the data.
    out: optional (labels, kind, n_clusters) tensors to write into.
    """
    F, T = _batch(xy, offsets)
    dev = xy.device
    if out is None:
        labels = torch.empty(T, dtype=torch.int32, device=dev)
        kind = torch.empty(T, dtype=torch.uint8, device=dev)
        ncl = torch.empty(max(F, 0), dtype=torch.int32, device=dev)
    else:
        labels, kind, ncl = out
    L = lib()
    ws_bytes = L.cluster_frames_workspace(F, T, int(max_frame_points))
    ws = _workspace(ws_bytes, dev, stream)
    _call(L.cluster_frames, dev, stream, _ptr(xy), _ptr(offsets), F, T, int(max_frame_points),
          eps_to_quanta(eps_px), int(min_pts), _ptr(labels), _ptr(kind), _ptr(ncl), _ptr(ws), ws_bytes)
    return labels, kind, ncl


def density_frames(xy: torch.Tensor, offsets: torch.Tensor, width_px: int, height_px: int,
                   grid_w: int, grid_h: int, sigma_px: float, max_frame_points: int = 0, out=None,
                   stream=None):
    """Gaussian density grid of every frame: float32[F, grid_h, grid_w] (birds / px^2).

    max_frame_points: an upper bound on birds per frame, or 0 (a planning hint).
    """
    F, T = _batch(xy, offsets)
    dev = xy.device
    dens = out if out is not None else torch.empty((max(F, 0), grid_h, grid_w), dtype=torch.float32,
                                                  device=dev)
    L = lib()
    ws_bytes = L.density_frames_workspace(F, T, int(grid_w), int(grid_h))
    ws = _workspace(ws_bytes, dev, stream)
    _call(L.density_frames, dev, stream, _ptr(xy), _ptr(offsets), F, T, int(max_frame_points), int(width_px),
          int(height_px), int(grid_w), int(grid_h), float(sigma_px), _ptr(dens), _ptr(ws), ws_bytes)
    return dens


def heatmap_frames(density: torch.Tensor, cell_area_px2: float, threshold: float, connectivity: int = 8,
                   out=None, stream=None):
    """Heatmap analytics of float32 density grids [F, grid_h, grid_w] on the device.

    Returns a dict of device tensors: labels int32[F, h, w] (smallest cell
    index of the component, -1 for cold cells), n_components int32[F],
    entropy float64[F], degree float64[F], comp_cells int32[F, h, w] and
    comp_mass float64[F, h, w] (at label cells, 0 elsewhere).
    out: optional dict of such tensors to write into.
    """
    if not density.is_cuda or density.dtype != torch.float32 or density.dim() != 3 \
            or not density.is_contiguous():
        raise ValueError("density must be a contiguous float32 device tensor [F, grid_h, grid_w]")
    F, gh, gw = density.shape
    dev = density.device
    if out is None:
        out = {"labels": torch.empty((F, gh, gw), dtype=torch.int32, device=dev),
               "n_components": torch.empty(F, dtype=torch.int32, device=dev),
               "entropy": torch.empty(F, dtype=torch.float64, device=dev),
               "degree": torch.empty(F, dtype=torch.float64, device=dev),
               "comp_cells": torch.empty((F, gh, gw), dtype=torch.int32, device=dev),
               "comp_mass": torch.empty((F, gh, gw), dtype=torch.float64, device=dev)}
    L = lib()
    ws_bytes = L.heatmap_frames_workspace(F, gw, gh)
    ws = _workspace(ws_bytes, dev, stream)
    _call(L.heatmap_frames, dev, stream, _ptr(density), F, gw, gh, float(cell_area_px2), float(threshold),
          int(connectivity), _ptr(out["labels"]), _ptr(out["n_components"]), _ptr(out["entropy"]),
          _ptr(out["degree"]), _ptr(out["comp_cells"]), _ptr(out["comp_mass"]), _ptr(ws), ws_bytes)
    return out


def roi_filter_frames(xy: torch.Tensor, offsets: torch.Tensor, roi_xy, with_index: bool = True, out=None,
                      stream=None):
    """Birds inside the closed ROI polygon roi_xy (host, [V, 2] int quanta).

    Returns a dict of device tensors: counts int32[F], xy int32[T, 2]
    (capacity; the first offsets[F] rows are the kept birds, frame after
    frame), offsets int32[F + 1], index int32[T] (capacity; input index of
    each kept bird) or None.
    """
    import numpy as np
    F, T = _batch(xy, offsets)
    poly = np.ascontiguousarray(np.asarray(roi_xy, dtype=np.int32).reshape(-1, 2))
    dev = xy.device
    if out is None:
        out = {"counts": torch.empty(max(F, 0), dtype=torch.int32, device=dev),
               "xy": torch.empty((T, 2), dtype=torch.int32, device=dev),
               "offsets": torch.empty(F + 1, dtype=torch.int32, device=dev),
               "index": torch.empty(T, dtype=torch.int32, device=dev) if with_index else None}
    L = lib()
    ws_bytes = L.roi_filter_frames_workspace(F, T)
    ws = _workspace(ws_bytes, dev, stream)
    _call(L.roi_filter_frames, dev, stream, _ptr(xy), _ptr(offsets), F, T, poly.ctypes.data, poly.shape[0],
          _ptr(out["counts"]), _ptr(out["xy"]), _ptr(out["offsets"]), _ptr(out.get("index")), _ptr(ws),
          ws_bytes)
    return out


def drinker_proximity_frames(xy: torch.Tensor, offsets: torch.Tensor, lines, threshold_q: int,
                             with_line: bool = True, out=None, stream=None):
    """Birds strictly closer than threshold_q (1/16 px) to some drinker-line
    segment; lines: host [L, 4] int (ax, ay, bx, by) in 1/16 px.

    Returns a dict of device tensors: drinking uint8[T], line int32[T]
    (smallest index of such a segment, -1 if none) or None, counts int32[F].
    """
    import numpy as np
    F, T = _batch(xy, offsets)
    ln = np.ascontiguousarray(np.asarray(lines, dtype=np.int32).reshape(-1, 4))
    dev = xy.device
    if out is None:
        out = {"drinking": torch.empty(T, dtype=torch.uint8, device=dev),
               "line": torch.empty(T, dtype=torch.int32, device=dev) if with_line else None,
               "counts": torch.empty(max(F, 0), dtype=torch.int32, device=dev)}
    L = lib()
    ws_bytes = L.drinker_proximity_frames_workspace(F, T)
    ws = _workspace(ws_bytes, dev, stream)
    _call(L.drinker_proximity_frames, dev, stream, _ptr(xy), _ptr(offsets), F, T, ln.ctypes.data, ln.shape[0],
          int(threshold_q), _ptr(out["drinking"]), _ptr(out.get("line")), _ptr(out["counts"]), _ptr(ws),
          ws_bytes)
    return out


def mask_capacity(n_frames: int, height: int, width: int, connectivity: int = 8) -> int:
    """Most components a batch of this shape can hold (isolated pixels on
    every other row and column with 8 neighbours, a checkerboard with 4)."""
    if connectivity == 8:
        return n_frames * ((height + 1) // 2) * ((width + 1) // 2)
    return n_frames * ((height * width + 1) // 2)


def mask_components_frames(prob: torch.Tensor, threshold: float, connectivity: int = 8, with_labels: bool = True,
                           capacity: int | None = None, out=None, stream=None):
    """Connected components of prob > threshold in float32 device masks
    [F, H, W], with statistics (the detection post-processing).

    Returns a dict of device tensors: labels int32[F, H, W] (first pixel of
    the component in raster order, -1 background) or None, n_components
    int32[F], offsets int32[F + 1] (offsets[F] = number of components K),
    and per component, in rows 0 .. min(K, capacity) - 1: label int32[C],
    area int32[C], box int32[C, 4] (x, y, width, height), centroid
    float64[C, 2], xy int32[C, 2] (1/16 px), score float32[C].  capacity
    defaults to the most components the shape can hold.
    """
    if not prob.is_cuda or prob.dtype != torch.float32 or prob.dim() != 3 or not prob.is_contiguous():
        raise ValueError("prob must be a contiguous float32 device tensor [F, H, W]")
    F, H, W = prob.shape
    dev = prob.device
    if capacity is None:
        capacity = mask_capacity(F, H, W, connectivity)
    C = int(capacity)
    if out is None:
        out = {"labels": torch.empty((F, H, W), dtype=torch.int32, device=dev) if with_labels else None,
               "n_components": torch.empty(F, dtype=torch.int32, device=dev),
               "offsets": torch.empty(F + 1, dtype=torch.int32, device=dev),
               "label": torch.empty(C, dtype=torch.int32, device=dev),
               "area": torch.empty(C, dtype=torch.int32, device=dev),
               "box": torch.empty((C, 4), dtype=torch.int32, device=dev),
               "centroid": torch.empty((C, 2), dtype=torch.float64, device=dev),
               "xy": torch.empty((C, 2), dtype=torch.int32, device=dev),
               "score": torch.empty(C, dtype=torch.float32, device=dev)}
    L = lib()
    ws_bytes = L.mask_components_frames_workspace(F, W, H, int(connectivity))
    ws = _workspace(ws_bytes, dev, stream)
    _call(L.mask_components_frames, dev, stream, _ptr(prob), F, W, H, float(threshold), int(connectivity),
          _ptr(out.get("labels")), _ptr(out["n_components"]), _ptr(out["offsets"]), C, _ptr(out.get("label")),
          _ptr(out.get("area")), _ptr(out.get("box")), _ptr(out.get("centroid")), _ptr(out.get("xy")),
          _ptr(out.get("score")), _ptr(ws), ws_bytes)
    return out


def version() -> str:
    return lib().flock_version().decode()
