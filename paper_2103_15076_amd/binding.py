"""Python binding of include/picasso.h: argument marshalling only.

The calls of a step (decimation, pooling, convolutions) go through the compiled
module _host (csrc/host.cpp), the others through ctypes.  torch supplies device
memory and the stream; every step of the path runs in libpicasso_hip.so.  There
is no fallback: if the library is missing or cannot be loaded, ``load_library`` raises.
"""
from __future__ import annotations

import ctypes
import os

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libpicasso_hip.so")

PICASSO_OK = 0
PICASSO_WARN_BUDGET_UNMET = 1
PICASSO_ERR_INVALID_ARG = -1
PICASSO_ERR_BAD_INDEX = -2
PICASSO_ERR_NONFINITE = -3
PICASSO_ERR_WORKSPACE = -4
PICASSO_ERR_HIP = -5
PICASSO_ERR_INTERNAL = -6

PICASSO_OPT_MAX_ROUNDS = 0
PICASSO_OPT_STAGE_TIMING = 1
PICASSO_OPT_SUBROUND_BATCH = 2
PICASSO_OPT_KERNEL_TIMING = 3
PICASSO_OPT_OVERLAP = 4
PICASSO_OPT_TRUNC_BLOCK_MAX = 5
PICASSO_OPT_PLACEMENT = 6
PICASSO_OPT_RCOND_MIN_BITS = 7
PICASSO_OPT_ABSORB = 8
PICASSO_OPT_SHUFFLE_SEED = 9
PICASSO_OPT_HOST_POLL = 10
PICASSO_OPT_LAUNCH_AHEAD = 11
PICASSO_OPT_TRUNC_WIDTH = 12
PICASSO_OPT_DROP_DEGENERATED = 13
PICASSO_OPT_TRUNC_SELECT = 14
PICASSO_PLACE_MEAN, PICASSO_PLACE_INVERSE = 0, 1

(PICASSO_KERNEL_SORT, PICASSO_KERNEL_UNIQUE_COST, PICASSO_KERNEL_SUBROUND0, PICASSO_KERNEL_FACET_INSERT,
 PICASSO_KERNEL_QUADRIC_ROWS, PICASSO_KERNEL_SORT_INCIDENCE, PICASSO_KERNEL_COUNT) = range(7)
TIMED_KERNEL_NAMES = (
    "bucket_keys_kernel (edge-key sort, per-bucket LDS sort, distinct edges)",
    "ring_costs_kernel, facet_costs_kernel; of sorted edges unique_cost_kernel (costs, first bids)",
    "suitor_kernel (the whole matching), select_facets_kernel; of sorted edges select_subround_kernel, select_first_kernel (first sub-round of the selection)",
    "final_facets_kernel; behind rounds of sorted edges edge_keys_kernel (facets and labels re-indexed; behind the last: facet hash set)",
    "bucket_keys_kernel (incidence-key sort, per-bucket LDS sort, vertex quadrics from facet planes)",
    "msd_scatter_kernel, xl_scatter_kernel (incidence-key sort, partition)",
)

PICASSO_STATS_ROUNDS = 32
PICASSO_ST_COUNT = 8
STAGE_NAMES = ("quadrics", "edges", "select", "contract", "facets")

EXPORTED_SYMBOLS = (
    "picasso_workspace_bytes", "picasso_create", "picasso_destroy", "picasso_set_option", "picasso_strerror",
    "picasso_last_hip_error", "picasso_decimate", "picasso_decimate_batch", "picasso_vertex_quadrics",
    "picasso_edge_costs", "picasso_radix_sort", "picasso_kernel_timing",
    "picasso_device_copy", "picasso_bucket_sort", "picasso_cluster_csr", "picasso_replace_mapping",
    "picasso_replace_mapping_static",
    "picasso_vertex_corner_csr", "picasso_facet_geometry", "picasso_fuzzy_coefficients", "picasso_v2f_forward",
    "picasso_v2f_backward", "picasso_f2f_forward", "picasso_f2f_backward", "picasso_f2f_clear_unowned", "picasso_f2v_forward",
    "picasso_f2v_backward", "picasso_pool_forward",
    "picasso_pool_backward", "picasso_unpool_forward", "picasso_unpool_backward",
)

PICASSO_POOL_AVG, PICASSO_POOL_MAX, PICASSO_POOL_WEIGHTED, PICASSO_POOL_SUM = 0, 1, 2, 3


class picasso_stats(ctypes.Structure):
    _fields_ = [
        ("rounds", ctypes.c_int32),
        ("nv_out", ctypes.c_int32),
        ("nf_out", ctypes.c_int32),
        ("nv", ctypes.c_int32 * PICASSO_STATS_ROUNDS),
        ("nf", ctypes.c_int32 * PICASSO_STATS_ROUNDS),
        ("ne", ctypes.c_int32 * PICASSO_STATS_ROUNDS),
        ("nsel", ctypes.c_int32 * PICASSO_STATS_ROUNDS),
        ("subrounds", ctypes.c_int32 * PICASSO_STATS_ROUNDS),
        ("ms_stage", (ctypes.c_float * PICASSO_ST_COUNT) * PICASSO_STATS_ROUNDS),
        ("ms_total", ctypes.c_float),
    ]

    def as_dict(self):
        r = min(self.rounds, PICASSO_STATS_ROUNDS)
        return dict(
            rounds=self.rounds, nv_out=self.nv_out, nf_out=self.nf_out, ms_total=self.ms_total,
            nv=list(self.nv[:r]), nf=list(self.nf[:r]), ne=list(self.ne[:r]), nsel=list(self.nsel[:r]),
            subrounds=list(self.subrounds[:r]),
            ms_stage=[{n: self.ms_stage[i][j] for j, n in enumerate(STAGE_NAMES)} for i in range(max(r, 1))],
        )


_lib = None
_host = None


class PicassoError(RuntimeError):
    def __init__(self, status, msg):
        super().__init__(f"picasso status {status}: {msg}")
        self.status = status


def load_library():
    """Loads libpicasso_hip.so; raises if it has not been built."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(
            f"{LIB_PATH} is missing: build it with `python -m paper_2103_15076_amd.build` "
            "(hipcc, gfx950).  There is no CPU fallback.")
    lib = ctypes.CDLL(LIB_PATH)
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    lib.picasso_workspace_bytes.restype = ctypes.c_size_t
    lib.picasso_workspace_bytes.argtypes = [i64, i64, i32]
    lib.picasso_create.restype = ctypes.c_int
    lib.picasso_create.argtypes = [ctypes.POINTER(vp), ctypes.c_int, i64, i64, i32]
    lib.picasso_destroy.restype = None
    lib.picasso_destroy.argtypes = [vp]
    lib.picasso_set_option.restype = ctypes.c_int
    lib.picasso_set_option.argtypes = [vp, ctypes.c_int, i64]
    lib.picasso_strerror.restype = ctypes.c_char_p
    lib.picasso_strerror.argtypes = [ctypes.c_int]
    lib.picasso_last_hip_error.restype = ctypes.c_char_p
    lib.picasso_last_hip_error.argtypes = [vp]
    lib.picasso_decimate.restype = ctypes.c_int
    lib.picasso_decimate.argtypes = [vp, vp, vp, i32, vp, i32, i32, vp, vp, vp, ctypes.POINTER(i32),
                                     ctypes.POINTER(i32), ctypes.POINTER(picasso_stats)]
    lib.picasso_decimate_batch.restype = ctypes.c_int
    lib.picasso_decimate_batch.argtypes = [vp, vp, i32, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp,
                                           ctypes.POINTER(picasso_stats)]
    lib.picasso_vertex_quadrics.restype = ctypes.c_int
    lib.picasso_vertex_quadrics.argtypes = [vp, vp, vp, i32, vp, i32, vp]
    lib.picasso_edge_costs.restype = ctypes.c_int
    lib.picasso_edge_costs.argtypes = [vp, vp, vp, i32, vp, i32, vp, vp, ctypes.POINTER(i32)]
    lib.picasso_kernel_timing.restype = ctypes.c_int
    lib.picasso_kernel_timing.argtypes = [vp, ctypes.c_int, ctypes.c_int, ctypes.POINTER(i64),
                                          ctypes.POINTER(ctypes.c_double), ctypes.POINTER(ctypes.c_double)]
    lib.picasso_device_copy.restype = ctypes.c_int
    lib.picasso_device_copy.argtypes = [vp, vp, vp, ctypes.c_size_t]
    lib.picasso_radix_sort.restype = ctypes.c_int
    lib.picasso_radix_sort.argtypes = [vp, vp, ctypes.c_int, vp, vp, i64, ctypes.c_int]
    lib.picasso_cluster_csr.restype = ctypes.c_int
    lib.picasso_cluster_csr.argtypes = [vp, vp, vp, i32, i32, vp, vp]
    lib.picasso_replace_mapping.restype = ctypes.c_int
    lib.picasso_replace_mapping.argtypes = [vp, vp, vp, i32, i32, vp, vp]
    lib.picasso_replace_mapping_static.restype = ctypes.c_int
    lib.picasso_replace_mapping_static.argtypes = [ctypes.c_int, vp, vp, i32, i32, vp, vp, vp]
    lib.picasso_vertex_corner_csr.restype = ctypes.c_int
    lib.picasso_vertex_corner_csr.argtypes = [vp, vp, vp, i32, i32, vp, vp]
    lib.picasso_facet_geometry.restype = ctypes.c_int
    lib.picasso_facet_geometry.argtypes = [vp, vp, vp, i32, vp, i32, i32, vp, i32, i32, vp, vp, vp]
    lib.picasso_fuzzy_coefficients.restype = ctypes.c_int
    lib.picasso_fuzzy_coefficients.argtypes = [vp, vp, vp, i32, vp, vp, i32, vp]
    lib.picasso_v2f_forward.restype = ctypes.c_int
    lib.picasso_v2f_forward.argtypes = [vp, vp, vp, i32, i32, vp, i32, vp, vp, vp]
    lib.picasso_v2f_backward.restype = ctypes.c_int
    lib.picasso_v2f_backward.argtypes = [vp, vp, vp, vp, i32, i32, vp, i32, vp, vp, vp, vp, vp, vp]
    lib.picasso_f2f_forward.restype = ctypes.c_int
    lib.picasso_f2f_forward.argtypes = [vp, vp, vp, vp, vp, i32, i32, i32, vp, vp]
    lib.picasso_f2f_backward.restype = ctypes.c_int
    lib.picasso_f2f_backward.argtypes = [vp, vp, vp, vp, vp, vp, i32, i32, i32, vp, vp, vp]
    lib.picasso_f2f_clear_unowned.restype = ctypes.c_int
    lib.picasso_f2f_clear_unowned.argtypes = [vp, vp, vp, i32, i32, i32, vp]
    lib.picasso_f2v_forward.restype = ctypes.c_int
    lib.picasso_f2v_forward.argtypes = [vp, vp, vp, i32, i32, vp, i32, vp, vp, vp, i32, vp]
    lib.picasso_f2v_backward.restype = ctypes.c_int
    lib.picasso_f2v_backward.argtypes = [vp, vp, vp, vp, i32, i32, vp, i32, vp, vp, vp, i32, vp, vp, vp]
    lib.picasso_pool_forward.restype = ctypes.c_int
    lib.picasso_pool_forward.argtypes = [vp, vp, ctypes.c_int, vp, i32, i32, vp, vp, i32, vp, vp, vp]
    lib.picasso_pool_backward.restype = ctypes.c_int
    lib.picasso_pool_backward.argtypes = [vp, vp, ctypes.c_int, vp, i32, i32, vp, vp, vp, i32, vp, vp, vp]
    lib.picasso_unpool_forward.restype = ctypes.c_int
    lib.picasso_unpool_forward.argtypes = [vp, vp, vp, i32, i32, vp, vp]
    lib.picasso_unpool_backward.restype = ctypes.c_int
    lib.picasso_unpool_backward.argtypes = [vp, vp, vp, i32, i32, vp, vp, i32, vp]
    lib.picasso_bucket_sort.restype = ctypes.c_int
    lib.picasso_bucket_sort.argtypes = [vp, vp, ctypes.c_int, vp, vp, i64, ctypes.c_int]
    _lib = lib
    return lib


def _load_host():
    """The compiled module through which the calls of every step go (checks, output tensors, the library's call)."""
    global _host
    if _host is not None:
        return _host
    import torch
    try:
        from . import _host as h
    except ImportError as e:
        raise RuntimeError("the package's _host module is missing or does not load: build it with "
                           "`python -m paper_2103_15076_amd.build`") from e
    h.set_callbacks(torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, _raise_status)
    _host = h
    return h


def _raise_status(handle, st):
    msg = picasso_strerror(st)
    if st == PICASSO_ERR_HIP:
        msg += ": " + load_library().picasso_last_hip_error(ctypes.c_void_p(handle)).decode()
    raise PicassoError(st, msg)


def picasso_strerror(status: int) -> str:
    return load_library().picasso_strerror(int(status)).decode()


def picasso_workspace_bytes(max_verts: int, max_facets: int, max_meshes: int = 1) -> int:
    return int(load_library().picasso_workspace_bytes(int(max_verts), int(max_facets), int(max_meshes)))


def _stream_ptr(stream):
    import torch
    s = stream if stream is not None else torch.cuda.current_stream()
    return ctypes.c_void_p(s.cuda_stream)


def _dev_ptr(t, dtype, what):
    import torch
    if t is None:
        return ctypes.c_void_p(0)
    if not (isinstance(t, torch.Tensor) and t.is_cuda and t.dtype == dtype and t.is_contiguous()):
        raise TypeError(f"{what}: expected a contiguous CUDA tensor of dtype {dtype}")
    return ctypes.c_void_p(t.data_ptr())


def picasso_device_copy(dst, src, stream=None):
    """dst[:] = src with the library's plain copy kernel (both contiguous CUDA tensors of equal byte size)."""
    nbytes = src.numel() * src.element_size()
    assert dst.numel() * dst.element_size() == nbytes and dst.is_cuda and src.is_cuda
    st = load_library().picasso_device_copy(_stream_ptr(stream), ctypes.c_void_p(dst.data_ptr()),
                                            ctypes.c_void_p(src.data_ptr()), nbytes)
    if st != PICASSO_OK:
        raise PicassoError(st, picasso_strerror(st))


PICASSO_STATIC_MAX_CLUSTERS = 1 << 22


def picasso_replace_mapping_static(cluster_id, n_out, replace, mapping, status, device=0, stream=None):
    """picasso_replace_mapping for callers that cannot allocate: no context; every tensor, outputs
    (replace, mapping int32[n_in], status int32[1]) included, comes from the caller; asynchronous.
    Returns the call's own status (argument checks and launch errors); the bad-index verdict is left
    in ``status`` on the device."""
    import torch
    return int(load_library().picasso_replace_mapping_static(
        int(device), _stream_ptr(stream), _dev_ptr(cluster_id, torch.int32, "cluster_id"), int(cluster_id.shape[0]),
        int(n_out), _dev_ptr(replace, torch.int32, "replace"), _dev_ptr(mapping, torch.int32, "mapping"),
        _dev_ptr(status, torch.int32, "status")))


class Context:
    """Owns a picasso_ctx (device workspace sized at creation)."""

    def __init__(self, max_verts: int, max_facets: int, max_meshes: int = 1, device: int = 0):
        self._lib, self._n = load_library(), _load_host()
        self._h = ctypes.c_void_p(0)
        st = self._lib.picasso_create(ctypes.byref(self._h), int(device), int(max_verts), int(max_facets),
                                      int(max_meshes))
        if st != PICASSO_OK:
            raise PicassoError(st, picasso_strerror(st))
        self._p = self._h.value
        self.max_verts, self.max_facets, self.max_meshes, self.device = max_verts, max_facets, max_meshes, device

    def close(self):
        if getattr(self, "_h", None) and self._h.value:
            self._lib.picasso_destroy(self._h)
            self._h, self._p = ctypes.c_void_p(0), 0

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def __enter__(self):
        return self

    def __exit__(self, *a):
        self.close()

    def set_option(self, option: int, value: int):
        st = self._lib.picasso_set_option(self._h, int(option), int(value))
        if st != PICASSO_OK:
            raise PicassoError(st, picasso_strerror(st))

    def set_placement(self, placement: int, rcond_min: float = 1e-3):
        """PICASSO_OPT_PLACEMENT and its binary32 threshold (passed on as a bit pattern)."""
        import struct
        self.set_option(PICASSO_OPT_RCOND_MIN_BITS, struct.unpack("<I", struct.pack("<f", float(rcond_min)))[0])
        self.set_option(PICASSO_OPT_PLACEMENT, placement)

    def picasso_kernel_timing(self, kernel, reset=False):
        """Totals for one of the bracketed kernels (PICASSO_KERNEL_*) while PICASSO_OPT_KERNEL_TIMING is on."""
        n, ms, by = ctypes.c_int64(0), ctypes.c_double(0.0), ctypes.c_double(0.0)
        st = self._lib.picasso_kernel_timing(self._h, int(kernel), int(bool(reset)), ctypes.byref(n), ctypes.byref(ms),
                                             ctypes.byref(by))
        if st != PICASSO_OK:
            self._raise(st)
        return dict(kernel=TIMED_KERNEL_NAMES[int(kernel)], launches=n.value, ms_total=ms.value, bytes_total=by.value)

    def last_hip_error(self) -> str:
        return self._lib.picasso_last_hip_error(self._h).decode()

    def _raise(self, st):
        _raise_status(self._h.value, st)

    # -- the calls of include/picasso.h, same names ---------------------------------------------

    def picasso_decimate(self, verts, facets, target_nv, verts_out=None, facets_out=None, cluster_id=None,
                         stats=None, stream=None, check=True):
        """Returns (status, verts_out[:nv], facets_out[:nf], cluster_id).  Output
        tensors are allocated with torch when not supplied (capacity = input sizes)."""
        r = self._n.decimate(self._p, stream, verts, facets, target_nv, verts_out, facets_out, cluster_id,
                             ctypes.addressof(stats) if stats is not None else 0)
        if r[0] < 0 and check:
            self._raise(r[0])
        return r

    def picasso_decimate_batch(self, verts, facets, nv_in, nf_in, target_nv, verts_out=None, facets_out=None,
                               cluster_id=None, stats=None, stream=None, check=True):
        """nv_in / nf_in / target_nv: host int sequences [B].  Returns
        (status, verts_out[:sum nv], facets_out[:sum nf], cluster_id, nv_out[B], nf_out[B])."""
        import numpy as np
        nv_in = np.ascontiguousarray(nv_in, dtype=np.int32)
        nf_in = np.ascontiguousarray(nf_in, dtype=np.int32)
        target_nv = np.ascontiguousarray(target_nv, dtype=np.int32)
        nvo = np.zeros(nv_in.shape[0], np.int32)
        nfo = np.zeros(nv_in.shape[0], np.int32)
        r = self._n.decimate_batch(self._p, stream, verts, facets, nv_in, nf_in, target_nv, verts_out, facets_out,
                                   cluster_id, nvo, nfo, ctypes.addressof(stats) if stats is not None else 0)
        if r[0] < 0:
            if check:
                self._raise(r[0])
            return r + (None, None)
        return r + (nvo, nfo)

    def picasso_vertex_quadrics(self, verts, facets, stream=None):
        import torch
        N, F = int(verts.shape[0]), int(facets.shape[0])
        out = torch.empty((N, 10), dtype=torch.float32, device=verts.device)
        st = self._lib.picasso_vertex_quadrics(self._h, _stream_ptr(stream), _dev_ptr(verts, torch.float32, "verts"),
                                               N, _dev_ptr(facets, torch.int32, "facets"), F,
                                               _dev_ptr(out, torch.float32, "out"))
        if st != PICASSO_OK:
            self._raise(st)
        return out

    def picasso_edge_costs(self, verts, facets, stream=None):
        import torch
        N, F = int(verts.shape[0]), int(facets.shape[0])
        edges = torch.empty((max(3 * F, 1), 2), dtype=torch.int32, device=verts.device)
        cost = torch.empty((max(3 * F, 1),), dtype=torch.float32, device=verts.device)
        ne = ctypes.c_int32(0)
        st = self._lib.picasso_edge_costs(self._h, _stream_ptr(stream), _dev_ptr(verts, torch.float32, "verts"), N,
                                          _dev_ptr(facets, torch.int32, "facets"), F,
                                          _dev_ptr(edges, torch.int32, "edges"), _dev_ptr(cost, torch.float32, "cost"),
                                          ctypes.byref(ne))
        if st != PICASSO_OK:
            self._raise(st)
        return edges[: ne.value], cost[: ne.value]

    # -- pooling / unpooling over cluster_id ------------------------------------------------------

    def picasso_replace_mapping(self, cluster_id, n_out, stream=None):
        """Returns (replace int32[n_in], mapping int32[n_in]) device tensors."""
        import torch
        n_in = int(cluster_id.shape[0])
        rep = torch.empty((n_in,), dtype=torch.int32, device=cluster_id.device)
        mp = torch.empty((n_in,), dtype=torch.int32, device=cluster_id.device)
        st = self._lib.picasso_replace_mapping(self._h, _stream_ptr(stream),
                                               _dev_ptr(cluster_id, torch.int32, "cluster_id"), n_in, int(n_out),
                                               _dev_ptr(rep, torch.int32, "replace"), _dev_ptr(mp, torch.int32, "mapping"))
        if st != PICASSO_OK:
            self._raise(st)
        return rep, mp

    def picasso_cluster_csr(self, cluster_id, n_out, stream=None):
        """Returns (offsets int32[n_out+1], members int32[n_in]) device tensors."""
        return self._n.cluster_csr(self._p, stream, cluster_id, n_out)

    def picasso_pool_forward(self, mode, x, offsets, members, weight=None, want_argmax=None, stream=None):
        """Returns y[n_out, C]; for PICASSO_POOL_MAX returns (y, argmax)."""
        if want_argmax is None:
            want_argmax = mode == PICASSO_POOL_MAX
        return self._n.pool_forward(self._p, stream, mode, x, offsets, members, weight, bool(want_argmax))

    def picasso_pool_backward(self, mode, gy, cluster_id, offsets, members, weight=None, argmax=None, stream=None):
        return self._n.pool_backward(self._p, stream, mode, gy, cluster_id, offsets, members, weight, argmax)

    def picasso_unpool_forward(self, y, cluster_id, stream=None):
        return self._n.unpool_forward(self._p, stream, y, cluster_id)

    def picasso_unpool_backward(self, gx, offsets, members, stream=None):
        return self._n.unpool_backward(self._p, stream, gx, offsets, members)

    # ---- mesh convolutions, depth-wise (Sec. 4; supplementary, backward propagations)

    def picasso_vertex_corner_csr(self, facets, n_verts, stream=None):
        """Returns (offsets int32[N+1], corners int32[3F]) device tensors."""
        return self._n.vertex_corner_csr(self._p, stream, facets, n_verts)

    def picasso_facet_geometry(self, verts, facets, nf=None, alpha=1, beta=1, stream=None):
        """Returns (normals f32[F,3], areas f32[F], level int32[F]); nf = facets per mesh of a batch."""
        return self._n.facet_geometry(self._p, stream, verts, facets, nf, alpha, beta)

    def picasso_fuzzy_coefficients(self, normals, mu, inv_var, stream=None):
        return self._n.fuzzy_coefficients(self._p, stream, normals, mu, inv_var)

    def picasso_v2f_forward(self, x, facets, level, w, out=None, stream=None):
        return self._n.v2f_forward(self._p, stream, x, facets, level, w, out)

    def picasso_v2f_backward(self, gy, x, facets, level, w, offsets, corners, stream=None):
        """Returns (gx[N,C], gw[3,C])."""
        return self._n.v2f_backward(self._p, stream, gy, x, facets, level, w, offsets, corners)

    def picasso_f2f_forward(self, tex, bary, poff, w, stream=None):
        return self._n.f2f_forward(self._p, stream, tex, bary, poff, w)

    def picasso_f2f_backward(self, gy, tex, bary, poff, w, stream=None):
        """Returns (gtex[P,C], gw[3,C])."""
        return self._n.f2f_backward(self._p, stream, gy, tex, bary, poff, w)

    def picasso_f2v_forward(self, y, pi, w, offsets, corners, n_verts, out=None, stream=None):
        return self._n.f2v_forward(self._p, stream, y, pi, w, offsets, corners, n_verts, out)

    def picasso_f2v_backward(self, gx, y, pi, w, facets, offsets, want_gpi=True, stream=None):
        """Returns (gy[F,C], gw[T,C], gpi[F,T] or None)."""
        return self._n.f2v_backward(self._p, stream, gx, y, pi, w, facets, offsets, bool(want_gpi))

    def picasso_bucket_sort(self, keys, vals=None, key_bits=None, stream=None):
        """Same as picasso_radix_sort, by top-digit partition + per-bucket LDS sort (n <= 2^20)."""
        return self.picasso_radix_sort(keys, vals, key_bits, stream, _fn="picasso_bucket_sort")

    def picasso_radix_sort(self, keys, vals=None, key_bits=None, stream=None, _fn="picasso_radix_sort"):
        """In-place stable sort of a uint32-as-int32 / uint64-as-int64 tensor on its low key_bits bits."""
        import torch
        if keys.dtype == torch.int64:
            kb = 8
        elif keys.dtype == torch.int32:
            kb = 4
        else:
            raise TypeError("keys must be int32 or int64 (bit patterns of unsigned keys)")
        if key_bits is None:
            key_bits = 8 * kb
        st = getattr(self._lib, _fn)(self._h, _stream_ptr(stream), kb, _dev_ptr(keys, keys.dtype, "keys"),
                                          _dev_ptr(vals, torch.int32, "vals") if vals is not None else None,
                                          int(keys.shape[0]), int(key_bits))
        if st != PICASSO_OK:
            self._raise(st)
        return keys, vals
