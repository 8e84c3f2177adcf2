"""ctypes marshalling for the C ABI declared in include/fpsched.h."""
from __future__ import annotations

import ctypes
import os

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libfpsched.so")

FLAG_DEADLOCK = 1
FLAG_INCOMPLETE = 2
FLAG_OVER_CAP = 4
NKINDS = 8
ERR_OVERFLOW = -4      # the problem's time bound does not fit
ERR_UNSUPPORTED = -6   # no kernel takes this problem, cost model or setting


class FpschedError(RuntimeError):
    def __init__(self, code, what):
        super().__init__(f"{what}: {code} ({_strerror(code)})")
        self.code = code


class _Desc(ctypes.Structure):
    _fields_ = [
        ("n_devices", ctypes.c_int32), ("n_stages", ctypes.c_int32),
        ("n_microbatches", ctypes.c_int32), ("has_w", ctypes.c_int32),
        ("stage_device", ctypes.c_void_p), ("n_edges", ctypes.c_int32),
        ("edge_src", ctypes.c_void_p), ("edge_dst", ctypes.c_void_p), ("edge_comm", ctypes.c_void_p),
        ("dur", ctypes.c_void_p), ("mem_units", ctypes.c_void_p), ("mem_cap", ctypes.c_void_p),
    ]


class _Results(ctypes.Structure):
    _fields_ = [("makespan", ctypes.c_void_p), ("idle", ctypes.c_void_p),
                ("peak", ctypes.c_void_p), ("flags", ctypes.c_void_p)]


_lib = None


def library_path() -> str:
    return _LIB_PATH


def load_library():
    """dlopen libfpsched.so (built in-tree by paper_2510_05112_amd/build.py).  Fails loudly."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise FileNotFoundError(
                f"{_LIB_PATH} is missing: build it with `python -m paper_2510_05112_amd.build`")
        lib = ctypes.CDLL(_LIB_PATH)
        vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
        lib.fpsched_version.restype = ctypes.c_int
        lib.fpsched_strerror.restype = ctypes.c_char_p
        lib.fpsched_strerror.argtypes = [ctypes.c_int]
        lib.fpsched_problem_create.restype = ctypes.c_int
        lib.fpsched_problem_create.argtypes = [ctypes.POINTER(_Desc), ctypes.c_int, i32, ctypes.POINTER(vp)]
        lib.fpsched_problem_destroy.restype = None
        lib.fpsched_problem_destroy.argtypes = [vp]
        lib.fpsched_problem_info.restype = ctypes.c_int
        lib.fpsched_problem_info.argtypes = [vp, ctypes.POINTER(i32), ctypes.POINTER(i32), ctypes.POINTER(i32)]
        lib.fpsched_problem_set_microbatch_costs.restype = ctypes.c_int
        lib.fpsched_problem_set_microbatch_costs.argtypes = [vp, vp]
        lib.fpsched_problem_set_link_occupancy.restype = ctypes.c_int
        lib.fpsched_problem_set_link_occupancy.argtypes = [vp, i32]
        lib.fpsched_problem_set_sync.restype = ctypes.c_int
        lib.fpsched_problem_set_sync.argtypes = [vp, vp, i32, vp]
        lib.fpsched_problem_set_copy_engine.restype = ctypes.c_int
        lib.fpsched_problem_set_copy_engine.argtypes = [vp, i32]
        lib.fpsched_problem_active_kernel.restype = ctypes.c_int
        lib.fpsched_problem_active_kernel.argtypes = [vp]
        lib.fpsched_problem_select_kernel.restype = ctypes.c_int
        lib.fpsched_problem_select_kernel.argtypes = [vp, ctypes.c_int]
        lib.fpsched_workspace_bytes.restype = ctypes.c_size_t
        lib.fpsched_workspace_bytes.argtypes = [vp, i64, i32]
        lib.fpsched_evaluate.restype = ctypes.c_int
        lib.fpsched_evaluate.argtypes = [vp, vp, i64, i32, _Results, vp, ctypes.c_size_t, vp]
        lib.fpsched_topk.restype = ctypes.c_int
        lib.fpsched_topk.argtypes = [vp, _Results, i64, i32, vp, vp, vp, vp, ctypes.c_size_t, vp]
        lib.fpsched_static_scratch_bytes.restype = ctypes.c_size_t
        lib.fpsched_static_scratch_bytes.argtypes = []
        lib.fpsched_evaluate_topk_static.restype = ctypes.c_int
        lib.fpsched_evaluate_topk_static.argtypes = [vp, vp, i64, i32, _Results, i32, vp, vp, vp, vp]
        lib.fpsched_rank_workspace_bytes.restype = ctypes.c_size_t
        lib.fpsched_rank_workspace_bytes.argtypes = [vp, i64, i32]
        lib.fpsched_rank.restype = ctypes.c_int
        lib.fpsched_rank.argtypes = [vp, _Results, i64, i32, i32, i32, vp, vp, vp, vp, ctypes.c_size_t, vp]
        lib.fpsched_wslide_workspace_bytes.restype = ctypes.c_size_t
        lib.fpsched_wslide_workspace_bytes.argtypes = [vp, i64, i32]
        lib.fpsched_wslide.restype = ctypes.c_int
        lib.fpsched_wslide.argtypes = [vp, vp, i64, i32, vp, i32, _Results, vp, ctypes.c_size_t, vp]
        lib.fpsched_wslide_evaluate.restype = ctypes.c_int
        lib.fpsched_wslide_evaluate.argtypes = [vp, vp, i64, i32, _Results, vp, ctypes.c_size_t, vp]
        lib.fpsched_pareto_workspace_bytes.restype = ctypes.c_size_t
        lib.fpsched_pareto_workspace_bytes.argtypes = [vp, i64]
        lib.fpsched_pareto.restype = ctypes.c_int
        lib.fpsched_pareto.argtypes = [vp, _Results, i64, i32, vp, vp, vp, vp, vp, ctypes.c_size_t, vp]
        lib.fpsched_apply_caps.restype = ctypes.c_int
        lib.fpsched_apply_caps.argtypes = [vp, vp, vp, i32, i64, vp, vp]
        lib.fpsched_generate.restype = ctypes.c_int
        lib.fpsched_generate.argtypes = [vp, vp, vp, i64, i32, vp, vp, vp, vp, ctypes.c_size_t, vp]
        lib.fpsched_generate_selected.restype = ctypes.c_int
        lib.fpsched_generate_selected.argtypes = [vp, vp, vp, i64, vp, i64, i32, vp, vp, vp, vp, ctypes.c_size_t, vp]
        lib.fpsched_generate_evaluate.restype = ctypes.c_int
        lib.fpsched_generate_evaluate.argtypes = [vp, vp, vp, i64, _Results, vp, vp, vp, ctypes.c_size_t, vp]
        lib.fpsched_generate_slide_evaluate.restype = ctypes.c_int
        lib.fpsched_generate_slide_evaluate.argtypes = lib.fpsched_generate_evaluate.argtypes
        lib.fpsched_encode.restype = ctypes.c_int
        lib.fpsched_encode.argtypes = [vp, vp, i32, i32, vp]
        lib.fpsched_validate.restype = ctypes.c_int64
        lib.fpsched_validate.argtypes = [vp, vp, i64, i32]
        _lib = lib
    return _lib


def _strerror(code):
    try:
        return load_library().fpsched_strerror(int(code)).decode()
    except Exception:  # pragma: no cover
        return "?"


def version() -> int:
    return load_library().fpsched_version()


def _i32(a):
    return np.ascontiguousarray(np.asarray(a, dtype=np.int32))


class Problem:
    """Handle on one problem (``fpsched_problem``).

    ``desc`` is any object with the fields of ``fpsched_problem_desc``
    (n_devices, n_stages, n_microbatches, has_w, stage_device, edge_src,
    edge_dst, edge_comm, dur[8][S], mem_units, mem_cap).  ``device`` is a CUDA/HIP
    device index, or None for a host-only handle (encode / validate only).
    """

    def __init__(self, desc, max_stride: int, device: int | None = 0):
        lib = load_library()
        self.D, self.S, self.m = int(desc.n_devices), int(desc.n_stages), int(desc.n_microbatches)
        self._keep = [_i32(desc.stage_device), _i32(desc.edge_src), _i32(desc.edge_dst),
                      _i32(desc.edge_comm), _i32(desc.dur), _i32(desc.mem_units), _i32(desc.mem_cap)]
        k = self._keep
        if k[0].size != self.S or k[4].size != NKINDS * self.S or k[5].size != self.S or k[6].size != self.D:
            raise ValueError("table sizes do not match n_stages / n_devices")
        if not (k[1].size == k[2].size == k[3].size):
            raise ValueError("edge arrays differ in length")
        d = _Desc(self.D, self.S, self.m, int(desc.has_w), k[0].ctypes.data, int(k[1].size),
                  k[1].ctypes.data, k[2].ctypes.data, k[3].ctypes.data, k[4].ctypes.data,
                  k[5].ctypes.data, k[6].ctypes.data)
        self.device = device
        self.max_stride = int(max_stride)
        self._h = ctypes.c_void_p()
        rc = lib.fpsched_problem_create(ctypes.byref(d), -1 if device is None else int(device),
                                        self.max_stride, ctypes.byref(self._h))
        if rc != 0:
            self._h = None
            raise FpschedError(rc, "fpsched_problem_create")

    def close(self):
        if getattr(self, "_h", None):
            load_library().fpsched_problem_destroy(self._h)
            self._h = None

    def __del__(self):  # pragma: no cover
        try:
            self.close()
        except Exception:
            pass

    def info(self):
        a, b, c = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
        load_library().fpsched_problem_info(self._h, ctypes.byref(a), ctypes.byref(b), ctypes.byref(c))
        return dict(lanes_per_candidate=a.value, candidates_per_wave=b.value, lds_bytes_per_wave=c.value)

    def select_kernel(self, which: str):
        """'auto', 'general' or 'slots' (both kernels compute the same results)."""
        rc = load_library().fpsched_problem_select_kernel(self._h, {"auto": 0, "general": 1, "slots": 2}[which])
        if rc != 0:
            raise FpschedError(rc, "fpsched_problem_select_kernel")

    def active_kernel(self) -> str:
        """'slots' or 'general': the kernel ``evaluate`` launches under the present cost model."""
        rc = load_library().fpsched_problem_active_kernel(self._h)
        if rc < 0:
            raise FpschedError(rc, "fpsched_problem_active_kernel")
        return {1: "general", 2: "slots"}[rc]

    def set_microbatch_costs(self, dur_mb):
        """dur_mb[8][S][m] (host array): per-micro-batch costs that replace dur[kind][stage] in evaluate;
        None switches back (see fpsched_problem_set_microbatch_costs)."""
        ptr = None
        if dur_mb is not None:
            table = np.ascontiguousarray(np.asarray(dur_mb, dtype=np.int32))
            if table.shape != (NKINDS, self.S, self.m):
                raise ValueError(f"dur_mb must be [{NKINDS}][{self.S}][{self.m}], got {table.shape}")
            ptr = table.ctypes.data
        rc = load_library().fpsched_problem_set_microbatch_costs(self._h, ptr)
        if rc != 0:
            raise FpschedError(rc, "fpsched_problem_set_microbatch_costs")

    def set_link_occupancy(self, on: bool = True):
        """Every ordered pair of devices becomes a link that carries one value at a time
        (see fpsched_problem_set_link_occupancy)."""
        rc = load_library().fpsched_problem_set_link_occupancy(self._h, 1 if on else 0)
        if rc != 0:
            raise FpschedError(rc, "fpsched_problem_set_link_occupancy")

    def set_sync(self, group=None, pairs=None):
        """Synchronisation stages and dependency pairs (see fpsched_problem_set_sync): group[S]
        micro-batches per item of each stage (None = 1), pairs = rows (kind_from, stage_from, kind_to,
        stage_to, latency).  set_sync() switches back to the plain model."""
        grp = None if group is None else _i32(group)
        if grp is not None and grp.shape != (self.S,):
            raise ValueError(f"group must have {self.S} entries")
        prs = _i32(np.zeros((0, 5), np.int32) if pairs is None else pairs).reshape(-1, 5)
        rc = load_library().fpsched_problem_set_sync(self._h, None if grp is None else grp.ctypes.data, len(prs),
                                                     prs.ctypes.data if len(prs) else None)
        if rc != 0:
            raise FpschedError(rc, "fpsched_problem_set_sync")

    def set_copy_engine(self, depth: int = 4):
        """Offload and reload items run on a copy engine that holds at most ``depth`` transfers
        (see fpsched_problem_set_copy_engine); 0 switches back."""
        rc = load_library().fpsched_problem_set_copy_engine(self._h, int(depth))
        if rc != 0:
            raise FpschedError(rc, "fpsched_problem_set_copy_engine")

    # ---- host helpers -----------------------------------------------------
    def encode(self, items, device: int) -> np.ndarray:
        """items: [(kind, stage, micro-batch), ...] of one device's list -> uint16 words."""
        a = _i32(items).reshape(-1, 3)
        out = np.zeros(len(a), np.uint16)
        rc = load_library().fpsched_encode(self._h, a.ctypes.data, int(device), len(a), out.ctypes.data)
        if rc != 0:
            raise FpschedError(rc, "fpsched_encode")
        return out

    def validate(self, words: np.ndarray) -> int:
        w = np.ascontiguousarray(np.asarray(words, np.uint16))
        assert w.ndim == 3 and w.shape[1] == self.D
        rc = load_library().fpsched_validate(self._h, w.ctypes.data, w.shape[0], w.shape[2])
        if rc < 0:
            raise FpschedError(rc, "fpsched_validate")
        return int(rc)

    # ---- device calls (torch tensors in, torch tensors out) --------------------
    def workspace_bytes(self, n_cand: int, k: int) -> int:
        return int(load_library().fpsched_workspace_bytes(self._h, int(n_cand), int(k)))

    def alloc_results(self, n_cand: int):
        import torch
        dev = torch.device("cuda", self.device)
        return dict(makespan=torch.empty(n_cand, dtype=torch.int64, device=dev),
                    idle=torch.empty((n_cand, self.D), dtype=torch.int64, device=dev),
                    peak=torch.empty((n_cand, self.D), dtype=torch.int32, device=dev),
                    flags=torch.empty(n_cand, dtype=torch.uint8, device=dev))

    def alloc_workspace(self, n_cand: int, k: int):
        import torch
        return torch.empty(self.workspace_bytes(n_cand, k), dtype=torch.uint8,
                           device=torch.device("cuda", self.device))

    @staticmethod
    def _res_struct(res):
        return _Results(res["makespan"].data_ptr(), res["idle"].data_ptr(),
                        res["peak"].data_ptr(), res["flags"].data_ptr())

    def _stream(self, stream):
        import torch
        s = torch.cuda.current_stream(self.device) if stream is None else stream
        return ctypes.c_void_p(s.cuda_stream)

    def evaluate(self, ops, results=None, workspace=None, stream=None):
        """ops: torch int16/uint16 CUDA tensor [C][D][stride] (resident in HBM).  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_evaluate")
        assert ops.is_cuda and ops.is_contiguous() and ops.dim() == 3 and ops.shape[1] == self.D
        assert ops.element_size() == 2
        C, _, stride = ops.shape
        if results is None:
            results = self.alloc_results(C)
        if workspace is None:
            workspace = self.alloc_workspace(C, 0)
        ws_ptr, ws_bytes = workspace.data_ptr(), workspace.numel()
        rc = load_library().fpsched_evaluate(self._h, ops.data_ptr(), C, stride, self._res_struct(results),
                                             ws_ptr, ws_bytes, self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_evaluate")
        return results

    def topk(self, results, k: int, workspace=None, out=None, stream=None):
        """k best feasible candidates of evaluated ``results``.  Returns dict(idx, makespan, count)
        of CUDA tensors.  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_topk")
        C = results["makespan"].numel()
        dev = torch.device("cuda", self.device)
        if workspace is None:
            workspace = self.alloc_workspace(C, k)
        if out is None:
            out = dict(idx=torch.empty(k, dtype=torch.int64, device=dev),
                       makespan=torch.empty(k, dtype=torch.int64, device=dev),
                       count=torch.empty(1, dtype=torch.int32, device=dev))
        rc = load_library().fpsched_topk(self._h, self._res_struct(results), C, int(k),
                                         out["idx"].data_ptr(), out["makespan"].data_ptr(),
                                         out["count"].data_ptr(), workspace.data_ptr(),
                                         workspace.numel(), self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_topk")
        return out

    def evaluate_topk_static(self, ops, k: int, results, out, stream=None):
        """fpsched_evaluate_topk_static: evaluate + top-k with the library's static scratch memory instead
        of a workspace.  ``results`` (alloc_results) and ``out`` (dict idx, makespan, count) are the
        caller's; nothing is allocated here or in the library.  Asynchronous."""
        if self.device is None:
            raise FpschedError(-5, "fpsched_evaluate_topk_static")
        assert ops.is_cuda and ops.is_contiguous() and ops.dim() == 3 and ops.shape[1] == self.D
        assert ops.element_size() == 2
        C, _, stride = ops.shape
        rc = load_library().fpsched_evaluate_topk_static(
            self._h, ops.data_ptr(), C, stride, self._res_struct(results), int(k), out["idx"].data_ptr(),
            out["makespan"].data_ptr(), out["count"].data_ptr(), self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_evaluate_topk_static")
        return out

    def generate(self, policy, inflight, stride: int, out=None, workspace=None, stream=None):
        """Run the scheduler on n parameter sets.  policy: torch int32 CUDA tensor [n][D][8]
        (fpsched_actor_policy per actor), inflight: torch int32 CUDA tensor [n][S].  Returns
        dict(ops int16 [n][D][stride], steps int32 [n], status uint8 [n]) of CUDA tensors.
        Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_generate")
        assert policy.is_cuda and policy.is_contiguous() and policy.dtype == torch.int32
        assert inflight.is_cuda and inflight.is_contiguous() and inflight.dtype == torch.int32
        n = policy.shape[0]
        assert tuple(policy.shape) == (n, self.D, 8) and tuple(inflight.shape) == (n, self.S)
        dev = torch.device("cuda", self.device)
        if out is None:
            out = dict(ops=torch.empty((n, self.D, int(stride)), dtype=torch.int16, device=dev),
                       steps=torch.empty(n, dtype=torch.int32, device=dev),
                       status=torch.empty(n, dtype=torch.uint8, device=dev))
        if workspace is None:
            workspace = self.alloc_workspace(n, 0)
        rc = load_library().fpsched_generate(self._h, policy.data_ptr(), inflight.data_ptr(), n, int(stride),
                                             out["ops"].data_ptr(), out["steps"].data_ptr(),
                                             out["status"].data_ptr(), workspace.data_ptr(), workspace.numel(),
                                             self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_generate")
        return out

    def generate_selected(self, policy, inflight, select, stride: int, out=None, workspace=None, stream=None):
        """fpsched_generate_selected: the schedules of the parameter sets ``select`` names (torch int64
        CUDA tensor [k], e.g. the indices of a top-k; negative = none).  Returns dict(ops int16
        [k][D][stride], steps, status).  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_generate_selected")
        assert policy.is_cuda and policy.is_contiguous() and policy.dtype == torch.int32
        assert inflight.is_cuda and inflight.is_contiguous() and inflight.dtype == torch.int32
        assert select.is_cuda and select.is_contiguous() and select.dtype == torch.int64 and select.dim() == 1
        n = policy.shape[0]
        assert tuple(policy.shape) == (n, self.D, 8) and tuple(inflight.shape) == (n, self.S)
        k = select.numel()
        dev = torch.device("cuda", self.device)
        if out is None:
            out = dict(ops=torch.empty((k, self.D, int(stride)), dtype=torch.int16, device=dev),
                       steps=torch.empty(k, dtype=torch.int32, device=dev),
                       status=torch.empty(k, dtype=torch.uint8, device=dev))
        if workspace is None:
            workspace = self.alloc_workspace(k, 0)
        rc = load_library().fpsched_generate_selected(
            self._h, policy.data_ptr(), inflight.data_ptr(), n, select.data_ptr(), k, int(stride),
            out["ops"].data_ptr(), out["steps"].data_ptr(), out["status"].data_ptr(), workspace.data_ptr(),
            workspace.numel(), self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_generate_selected")
        return out

    def generate_evaluate(self, policy, inflight, results=None, out=None, workspace=None, stream=None, slide=False):
        """fpsched_generate_evaluate: the schedules of n parameter sets timed while they are generated;
        no op words are written.  slide: fpsched_generate_slide_evaluate, the same with the weight-gradient
        sliding pass in it.  Returns (results as alloc_results gives them, dict(steps, status)).
        Asynchronous."""
        import torch
        name = "fpsched_generate_slide_evaluate" if slide else "fpsched_generate_evaluate"
        if self.device is None:
            raise FpschedError(-5, name)
        assert policy.is_cuda and policy.is_contiguous() and policy.dtype == torch.int32
        assert inflight.is_cuda and inflight.is_contiguous() and inflight.dtype == torch.int32
        n = policy.shape[0]
        assert tuple(policy.shape) == (n, self.D, 8) and tuple(inflight.shape) == (n, self.S)
        dev = torch.device("cuda", self.device)
        if results is None:
            results = self.alloc_results(n)
        if out is None:
            out = dict(steps=torch.empty(n, dtype=torch.int32, device=dev),
                       status=torch.empty(n, dtype=torch.uint8, device=dev))
        if workspace is None:
            workspace = self.alloc_workspace(n, 0)
        rc = getattr(load_library(), name)(
            self._h, policy.data_ptr(), inflight.data_ptr(), n, self._res_struct(results),
            out["steps"].data_ptr(), out["status"].data_ptr(), workspace.data_ptr(), workspace.numel(),
            self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, name)
        return results, out

    RANK_MODES = {"makespan": 0, "makespan_peak": 1, "peak_makespan": 2, "idle": 3}

    def rank(self, results, k: int, mode: str = "makespan_peak", include_over_cap: bool = False, stream=None):
        """k best evaluated candidates by a two-part key (see fpsched_rank).  Returns dict(idx, key,
        count) of CUDA tensors.  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_rank")
        C = results["makespan"].numel()
        dev = torch.device("cuda", self.device)
        nbytes = int(load_library().fpsched_rank_workspace_bytes(self._h, C, int(k)))
        workspace = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        out = dict(idx=torch.empty(k, dtype=torch.int64, device=dev),
                   key=torch.empty(k, dtype=torch.int64, device=dev),
                   count=torch.empty(1, dtype=torch.int32, device=dev))
        rc = load_library().fpsched_rank(self._h, self._res_struct(results), C, int(k), self.RANK_MODES[mode],
                                         int(bool(include_over_cap)), out["idx"].data_ptr(), out["key"].data_ptr(),
                                         out["count"].data_ptr(), workspace.data_ptr(), workspace.numel(),
                                         self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_rank")
        return out

    def wslide(self, ops, stride_out: int | None = None, out=None, workspace=None, stream=None):
        """Slide the weight-gradient items of ``ops`` (int16/uint16 CUDA tensor [n][D][stride]) into idle
        time (see fpsched_wslide).  Returns dict(ops, makespan, idle, peak, flags) of the new lists.
        out / workspace: reuse earlier results / a uint8 CUDA tensor of at least
        fpsched_wslide_workspace_bytes.  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_wslide")
        assert ops.is_cuda and ops.is_contiguous() and ops.dim() == 3 and ops.shape[1] == self.D
        assert ops.dtype in (torch.int16, torch.uint16)
        n, _, stride = ops.shape
        stride_out = int(stride if stride_out is None else stride_out)
        dev = torch.device("cuda", self.device)
        if out is None:
            out = dict(ops=torch.empty((n, self.D, stride_out), dtype=ops.dtype, device=dev),
                       makespan=torch.empty(n, dtype=torch.int64, device=dev),
                       idle=torch.empty((n, self.D), dtype=torch.int64, device=dev),
                       peak=torch.empty((n, self.D), dtype=torch.int32, device=dev),
                       flags=torch.empty(n, dtype=torch.uint8, device=dev))
        nbytes = int(load_library().fpsched_wslide_workspace_bytes(self._h, n, int(stride)))
        if workspace is None:
            workspace = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=dev)
        rc = load_library().fpsched_wslide(self._h, ops.data_ptr(), n, int(stride), out["ops"].data_ptr(), stride_out,
                                           self._res_struct(out), workspace.data_ptr(), workspace.numel(),
                                           self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_wslide")
        return out

    def wslide_evaluate(self, ops, out=None, workspace=None, stream=None):
        """The evaluation of the lists ``wslide`` would write for ``ops``, without the lists (see
        fpsched_wslide_evaluate).  Returns dict(makespan, idle, peak, flags).  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_wslide_evaluate")
        assert ops.is_cuda and ops.is_contiguous() and ops.dim() == 3 and ops.shape[1] == self.D
        assert ops.dtype in (torch.int16, torch.uint16)
        n, _, stride = ops.shape
        dev = torch.device("cuda", self.device)
        if out is None:
            out = dict(makespan=torch.empty(n, dtype=torch.int64, device=dev),
                       idle=torch.empty((n, self.D), dtype=torch.int64, device=dev),
                       peak=torch.empty((n, self.D), dtype=torch.int32, device=dev),
                       flags=torch.empty(n, dtype=torch.uint8, device=dev))
        if workspace is None:
            workspace = torch.empty(256, dtype=torch.uint8, device=dev)
        rc = load_library().fpsched_wslide_evaluate(self._h, ops.data_ptr(), n, int(stride), self._res_struct(out),
                                                    workspace.data_ptr(), workspace.numel(), self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_wslide_evaluate")
        return out

    def pareto(self, results, kmax: int, stream=None):
        """Pareto front of (makespan, largest peak) over the completed candidates (see fpsched_pareto).
        Returns dict(idx, makespan, peak, count) of CUDA tensors.  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_pareto")
        C = results["makespan"].numel()
        dev = torch.device("cuda", self.device)
        nbytes = int(load_library().fpsched_pareto_workspace_bytes(self._h, C))
        workspace = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=dev)
        out = dict(idx=torch.empty(kmax, dtype=torch.int64, device=dev),
                   makespan=torch.empty(kmax, dtype=torch.int64, device=dev),
                   peak=torch.empty(kmax, dtype=torch.int32, device=dev),
                   count=torch.empty(1, dtype=torch.int32, device=dev))
        rc = load_library().fpsched_pareto(self._h, self._res_struct(results), C, int(kmax), out["idx"].data_ptr(),
                                           out["makespan"].data_ptr(), out["peak"].data_ptr(),
                                           out["count"].data_ptr(), workspace.data_ptr(), workspace.numel(),
                                           self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_pareto")
        return out

    def apply_caps(self, results, caps, stream=None):
        """Rewrite the OVER_CAP bit of results["flags"] in place for other caps: an int32 CUDA tensor
        [D] (one cap per device) or [n][D] (caps per candidate).  Asynchronous."""
        import torch
        if self.device is None:
            raise FpschedError(-5, "fpsched_apply_caps")
        C = results["flags"].numel()
        per = caps.dim() == 2
        if caps.dtype != torch.int32 or not caps.is_cuda or not caps.is_contiguous() or \
                tuple(caps.shape) != ((C, self.D) if per else (self.D,)):
            raise ValueError("caps: contiguous int32 CUDA tensor [D] or [n][D]")
        rc = load_library().fpsched_apply_caps(self._h, results["peak"].data_ptr(), caps.data_ptr(), int(per), C,
                                               results["flags"].data_ptr(), self._stream(stream))
        if rc != 0:
            raise FpschedError(rc, "fpsched_apply_caps")
        return results
