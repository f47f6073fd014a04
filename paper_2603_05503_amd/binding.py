"""ctypes marshalling for include/calibatt.h."""
from __future__ import annotations

import ctypes as C
import functools
import os
import threading
from dataclasses import dataclass
from typing import Optional

import numpy as np

_PKG_DIR = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_PKG_DIR, "libcalibatt.so")
_lib = None


class CalibattError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {strerror(status)} (status {status})")


class _CStrides(C.Structure):
    _fields_ = [("b", C.c_int64), ("h", C.c_int64), ("n", C.c_int64)]


class _CFwdOptions(C.Structure):
    _fields_ = [("in_strides", C.POINTER(_CStrides)), ("out_strides", C.POINTER(_CStrides)),
                ("dtype", C.c_int32), ("lse", C.c_void_p), ("kernel", C.c_int32)]


KERNEL_AUTO, KERNEL_TWO_WORKGROUPS, KERNEL_INTERLEAVED = 0, 1, 2
ENERGY_ONE_BLOCK, ENERGY_TWO_BLOCKS, ENERGY_OVERLAPPED = 0, 1, 2  # forms of the one-pass block energies


class _CPattern(C.Structure):
    _fields_ = [
        ("H", C.c_int32), ("N", C.c_int32), ("block_q", C.c_int32), ("block_k", C.c_int32),
        ("nbq", C.c_int32), ("nbk", C.c_int32),
        ("n_work", C.c_int32), ("n_repeat", C.c_int32),
        ("order", C.c_int32), ("max_row", C.c_int32),
        ("nnz", C.c_int64),
        ("row_ptr", C.c_void_p), ("col_idx", C.c_void_p), ("repeat_src", C.c_void_p),
        ("work", C.c_void_p), ("fan_ptr", C.c_void_p), ("fan_dst", C.c_void_p),
        ("work_counter", C.c_void_p),
        ("n_groups", C.c_int32),
        ("group_ptr", C.c_int32 * 9),
        ("iv_ptr", C.c_void_p), ("iv", C.c_void_p),
        ("head_map", C.c_void_p),
    ]


class _CSplit(C.Structure):
    _fields_ = [("B", C.c_int32), ("n_parts", C.c_int32), ("n_rows", C.c_int32), ("n_slots", C.c_int32),
                ("parts", C.c_void_p), ("arrivals", C.c_void_p)]


def library_path() -> str:
    return _LIB_PATH


def load_library():
    """Load libcalibatt.so (built by ``python -m paper_2603_05503_amd.build``)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise RuntimeError(
            f"{_LIB_PATH} is missing: build it with `python -m paper_2603_05503_amd.build` "
            "(there is no fallback path)"
        )
    # Device pointers and streams handed to the library come from torch, so both must sit on ONE HIP
    # runtime.  torch ships its own copy; loading torch first makes the dynamic linker resolve the
    # library's libamdhip64 dependency to that already loaded copy instead of a second runtime
    # (which would not see torch's device context).
    import torch  # noqa: F401

    lib = C.CDLL(_LIB_PATH)
    i32p, u8p, i64p = C.POINTER(C.c_int32), C.POINTER(C.c_uint8), C.POINTER(C.c_int64)
    lib.calibatt_pattern_sizes.restype = C.c_int
    lib.calibatt_pattern_sizes.argtypes = [u8p, i32p, C.c_int, C.c_int, C.c_int, C.c_int, i64p, i32p, i32p]
    lib.calibatt_compile_pattern.restype = C.c_int
    lib.calibatt_compile_pattern.argtypes = [
        u8p, i32p, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int,
        i32p, i32p, C.c_int64, i32p, i32p, i32p, i32p, C.POINTER(_CPattern),
    ]
    lib.calibatt_sparse_attn_fwd.restype = C.c_int
    lib.calibatt_sparse_attn_fwd.argtypes = [
        C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
        C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int,
        C.POINTER(_CPattern), C.c_float, C.c_void_p,
    ]
    lib.calibatt_anchor_map.restype = C.c_int
    lib.calibatt_anchor_map.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, i32p, i32p, i32p, i32p]
    lib.calibatt_anchor_attn_fwd.restype = C.c_int
    lib.calibatt_anchor_attn_fwd.argtypes = [
        C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
        C.c_int, C.c_int, C.c_int, C.c_int,
        C.c_void_p, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int,
        C.c_float, C.c_void_p,
    ]
    lib.calibatt_block_energy.restype = C.c_int
    lib.calibatt_block_energy.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int,
                                          C.c_int, C.c_int, C.c_float, C.c_void_p]
    lib.calibatt_select_blocks.restype = C.c_int
    lib.calibatt_select_blocks.argtypes = [C.POINTER(C.c_float), C.c_int64, C.c_int, C.c_double, u8p]
    lib.calibatt_vote_masks.restype = C.c_int
    lib.calibatt_vote_masks.argtypes = [u8p, C.c_int, C.c_int64, C.c_double, u8p]
    u16p = C.POINTER(C.c_uint16)
    lib.calibatt_vote_accumulate.restype = C.c_int
    lib.calibatt_vote_accumulate.argtypes = [u8p, C.c_int64, u16p]
    lib.calibatt_vote_finish.restype = C.c_int
    lib.calibatt_vote_finish.argtypes = [u16p, C.c_int, C.c_int64, C.c_double, u8p]
    lib.calibatt_epsilon_schedule.restype = C.c_double
    lib.calibatt_epsilon_schedule.argtypes = [C.c_int, C.c_int, C.c_double, C.c_double, C.c_double]
    lib.calibatt_schedule_base_level.restype = C.c_double
    lib.calibatt_schedule_base_level.argtypes = [C.c_int]
    u32p = C.POINTER(C.c_uint32)
    lib.calibatt_encode_intervals.restype = C.c_int
    lib.calibatt_encode_intervals.argtypes = [i32p, i32p, C.c_int64, i32p, u32p, C.c_int64, i64p]
    lib.calibatt_merge_intervals.restype = C.c_int
    lib.calibatt_merge_intervals.argtypes = [u8p, C.c_int64, C.c_int, C.c_double, u8p, i32p]
    lib.calibatt_share_timesteps.restype = C.c_int
    lib.calibatt_share_timesteps.argtypes = [u8p, C.c_int, C.c_int64, C.c_double, i32p, u8p, i32p]
    lib.calibatt_sparse_attn_fwd_strided.restype = C.c_int
    lib.calibatt_sparse_attn_fwd_strided.argtypes = [
        C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
        C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int,
        C.POINTER(_CPattern), C.c_float, C.POINTER(_CStrides), C.POINTER(_CStrides), C.c_void_p,
    ]
    lib.calibatt_schedule_constants.restype = C.c_int
    lib.calibatt_schedule_constants.argtypes = [C.c_int, C.c_int, C.POINTER(C.c_double), C.POINTER(C.c_double),
                                                C.POINTER(C.c_double)]
    lib.calibatt_flag_heads.restype = C.c_int
    lib.calibatt_flag_heads.argtypes = [C.POINTER(C.c_float), C.c_int, C.c_int, C.c_double, C.POINTER(C.c_uint8),
                                        C.POINTER(C.c_double)]
    lib.calibatt_anchor_partner.restype = C.c_int
    lib.calibatt_anchor_partner.argtypes = [C.c_int, C.c_int, C.c_int, C.c_int, i32p]
    lib.calibatt_spatial_similarity.restype = C.c_int
    lib.calibatt_spatial_similarity.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int,
                                                C.c_void_p, C.c_int, C.c_int, C.c_float, C.c_void_p, C.c_void_p,
                                                C.c_void_p]
    lib.calibatt_similarity_lists_bytes.restype = C.c_int
    lib.calibatt_similarity_lists_bytes.argtypes = [C.c_int, C.c_int, C.c_int, C.POINTER(C.c_int64)]
    lib.calibatt_spatial_similarity_grouped.restype = C.c_int
    lib.calibatt_spatial_similarity_grouped.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int,
                                                        C.c_void_p, C.c_int, C.c_int, C.c_float, C.c_void_p,
                                                        C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p]
    lib.calibatt_spatial_similarity_static.restype = C.c_int
    lib.calibatt_spatial_similarity_static.argtypes = [C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int,
                                                       C.c_void_p, C.c_int, C.c_int, C.c_float, C.c_void_p, C.c_void_p]
    lib.calibatt_sparse_attn_fwd_ex.restype = C.c_int
    lib.calibatt_sparse_attn_fwd_ex.argtypes = [
        C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p,
        C.c_int, C.c_int, C.c_int, C.c_int, C.c_int, C.c_int,
        C.POINTER(_CPattern), C.c_float, C.POINTER(_CFwdOptions), C.c_void_p,
    ]
    lib.calibatt_plan_split.restype = C.c_int
    lib.calibatt_plan_split.argtypes = [C.POINTER(_CPattern), C.c_int, C.c_int, i32p, C.c_int64, C.POINTER(_CSplit)]
    lib.calibatt_split_workspace_bytes.restype = C.c_int64
    lib.calibatt_split_workspace_bytes.argtypes = [C.POINTER(_CSplit), C.c_int, C.c_int]
    lib.calibatt_sparse_attn_fwd_split.restype = C.c_int
    lib.calibatt_sparse_attn_fwd_split.argtypes = lib.calibatt_sparse_attn_fwd_ex.argtypes[:-1] + [
        C.POINTER(_CSplit), C.c_void_p, C.c_int64, C.c_void_p]
    lib.calibatt_anchor_attn_fwd_strided.restype = C.c_int
    lib.calibatt_anchor_attn_fwd_strided.argtypes = lib.calibatt_anchor_attn_fwd.argtypes[:-1] + [
        C.POINTER(_CStrides), C.POINTER(_CStrides), C.c_void_p]
    lib.calibatt_anchor_attn_fwd_split.restype = C.c_int
    lib.calibatt_anchor_attn_fwd_split.argtypes = lib.calibatt_anchor_attn_fwd_strided.argtypes[:-1] + [
        C.c_void_p, C.c_int64, C.c_void_p]
    lib.calibatt_anchor_split_plan.restype = C.c_int
    lib.calibatt_anchor_split_plan.argtypes = [C.c_int] * 5 + [C.POINTER(C.c_int32), C.POINTER(C.c_int64)]
    lib.calibatt_block_energy_workspace_bytes.restype = C.c_int
    lib.calibatt_block_energy_workspace_bytes.argtypes = [C.c_int, C.c_int, C.c_int, C.POINTER(C.c_int64)]
    lib.calibatt_block_energy_onepass_form.restype = C.c_int
    lib.calibatt_block_energy_onepass_form.argtypes = [C.c_int] * 6 + [C.c_int64, C.POINTER(C.c_int32)]
    lib.calibatt_block_energy_onepass.restype = C.c_int
    lib.calibatt_block_energy_onepass.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p] + [C.c_int] * 6 + [
        C.c_float, C.c_void_p, C.c_int64, C.c_void_p]
    lib.calibatt_select_blocks_device.restype = C.c_int
    lib.calibatt_select_blocks_device.argtypes = [C.c_void_p, C.c_int64, C.c_int, C.c_double, C.c_void_p, C.c_void_p]
    lib.calibatt_vote_accumulate_device.restype = C.c_int
    lib.calibatt_vote_accumulate_device.argtypes = [C.c_void_p, C.c_int64, C.c_void_p, C.c_void_p]
    lib.calibatt_strerror.restype = C.c_char_p
    lib.calibatt_strerror.argtypes = [C.c_int]
    lib.calibatt_version.restype = C.c_int
    lib.calibatt_version.argtypes = []
    _lib = lib
    return lib


def strerror(status: int) -> str:
    return load_library().calibatt_strerror(int(status)).decode()


def version() -> int:
    return int(load_library().calibatt_version())


def _as_mask(mask, H, nbq, nbk):
    m = np.ascontiguousarray(mask, dtype=np.uint8)
    if m.size != H * nbq * nbk:
        raise ValueError(f"mask has {m.size} entries, expected {H}x{nbq}x{nbk}")
    return m


def _as_repeat(repeat, H, nbq):
    if repeat is None:
        return None
    r = np.ascontiguousarray(repeat, dtype=np.int32)
    if r.size != H * nbq:
        raise ValueError(f"repeat has {r.size} entries, expected {H}x{nbq}")
    return r


def _ptr(a, ctype):
    return None if a is None else a.ctypes.data_as(C.POINTER(ctype))


def pattern_sizes(mask, repeat, H, N, block_q, block_k):
    """(nnz, n_work, n_repeat) via calibatt_pattern_sizes."""
    lib = load_library()
    nbq, nbk = -(-N // block_q), -(-N // block_k)
    m, r = _as_mask(mask, H, nbq, nbk), _as_repeat(repeat, H, nbq)
    nnz, nw, nr = C.c_int64(0), C.c_int32(0), C.c_int32(0)
    st = lib.calibatt_pattern_sizes(_ptr(m, C.c_uint8), _ptr(r, C.c_int32), H, N, block_q, block_k,
                                    C.byref(nnz), C.byref(nw), C.byref(nr))
    if st != 0:
        raise CalibattError(st, "calibatt_pattern_sizes")
    return int(nnz.value), int(nw.value), int(nr.value)


@dataclass
class HostPattern:
    """Output of calibatt_compile_pattern in host (NumPy) buffers."""
    H: int
    N: int
    block_q: int
    block_k: int
    nbq: int
    nbk: int
    n_work: int
    n_repeat: int
    order: int
    max_row: int
    nnz: int
    row_ptr: np.ndarray
    col_idx: np.ndarray
    repeat_src: np.ndarray
    work: np.ndarray
    fan_ptr: np.ndarray
    fan_dst: np.ndarray
    n_groups: int = 1
    group_ptr: Optional[np.ndarray] = None

    def to_device(self, device="cuda", persistent=True, intervals=False, head_map=None) -> "DevicePattern":
        """``intervals=True`` uploads the interval form of the kept-block lists instead of col_idx;
        ``head_map`` (one tensor head per pattern head) makes the pattern act on a subset of heads."""
        return DevicePattern(self, device, persistent, intervals, head_map)

    def plan_split(self, B: int, max_blocks: int = 0, iv_ptr=None):
        """calibatt_plan_split for batch ``B``: (struct without device pointers, int32 records [n_parts, 12]), or None
        where whole rows are the better choice.  ``max_blocks``: longest part in key blocks, 0 = the library's choice."""
        lib = load_library()
        c = _CPattern()
        for f in ("H", "N", "block_q", "block_k", "nbq", "nbk", "n_work", "n_repeat", "order", "max_row", "nnz"):
            setattr(c, f, getattr(self, f))
        # the library reads packed int32; `lists` keeps what is copied for that
        lists = [np.ascontiguousarray(a, np.int32) for a in (self.row_ptr, self.work, self.fan_ptr, self.col_idx)]
        c.row_ptr, c.work, c.fan_ptr, c.col_idx = (a.ctypes.data for a in lists)
        if iv_ptr is not None:
            iv_ptr = np.ascontiguousarray(iv_ptr, np.int32)
            c.iv_ptr = iv_ptr.ctypes.data
        split = _CSplit()
        cap = 2 * (self.n_work * B + 1024)  # more than most plans have
        while True:
            parts = np.empty((cap, 12), np.int32)
            st = lib.calibatt_plan_split(C.byref(c), B, max_blocks, _ptr(parts, C.c_int32), cap, C.byref(split))
            if st != -7 or cap >= split.n_parts:
                break
            cap = split.n_parts
        if st != 0:
            raise CalibattError(st, "calibatt_plan_split")
        parts = parts[:split.n_parts]
        return (split, parts) if split.n_parts else None

    def encode_intervals(self):
        """(iv_ptr int32 [rows + 1], iv uint32 words) via calibatt_encode_intervals."""
        return encode_intervals(self.row_ptr, self.col_idx)


def compile_pattern(mask, repeat, H, N, block_q, block_k, order=4) -> HostPattern:
    lib = load_library()
    if min(H, N, block_q, block_k) <= 0:
        raise CalibattError(-2, "calibatt_compile_pattern")
    nbq, nbk = -(-N // block_q), -(-N // block_k)
    m, r = _as_mask(mask, H, nbq, nbk), _as_repeat(repeat, H, nbq)
    nnz, _, _ = pattern_sizes(m, r, H, N, block_q, block_k)
    rows = H * nbq
    row_ptr = np.empty(rows + 1, np.int32)
    col_idx = np.empty(max(nnz, 1), np.int32)
    repeat_src = np.empty(rows, np.int32)
    work = np.empty(rows, np.int32)
    fan_ptr = np.empty(rows + 1, np.int32)
    fan_dst = np.empty(rows, np.int32)
    cp = _CPattern()
    st = lib.calibatt_compile_pattern(
        _ptr(m, C.c_uint8), _ptr(r, C.c_int32), H, N, block_q, block_k, order,
        _ptr(row_ptr, C.c_int32), _ptr(col_idx, C.c_int32), nnz, _ptr(repeat_src, C.c_int32),
        _ptr(work, C.c_int32), _ptr(fan_ptr, C.c_int32), _ptr(fan_dst, C.c_int32), C.byref(cp))
    if st != 0:
        raise CalibattError(st, "calibatt_compile_pattern")
    return HostPattern(
        H=cp.H, N=cp.N, block_q=cp.block_q, block_k=cp.block_k, nbq=cp.nbq, nbk=cp.nbk,
        n_work=cp.n_work, n_repeat=cp.n_repeat, order=cp.order, max_row=cp.max_row, nnz=cp.nnz,
        row_ptr=row_ptr, col_idx=col_idx[:nnz], repeat_src=repeat_src,
        work=work[: cp.n_work], fan_ptr=fan_ptr[: cp.n_work + 1], fan_dst=fan_dst[: cp.n_repeat],
        n_groups=cp.n_groups, group_ptr=np.array(list(cp.group_ptr), dtype=np.int32),
    )


class _StreamState:
    """What the calls of one stream use of a pattern."""

    def __init__(self, c, words, splits):
        self.c, self.c_ref, self.words, self.splits = c, C.byref(c), words, splits
        self.stream = None  # as a torch stream, for calls while another one is current


def _upload(arrays, device):
    """{name: int32 tensor on ``device``} of host integer arrays; an empty one becomes one zero.  A copy takes 8 us however
    little it moves, so small arrays go together, each at a cache line of its own; from 64 KB on an array goes by itself."""
    import torch

    out, small, n = {}, [], 0
    for name, a in arrays.items():
        if a.size > 1 << 14:
            out[name] = torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(device)
        else:
            small.append((name, a, n))
            n += -(-max(a.size, 1) // 32) * 32
    flat = np.zeros(n, np.int32)
    for _, a, at in small:
        flat[at:at + a.size] = a.reshape(-1)
    dev = torch.from_numpy(flat).to(device)
    for name, a, at in small:
        out[name] = dev[at:at + max(a.size, 1)].view(a.shape if a.size else (1,))
    return out


class DevicePattern:
    """The six index arrays as int32 torch tensors on the GPU plus the C struct
    that points at them."""

    _NAMES = ("row_ptr", "col_idx", "repeat_src", "work", "fan_ptr", "fan_dst")

    def __init__(self, hp: HostPattern, device="cuda", persistent=True, intervals=False, head_map=None):
        self.host = hp
        self.device = device
        self.intervals = bool(intervals)
        self._iv_ptr = None
        lists = {name: getattr(hp, name) for name in self._NAMES if not (intervals and name == "col_idx")}
        if intervals:
            self._iv_ptr, iv = hp.encode_intervals()
            lists["iv_ptr"], lists["iv"] = self._iv_ptr, iv.view(np.int32)
        if head_map is not None:
            lists["head_map"] = np.asarray(head_map).reshape(-1)
            if lists["head_map"].size != hp.H:
                raise ValueError(f"head_map has {lists['head_map'].size} entries, the pattern has {hp.H} heads")
        c = _CPattern()
        for f in ("H", "N", "block_q", "block_k", "nbq", "nbk", "n_work", "n_repeat", "order", "max_row", "nnz"):
            setattr(c, f, getattr(hp, f))
        c.n_groups = hp.n_groups
        gp = hp.group_ptr if hp.group_ptr is not None else np.array([0] + [hp.n_work] * 8, np.int32)
        for i in range(9):
            c.group_ptr[i] = int(gp[i])
        self.c = c
        self.tensors = self._plan(persistent, lists=lists)
        for name in (*self._NAMES, "iv_ptr", "iv", "head_map"):
            setattr(c, name, self.tensors[name].data_ptr() if name in self.tensors else None)

    def _plan(self, persistent, max_blocks=0, lists=None):
        """Plans of the calls cut along the keys (batches of one and, for two guidance branches, two), and the counters:
        per stream an int32[16] workspace of the persistent-workgroup scheduler and the arrivals of the cut rows' parts,
        both kept zero between calls, here for eight streams.  All of it goes to the GPU together with ``lists`` and is there
        when the call returns; the tensors of the lists are returned.  ``max_blocks``: as of ``plan_split``, None = no plans,
        every call takes whole rows."""
        host, plans = dict(lists or {}), {}
        if persistent:
            for B in (1, 2) if max_blocks is not None else ():
                plan = self.host.plan_split(B, max_blocks, self._iv_ptr)
                if plan:
                    plans[B], host[B] = plan
            # the arrivals behind the scheduler's words, whole cache lines for every stream
            arrivals = max((p.n_rows for p in plans.values()), default=0)
            self._words = 32 + -(-arrivals // 32) * 32
            host["words"] = np.zeros((8, self._words), np.int32)
        tensors = _upload(host, self.device)
        self._plans = {B: (plan, tensors.pop(B)) for B, plan in plans.items()}
        self._spare = list(tensors.pop("words")) if persistent else []
        words = self._spare.pop(0) if persistent else None
        self.counter = words[:16] if persistent else None
        self.c.work_counter = self.counter.data_ptr() if persistent else None
        self._stream_of_c = None  # stream handle that uses self.c
        self._own = _StreamState(self.c, words, self._splits_with(words))
        self._per_stream = {}     # other streams: clone of the struct, its own words, splits with its own arrivals
        self._lock = threading.Lock()
        return tensors

    def _splits_with(self, words):
        """{B: struct of the planned split whose arrivals are counted behind the scheduler's ``words``}"""
        out = {}
        for B, (plan, parts) in self._plans.items():
            out[B] = _CSplit(plan.B, plan.n_parts, plan.n_rows, plan.n_slots, parts.data_ptr(), words.data_ptr() + 32 * 4)
        return out

    def _for_stream(self, stream_handle: int):
        if self.counter is None or self._stream_of_c == stream_handle:
            return self._own
        with self._lock:
            if self._stream_of_c is None:
                self._stream_of_c = stream_handle
            if self._stream_of_c == stream_handle:
                return self._own
            if stream_handle not in self._per_stream:
                import torch

                clone = _CPattern()
                C.memmove(C.byref(clone), C.byref(self.c), C.sizeof(_CPattern))
                if self._spare:
                    words = self._spare.pop()
                else:  # cleared on the stream that uses it: nothing orders a fill on another one before the call
                    with torch.cuda.stream(_torch_stream(stream_handle, self.counter.device)):
                        words = torch.zeros(self._words, dtype=torch.int32, device=self.counter.device)
                clone.work_counter = words.data_ptr()
                self._per_stream[stream_handle] = _StreamState(clone, words, self._splits_with(words))
            return self._per_stream[stream_handle]

    def c_for(self, stream_handle: int):
        """The C struct to pass for a call on ``stream_handle``.  Calls on different streams may overlap on
        the GPU, and overlapping calls must not share the scheduler's work counters: every stream after the
        first gets a clone of the struct that points at counters of its own (the index arrays are shared)."""
        return self._for_stream(stream_handle).c

    @property
    def nnz(self) -> int:
        return self.host.nnz

    @property
    def index_bytes(self) -> int:
        """Bytes of the kept-block lists on the GPU (col_idx, or iv_ptr + iv in the interval form), without ``plan_bytes``."""
        names = ("iv_ptr", "iv") if self.intervals else ("col_idx",)
        return sum(self.tensors[n].numel() * 4 for n in names)

    @property
    def plan_bytes(self) -> int:
        """Bytes on the GPU that calls cut along the keys need beside the lists: the records of the plans, and the arrivals
        of the streams so far."""
        if self.counter is None:
            return 0
        streams = 1 + len(self._spare) + len(self._per_stream)
        return sum(parts.numel() * 4 for _, parts in self._plans.values()) + streams * (self._words - 32) * 4


def sparse_attn_fwd(q, k, v, out, pattern: DevicePattern, scale: float,
                    block_q: Optional[int] = None, block_k: Optional[int] = None, stream=None, lse=None,
                    kernel: int = KERNEL_AUTO):
    """The sparse forward on torch CUDA tensors of logical shape [B, H, N, D], bf16 or fp16 (all four
    alike).  The tensors may be strided views (e.g. ``x.transpose(1, 2)`` of a [B, N, H, D] tensor, or
    slices of a fused [B, N, 3, H, D] projection) as long as D is contiguous and q, k, v share their
    strides.  ``lse``: optional contiguous fp32 CUDA tensor [B, H, N] that receives the log-sum-exp of
    every query's kept logits.  ``kernel``: KERNEL_AUTO, KERNEL_TWO_WORKGROUPS or KERNEL_INTERLEAVED (the
    ``kernel`` field of calibatt_fwd_options).  Calls that the pattern has a split for (``DevicePattern``)
    go through calibatt_sparse_attn_fwd_split (with whole rows where its workspace cannot be had), other packed bf16 calls without ``lse`` and with the automatic
    kernel choice through calibatt_sparse_attn_fwd, everything else through calibatt_sparse_attn_fwd_ex."""
    import torch

    lib = load_library()
    shape, dtype, strides, out_strides = q.shape, q.dtype, q.stride(), out.stride()
    if not (len(shape) == 4 and dtype in (torch.bfloat16, torch.float16) and strides[3] == 1 and len(out_strides) == 4
            and out_strides[3] == 1 and q.is_cuda and k.is_cuda and v.is_cuda and out.is_cuda
            and k.dtype == dtype and v.dtype == dtype and out.dtype == dtype
            and k.shape == shape and v.shape == shape and out.shape == shape
            and k.stride() == strides and v.stride() == strides):
        for t in (q, k, v, out):
            if not (t.is_cuda and t.dtype in (torch.bfloat16, torch.float16) and t.dim() == 4 and t.stride(3) == 1):
                raise ValueError("q, k, v, out must be bf16 or fp16 CUDA tensors [B, H, N, D] with contiguous D")
            if t.shape != q.shape or t.dtype != q.dtype:
                raise ValueError("q, k, v, out must have the same shape and element type")
        raise ValueError("q, k, v must share their strides")
    B, H, N, D = shape
    if lse is not None and not (lse.is_cuda and lse.dtype == torch.float32 and lse.is_contiguous()
                                and tuple(lse.shape) == (B, H, N)):
        raise ValueError("lse must be a contiguous fp32 CUDA tensor [B, H, N]")
    bq = pattern.host.block_q if block_q is None else block_q
    bk = pattern.host.block_k if block_k is None else block_k
    current = _current_handle(q.device)
    stream = current if stream is None else int(stream)
    state = pattern._for_stream(stream)
    split = state.splits.get(B) if kernel != KERNEL_TWO_WORKGROUPS and bq == pattern.host.block_q else None
    packed = q.is_contiguous() and out.is_contiguous()
    args = (q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), B, H, N, D, bq, bk, state.c_ref, float(scale))
    if split is None and packed and lse is None and dtype == torch.bfloat16 and kernel == KERNEL_AUTO:
        st = lib.calibatt_sparse_attn_fwd(*args, stream)
    else:
        si, so = _CStrides(*strides[:3]), _CStrides(*out_strides[:3])
        opt = _CFwdOptions(None if packed else C.pointer(si), None if packed else C.pointer(so),
                           0 if dtype == torch.bfloat16 else 1, None if lse is None else lse.data_ptr(), int(kernel))
        st = None
        if split is not None:
            split_args = lib, args, opt, split, bq, D, q.device, stream
            if stream == current or not split.n_slots:
                st = _split_call(*split_args)
            else:
                if state.stream is None:
                    state.stream = _torch_stream(stream, q.device)
                if torch.cuda.current_device() == q.device.index:
                    # torch.cuda.stream() takes 3 us more: it looks after the device as well
                    back = torch.cuda.current_stream()
                    torch.cuda.set_stream(state.stream)
                    try:
                        st = _split_call(*split_args)
                    finally:
                        torch.cuda.set_stream(back)
                else:
                    with torch.cuda.stream(state.stream):
                        st = _split_call(*split_args)
        if st is None:
            st = lib.calibatt_sparse_attn_fwd_ex(*args, C.byref(opt), stream)
    if st != 0:
        raise CalibattError(st, "calibatt_sparse_attn_fwd")
    return out


def _split_call(lib, args, opt, split, block_q, D, device, stream):
    """calibatt_sparse_attn_fwd_split with a workspace of torch's current stream, which is the call's; None where the
    memory for it is not there (the call then runs with whole rows, which take none)."""
    import torch

    if not split.n_slots:  # no row is cut: nothing is left anywhere
        return lib.calibatt_sparse_attn_fwd_split(*args, C.byref(opt), C.byref(split), None, 0, stream)
    nbytes = split.n_slots * _part_bytes(block_q, D)
    try:
        workspace = torch.empty(nbytes // 4, dtype=torch.float32, device=device)
        if torch.cuda.is_current_stream_capturing():
            # a captured call counts in memory of its own graph: replays may overlap calls of the stream it is captured on
            arrivals = torch.zeros(split.n_rows, dtype=torch.int32, device=device)
            split = _CSplit(split.B, split.n_parts, split.n_rows, split.n_slots, split.parts, arrivals.data_ptr())
    except torch.OutOfMemoryError:
        return None
    return lib.calibatt_sparse_attn_fwd_split(*args, C.byref(opt), C.byref(split), workspace.data_ptr(), nbytes, stream)


@functools.lru_cache(maxsize=16)
def _part_bytes(block_q: int, D: int) -> int:
    """Workspace of one part of a cut row (calibatt_split_workspace_bytes)."""
    return load_library().calibatt_split_workspace_bytes(C.byref(_CSplit(1, 0, 0, 1, None, None)), block_q, D)


@dataclass
class HostAnchorMap:
    """Output of calibatt_anchor_map in host (NumPy) buffers."""
    N: int
    n_q: int
    q_index: np.ndarray
    dst_ptr: np.ndarray
    dst_idx: np.ndarray

    def to_device(self, device="cuda") -> "DeviceAnchorMap":
        return DeviceAnchorMap(self, device)


def anchor_map(N, F, Hs, Ws, k) -> HostAnchorMap:
    lib = load_library()
    n_q = C.c_int32(0)
    st = lib.calibatt_anchor_map(N, F, Hs, Ws, k, None, None, None, C.byref(n_q))
    if st != 0:
        raise CalibattError(st, "calibatt_anchor_map")
    q_index = np.empty(n_q.value, np.int32)
    dst_ptr = np.empty(n_q.value + 1, np.int32)
    dst_idx = np.empty(N, np.int32)
    st = lib.calibatt_anchor_map(N, F, Hs, Ws, k, _ptr(q_index, C.c_int32), _ptr(dst_ptr, C.c_int32),
                                 _ptr(dst_idx, C.c_int32), C.byref(n_q))
    if st != 0:
        raise CalibattError(st, "calibatt_anchor_map")
    return HostAnchorMap(N=N, n_q=int(n_q.value), q_index=q_index, dst_ptr=dst_ptr, dst_idx=dst_idx)


class DeviceAnchorMap:
    """The three lists of an anchor map as int32 torch tensors on the GPU."""

    def __init__(self, hm: HostAnchorMap, device="cuda"):
        import torch

        self.host = hm
        self.n_q = hm.n_q
        self.q_index = torch.from_numpy(np.ascontiguousarray(hm.q_index, dtype=np.int32)).to(device)
        self.dst_ptr = torch.from_numpy(np.ascontiguousarray(hm.dst_ptr, dtype=np.int32)).to(device)
        self.dst_idx = torch.from_numpy(np.ascontiguousarray(hm.dst_idx, dtype=np.int32)).to(device)


def anchor_split_plan(B: int, N: int, D: int, n_heads: int, n_q: int):
    """calibatt_anchor_split_plan on the current device: (n_split, workspace_bytes)."""
    lib = load_library()
    n_split, nbytes = C.c_int32(0), C.c_int64(0)
    st = lib.calibatt_anchor_split_plan(B, N, D, n_heads, n_q, C.byref(n_split), C.byref(nbytes))
    if st != 0:
        raise CalibattError(st, "calibatt_anchor_split_plan")
    return n_split.value, nbytes.value


def anchor_attn_fwd(q, k, v, out, head_ids, amap: DeviceAnchorMap, scale: float, stream=None, workspace=None):
    """calibatt_anchor_attn_fwd on torch bf16 CUDA tensors of logical shape [B, H, N, D] (strided views
    with contiguous D allowed, q, k, v sharing their strides); ``head_ids`` is an int32 CUDA tensor of
    the heads to process.  ``workspace``: a contiguous CUDA tensor of at least the bytes
    ``anchor_split_plan`` names for the shape selects calibatt_anchor_attn_fwd_split."""
    import torch

    lib = load_library()
    for t in (q, k, v, out):
        if not (t.is_cuda and t.dtype == torch.bfloat16 and t.dim() == 4 and t.stride(3) == 1):
            raise ValueError("q, k, v, out must be bf16 CUDA tensors [B, H, N, D] with contiguous D")
        if t.shape != q.shape:
            raise ValueError("q, k, v, out must have the same shape")
    if not (q.stride() == k.stride() == v.stride()):
        raise ValueError("q, k, v must share their strides")
    if not (head_ids.is_cuda and head_ids.dtype == torch.int32 and head_ids.is_contiguous() and head_ids.dim() == 1):
        raise ValueError("head_ids must be a contiguous 1-d int32 CUDA tensor")
    B, H, N, D = q.shape
    if stream is None:
        stream = torch.cuda.current_stream(q.device).cuda_stream
    args = (q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), B, H, N, D,
            head_ids.data_ptr(), head_ids.numel(), amap.q_index.data_ptr(),
            amap.dst_ptr.data_ptr(), amap.dst_idx.data_ptr(), amap.n_q, float(scale))
    if workspace is not None:
        if not (workspace.is_cuda and workspace.is_contiguous() and workspace.device == q.device):
            raise ValueError("workspace must be a contiguous CUDA tensor on the tensors' device")
        si = _CStrides(q.stride(0), q.stride(1), q.stride(2))
        so = _CStrides(out.stride(0), out.stride(1), out.stride(2))
        st = lib.calibatt_anchor_attn_fwd_split(*args, C.byref(si), C.byref(so), C.c_void_p(workspace.data_ptr()),
                                                workspace.numel() * workspace.element_size(), C.c_void_p(stream))
    elif all(t.is_contiguous() for t in (q, k, v, out)):
        st = lib.calibatt_anchor_attn_fwd(*args, C.c_void_p(stream))
    else:
        si = _CStrides(q.stride(0), q.stride(1), q.stride(2))
        so = _CStrides(out.stride(0), out.stride(1), out.stride(2))
        st = lib.calibatt_anchor_attn_fwd_strided(*args, C.byref(si), C.byref(so), C.c_void_p(stream))
    if st != 0:
        raise CalibattError(st, "calibatt_anchor_attn_fwd")
    return out


def _torch_stream(handle: int, device):
    """The torch stream of a handle (ExternalStream(0) is not the default stream but one of torch's own)."""
    import torch

    return torch.cuda.ExternalStream(handle, device=device) if handle else torch.cuda.default_stream(device)


def _current_handle(device) -> int:
    """Handle of torch's current stream (a stream object costs 2 us, as much as half a launch)."""
    import torch

    index = device.index
    return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device() if index is None else index)


def _stream_of(stream, device):
    """(handle, other): the stream handle of a call (None = torch's current stream), and that stream as a torch stream
    where it is not the current one.  What a call allocates is allocated under ``torch.cuda.stream(other)`` (None = the
    current one): free memory of the current stream may still be in use by work of its last owner there, which nothing
    orders before another stream."""
    current = _current_handle(device)
    if stream is None or int(stream) == current:
        return current, None
    return int(stream), _torch_stream(int(stream), device)


def _empty(shape, dtype, device, other, returned=False):
    """An uninitialised tensor of the call's stream (see ``_stream_of``); one that is returned may be read and released
    on the current stream."""
    import torch

    if other is None:
        return torch.empty(shape, dtype=dtype, device=device)
    current = torch.cuda.current_stream(device)
    with torch.cuda.stream(other):
        t = torch.empty(shape, dtype=dtype, device=device)
    if returned:
        t.record_stream(current)
    return t


def block_energy_workspace_bytes(N: int, block_q: int, block_k: int) -> int:
    lib = load_library()
    n = C.c_int64(0)
    st = lib.calibatt_block_energy_workspace_bytes(N, block_q, block_k, C.byref(n))
    if st != 0:
        raise CalibattError(st, "calibatt_block_energy_workspace_bytes")
    return n.value


def block_energy_onepass_form(B: int, H: int, N: int, D: int, block_q: int, block_k: int, workspace_bytes: int) -> int:
    """calibatt_block_energy_onepass_form: the form of such a call on the current device, ENERGY_*."""
    lib = load_library()
    n = C.c_int32(0)
    st = lib.calibatt_block_energy_onepass_form(B, H, N, D, block_q, block_k, workspace_bytes, C.byref(n))
    if st != 0:
        raise CalibattError(st, "calibatt_block_energy_onepass_form")
    return n.value


def block_energy(q, k, block_q: int, block_k: int, scale: float, out=None, stream=None, workspace=None):
    """calibatt_block_energy on torch bf16 CUDA tensors [B, H, N, D]; returns the fp32 CUDA tensor
    [B, H, ceil(N/block_q), ceil(N/block_k)] (``out`` if given).  ``workspace`` (a contiguous CUDA
    tensor, see ``block_energy_workspace_bytes``) selects calibatt_block_energy_onepass."""
    import torch

    lib = load_library()
    for t in (q, k):
        if not (t.is_cuda and t.dtype == torch.bfloat16 and t.is_contiguous() and t.dim() == 4):
            raise ValueError("q, k must be contiguous bf16 CUDA tensors [B, H, N, D]")
    if q.shape != k.shape:
        raise ValueError("q and k must have the same shape")
    B, H, N, D = q.shape
    shape = (B, H, -(-N // block_q), -(-N // block_k))
    stream, other = _stream_of(stream, q.device)
    if out is None:
        out = _empty(shape, torch.float32, q.device, other, returned=True)
    elif not (out.is_cuda and out.dtype == torch.float32 and out.is_contiguous() and tuple(out.shape) == shape):
        raise ValueError(f"out must be a contiguous fp32 CUDA tensor of shape {shape}")
    if workspace is not None:
        if not (workspace.is_cuda and workspace.is_contiguous() and workspace.device == q.device):
            raise ValueError("workspace must be a contiguous CUDA tensor on the tensors' device")
        st = lib.calibatt_block_energy_onepass(q.data_ptr(), k.data_ptr(), out.data_ptr(), B, H, N, D, block_q, block_k,
                                               float(scale), workspace.data_ptr(),
                                               workspace.numel() * workspace.element_size(), C.c_void_p(stream))
    else:
        st = lib.calibatt_block_energy(q.data_ptr(), k.data_ptr(), out.data_ptr(), B, H, N, D, block_q, block_k,
                                       float(scale), C.c_void_p(stream))
    if st != 0:
        raise CalibattError(st, "calibatt_block_energy")
    return out


def select_blocks_device(energy, eps: float, out=None, stream=None):
    """calibatt_select_blocks_device on a contiguous fp32 CUDA tensor [..., nbk]: uint8 CUDA mask of the
    same shape (``out`` if given)."""
    import torch

    lib = load_library()
    if not (energy.is_cuda and energy.dtype == torch.float32 and energy.is_contiguous() and energy.dim() >= 1):
        raise ValueError("energy must be a contiguous fp32 CUDA tensor [..., nbk]")
    stream, other = _stream_of(stream, energy.device)
    if out is None:
        out = _empty(energy.shape, torch.uint8, energy.device, other, returned=True)
    elif not (out.is_cuda and out.dtype == torch.uint8 and out.is_contiguous() and out.shape == energy.shape):
        raise ValueError("out must be a contiguous uint8 CUDA tensor of the energies' shape")
    nbk = energy.shape[-1]
    st = lib.calibatt_select_blocks_device(energy.data_ptr(), energy.numel() // max(nbk, 1), nbk, float(eps),
                                           out.data_ptr(), C.c_void_p(stream))
    if st != 0:
        raise CalibattError(st, "calibatt_select_blocks_device")
    return out


def vote_accumulate_device(mask, counts, stream=None):
    """calibatt_vote_accumulate_device: ``mask`` uint8 CUDA tensor of n entries, ``counts`` int16 CUDA
    tensor of n entries holding uint16 counters (torch has no arithmetic on uint16; read them back with
    ``counts.cpu().numpy().view(numpy.uint16)``)."""
    import torch

    lib = load_library()
    if not (mask.is_cuda and mask.dtype == torch.uint8 and mask.is_contiguous()):
        raise ValueError("mask must be a contiguous uint8 CUDA tensor")
    if not (counts.is_cuda and counts.dtype == torch.int16 and counts.is_contiguous() and counts.numel() == mask.numel()):
        raise ValueError("counts must be a contiguous int16 CUDA tensor with one entry per mask entry")
    if stream is None:
        stream = torch.cuda.current_stream(mask.device).cuda_stream
    st = lib.calibatt_vote_accumulate_device(mask.data_ptr(), mask.numel(), counts.data_ptr(), C.c_void_p(stream))
    if st != 0:
        raise CalibattError(st, "calibatt_vote_accumulate_device")
    return counts


def select_blocks(energy, eps: float) -> np.ndarray:
    """calibatt_select_blocks on a host array [..., nbk] (converted to fp32): uint8 mask of the same shape."""
    lib = load_library()
    e = np.ascontiguousarray(energy, dtype=np.float32)
    if e.ndim < 1 or e.shape[-1] == 0:
        raise CalibattError(-2, "calibatt_select_blocks")
    mask = np.empty(e.shape, np.uint8)
    st = lib.calibatt_select_blocks(_ptr(e, C.c_float), e.size // e.shape[-1], e.shape[-1], float(eps),
                                    _ptr(mask, C.c_uint8))
    if st != 0:
        raise CalibattError(st, "calibatt_select_blocks")
    return mask


def vote_masks(masks, rho: float) -> np.ndarray:
    """calibatt_vote_masks on a host array [n_prompts, ...]: uint8 mask of the trailing shape."""
    lib = load_library()
    m = np.ascontiguousarray(masks, dtype=np.uint8)
    if m.ndim < 1 or m.shape[0] == 0:
        raise CalibattError(-2, "calibatt_vote_masks")
    out = np.empty(m.shape[1:], np.uint8)
    st = lib.calibatt_vote_masks(_ptr(m, C.c_uint8), m.shape[0], out.size, float(rho), _ptr(out, C.c_uint8))
    if st != 0:
        raise CalibattError(st, "calibatt_vote_masks")
    return out


def vote_accumulate(mask, counts: np.ndarray) -> None:
    """calibatt_vote_accumulate: adds one prompt's mask to the uint16 counters (same shape), in place."""
    lib = load_library()
    m = np.ascontiguousarray(mask, dtype=np.uint8)
    if not (counts.dtype == np.uint16 and counts.flags.c_contiguous and counts.shape == m.shape):
        raise ValueError("counts must be a C-contiguous uint16 array of the mask's shape")
    st = lib.calibatt_vote_accumulate(_ptr(m, C.c_uint8), m.size, _ptr(counts, C.c_uint16))
    if st != 0:
        raise CalibattError(st, "calibatt_vote_accumulate")


def vote_finish(counts: np.ndarray, n_prompts: int, rho: float) -> np.ndarray:
    """calibatt_vote_finish: uint8 mask of the counters' shape."""
    lib = load_library()
    c = np.ascontiguousarray(counts, dtype=np.uint16)
    out = np.empty(c.shape, np.uint8)
    st = lib.calibatt_vote_finish(_ptr(c, C.c_uint16), int(n_prompts), c.size, float(rho), _ptr(out, C.c_uint8))
    if st != 0:
        raise CalibattError(st, "calibatt_vote_finish")
    return out


def epsilon_schedule(t: int, T: int, A: float, Cc: float, k: float) -> float:
    return float(load_library().calibatt_epsilon_schedule(int(t), int(T), float(A), float(Cc), float(k)))


def schedule_base_level(N: int) -> float:
    return float(load_library().calibatt_schedule_base_level(int(N)))


REGIME_MANY_STEP, REGIME_DISTILLED = 0, 1


def schedule_constants(regime: int, N: int):
    """calibatt_schedule_constants: (A, C, k) of Eq. 7 for the many-step (0) or distilled (1) regime."""
    lib = load_library()
    A, Cc, k = C.c_double(), C.c_double(), C.c_double()
    st = lib.calibatt_schedule_constants(int(regime), int(N), C.byref(A), C.byref(Cc), C.byref(k))
    if st != 0:
        raise CalibattError(st, "calibatt_schedule_constants")
    return A.value, Cc.value, k.value


def flag_heads(scores, gamma: float):
    """calibatt_flag_heads: scores [n_prompts, H] -> (flags uint8 [H], mean float64 [H])."""
    lib = load_library()
    s = np.ascontiguousarray(scores, dtype=np.float32)
    if s.ndim != 2:
        raise ValueError("scores must be [n_prompts, H]")
    flags = np.zeros(s.shape[1], dtype=np.uint8)
    mean = np.zeros(s.shape[1], dtype=np.float64)
    st = lib.calibatt_flag_heads(s.ctypes.data_as(C.POINTER(C.c_float)), int(s.shape[0]), int(s.shape[1]), float(gamma),
                                 flags.ctypes.data_as(C.POINTER(C.c_uint8)), mean.ctypes.data_as(C.POINTER(C.c_double)))
    if st != 0:
        raise CalibattError(st, "calibatt_flag_heads")
    return flags, mean


def encode_intervals(row_ptr, col_idx):
    """calibatt_encode_intervals: (iv_ptr int32 [rows + 1], iv uint32 words)."""
    lib = load_library()
    rp = np.ascontiguousarray(row_ptr, dtype=np.int32)
    ci = np.ascontiguousarray(col_idx, dtype=np.int32)
    if ci.size == 0:
        ci = np.zeros(1, np.int32)
    n_rows = rp.size - 1
    n_words = C.c_int64(0)
    st = lib.calibatt_encode_intervals(_ptr(rp, C.c_int32), _ptr(ci, C.c_int32), n_rows, None, None, 0, C.byref(n_words))
    if st != 0:
        raise CalibattError(st, "calibatt_encode_intervals")
    iv_ptr = np.empty(n_rows + 1, np.int32)
    iv = np.empty(max(n_words.value, 1), np.uint32)
    st = lib.calibatt_encode_intervals(_ptr(rp, C.c_int32), _ptr(ci, C.c_int32), n_rows, _ptr(iv_ptr, C.c_int32),
                                       _ptr(iv, C.c_uint32), iv.size, C.byref(n_words))
    if st != 0:
        raise CalibattError(st, "calibatt_encode_intervals")
    return iv_ptr, iv[: n_words.value]


def merge_intervals(mask, pct: float):
    """calibatt_merge_intervals over all rows of ``mask[..., nbk]``: (merged uint8 mask, width)."""
    lib = load_library()
    m = np.ascontiguousarray(mask, dtype=np.uint8)
    if m.ndim < 1 or m.shape[-1] == 0:
        raise CalibattError(-2, "calibatt_merge_intervals")
    out = np.empty_like(m)
    width = C.c_int32(0)
    st = lib.calibatt_merge_intervals(_ptr(m, C.c_uint8), m.size // m.shape[-1], m.shape[-1], float(pct),
                                      _ptr(out, C.c_uint8), C.byref(width))
    if st != 0:
        raise CalibattError(st, "calibatt_merge_intervals")
    return out, int(width.value)


def share_timesteps(masks, tau: float):
    """calibatt_share_timesteps on ``masks[T, ...]`` of one (layer, head): (cluster ids int32 [T],
    shared masks uint8 [n_clusters, ...])."""
    lib = load_library()
    m = np.ascontiguousarray(masks, dtype=np.uint8)
    if m.ndim < 1 or m.shape[0] == 0:
        raise CalibattError(-2, "calibatt_share_timesteps")
    T = m.shape[0]
    n = m.size // T
    cluster = np.empty(T, np.int32)
    shared = np.empty_like(m)
    n_clusters = C.c_int32(0)
    st = lib.calibatt_share_timesteps(_ptr(m, C.c_uint8), T, n, float(tau), _ptr(cluster, C.c_int32),
                                      _ptr(shared, C.c_uint8), C.byref(n_clusters))
    if st != 0:
        raise CalibattError(st, "calibatt_share_timesteps")
    return cluster, shared[: n_clusters.value].copy()


def anchor_partner(F, Hs, Ws, k) -> np.ndarray:
    """calibatt_anchor_partner: int32 [F*Hs*Ws], the token each video token is compared with."""
    lib = load_library()
    if min(F, Hs, Ws) <= 0:
        raise CalibattError(-2, "calibatt_anchor_partner")
    partner = np.empty(F * Hs * Ws, np.int32)
    st = lib.calibatt_anchor_partner(F, Hs, Ws, k, _ptr(partner, C.c_int32))
    if st != 0:
        raise CalibattError(st, "calibatt_anchor_partner")
    return partner


def spatial_similarity(q, k, partner, row_len: int, scale: float, workspace=None, stream=None):
    """calibatt_spatial_similarity on torch bf16 CUDA tensors [B, H, N, D]; ``partner`` is an int32
    CUDA tensor [n_tok].  Returns the fp32 CUDA tensor [B, H] of scores."""
    import torch

    lib = load_library()
    for t in (q, k):
        if not (t.is_cuda and t.dtype == torch.bfloat16 and t.is_contiguous() and t.dim() == 4):
            raise ValueError("q, k must be contiguous bf16 CUDA tensors [B, H, N, D]")
    if q.shape != k.shape:
        raise ValueError("q and k must have the same shape")
    if not (partner.is_cuda and partner.dtype == torch.int32 and partner.is_contiguous() and partner.dim() == 1):
        raise ValueError("partner must be a contiguous 1-d int32 CUDA tensor")
    B, H, N, D = q.shape
    n_tok = partner.numel()
    stream, other = _stream_of(stream, q.device)
    if workspace is None:
        workspace = _empty((B, H, max(n_tok, 1), 3), torch.float32, q.device, other)
    score = _empty((B, H), torch.float32, q.device, other, returned=True)
    nbytes = C.c_int64(0)
    lists = None
    if lib.calibatt_similarity_lists_bytes(B, H, n_tok, C.byref(nbytes)) == 0 and nbytes.value > 0:
        lists = _empty(nbytes.value, torch.uint8, q.device, other)
    st = lib.calibatt_spatial_similarity_grouped(q.data_ptr(), k.data_ptr(), B, H, N, D, partner.data_ptr(), n_tok,
                                                 int(row_len), float(scale), workspace.data_ptr(),
                                                 None if lists is None else lists.data_ptr(), nbytes.value,
                                                 score.data_ptr(), C.c_void_p(stream))
    if st != 0:
        raise CalibattError(st, "calibatt_spatial_similarity")
    return score


SIMILARITY_STATIC_MAX_BYTES = 16 * 1024 * 1024


def spatial_similarity_static(q, k, partner, row_len: int, scale: float, score, stream=None):
    """calibatt_spatial_similarity_static: the call that allocates nothing.  ``score`` is the caller's
    fp32 CUDA tensor [B, H]; the per-token sums live in the library's own buffer (one per GPU, shared by
    all calls on it)."""
    import torch

    lib = load_library()
    for t in (q, k):
        if not (t.is_cuda and t.dtype == torch.bfloat16 and t.is_contiguous() and t.dim() == 4):
            raise ValueError("q, k must be contiguous bf16 CUDA tensors [B, H, N, D]")
    if q.shape != k.shape:
        raise ValueError("q and k must have the same shape")
    if not (partner.is_cuda and partner.dtype == torch.int32 and partner.is_contiguous() and partner.dim() == 1):
        raise ValueError("partner must be a contiguous 1-d int32 CUDA tensor")
    B, H, N, D = q.shape
    if not (score.is_cuda and score.dtype == torch.float32 and score.is_contiguous() and tuple(score.shape) == (B, H)):
        raise ValueError("score must be a contiguous fp32 CUDA tensor [B, H]")
    if stream is None:
        stream = torch.cuda.current_stream(q.device).cuda_stream
    st = lib.calibatt_spatial_similarity_static(q.data_ptr(), k.data_ptr(), B, H, N, D, partner.data_ptr(),
                                                partner.numel(), int(row_len), float(scale), score.data_ptr(),
                                                C.c_void_p(stream))
    if st != 0:
        raise CalibattError(st, "calibatt_spatial_similarity_static")
    return score
