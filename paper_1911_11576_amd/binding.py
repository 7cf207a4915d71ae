"""Binding of include/fs.h: same entry points, argument marshalling only, by ctypes; the launch calls by the module
_launch (csrc/py_launch.cpp) where it was built for this interpreter, else by ctypes too, a microsecond a call slower.

Every step of the path runs in the HIP library.  PyTorch appears here only as the
owner of device memory and streams (`tensor.data_ptr()`, the current stream's
handle).  If the built library is missing, loading fails loudly: there is no CPU
or eager fallback.
"""
from __future__ import annotations

import ctypes as C
import os
from array import array
from collections import namedtuple
from math import prod

FS_MAX_RANK = 4
LIB_PATH = os.environ.get("FS_LIB_PATH") or os.path.join(os.path.dirname(os.path.abspath(__file__)),
                                                        "libfusionstitch.so")

FS_OK, FS_ERR_INVALID, FS_ERR_UNSUPPORTED, FS_ERR_LDS, FS_ERR_HIP, FS_ERR_NOMEM = range(6)
STATUS_NAMES = ["FS_OK", "FS_ERR_INVALID", "FS_ERR_UNSUPPORTED", "FS_ERR_LDS", "FS_ERR_HIP", "FS_ERR_NOMEM"]
FS_MODE_STITCHED, FS_MODE_PER_OP, FS_MODE_STITCHED_PREBUILT, FS_MODE_STITCHED_GENERATED = 0, 1, 2, 3
SCHEDULE_NAMES = ["per_op", "row", "row_col", "bdot_softmax", "elementwise", "block_dot", "two_step"]

DTYPES = {"f32": 0, "f16": 1, "bf16": 2}
OPKINDS = {name: i for i, name in enumerate((
    "parameter", "constant", "add", "subtract", "multiply", "divide", "maximum", "negate",
    "exp", "log", "tanh", "rsqrt", "sqrt", "convert", "broadcast", "reduce_sum", "reduce_max",
    "dot", "causal_mask", "output", "erf", "logistic"))}


class fs_op_desc(C.Structure):
    _fields_ = [("kind", C.c_int32), ("dtype", C.c_int32), ("rank", C.c_int32), ("axis", C.c_int32),
                ("shape", C.c_int64 * FS_MAX_RANK), ("operand", C.c_int32 * 3),
                ("reserved", C.c_int32), ("attr", C.c_double)]


class fs_plan_options(C.Structure):
    _fields_ = [("mode", C.c_int32), ("wg_size", C.c_int32), ("rows_per_wave", C.c_int32),
                ("grid", C.c_int32)]


class fs_fusion_options(C.Structure):
    _fields_ = [("launch_us", C.c_double), ("max_patterns", C.c_int32), ("explore_budget", C.c_int32),
                ("seed_bytes", C.c_int64), ("bw_bytes", C.POINTER(C.c_int64)), ("bw_gbs", C.POINTER(C.c_double)),
                ("n_bw", C.c_int32), ("n_extra", C.c_int32), ("extra_sizes", C.POINTER(C.c_int32)),
                ("extra_ops", C.POINTER(C.c_int32)), ("extra_scores", C.POINTER(C.c_double))]


class FsError(RuntimeError):
    def __init__(self, status, message):
        super().__init__(f"{STATUS_NAMES[status] if 0 <= status < 6 else status}: {message}")
        self.status = status
        self.message = message


_lib = None
_native = None              # the launch entry points on Python lists (_launch or _CtypesCalls), with lib()


def lib():
    """The loaded shared library (loaded on first use)."""
    global _lib, _native
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise ImportError(
                f"{LIB_PATH} is not built: run `python -m paper_1911_11576_amd.build` "
                "(there is no fallback path)")
        L = C.CDLL(LIB_PATH)
        vp, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
        L.fs_plan_create.argtypes = [C.POINTER(fs_op_desc), i32, C.POINTER(fs_plan_options), C.POINTER(vp)]
        L.fs_plan_create.restype = i32
        L.fs_plan_create_packed.argtypes = [C.POINTER(C.POINTER(fs_op_desc)), C.POINTER(i32), i32, C.POINTER(C.c_uint8), C.POINTER(vp)]
        L.fs_plan_create_packed.restype = i32
        L.fs_plan_create_two_step.argtypes = [C.POINTER(fs_op_desc), i32, C.POINTER(i64), C.POINTER(vp)]
        L.fs_plan_create_two_step.restype = i32
        L.fs_launch.argtypes = [vp, C.POINTER(vp), i32, C.POINTER(vp), i32, vp]
        L.fs_launch.restype = i32
        L.fs_launch_static.argtypes = [vp, C.POINTER(vp), i32, C.POINTER(vp), i32, vp]
        L.fs_launch_static.restype = i32
        L.fs_destroy.argtypes = [vp]
        L.fs_destroy.restype = i32
        L.fs_last_error.argtypes = []
        L.fs_last_error.restype = C.c_char_p
        L.fs_plan_info.argtypes = [vp, C.POINTER(i32), C.POINTER(i32), C.POINTER(i64), C.POINTER(i64),
                                   C.POINTER(i64), C.POINTER(i64)]
        L.fs_plan_info.restype = i32
        L.fs_plan_describe.argtypes = [vp]
        L.fs_plan_describe.restype = C.c_char_p
        L.fs_plan_tune.argtypes = [C.POINTER(fs_op_desc), i32, C.POINTER(vp), i32, C.POINTER(vp), i32, vp, i32,
                                   C.POINTER(vp), C.POINTER(fs_plan_options), C.POINTER(C.c_double)]
        L.fs_plan_tune.restype = i32
        L.fs_stream_copy.argtypes = [vp, vp, i64, vp]
        L.fs_stream_copy.restype = i32
        L.fs_kernel_cache_dir.argtypes = [C.c_char_p]
        L.fs_kernel_cache_dir.restype = i32
        L.fs_kernel_cache_stats.argtypes = [C.POINTER(i64), C.POINTER(i64), C.POINTER(i64)]
        L.fs_kernel_cache_stats.restype = i32
        L.fs_kernel_cache_drop_memory.argtypes = []
        L.fs_kernel_cache_drop_memory.restype = i32
        L.fs_group_key.argtypes = [C.POINTER(fs_op_desc), i32, C.POINTER(C.c_uint64)]
        L.fs_group_key.restype = i32
        L.fs_tune_cache_has.argtypes = [C.c_uint64]
        L.fs_tune_cache_has.restype = i32
        L.fs_tune_cache_size.argtypes = []
        L.fs_tune_cache_size.restype = i32
        L.fs_tune_cache_clear.argtypes = []
        L.fs_tune_cache_clear.restype = i32
        L.fs_tune_cache_save.argtypes = [C.c_char_p]
        L.fs_tune_cache_save.restype = i32
        L.fs_tune_cache_load.argtypes = [C.c_char_p]
        L.fs_tune_cache_load.restype = i32
        L.fs_shared_plan.argtypes = [C.POINTER(i32), C.POINTER(i64), C.POINTER(C.c_uint8), i32, C.POINTER(i64),
                                     C.POINTER(i32), C.POINTER(i64)]
        L.fs_shared_plan.restype = i32
        L.fs_fusion_create.argtypes = [C.POINTER(fs_op_desc), i32, C.POINTER(fs_fusion_options), C.POINTER(vp)]
        L.fs_fusion_create.restype = i32
        L.fs_fusion_destroy.argtypes = [vp]
        L.fs_fusion_destroy.restype = i32
        L.fs_fusion_info.argtypes = [vp, C.POINTER(i32), C.POINTER(i32), C.POINTER(C.c_double), C.POINTER(i32)]
        L.fs_fusion_info.restype = i32
        L.fs_fusion_group_size.argtypes = [vp, i32, C.POINTER(i32), C.POINTER(i32), C.POINTER(i32), C.POINTER(i32),
                                           C.POINTER(C.c_double)]
        L.fs_fusion_group_size.restype = i32
        L.fs_fusion_group.argtypes = [vp, i32, C.POINTER(fs_op_desc), C.POINTER(i32), C.POINTER(i32), C.POINTER(i32)]
        L.fs_fusion_group.restype = i32
        L.fs_fusion_pattern.argtypes = [vp, i32, C.POINTER(i32), C.POINTER(i32), i32, C.POINTER(i32), C.POINTER(i64),
                                        C.POINTER(C.c_double), C.POINTER(i32)]
        L.fs_fusion_pattern.restype = i32
        L.fs_fusion_pattern_group_size.argtypes = [vp, i32, C.POINTER(i32), C.POINTER(i32), C.POINTER(i32), C.POINTER(i32)]
        L.fs_fusion_pattern_group_size.restype = i32
        L.fs_fusion_pattern_group.argtypes = [vp, i32, C.POINTER(fs_op_desc), C.POINTER(i32), C.POINTER(i32)]
        L.fs_fusion_pattern_group.restype = i32
        _native = _launch_calls(L)
        _lib = L
    return _lib


class _CtypesCalls:
    """The calls of the module _launch by ctypes, for an interpreter that it was not built for."""

    def __init__(self):
        raw = C.CDLL(LIB_PATH)          # a handle of its own: plain addresses in place of lib()'s typed pointers
        for f in (raw.fs_launch, raw.fs_launch_static):
            f.argtypes = [C.c_void_p, C.c_void_p, C.c_int32, C.c_void_p, C.c_int32, C.c_void_p]
            f.restype = C.c_int32
        self.launch_arrays, self._launch_static, self._stream = raw.fs_launch, raw.fs_launch_static, None

    def current_stream(self):
        if self._stream is None:
            self._stream = _stream_source()
        raw, device = self._stream
        return raw(device()) if device else raw()

    def _call(self, f, plan, inputs, outputs, stream):
        if stream is None:
            stream = self.current_stream()
        ins, n_in = self._addresses(inputs)
        outs, n_out = self._addresses(outputs)
        return f(plan, ins.buffer_info()[0], n_in, outs.buffer_info()[0], n_out, stream)

    @staticmethod
    def _addresses(tensors):
        len(tensors)                    # an iterator has no length: refused
        taken = [t if isinstance(t, int) else t.data_ptr() for t in tensors]
        return array("Q", taken or [0]), len(taken)

    def launch(self, plan, inputs, outputs, stream):
        return self._call(self.launch_arrays, plan, inputs, outputs, stream)

    def launch_static(self, plan, inputs, outputs, stream):
        return self._call(self._launch_static, plan, inputs, outputs, stream)


def _launch_calls(L):
    try:
        from . import _launch
    except ImportError:
        return _CtypesCalls()
    _launch.bind(C.cast(L.fs_launch, C.c_void_p).value, C.cast(L.fs_launch_static, C.c_void_p).value, _stream_source,
                 C.c_void_p, lambda o: C.cast(o, C.c_void_p).value)
    return _launch


def fs_last_error():
    return lib().fs_last_error().decode()


def _check(status):
    if status != FS_OK:
        raise FsError(status, fs_last_error())


def marshal_ops(ops):
    """Sequence of records with fields kind, dtype, shape, operands, axis, attr ->
    a C array of fs_op_desc."""
    arr = (fs_op_desc * len(ops))()
    for d, op in zip(arr, ops):
        d.kind = OPKINDS[op.kind]
        d.dtype = DTYPES[op.dtype]
        d.rank = len(op.shape)
        d.axis = op.axis if op.axis >= 0 else 0
        for k in range(FS_MAX_RANK):
            d.shape[k] = op.shape[k] if k < len(op.shape) else 0
        for k in range(3):
            d.operand[k] = op.operands[k] if k < len(op.operands) else -1
        d.reserved = 0
        d.attr = op.attr
    return arr


def fs_plan_create(ops, mode=FS_MODE_STITCHED, wg_size=0, rows_per_wave=0, grid=0):
    """-> opaque plan handle (int).  `ops` may be a marshalled array or op records."""
    arr = ops if isinstance(ops, C.Array) else marshal_ops(ops)
    opt = fs_plan_options(mode, wg_size, rows_per_wave, grid)
    out = C.c_void_p()
    _check(lib().fs_plan_create(arr, len(arr), C.byref(opt), C.byref(out)))
    return out.value


def fs_plan_create_packed(groups):
    """groups: marshalled op lists of independent groups -> (plan handle, indices of the groups it runs), or
    FsError with FS_ERR_UNSUPPORTED if no two of them can share a launch."""
    n = len(groups)
    ptrs = (C.POINTER(fs_op_desc) * max(1, n))(*[C.cast(g, C.POINTER(fs_op_desc)) for g in groups])
    sizes = (C.c_int32 * max(1, n))(*[len(g) for g in groups])
    taken, out = (C.c_uint8 * max(1, n))(), C.c_void_p()
    _check(lib().fs_plan_create_packed(ptrs, sizes, n, taken, C.byref(out)))
    return out.value, [k for k in range(n) if taken[k]]


def fs_plan_create_two_step(ops):
    """A group in which values reduced over whole tensors feed ops on whole tensors -> (plan handle, bytes of the partial
    results, for which the plan takes a buffer as one more output), or FsError with FS_ERR_UNSUPPORTED."""
    arr = ops if isinstance(ops, C.Array) else marshal_ops(ops)
    nbytes, out = C.c_int64(), C.c_void_p()
    _check(lib().fs_plan_create_two_step(arr, len(arr), C.byref(nbytes), C.byref(out)))
    return out.value, nbytes.value


def _pointers(tensors):
    arr = (C.c_void_p * max(1, len(tensors)))()
    for i, t in enumerate(tensors):
        arr[i] = t if isinstance(t, int) else t.data_ptr()
    return arr


def _stream_source():
    """Where the handle of torch's current stream comes from (without the stream object that torch.cuda.current_stream()
    makes): a function of the device's ordinal and the one that gives the ordinal, or a function of nothing and None."""
    import torch
    raw = getattr(torch._C, "_cuda_getCurrentRawStream", None)
    if raw is None:
        return (lambda: torch.cuda.current_stream().cuda_stream), None
    return raw, torch.cuda.current_device


def _current_stream():
    if _native is None:
        lib()
    return _native.current_stream()


def fs_launch(plan, inputs, outputs, stream=None):
    """inputs/outputs: device tensors (anything with .data_ptr()) or raw addresses.
    stream: a hipStream_t address; None = torch's current stream."""
    if _native is None:
        lib()
    status = _native.launch(plan, inputs, outputs, stream)
    if status != FS_OK:
        raise FsError(status, fs_last_error())


def fs_launch_static(plan, inputs, outputs, stream=None):
    """fs_launch without any allocation: the plan's scratch memory is the library's static device array."""
    if _native is None:
        lib()
    _check(_native.launch_static(plan, inputs, outputs, stream))


def fs_plan_tune(ops, inputs, outputs, stream=None, trials=20):
    """-> (plan handle, winning options as a dict, microseconds per launch)."""
    arr = ops if isinstance(ops, C.Array) else marshal_ops(ops)
    if stream is None:
        import torch
        stream = torch.cuda.current_stream().cuda_stream
    out, opt, us = C.c_void_p(), fs_plan_options(), C.c_double()
    _check(lib().fs_plan_tune(arr, len(arr), _pointers(inputs), len(inputs), _pointers(outputs), len(outputs),
                              stream, trials, C.byref(out), C.byref(opt), C.byref(us)))
    return out.value, {"wg_size": opt.wg_size, "rows_per_wave": opt.rows_per_wave, "grid": opt.grid}, us.value


def fs_destroy(plan):
    _check(lib().fs_destroy(plan))


def fs_plan_info(plan):
    sched, nk = C.c_int32(), C.c_int32()
    lds, ws, algo, moved = C.c_int64(), C.c_int64(), C.c_int64(), C.c_int64()
    _check(lib().fs_plan_info(plan, C.byref(sched), C.byref(nk), C.byref(lds), C.byref(ws),
                              C.byref(algo), C.byref(moved)))
    return {"schedule": SCHEDULE_NAMES[sched.value], "n_kernels": nk.value, "lds_bytes": lds.value,
            "workspace_bytes": ws.value, "algorithmic_bytes": algo.value, "moved_bytes": moved.value}


def fs_plan_describe(plan):
    return lib().fs_plan_describe(plan).decode()


def fs_shared_plan(operands, req_bytes, is_output=None):
    """Algorithm 4 on a DAG given as per-op operand lists (indices of earlier ops) and shared-
    space requests in bytes.  -> (offsets, shares_with, total_bytes)."""
    n = len(operands)
    ops = (C.c_int32 * (3 * max(n, 1)))(*([-1] * (3 * max(n, 1))))
    for i, lst in enumerate(operands):
        assert len(lst) <= 3
        for j, o in enumerate(lst):
            ops[3 * i + j] = o
    req = (C.c_int64 * max(n, 1))(*req_bytes) if n else (C.c_int64 * 1)()
    outs = None if is_output is None else (C.c_uint8 * max(n, 1))(*[1 if b else 0 for b in is_output])
    off = (C.c_int64 * max(n, 1))()
    shr = (C.c_int32 * max(n, 1))()
    total = C.c_int64(0)
    _check(lib().fs_shared_plan(ops, req, outs, n, off, shr, C.byref(total)))
    return list(off[:n]), list(shr[:n]), total.value


def fs_kernel_cache_dir(path):
    """Directory for compiled kernels shared between processes (None turns it off)."""
    _check(lib().fs_kernel_cache_dir(None if path is None else str(path).encode()))


def fs_kernel_cache_stats():
    """-> dict(compiled, from_memory, from_disk): where generated kernels came from so far."""
    c, m, d = C.c_int64(), C.c_int64(), C.c_int64()
    _check(lib().fs_kernel_cache_stats(C.byref(c), C.byref(m), C.byref(d)))
    return {"compiled": c.value, "from_memory": m.value, "from_disk": d.value}


def fs_kernel_cache_drop_memory():
    _check(lib().fs_kernel_cache_drop_memory())


def fs_group_key(ops):
    """Key of a group in the tuning cache (an int)."""
    arr = ops if isinstance(ops, C.Array) else marshal_ops(ops)
    key = C.c_uint64()
    _check(lib().fs_group_key(arr, len(arr), C.byref(key)))
    return key.value


def fs_tune_cache_has(key):
    return bool(lib().fs_tune_cache_has(key))


def fs_tune_cache_size():
    return lib().fs_tune_cache_size()


def fs_tune_cache_clear():
    _check(lib().fs_tune_cache_clear())


def fs_tune_cache_save(path):
    _check(lib().fs_tune_cache_save(str(path).encode()))


def fs_tune_cache_load(path):
    _check(lib().fs_tune_cache_load(str(path).encode()))


def fs_stream_copy(dst, src, nbytes, stream=None):
    if stream is None:
        import torch
        stream = torch.cuda.current_stream().cuda_stream
    _check(lib().fs_stream_copy(dst if isinstance(dst, int) else dst.data_ptr(),
                                src if isinstance(src, int) else src.data_ptr(), nbytes, stream))


class BoundArgs:
    """Pointer arrays of one (inputs, outputs) set, marshalled once so that repeated
    launches of the same buffers cost a single foreign call.  Keeps the tensors alive."""

    def __init__(self, inputs, outputs):
        self.keep = (list(inputs), list(outputs))
        self.n_in, self.n_out = len(inputs), len(outputs)
        self.in_ptrs, self.out_ptrs = _pointers(inputs), _pointers(outputs)
        self.in_addr, self.out_addr = C.addressof(self.in_ptrs), C.addressof(self.out_ptrs)


class Plan:
    """Owner of one fs_plan handle."""

    def __init__(self, ops, mode="stitched", wg_size=0, rows_per_wave=0, grid=0, _handle=None):
        self._h = _handle
        if _handle is None:
            m = {"stitched": FS_MODE_STITCHED, "per_op": FS_MODE_PER_OP, "prebuilt": FS_MODE_STITCHED_PREBUILT,
                 "generated": FS_MODE_STITCHED_GENERATED}[mode]
            self._h = fs_plan_create(ops, m, wg_size, rows_per_wave, grid)
        self.tuned = None

    @classmethod
    def packed(cls, groups):
        """Independent groups as one launch (fs_plan_create_packed) -> (plan, indices of the groups it runs)."""
        h, taken = fs_plan_create_packed(groups)
        return cls(None, _handle=h), taken

    @classmethod
    def two_step(cls, ops):
        """fs_plan_create_two_step -> (plan, bytes of the buffer it takes as its last output)."""
        h, nbytes = fs_plan_create_two_step(ops)
        return cls(None, _handle=h), nbytes

    @classmethod
    def tune(cls, ops, inputs, outputs, stream=None, trials=20):
        """The fastest of the schedule's launch templates for these buffers (fs_plan_tune)."""
        h, opts, us = fs_plan_tune(ops, inputs, outputs, stream, trials)
        plan = cls(ops, _handle=h)
        plan.tuned = dict(opts, us=us)
        return plan

    def launch(self, inputs, outputs, stream=None):
        st = _native.launch(self._h, inputs, outputs, stream)
        if st != FS_OK:
            raise FsError(st, fs_last_error())

    def launch_static(self, inputs, outputs, stream=None):
        fs_launch_static(self._h, inputs, outputs, stream)

    def launch_bound(self, bound, stream):
        """Launch with pre-marshalled arguments (see BoundArgs) on an explicit stream handle."""
        st = _native.launch_arrays(self._h, bound.in_addr, bound.n_in, bound.out_addr, bound.n_out, stream)
        if st != FS_OK:
            raise FsError(st, fs_last_error())

    def info(self):
        return fs_plan_info(self._h)

    def describe(self):
        return fs_plan_describe(self._h)

    def close(self):
        if self._h is not None:
            h, self._h = self._h, None
            fs_destroy(h)

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.close()


# ---------------------------------------------------------------- fusion planning (Section 4)

_KIND_NAMES = {v: k for k, v in OPKINDS.items()}
_DTYPE_NAMES = {v: k for k, v in DTYPES.items()}


class FusionPlan:
    """fs_fusion_create on a computation graph (op records as for Plan).

    .groups     list of dicts in execution order: ops (marshalled fs_op_desc array, ready for
                fs_plan_create), input_of / output_of (indices into the original list), members
                (the original ops it fuses), score_us
    .patterns   every scored candidate: ops, origin, saved_bytes, score_us, chosen, measured, and (where a
                stitched plan exists for it) group_ops / input_of / output_of like a group's

    extra_scores: per extra pattern the microseconds it was measured to save (None or NaN: the model's score).
    """

    def __init__(self, ops, launch_us=0.0, max_patterns=0, explore_budget=0, seed_bytes=0, bandwidth=None, extra_patterns=None,
                 extra_scores=None):
        arr = ops if isinstance(ops, C.Array) else marshal_ops(ops)
        opt = fs_fusion_options()
        opt.launch_us, opt.max_patterns, opt.explore_budget, opt.seed_bytes = launch_us, max_patterns, explore_budget, seed_bytes
        keep = None
        if bandwidth:
            bb = (C.c_int64 * len(bandwidth))(*[int(b) for b, _ in bandwidth])
            gg = (C.c_double * len(bandwidth))(*[float(g) for _, g in bandwidth])
            opt.bw_bytes, opt.bw_gbs, opt.n_bw = bb, gg, len(bandwidth)
            keep = (bb, gg)
        keep2 = None
        if extra_patterns:
            sizes = (C.c_int32 * len(extra_patterns))(*[len(p) for p in extra_patterns])
            flat = [o for p in extra_patterns for o in p]
            eo = (C.c_int32 * len(flat))(*flat)
            opt.n_extra, opt.extra_sizes, opt.extra_ops = len(extra_patterns), sizes, eo
            keep2 = (sizes, eo)
            if extra_scores is not None:
                if len(extra_scores) != len(extra_patterns):
                    raise ValueError("extra_scores: one entry per extra pattern")
                es = (C.c_double * len(extra_scores))(*[float("nan") if v is None else float(v) for v in extra_scores])
                opt.extra_scores = es
                keep2 = (sizes, eo, es)
        h = C.c_void_p()
        _check(lib().fs_fusion_create(arr, len(arr), C.byref(opt), C.byref(h)))
        del keep, keep2
        try:
            ng, npat, total, rounds = C.c_int32(), C.c_int32(), C.c_double(), C.c_int32()
            _check(lib().fs_fusion_info(h, C.byref(ng), C.byref(npat), C.byref(total), C.byref(rounds)))
            self.total_score_us, self.solver_rounds = total.value, rounds.value
            self.groups, self.patterns = [], []
            for g in range(ng.value):
                n_ops, n_in, n_out, n_mem, score = C.c_int32(), C.c_int32(), C.c_int32(), C.c_int32(), C.c_double()
                _check(lib().fs_fusion_group_size(h, g, C.byref(n_ops), C.byref(n_in), C.byref(n_out), C.byref(n_mem), C.byref(score)))
                gops = (fs_op_desc * max(1, n_ops.value))()
                gin, gout = (C.c_int32 * max(1, n_in.value))(), (C.c_int32 * max(1, n_out.value))()
                gmem = (C.c_int32 * max(1, n_mem.value))()
                _check(lib().fs_fusion_group(h, g, gops, gin, gout, gmem))
                trimmed = (fs_op_desc * n_ops.value)(*gops[:n_ops.value])
                self.groups.append(dict(ops=trimmed, input_of=list(gin[:n_in.value]), output_of=list(gout[:n_out.value]),
                                        members=list(gmem[:n_mem.value]), score_us=score.value))
            for k in range(npat.value):
                n_ops, origin, saved, score, chosen = C.c_int32(), C.c_int32(), C.c_int64(), C.c_double(), C.c_int32()
                _check(lib().fs_fusion_pattern(h, k, C.byref(n_ops), None, 0, None, None, None, None))      # its size first
                buf = (C.c_int32 * max(1, n_ops.value))()
                _check(lib().fs_fusion_pattern(h, k, C.byref(n_ops), buf, n_ops.value, C.byref(origin), C.byref(saved), C.byref(score), C.byref(chosen)))
                pat = dict(ops=list(buf[:n_ops.value]), n_ops=n_ops.value, origin=origin.value,
                           saved_bytes=saved.value, score_us=score.value, chosen=bool(chosen.value))
                l_ops, l_in, l_out, measured = C.c_int32(), C.c_int32(), C.c_int32(), C.c_int32()
                _check(lib().fs_fusion_pattern_group_size(h, k, C.byref(l_ops), C.byref(l_in), C.byref(l_out), C.byref(measured)))
                pat["measured"] = bool(measured.value)
                if l_ops.value:
                    gops = (fs_op_desc * l_ops.value)()
                    gin, gout = (C.c_int32 * max(1, l_in.value))(), (C.c_int32 * max(1, l_out.value))()
                    _check(lib().fs_fusion_pattern_group(h, k, gops, gin, gout))
                    pat.update(group_ops=gops, input_of=list(gin[:l_in.value]), output_of=list(gout[:l_out.value]))
                self.patterns.append(pat)
        finally:
            lib().fs_fusion_destroy(h)


def describe_group_ops(arr):
    """The ops of a marshalled list as (kind, dtype, shape, operands) tuples, for logs and tests."""
    out = []
    for d in arr:
        nop = 0 if d.kind in (OPKINDS["parameter"], OPKINDS["constant"]) else 2 if (2 <= d.kind <= 6 or d.kind == OPKINDS["dot"]) else 1
        out.append((_KIND_NAMES[d.kind], _DTYPE_NAMES[d.dtype], tuple(d.shape[:d.rank]), tuple(d.operand[:nop])))
    return out


# A launch of a program: its plan (None: its one group's own), its groups, the values it reads and writes, the bytes of the buffer
# that it takes as one more output (0: none)
_Launch = namedtuple("_Launch", "plan members inputs outputs extra")
_OpRecord = namedtuple("_OpRecord", "kind dtype shape operands axis attr")


# What a launch is worth in bytes, for a two-step plan that moves more than the launches it replaces (its two kernels both read what a reduced value is
# made of, where a launch of its own would have written the value once).  y = u / |u|, u the sum of n fp32 tensors, replayed: 2048 x 4096, n 3, 34 MB more
# and two launches fewer, 38.3 us apart and 37.3 as a two-step plan; n 4, 67 MB more, 43.5 and 46.1; n 8, 201 MB more, 65 and 87; 1024 x 2048, n 8, 42 MB
# more and three launches fewer, 23.5 and 23.2; 512 x 2048, n 8, 20.1 and 11.0.
_BYTES_OF_A_LAUNCH = 20e6


class FusedProgram:
    """A whole computation graph run as the groups its fusion plan chose: one Plan per group, one per
    several small row groups that do not depend on each other, or one of two kernels for groups that pass scalars reduced
    over whole tensors on to ops on whole tensors; intermediates between launches in device
    tensors.  Inputs: one tensor per parameter op of the original list, in order; outputs: one per output op."""

    def __init__(self, ops, fusion=None, **fusion_options):
        import torch
        self._torch = torch
        self.ops = list(ops)
        self.fusion = fusion if fusion is not None else FusionPlan(self.ops, **fusion_options)
        self.param_ops = [i for i, op in enumerate(self.ops) if op.kind == "parameter"]
        self.output_ops = [i for i, op in enumerate(self.ops) if op.kind == "output"]
        self._plans = [None] * len(self.fusion.groups)      # per group; None: not built, the group runs in a launch with others
        self._packed_units = None
        self._levels()
        self._launches = self._pack(self._two_steps())
        self._build_single_plans()

    def _levels(self):
        """made_by: the group that makes a value; level: the length of the longest chain of groups a group depends on."""
        self._made_by, self._level = {}, []
        for k, g in enumerate(self.fusion.groups):
            self._level.append(1 + max((self._level[self._made_by[i]] for i in g["input_of"] if i in self._made_by), default=-1))
            for i in g["output_of"]:
                self._made_by[i] = k

    def _build_single_plans(self):
        for u in self._launches:
            if u.plan is None and self._plans[u.members[0]] is None:
                self._plans[u.members[0]] = self._group_plan(u.members[0])
        self._count_kernels()

    @property
    def plans(self):
        """Every group's own plan, in execution order.  That of a group that runs in a launch with others is built when it is asked for."""
        for k, plan in enumerate(self._plans):
            if plan is None:
                self._plans[k] = self._group_plan(k)
        return self._plans

    @property
    def _units(self):
        """The program as launches of groups and of packed groups: (packed plan or None, groups).  Where it has two-step plans instead,
        built when it is asked for."""
        if not any(u.extra for u in self._launches):
            return [(u.plan, u.members) for u in self._launches]
        if self._packed_units is None:
            self._packed_units = [(u.plan, u.members) for u in self._pack([])]
        return self._packed_units

    def _group_plan(self, k):
        try:
            return Plan(self.fusion.groups[k]["ops"])
        except FsError as e:
            if e.status != FS_ERR_UNSUPPORTED:
                raise
            return Plan(self.fusion.groups[k]["ops"], "per_op")   # an op left alone that no stitched schedule takes (a lone dot)

    def _two_steps(self):
        """Launches of two-step plans: a group that reads scalars other groups make, with all that makes them, where nothing else
        reads what is made on the way.  A group with recorded tuning options keeps its own plan; so does one whose two-step plan
        would move more bytes than the launches saved are worth."""
        groups, ops = self.fusion.groups, self.ops

        def nbytes(values):
            return sum(prod(ops[i].shape) * (4 if ops[i].dtype == "f32" else 2) for i in values)

        def leaves_below(i, leaves):
            seen, stack = set(), [i]
            while stack:
                k = stack.pop()
                if k not in seen:
                    seen.add(k)
                    if k not in leaves:
                        stack += ops[k].operands
            return seen & leaves

        used_by = {}
        for k, g in enumerate(groups):
            for i in g["input_of"]:
                used_by.setdefault(i, set()).add(k)
        returned = {ops[i].operands[0] for i in self.output_ops}
        taken, launches = set(), []
        tuned = fs_tune_cache_size() > 0
        for last, g in enumerate(groups):
            if all(ops[i].shape == () for i in g["output_of"]):
                continue                                   # (makes scalars itself)
            made = [i for i in g["input_of"] if ops[i].shape == () and i in self._made_by]
            members, stack = {last}, [self._made_by[i] for i in made]
            while stack:
                k = stack.pop()
                if k not in members:
                    members.add(k)
                    stack += [self._made_by[i] for i in groups[k]["input_of"] if i in self._made_by]
            if len(members) < 2 or members & taken:
                continue
            if any(used_by.get(i, set()) - members or i in returned for k in members - {last} for i in groups[k]["output_of"]):
                continue
            if tuned and any(fs_tune_cache_has(fs_group_key(groups[k]["ops"])) for k in members):
                continue
            outputs = list(g["output_of"])
            inside, leaves, stack = set(), set(), list(outputs)
            while stack:
                i = stack.pop()
                if i in inside or i in leaves:
                    continue
                if ops[i].kind == "parameter" or (i in self._made_by and self._made_by[i] not in members):
                    leaves.add(i)
                else:
                    inside.add(i)
                    stack += ops[i].operands
            # both kernels' reads and the outputs, against what goes in and out of the groups, in as many launches as they have levels
            more = nbytes(leaves) + sum(nbytes(leaves_below(i, leaves)) for i in inside if ops[i].kind in ("reduce_sum", "reduce_max") and ops[i].shape == ())
            more += nbytes(outputs) - sum(nbytes(groups[k]["input_of"]) + nbytes(groups[k]["output_of"]) for k in members)
            if more > (len({self._level[k] for k in members}) - 2) * _BYTES_OF_A_LAUNCH:
                continue
            inputs = sorted(leaves)
            number, listed = {}, []
            for i in inputs + sorted(inside):
                op = ops[i]
                number[i] = len(listed)
                if i in leaves:
                    listed.append(_OpRecord("parameter", op.dtype, op.shape, (), -1, 0.0))
                else:
                    listed.append(_OpRecord(op.kind, op.dtype, op.shape, tuple(number[o] for o in op.operands), op.axis, op.attr))
            for i in outputs:
                listed.append(_OpRecord("output", ops[i].dtype, ops[i].shape, (number[i],), -1, 0.0))
            try:
                plan, extra = Plan.two_step(listed)
            except FsError as e:
                if e.status not in (FS_ERR_UNSUPPORTED, FS_ERR_INVALID):      # (invalid: more inputs, outputs or ops than a list may have)
                    raise
                continue
            taken |= members
            launches.append(_Launch(plan, sorted(members), inputs, outputs, extra))
        return launches

    def _pack(self, two_steps):
        """The program's launches in order: groups sorted by their level, which leaves those of one level independent of each
        other; of a level, what can share a launch does.  A two-step plan runs at the level of its last group."""
        groups = self.fusion.groups
        inside = {k for u in two_steps for k in u.members}
        launches = []

        def add(plan, members):
            launches.append(_Launch(plan, members, [i for k in members for i in groups[k]["input_of"]],
                                    [i for k in members for i in groups[k]["output_of"]], 0))

        for lv in range(max(self._level, default=-1) + 1):
            left = [k for k in range(len(groups)) if self._level[k] == lv and k not in inside]
            while len(left) > 1:
                try:
                    plan, taken = Plan.packed([groups[k]["ops"] for k in left])
                except FsError as e:
                    if e.status != FS_ERR_UNSUPPORTED:
                        raise
                    break
                add(plan, [left[t] for t in taken])
                left = [k for t, k in enumerate(left) if t not in taken]
            for k in left:
                add(None, [k])
            launches += [u for u in two_steps if max(self._level[k] for k in u.members) == lv]
        return launches

    def _count_kernels(self):
        self.n_kernels = sum((u.plan or self._plans[u.members[0]]).info()["n_kernels"] for u in self._launches)

    def _launch_args(self, values, launch, device):
        """Inputs and freshly allocated outputs of a launch, in order."""
        torch = self._torch
        dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
        gin, gout = [values[i] for i in launch.inputs], []
        device = device or (gin[0].device if gin else "cuda:0")
        for i in launch.outputs:
            op = self.ops[i]
            values[i] = torch.empty(op.shape, dtype=dt[op.dtype], device=device)
            gout.append(values[i])
        if launch.extra:
            gout.append(torch.empty(launch.extra, dtype=torch.uint8, device=device))
        return gin, gout

    def run(self, inputs, stream=None):
        values = {i: t for i, t in zip(self.param_ops, inputs)}
        for u in self._launches:
            gin, gout = self._launch_args(values, u, None)
            (u.plan or self._plans[u.members[0]]).launch(gin, gout, stream)
        return [values[self.ops[i].operands[0]] for i in self.output_ops]

    @classmethod
    def best_of(cls, ops, inputs, option_sets=None, trials=20):
        """The execution-based side of Section 4.3 at the level of whole plans: build the program under
        each set of planning options, time it on the given inputs (HIP events, `trials` runs after two
        warm-ups), keep the fastest.  -> (program, microseconds per run, the winning options)."""
        import torch
        if option_sets is None:
            option_sets = [dict(), dict(explore_budget=-1), dict(seed_bytes=1), dict(launch_us=10.0), dict(launch_us=0.5)]
        best = None
        for kw in option_sets:
            prog = cls(ops, **kw)
            prog.bind(inputs)
            for _ in range(2):
                prog.run_bound()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(trials):
                prog.run_bound()
            e1.record()
            torch.cuda.synchronize()
            us = e0.elapsed_time(e1) * 1e3 / trials
            if best is None or us < best[1]:
                if best is not None:
                    best[0].close()
                best = (prog, us, dict(kw))
            else:
                prog.close()
        return best

    @classmethod
    def measured(cls, ops, top=12, trials=20, device="cuda:0", **fusion_options):
        """The hybrid scoring policy of Section 4.3.  Plan with the model's scores; build the plan's
        patterns and the `top` best other candidates, time each stitched and as one kernel per op on
        buffers of the right shapes (`trials` launches recorded and replayed, the medians of seven replays), and
        plan again with the measured savings in place of the model's for those patterns.  Groups are timed one by one: what
        sharing launches saves beyond that is not in the scores.
        -> (program, list of (pattern ops, model score, measured score))."""
        import torch
        ops = list(ops)
        dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
        first = FusionPlan(ops, **fusion_options)
        ranked = sorted((p for p in first.patterns if p["score_us"] >= 0 and "group_ops" in p),
                        key=lambda p: (not p["chosen"], -p["score_us"]))
        n_chosen = sum(1 for p in ranked if p["chosen"])
        picked = ranked[:n_chosen + top]

        def replayed(plan, bound):
            """`trials` launches of the plan, recorded after an ordinary one (kernel loaded, workspace allocated)."""
            plan.launch_bound(bound, _current_stream())
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
                for _ in range(trials):
                    plan.launch_bound(bound, _current_stream())
            return graph

        def timed(graph):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            graph.replay()
            e1.record()
            torch.cuda.synchronize()
            return e0.elapsed_time(e1) * 1e3 / trials

        def saving(apart, fused, bound):
            # Kernels and the gaps between them, as the device runs them: a replayed graph, since the host's share of a launch (4 to
            # 10 us on one machine within a minute, for one kernel or seventeen) would drown what patterns differ by.  Both in turn, medians.
            graphs = [replayed(apart, bound), replayed(fused, bound)]
            us = [[], []]
            for _ in range(7):
                for k, graph in enumerate(graphs):
                    us[k].append(timed(graph))
            return sorted(us[0])[3] - sorted(us[1])[3]

        report = []
        for p in picked:
            shapes = [(ops[i].shape, ops[i].dtype) for i in p["input_of"]]
            gin = [torch.randn(sh, dtype=torch.float32, device=device).to(dt[d]) for sh, d in shapes]
            gout = [torch.empty(ops[i].shape, dtype=dt[ops[i].dtype], device=device) for i in p["output_of"]]
            with Plan(p["group_ops"]) as fused, Plan(p["group_ops"], "per_op") as apart:
                saved = saving(apart, fused, BoundArgs(gin, gout))
            report.append((p["ops"], p["score_us"], saved))
        kw = dict(fusion_options)
        extra = list(kw.pop("extra_patterns", None) or [])
        scores = list(kw.pop("extra_scores", None) or [None] * len(extra))
        second = FusionPlan(ops, extra_patterns=extra + [r[0] for r in report], extra_scores=scores + [r[2] for r in report], **kw)
        return cls(ops, fusion=second), report

    def tune(self, inputs, trials=10):
        """Time every group's launch templates on the program's own data (fs_plan_tune, group by group in
        execution order) and keep the winners; every group is then a launch of its own.  -> the program's
        outputs, as run() would return them."""
        torch = self._torch
        plans = self.plans
        self._close_shared()
        self._launches = [_Launch(None, [k], g["input_of"], g["output_of"], 0) for k, g in enumerate(self.fusion.groups)]
        dt = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
        values = {i: t for i, t in zip(self.param_ops, inputs)}
        for k, g in enumerate(self.fusion.groups):
            gin = [values[i] for i in g["input_of"]]
            gout = []
            for i in g["output_of"]:
                op = self.ops[i]
                values[i] = torch.empty(op.shape, dtype=dt[op.dtype], device=gin[0].device if gin else "cuda:0")
                gout.append(values[i])
            if plans[k].info()["schedule"] == "per_op":
                plans[k].launch(gin, gout)
                continue
            tuned = Plan.tune(g["ops"], gin, gout, trials=trials)      # leaves the group's outputs written
            plans[k].close()
            plans[k] = tuned
        self._count_kernels()
        return [values[self.ops[i].operands[0]] for i in self.output_ops]

    def bind(self, inputs):
        """Fix the program's buffers: the given input tensors, and one freshly allocated tensor per value
        that crosses a group boundary.  -> the output tensors; run_bound() then launches every group on
        those buffers without allocating, which is what a HIP graph capture needs."""
        values = {i: t for i, t in zip(self.param_ops, inputs)}
        device = inputs[0].device if inputs else "cuda:0"
        self._bound = []
        for u in self._launches:
            gin, gout = self._launch_args(values, u, device)
            self._bound.append((u.plan or self._plans[u.members[0]], BoundArgs(gin, gout)))
        self._bound_outputs = [values[self.ops[i].operands[0]] for i in self.output_ops]
        return self._bound_outputs

    def run_bound(self, stream=None):
        if stream is None:
            stream = _current_stream()
        for plan, args in self._bound:
            plan.launch_bound(args, stream)
        return self._bound_outputs

    def capture(self, inputs):
        """bind(inputs), one ordinary run (kernels loaded, workspaces allocated), then the same launches
        recorded into a HIP graph.  -> (graph, outputs): graph.replay() recomputes the outputs from whatever
        the input tensors hold then."""
        torch = self._torch
        outs = self.bind(inputs)
        self.run_bound()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            self.run_bound()
        return graph, outs

    def _close_shared(self):
        """The plans that run more than one group."""
        for p in [u.plan for u in self._launches] + [plan for plan, _ in self._packed_units or []]:
            if p is not None:
                p.close()
        self._launches, self._packed_units = [], None

    def close(self):
        for p in self._plans:
            if p is not None:
                p.close()
        self._close_shared()
        self._plans = []
        self._bound = []

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        self.close()
