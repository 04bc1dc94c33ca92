"""ctypes marshalling for libalt.so, with a native module for the calls that programs repeat.  Function names follow include/alt.h."""
import ctypes
import os
import struct

try:
    from . import _altcall as _native
except ImportError:                       # built where Python's headers are (build.py)
    _native = None

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIBPATH = os.environ.get("ALT_LIBRARY", os.path.join(_HERE, "libalt.so"))   # ALT_LIBRARY: developer builds

F32, BF16 = 0, 1
EPI_BIAS, EPI_RELU = 1, 2
MAX_RANK, MAX_PRIMS, MAX_CAND, MAX_CHAIN = 8, 8, 16, 8

_STATUS = ["ok", "invalid argument", "invalid layout", "shape mismatch", "unsupported",
           "workspace too small", "HIP error", "not tuned"]


class AltError(RuntimeError):
    def __init__(self, status, msg=""):
        self.status = status
        name = _STATUS[status] if 0 <= status < len(_STATUS) else str(status)
        super().__init__("%s%s" % (name, (": " + msg) if msg else ""))


class Prim(ctypes.Structure):
    _fields_ = [("kind", ctypes.c_int32), ("dim", ctypes.c_int32), ("count", ctypes.c_int32),
                ("reserved", ctypes.c_int32), ("v", ctypes.c_int64 * MAX_RANK)]


def split(dim, factors):
    p = Prim(0, dim, len(factors), 0)
    for i, f in enumerate(factors):
        p.v[i] = f
    return p


def reorder(perm):
    p = Prim(1, 0, len(perm), 0)
    for i, f in enumerate(perm):
        p.v[i] = f
    return p


def fuse(dim, count):
    return Prim(2, dim, count, 0)


class Layout(ctypes.Structure):
    _fields_ = [("ndim", ctypes.c_int32), ("nsub", ctypes.c_int32), ("separable", ctypes.c_int32),
                ("nprims", ctypes.c_int32),
                ("sub_dim", ctypes.c_int32 * MAX_RANK), ("sub_group", ctypes.c_int32 * MAX_RANK),
                ("sub_div", ctypes.c_int64 * MAX_RANK), ("sub_extent", ctypes.c_int64 * MAX_RANK),
                ("shape", ctypes.c_int64 * MAX_RANK), ("prims", Prim * MAX_PRIMS)]


class ConvDesc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("N", "C", "H", "W", "K", "R", "S")] + \
               [(n, ctypes.c_int32) for n in ("stride_h", "stride_w", "pad_h", "pad_w", "dil_h", "dil_w",
                                              "in_dtype", "out_dtype", "epilogue", "variant")] + \
               [("x_layout", Layout), ("w_layout", Layout), ("y_layout", Layout),
                ("groups", ctypes.c_int32), ("reserved", ctypes.c_int32)]


class Conv3dDesc(ctypes.Structure):
    _fields_ = [("plane", ConvDesc), ("D", ctypes.c_int64), ("T", ctypes.c_int64),
                ("stride_d", ctypes.c_int32), ("pad_d", ctypes.c_int32), ("dil_d", ctypes.c_int32),
                ("reserved", ctypes.c_int32)]


class GemmDesc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int64) for n in ("batch", "M", "N", "K")] + \
               [(n, ctypes.c_int32) for n in ("in_dtype", "out_dtype", "variant", "reserved")] + \
               [("a_layout", Layout), ("b_layout", Layout), ("c_layout", Layout)]


class TuneOpts(ctypes.Structure):
    _fields_ = [("max_trials", ctypes.c_int32), ("warmup", ctypes.c_int32), ("reps", ctypes.c_int32),
                ("layout_mask", ctypes.c_int32), ("arena", ctypes.c_void_p),
                ("arena_bytes", ctypes.c_size_t), ("stream", ctypes.c_void_p)]


class TuneReport(ctypes.Structure):
    _fields_ = [("trials", ctypes.c_int32), ("n_layouts", ctypes.c_int32),
                ("best_us", ctypes.c_float), ("default_us", ctypes.c_float),
                ("layout_best_us", ctypes.c_float * MAX_CAND),
                ("layout_best_variant", ctypes.c_int32 * MAX_CAND),
                ("layout_name", (ctypes.c_char * 48) * MAX_CAND)]


class ChainPlan(ctypes.Structure):
    _fields_ = [("nops", ctypes.c_int32), ("trials", ctypes.c_int32),
                ("op", ConvDesc * MAX_CHAIN), ("transform_before", ctypes.c_int32 * MAX_CHAIN),
                ("edge_layout", Layout * (MAX_CHAIN + 1)),
                ("op_us", ctypes.c_float * MAX_CHAIN), ("transform_us", ctypes.c_float * MAX_CHAIN),
                ("total_us", ctypes.c_float), ("default_total_us", ctypes.c_float)]


class ConvCall(ctypes.Structure):
    _fields_ = [("d", ctypes.POINTER(ConvDesc)), ("x", ctypes.c_void_p), ("w", ctypes.c_void_p),
                ("bias", ctypes.c_void_p), ("y", ctypes.c_void_p), ("workspace", ctypes.c_void_p),
                ("ws_bytes", ctypes.c_size_t), ("stream", ctypes.c_void_p)]


MAX_GRAPH = 8
NODE_CONV, NODE_ADD = 0, 1


class GraphNode(ctypes.Structure):
    _fields_ = [("kind", ctypes.c_int32), ("in0", ctypes.c_int32), ("in1", ctypes.c_int32),
                ("relu", ctypes.c_int32), ("conv", ConvDesc)]


class GraphPlan(ctypes.Structure):
    _fields_ = [("nnodes", ctypes.c_int32), ("trials", ctypes.c_int32),
                ("conv", ConvDesc * MAX_GRAPH), ("tensor_layout", Layout * (MAX_GRAPH + 1)),
                ("read_layout", (Layout * 2) * MAX_GRAPH), ("convert", (ctypes.c_int32 * 2) * MAX_GRAPH),
                ("convert_us", (ctypes.c_float * 2) * MAX_GRAPH), ("node_us", ctypes.c_float * MAX_GRAPH),
                ("total_us", ctypes.c_float), ("default_total_us", ctypes.c_float),
                ("fused_into", ctypes.c_int32 * MAX_GRAPH)]


class MultiPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("launch", "family", "body", "slices", "kept")]


class TransformPlan(ctypes.Structure):
    _fields_ = [("kind", ctypes.c_int32), ("src_flat", ctypes.c_int32), ("dst_flat", ctypes.c_int32),
                ("load_bytes", ctypes.c_int32), ("store_bytes", ctypes.c_int32),
                ("tile_a", ctypes.c_int32), ("tile_b", ctypes.c_int32), ("tile_g", ctypes.c_int32),
                ("workgroups", ctypes.c_int64), ("lds_bytes", ctypes.c_int64), ("mismatches", ctypes.c_int64)]


class SplitkStatus(ctypes.Structure):
    _fields_ = [("streams_bound", ctypes.c_int32), ("max_streams", ctypes.c_int32), ("counters_nonzero", ctypes.c_int32)]


class Peaks(ctypes.Structure):
    _fields_ = [("copy_gbps", ctypes.c_float), ("mfma_bf16_tflops", ctypes.c_float),
                ("nominal_hbm_gbps", ctypes.c_float), ("nominal_bf16_tflops", ctypes.c_float),
                ("compute_units", ctypes.c_int32), ("clock_mhz", ctypes.c_int32),
                ("arch", ctypes.c_char * 32), ("read_gbps", ctypes.c_float), ("write_gbps", ctypes.c_float)]


_lib = None


def library_path():
    return _LIBPATH


def lib():
    """Loads libalt.so; raises if it has not been built (python -m
    paper_2210_12415_amd.build)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIBPATH):
            raise AltError(6, "libalt.so is not built: run python -m paper_2210_12415_amd.build")
        L = ctypes.CDLL(_LIBPATH)
        L.alt_last_error.restype = ctypes.c_char_p
        L.alt_status_string.restype = ctypes.c_char_p
        L.alt_version.restype = ctypes.c_char_p
        if _native is not None:
            _native.setup(*[ctypes.cast(getattr(L, n), ctypes.c_void_p).value for n in _REPEATED],
                          ctypes.c_void_p, ConvDesc, Conv3dDesc, GemmDesc, Layout)
        _lib = L
    return _lib


# The calls a program repeats, with prototypes of their own: addresses go through as plain integers, not each wrapped in an object, and
# the current stream is asked for by its address.  Host time set short calls: nine conversions of 4 to 7 us on the device took 66 us, and
# 45 so; four products of one short sequence 29 us, 25 so.
_V, _I, _L = ctypes.c_void_p, ctypes.c_int, ctypes.c_int64
_OPERATOR = (_V, _V, _V, _V, _V, _V, _V, ctypes.c_size_t, _V)
_PROTOTYPES = {"alt_layout_transform": (_V, _I, _I, _V, _V, _V, _V, _V, _V), "alt_eltwise_add": (_V, _I, _L, _V, _V, _V, _I, _V),
               "alt_gemm": (_V, _V, _V, _V, _V, _V, ctypes.c_size_t, _V), "alt_conv2d": _OPERATOR, "alt_conv3d": _OPERATOR,
               "alt_conv2d_transpose": _OPERATOR, "alt_conv3d_transpose": _OPERATOR}
_calls = {}

# The same calls by the native module (native/altcall.c), for arguments of plain types; it answers None to others, and without the module
# everything is another.  (A conversion's arguments took 1.8 us through ctypes, beside 3.5 for the launch.)
_REPEATED = ("alt_conv2d", "alt_conv3d", "alt_conv2d_transpose", "alt_conv3d_transpose", "alt_gemm", "alt_layout_transform", "alt_eltwise_add")


def _not_taken(*_):
    return None


def _quick(name):
    return getattr(_native, name) if _native is not None else _not_taken


_quick_conv2d, _quick_conv3d = _quick("conv2d"), _quick("conv3d")
_quick_conv2d_transpose, _quick_conv3d_transpose = _quick("conv2d_transpose"), _quick("conv3d_transpose")
_quick_gemm, _quick_transform, _quick_add, _quick_prepare = _quick("gemm"), _quick("layout_transform"), _quick("eltwise_add"), _quick("prepare_conv2d")


def _call(name):
    fn = _calls.get(name)
    if fn is None:
        fn = _calls[name] = ctypes.CFUNCTYPE(ctypes.c_int, *_PROTOTYPES[name])((name, lib()))
    return fn


def exported_symbols():
    """Names declared in include/alt.h that the binding expects to find."""
    return ["alt_create", "alt_destroy", "alt_last_error", "alt_status_string", "alt_version",
            "alt_layout_parse", "alt_layout_from_prims", "alt_layout_physical_shape",
            "alt_layout_offset", "alt_layout_index_of", "alt_layout_transform",
            "alt_conv2d", "alt_conv2d_add", "alt_conv2d_multi", "alt_conv2d_multi_plan", "alt_conv2d_transpose", "alt_conv2d_transpose_workspace_size",
            "alt_conv2d_transpose_output_shape", "alt_conv2d_transpose_weight_shape", "alt_pack_weights_transpose",
            "alt_conv3d", "alt_conv3d_workspace_size", "alt_conv3d_output_shape", "alt_pack_weights3d",
            "alt_conv3d_transpose", "alt_conv3d_transpose_workspace_size", "alt_conv3d_transpose_output_shape",
            "alt_pack_weights3d_transpose", "alt_conv2d_transpose_problem", "alt_conv3d_problem", "alt_conv3d_transpose_problem", "alt_conv3d_transpose_weight_shape", "alt_conv2d_workspace_size", "alt_conv2d_output_shape", "alt_pack_weights",
            "alt_conv2d_variant_count", "alt_conv2d_variant_name",
            "alt_gemm", "alt_gemm_workspace_size", "alt_gemm_variant_count", "alt_gemm_variant_name",
            "alt_tune_conv2d_arena_size", "alt_tune_gemm_arena_size", "alt_tune_conv2d", "alt_tune_gemm",
            "alt_tune_conv2d_variants", "alt_tune_conv2d_multi", "alt_tune_chain", "alt_plan_chain",
            "alt_eltwise_add", "alt_tune_graph", "alt_plan_graph", "alt_unfold", "alt_unfold_shape",
            "alt_cache_save", "alt_cache_load", "alt_cache_clear", "alt_get_peak", "alt_layout_transform_plan", "alt_splitk_status", "alt_conv2d_static", "alt_layout_transform_pad"]


def version():
    return lib().alt_version().decode()


def _i64(a):
    return (ctypes.c_int64 * len(a))(*[int(x) for x in a])


def _ck(status, h=None):
    if status != 0:
        msg = lib().alt_last_error(h).decode() if h else ""
        raise AltError(status, msg)


def _ptr(x):
    """Device pointer of a torch tensor, or the integer itself."""
    if x is None:
        return None
    if hasattr(x, "data_ptr"):
        return ctypes.c_void_p(x.data_ptr())
    return ctypes.c_void_p(int(x))


def _stream(s):
    if s is None:
        import torch
        return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    if hasattr(s, "cuda_stream"):
        return ctypes.c_void_p(s.cuda_stream)
    return ctypes.c_void_p(int(s))


def _address(x):
    """_ptr as a plain integer (or None)."""
    try:
        return x.data_ptr()
    except AttributeError:
        return None if x is None else int(x)


_raw_stream = None


def _stream_address(s):
    """_stream as a plain integer.  The current stream is asked for by its address where torch offers that: making the Stream object
    first takes 2 us."""
    global _raw_stream
    if s is None:
        import torch
        if not torch.cuda.is_initialized():
            return torch.cuda.current_stream().cuda_stream
        if _raw_stream is None:
            c = torch._C
            if hasattr(c, "_cuda_getCurrentRawStream") and hasattr(c, "_cuda_getDevice"):
                _raw_stream = lambda: c._cuda_getCurrentRawStream(c._cuda_getDevice())
                if _native is not None:
                    _native.streams(c._cuda_getCurrentRawStream, c._cuda_getDevice)
            else:
                _raw_stream = lambda: torch.cuda.current_stream().cuda_stream
        return _raw_stream()
    try:
        return s.cuda_stream
    except AttributeError:
        return int(s)


_packers = {}


def _extents(a):
    """_i64 as packed bytes, which take half as long to make; what is no whole number of 64 bits is converted there."""
    n = len(a)
    pack = _packers.get(n)
    if pack is None:
        pack = _packers[n] = struct.Struct("=%dq" % n).pack
    try:
        return pack(*a)
    except struct.error:
        return _i64(a)


# What a prototype is given: an int goes through as it is; anything else (a numpy integer, None, an object of ctypes, what is no number at all)
# takes the call without prototypes, which decides as ever what it accepts and what it raises.
_CODES = frozenset(range(256))


# ------------------------------------------------------------- layouts (host) ----

def layout_parse(text):
    out = Layout()
    _ck(lib().alt_layout_parse(text.encode(), ctypes.byref(out)))
    return out


def layout_from_prims(shape, seq):
    out = Layout()
    arr = (Prim * max(1, len(seq)))(*seq)
    _ck(lib().alt_layout_from_prims(len(shape), _i64(shape), arr, len(seq), ctypes.byref(out)))
    return out


def _as_layout(l):
    return layout_parse(l) if isinstance(l, str) else l


def layout_physical_shape(layout, shape):
    out = (ctypes.c_int64 * MAX_RANK)()
    rank = ctypes.c_int()
    _ck(lib().alt_layout_physical_shape(ctypes.byref(_as_layout(layout)), _i64(shape), out, ctypes.byref(rank)))
    return tuple(out[i] for i in range(rank.value))


def layout_offset(layout, shape, idx):
    off = ctypes.c_int64()
    _ck(lib().alt_layout_offset(ctypes.byref(_as_layout(layout)), _i64(shape), _i64(idx), ctypes.byref(off)))
    return off.value


def layout_index_of(layout, shape, offset):
    out = (ctypes.c_int64 * MAX_RANK)()
    _ck(lib().alt_layout_index_of(ctypes.byref(_as_layout(layout)), _i64(shape), ctypes.c_int64(offset), out))
    return tuple(out[i] for i in range(len(shape)))


def plan_chain(op_cost, conv_cost, in_layout):
    """op_cost, conv_cost: nested lists [nops][nl][nl] of latencies."""
    nops, nl = len(op_cost), len(op_cost[0])
    flat = lambda c: (ctypes.c_float * (nops * nl * nl))(*[float(v) for o in c for r in o for v in r])
    ins, outs = (ctypes.c_int * nops)(), (ctypes.c_int * nops)()
    total = ctypes.c_float()
    _ck(lib().alt_plan_chain(nops, nl, flat(op_cost), flat(conv_cost), in_layout, ins, outs, ctypes.byref(total)))
    return list(ins), list(outs), total.value


def unfold_shape(shape, dim, B, S):
    out = (ctypes.c_int64 * (len(shape) + 1))()
    _ck(lib().alt_unfold_shape(len(shape), _i64(shape), dim, ctypes.c_int64(B), ctypes.c_int64(S), out))
    return tuple(out)


def plan_graph(kind, in0, in1, op_cost, conv_cost, add_cost, in_layout):
    """kind/in0/in1: per node; op_cost [nnodes][nl][nl], conv_cost [nnodes+1][nl][nl],
    add_cost [nnodes].  Returns (stored layout per tensor, read layouts per node, total)."""
    n, nl = len(kind), len(op_cost[0])
    i32 = lambda a: (ctypes.c_int32 * len(a))(*[int(v) for v in a])
    flat = lambda c, m: (ctypes.c_float * (m * nl * nl))(*[float(v) for o in c for r in o for v in r])
    tl, rl = (ctypes.c_int32 * (n + 1))(), (ctypes.c_int32 * (2 * n))()
    total = ctypes.c_float()
    _ck(lib().alt_plan_graph(n, i32(kind), i32(in0), i32(in1), nl, flat(op_cost, n), flat(conv_cost, n + 1),
                             (ctypes.c_float * n)(*[float(v) for v in add_cost]), in_layout, tl, rl,
                             ctypes.byref(total)))
    return list(tl), [list(rl[2 * i:2 * i + 2]) for i in range(n)], total.value


def graph_node(kind, in0, in1=0, relu=0, conv=None):
    nd = GraphNode(kind, in0, in1, relu)
    if conv is not None:
        nd.conv = conv
    return nd


# ------------------------------------------------------------------ descriptors ----

def conv_desc(N, C, H, W, K, R, S, stride=1, pad=0, dil=1, in_dtype=BF16, out_dtype=F32,
              epilogue=0, variant=-1, x_layout="NCHW->NCHW", w_layout="OIHW->OIHW",
              y_layout="NCHW->NCHW", groups=1):
    d = ConvDesc(N, C, H, W, K, R, S, stride, stride, pad, pad, dil, dil, in_dtype, out_dtype,
                 epilogue, variant)
    d.x_layout, d.w_layout, d.y_layout = _as_layout(x_layout), _as_layout(w_layout), _as_layout(y_layout)
    d.groups = groups
    return d


def _triple(v):
    return tuple(v) if isinstance(v, (tuple, list)) else (v, v, v)


def conv3d_desc(N, C, D, H, W, K, T, R, S, stride=1, pad=0, dil=1, **plane):
    """stride, pad, dil: one number or (depth, height, width); the rest as conv_desc."""
    (sd, sh, sw), (pd, ph, pw), (dd, dh, dw) = _triple(stride), _triple(pad), _triple(dil)
    q = conv_desc(N, C, H, W, K, R, S, **plane)
    q.stride_h, q.stride_w, q.pad_h, q.pad_w, q.dil_h, q.dil_w = sh, sw, ph, pw, dh, dw
    return Conv3dDesc(q, D, T, sd, pd, dd, 0)


def gemm_desc(M, N, K, batch=1, in_dtype=BF16, out_dtype=F32, variant=-1,
              a_layout="MK->MK", b_layout="KN->KN", c_layout="MN->MN"):
    d = GemmDesc(batch, M, N, K, in_dtype, out_dtype, variant, 0)
    d.a_layout, d.b_layout, d.c_layout = _as_layout(a_layout), _as_layout(b_layout), _as_layout(c_layout)
    return d


# ----------------------------------------------------------------------- handle ----

class Handle:
    """One library handle on the current device."""

    def __init__(self):
        self._h = ctypes.c_void_p()
        _ck(lib().alt_create(ctypes.byref(self._h)))

    def close(self):
        if self._h:
            h = ctypes.c_void_p(self._h.value)
            self._h.value = None              # in place: calls prepared with it find no handle
            lib().alt_destroy(h)

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def last_error(self):
        return lib().alt_last_error(self._h).decode()

    def layout_transform(self, dtype, shape, src_layout, src, dst_layout, dst, stream=None):
        status = _quick_transform(self._h, dtype, shape, src_layout, src, dst_layout, dst, stream)
        if status is not None:
            pass
        elif dtype.__class__ is int and dtype in _CODES:
            status = _call("alt_layout_transform")(self._h, dtype, len(shape), _extents(shape),
                                                   ctypes.byref(_as_layout(src_layout)), _address(src),
                                                   ctypes.byref(_as_layout(dst_layout)), _address(dst), _stream_address(stream))
        else:
            status = lib().alt_layout_transform(self._h, dtype, len(shape), _i64(shape),
                                                ctypes.byref(_as_layout(src_layout)), _ptr(src),
                                                ctypes.byref(_as_layout(dst_layout)), _ptr(dst), _stream(stream))
        if status != 0:
            _ck(status, self._h)

    def layout_transform_plan(self, dtype, shape, src_layout, dst_layout, src_misalign=0, dst_misalign=0, replay=False):
        out = TransformPlan()
        _ck(lib().alt_layout_transform_plan(self._h, dtype, len(shape), _i64(shape), ctypes.byref(_as_layout(src_layout)),
                                            int(src_misalign), ctypes.byref(_as_layout(dst_layout)), int(dst_misalign),
                                            int(bool(replay)), ctypes.byref(out)), self._h)
        return out

    def _operator(self, name, d, x, w, bias, y, workspace, ws_bytes, stream):
        if ws_bytes.__class__ is not int:
            ws_bytes = ctypes.c_size_t(ws_bytes).value
        status = _call(name)(self._h, ctypes.byref(d), _address(x), _address(w), _address(bias), _address(y), _address(workspace),
                             ws_bytes, _stream_address(stream))
        if status != 0:
            _ck(status, self._h)

    # conv
    def conv2d(self, d, x, w, y, bias=None, workspace=None, ws_bytes=0, stream=None):
        status = _quick_conv2d(self._h, d, x, w, bias, y, workspace, ws_bytes, stream)
        if status is None:
            self._operator("alt_conv2d", d, x, w, bias, y, workspace, ws_bytes, stream)
        elif status != 0:
            _ck(status, self._h)

    def conv2d_static(self, d, x, w, y, bias=None, stream=None):
        _ck(lib().alt_conv2d_static(self._h, ctypes.byref(d), _ptr(x), _ptr(w), _ptr(bias), _ptr(y), _stream(stream)), self._h)

    def conv2d_add(self, d, x, w, addend, y, bias=None, workspace=None, ws_bytes=0, stream=None):
        _ck(lib().alt_conv2d_add(self._h, ctypes.byref(d), _ptr(x), _ptr(w), _ptr(bias), _ptr(addend), _ptr(y),
                                 _ptr(workspace), ctypes.c_size_t(ws_bytes), _stream(stream)), self._h)

    def conv2d_prepared(self, d, x, w, y, bias=None, workspace=None, ws_bytes=0, stream=None):
        """The same call as conv2d with its arguments marshalled once: returns a
        function of no arguments that launches it (for loops that repeat one call)."""
        call = _quick_prepare(self._h, d, x, w, bias, y, workspace, ws_bytes, stream, _ck, self)
        if call is not None:
            return call
        fn = _call("alt_conv2d")
        ws_bytes = ctypes.c_size_t(ws_bytes).value
        args = (self._h, ctypes.byref(d), _address(x), _address(w), _address(bias), _address(y), _address(workspace),
                ws_bytes, _stream_address(stream))
        keep = (self, d, x, w, y, bias, workspace)

        def run():
            status = fn(*args)
            if status != 0:
                _ck(status, self._h)
            return keep is None
        return run

    @staticmethod
    def _call_array(calls):
        n = len(calls)
        arr = (ConvCall * n)()
        for i, c in enumerate(calls):
            arr[i].d = ctypes.pointer(c["d"])
            for k in ("x", "w", "bias", "y", "workspace"):
                setattr(arr[i], k, _ptr(c.get(k)))
            arr[i].ws_bytes = int(c.get("ws_bytes", 0))
            arr[i].stream = _stream(c.get("stream"))
        return arr

    def conv2d_multi_prepared(self, calls):
        """alt_conv2d_multi over `calls`, a list of dicts with the keyword arguments of
        conv2d (d, x, w, y and optionally bias, workspace, ws_bytes, stream), marshalled
        once: returns a function of no arguments that issues them all, and keeps the Handle and the arguments."""
        n = len(calls)
        arr = self._call_array(calls)
        keep = (self, [tuple(c.values()) for c in calls])
        fn, hh, nn = lib().alt_conv2d_multi, self._h, ctypes.c_int32(n)

        def run():
            status = fn(hh, arr, nn)
            if status != 0:
                _ck(status, hh)
            return keep is None
        return run

    def layout_transform_pad(self, dtype, src_shape, src_layout, src, dst_shape, dst_layout, dst, stream=None):
        _ck(lib().alt_layout_transform_pad(self._h, dtype, len(src_shape), _i64(src_shape),
                                           ctypes.byref(_as_layout(src_layout)), _ptr(src), _i64(dst_shape),
                                           ctypes.byref(_as_layout(dst_layout)), _ptr(dst), _stream(stream)), self._h)

    def conv2d_multi(self, calls):
        self.conv2d_multi_prepared(calls)()

    def conv2d_multi_plan(self, calls):
        """How conv2d_multi issues `calls`: a MultiPlan for each (host only)."""
        out = (MultiPlan * len(calls))()
        _ck(lib().alt_conv2d_multi_plan(self._h, self._call_array(calls), ctypes.c_int32(len(calls)), out), self._h)
        return list(out)

    def conv2d_workspace_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_conv2d_workspace_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def conv2d_output_shape(self, d):
        out = (ctypes.c_int64 * 4)()
        _ck(lib().alt_conv2d_output_shape(ctypes.byref(d), out))
        return tuple(out)

    def conv2d_transpose(self, d, x, w, y, bias=None, workspace=None, ws_bytes=0, stream=None):
        status = _quick_conv2d_transpose(self._h, d, x, w, bias, y, workspace, ws_bytes, stream)
        if status is None:
            self._operator("alt_conv2d_transpose", d, x, w, bias, y, workspace, ws_bytes, stream)
        elif status != 0:
            _ck(status, self._h)

    def conv2d_transpose_workspace_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_conv2d_transpose_workspace_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def conv2d_transpose_output_shape(self, d):
        out = (ctypes.c_int64 * 4)()
        _ck(lib().alt_conv2d_transpose_output_shape(ctypes.byref(d), out))
        return tuple(out)

    def conv2d_transpose_problem(self, d):
        out = ConvDesc()
        _ck(lib().alt_conv2d_transpose_problem(self._h, ctypes.byref(d), ctypes.byref(out)), self._h)
        return out

    def conv3d_problem(self, d):
        out = ConvDesc()
        _ck(lib().alt_conv3d_problem(self._h, ctypes.byref(d), ctypes.byref(out)), self._h)
        return out

    def conv3d_transpose_problem(self, d):
        out = ConvDesc()
        _ck(lib().alt_conv3d_transpose_problem(self._h, ctypes.byref(d), ctypes.byref(out)), self._h)
        return out

    def conv3d_transpose_weight_shape(self, d):
        out = (ctypes.c_int64 * 4)()
        _ck(lib().alt_conv3d_transpose_weight_shape(self._h, ctypes.byref(d), out), self._h)
        return tuple(out)

    def conv2d_transpose_weight_shape(self, d):
        out = (ctypes.c_int64 * 4)()
        _ck(lib().alt_conv2d_transpose_weight_shape(ctypes.byref(d), out))
        return tuple(out)

    def pack_weights_transpose(self, d, w_ckrs, w_packed, stream=None):
        _ck(lib().alt_pack_weights_transpose(self._h, ctypes.byref(d), _ptr(w_ckrs), _ptr(w_packed),
                                             _stream(stream)), self._h)

    def conv3d(self, d, x, w, y, bias=None, workspace=None, ws_bytes=0, stream=None):
        status = _quick_conv3d(self._h, d, x, w, bias, y, workspace, ws_bytes, stream)
        if status is None:
            self._operator("alt_conv3d", d, x, w, bias, y, workspace, ws_bytes, stream)
        elif status != 0:
            _ck(status, self._h)

    def conv3d_workspace_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_conv3d_workspace_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def conv3d_output_shape(self, d):
        out = (ctypes.c_int64 * 5)()
        _ck(lib().alt_conv3d_output_shape(ctypes.byref(d), out))
        return tuple(out)

    def pack_weights3d(self, d, w_kctrs, w_packed, stream=None):
        _ck(lib().alt_pack_weights3d(self._h, ctypes.byref(d), _ptr(w_kctrs), _ptr(w_packed),
                                     _stream(stream)), self._h)

    def conv3d_transpose(self, d, x, w, y, bias=None, workspace=None, ws_bytes=0, stream=None):
        status = _quick_conv3d_transpose(self._h, d, x, w, bias, y, workspace, ws_bytes, stream)
        if status is None:
            self._operator("alt_conv3d_transpose", d, x, w, bias, y, workspace, ws_bytes, stream)
        elif status != 0:
            _ck(status, self._h)

    def conv3d_transpose_workspace_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_conv3d_transpose_workspace_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def conv3d_transpose_output_shape(self, d):
        out = (ctypes.c_int64 * 5)()
        _ck(lib().alt_conv3d_transpose_output_shape(ctypes.byref(d), out))
        return tuple(out)

    def pack_weights3d_transpose(self, d, w_cktrs, w_packed, stream=None):
        _ck(lib().alt_pack_weights3d_transpose(self._h, ctypes.byref(d), _ptr(w_cktrs), _ptr(w_packed),
                                               _stream(stream)), self._h)

    def pack_weights(self, d, w_oihw, w_packed, stream=None):
        _ck(lib().alt_pack_weights(self._h, ctypes.byref(d), _ptr(w_oihw), _ptr(w_packed),
                                   _stream(stream)), self._h)

    def conv2d_variant_count(self, d):
        n = ctypes.c_int()
        _ck(lib().alt_conv2d_variant_count(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def conv2d_variant_name(self, d, variant):
        buf = ctypes.create_string_buffer(96)
        _ck(lib().alt_conv2d_variant_name(self._h, ctypes.byref(d), variant, buf, ctypes.c_size_t(96)), self._h)
        return buf.value.decode()

    # gemm
    def gemm(self, d, A, B, C, workspace=None, ws_bytes=0, stream=None):
        status = _quick_gemm(self._h, d, A, B, C, workspace, ws_bytes, stream)
        if status is not None:
            if status != 0:
                _ck(status, self._h)
            return
        if ws_bytes.__class__ is not int:
            ws_bytes = ctypes.c_size_t(ws_bytes).value
        status = _call("alt_gemm")(self._h, ctypes.byref(d), _address(A), _address(B), _address(C), _address(workspace),
                                   ws_bytes, _stream_address(stream))
        if status != 0:
            _ck(status, self._h)

    def gemm_workspace_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_gemm_workspace_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def gemm_variant_count(self, d):
        n = ctypes.c_int()
        _ck(lib().alt_gemm_variant_count(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def gemm_variant_name(self, d, variant):
        buf = ctypes.create_string_buffer(96)
        _ck(lib().alt_gemm_variant_name(self._h, ctypes.byref(d), variant, buf, ctypes.c_size_t(96)), self._h)
        return buf.value.decode()

    # tuning
    def _opts(self, arena, arena_bytes, max_trials, warmup, reps, layout_mask, stream):
        return TuneOpts(max_trials, warmup, reps, layout_mask, _ptr(arena), arena_bytes, _stream(stream))

    def tune_conv2d_arena_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_tune_conv2d_arena_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def tune_gemm_arena_size(self, d):
        n = ctypes.c_size_t()
        _ck(lib().alt_tune_gemm_arena_size(self._h, ctypes.byref(d), ctypes.byref(n)), self._h)
        return n.value

    def tune_conv2d(self, d, arena, arena_bytes, max_trials=0, warmup=3, reps=20, layout_mask=0, stream=None):
        best, rep = ConvDesc(), TuneReport()
        o = self._opts(arena, arena_bytes, max_trials, warmup, reps, layout_mask, stream)
        _ck(lib().alt_tune_conv2d(self._h, ctypes.byref(d), ctypes.byref(o), ctypes.byref(best),
                                  ctypes.byref(rep)), self._h)
        return best, rep

    def tune_gemm(self, d, arena, arena_bytes, max_trials=0, warmup=3, reps=20, layout_mask=0, stream=None):
        best, rep = GemmDesc(), TuneReport()
        o = self._opts(arena, arena_bytes, max_trials, warmup, reps, layout_mask, stream)
        _ck(lib().alt_tune_gemm(self._h, ctypes.byref(d), ctypes.byref(o), ctypes.byref(best),
                                ctypes.byref(rep)), self._h)
        return best, rep

    def tune_conv2d_variants(self, d, arena, arena_bytes, max_trials=0, warmup=3, reps=20, stream=None):
        us, trials = ctypes.c_float(), ctypes.c_int()
        o = self._opts(arena, arena_bytes, max_trials, warmup, reps, 0, stream)
        _ck(lib().alt_tune_conv2d_variants(self._h, ctypes.byref(d), ctypes.byref(o), ctypes.byref(us),
                                           ctypes.byref(trials)), self._h)
        return us.value, trials.value

    def tune_conv2d_multi(self, calls, max_trials=0, warmup=3, reps=20):
        """alt_tune_conv2d_multi over `calls` (as for conv2d_multi): returns (variants, order,
        step_us, measurements)."""
        n = len(calls)
        arr = self._call_array(calls)
        variants, order = (ctypes.c_int32 * n)(), (ctypes.c_int32 * n)()
        us, meas = ctypes.c_float(), ctypes.c_int32()
        o = TuneOpts(max_trials, warmup, reps, 0, None, 0, None)
        _ck(lib().alt_tune_conv2d_multi(self._h, arr, ctypes.c_int32(n), ctypes.byref(o), variants, order,
                                        ctypes.byref(us), ctypes.byref(meas)), self._h)
        return list(variants), list(order), us.value, meas.value

    def tune_chain(self, ops, in_layout, arena, arena_bytes, max_trials=0, warmup=3, reps=20, stream=None):
        arr = (ConvDesc * len(ops))(*ops)
        plan = ChainPlan()
        o = self._opts(arena, arena_bytes, max_trials, warmup, reps, 0, stream)
        _ck(lib().alt_tune_chain(self._h, arr, len(ops), ctypes.byref(_as_layout(in_layout)),
                                 ctypes.byref(o), ctypes.byref(plan)), self._h)
        return plan

    def unfold(self, dtype, shape, dim, B, S, src, dst, stream=None):
        _ck(lib().alt_unfold(self._h, dtype, len(shape), _i64(shape), dim, ctypes.c_int64(B), ctypes.c_int64(S),
                             _ptr(src), _ptr(dst), _stream(stream)), self._h)

    def eltwise_add(self, dtype, numel, a, b, y, relu=False, stream=None):
        status = _quick_add(self._h, dtype, numel, a, b, y, relu, stream)
        if status is not None:
            pass
        elif dtype.__class__ is int and dtype in _CODES and numel.__class__ is int:
            status = _call("alt_eltwise_add")(self._h, dtype, numel, _address(a), _address(b), _address(y), int(bool(relu)),
                                              _stream_address(stream))
        else:
            status = lib().alt_eltwise_add(self._h, dtype, ctypes.c_int64(numel), _ptr(a), _ptr(b), _ptr(y), int(bool(relu)),
                                           _stream(stream))
        if status != 0:
            _ck(status, self._h)

    def tune_graph(self, nodes, in_layout, arena, arena_bytes, max_trials=0, warmup=3, reps=20, stream=None):
        arr = (GraphNode * len(nodes))(*nodes)
        plan = GraphPlan()
        o = self._opts(arena, arena_bytes, max_trials, warmup, reps, 0, stream)
        _ck(lib().alt_tune_graph(self._h, arr, len(nodes), ctypes.byref(_as_layout(in_layout)),
                                 ctypes.byref(o), ctypes.byref(plan)), self._h)
        return plan

    def cache_save(self, path):
        _ck(lib().alt_cache_save(self._h, path.encode()), self._h)

    def cache_load(self, path):
        _ck(lib().alt_cache_load(self._h, path.encode()), self._h)

    def cache_clear(self):
        _ck(lib().alt_cache_clear(self._h), self._h)

    def splitk_status(self):
        out = SplitkStatus()
        _ck(lib().alt_splitk_status(self._h, ctypes.byref(out)), self._h)
        return out

    def get_peak(self, arena, arena_bytes):
        p = Peaks()
        _ck(lib().alt_get_peak(self._h, _ptr(arena), ctypes.c_size_t(arena_bytes), ctypes.byref(p)), self._h)
        return p
