"""ctypes binding of libdlm (include/dlm.h): argument marshalling only.

Every function has the name of the C entry point it calls.  Device buffers are
torch tensors (torch only allocates memory and supplies the stream); host
arrays are plain int lists.  A missing library is an error: there is no
fallback path.
"""
import ctypes as C
import functools
import os
import struct

import torch  # loaded first so that libdlm binds to the HIP runtime torch already opened

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libdlm.so")
_lib = None

DLM_F32, DLM_BF16 = 0, 1
ERRORS = {-1: "DLM_EINVAL", -2: "DLM_ESHAPE", -3: "DLM_ECAPACITY", -4: "DLM_ENOMEM", -5: "DLM_EHIP"}


class DlmError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__(f"{ERRORS.get(code, code)}: {msg}")
        self.code = code


class dlm_config(C.Structure):
    _fields_ = [(n, C.c_int32) for n in
                ("n_layers", "d_model", "n_q_heads", "n_kv_heads", "head_dim", "d_ffn", "vocab", "mask_id", "dtype")] + \
               [("rms_eps", C.c_float), ("rope_theta", C.c_float)]


class dlm_weights(C.Structure):
    _fields_ = [("embed", C.c_void_p), ("wqkv", C.POINTER(C.c_void_p)), ("wo", C.POINTER(C.c_void_p)),
                ("w_gate_up", C.POINTER(C.c_void_p)), ("w_down", C.POINTER(C.c_void_p)), ("norm1", C.POINTER(C.c_void_p)),
                ("norm2", C.POINTER(C.c_void_p)), ("final_norm", C.c_void_p), ("lm_head", C.c_void_p)]


_I32P = C.POINTER(C.c_int32)


class dlm_step_desc(C.Structure):
    _fields_ = [("n_seqs", C.c_int32)] + [(n, _I32P) for n in
                ("slot", "row_offsets", "span_start", "commit_len", "kl_first", "kl_count", "save_first", "save_count", "tok_start", "suffix_len")] + \
               [(n, C.c_void_p) for n in ("tokens", "logits", "max_logit", "lse", "entropy", "kl", "conf", "argmax")]


class dlm_boundary_params(C.Structure):
    _fields_ = [("lam", C.c_float), ("l_min", C.c_int32), ("smooth_radius", C.c_int32), ("norm_mode", C.c_int32), ("rule", C.c_int32)]


class dlm_select_params(C.Structure):
    _fields_ = [("tau_low", C.c_float), ("tau_high", C.c_float), ("gamma", C.c_float), ("mode", C.c_int32)]


EXPORTS = ["dlm_last_error", "dlm_model_create", "dlm_model_destroy", "dlm_state_create", "dlm_state_destroy", "dlm_state_reset",
           "dlm_state_kv_len", "dlm_step", "block_boundary", "select_parallel", "dlm_vocab_stats_workspace", "dlm_vocab_stats",
           "dlm_gemm_nt", "dlm_attention", "dlm_profile_enable", "dlm_profile_read", "dlm_probe_hbm_read", "dlm_probe_mfma",
           "dlm_state_fuse_stats", "dlm_vocab_stats_static", "dlm_plan_attention",
           "dlm_plan_vocab_stats", "dlm_plan_gemm"]


def lib():
    """The loaded library; raises if it has not been built."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"{LIB_PATH} is missing: run `python -m paper_2604_15750_amd.build` (there is no fallback path)")
        L = C.CDLL(LIB_PATH)
        L.dlm_last_error.restype = C.c_char_p
        L.dlm_vocab_stats_workspace.restype = C.c_size_t
        L.dlm_vocab_stats_workspace.argtypes = [C.c_int]
        L.dlm_model_create.argtypes = [C.POINTER(dlm_config), C.POINTER(dlm_weights), C.c_void_p, C.POINTER(C.c_void_p)]
        L.dlm_model_destroy.argtypes = [C.c_void_p]
        L.dlm_model_destroy.restype = None
        L.dlm_state_create.argtypes = [C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int, C.POINTER(C.c_void_p)]
        L.dlm_state_destroy.argtypes = [C.c_void_p]
        L.dlm_state_destroy.restype = None
        L.dlm_state_reset.argtypes = [C.c_void_p, C.c_int]
        L.dlm_state_kv_len.argtypes = [C.c_void_p, C.c_int]
        L.dlm_step.argtypes = [C.c_void_p, C.POINTER(dlm_step_desc), C.c_void_p]
        # (the host arrays and parameters of the two decisions are void pointers: they are handed over as bytes)
        L.block_boundary.argtypes = [C.c_void_p] * 5 + [C.c_int] + [C.c_void_p] * 5
        L.select_parallel.argtypes = [C.c_void_p, C.c_int, C.c_int] + [C.c_void_p] * 7 + \
                                     [C.c_int, C.c_int, C.c_void_p, C.c_int] + [C.c_void_p] * 4
        L.dlm_vocab_stats.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int] + [C.c_void_p] * 7 + \
                                     [C.c_size_t, C.c_void_p]
        L.dlm_vocab_stats_static.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int] + [C.c_void_p] * 7
        L.dlm_gemm_nt.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_int, C.c_void_p]
        L.dlm_attention.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p] + [C.c_int] * 6 + [C.c_void_p]
        L.dlm_probe_hbm_read.argtypes = [C.c_void_p, C.c_size_t, C.c_int, C.POINTER(C.c_double), C.c_void_p]
        L.dlm_probe_mfma.argtypes = [C.c_int, C.POINTER(C.c_double), C.c_void_p]
        L.dlm_plan_attention.argtypes = [C.c_int] * 4 + [_I32P]
        L.dlm_plan_vocab_stats.argtypes = [C.c_int] * 3 + [_I32P]
        L.dlm_plan_gemm.argtypes = [C.c_int] * 4 + [_I32P]
        L.dlm_state_fuse_stats.argtypes = [C.c_void_p, C.c_int]
        L.dlm_profile_enable.argtypes = [C.c_void_p, C.c_uint]
        L.dlm_profile_read.argtypes = [C.c_void_p, C.c_int, C.POINTER(C.c_double), C.POINTER(C.c_int64), C.c_int]
        _lib = L
    return _lib


def _check(rc):
    if rc < 0:
        raise DlmError(rc, lib().dlm_last_error().decode())
    return rc


def _ptr(t):
    return None if t is None else t.data_ptr()


def _enough(v, n):
    """The library reads n entries of a host array, whatever its length: one that is shorter is refused here."""
    if v is not None and len(v) < n:
        raise ValueError(f"a host array of {len(v)} entries where the call reads {n}")
    return v


def _ints(v, n=0):
    if v is None:
        return None
    k = len(v)
    if k < n:
        _enough(v, n)
    return (C.c_int32 * k)(*map(int, v))


# The two decisions are bound by what their calls cost the host: plain arguments go through a small extension (csrc/decisions_py.c),
# any others through ctypes, host arrays and parameters as bytes (marshalling alone 3.8 and 6.1 us with ctypes structs and a format
# string per array, 2.7 and 4.8 as bytes, 1.2 and 2.1 through the extension; both decisions of one sequence x 8 rows 11.8 -> 10.0 us a
# pass, of 16 x 64 12.3 -> 10.3, on another box 10.3 -> 9.6 and 10.7 -> 9.7).
@functools.lru_cache(maxsize=None)
def _decisions():
    """The extension, bound to the library; None where it has not been built."""
    try:
        from . import _decisions as m
    except ImportError:
        return None
    L = lib()
    m.bind(C.cast(L.block_boundary, C.c_void_p).value, C.cast(L.select_parallel, C.c_void_p).value, torch.float32, torch.bfloat16)
    return m


@functools.lru_cache(maxsize=64)
def _int_packer(n):
    return struct.Struct(f"{n}i").pack


def _packed(v):
    """A host array as bytes (a ctypes array of 16 takes 2.1 us, this 0.3).  What struct does not take as a 32-bit integer goes
    the way of _ints."""
    if v is None:
        return None
    try:
        return _int_packer(len(v))(*v)
    except (struct.error, TypeError, OverflowError):
        return bytes(_ints(v))


_pack_boundary, _pack_select = struct.Struct("f4i").pack, struct.Struct("3fi").pack


def _params(pack, cls, v):
    """A parameter struct as bytes; values that struct does not take go the way of the ctypes struct."""
    try:
        return pack(*v)
    except (struct.error, TypeError, OverflowError):
        return bytes(cls(*v))


# what torch.cuda.current_stream() asks, without its Stream object (0.3 us against 2.7); a private name, so the public way stays beside it
_raw_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)


def _stream():
    if _raw_stream is None:
        return torch.cuda.current_stream().cuda_stream
    return _raw_stream(torch.cuda.current_device())


_DTYPE_CODES = {torch.float32: DLM_F32, torch.bfloat16: DLM_BF16}


def dtype_code(t):
    return _DTYPE_CODES[t if isinstance(t, torch.dtype) else t.dtype]


class Model:
    """dlm_model_create / dlm_model_destroy.  cfg: dict of inputs.model_config; W: dict of device tensors.
    weight_copies=False sets DLM_W_STEPS=0 for the call: no step-major second copies of the layer matrices."""

    def __init__(self, cfg, W, weight_copies=True):
        self.cfg = dict(cfg)
        dt = DLM_F32 if cfg["dtype"] == "f32" else DLM_BF16
        c = dlm_config(cfg["n_layers"], cfg["d_model"], cfg["n_q_heads"], cfg["n_kv_heads"], cfg["head_dim"], cfg["d_ffn"],
                       cfg["vocab"], cfg["mask_id"], dt, cfg["rms_eps"], cfg["rope_theta"])
        arr = lambda ts: (C.c_void_p * len(ts))(*[t.data_ptr() for t in ts])
        keep = [arr(W[k]) for k in ("wqkv", "wo", "w_gate_up", "w_down", "norm1", "norm2")]
        w = dlm_weights(W["embed"].data_ptr(), *keep, W["final_norm"].data_ptr(), W["lm_head"].data_ptr())
        h = C.c_void_p()
        before = os.environ.get("DLM_W_STEPS")
        if not weight_copies:
            os.environ["DLM_W_STEPS"] = "0"
        try:
            _check(lib().dlm_model_create(C.byref(c), C.byref(w), _stream(), C.byref(h)))
        finally:
            if not weight_copies:
                if before is None:
                    del os.environ["DLM_W_STEPS"]
                else:
                    os.environ["DLM_W_STEPS"] = before
        torch.cuda.current_stream().synchronize()  # the caller may now drop W
        self.handle = h
        self.torch_dtype = torch.float32 if dt == DLM_F32 else torch.bfloat16

    def close(self):
        if self.handle and lib is not None:  # at interpreter shutdown the module's globals may already be gone
            lib().dlm_model_destroy(self.handle)
            self.handle = None

    __del__ = close


class State:
    """dlm_state_create / dlm_state_destroy."""

    def __init__(self, model, max_seqs, max_seq_len, max_rows, max_lookahead):
        self.model = model
        h = C.c_void_p()
        _check(lib().dlm_state_create(model.handle, max_seqs, max_seq_len, max_rows, max_lookahead, C.byref(h)))
        self.handle = h
        self.max_rows = max_rows

    def reset(self, slot):
        _check(lib().dlm_state_reset(self.handle, slot))

    def kv_len(self, slot):
        return _check(lib().dlm_state_kv_len(self.handle, slot))

    def fuse_stats(self, enable):
        """dlm_state_fuse_stats: statistics of qualifying passes from the LM head's epilogue (default) or from the streamed reduction."""
        _check(lib().dlm_state_fuse_stats(self.handle, int(bool(enable))))

    PROFILE_CLASSES = ("gemm_qkv", "gemm_o", "gemm_gate_up", "gemm_down", "gemm_lm_head", "attention", "vocab_stats", "other")

    def profile_enable(self, classes):
        """classes: True (all), False (none) or an iterable of names from PROFILE_CLASSES."""
        if classes is True:
            mask = (1 << len(self.PROFILE_CLASSES)) - 1
        elif not classes:
            mask = 0
        else:
            mask = sum(1 << self.PROFILE_CLASSES.index(c) for c in classes)
        _check(lib().dlm_profile_enable(self.handle, mask))

    def profile_read(self, reset=True):
        """{class name: (milliseconds, launches)} since the last reset."""
        k = len(self.PROFILE_CLASSES)
        ms = (C.c_double * k)()
        n = (C.c_int64 * k)()
        _check(lib().dlm_profile_read(self.handle, k, ms, n, int(reset)))
        return {name: (ms[i], n[i]) for i, name in enumerate(self.PROFILE_CLASSES)}

    def close(self):
        if self.handle and lib is not None:
            lib().dlm_state_destroy(self.handle)
            self.handle = None

    __del__ = close


class StepOutputs:
    """Caller-owned output buffers of dlm_step for up to `rows` rows."""

    def __init__(self, rows, vocab, dtype, device):
        self.logits = torch.empty((rows, vocab), dtype=dtype, device=device)
        f = lambda: torch.empty(rows, dtype=torch.float32, device=device)
        self.max_logit, self.lse, self.entropy, self.kl, self.conf = f(), f(), f(), f(), f()
        self.argmax = torch.empty(rows, dtype=torch.int32, device=device)


def dlm_step(state, tokens, out, row_offsets, span_start, commit_len, tok_start, slot=None, kl_first=None, kl_count=None,
             save_first=None, save_count=None, suffix_len=None):
    """tokens: device int32 tensor; out: StepOutputs; the rest: host int lists (see include/dlm.h)."""
    n = len(span_start)
    keep = [_ints(slot, n), _ints(row_offsets, n + 1)]
    keep += [_ints(v, n) for v in (span_start, commit_len, kl_first, kl_count, save_first, save_count, tok_start, suffix_len)]
    d = dlm_step_desc(n, *keep, tokens.data_ptr(), out.logits.data_ptr(), out.max_logit.data_ptr(), out.lse.data_ptr(),
                      out.entropy.data_ptr(), out.kl.data_ptr(), out.conf.data_ptr(), out.argmax.data_ptr())
    _check(lib().dlm_step(state.handle, C.byref(d), _stream()))


def block_boundary(I, H, win_start, win_len, L_out, lam, l_min, smooth_radius=1, norm_mode=0, rule=0, cold=None, S_out=None,
                   margin_out=None):
    ext = _decisions()
    if ext is not None:
        rc = ext.boundary(I, H, win_start, win_len, cold, L_out, S_out, margin_out, lam, l_min, smooth_radius, norm_mode, rule, _stream())
        if rc is not None:  # (None: not plain arguments, nothing has been called)
            if rc < 0:
                _check(rc)
            return
    n = len(win_start)
    _check(lib().block_boundary(_ptr(I), _ptr(H), _packed(win_start), _packed(_enough(win_len, n)), _packed(_enough(cold, n)), n,
                                _params(_pack_boundary, dlm_boundary_params, (lam, l_min, smooth_radius, norm_mode, rule)), _ptr(L_out),
                                _ptr(S_out), _ptr(margin_out), _stream()))


def select_parallel(logits, lse, conf, argmax, tokens, row_start, tok_start, block_len, mask_id, tau_low, tau_high, gamma, mode,
                    selected_out, n_selected_out, apply_tokens=True, margin_out=None):
    ext = _decisions()
    if ext is not None:
        rc = ext.select(logits, lse, conf, argmax, tokens, row_start, tok_start, block_len, mask_id, tau_low, tau_high, gamma, mode,
                        selected_out, n_selected_out, apply_tokens, margin_out, _stream())
        if rc is not None:
            if rc < 0:
                _check(rc)
            return
    n = len(row_start)
    _check(lib().select_parallel(_ptr(logits), logits.size(-1), dtype_code(logits), _ptr(lse), _ptr(conf), _ptr(argmax), _ptr(tokens),
                                 _packed(row_start), _packed(_enough(tok_start, n)), _packed(_enough(block_len, n)), n, mask_id,
                                 _params(_pack_select, dlm_select_params, (tau_low, tau_high, gamma, mode)), int(apply_tokens),
                                 _ptr(selected_out), _ptr(n_selected_out), _ptr(margin_out), _stream()))


def dlm_vocab_stats(logits, mask_id, prev=None, workspace=None, prev_lse=None):
    rows, vocab = logits.shape
    dev = logits.device
    f = lambda: torch.empty(rows, dtype=torch.float32, device=dev)
    out = dict(max_logit=f(), lse=f(), entropy=f(), kl=f(), conf=f(), argmax=torch.empty(rows, dtype=torch.int32, device=dev))
    if workspace is None:
        workspace = torch.empty(lib().dlm_vocab_stats_workspace(rows), dtype=torch.uint8, device=dev)
    _check(lib().dlm_vocab_stats(_ptr(logits), _ptr(prev), _ptr(prev_lse), rows, vocab, dtype_code(logits), mask_id, _ptr(out["max_logit"]),
                                 _ptr(out["lse"]), _ptr(out["entropy"]), _ptr(out["kl"]), _ptr(out["conf"]), _ptr(out["argmax"]),
                                 _ptr(workspace), workspace.numel(), _stream()))
    return out


def dlm_vocab_stats_static(logits, mask_id, prev=None, out=None, prev_lse=None):
    """dlm_vocab_stats_static: the partial states live in the library's file-scope scratch.  `out`: a dict of preallocated
    output tensors as dlm_vocab_stats returns (so that the call allocates nothing at all); None: new ones."""
    rows, vocab = logits.shape
    dev = logits.device
    if out is None:
        f = lambda: torch.empty(rows, dtype=torch.float32, device=dev)
        out = dict(max_logit=f(), lse=f(), entropy=f(), kl=f(), conf=f(), argmax=torch.empty(rows, dtype=torch.int32, device=dev))
    _check(lib().dlm_vocab_stats_static(_ptr(logits), _ptr(prev), _ptr(prev_lse), rows, vocab, dtype_code(logits), mask_id, _ptr(out["max_logit"]),
                                        _ptr(out["lse"]), _ptr(out["entropy"]), _ptr(out["kl"]), _ptr(out["conf"]), _ptr(out["argmax"]),
                                        _stream()))
    return out


def dlm_gemm_nt(x, w):
    M, K = x.shape
    N = w.shape[0]
    y = torch.empty((M, N), dtype=x.dtype, device=x.device)
    _check(lib().dlm_gemm_nt(_ptr(x), _ptr(w), _ptr(y), M, N, K, dtype_code(x), _stream()))
    return y


def probe_hbm_read(buf, reps=10):
    """GB/s of a plain streaming read of the device tensor `buf` (see include/dlm.h)."""
    out = C.c_double()
    _check(lib().dlm_probe_hbm_read(_ptr(buf), C.c_size_t(buf.numel() * buf.element_size()), reps, C.byref(out), _stream()))
    return out.value


def probe_mfma(reps=5):
    """TFLOP/s of independent half-precision matrix-core products out of registers, on operands of pseudo-random values."""
    out = C.c_double()
    _check(lib().dlm_probe_mfma(reps, C.byref(out), _stream()))
    return out.value


def dlm_attention(q, k, v):
    A, n_q, hd = q.shape
    T, n_kv, _ = k.shape
    out = torch.empty_like(q)
    _check(lib().dlm_attention(_ptr(q), _ptr(k), _ptr(v), _ptr(out), A, T, n_q, n_kv, hd, dtype_code(q), _stream()))
    return out


def plan_attention(max_seq_rows, n_seqs, n_q, head_dim):
    """How the attention of such a pass is launched (include/dlm.h): wavefronts of a workgroup, workgroups that share a head's
    output dims, 16-query tiles of a workgroup."""
    out = (C.c_int32 * 3)()
    _check(lib().dlm_plan_attention(max_seq_rows, n_seqs, n_q, head_dim, out))
    return dict(zip(("waves", "shares", "tiles"), out))


def plan_vocab_stats(rows, vocab, dtype):
    """How the streamed vocabulary reduction is launched (include/dlm.h): threads of a workgroup, chunks of a row."""
    out = (C.c_int32 * 2)()
    _check(lib().dlm_plan_vocab_stats(rows, vocab, dtype_code(dtype), out))
    return dict(zip(("threads", "chunks"), out))


EPILOGUES = ("direct", "qkv", "swiglu", "resid", "sum", "stats")


def plan_gemm(M, N, K, epilogue):
    """How a bf16 model's product is launched (include/dlm.h); epilogue: a name from EPILOGUES."""
    out = (C.c_int32 * 7)()
    _check(lib().dlm_plan_gemm(M, N, K, EPILOGUES.index(epilogue), out))
    return dict(zip(("kernel", "rows", "cols", "splits", "k_parts", "workgroups", "ssq_parts"), (("skinny", "mid", "macro")[out[0]], *out[1:])))
