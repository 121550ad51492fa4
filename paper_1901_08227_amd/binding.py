"""ctypes binding of libtng (include/tng.h).  Argument marshalling only: every step of the
iteration runs in the HIP kernels of the library; torch tensors are used as device memory.  The calls of
a training loop are marshalled by a native function (csrc/tng_call.cpp) where their arguments are plain.

The module-level functions carry the names of the C entry points and take a context handle
plus torch CUDA tensors; `Context` owns the workspace and keeps problem data alive.
There is no fallback for the library: if it has not been built, loading raises.  Without the native function, or with one that
was built for another torch or Python, the calls all go through ctypes.
"""
from __future__ import annotations

import ctypes
import importlib.machinery
import importlib.util
import os

import torch

from . import build

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libtng.so")
CALL_PATH = os.path.join(_HERE, "tng_call.so")

TNG_OK = 0
TNG_ERR_INVALID_ARG, TNG_ERR_BAD_STATE, TNG_ERR_WORKSPACE, TNG_ERR_UNSUPPORTED, TNG_ERR_HIP = 1, 2, 3, 4, 5
TNG_ERR_TOO_LARGE, TNG_ERR_HOST_MEMORY = 6, 7
NORM_NONE, NORM_SUB, NORM_QUOT, NORM_COMB, NORM_MEAN = 0, 1, 2, 3, 4
SCALE_MAX, SCALE_L2 = 0, 1
REF_ZERO, REF_LAST_AVG, REF_WINDOW_AVG = 0, 1, 2
PROB_EXTERNAL, PROB_LOGREG_DENSE, PROB_LOGREG_CSR, PROB_ROSENBROCK = 0, 1, 2, 3


class TngConfig(ctypes.Structure):
    _fields_ = [
        ("d", ctypes.c_uint64), ("M", ctypes.c_uint32), ("bits", ctypes.c_uint32),
        ("norm", ctypes.c_int32), ("quot_eps", ctypes.c_float),
        ("ref_policy", ctypes.c_int32), ("ref_period", ctypes.c_uint32),
        ("seed", ctypes.c_uint64), ("lr", ctypes.c_float), ("l2", ctypes.c_float),
        ("batch", ctypes.c_uint32), ("problem", ctypes.c_int32), ("ref_window", ctypes.c_uint32),
        ("scale", ctypes.c_int32),
    ]


class TngError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {status_string(status)} (tng_status {status})")


_lib = None
_call = None      # the extension's call() or _through_ctypes; set with the library
_address = None   # {entry point: its address} of those that go through it


def _through_ctypes(*_):
    """In the place of tng_call.call: no case is plain."""
    return None


def _load_call():
    """tng_call.call of the built extension; _through_ctypes where there is none that fits this torch and Python."""
    if not os.path.exists(CALL_PATH):
        return _through_ctypes
    try:
        loader = importlib.machinery.ExtensionFileLoader("tng_call", CALL_PATH)
        module = importlib.util.module_from_spec(importlib.util.spec_from_loader("tng_call", loader))
        loader.exec_module(module)
    except ImportError:
        return _through_ctypes
    return module.call if getattr(module, "built_for", None) == build.call_target() else _through_ctypes


def lib() -> ctypes.CDLL:
    """The loaded library; raises if it has not been built (python -m paper_1901_08227_amd.build)."""
    global _lib, _call, _address
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(f"libtng is not built: {LIB_PATH} is missing; run __graft_entry__.build()")
        L = ctypes.CDLL(LIB_PATH)
        vp, u32, u64, cfgp = ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint64, ctypes.POINTER(TngConfig)
        L.tng_words_per_row.restype, L.tng_words_per_row.argtypes = u64, [u64, u32]
        L.tng_workspace_bytes.restype, L.tng_workspace_bytes.argtypes = ctypes.c_size_t, [cfgp]
        L.tng_status_string.restype, L.tng_status_string.argtypes = ctypes.c_char_p, [ctypes.c_int]
        L.tng_csr_index_bytes.restype = ctypes.c_size_t
        L.tng_csr_index_bytes.argtypes = [cfgp, ctypes.POINTER(ctypes.c_uint64)]
        sigs = {
            "tng_create": [cfgp, vp, ctypes.c_size_t, vp, ctypes.POINTER(vp)],
            "tng_destroy": [vp],
            "tng_set_logreg_dense": [vp, ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(u64)],
            "tng_set_logreg_csr": [vp, ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(vp),
                                   ctypes.POINTER(vp), ctypes.POINTER(u64)],
            "tng_set_logreg_csr_pairs": [vp, ctypes.POINTER(vp), ctypes.POINTER(vp), ctypes.POINTER(vp),
                                         ctypes.POINTER(u64)],
            "tng_validate_csr": [vp, ctypes.POINTER(u64)],
            "tng_set_noise": [vp, vp],
            "tng_set_noise_variance": [vp, ctypes.c_float],
            "tng_set_csr_index": [vp, vp, ctypes.c_size_t],
            "tng_set_second_reference": [vp, vp],
            "tng_set_worker_means": [vp, vp],
            "tng_set_reference_history": [vp, vp],
            "tng_set_profile_events": [vp, ctypes.POINTER(vp), u32],
            "tng_rng_draws": [vp, u32, u32, u32, u64, u64, vp],
            "tng_minibatch_indices": [vp, u32, vp],
            "tng_local_grad": [vp, u32, vp, vp],
            "tng_normalize_encode": [vp, u32, vp, vp, vp, vp],
            "tng_normalize_encode_static": [cfgp, vp, u32, vp, vp, vp, vp],
            "tng_decode_aggregate": [vp, vp, vp, vp, vp],
            "tng_update_reference": [vp, u32, vp, vp],
            "tng_step": [vp, u32, vp, vp, vp, vp, vp, vp],
        }
        for name, argtypes in sigs.items():
            fn = getattr(L, name)
            fn.restype, fn.argtypes = ctypes.c_int, argtypes
        _call = _load_call()
        _address = {name: ctypes.cast(getattr(L, name), vp).value
                    for name in ("tng_local_grad", "tng_normalize_encode", "tng_decode_aggregate", "tng_update_reference",
                                 "tng_step")}
        _lib = L
    return _lib


def status_string(status: int) -> str:
    return lib().tng_status_string(int(status)).decode()


def tng_words_per_row(d: int, bits: int) -> int:
    return int(lib().tng_words_per_row(d, bits))


def tng_workspace_bytes(cfg: TngConfig) -> int:
    return int(lib().tng_workspace_bytes(ctypes.byref(cfg)))


def _check(status: int, where: str):
    if status != TNG_OK:
        raise TngError(status, where)


def _ptr(t, dtype, numel, name):
    """Device address of a contiguous CUDA tensor of the given dtype and at least numel elements."""
    if t is None:
        return None
    if not isinstance(t, torch.Tensor) or not t.is_cuda:
        raise TypeError(f"{name}: expected a CUDA tensor")
    if t.dtype != dtype or not t.is_contiguous():
        raise TypeError(f"{name}: expected contiguous {dtype}, got {t.dtype}")
    if t.numel() < numel:
        raise ValueError(f"{name}: needs {numel} elements, has {t.numel()}")
    return ctypes.c_void_p(t.data_ptr())


def csr_pairs(col, val):
    """(column, value) pairs for set_logreg_csr_pairs from parallel arrays: an int32 tensor [nnz][2] whose
    second column holds the bit patterns of the float32 values (layout only; nothing is computed)."""
    out = torch.empty((col.numel(), 2), dtype=torch.int32, device=col.device)
    out[:, 0] = col
    out[:, 1] = val.view(torch.int32)
    return out


class Context:
    """A tng_ctx plus the device workspace it was created on (torch owns the memory)."""

    def __init__(self, *, d, M, bits=2, norm=NORM_SUB, quot_eps=1e-8, ref_policy=REF_LAST_AVG, ref_period=1,
                 seed=0, lr=0.1, l2=0.0, batch=0, problem=PROB_EXTERNAL, ref_window=1, scale=SCALE_MAX, device="cuda:0",
                 stream=None):
        self.cfg = TngConfig(d=d, M=M, bits=bits, norm=norm, quot_eps=quot_eps, ref_policy=ref_policy,
                             ref_period=ref_period, seed=seed, lr=lr, l2=l2, batch=batch, problem=problem,
                             ref_window=ref_window, scale=scale)
        nbytes = tng_workspace_bytes(self.cfg)
        if nbytes == 0:
            raise TngError(TNG_ERR_INVALID_ARG, "tng_workspace_bytes")
        self.device = torch.device(device)
        if stream is None:
            stream = torch.cuda.current_stream(self.device)
        self.stream = stream
        # the zero fill goes on the context's own stream: on another stream it could still be pending, and
        # wipe the pointer tables, after the library has begun to use the workspace
        with torch.cuda.stream(stream):
            self.workspace = torch.zeros(nbytes, dtype=torch.uint8, device=self.device)
        self.handle = ctypes.c_void_p()
        _check(lib().tng_create(ctypes.byref(self.cfg), ctypes.c_void_p(self.workspace.data_ptr()), nbytes,
                                ctypes.c_void_p(stream.cuda_stream), ctypes.byref(self.handle)), "tng_create")
        self.d, self.M, self.bits, self.batch = int(d), int(M), int(bits), int(batch)
        self.words = tng_words_per_row(d, bits)
        self._keep = {}

    def close(self):
        if self.handle:
            lib().tng_destroy(self.handle)
            self.handle = ctypes.c_void_p()

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    # ---- problem data
    def _table(self, tensors, dtype, numels, name):
        arr = (ctypes.c_void_p * self.M)()
        for m, t in enumerate(tensors):
            arr[m] = _ptr(t, dtype, numels[m], f"{name}[{m}]").value
        return arr

    def set_logreg_dense(self, X, y):
        """X: list of M tensors [n_m][d] float32; y: list of M tensors [n_m] float32 (0/1)."""
        n = [int(x.shape[0]) for x in X]
        rows = (ctypes.c_uint64 * self.M)(*n)
        tx = self._table(X, torch.float32, [k * self.d for k in n], "X")
        ty = self._table(y, torch.float32, n, "y")
        self._keep["data"] = (list(X), list(y))
        self.n_rows = n
        _check(lib().tng_set_logreg_dense(self.handle, tx, ty, rows), "tng_set_logreg_dense")

    def set_logreg_csr(self, rowptr, col, val, y):
        n = [int(r.numel()) - 1 for r in rowptr]
        rows = (ctypes.c_uint64 * self.M)(*n)
        nnz = [int(c.numel()) for c in col]
        tr = self._table(rowptr, torch.int64, [k + 1 for k in n], "rowptr")
        tc = self._table(col, torch.int32, nnz, "col")
        tv = self._table(val, torch.float32, nnz, "val")
        ty = self._table(y, torch.float32, n, "y")
        self._keep["data"] = (list(rowptr), list(col), list(val), list(y))
        self._keep["nnz"] = nnz
        self.n_rows = n
        _check(lib().tng_set_logreg_csr(self.handle, tr, tc, tv, ty, rows), "tng_set_logreg_csr")

    def set_logreg_csr_pairs(self, rowptr, entries, y):
        """entries: list of M int32 tensors [nnz_m][2]: column id and the bit pattern of the float32 value
        (see csr_pairs), i.e. an array of tng_csr_entry."""
        n = [int(r.numel()) - 1 for r in rowptr]
        rows = (ctypes.c_uint64 * self.M)(*n)
        nnz = [int(e.numel()) // 2 for e in entries]
        tr = self._table(rowptr, torch.int64, [k + 1 for k in n], "rowptr")
        te = self._table(entries, torch.int32, [2 * k for k in nnz], "entries")
        ty = self._table(y, torch.float32, n, "y")
        self._keep["data"] = (list(rowptr), list(entries), None, list(y))
        self._keep["nnz"] = nnz
        self.n_rows = n
        _check(lib().tng_set_logreg_csr_pairs(self.handle, tr, te, ty, rows), "tng_set_logreg_csr_pairs")

    def validate_csr(self):
        """Device pass over the CSR shards set last: raises TngError(TNG_ERR_INVALID_ARG) if row pointers or
        column ids break what the gradient kernels assume."""
        nnz = (ctypes.c_uint64 * self.M)(*self._keep["nnz"])
        _check(lib().tng_validate_csr(self.handle, nnz), "tng_validate_csr")

    def build_csr_index(self):
        """Allocates and builds the per-row tile index for the CSR shards set last (optional speed-up)."""
        rows = (ctypes.c_uint64 * self.M)(*self.n_rows)
        nbytes = lib().tng_csr_index_bytes(ctypes.byref(self.cfg), rows)
        if nbytes == 0:
            raise TngError(TNG_ERR_UNSUPPORTED, "tng_csr_index_bytes")
        index = torch.empty(nbytes, dtype=torch.uint8, device=self.device)
        self._keep["csr_index"] = index
        _check(lib().tng_set_csr_index(self.handle, ctypes.c_void_p(index.data_ptr()), nbytes), "tng_set_csr_index")

    def set_noise(self, noise):
        self._keep["noise"] = noise
        _check(lib().tng_set_noise(self.handle, _ptr(noise, torch.float32, self.M * self.d, "noise")), "tng_set_noise")

    def set_noise_variance(self, variance):
        """Rosenbrock: N(0, variance) noise generated on the device (0 switches it off)."""
        _check(lib().tng_set_noise_variance(self.handle, float(variance)), "tng_set_noise_variance")
        if variance > 0:
            self._keep.pop("noise", None)

    def set_reference_history(self, history):
        """history: zero-filled float32 tensor [ref_window][d]; the library keeps the decoded averages in it."""
        self._keep["history"] = history
        _check(lib().tng_set_reference_history(
            self.handle, _ptr(history, torch.float32, int(self.cfg.ref_window) * self.d, "history")),
            "tng_set_reference_history")

    def set_second_reference(self, gref2):
        self._keep["gref2"] = gref2
        _check(lib().tng_set_second_reference(self.handle, _ptr(gref2, torch.float32, self.d, "gref2")),
               "tng_set_second_reference")

    def set_worker_means(self, means):
        """means: float32 tensor [M]; written by encode, read by decode (per-worker mean reference)."""
        self._keep["means"] = means
        _check(lib().tng_set_worker_means(self.handle, _ptr(means, torch.float32, self.M, "means")),
               "tng_set_worker_means")

    def set_profile_events(self, events, slots):
        """events: list of 5*slots hipEvent_t handles (ints), or None to switch the hook off."""
        if not events:
            _check(lib().tng_set_profile_events(self.handle, None, 0), "tng_set_profile_events")
            return
        arr = (ctypes.c_void_p * len(events))(*events)
        _check(lib().tng_set_profile_events(self.handle, arr, slots), "tng_set_profile_events")

    # ---- the calls
    def rng_draws(self, it, worker, stream, first, count, out):
        _check(lib().tng_rng_draws(self.handle, it, worker, stream, first, count,
                                   _ptr(out, torch.int32, count, "out")), "tng_rng_draws")

    def minibatch_indices(self, it, idx):
        _check(lib().tng_minibatch_indices(self.handle, it, _ptr(idx, torch.int32, self.M * self.batch, "idx")),
               "tng_minibatch_indices")

    # (each first by the native function; None: not a plain case, ctypes converts the arguments or says what is wrong)
    def local_grad(self, it, w, g):
        status = _call(_address["tng_local_grad"], self.handle.value, it, "dg", self.d, self.M, self.words, w, g)
        if status is None:
            status = lib().tng_local_grad(self.handle, it, _ptr(w, torch.float32, self.d, "w"),
                                          _ptr(g, torch.float32, self.M * self.d, "g"))
        _check(status, "tng_local_grad")

    def normalize_encode(self, it, g, gref, codes, scales):
        status = _call(_address["tng_normalize_encode"], self.handle.value, it, "gdcs", self.d, self.M, self.words, g, gref,
                       codes, scales)
        if status is None:
            status = lib().tng_normalize_encode(
                self.handle, it, _ptr(g, torch.float32, self.M * self.d, "g"), _ptr(gref, torch.float32, self.d, "gref"),
                _ptr(codes, torch.int32, self.M * self.words, "codes"), _ptr(scales, torch.float32, self.M, "scales"))
        _check(status, "tng_normalize_encode")

    def decode_aggregate(self, codes, scales, gref, vbar):
        status = _call(_address["tng_decode_aggregate"], self.handle.value, None, "-csdd", self.d, self.M, self.words, codes,
                       scales, gref, vbar)
        if status is None:
            status = lib().tng_decode_aggregate(
                self.handle, _ptr(codes, torch.int32, self.M * self.words, "codes"),
                _ptr(scales, torch.float32, self.M, "scales"), _ptr(gref, torch.float32, self.d, "gref"),
                _ptr(vbar, torch.float32, self.d, "vbar"))
        _check(status, "tng_decode_aggregate")

    def update_reference(self, it, vbar, gref):
        status = _call(_address["tng_update_reference"], self.handle.value, it, "dd", self.d, self.M, self.words, vbar, gref)
        if status is None:
            status = lib().tng_update_reference(self.handle, it, _ptr(vbar, torch.float32, self.d, "vbar"),
                                                _ptr(gref, torch.float32, self.d, "gref"))
        _check(status, "tng_update_reference")

    def step(self, it, w, gref, g, codes, scales, vbar):
        status = _call(_address["tng_step"], self.handle.value, it, "ddgcsd", self.d, self.M, self.words, w, gref, g, codes,
                       scales, vbar)
        if status is None:
            status = lib().tng_step(
                self.handle, it, _ptr(w, torch.float32, self.d, "w"), _ptr(gref, torch.float32, self.d, "gref"),
                _ptr(g, torch.float32, self.M * self.d, "g"), _ptr(codes, torch.int32, self.M * self.words, "codes"),
                _ptr(scales, torch.float32, self.M, "scales"), _ptr(vbar, torch.float32, self.d, "vbar"))
        _check(status, "tng_step")


# Module-level spellings of the C entry points (same names, same argument order).
def tng_local_grad(ctx: Context, it, w, g):
    ctx.local_grad(it, w, g)


def tng_normalize_encode(ctx: Context, it, g, gref, codes, scales):
    ctx.normalize_encode(it, g, gref, codes, scales)


def tng_decode_aggregate(ctx: Context, codes, scales, gref, vbar):
    ctx.decode_aggregate(codes, scales, gref, vbar)


def tng_update_reference(ctx: Context, it, vbar, gref):
    ctx.update_reference(it, vbar, gref)


def tng_step(ctx: Context, it, w, gref, g, codes, scales, vbar):
    ctx.step(it, w, gref, g, codes, scales, vbar)


def tng_normalize_encode_static(cfg: TngConfig, stream, it, g, gref, codes, scales):
    """The encoder without a context or a workspace (fixed scratch inside the library; M <= 64)."""
    words = tng_words_per_row(int(cfg.d), int(cfg.bits))
    M, d = int(cfg.M), int(cfg.d)
    _check(lib().tng_normalize_encode_static(
        ctypes.byref(cfg), ctypes.c_void_p(stream.cuda_stream if stream is not None else 0), it,
        _ptr(g, torch.float32, M * d, "g"), _ptr(gref, torch.float32, d, "gref"),
        _ptr(codes, torch.int32, M * words, "codes"), _ptr(scales, torch.float32, M, "scales")),
        "tng_normalize_encode_static")
