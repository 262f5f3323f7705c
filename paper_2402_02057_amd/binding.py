"""Thin binding of the C-ABI HIP library (include/la.h): argument marshalling only.

Every step of the hot path runs in the library's kernels.  There is no fallback: if the
library has not been built (python -m paper_2402_02057_amd.buildlib, or
__graft_entry__.build()) loading fails loudly.

The calls of a decoding step are marshalled by an extension module (csrc/la_binding.cpp): an entry
point is called once per layer and step, and checking its tensors in Python took longer than the
shorter launches take on the GPU.  The functions below document the arguments and hand them on;
queries and testing hooks, and whoever wants the C functions themselves (load()), go through ctypes.
"""
import ctypes
import importlib
import os

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libla_hip.so")

LA_OK = 0
LA_EINVAL, LA_EUNSUPPORTED, LA_ENOMEM, LA_EHIP = -1, -2, -3, -4
_lib = None


# (the C structures below are for callers of load())

class StepDesc(ctypes.Structure):
    """la_step_desc of include/la.h."""
    _fields_ = [("q", ctypes.c_void_p), ("k_cache", ctypes.c_void_p), ("v_cache", ctypes.c_void_p),
                ("step_k", ctypes.c_void_p), ("step_v", ctypes.c_void_p), ("out", ctypes.c_void_p),
                ("P", ctypes.c_int), ("reserved", ctypes.c_int)]


class StepDescPaged(ctypes.Structure):
    """la_step_desc_paged of include/la.h."""
    _fields_ = [("q", ctypes.c_void_p), ("block_table", ctypes.c_void_p), ("step_k", ctypes.c_void_p),
                ("step_v", ctypes.c_void_p), ("out", ctypes.c_void_p), ("P", ctypes.c_int), ("reserved", ctypes.c_int)]


class CommitDesc(ctypes.Structure):
    """la_commit_desc of include/la.h."""
    _fields_ = [("k_cache", ctypes.c_void_p), ("v_cache", ctypes.c_void_p), ("block_table", ctypes.c_void_p),
                ("step_k", ctypes.c_void_p), ("step_v", ctypes.c_void_p), ("best", ctypes.c_void_p),
                ("n_out", ctypes.c_void_p), ("capacity", ctypes.c_longlong), ("P", ctypes.c_int),
                ("reserved", ctypes.c_int)]


class VerifyDesc(ctypes.Structure):
    """la_verify_desc of include/la.h."""
    _fields_ = [(n, ctypes.c_void_p) for n in ("logits_cur", "logits_look", "logits_cand", "cand_tokens",
                                                "out_tokens", "n_out", "best", "new_window", "accept_len")]


class SampleDesc(ctypes.Structure):
    """la_sample_desc of include/la.h."""
    _fields_ = [(n, ctypes.c_void_p) for n in ("logits_cur", "logits_cand", "cand_tokens", "u_test", "u_final",
                                                "out_tokens", "n_out")] + \
               [("temperature", ctypes.c_float), ("reserved", ctypes.c_int)]


class LaError(RuntimeError):
    def __init__(self, code, message):
        super().__init__("la error %d: %s" % (code, message))
        self.code = code


def load():
    """Open libla_hip.so (once).  Raises if it is missing: the HIP path is the only path."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError("HIP library %s is not built; run __graft_entry__.build()" % LIB_PATH)
    lib = ctypes.CDLL(LIB_PATH)
    i, p = ctypes.c_int, ctypes.c_void_p
    lib.la_step_attention.argtypes = [p, p, p, p, p, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention.restype = i
    lib.la_step_attention_noalloc.argtypes = [p, p, p, p, p, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention_noalloc.restype = i
    lib.la_step_attention_fp8kv.argtypes = [p, p, p, p, p, p, p, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention_fp8kv.restype = i
    lib.la_step_attention_rope.argtypes = [p, p, p, p, p, p, p, i, i, i, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention_rope.restype = i
    ll = ctypes.c_longlong
    lib.la_step_attention_cap.argtypes = [p, p, p, ll, p, p, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention_cap.restype = i
    lib.la_kv_commit.argtypes = [p, p, ll, p, p, i, i, i, i, i, i, p, p, p]
    lib.la_kv_commit.restype = i
    lib.la_kv_commit_rope.argtypes = [p, p, ll, p, p, p, p, i, i, i, i, i, i, i, i, p, p, p]
    lib.la_kv_commit_rope.restype = i
    lib.la_verify_sample_batch.argtypes = [p, i, i, i, i, p]
    lib.la_verify_sample_batch.restype = i
    lib.la_step_rope.argtypes = [p, p, p, p, i, i, i, i, i, i, i, i, i, p]
    lib.la_step_rope.restype = i
    lib.la_verify_step_batch.argtypes = [p, i, i, i, i, i, p]
    lib.la_verify_step_batch.restype = i
    lib.la_kv_commit_batch.argtypes = [p, i, i, i, i, i, i, i, i, p]
    lib.la_kv_commit_batch.restype = i
    lib.la_step_attention_batch.argtypes = [p, i, i, i, i, i, i, i, p]
    lib.la_step_attention_batch.restype = i
    lib.la_step_attention_batch_paged.argtypes = [p, i, p, p, i, i, i, i, i, i, i, i, p]
    lib.la_step_attention_batch_paged.restype = i
    lib.la_step_attention_rows.argtypes = [p, p, p, p, p, p, i, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention_rows.restype = i
    lib.la_step_attention_paged.argtypes = [p, p, p, p, i, i, p, p, i, i, i, i, i, i, i, p, p]
    lib.la_step_attention_paged.restype = i
    lib.la_kv_commit_paged.argtypes = [p, p, p, i, i, p, p, i, i, i, i, i, i, p, p, p]
    lib.la_kv_commit_paged.restype = i
    lib.la_verify.argtypes = [p, p, i, i, i, p, p, p]
    lib.la_verify.restype = i
    lib.la_verify_step.argtypes = [p, p, p, p, i, i, i, i, p, p, p, p, p, p]
    lib.la_verify_step.restype = i
    lib.la_verify_sample.argtypes = [p, p, p, p, p, ctypes.c_float, i, i, i, p, p, p]
    lib.la_verify_sample.restype = i
    lib.la_step_attention_workspace_bytes.argtypes = [i, i, i, i, i, i, i]
    lib.la_step_attention_workspace_bytes.restype = ctypes.c_longlong
    lib.la_step_attention_kernel.argtypes = [i, i, i, i, i, i, i]
    lib.la_step_attention_kernel.restype = i
    lib.la_shutdown.argtypes = []
    lib.la_shutdown.restype = None
    lib.la_last_error.argtypes = []
    lib.la_last_error.restype = ctypes.c_char_p
    lib.la_probe_stream_read.argtypes = [p, ll, p, p]
    lib.la_probe_stream_read.restype = i
    lib.la_probe_mfma.argtypes = [i, p, p]
    lib.la_probe_mfma.restype = ll
    lib.la_debug_override.argtypes = [ctypes.c_char_p, ctypes.c_char_p]
    lib.la_debug_override.restype = i
    lib.la_select_workspace.argtypes = [i]
    lib.la_select_workspace.restype = i
    lib.la_version.argtypes = []
    lib.la_version.restype = i
    _lib = lib
    return lib


class _Native:
    """The extension module, opened on the first call into it."""

    def __getattr__(self, name):
        load()
        try:
            module = importlib.import_module("._la_native", __package__)
        except ImportError as e:
            raise RuntimeError("the extension module _la_native is not built or does not load (%s); run "
                               "__graft_entry__.build()" % e) from e
        module.set_error_class(LaError)
        for key in dir(module):
            setattr(self, key, getattr(module, key))
        return getattr(module, name)


_native = _Native()


EXPORTS = ("la_step_rope", "la_step_attention", "la_step_attention_noalloc", "la_step_attention_fp8kv", "la_step_attention_rope", "la_step_attention_cap", "la_kv_commit", "la_kv_commit_rope", "la_step_attention_paged", "la_kv_commit_paged", "la_kv_commit_batch", "la_step_attention_rows", "la_step_attention_batch", "la_step_attention_batch_paged", "la_verify", "la_verify_step", "la_verify_step_batch", "la_verify_sample", "la_verify_sample_batch", "la_step_attention_workspace_bytes", "la_step_attention_kernel", "la_shutdown", "la_select_workspace", "la_debug_override", "la_probe_stream_read", "la_probe_mfma",
           "la_last_error", "la_version")


def _check(rc):
    if rc != LA_OK:
        raise LaError(rc, load().la_last_error().decode())


def _stream(stream):
    if stream is None:
        return torch.cuda.current_stream().cuda_stream
    if isinstance(stream, torch.cuda.Stream):
        return stream.cuda_stream
    return int(stream)


def la_step_attention(q, k_cache, v_cache, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim,
                      out, stream=None):
    """out[T, heads, head_dim] (bf16) <- lookahead-step attention; asynchronous on `stream`."""
    _native.step_attention(q, k_cache, v_cache, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim, out, stream)
    return out


def la_step_attention_noalloc(q, k_cache, v_cache, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim,
                              out, stream=None):
    """la_step_attention through the entry point that allocates nothing (fixed scratch block)."""
    _native.step_attention_noalloc(q, k_cache, v_cache, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim, out,
                                   stream)
    return out


def la_step_attention_fp8kv(q, k_cache, v_cache, step_k, step_v, k_scale, v_scale, P, W, N, G, heads, kv_heads,
                            head_dim, out, stream=None):
    """The step over a cache of 8-bit floats (uint8 codes, cache and step rows) with one fp32 scale per
    KV head for the keys and one for the values; q and out are bf16.  Asynchronous."""
    _native.step_attention_fp8kv(q, k_cache, v_cache, step_k, step_v, k_scale, v_scale, P, W, N, G, heads, kv_heads,
                                 head_dim, out, stream)
    return out


def la_step_attention_cap(q, k_cache, v_cache, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim, out,
                          stream=None):
    """la_step_attention over caches [kv_heads, capacity, head_dim] whose first P rows per head are
    the prefix (capacity is read from the tensors); asynchronous."""
    _native.step_attention_cap(q, k_cache, v_cache, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim, out, stream)
    return out


def la_step_rope(q, step_k, cos, sin, P, W, N, G, heads, kv_heads, head_dim, interleaved=False, stream=None):
    """Rotate q [T, heads, d] and step_k [T, kv_heads, d] (bf16, in place) by the step's positions with
    the fp32 tables cos, sin [max_pos, d/2]; asynchronous."""
    _native.step_rope(q, step_k, cos, sin, P, W, N, G, heads, kv_heads, head_dim, interleaved, stream)


def la_step_attention_rope(q, k_cache, v_cache, step_k, step_v, cos, sin, P, W, N, G, heads, kv_heads, head_dim, out,
                           interleaved=False, stream=None, rotate_keys=False):
    """la_step_attention with q rotated inside the kernel (q is left as it is).  rotate_keys False:
    step_k must be rotated already, e.g. by la_step_rope(None, step_k, ...); True: step_k comes
    unrotated too and the kernel turns the step keys it stages (append with la_kv_commit_rope then);
    asynchronous."""
    _native.step_attention_rope(q, k_cache, v_cache, step_k, step_v, cos, sin, P, W, N, G, heads, kv_heads, head_dim,
                                out, interleaved, rotate_keys, stream)
    return out


def la_kv_commit(k_cache, v_cache, step_k, step_v, P, W, N, G, kv_heads, head_dim, best, n_out, stream=None):
    """Append the rows of the tokens la_verify_step accepted (device-side best, n_out) to the caches
    [kv_heads, capacity, head_dim] at row P; asynchronous."""
    _native.kv_commit(k_cache, v_cache, step_k, step_v, P, W, N, G, kv_heads, head_dim, best, n_out, stream)


def la_kv_commit_rope(k_cache, v_cache, step_k, step_v, cos, sin, P, W, N, G, kv_heads, head_dim, best, n_out,
                      interleaved=False, stream=None):
    """la_kv_commit for unrotated step keys: the appended key rows are turned by their cache positions
    (tables as for la_step_rope); asynchronous."""
    _native.kv_commit_rope(k_cache, v_cache, step_k, step_v, cos, sin, P, W, N, G, kv_heads, head_dim, best, n_out,
                           interleaved, stream)


def la_step_attention_batch(seqs, W, N, G, heads, kv_heads, head_dim, stream=None):
    """Several steps in one launch.  `seqs` is a list of dicts with q, k_cache, v_cache, step_k,
    step_v, out (tensors as for la_step_attention) and P; asynchronous."""
    _native.step_attention_batch(seqs, W, N, G, heads, kv_heads, head_dim, stream)


def la_step_attention_batch_paged(seqs, k_pages, v_pages, W, N, G, heads, kv_heads, head_dim, stream=None):
    """Several steps over one paged cache in one launch.  `seqs`: dicts with q, block_table (int32
    tensor, >= ceil(P / page_size) entries, or None if P == 0), step_k, step_v, out, P; asynchronous."""
    _native.step_attention_batch_paged(seqs, k_pages, v_pages, W, N, G, heads, kv_heads, head_dim, stream)


def la_step_attention_rows(q, k_cache, v_cache, step_k, step_v, row_ids, P, W, N, G, heads, kv_heads, head_dim, out,
                           stream=None):
    """la_step_attention over the rows `row_ids` (int32 tensor) of the (W, N, G) layout: a device's
    share under lookahead parallelism; asynchronous."""
    _native.step_attention_rows(q, k_cache, v_cache, step_k, step_v, row_ids, P, W, N, G, heads, kv_heads, head_dim, out,
                                stream)
    return out


def la_step_attention_paged(q, k_pages, v_pages, block_table, step_k, step_v, P, W, N, G, heads, kv_heads,
                            head_dim, out, stream=None):
    """la_step_attention over pages [n_pages, kv_heads, page_size, head_dim] named by the int32
    block_table (>= ceil(P / page_size) entries); asynchronous."""
    _native.step_attention_paged(q, k_pages, v_pages, block_table, step_k, step_v, P, W, N, G, heads, kv_heads, head_dim,
                                 out, stream)
    return out


def la_kv_commit_paged(k_pages, v_pages, block_table, step_k, step_v, P, W, N, G, kv_heads, head_dim, best,
                       n_out, stream=None):
    """la_kv_commit into pages; block_table needs >= ceil((P + N) / page_size) entries; asynchronous."""
    _native.kv_commit_paged(k_pages, v_pages, block_table, step_k, step_v, P, W, N, G, kv_heads, head_dim, best, n_out, stream)


def la_kv_commit_batch(appends, W, N, G, kv_heads, head_dim, stream=None):
    """Several appends in one launch.  `appends`: dicts with k_cache, v_cache, step_k, step_v, best,
    n_out, P and, for a paged cache, block_table (then k_cache / v_cache are the page pools
    [n_pages, kv_heads, page_size, head_dim], the same geometry in all of them); asynchronous."""
    _native.kv_commit_batch(appends, W, N, G, kv_heads, head_dim, stream)


def la_verify(logits, cand_tokens, G, N, V, accept_len, accepted, stream=None):
    """accept_len[G], accepted[G, N-1] (int32) <- greedy verification; asynchronous."""
    _native.verify(logits, cand_tokens, G, N, V, accept_len, accepted, stream)
    return accept_len, accepted


def la_verify_step(logits_cur, logits_look, logits_cand, cand_tokens, W, N, G, V, out_tokens, n_out, best,
                   new_window, accept_len=None, stream=None):
    """out_tokens[N], n_out[1], best[1], new_window[W], accept_len[G] (int32) <- the end of a greedy
    step (accepted tokens of the best candidate plus correction or bonus token; new window tokens);
    asynchronous."""
    _native.verify_step(logits_cur, logits_look, logits_cand, cand_tokens, W, N, G, V, out_tokens, n_out, best, new_window,
                        accept_len, stream)
    return out_tokens, n_out, best, new_window, accept_len


def la_verify_step_batch(seqs, W, N, G, V, stream=None):
    """The ends of several sequences' steps in one launch.  `seqs`: dicts with logits_cur, logits_look,
    logits_cand, cand_tokens, out_tokens, n_out, best, new_window and optionally accept_len (tensors
    as for la_verify_step); asynchronous."""
    _native.verify_step_batch(seqs, W, N, G, V, stream)


def la_verify_sample(logits_cur, logits_cand, cand_tokens, u_test, u_final, temperature, N, G, V, out_tokens,
                     n_out, stream=None):
    """out_tokens[N], n_out[1] (int32) <- sampling verification (Algorithm 4); asynchronous."""
    _native.verify_sample(logits_cur, logits_cand, cand_tokens, u_test, u_final, temperature, N, G, V, out_tokens, n_out,
                          stream)
    return out_tokens, n_out


def la_verify_sample_batch(seqs, N, G, V, stream=None):
    """Sampling verification of several sequences in one launch.  `seqs`: dicts with logits_cur,
    logits_cand, cand_tokens, u_test, u_final, temperature, out_tokens, n_out (tensors as for
    la_verify_sample); asynchronous."""
    _native.verify_sample_batch(seqs, N, G, V, stream)


def la_step_attention_kernel(P, W, N, G, heads, kv_heads, head_dim):
    """0: the staged kernel, 1: the row-tile kernel (what la_step_attention takes for this shape)."""
    return int(load().la_step_attention_kernel(P, W, N, G, heads, kv_heads, head_dim))


def la_step_attention_workspace_bytes(P, W, N, G, heads, kv_heads, head_dim):
    return int(load().la_step_attention_workspace_bytes(P, W, N, G, heads, kv_heads, head_dim))


def la_shutdown():
    load().la_shutdown()


def la_select_workspace(index):
    """The calling thread's next calls use workspace set `index` (0..15): calls on different streams
    that may overlap need different sets."""
    _check(load().la_select_workspace(int(index)))


def la_version():
    return int(load().la_version())


def bf16_tensor(bits, device="cuda"):
    """numpy uint16 bit patterns -> bf16 tensor on the device (no value conversion)."""
    import numpy as np
    t = torch.from_numpy(np.ascontiguousarray(bits).view(np.int16).copy())
    return t.view(torch.bfloat16).to(device)


def bf16_bits(t):
    """bf16 tensor -> numpy uint16 bit patterns on the host."""
    import numpy as np
    return t.detach().contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def la_debug_override(key, value):
    """Testing hook: force a decomposition ("attn_plan", "batch_plan") or the recompute path
    ("force_recompute"); value None clears it."""
    _check(load().la_debug_override(key.encode(), None if value is None else str(value).encode()))


def la_probe_stream_read(buf, sink, stream=None):
    """Measurement aid: read every byte of the uint8 tensor `buf` once (asynchronous)."""
    _check(load().la_probe_stream_read(buf.data_ptr(), buf.numel() * buf.element_size(), sink.data_ptr(), _stream(stream)))


def la_probe_mfma(iters, sink, stream=None):
    """Measurement aid: a register-resident bf16 MFMA loop; returns the flops of the launch."""
    flops = load().la_probe_mfma(int(iters), sink.data_ptr(), _stream(stream))
    if flops < 0:
        raise LaError(LA_EHIP, load().la_last_error().decode())
    return int(flops)
