"""Python binding of liblynx.so (include/lynx.h): argument marshalling only.

Every function has the name and argument order of its C entry point.  Tensors
are torch CUDA tensors; their device pointers and the current HIP stream are
passed through ctypes.  Nothing here computes any part of the method: if the
library is missing the binding raises instead of falling back to anything.
"""
from __future__ import annotations

import ctypes
from dataclasses import dataclass
from pathlib import Path

import torch

LIBRARY = Path(__file__).resolve().parent / "liblynx.so"

LYNX_OK, LYNX_EINVAL, LYNX_ENOTSUP, LYNX_EWORKSPACE, LYNX_EHIP = 0, -1, -2, -3, -4
HEAD_DIM = 128
K_GROUP = 128
MAX_DRAFTS = 64


class LynxError(RuntimeError):
    def __init__(self, fn: str, status: int):
        self.status = status
        super().__init__(f"{fn} failed: {lynx_strerror(status)} ({status})")


class lynx_layout(ctypes.Structure):
    _fields_ = [("num_kv_heads", ctypes.c_int32), ("head_dim", ctypes.c_int32),
                ("k_group_tokens", ctypes.c_int32), ("block_tokens", ctypes.c_int32),
                ("max_blocks_per_seq", ctypes.c_int32), ("num_blocks", ctypes.c_int32),
                ("max_tokens", ctypes.c_int32)]


class lynx_meta(ctypes.Structure):
    _fields_ = [("k_scale", ctypes.c_void_p), ("k_zero", ctypes.c_void_p),
                ("v_scale", ctypes.c_void_p), ("v_zero", ctypes.c_void_p)]


_lib = None


_HMETA_NAMES = ("k_gmin", "k_gscale", "k_mu", "k_sigma", "v_gmin", "v_gscale", "v_mu", "v_sigma")


class lynx_hmeta(ctypes.Structure):
    _fields_ = [(name, ctypes.c_void_p) for name in _HMETA_NAMES]


def load():
    """Load liblynx.so (raises if it has not been built)."""
    global _lib
    if _lib is not None:
        return _lib
    if not LIBRARY.exists():
        raise RuntimeError(f"{LIBRARY} is not built: run `python -m paper_2607_01831_amd.build` "
                           "(or __graft_entry__.build()) first")
    lib = ctypes.CDLL(str(LIBRARY))
    P, I32, SZ = ctypes.c_void_p, ctypes.c_int32, ctypes.c_size_t
    LP, MP = ctypes.POINTER(lynx_layout), ctypes.POINTER(lynx_meta)
    sigs = {
        "lynx_kv_encode": ([LP, I32, I32, P, P, P, P, P, P, P, MP, P], ctypes.c_int),
        "lynx_kv_merge": ([P, P, P, SZ, P], ctypes.c_int),
        "lynx_attn_workspace_bytes": ([LP, I32, I32, I32, I32], SZ),
        "lynx_attn_anchor_decode": ([LP, I32, I32, I32, P, P, P, P, MP, P, P, P, P, SZ, P],
                                    ctypes.c_int),
        "lynx_attn_anchor_decode_split": ([I32, LP, I32, I32, I32, P, P, P, P, MP, P, P, P, P, SZ, P],
                                          ctypes.c_int),
        "lynx_attn_anchor_decode_noalloc": ([LP, I32, I32, I32, P, P, P, P, MP, P, P, P, P],
                                            ctypes.c_int),
        "lynx_attn_verify": ([LP, I32, I32, I32, I32, P, P, P, P, MP, P, P, P, P, P, SZ, P],
                             ctypes.c_int),
        "lynx_attn_anchor_decode_tail": ([LP, I32, I32, I32, P, P, P, P, MP, P, I32, P, P, P, P, P,
                                          SZ, P], ctypes.c_int),
        "lynx_spec_accept_workspace_bytes": ([I32, I32, I32], SZ),
        "lynx_spec_accept_greedy": ([I32, I32, I32, P, P, P, P, P, SZ, P], ctypes.c_int),
        "lynx_spec_accept_sample": ([I32, I32, I32, P, P, P, P, P, P, P, SZ, P], ctypes.c_int),
        "lynx_serialized_bytes": ([I32, I32, ctypes.POINTER(SZ), ctypes.POINTER(SZ)], ctypes.c_int),
        "lynx_kv_serialize": ([I32, I32, P, P, P, P, P], ctypes.c_int),
        "lynx_kv_deserialize_anchor": ([LP, I32, I32, I32, P, P, P, P, MP, P], ctypes.c_int),
        "lynx_kv_deserialize_residual": ([LP, I32, I32, I32, P, P, P, P, P, P, P], ctypes.c_int),
        "lynx_hkv_encode": ([LP, I32, I32, P, P, P, ctypes.c_float, I32, P, P, P, P,
                             ctypes.POINTER(lynx_hmeta), P], ctypes.c_int),
        "lynx_hkv_dequant": ([LP, I32, I32, P, I32, P, P, ctypes.c_float, I32,
                              ctypes.POINTER(lynx_hmeta), P, P, P], ctypes.c_int),
        "lynx_kv_encode_split": ([LP, I32, I32, I32, P, P, P, P, P, P, P, MP, P], ctypes.c_int),
        "lynx_kv_merge_split": ([I32, SZ, P, P, P, P], ctypes.c_int),
        "lynx_kv_dequant_anchor_split": ([LP, I32, I32, I32, P, P, P, MP, P, P, P], ctypes.c_int),
        "lynx_strerror": ([ctypes.c_int], ctypes.c_char_p),
    }
    for name, (args, res) in sigs.items():
        fn = getattr(lib, name)
        fn.argtypes = args
        fn.restype = res
    _lib = lib
    return lib


def lynx_strerror(status: int) -> str:
    return load().lynx_strerror(status).decode()


def _ptr(t):
    if t is None:
        return None
    if isinstance(t, int):
        return t
    if not t.is_cuda:
        raise ValueError("liblynx takes device tensors")
    if not t.is_contiguous():
        raise ValueError("liblynx takes contiguous tensors")
    return t.data_ptr()


def _stream(stream):
    if stream is None:
        if torch.cuda.is_initialized():
            # the same handle without a Stream object around it (1.4 us a call)
            return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
        return torch.cuda.current_stream().cuda_stream
    if isinstance(stream, torch.cuda.Stream):
        return stream.cuda_stream
    return stream


def _check(fn: str, status: int):
    if status != LYNX_OK:
        raise LynxError(fn, status)


# Size checks of the tensors a call reads or writes.  The C ABI sees only
# pointers, so a short tensor would become an out-of-bounds device access:
# the binding rejects it first.  A call makes a dozen of these, and a short
# kernel waits for them (the checks and the pointers in one function each,
# sizes computed once a call: an anchor decode 14.2 -> 10.5 us on the host).
def _arg(fn: str, what: str, t, nbytes: int):
    """The device pointer of tensor `t`, which holds at least nbytes bytes; an
    int is a pointer already, None is NULL."""
    if t is None:
        return None
    if isinstance(t, int):
        return t
    if t.nbytes < nbytes:
        raise ValueError(f"{fn}: {what} holds {t.nbytes} bytes; the call uses {nbytes}")
    if not t.is_cuda:
        raise ValueError("liblynx takes device tensors")
    if not t.is_contiguous():
        raise ValueError("liblynx takes contiguous tensors")
    return t.data_ptr()


def _meta_arg(fn: str, L: "Layout", meta: "Meta", rows: int) -> lynx_meta:
    """fp32 metadata rows 0 .. rows - 1 (sequences) of the layout."""
    heads = rows * L.num_kv_heads
    k = heads * -(-L.max_tokens // K_GROUP) * HEAD_DIM * 4
    v = heads * L.max_tokens * 4
    return lynx_meta(_arg(fn, "meta.k_scale", meta.k_scale, k), _arg(fn, "meta.k_zero", meta.k_zero, k),
                     _arg(fn, "meta.v_scale", meta.v_scale, v), _arg(fn, "meta.v_zero", meta.v_zero, v))


def _hmeta_arg(fn: str, L: "Layout", hmeta: "HMeta", rows: int) -> lynx_hmeta:
    heads = rows * L.num_kv_heads
    page = heads * -(-L.max_tokens // 256) * HEAD_DIM * 4
    chunk = heads * -(-L.max_tokens // 32) * HEAD_DIM * 4
    return lynx_hmeta(*(_arg(fn, f"hmeta.{name}", getattr(hmeta, name), page if name[2] == "g" else chunk)
                        for name in _HMETA_NAMES))


def _attn_args(fn: str, L: "Layout", B: int, Hq: int, seq_lens, block_table, k_plane, v_plane, row_bytes: int,
               meta: "Meta", q, nq: int = 1):
    """The arguments every attention call starts with, up to q."""
    if B <= 0:
        return (ctypes.byref(L.c()),), (_ptr(seq_lens), _ptr(block_table), _ptr(k_plane), _ptr(v_plane),
                                        ctypes.byref(meta.c()), _ptr(q))
    plane = L.plane_bytes(row_bytes)
    return (ctypes.byref(L.c()),), (
        _arg(fn, "seq_lens", seq_lens, B * 4),
        _arg(fn, "block_table", block_table, B * L.max_blocks_per_seq * 4),
        _arg(fn, "plane 0", k_plane, plane), _arg(fn, "plane 1", v_plane, plane),
        ctypes.byref(_meta_arg(fn, L, meta, B)), _arg(fn, "q", q, B * nq * Hq * HEAD_DIM * 2))


@dataclass
class Layout:
    """Cache geometry (see lynx_layout in include/lynx.h)."""
    num_kv_heads: int
    block_tokens: int
    max_blocks_per_seq: int
    num_blocks: int
    max_tokens: int
    head_dim: int = HEAD_DIM
    k_group_tokens: int = K_GROUP

    def c(self) -> lynx_layout:
        return lynx_layout(self.num_kv_heads, self.head_dim, self.k_group_tokens,
                           self.block_tokens, self.max_blocks_per_seq, self.num_blocks,
                           self.max_tokens)

    @property
    def n_groups(self) -> int:
        return -(-self.max_tokens // K_GROUP)

    def plane_bytes(self, row_bytes: int = 64) -> int:
        return self.num_blocks * self.num_kv_heads * self.block_tokens * row_bytes


@dataclass
class Meta:
    """fp32 metadata tensors of a batch (device)."""
    k_scale: torch.Tensor  # [B][Hkv][n_groups][128]
    k_zero: torch.Tensor
    v_scale: torch.Tensor  # [B][Hkv][max_tokens]
    v_zero: torch.Tensor

    @staticmethod
    def empty(L: Layout, B: int, device="cuda") -> "Meta":
        ks = (B, L.num_kv_heads, L.n_groups, HEAD_DIM)
        vs = (B, L.num_kv_heads, L.max_tokens)
        f = dict(dtype=torch.float32, device=device)
        return Meta(torch.zeros(ks, **f), torch.zeros(ks, **f), torch.zeros(vs, **f),
                    torch.zeros(vs, **f))

    def c(self) -> lynx_meta:
        return lynx_meta(_ptr(self.k_scale), _ptr(self.k_zero), _ptr(self.v_scale),
                         _ptr(self.v_zero))


def lynx_kv_encode(L: Layout, b: int, T: int, block_table, k, v, k_anc, v_anc, k_res, v_res,
                   meta: Meta, stream=None) -> None:
    fn = "lynx_kv_encode"
    n, plane = T * L.num_kv_heads * HEAD_DIM * 2, L.plane_bytes(64)
    _check(fn, load().lynx_kv_encode(
        ctypes.byref(L.c()), b, T, _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4),
        _arg(fn, "k", k, n), _arg(fn, "v", v, n), _arg(fn, "k_anc", k_anc, plane), _arg(fn, "v_anc", v_anc, plane),
        _arg(fn, "k_res", k_res, plane), _arg(fn, "v_res", v_res, plane),
        ctypes.byref(_meta_arg(fn, L, meta, b + 1)), _stream(stream)))


def lynx_kv_merge(anc, res, codes, n_packed_bytes: int | None = None, stream=None) -> None:
    n = anc.numel() if n_packed_bytes is None else n_packed_bytes
    if n > anc.numel() or n > res.numel() or 2 * n > codes.numel():
        raise ValueError("lynx_kv_merge: the planes hold fewer bytes than asked for")
    _check("lynx_kv_merge", load().lynx_kv_merge(_ptr(anc), _ptr(res), _ptr(codes), n,
                                                 _stream(stream)))


def lynx_attn_workspace_bytes(L: Layout, B: int, Hq: int, num_queries: int,
                              max_seq_len: int) -> int:
    lay = L.c()
    return int(load().lynx_attn_workspace_bytes(ctypes.byref(lay), B, Hq, num_queries,
                                                 max_seq_len))


# Arrival counters at the head of every attention workspace (lynx.h).
ATTN_COUNTER_BYTES = 262144


def workspace(L: Layout, B: int, Hq: int, num_queries: int, max_seq_len: int,
              device="cuda") -> torch.Tensor:
    """A device buffer of lynx_attn_workspace_bytes() bytes (allocated by
    torch), zero-filled: the arrival counters at its head must start at zero."""
    n = lynx_attn_workspace_bytes(L, B, Hq, num_queries, max_seq_len)
    return torch.zeros(max(n, ATTN_COUNTER_BYTES), dtype=torch.uint8, device=device)


def lynx_attn_anchor_decode(L: Layout, B: int, Hq: int, max_seq_len: int, seq_lens,
                            block_table, k_anc, v_anc, meta: Meta, q, out, lse=None,
                            workspace_buf=None, stream=None) -> None:
    fn = "lynx_attn_anchor_decode"
    lay, args = _attn_args(fn, L, B, Hq, seq_lens, block_table, k_anc, v_anc, 64, meta, q)
    ws = workspace_buf
    _check(fn, load().lynx_attn_anchor_decode(
        *lay, B, Hq, max_seq_len, *args, _arg(fn, "out", out, B * Hq * HEAD_DIM * 2), _arg(fn, "lse", lse, B * Hq * 4),
        _ptr(ws), 0 if ws is None else ws.nbytes, _stream(stream)))


def lynx_attn_anchor_decode_split(anchor_bits: int, L: Layout, B: int, Hq: int, max_seq_len: int,
                                  seq_lens, block_table, k_anc, v_anc, meta: Meta, q, out, lse=None,
                                  workspace_buf=None, stream=None) -> None:
    """Decode over the A-bit anchor planes of a split width (rows of 16 A bytes)."""
    fn = "lynx_attn_anchor_decode_split"
    if anchor_bits not in (2, 4, 6):
        raise LynxError(fn, LYNX_EINVAL)
    lay, args = _attn_args(fn, L, B, Hq, seq_lens, block_table, k_anc, v_anc, 16 * anchor_bits, meta, q)
    ws = workspace_buf
    _check(fn, load().lynx_attn_anchor_decode_split(
        anchor_bits, *lay, B, Hq, max_seq_len, *args, _arg(fn, "out", out, B * Hq * HEAD_DIM * 2),
        _arg(fn, "lse", lse, B * Hq * 4), _ptr(ws), 0 if ws is None else ws.nbytes, _stream(stream)))


# Scratch held by the library for lynx_attn_anchor_decode_noalloc (lynx.h).
NOALLOC_SCRATCH_BYTES = 16 << 20


def lynx_attn_anchor_decode_noalloc(L: Layout, B: int, Hq: int, max_seq_len: int, seq_lens,
                                    block_table, k_anc, v_anc, meta: Meta, q, out, lse=None,
                                    stream=None) -> None:
    """lynx_attn_anchor_decode without a workspace: the library's own static
    scratch (calls that overlap on one GPU race)."""
    fn = "lynx_attn_anchor_decode_noalloc"
    lay, args = _attn_args(fn, L, B, Hq, seq_lens, block_table, k_anc, v_anc, 64, meta, q)
    _check(fn, load().lynx_attn_anchor_decode_noalloc(
        *lay, B, Hq, max_seq_len, *args, _arg(fn, "out", out, B * Hq * HEAD_DIM * 2),
        _arg(fn, "lse", lse, B * Hq * 4), _stream(stream)))


def lynx_attn_anchor_decode_tail(L: Layout, B: int, Hq: int, max_seq_len: int, seq_lens,
                                 block_table, k_anc, v_anc, meta: Meta, q, k_tail, v_tail, out,
                                 lse=None, workspace_buf=None, stream=None) -> None:
    """Anchor decode that also attends the BF16 tail k_tail / v_tail
    ([B][n_tail][Hkv][128], or None for n_tail = 0)."""
    fn = "lynx_attn_anchor_decode_tail"
    lay, args = _attn_args(fn, L, B, Hq, seq_lens, block_table, k_anc, v_anc, 64, meta, q)
    n_tail = 0 if k_tail is None else int(k_tail.shape[1])
    n = B * n_tail * L.num_kv_heads * HEAD_DIM * 2
    ws = workspace_buf
    _check(fn, load().lynx_attn_anchor_decode_tail(
        *lay, B, Hq, max_seq_len, *args, n_tail, _arg(fn, "k_tail", k_tail, n),
        _ptr(v_tail) if k_tail is None else _arg(fn, "v_tail", v_tail, n), _arg(fn, "out", out, B * Hq * HEAD_DIM * 2),
        _arg(fn, "lse", lse, B * Hq * 4), _ptr(ws), 0 if ws is None else ws.nbytes, _stream(stream)))


def lynx_spec_accept_workspace_bytes(B: int, k: int, vocab: int) -> int:
    return int(load().lynx_spec_accept_workspace_bytes(B, k, vocab))


def lynx_spec_accept_greedy(target_logits, draft_tokens, accepted, next_token,
                            workspace_buf=None, stream=None) -> None:
    """target_logits fp32 [B][k+1][V], draft_tokens int32 [B][k]; writes
    accepted and next_token (int32 [B]).  workspace_buf: None allocates
    lynx_spec_accept_workspace_bytes() bytes with torch."""
    B, k1, V = (int(x) for x in target_logits.shape)
    ws = workspace_buf
    if ws is None:
        n = lynx_spec_accept_workspace_bytes(B, k1 - 1, V)
        ws = torch.empty(max(n, 16), dtype=torch.uint8, device=target_logits.device)
    _check("lynx_spec_accept_greedy", load().lynx_spec_accept_greedy(
        B, k1 - 1, V, _ptr(target_logits), _ptr(draft_tokens), _ptr(accepted), _ptr(next_token),
        _ptr(ws), ws.nbytes, _stream(stream)))


def lynx_spec_accept_sample(target_probs, draft_probs, draft_tokens, uniforms, accepted,
                            next_token, workspace_buf=None, stream=None) -> None:
    """target_probs fp32 [B][k+1][V], draft_probs fp32 [B][k][V], draft_tokens
    int32 [B][k], uniforms fp32 [B][k+1]; writes accepted and next_token
    (int32 [B]).  workspace_buf: None allocates
    lynx_spec_accept_workspace_bytes() bytes with torch."""
    B, k1, V = (int(x) for x in target_probs.shape)
    ws = workspace_buf
    if ws is None:
        n = lynx_spec_accept_workspace_bytes(B, k1 - 1, V)
        ws = torch.empty(max(n, 16), dtype=torch.uint8, device=target_probs.device)
    _check("lynx_spec_accept_sample", load().lynx_spec_accept_sample(
        B, k1 - 1, V, _ptr(target_probs), _ptr(draft_probs), _ptr(draft_tokens), _ptr(uniforms),
        _ptr(accepted), _ptr(next_token), _ptr(ws), ws.nbytes, _stream(stream)))


def lynx_attn_verify(L: Layout, B: int, Hq: int, k: int, max_seq_len: int, seq_lens,
                     block_table, k_codes, v_codes, meta: Meta, q, k_new, v_new, out,
                     workspace_buf=None, stream=None) -> None:
    fn = "lynx_attn_verify"
    lay, args = _attn_args(fn, L, B, Hq, seq_lens, block_table, k_codes, v_codes, 128, meta, q, k)
    n = B * k * L.num_kv_heads * HEAD_DIM * 2
    ws = workspace_buf
    _check(fn, load().lynx_attn_verify(
        *lay, B, Hq, k, max_seq_len, *args, _arg(fn, "k_new", k_new, n), _arg(fn, "v_new", v_new, n),
        _arg(fn, "out", out, B * k * Hq * HEAD_DIM * 2), _ptr(ws), 0 if ws is None else ws.nbytes, _stream(stream)))


# ----------------------------------------------------------------------------
# Allocation helpers (torch device memory only)
# ----------------------------------------------------------------------------

@dataclass
class HMeta:
    """fp32 metadata of the hierarchical codec (device): page minimum and
    range [B][Hkv][ceil(max_tokens/256)][128], chunk mean and scale
    [B][Hkv][ceil(max_tokens/32)][128], for K and V."""
    k_gmin: torch.Tensor
    k_gscale: torch.Tensor
    k_mu: torch.Tensor
    k_sigma: torch.Tensor
    v_gmin: torch.Tensor
    v_gscale: torch.Tensor
    v_mu: torch.Tensor
    v_sigma: torch.Tensor

    @staticmethod
    def empty(L: Layout, B: int, device="cuda") -> "HMeta":
        pg = (B, L.num_kv_heads, -(-L.max_tokens // 256), HEAD_DIM)
        ch = (B, L.num_kv_heads, -(-L.max_tokens // 32), HEAD_DIM)
        z = lambda shape: torch.zeros(shape, dtype=torch.float32, device=device)
        return HMeta(z(pg), z(pg), z(ch), z(ch), z(pg), z(pg), z(ch), z(ch))

    def c(self) -> lynx_hmeta:
        return lynx_hmeta(*(_ptr(getattr(self, f)) for f, _ in lynx_hmeta._fields_))


def lynx_kv_encode_split(L: Layout, anchor_bits: int, b: int, T: int, block_table, k, v, k_anc, v_anc,
                         k_res, v_res, meta: Meta, stream=None) -> None:
    """k, v: BF16 [T][Hkv][128]; planes: uint8 device tensors of rows of
    16 anchor_bits (anchor) and 16 (8 - anchor_bits) (residual) bytes."""
    fn = "lynx_kv_encode_split"
    n = T * L.num_kv_heads * HEAD_DIM * 2
    # (a width that the library rejects needs no plane)
    wa, wr = (anchor_bits, 8 - anchor_bits) if 0 < anchor_bits < 8 else (0, 0)
    anc, res = L.plane_bytes(16 * wa), L.plane_bytes(16 * wr)
    _check(fn, load().lynx_kv_encode_split(
        ctypes.byref(L.c()), anchor_bits, b, T,
        _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4), _arg(fn, "k", k, n),
        _arg(fn, "v", v, n), _arg(fn, "k_anc", k_anc, anc), _arg(fn, "v_anc", v_anc, anc),
        _arg(fn, "k_res", k_res, res), _arg(fn, "v_res", v_res, res),
        ctypes.byref(_meta_arg(fn, L, meta, b + 1)), _stream(stream)))


def lynx_kv_merge_split(anchor_bits: int, anc, res, codes, stream=None) -> None:
    """Rows of A-bit anchors and (8 - A)-bit residuals -> rows of 128 codes."""
    n_rows = anc.numel() // (16 * anchor_bits)
    if (anc.numel() != n_rows * 16 * anchor_bits or res.numel() != n_rows * 16 * (8 - anchor_bits)
            or codes.numel() < n_rows * 128):
        raise ValueError("lynx_kv_merge_split: plane sizes do not match one another")
    _check("lynx_kv_merge_split", load().lynx_kv_merge_split(
        anchor_bits, n_rows, _ptr(anc), _ptr(res), _ptr(codes), _stream(stream)))


def lynx_kv_dequant_anchor_split(L: Layout, anchor_bits: int, b: int, T: int, block_table, k_anc, v_anc,
                                 meta: Meta, k_out, v_out, stream=None) -> None:
    """k_out, v_out: BF16 [T][Hkv][128] (device, written)."""
    fn = "lynx_kv_dequant_anchor_split"
    n = T * L.num_kv_heads * HEAD_DIM * 2
    anc = L.plane_bytes(16 * anchor_bits) if 0 < anchor_bits < 8 else 0
    _check(fn, load().lynx_kv_dequant_anchor_split(
        ctypes.byref(L.c()), anchor_bits, b, T,
        _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4), _arg(fn, "k_anc", k_anc, anc),
        _arg(fn, "v_anc", v_anc, anc), ctypes.byref(_meta_arg(fn, L, meta, b + 1)), _arg(fn, "k_out", k_out, n),
        _arg(fn, "v_out", v_out, n), _stream(stream)))


# codec variants of the hierarchical codec (lynx.h LYNX_HQ_*)
LYNX_HQ_BIASED, LYNX_HQ_CENTRED, LYNX_HQ_INT4 = 0, 1, 2


def lynx_hkv_encode(L: Layout, b: int, T: int, block_table, k, v, alpha: float, variant: int,
                    k_anc, v_anc, k_res, v_res, hmeta: HMeta, stream=None) -> None:
    """k_res, v_res may be None for LYNX_HQ_INT4."""
    fn = "lynx_hkv_encode"
    n, plane = T * L.num_kv_heads * HEAD_DIM * 2, L.plane_bytes(64)
    _check(fn, load().lynx_hkv_encode(
        ctypes.byref(L.c()), b, T, _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4),
        _arg(fn, "k", k, n), _arg(fn, "v", v, n), alpha, variant, _arg(fn, "k_anc", k_anc, plane),
        _arg(fn, "v_anc", v_anc, plane), _arg(fn, "k_res", k_res, plane), _arg(fn, "v_res", v_res, plane),
        ctypes.byref(_hmeta_arg(fn, L, hmeta, b + 1)), _stream(stream)))


def lynx_hkv_dequant(L: Layout, b: int, T: int, block_table, full: bool, k_plane, v_plane,
                     alpha: float, variant: int, hmeta: HMeta, k_out, v_out, stream=None) -> None:
    """k_out, v_out: BF16 [T][Hkv][128] (device, written)."""
    fn = "lynx_hkv_dequant"
    n, plane = T * L.num_kv_heads * HEAD_DIM * 2, L.plane_bytes(128 if full else 64)
    _check(fn, load().lynx_hkv_dequant(
        ctypes.byref(L.c()), b, T, _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4),
        1 if full else 0, _arg(fn, "k_plane", k_plane, plane), _arg(fn, "v_plane", v_plane, plane), alpha, variant,
        ctypes.byref(_hmeta_arg(fn, L, hmeta, b + 1)), _arg(fn, "k_out", k_out, n), _arg(fn, "v_out", v_out, n),
        _stream(stream)))


def lynx_serialized_bytes(num_kv_heads: int, n_tokens: int) -> tuple[int, int]:
    """(anchor_bytes, residual_bytes) of an object of n_tokens tokens."""
    a, r = ctypes.c_size_t(), ctypes.c_size_t()
    _check("lynx_serialized_bytes", load().lynx_serialized_bytes(num_kv_heads, n_tokens,
                                                                 ctypes.byref(a), ctypes.byref(r)))
    return int(a.value), int(r.value)


def lynx_kv_serialize(num_kv_heads: int, n_tokens: int, k, v, anchor_buf, residual_buf,
                      stream=None) -> None:
    """k, v: BF16 [n_tokens][Hkv][128] (an object's tokens); the buffers are
    uint8 device tensors of lynx_serialized_bytes() bytes."""
    fn = "lynx_kv_serialize"
    n, na, nr = n_tokens * num_kv_heads * HEAD_DIM * 2, 0, 0
    if num_kv_heads > 0 and n_tokens > 0:
        na, nr = lynx_serialized_bytes(num_kv_heads, n_tokens)
    _check(fn, load().lynx_kv_serialize(
        num_kv_heads, n_tokens, _arg(fn, "k", k, n), _arg(fn, "v", v, n), _arg(fn, "anchor_buf", anchor_buf, na),
        _arg(fn, "residual_buf", residual_buf, nr), _stream(stream)))


def lynx_kv_deserialize_anchor(L: Layout, b: int, t0: int, n_tokens: int, block_table, anchor_buf,
                               k_anc, v_anc, meta: Meta, stream=None) -> None:
    fn = "lynx_kv_deserialize_anchor"
    na = lynx_serialized_bytes(L.num_kv_heads, n_tokens)[0] if n_tokens > 0 else 0
    plane = L.plane_bytes(64)
    _check(fn, load().lynx_kv_deserialize_anchor(
        ctypes.byref(L.c()), b, t0, n_tokens,
        _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4),
        _arg(fn, "anchor_buf", anchor_buf, na), _arg(fn, "k_anc", k_anc, plane), _arg(fn, "v_anc", v_anc, plane),
        ctypes.byref(_meta_arg(fn, L, meta, b + 1)), _stream(stream)))


def lynx_kv_deserialize_residual(L: Layout, b: int, t0: int, n_tokens: int, block_table,
                                 residual_buf, k_anc, v_anc, k_codes, v_codes,
                                 stream=None) -> None:
    fn = "lynx_kv_deserialize_residual"
    nr = lynx_serialized_bytes(L.num_kv_heads, n_tokens)[1] if n_tokens > 0 else 0
    plane = L.plane_bytes(64)
    _check(fn, load().lynx_kv_deserialize_residual(
        ctypes.byref(L.c()), b, t0, n_tokens,
        _arg(fn, "block_table", block_table, (b + 1) * L.max_blocks_per_seq * 4),
        _arg(fn, "residual_buf", residual_buf, nr), _arg(fn, "k_anc", k_anc, plane), _arg(fn, "v_anc", v_anc, plane),
        _arg(fn, "k_codes", k_codes, 2 * plane), _arg(fn, "v_codes", v_codes, 2 * plane), _stream(stream)))


@dataclass
class KVPool:
    """Nibble planes, metadata and (after merge) code planes of one layer."""
    layout: Layout
    B: int
    k_anc: torch.Tensor
    v_anc: torch.Tensor
    k_res: torch.Tensor
    v_res: torch.Tensor
    meta: Meta
    k_codes: torch.Tensor | None = None
    v_codes: torch.Tensor | None = None

    @staticmethod
    def allocate(L: Layout, B: int, device="cuda", codes: bool = True) -> "KVPool":
        n = L.plane_bytes(64)
        u8 = dict(dtype=torch.uint8, device=device)
        pool = KVPool(L, B, torch.zeros(n, **u8), torch.zeros(n, **u8), torch.zeros(n, **u8),
                      torch.zeros(n, **u8), Meta.empty(L, B, device))
        if codes:
            pool.k_codes = torch.zeros(2 * n, **u8)
            pool.v_codes = torch.zeros(2 * n, **u8)
        return pool

    @staticmethod
    def allocate_layers(L: Layout, B: int, layers: int, device="cuda", codes: bool = True):
        """Pools for `layers` layers whose planes are consecutive slices of one
        allocation per plane kind, so that a whole cache's residual planes can
        be transported and merged in one call each.  Returns (pools, whole),
        whole being a KVPool-like record of the full-length planes (its meta
        is that of layer 0 and is not used)."""
        n = L.plane_bytes(64)
        u8 = dict(dtype=torch.uint8, device=device)
        big = {name: torch.zeros(layers * n, **u8) for name in ("k_anc", "v_anc", "k_res", "v_res")}
        if codes:
            big["k_codes"] = torch.zeros(layers * 2 * n, **u8)
            big["v_codes"] = torch.zeros(layers * 2 * n, **u8)
        pools = []
        for l in range(layers):
            pool = KVPool(L, B, *(big[name][l * n:(l + 1) * n] for name in ("k_anc", "v_anc", "k_res", "v_res")),
                          Meta.empty(L, B, device))
            if codes:
                pool.k_codes = big["k_codes"][l * 2 * n:(l + 1) * 2 * n]
                pool.v_codes = big["v_codes"][l * 2 * n:(l + 1) * 2 * n]
            pools.append(pool)
        whole = KVPool(L, B, big["k_anc"], big["v_anc"], big["k_res"], big["v_res"], pools[0].meta,
                       big.get("k_codes"), big.get("v_codes"))
        return pools, whole

    def encode(self, b: int, T: int, block_table, k, v, stream=None) -> None:
        lynx_kv_encode(self.layout, b, T, block_table, k, v, self.k_anc, self.v_anc, self.k_res,
                       self.v_res, self.meta, stream)

    def merge(self, stream=None) -> None:
        lynx_kv_merge(self.k_anc, self.k_res, self.k_codes, stream=stream)
        lynx_kv_merge(self.v_anc, self.v_res, self.v_codes, stream=stream)


def contiguous_layout(Hkv: int, B: int, T: int) -> Layout:
    """One block of T tokens per sequence; block_table[b] = [b]."""
    return Layout(num_kv_heads=Hkv, block_tokens=T, max_blocks_per_seq=1, num_blocks=B,
                  max_tokens=T)
