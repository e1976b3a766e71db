"""Argument marshalling of the binding's hot calls through ctypes: what ``csrc/marshal.cpp`` does, for a tree whose native module was
not built (it needs the headers of Python and torch, which the library itself does not).  A call takes 10 to 15 us longer on the
host.  Functions return the C call's code; a failed check raises AssertionError."""
from __future__ import annotations

import ctypes

import torch

from . import binding as b


def _rows(t):
    return t.dim() == 2 and t.is_contiguous()


def store(cache, K, V, page_table, slots):
    T = K.shape[0]
    assert K.dim() == 3 and K.dtype == V.dtype and K.shape == V.shape and K.stride(2) == 1 and K.stride(1) == cache.head_dim
    assert V.stride() == K.stride() and page_table.dtype == torch.int32 and slots.dtype == torch.int32
    assert _rows(page_table) and slots.is_contiguous() and slots.shape == (T, 2)
    st = cache.struct()
    return b.lib().saw_rotate_quant_store(ctypes.byref(st), b._ptr(K), b._ptr(V), b._DT[K.dtype], T,
                                          K.stride(0) if T > 1 else cache.n_kv_heads * cache.head_dim, b._ptr(page_table),
                                          page_table.shape[0], page_table.shape[1], b._ptr(slots), b._stream())


def store_layers(caches, Ks, Vs, page_table, slots):
    n = len(caches)
    c0, K0 = caches[0], Ks[0]
    T = K0.shape[0]
    stride = K0.stride(0) if T > 1 else c0.n_kv_heads * c0.head_dim
    assert len(Ks) == n == len(Vs) and K0.dim() == 3
    for K, V in zip(Ks, Vs):
        assert K.dtype == K0.dtype and K.shape == K0.shape == V.shape and K.stride(2) == 1 and K.stride(1) == c0.head_dim
        assert V.stride() == K.stride() and (T <= 1 or K.stride(0) == stride)
    assert _rows(page_table) and slots.is_contiguous() and slots.shape == (T, 2)
    sts = (b.SawCacheStruct * n)(*[c.struct() for c in caches])
    kp = (ctypes.c_void_p * n)(*[K.data_ptr() for K in Ks])
    vp = (ctypes.c_void_p * n)(*[V.data_ptr() for V in Vs])
    return b.lib().saw_rotate_quant_store_layers(sts, kp, vp, n, b._DT[K0.dtype], T, stride, b._ptr(page_table), page_table.shape[0],
                                                 page_table.shape[1], b._ptr(slots), b._stream())


def _hints(order, B):
    if order is None:
        return b.SawHints(None)
    assert order.dtype == torch.int32 and order.numel() == B and order.is_contiguous()
    return b.SawHints(order.data_ptr())


def decode(cache, q, page_table, seq_lens, max_seq_len, sm_scale, out, workspace, num_splits, order):
    B, Hq, _ = q.shape
    assert q.is_contiguous() and _rows(page_table) and seq_lens.dtype == torch.int32
    st, hints = cache.struct(), _hints(order, B)
    return b.lib().saw_paged_decode_attn_hinted(ctypes.byref(st), b._ptr(q), b._DT[q.dtype], B, Hq, b._ptr(page_table),
                                                page_table.shape[1], b._ptr(seq_lens), max_seq_len, float(sm_scale), b._ptr(out),
                                                b._DT[out.dtype], b._ptr(workspace), workspace.numel(), num_splits,
                                                ctypes.byref(hints), b._stream())


def append(cache, K_new, V_new, q, page_table, seq_lens, max_seq_len, sm_scale, out, workspace, order):
    B, Hq, _ = q.shape
    assert q.is_contiguous() and K_new.is_contiguous() and V_new.is_contiguous() and K_new.dtype == V_new.dtype
    assert _rows(page_table) and seq_lens.dtype == torch.int32
    st, hints = cache.struct(), _hints(order, B)
    return b.lib().saw_append_decode_attn_hinted(ctypes.byref(st), b._ptr(K_new), b._ptr(V_new), b._DT[K_new.dtype], b._ptr(q),
                                                 b._DT[q.dtype], B, Hq, b._ptr(page_table), page_table.shape[1], b._ptr(seq_lens),
                                                 max_seq_len, float(sm_scale), b._ptr(out), b._DT[out.dtype], b._ptr(workspace),
                                                 workspace.numel(), ctypes.byref(hints), b._stream())


def flatten(cache, page_table, seq, pos_begin, pos_end, unrotate, k_out, v_out):
    ref = k_out if k_out is not None else v_out
    stride = ref.stride(0) if pos_end > pos_begin else cache.n_kv_heads * cache.head_dim
    st = cache.struct()
    return b.lib().saw_flatten_dequant(ctypes.byref(st), b._ptr(page_table), page_table.shape[1], seq, pos_begin, pos_end,
                                       int(bool(unrotate)), b._DT[ref.dtype], b._ptr(k_out), b._ptr(v_out), stride, b._stream())


def kv16_decode(cache, q, page_table, seq_lens, max_seq_len, sm_scale, out, workspace, num_splits):
    B, Hq, _ = q.shape
    st = cache.struct()
    return b.lib().saw_kv16_paged_decode_attn(ctypes.byref(st), b._ptr(cache.k_pages), b._ptr(cache.v_pages), b._DT[cache.dtype],
                                              b._ptr(q), b._DT[q.dtype], B, Hq, b._ptr(page_table), page_table.shape[1],
                                              b._ptr(seq_lens), max_seq_len, float(sm_scale), b._ptr(out), b._DT[out.dtype],
                                              b._ptr(workspace), workspace.numel(), num_splits, b._stream())
