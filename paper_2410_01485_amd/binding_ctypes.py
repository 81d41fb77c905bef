"""The calls of csrc/lg_bind.cpp in Python over ctypes, for an interpreter or a torch that the extension module is not
built for: the same functions with the same arguments, checks and errors, each returning the lg_status of the call.  A
call takes the host a few microseconds longer."""
from .binding import _check, _check_lse, _cu_array, _dtype_code, _ptr, _stream, _ws_bytes, lib


def _rank(t, dims):
    import torch
    if not isinstance(t, torch.Tensor):
        raise TypeError("expected a torch tensor, got %s" % type(t).__name__)
    if len(t.shape) != dims:
        raise ValueError("expected a tensor of %d dimensions, got %s" % (dims, tuple(t.shape)))
    return t.shape


def _all(shape, like, *tensors):
    for t in tensors:
        _check(t, *shape, like=like)


def _lse(t, *shape):
    if t is not None:
        _check_lse(t, *shape)
    return _ptr(t)


def _offsets(cu_seqlens, total):
    cu, n = _cu_array(cu_seqlens)
    if cu[n] != total:
        raise ValueError("cu_seqlens ends at %d, the tensors hold %d tokens" % (cu[n], total))
    return cu, n


def fwd(q, k, v, out, lse, sink, window, block, stride, scale):
    (B, Hq, N, D), Hkv = _rank(q, 4), _rank(k, 4)[1]
    _all((B, Hq, N, D), q, q, out), _all((B, Hkv, N, D), q, k, v)
    return lib().lg_sparse_attn_fwd(_ptr(q), _ptr(k), _ptr(v), _ptr(out), _lse(lse, B, Hq, N), B, Hq, Hkv, N, D, sink,
                                    window, block, stride, _dtype_code(q), scale, _stream(q))


def bwd(q, k, v, out, lse, dout, dq, dk, dv, workspace, sink, window, block, stride, scale):
    (B, Hq, N, D), Hkv = _rank(q, 4), _rank(k, 4)[1]
    _all((B, Hq, N, D), q, q, out, dout, dq), _all((B, Hkv, N, D), q, k, v, dk, dv), _check_lse(lse, B, Hq, N)
    return lib().lg_sparse_attn_bwd(*map(_ptr, (q, k, v, out, lse, dout, dq, dk, dv, workspace)), _ws_bytes(workspace), B,
                                    Hq, Hkv, N, D, sink, window, block, stride, _dtype_code(q), scale, _stream(q))


def fwd_varlen(q, k, v, out, lse, cu_seqlens, sink, window, block, stride, scale):
    (Hq, T, D), Hkv = _rank(q, 3), _rank(k, 3)[0]
    cu, n = _offsets(cu_seqlens, T)
    _all((Hq, T, D), q, q, out), _all((Hkv, T, D), q, k, v)
    return lib().lg_sparse_attn_fwd_varlen(_ptr(q), _ptr(k), _ptr(v), _ptr(out), _lse(lse, Hq, T), cu, n, Hq, Hkv, D, sink,
                                           window, block, stride, _dtype_code(q), scale, _stream(q))


def bwd_varlen(q, k, v, out, lse, dout, dq, dk, dv, workspace, cu_seqlens, sink, window, block, stride, scale):
    (Hq, T, D), Hkv = _rank(q, 3), _rank(k, 3)[0]
    cu, n = _offsets(cu_seqlens, T)
    _all((Hq, T, D), q, q, out, dout, dq), _all((Hkv, T, D), q, k, v, dk, dv), _check_lse(lse, Hq, T)
    return lib().lg_sparse_attn_bwd_varlen(*map(_ptr, (q, k, v, out, lse, dout, dq, dk, dv, workspace)),
                                           _ws_bytes(workspace), cu, n, Hq, Hkv, D, sink, window, block, stride,
                                           _dtype_code(q), scale, _stream(q))


def _cached(q, k_cache, v_cache, out, lse, slots):
    (B, Hq, D), Hkv = _rank(q, 3), _rank(k_cache, 4)[1]
    _all((B, Hq, D), q, q, out), _all((B, Hkv, slots, D), q, k_cache, v_cache)
    return (_ptr(q), _ptr(k_cache), _ptr(v_cache), _ptr(out), _lse(lse, B, Hq)), (B, Hq, Hkv), D


def decode(q, k_cache, v_cache, out, lse, workspace, N, sink, window, block, stride, scale):
    ptrs, heads, D = _cached(q, k_cache, v_cache, out, lse, sink + window)
    return lib().lg_sparse_attn_decode(*ptrs, _ptr(workspace), _ws_bytes(workspace), *heads, N, D, sink, window, block,
                                       stride, _dtype_code(q), scale, _stream(q))


def decode_cache(q, k_cache, v_cache, out, lse, workspace, N, sink, window, block, stride, scale):
    slots = _rank(k_cache, 4)[2]
    ptrs, heads, D = _cached(q, k_cache, v_cache, out, lse, slots)
    return lib().lg_sparse_attn_decode_cache(*ptrs, _ptr(workspace), _ws_bytes(workspace), *heads, N, D, sink, window,
                                             block, stride, slots, _dtype_code(q), scale, _stream(q))


def decode_cache_static(q, k_cache, v_cache, out, lse, N, sink, window, block, stride, scale):
    slots = _rank(k_cache, 4)[2]
    ptrs, heads, D = _cached(q, k_cache, v_cache, out, lse, slots)
    return lib().lg_sparse_attn_decode_cache_static(*ptrs, *heads, N, D, sink, window, block, stride, slots,
                                                    _dtype_code(q), scale, _stream(q))


def ring_append(k_new, v_new, k_cache, v_cache, pos, sink, window, block, stride):
    (B, Hkv, T, D), slots = _rank(k_new, 4), _rank(k_cache, 4)[2]
    _all((B, Hkv, T, D), k_new, k_new, v_new), _all((B, Hkv, slots, D), k_new, k_cache, v_cache)
    return lib().lg_kv_ring_append(*map(_ptr, (k_new, v_new, k_cache, v_cache)), B, Hkv, D, T, pos, slots, sink, window,
                                   block, stride, _dtype_code(k_new), _stream(k_new))


def _ints(*tensors_and_shapes):
    import torch
    for t, shape in tensors_and_shapes:
        _check(t, *shape, dtype=torch.int32)


def decode_paged(q, k_pages, v_pages, page_table, seq_lens, out, lse, workspace, n_max, sink, window, block, stride, scale):
    (B, Hq, D), (pages, Hkv, ps, _), per_seq = _rank(q, 3), _rank(k_pages, 4), _rank(page_table, 2)[1]
    _all((B, Hq, D), q, q, out), _all((pages, Hkv, ps, D), q, k_pages, v_pages)
    _ints((page_table, (B, per_seq)), (seq_lens, (B,)))
    return lib().lg_sparse_attn_decode_paged(*map(_ptr, (q, k_pages, v_pages, page_table, seq_lens, out)),
                                             _lse(lse, B, Hq), _ptr(workspace), _ws_bytes(workspace), B, Hq, Hkv, n_max, D,
                                             sink, window, block, stride, ps, per_seq, pages, _dtype_code(q), scale,
                                             _stream(q))


def paged_append(k_new, v_new, k_pages, v_pages, page_table, positions, n_max, sink, window, block, stride):
    (B, Hkv, T, D), (pages, _, ps, _), per_seq = _rank(k_new, 4), _rank(k_pages, 4), _rank(page_table, 2)[1]
    _all((B, Hkv, T, D), k_new, k_new, v_new), _all((pages, Hkv, ps, D), k_new, k_pages, v_pages)
    _ints((page_table, (B, per_seq)), (positions, (B,)))
    return lib().lg_kv_paged_append(*map(_ptr, (k_new, v_new, k_pages, v_pages, page_table, positions)), B, Hkv, D, T,
                                    n_max, sink, window, block, stride, ps, per_seq, pages, _dtype_code(k_new),
                                    _stream(k_new))
