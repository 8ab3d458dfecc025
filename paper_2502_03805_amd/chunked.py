"""Chunked prefill with eviction between chunks: a host loop over the three C-ABI calls.

After each chunk of the prompt the cache kept so far, followed by the chunk's new K/V rows, is scored with
the chunk's last W queries (causal inside the window, the window's own tokens protected), cut down to the
budget and compacted; the compacted cache, which the gather writes with the next chunk's rows behind it, is what the
next pass sees.  Only orchestration happens here; every step of each pass runs in the library's kernels.
"""
from __future__ import annotations

from typing import Callable, List, Sequence, Tuple

from . import binding as B


def _appendable(cache, new) -> bool:
    """Whether the gather can write `new`'s rows behind the kept ones itself (else they are concatenated)."""
    per16 = 16 // cache.element_size()
    return (new.dim() == 4 and new.shape[2] > 0 and new.shape[:2] == cache.shape[:2] and new.shape[3] == cache.shape[3] and
            new.dtype == cache.dtype and new.device == cache.device and new.stride(3) == 1 and new.data_ptr() % 16 == 0 and
            all(s % per16 == 0 for s in new.stride()[:3]))


def chunked_prefill_evict(make_desc: Callable[[int], "B.LayerDesc"], q_windows: Sequence, k_chunks: Sequence,
                          v_chunks: Sequence, w_o, budget: int, alpha: float, stream=None) -> Tuple[object, object, List]:
    """q_windows[c]: [b,H,W,d_h] last W queries of chunk c; k_chunks[c], v_chunks[c]: [b,Hkv,len_c,d_h].
    make_desc(n) builds the layer descriptor for n cached entries (flags should include CKV_CAUSAL_TAIL and
    CKV_PROTECT_WINDOW).  Returns (k_cache, v_cache, kept) where kept[c] is the idx tensor of chunk c's pass
    (positions in that pass's concatenated cache) or None when everything fitted the budget."""
    import torch
    chunks = iter(zip(q_windows, k_chunks, v_chunks))
    chunk = next(chunks, None)
    k_cache = v_cache = k_all = v_all = bud = None
    kept = []
    while chunk is not None:
        q_win, k_new, v_new = chunk
        if k_all is None: # (else written behind the kept rows by the pass before)
            k_all = k_new if k_cache is None else torch.cat([k_cache, k_new], dim=2).contiguous()
            v_all = v_new if v_cache is None else torch.cat([v_cache, v_new], dim=2).contiguous()
        chunk = next(chunks, None)
        b, Hkv, n, dh = k_all.shape
        if n <= budget:
            k_cache, v_cache = k_all, v_all
            k_all = v_all = None
            kept.append(None)
            continue
        desc = make_desc(n)
        ws = torch.empty(B.workspace_bytes(desc, budget), dtype=torch.uint8, device=k_all.device)
        attn = torch.empty((b, Hkv, n), dtype=torch.float32, device=k_all.device)
        crit = torch.empty_like(attn)
        idx = torch.empty((b, Hkv, budget), dtype=torch.int32, device=k_all.device)
        count = torch.empty((b, Hkv), dtype=torch.int32, device=k_all.device)
        if bud is None or bud.shape != (b, Hkv) or bud.device != k_all.device:
            bud = torch.full((b, Hkv), budget, dtype=torch.int32, device=k_all.device)
        B.criticalkv_score(desc, q_win, k_all, v_all, w_o, attn, crit, None, workspace=ws, stream=stream)
        B.criticalkv_select(desc, attn, crit, bud, alpha, budget, idx, count, workspace=ws, stream=stream)
        appended = (chunk is not None and chunk[1].shape == chunk[2].shape and _appendable(k_all, chunk[1]) and
                    _appendable(v_all, chunk[2]))
        rows = budget + (chunk[1].shape[2] if appended else 0)
        k_out = torch.empty((b, Hkv, rows, dh), dtype=k_all.dtype, device=k_all.device)
        v_out = torch.empty_like(k_out)
        if appended:
            B.criticalkv_compact_append(desc, k_all, v_all, idx, count, budget, chunk[1], chunk[2], k_out, v_out, stream=stream)
            k_all, v_all = k_out, v_out
        else:
            B.criticalkv_compact(desc, k_all, v_all, idx, count, budget, k_out, v_out, stream=stream)
            k_cache, v_cache = k_out, v_out
            k_all = v_all = None
        kept.append(idx)
    return k_cache, v_cache, kept
