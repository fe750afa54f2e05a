"""Decode launches whose shape is chosen by predicted time (paper Section 3, Eq. (3) over the packed
cache): head counts between and beyond one workgroup per CU, where the number of workgroups per head
and their size change with the token count, against the checker; and the workspace such calls want."""
import numpy as np
import pytest
import torch

from paper_2412_12706_amd import kvqp, synth
from tests.gpu_util import attn_excess, dev, upload_cache

pytestmark = pytest.mark.gpu


def cache_of(orc, B, Hkv, Gq, n, bits, axis=0, G=32, W=8, tau=0.0):
    L = n + W
    _, k, v = synth.prompt_host(B, Hkv * Gq, Hkv, L, W, 128, config=90 + bits)
    idx = np.broadcast_to(np.arange(n, dtype=np.int32), (B, Hkv, n)).copy()
    kw = dict(tau=tau, ovf_cap=512) if tau else {}
    oc = orc.quantize_selected(k, v, idx, W=W, bits=bits, G=G, key_axis=axis, **kw)
    cfg = kvqp.Cfg(batch=B, n_q_heads=Hkv * Gq, n_kv_heads=Hkv, seq_len=L, window=W, budget=n, bits=bits, group_size=G, key_axis=axis,
                   outlier_threshold=tau, outlier_overflow_cap=512 if tau else 0)
    return cfg, oc


@pytest.mark.parametrize("B,Hkv,Gq,n,bits,axis,tau", [
    (3, 8, 4, 1500, 4, 0, 0.0), (12, 8, 4, 1100, 4, 0, 0.0), (24, 8, 4, 700, 4, 0, 0.0), (24, 8, 2, 1300, 16, 0, 0.0),
    (40, 8, 2, 900, 4, 1, 0.0), (40, 8, 1, 640, 8, 0, 0.0), (4, 8, 8, 1500, 2, 1, 0.0), (28, 8, 8, 300, 2, 0, 0.0),
    (14, 8, 4, 600, 4, 0, 6.0), (65, 8, 1, 200, 2, 0, 0.0)])
def test_shapes_between_and_beyond_one_workgroup_per_cu(orc, B, Hkv, Gq, n, bits, axis, tau):
    print(f"case B={B} Hkv={Hkv} Gq={Gq} n={n} bits={bits} axis={axis} tau={tau}", flush=True)
    cfg, oc = cache_of(orc, B, Hkv, Gq, n, bits, axis=axis, tau=tau)
    gc = upload_cache(oc)
    ws = kvqp.alloc_decode_workspace(cfg)
    for step in range(2):
        q = synth.decode_query_host(B, cfg.n_q_heads, 128, config=91, step=step)
        ref = orc.decode_attn(q, oc, float(np.float32(cfg.sm_scale)))
        assert attn_excess(kvqp.decode_attn(cfg, dev(q), gc, workspace=ws), ref) <= 0
        out = torch.empty((B, cfg.n_q_heads, 128), dtype=torch.float16, device="cuda")
        kvqp.decode_attn_static(cfg, dev(q), gc, out)
        assert attn_excess(out, ref) <= 0


def test_a_workspace_that_holds_the_counters_only_still_serves_a_full_chip(orc):
    """320 heads fill the chip with one workgroup each, which needs the arrival counters and nothing
    else; a plan that splits heads for speed must not take that away, nor accept less."""
    print("case counters-only workspace", flush=True)
    cfg, oc = cache_of(orc, 40, 8, 2, 1200, 4)
    gc = upload_cache(oc)
    q = synth.decode_query_host(40, 16, 128, config=92)
    ref = orc.decode_attn(q, oc, float(np.float32(cfg.sm_scale)))
    counters = 320 * 4
    ws = kvqp.decode_workspace_init(cfg, kvqp.alloc_workspace((counters + 255) // 256 * 256))
    assert attn_excess(kvqp.decode_attn(cfg, dev(q), gc, workspace=ws), ref) <= 0
    with pytest.raises(kvqp.KvqpError):
        kvqp.decode_attn(cfg, dev(q), gc, workspace=ws[:-16])


def test_one_workspace_and_the_static_array_serve_head_counts_in_any_order(orc):
    """A split call leaves partial results in the workspace and its arrival counters at zero; neither
    may be in the way of a later call with more heads, whose counters reach further."""
    jobs = [cache_of(orc, B, 8, 2, n, 4) for B, n in ((12, 1100), (3, 1500), (24, 900))]
    ws = kvqp.decode_workspace_init(jobs[2][0], kvqp.alloc_workspace(max(kvqp.workspace_bytes(cfg)[1] for cfg, _ in jobs)))
    data = []
    for cfg, oc in jobs:
        q = synth.decode_query_host(cfg.batch, cfg.n_q_heads, 128, config=93)
        data.append((cfg, upload_cache(oc), dev(q), orc.decode_attn(q, oc, float(np.float32(cfg.sm_scale)))))
    for i in (1, 0, 2, 1, 2, 0):
        print(f"case order job {i}", flush=True)
        cfg, gc, q, ref = data[i]
        assert attn_excess(kvqp.decode_attn(cfg, q, gc, workspace=ws), ref) <= 0
        out = torch.empty((cfg.batch, cfg.n_q_heads, 128), dtype=torch.float16, device="cuda")
        kvqp.decode_attn_static(cfg, q, gc, out)
        assert attn_excess(out, ref) <= 0


@pytest.mark.parametrize("order", [(19, 44, 23, 43), (44, 19, 44, 23, 44)])
def test_splits_that_fill_the_stated_workspace_leave_other_calls_counters_alone(orc, order):
    """Batches whose splits use all the partials a workspace is stated for, on one workspace that is
    prepared once: every call's counters have to be zero when it starts, whichever came before."""
    jobs = {}
    for b in set(order):
        cfg, oc = cache_of(orc, b, 8, 2, 900, 4)
        q = synth.decode_query_host(b, 16, 128, config=94)
        jobs[b] = (cfg, upload_cache(oc), dev(q), orc.decode_attn(q, oc, float(np.float32(cfg.sm_scale))))
    ws = kvqp.decode_workspace_init(jobs[max(order)][0], kvqp.alloc_workspace(max(kvqp.workspace_bytes(cfg)[1] for cfg, *_ in jobs.values())))
    for b in order:
        print(f"case shared workspace batch {b} of {order}", flush=True)
        cfg, gc, q, ref = jobs[b]
        out = torch.full((b, 16, 128), float("nan"), dtype=torch.float16, device="cuda")   # (a head that is not merged stays)
        assert attn_excess(kvqp.decode_attn(cfg, q, gc, out, ws), ref) <= 0


@pytest.mark.parametrize("Hkv,Gq,n,bits,axis", [(8, 4, 1024, 4, 0), (2, 8, 3000, 8, 1), (4, 4, 700, 2, 0)])
def test_small_calls_in_workspaces_of_several_sizes(orc, Hkv, Gq, n, bits, axis):
    """Chunks of 32 tokens where their partial results have room behind the counters (the stated size); in less, down to this
    call's own counters and the plain rule's partials, the plain rule's launch.  The library's own array beside them."""
    cfg, oc = cache_of(orc, 1, Hkv, Gq, n, bits, axis=axis)
    gc = upload_cache(oc)
    q = synth.decode_query_host(1, Hkv * Gq, 128, config=95)
    ref = orc.decode_attn(q, oc, float(np.float32(cfg.sm_scale)))
    stated = kvqp.workspace_bytes(cfg)[1]
    room = kvqp.alloc_workspace(stated)
    taken = 0
    for size in [stated] + [256 + i * (stated - 65536 * 4) // 8 // 16 * 16 for i in range(9)]:
        print(f"case small call Hkv={Hkv} Gq={Gq} n={n} bits={bits} workspace={size} of {stated}", flush=True)
        ws = kvqp.decode_workspace_init(cfg, room[:size])
        out = torch.full((1, Hkv * Gq, 128), float("nan"), dtype=torch.float16, device="cuda")
        try:
            kvqp.decode_attn(cfg, dev(q), gc, out, ws)
        except kvqp.KvqpError:
            assert size < stated      # (fewer bytes than the plain rule's partials)
            continue
        taken += 1
        assert attn_excess(out, ref) <= 0, size
        assert attn_excess(kvqp.decode_attn(cfg, dev(q), gc, workspace=ws), ref) <= 0, size      # (the counters are back at zero)
    assert taken >= 2
    out = torch.empty((1, Hkv * Gq, 128), dtype=torch.float16, device="cuda")
    kvqp.decode_attn_static(cfg, dev(q), gc, out)
    assert attn_excess(out, ref) <= 0
