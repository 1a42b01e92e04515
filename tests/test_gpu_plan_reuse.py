"""Plans a context keeps from call to call: a call that repeats the host arrays of
the last one of its kind uses the plan already on the device, any other call (other
lengths, heads, speeds, stream, or after sa_reserve moved the buffers) plans again.
Every call in a sequence that alternates between them must give the bits a fresh
context gives."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_00151_amd as sa
from workloads.configs import build

from harness import build_cache, build_source_cache, compare, dev_u16, host_u16, layout_of

pytestmark = pytest.mark.gpu


def attend(fn, ctx, w, cache, stream=None):
    L = layout_of(w)
    kp, vp, ip, ix = cache
    T = int(w.qlen.sum())
    o = torch.full((T, w.num_q_heads, 128), -1, dtype=torch.int16, device="cuda")
    lse = torch.full((T, w.num_q_heads), float("nan"), dtype=torch.float32, device="cuda")
    q = dev_u16(w.q)
    if stream is not None:
        stream.wait_stream(torch.cuda.current_stream())
    fn(ctx, L, 0, q, kp, vp, w.qlen, w.kv, ip, ix, w.scale, o, lse, stream=stream)
    torch.cuda.synchronize()
    return o, lse


# same token counts, other splits between sequences, heads or rows; one that splits by key range
CASES = {
    "a": lambda: build("reuse_a", 301, 8, 2, 128, 16, [700, 40], [3, 60]),
    "b": lambda: build("reuse_b", 302, 8, 2, 128, 16, [40, 700], [60, 3]),
    "heads": lambda: build("reuse_h", 303, 8, 4, 128, 16, [700, 40], [3, 60]),
    "split": lambda: build("reuse_s", 304, 8, 1, 128, 32, [5000, 20], [1, 1]),
}


@pytest.mark.parametrize("entry", ["sa_segment_prefill_attn", "sa_segment_prefill_attn_noalloc"])
def test_attention_plans_reused_and_replaced(entry):
    fn = getattr(sa, entry)
    ws = {k: f() for k, f in CASES.items()}
    caches = {k: build_cache(w) for k, w in ws.items()}
    want = {}
    for k, w in ws.items():
        with sa.Context(0) as fresh:
            want[k] = attend(fn, fresh, w, caches[k])
    side = torch.cuda.Stream()
    with sa.Context(0) as ctx:
        steps = ["a", "a", "b", "a", "heads", "a", "split", "split", "a", "reserve", "a", "side", "a", "xcd", "a", "split"]
        for i, k in enumerate(steps):
            stream = None
            if k == "reserve":
                sa.sa_reserve(ctx, 1 << 20, 1 << 20)
                continue
            if k == "xcd":
                sa.sa_set_xcd_weights(ctx, [1.0, 0.9, 1.1, 1.0, 0.8, 1.0, 1.2, 1.0])
                continue
            if k == "side":
                k, stream = "a", side
            o, lse = attend(fn, ctx, ws[k], caches[k], stream)
            assert torch.equal(o, want[k][0]) and torch.equal(lse, want[k][1]), (i, k)
        sa.sa_sync_check(ctx)


def test_bad_lengths_are_refused_after_a_kept_plan():
    """A repeated call's checks: what the lengths of a kept plan do not cover is still refused."""
    w = CASES["a"]()
    cache = build_cache(w)
    L = layout_of(w)
    with sa.Context(0) as ctx:
        attend(sa.sa_segment_prefill_attn, ctx, w, cache)
        kp, vp, ip, ix = cache
        o = torch.zeros((int(w.qlen.sum()), 8, 128), dtype=torch.int16, device="cuda")
        for bad in (dict(layer=1), dict(scale=-1.0), dict(kv=np.array([2, 100]))):
            with pytest.raises(sa.SaError) as e:
                sa.sa_segment_prefill_attn(ctx, L, bad.get("layer", 0), dev_u16(w.q), kp, vp, w.qlen,
                                           bad.get("kv", w.kv), ip, ix, bad.get("scale", w.scale), o)
            assert e.value.name == "SA_ERR_SHAPE"
        with pytest.raises(sa.SaError) as e:
            sa._check(sa.load_library().sa_segment_prefill_attn(
                ctx.handle, sa.ctypes.byref(L), 0, None, kp.data_ptr(), vp.data_ptr(), w.batch,
                sa._host_i32(w.qlen).ctypes.data, sa._host_i32(w.kv).ctypes.data,
                sa._Pages(ip.data_ptr(), ix.data_ptr()), w.scale, o.data_ptr(), None, None))
        assert e.value.name == "SA_ERR_NULL"


@pytest.mark.parametrize("entry", ["sa_segment_prefill_attn", "sa_segment_prefill_attn_noalloc"])
def test_arrival_counters_left_off_are_reported_and_cleared(entry):
    """Counters that overlapping launches would leave off (set here from the host, between
    launches): sa_sync_check reports and clears them, and the next split launch is whole again."""
    fn = getattr(sa, entry)
    w = CASES["split"]()
    cache = build_cache(w)
    hip = sa.load_library()                                  # its HIP runtime's entry points too
    hip.hipMemcpy.restype = sa.ctypes.c_int
    with sa.Context(0) as ctx:
        want = attend(fn, ctx, w, cache)
        sa.sa_sync_check(ctx)
        head = (sa.ctypes.c_int32 * 2).from_address(ctx.handle.value)   # {device, compute units}, then the flag's address
        assert list(head) == [0, torch.cuda.get_device_properties(0).multi_processor_count]
        flag = sa.ctypes.c_uint64.from_address(ctx.handle.value + 8).value
        one = np.ones(1, dtype=np.int32)
        assert hip.hipMemcpy(sa.ctypes.c_void_p(flag + 256), sa.ctypes.c_void_p(one.ctypes.data), sa.ctypes.c_size_t(4), 1) == 0
        with pytest.raises(sa.SaError) as e:
            sa.sa_sync_check(ctx)
        assert e.value.name == "SA_ERR_OVERLAP"
        sa.sa_sync_check(ctx)
        o, lse = attend(fn, ctx, w, cache)
        assert torch.equal(o, want[0]) and torch.equal(lse, want[1])
        sa.sa_sync_check(ctx)


@pytest.mark.parametrize("entry", ["sa_segment_prefill_attn", "sa_segment_prefill_attn_noalloc"])
@pytest.mark.parametrize("batch", [200, 285, 291, 299, 583, 595, 1165, 1185])
def test_plans_of_one_and_several_copies(batch, entry):
    """One item a request (56 bytes of plan): plans around 16, 32 and 64 KB, which go to the device in
    one copy, in pieces or in one copy again; every row against the oracle."""
    r = np.random.default_rng(batch)
    w = build("pieces", 320 + batch, 2, 1, 128, 16, [int(x) for x in r.integers(0, 40, batch)], [1] * batch)
    with sa.Context(0) as ctx:
        o, lse = attend(getattr(sa, entry), ctx, w, build_cache(w))
        sa.sa_sync_check(ctx)
    ref, ref_lse, _ = oracle.attention_all(w.q, w.k, w.v, w.q_indptr, w.kv_indptr, 2, 1, w.scale)
    compare(host_u16(o), ref, 2e-2, 2e-3)
    assert np.abs(lse.cpu().numpy() - ref_lse).max() <= 1e-3


@pytest.mark.parametrize("mode", ["copy", "alias"])
def test_splice_and_append_plans_reused_and_replaced(mode):
    """Two batches of one shape but other spans, kept lengths and capacities, in turn on one context."""
    ws = [build("reuse_c", 311, 8, 2, 128, 16, [333, 90], [20, 70], assemble=True),
          build("reuse_d", 312, 8, 2, 128, 16, [320, 103], [33, 57], assemble=True)]

    def step(ctx, w):
        L = layout_of(w)
        kp, vp, sip, sid, fresh = build_source_cache(w)
        dip = torch.zeros(w.batch + 1, dtype=torch.int32, device="cuda")
        did = torch.full((len(w.asm.fresh),), -1, dtype=torch.int32, device="cuda")
        a, ks, vs = w.asm, dev_u16(w.k_seg()), dev_u16(w.v_seg())
        if mode == "alias":
            kept = sa.sa_kv_splice_alias(ctx, L, a.src_len, a.keep_indptr, a.keep_spans, a.reserve, sip, sid,
                                         fresh, dip, did)
        else:
            kept = sa.sa_kv_assemble(ctx, L, kp, vp, kp, vp, a.src_len, a.keep_indptr, a.keep_spans, a.reserve,
                                     sip, sid, fresh, dip, did)
        sa.sa_kv_append(ctx, L, 0, kp, vp, ks, vs, kept, w.qlen, dip, did)
        if mode == "copy":      # the same splice with the append in its launch replaces the kept splice plan
            again = sa.sa_kv_assemble_append(ctx, L, kp, vp, kp, vp, a.src_len, a.keep_indptr, a.keep_spans,
                                             a.reserve, sip, sid, fresh, dip, did, 0, ks, vs, w.qlen)
            assert np.array_equal(kept, again)
        sa.sa_sync_check(ctx)
        return [kept] + [t.cpu() for t in (kp, vp, dip, did)]

    want = []
    for w in ws:
        with sa.Context(0) as fresh_ctx:
            want.append(step(fresh_ctx, w))
    with sa.Context(0) as ctx:
        for i in (0, 0, 1, 0, 1, 1):
            got = step(ctx, ws[i])
            assert np.array_equal(got[0], want[i][0])
            assert all(torch.equal(x, y) for x, y in zip(got[1:], want[i][1:])), i
