"""Split items merged inside the attention launch, and the decode path at the edges of
its blocks: rows 1 to 32 of a request (one or two 16-row blocks, query-head counts that
do not divide the merging threads), parts of a few tiles, parts whose keys some rows do
not see, lengths around a tile boundary, the part limit, and a layer's pool past 2 GiB.
Every row against the oracle within the tests' bars (2e-2 / 2e-3; LSE 1e-3); three
launches in a row give the same bits (the arrival counters come back to zero, and the
merge sums in part order whichever part arrives last)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2607_00151_amd as sa
from workloads.configs import build

from harness import build_cache, compare, dev_u16, host_u16, layout_of

pytestmark = pytest.mark.gpu

CASES = {
    # name: Hq, Hkv, page, prefixes, segments
    "one_row": (1, 1, 16, [9000], [1]),
    "three_heads": (3, 1, 32, [5000, 100], [1, 1]),
    "five_heads": (10, 2, 16, [3000], [1]),
    "twelve_heads": (12, 1, 16, [2500], [1]),
    "part_limit": (8, 1, 32, [40000], [1]),
    "seventeen_rows": (17, 1, 16, [2000], [1]),
    "twenty_rows": (4, 1, 16, [7000, 63], [5, 5]),
    "thirty_two_rows": (1, 1, 16, [3000], [32]),
    "thirty_three_rows": (1, 1, 16, [3000], [33]),
    "tile_edges": (8, 2, 16, [255, 256, 257, 511, 64], [1, 1, 1, 65, 64]),
    "no_prefix": (8, 2, 32, [0, 0], [700, 1]),
    "unseen_parts": (8, 2, 16, [700, 10], [100, 300]),
    "ragged_decode": (8, 1, 16, [100, 20000, 3000, 0, 64], [1, 1, 1, 1, 1]),
    "mixed": (8, 1, 16, [4000, 4000, 900], [1, 200, 1]),
    "part_limit_8_rows": (8, 1, 32, [190000], [1]),
    "part_limit_32_rows": (32, 1, 32, [720000], [1]),
    # 320 and 448 items, one long context among short ones: more than CUs, not two per CU
    "long_among_short": (64, 64, 16, [6000, 300, 300, 300, 300], [1, 1, 1, 1, 1]),
    "long_among_short_mixed": (128, 64, 16, [6000, 300, 300, 300, 300], [40, 100, 70, 1, 1]),
}


def launches(ctx, w, fn, n=3):
    L = layout_of(w)
    kp, vp, ip, ix = build_cache(w)
    q, T = dev_u16(w.q), int(w.qlen.sum())
    out = []
    for _ in range(n):
        o = torch.full((T, w.num_q_heads, 128), -1, dtype=torch.int16, device="cuda")
        lse = torch.full((T, w.num_q_heads), float("nan"), dtype=torch.float32, device="cuda")
        fn(ctx, L, 0, q, kp, vp, w.qlen, w.kv, ip, ix, w.scale, o, lse)
        out.append((o, lse))
    sa.sa_sync_check(ctx)
    return out


def check(w, out):
    for o, lse in out[1:]:
        assert torch.equal(o, out[0][0]) and torch.equal(lse, out[0][1])
    ref, ref_lse, _ = oracle.attention_all(w.q, w.k, w.v, w.q_indptr, w.kv_indptr, w.num_q_heads, w.num_kv_heads,
                                           w.scale)
    compare(host_u16(out[0][0]), ref, 2e-2, 2e-3)
    assert np.abs(out[0][1].cpu().numpy() - ref_lse).max() <= 1e-3


@pytest.mark.parametrize("entry", ["sa_segment_prefill_attn", "sa_segment_prefill_attn_noalloc"])
@pytest.mark.parametrize("name", list(CASES))
def test_split_items(name, entry):
    Hq, Hkv, P, pre, q = CASES[name]
    w = build(name, 400 + list(CASES).index(name), Hq, Hkv, 128, P, pre, q)
    st = sa.sa_attn_plan_stats(layout_of(w), w.qlen, w.kv)
    print(f"{name} {entry}: {st}", flush=True)
    assert st["parts"] > 0 and st["items"] < 2 ** 14
    if name.startswith("part_limit_"):         # as many as the merge has LDS for
        assert st["parts"] == 128
    with sa.Context(0) as ctx:
        check(w, launches(ctx, w, getattr(sa, entry)))


def test_folded_scale_split_decode():
    Hq, Hkv, P, pre, q = CASES["twenty_rows"]
    w = build("folded_split", 431, Hq, Hkv, 128, P, pre, q)
    with sa.Context(0) as ctx:
        sa.sa_set_exact_scale(ctx, False)
        out = launches(ctx, w, sa.sa_segment_prefill_attn)
    ref, _, _ = oracle.attention_all(w.q, w.k, w.v, w.q_indptr, w.kv_indptr, Hq, Hkv, w.scale)
    compare(host_u16(out[0][0]), ref, 2e-2, 2e-3)
    assert torch.equal(out[0][0], out[2][0])


@pytest.mark.parametrize("q", [[1, 1, 1], [1, 40, 9]])
def test_pool_past_two_gib(q):
    """Slots beyond the reach of one 32-bit buffer resource, decode and prefill items."""
    slots = (1 << 31) // (2 * 32 * 128 * 2) + 4096           # Hkv 2, page 32: 16 KiB a slot
    w = build("big_pool", 432, 8, 2, 128, 32, [3000, 50, 700], q, num_slots=slots)
    assert (w.pages.astype(np.int64) * 2 * 32 * 128 * 2 >= 1 << 31).any()
    with sa.Context(0) as ctx:
        check(w, launches(ctx, w, sa.sa_segment_prefill_attn))


def test_missing_pages_of_a_split_decode_item_are_reported():
    """A slot outside the pool in one part: reported, the rest of the launch whole, the next launch clean."""
    w = build("bad_page", 433, 8, 1, 128, 16, [6000, 900], [1, 1])
    L = layout_of(w)
    kp, vp, ip, ix = build_cache(w)
    q = dev_u16(w.q)
    with sa.Context(0) as ctx:
        o = torch.zeros((2, 8, 128), dtype=torch.int16, device="cuda")
        bad = ix.clone()
        bad[200] = L.num_slots
        sa.sa_segment_prefill_attn(ctx, L, 0, q, kp, vp, w.qlen, w.kv, ip, bad, w.scale, o)
        with pytest.raises(sa.SaError) as e:
            sa.sa_sync_check(ctx)
        assert e.value.name == "SA_ERR_RANGE"
        ref, _, _ = oracle.attention_all(w.q, w.k, w.v, w.q_indptr, w.kv_indptr, 8, 1, w.scale)
        compare(host_u16(o)[1:], ref[1:], 2e-2, 2e-3)
        sa.sa_segment_prefill_attn(ctx, L, 0, q, kp, vp, w.qlen, w.kv, ip, ix, w.scale, o)
        sa.sa_sync_check(ctx)
        compare(host_u16(o), ref, 2e-2, 2e-3)


def test_split_buffer_grows_by_doubling():
    """A context whose part counts creep up call by call (16, 24, ... 256 parts of 66 KB) allocates for
    them at 16, 24, 40, 72 and 136 parts, not at each of the 31."""
    L = sa.Layout(num_q_heads=8, num_kv_heads=8, head_dim=128, page_size=32, num_layers=1, num_slots=256)
    pools = [torch.zeros((256, 8, 32, 128), dtype=torch.int16, device="cuda") for _ in range(2)]
    q = torch.zeros((1, 8, 128), dtype=torch.int16, device="cuda")
    o = torch.zeros_like(q)
    ip = torch.tensor([0, 256], dtype=torch.int32, device="cuda")
    ix = torch.arange(256, dtype=torch.int32, device="cuda")
    parts, free = [], []
    with sa.Context(0) as ctx:
        for k in range(2, 33):
            kv = [256 * k]
            parts.append(sa.sa_attn_plan_stats(L, [1], kv)["parts"])
            sa.sa_segment_prefill_attn(ctx, L, 0, q, pools[0], pools[1], [1], kv, ip, ix, 0.088, o)
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info(0)[0])
        sa.sa_sync_check(ctx)
    assert parts == [8 * k for k in range(2, 33)]
    assert sum(a != b for a, b in zip(free, free[1:])) <= 6
