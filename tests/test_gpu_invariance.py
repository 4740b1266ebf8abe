"""GPU bitwise invariance: the output of a logical (prompt, position, head)
row is bit-identical across batch composition and order, chunking, query
length (decode vs verify vs prefill), page placement and sharing, and
metadata that must not matter (hints, table stride, pool size, workspace
contents, stream, repetition) -- the causal contract of the paper's
Section 5.3 / Appendix A.1."""
from __future__ import annotations

import json
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2609_38981_amd import staging as S
from paper_2609_38981_amd import vdattn as V
from paper_2609_38981_amd import workloads as W
from tests import gpu_util as U

pytestmark = pytest.mark.gpu
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    U.require_gpu()


def outs(call, **kw):
    return U.by_position(call, U.gpu_run(call, **kw))


# -- tiny workload (config 1) ---------------------------------------------------
def test_tiny_variants():
    base = outs(W.config1(variant="both"))
    n = 0
    for v in ["BA", "A", "B", "B44a", "B44b"]:
        n += U.assert_same_bits(base, outs(W.config1(variant=v)))
    n += U.assert_same_bits(base, outs(W.config1(perm_stream=5)), min_common=9)
    U.say("tiny variants: %d rows bit-identical" % n)


def test_fig4_example_on_gpu():
    """Paper Fig. 4: prefill row 3 of q_len = k_len = 6 equals the decode row
    of q_len 1, k_len 4, on different physical pages (page size 16 here)."""
    ex = json.load(open(os.path.join(GOLDEN, "fig4_position_example.json")))
    pre, dec = ex["prefill"], ex["decode"]
    for sh in (W.TINY, W.LLAMA8B):
        pr = W.make_prompt(sh, pre["k_len"], 11, 0)
        a = W.place(sh, [pr], [W.Req(0, pre["k_len"], pre["q_len"])], W.rng_for(11, 4), min_pages=12)
        b = W.place(sh, [pr], [W.Req(0, dec["k_len"], dec["q_len"])], W.rng_for(11, 5), min_pages=12)
        assert a.page_table[0, 0] != b.page_table[0, 0]
        oa, ob = U.gpu_run(a), U.gpu_run(b)
        assert np.array_equal(oa[pre["row"]], ob[dec["row"]])


# -- query length: whole prefill vs chunks vs verify vs decode stepping --------
@pytest.mark.parametrize("shape", [W.LLAMA8B, W.TINY], ids=["8b", "tiny"])
def test_chunking_and_query_length(shape):
    """One prompt of 1100 tokens: whole (s = n), chunks of 512 and 128, 4-token
    verify steps and 1-token decode steps give the same bits per position."""
    n_total = 1100
    pr = W.make_prompt(shape, n_total, 12, 0)
    rng = W.rng_for(12, 4)

    def run(pieces):
        # pieces: list of (n, s) calls, each a separate invocation
        res = {}
        for n, s in pieces:
            call = W.place(shape, [pr], [W.Req(0, n, s)], rng)
            res.update(outs(call))
        return res

    whole = run([(n_total, n_total)])
    assert len(whole) == n_total
    c512 = run([(min(n_total, e + 512), min(512, n_total - e)) for e in range(0, n_total, 512)])
    c128 = run([(min(n_total, e + 128), min(128, n_total - e)) for e in range(0, n_total, 128)])
    U.assert_same_bits(whole, c512, min_common=n_total)
    U.assert_same_bits(whole, c128, min_common=n_total)
    # verify (s = 4) and decode (s = 1) steps around split and tile edges
    spots = [1, 2, 63, 64, 65, 511, 512, 513, 1023, 1024, 1025, 1099]
    steps = [(p + 1, 1) for p in spots] + [(p + 1, 4) for p in spots if p >= 3]
    U.assert_same_bits(whole, run(steps), min_common=len(spots))
    # a batch that mixes all of them in one call
    reqs = [W.Req(0, n, s) for n, s in [(1100, 600), (513, 1), (700, 4), (65, 65), (1025, 8)]]
    call = W.place(shape, [pr], reqs, rng)
    U.assert_same_bits(whole, outs(call), min_common=600)


# -- batch composition and order (config 2 family) -----------------------------
def test_probe_request_batch_invariance():
    """A fixed probe request alone, and at random slots in batches of 17 and
    64, gives the same bits; page placement and order do not matter."""
    kw = dict(lo=200, hi=2600)
    solo = outs(W.config2(batch=1, probe_slot=0, **kw))
    n = 0
    for batch, slot, perm in [(17, 5, 4), (64, 41, 4), (64, 0, 5), (17, 16, 5)]:
        n += U.assert_same_bits(solo, outs(W.config2(batch=batch, probe_slot=slot,
                                                     perm_stream=perm, **kw)))
    U.say("probe invariance: %d comparisons" % n)


def test_metadata_does_not_matter():
    """Oversized hints, a wider page-table stride, a bigger pool, a NaN-filled
    workspace, another stream, a repeat run and a prepared call (whole or
    phase by phase) give the same bits."""
    mk = lambda **kw: W.config2(batch=9, lo=300, hi=1800, **kw)
    base = outs(mk())
    call = mk()
    variants = {
        "hints": dict(hint_extra_q=7, hint_extra_ctx=3000),
        "hints_long": dict(hint_extra_ctx=20000),
        "ws_nan": dict(workspace_fill=-1),
        "stream": dict(stream=torch.cuda.Stream()),
        "repeat": {},
        "prepared_forward": dict(prepared="forward"),
        "prepared_phases": dict(prepared="phases"),
        "prepared_timed": dict(prepared="timed"),
        # ordinary (cached) K/V loads instead of non-temporal ones
        "shared_pages_hint": dict(shared_pages=True),
    }
    for name, kw in variants.items():
        U.assert_same_bits(base, U.by_position(call, U.gpu_run(call, **kw)), min_common=9)
    wide = W.place(call.shape, call.prompts, call.reqs, W.rng_for(2, 4), stride_extra=37,
                   pool_factor=3.0)
    U.assert_same_bits(base, outs(wide), min_common=9)


def test_mixed_batch_orders():
    """Config 3 family: prefill chunks and decodes in one call, rows ordered
    prefill-first or shuffled, and the timed phase launches, give the same
    bits."""
    kw = dict(num_prefill=3, chunk=96, max_off=900, num_decode=10, dec_lo=60, dec_hi=1500)
    a = outs(W.config3(**kw))
    b = outs(W.config3(shuffle=True, perm_stream=5, **kw))
    U.assert_same_bits(a, b, min_common=3 * 96 + 10)
    # the timed split and chunk launches compute the same bits
    c = outs(W.config3(**kw), prepared="timed")
    U.assert_same_bits(a, c, min_common=3 * 96 + 10)


def test_prefix_sharing_and_verify_steps():
    """Config 5 family: shared vs copied prefix pages, and 4-token verify vs
    single-token steps at each of the 4 positions."""
    kw = dict(num_req=8, prefix=512, suf_lo=30, suf_hi=200)
    shared = outs(W.config5(shared=True, **kw))
    copied = outs(W.config5(shared=False, perm_stream=5, **kw))
    U.assert_same_bits(shared, copied, min_common=4 * 4 + 4)
    for step in range(4):
        U.assert_same_bits(shared, outs(W.config5(step=step, **kw)), min_common=8)
    # non-temporal K/V loads although pages are shared
    U.assert_same_bits(shared, outs(W.config5(shared=True, **kw), shared_pages=False),
                       min_common=4 * 4 + 4)


def test_large_batch_plan_launch():
    """More than 256 requests: the plan launch lists the split items and, with
    the query rows' K/V handed over, writes them.  A probe request gives the
    same bits there as alone or among 17 requests, where the split workgroups
    find their items and write the new tokens themselves."""
    kw = dict(lo=20, hi=600)
    solo = outs(W.config2(batch=1, probe_slot=0, **kw))
    big = W.config2(batch=300, probe_slot=211, perm_stream=5, **kw)
    U.assert_same_bits(solo, outs(big))
    out_append = U.gpu_run(big, append=True)
    U.assert_same_bits(solo, U.by_position(big, out_append))
    U.assert_same_bits(outs(big), U.by_position(big, out_append), min_common=300)
    U.assert_same_bits(solo, outs(W.config2(batch=17, probe_slot=3, **kw), append=True))
    U.say("  300 requests, appended: %s" % U.parity(big, out_append, rows=[0, 150, 211, 299]))
    # prefill rows too: the plan launch's chunk list (263 requests) against the
    # chunk workgroups' own planning (13 requests)
    kw3 = dict(num_prefill=3, chunk=96, max_off=900, dec_lo=20, dec_hi=400)
    small = outs(W.config3(num_decode=10, **kw3))
    large = W.config3(num_decode=260, **kw3)
    U.assert_same_bits(small, outs(large), min_common=3 * 96 + 10)
    U.assert_same_bits(small, outs(large, append=True), min_common=3 * 96 + 10)
    U.assert_same_bits(small, outs(W.config3(num_decode=10, **kw3), append=True),
                       min_common=3 * 96 + 10)


def test_large_batch_column_halves():
    """More than 256 requests with 32 query-head rows per KV head (70B verify,
    s = 4): the plan launch lists one wide item per split (both 16-row
    blocks).  Rows equal those of a few of the requests run alone (the split
    workgroups' own planning), and those without the shared-prefix pass."""
    big = W.config5(num_req=300, prefix=V.SPLIT_KEYS, suf_lo=20, suf_hi=300)
    a = outs(big)
    U.assert_same_bits(a, outs(big.subcall([0, 1, 150, 298, 299])), min_common=4 * 3 + 2)
    U.assert_same_bits(a, outs(big, shared_pages=False), min_common=big.total_q_tokens)
    U.say("  300 verify requests: %s" % U.parity(big, U.gpu_run(big), rows=[0, 3, 601, 749]))


def test_wide_items_vs_column_halves():
    """70B verify (s = 4: 32 query-head rows per KV head) runs as wide split
    items, one per split over both 16-row blocks, when every request is on
    the split path, and as two column-half items per split when the call also
    carries a prefill chunk (40 G rows: the chunk path).  The verify rows are
    the same bits either way, below and above 256 requests (in-wave planning
    and the plan launch), with and without the shared-prefix pass; suffixes
    up to 1500 keys give rows of up to three splits."""
    for num_req in (12, 300):
        base = W.config5(num_req=num_req, prefix=V.SPLIT_KEYS + 304, suf_lo=20, suf_hi=1500)
        sh = base.shape
        wide = outs(base)
        extra = W.make_prompt(sh, 700, 16, 0, q_window=40)
        mixed = W.place(sh, base.prompts + [extra], base.reqs + [W.Req(len(base.prompts), 700, 40)],
                        W.rng_for(16, 4), shared_prefix_pages=(V.SPLIT_KEYS + 304) // sh.page_size)
        assert mixed.max_q_len * sh.group > 32 and base.max_q_len * sh.group == 32
        n = U.assert_same_bits(wide, outs(mixed), min_common=base.total_q_tokens)
        n += U.assert_same_bits(wide, outs(mixed, shared_pages=False), min_common=base.total_q_tokens)
        n += U.assert_same_bits(wide, outs(base, shared_pages=False), min_common=base.total_q_tokens)
        U.say("  %d verify requests, wide vs column halves: %d rows bit-identical" % (num_req, n))


def test_wide_items_head_dim_64():
    """Head dim 64, 2 query heads per KV head: 12-token verify rows (24
    query-head rows per KV head, wide split items) against the same rows in a
    call that also prefills a 40-token chunk (16-row column halves), and
    against single-token steps at each position."""
    sh = W.TINY
    prompts = [W.make_prompt(sh, n, 17, i, q_window=12) for i, n in enumerate((700, 1500, 2100, 90))]
    reqs = [W.Req(i, pr.length, 12) for i, pr in enumerate(prompts)]
    wide = outs(W.place(sh, prompts, reqs, W.rng_for(17, 4)))
    extra = W.make_prompt(sh, 300, 17, 9, q_window=40)
    mixed = W.place(sh, prompts + [extra], reqs + [W.Req(len(prompts), 300, 40)], W.rng_for(17, 5))
    n = U.assert_same_bits(wide, outs(mixed), min_common=48)
    steps = [W.Req(i, pr.length - j, 1) for i, pr in enumerate(prompts) for j in range(12)]
    n += U.assert_same_bits(wide, outs(W.place(sh, prompts, steps, W.rng_for(17, 6))), min_common=48)
    U.say("  head dim 64, wide vs column halves vs steps: %d rows bit-identical" % n)


def test_chunk_order_above_64_requests():
    """70 prefill chunks (more than 64 on the chunk path: the in-wave planner
    keeps request order) against 9 of them alone (listed longest first), and
    in reverse order."""
    kw = dict(chunk=96, max_off=1500, num_decode=3, dec_lo=20, dec_hi=400)
    big = W.config3(num_prefill=70, **kw)
    a = outs(big)
    sub = [0, 1, 5, 17, 33, 40, 64, 69, 71]
    n = U.assert_same_bits(a, outs(big.subcall(sub)), min_common=8 * 96 + 1)
    rev = W.place(big.shape, big.prompts, big.reqs[::-1], W.rng_for(3, 9))
    n += U.assert_same_bits(a, outs(rev), min_common=big.total_q_tokens)
    U.say("  70 chunk-path requests vs 9 alone and reversed: %d rows bit-identical" % n)


def test_long_context_batch_and_placement():
    """Config 4 family (scaled down): batch 1 vs batch 4, two placements."""
    kw = dict(lo=6000, hi=12000)
    b4 = outs(W.config4(batch=4, **kw))
    for i in range(4):
        U.assert_same_bits(b4, outs(W.config4(batch=4, only=i, perm_stream=5, **kw)))


def test_full_size_long_decode_batch_one_vs_eight():
    """Long-context decode at full size: requests alone (another placement)
    and in the batch of 8 give the same bits."""
    b8 = outs(W.config4())
    for i in (2, 6):
        U.assert_same_bits(b8, outs(W.config4(only=i, perm_stream=5)))


def test_full_size_decode_probe_batch_1_17_64():
    """Llama-3-8B decode at full size: the probe request alone, in 17 and in
    64 requests (contexts 512..4096)."""
    solo = outs(W.config2(batch=1, probe_slot=0))
    for batch, slot in [(17, 9), (64, 33)]:
        U.assert_same_bits(solo, outs(W.config2(batch=batch, probe_slot=slot, perm_stream=5)))


PAIR_SHAPES = [W.LLAMA8B, W.Shape(14, 2, 64), W.Shape(32, 8, 128, window=1500)]


@pytest.mark.parametrize("shape", PAIR_SHAPES, ids=["d128-g4", "d64-g7", "d128-window"])
@pytest.mark.parametrize("n,s", [
    (1025, 33),    # a second split of one key
    (2048, 65),    # two whole splits
    (2049, 128),   # a third of one key, alone in its round
    (3100, 17),    # rows in one split, an odd count of splits
    (4097, 90),    # rows on both sides of a split edge
    (5000, 257),
])
def test_paired_chunks_equal_chunks(shape, n, s):
    """A prefill chunk alone (few items: the paired chunk kernel, where its
    context is longer than a split) equals, bit for bit and in its log-sum-exp,
    the same chunk in a call with enough other rows for the chunk kernel; and
    sampled rows match the oracle."""
    p = W.make_prompt(shape, n, 71, n, q_window=s)
    other = W.make_prompt(shape, 1200 * 32 // shape.num_q_heads, 71, 1)
    rng = W.rng_for(71, 4)
    alone = W.place(shape, [p], [W.Req(0, n, s)], rng)
    both = W.place(shape, [other, p], [W.Req(0, other.length, other.length), W.Req(1, n, s)], rng)
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def items(call):  # an upper bound, 64 query-head rows each
        rows = call.total_q_tokens * shape.group + 63 * call.num_seqs
        return shape.num_kv_heads * (rows // 64)

    assert items(alone) <= cus < items(both)
    a, la = U.gpu_run(alone, with_lse=True)
    b, lb = U.gpu_run(both, with_lse=True)
    assert np.array_equal(a, b[other.length:]) and np.array_equal(la, lb[other.length:])
    U.assert_written(U.by_position(alone, a))
    U.parity(alone, a, rows=[0, s // 2, s - 1])


@pytest.mark.parametrize("shape", PAIR_SHAPES, ids=["d128-g4", "d64-g7", "d128-window"])
@pytest.mark.parametrize("pages", [
    [106],                      # one page of a tile in split 1
    [128, 129, 130, 131, 190],  # a whole tile, split 2's first, and another page of it
    [193],                      # the last, ragged tile (split 3)
    [10, 106, 150, 193],        # both splits of each round
], ids=["split1", "split2", "last", "all"])
def test_chunks_read_invalid_pages_as_zeros(shape, pages):
    """A prefill chunk whose table holds page ids outside the pool, in one split
    of a round of the paired chunk kernel or in both, within a tile, over a whole
    tile and in the last one: alone (paired) and beside enough other rows (the
    chunk kernel) the same bits and log-sum-exp, and the oracle's values with
    zeros in those pages."""
    n, s = 3100, 257
    p = W.make_prompt(shape, n, 77, n, q_window=s)
    other = W.make_prompt(shape, 1200 * 32 // shape.num_q_heads, 77, 1)
    alone = W.place(shape, [p], [W.Req(0, n, s)], W.rng_for(77, 4))
    both = W.place(shape, [other, p], [W.Req(0, other.length, other.length), W.Req(1, n, s)],
                   W.rng_for(77, 5))
    attn = U.handle(shape)
    got = []
    for call in (alone, both):
        b = S.to_device(attn, call, lse=True).batch
        for i, pg in enumerate(pages):
            b.page_table[-1, pg] = [-1, call.num_pages, -7, 2**31 - 1][i % 4]
        out = S.bits_of(attn.forward(b))
        got.append((out[-s:], b.lse.cpu().numpy()[-s:]))
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    kp, vp = (x.copy() for x in alone.std_pool())
    for x in (kp, vp):
        x[alone.page_table[0, pages]] = 0
    rows = [0, s // 2, s - 1]
    ref = oracle.paged_attention(alone.q_bits(), alone.cu_q_lens, alone.context_lens, alone.page_table,
                                 kp, vp, num_q_heads=shape.num_q_heads,
                                 num_kv_heads=shape.num_kv_heads, head_dim=shape.head_dim,
                                 page_size=shape.page_size, window=shape.window, rows=rows)[rows]
    val = W.bf16_to_f32(got[0][0][rows]).astype(np.float64)
    assert np.isfinite(val).all()
    bound = np.minimum(U.TOL, U.REL_TOL * np.abs(ref).max(axis=-1, keepdims=True) + 1e-7)
    assert (np.abs(val - ref) <= bound).all()


@pytest.mark.parametrize("shape", [W.LLAMA8B, W.TINY], ids=["d128", "d64"])
@pytest.mark.parametrize("append", [False, True], ids=["written", "append"])
def test_calls_of_prefill_rows_only(shape, append):
    """Calls whose sizes leave every request chunk-path rows (one chunk; chunks
    of one length): the same bits as beside a decode row, new tokens written or
    handed over; and a request with fewer rows than total_q_tokens and max_q_len
    promise still gets its output."""
    rng = W.rng_for(72, 4)
    ps = [W.make_prompt(shape, n, 72, i, q_window=60) for i, n in enumerate([1100, 700, 60, 300])]
    decode = [W.Req(3, 300, 1)]
    for reqs in ([W.Req(0, 1100, 60)], [W.Req(i, ps[i].length, 40) for i in range(3)]):
        alone, mixed = W.place(shape, ps, reqs, rng), W.place(shape, ps, reqs + decode, rng)
        a, la = U.gpu_run(alone, append=append, with_lse=True)
        b, lb = U.gpu_run(mixed, append=append, with_lse=True)
        assert np.array_equal(a, b[:-1]) and np.array_equal(la, lb[:-1])
        U.assert_written(U.by_position(alone, a))
    one = W.place(shape, ps, decode, rng)
    want = U.gpu_run(one)
    attn = U.handle(shape)
    b = S.to_device(attn, one).batch
    b.q = torch.cat([b.q] * 40)
    b.max_q_len = 40
    got = S.bits_of(attn.forward(b))
    assert np.array_equal(got[:1], want)


CAPACITY_SHAPES = [W.LLAMA8B, W.Shape(14, 2, 64), W.Shape(8, 8, 64), W.Shape(32, 8, 128, window=1500)]


@pytest.mark.parametrize("shape", CAPACITY_SHAPES, ids=["d128-g4", "d64-g7", "d64-g1", "d128-window"])
@pytest.mark.parametrize("append", [False, True], ids=["written", "append"])
@pytest.mark.parametrize("shared", [False, True], ids=["own", "shared"])
def test_short_requests_in_a_call_sized_for_chunks(shape, append, shared):
    """Decode and verify rows, alone and beside a chunk, in a call whose
    total_q_tokens and max_q_len leave room for chunks (a captured call's): they
    run in the split launch like in a call of their own size (the splits phase
    alone writes the rows of one split), and output and log-sum-exp are the
    same, folded by the paired chunk kernel's launch and, beside the chunk kernel
    (more room) or with more splits than that folds, by the merge."""
    ns = [1, 60, 1024, 1025, 2500, 5000, 3000]
    attn = U.handle(shape)
    for last, room in ((40, 40), (40, 100), (34816, 40)):  # last request's keys: up to 34 splits
        ps = [W.make_prompt(shape, n, 76, n, q_window=40) for n in ns + [last]]
        if shared:  # the prompts of 2500 and 5000 keys begin with the same pages
            ps[5] = W.make_prompt(shape, ns[5], 76, 1, q_window=40, prefix=ps[4], prefix_len=2048)
        reqs = [W.Req(i, p.length, min(p.length, s)) for i, (p, s) in enumerate(
            zip(ps, [1, 4, 1, 2, 1, 3, 40, 4]))]
        call = W.place(shape, ps, reqs, W.rng_for(76, 4))
        want, lse = U.gpu_run(call, append=append, with_lse=True)
        b = S.to_device(attn, call, append=append, lse=True, shared_pages=shared).batch
        T, pad = call.total_q_tokens, room * len(reqs) - call.total_q_tokens

        def longer(x):
            return torch.cat([x, x[:1].expand(pad, *x.shape[1:])])

        b.q, b.lse, b.max_q_len = longer(b.q), longer(b.lse), room
        if append:
            b.k_new, b.v_new = longer(b.k_new), longer(b.v_new)
        ws = attn.new_workspace(len(reqs), room, b.max_context_len)
        out = torch.full_like(b.q, float("nan"))
        attn.forward_plan(b, ws)
        attn.forward_splits(b, out, ws)
        single = [r for r, q in enumerate(reqs) if q.n <= 1024 and q.s * shape.group <= 32]
        for r in single:
            row = call.row_of(r, reqs[r].n - reqs[r].s)
            got = S.bits_of(out)[row:row + reqs[r].s]
            assert np.array_equal(got, want[row:row + reqs[r].s]), reqs[r]
        assert len(single) >= 3
        attn.forward_chunks(b, out, ws)
        attn.forward_merge(b, out, ws)
        assert np.array_equal(S.bits_of(out)[:T], want)
        assert np.array_equal(b.lse[:T].cpu().numpy(), lse)


@pytest.mark.parametrize("append", [False, True], ids=["written", "append"])
def test_query_buffer_longer_than_its_rows(append):
    """Decode rows at the start of a longer query buffer (total_q_tokens past
    cu_q_lens[B], max_q_len 1), and beside a request with more rows than
    max_q_len (skipped): output, log-sum-exp and new tokens' slots as without
    the further rows."""
    shape = W.LLAMA8B
    ps = [W.make_prompt(shape, n, 75, n, q_window=40) for n in (300, 1100, 2500, 60)]
    attn = U.handle(shape)
    rng = W.rng_for(75, 4)
    cut = W.place(shape, ps, [W.Req(i, p.length, 1) for i, p in enumerate(ps)], rng)
    past = W.place(shape, ps, [W.Req(i, p.length, 40 if i == 3 else 1) for i, p in enumerate(ps)], rng)
    for call, rows, pad in ((cut, 4, 60), (past, 3, 0)):
        alone = call.subcall(range(rows))
        want = S.to_device(attn, alone, append=append, lse=True).batch
        wo = attn.forward(want)
        b = S.to_device(attn, call, append=append, lse=True).batch
        b.q = torch.cat([b.q, b.q[:1].expand(pad, -1, -1)])
        b.lse = torch.empty(b.q.shape[:2], dtype=torch.float32, device="cuda")
        if append:
            b.k_new = torch.cat([b.k_new, b.k_new[:1].expand(pad, -1, -1)])
            b.v_new = torch.cat([b.v_new, b.v_new[:1].expand(pad, -1, -1)])
        b.max_q_len = 1
        got = attn.forward(b)
        assert np.array_equal(S.bits_of(got)[:rows], S.bits_of(wo))
        assert torch.equal(b.lse[:rows], want.lse)
        for r in range(rows):  # the requests' pages, in the call's and in their own placement
            n = alone.reqs[r].n
            for pool in ("k_pool", "v_pool"):
                x = getattr(b, pool).view(torch.int16).view(b.num_pages, -1)
                y = getattr(want, pool).view(torch.int16).view(want.num_pages, -1)
                k = (n + 15) // 16
                assert torch.equal(x[b.page_table[r, :k].long()], y[want.page_table[r, :k].long()])


SHARE_SHAPES = [W.LLAMA8B, W.LLAMA70B, W.Shape(8, 8, 64), W.Shape(21, 3, 64, window=700),
                W.Shape(32, 8, 128, window=1100)]


@pytest.mark.parametrize("shape", SHARE_SHAPES, ids=["d128-g4", "d128-g8", "d64-g1", "d64-g7-window",
                                                     "d128-window"])
@pytest.mark.parametrize("append", [False, True], ids=["written", "append"])
@pytest.mark.parametrize("s", [1, 4])
def test_shared_out_splits_equal_splits(shape, append, s):
    """Decode and verify rows in calls of one request (few items: a workgroup per
    split) equal, bit for bit, in output, log-sum-exp and the new tokens' pool
    slots, the same rows in a call of 70 requests (a wavefront per split):
    contexts of 3 tiles, at split and tile edges, with new tokens on both sides of
    a tile or split edge; and match the oracle."""
    check_shared_out(shape, append, s)


@pytest.mark.parametrize("shape,s", [
    (W.Shape(8, 8, 64), 9), (W.Shape(8, 8, 64), 16), (W.Shape(16, 8, 128), 9), (W.Shape(16, 8, 128), 16),
    (W.Shape(8, 8, 128), 17), (W.Shape(6, 6, 64), 32),
], ids=["d64-g1-9", "d64-g1-16", "d128-g2-9", "d128-g2-16", "d128-g1-17", "d64-g1-32"])
@pytest.mark.parametrize("append", [False, True], ids=["written", "append"])
def test_shared_out_splits_of_many_rows(shape, append, s):
    """The same for 9 to 16 new rows, which the split launch writes, and 17 to
    32 rows of one query head per KV head, which the plan launch writes."""
    check_shared_out(shape, append, s)


def check_shared_out(shape, append, s):
    ns = [129, 577, 1024, 1025, 1026, 1100, 1984, 2050, 3071, 4096 + 64]
    ps = [W.make_prompt(shape, n, 73, n, q_window=s) for n in ns]
    ps += [W.make_prompt(shape, 100 + i, 73, i, q_window=1) for i in range(60)]
    rng = W.rng_for(73, 4)
    reqs = [W.Req(i, p.length, s if i < len(ns) else 1) for i, p in enumerate(ps)]
    big = W.place(shape, ps, reqs, rng)
    want, lse = U.gpu_run(big, append=append, with_lse=True)
    U.assert_written(U.by_position(big, want))
    for i, n in enumerate(ns):
        one = big.subcall([i])
        got, l1 = U.gpu_run(one, append=append, with_lse=True)
        row = big.row_of(i, n - s)
        assert np.array_equal(got, want[row:row + s]), n
        assert np.array_equal(l1, lse[row:row + s]), n
        if append:
            attn = U.handle(shape)
            a = S.to_device(attn, one, append=True).batch
            b = S.to_device(attn, one, append=False).batch
            attn.forward(a)
            assert torch.equal(a.k_pool.view(torch.int16), b.k_pool.view(torch.int16)), n
            assert torch.equal(a.v_pool.view(torch.int16), b.v_pool.view(torch.int16)), n
    U.parity(big, want, rows=[big.row_of(i, n - 1) for i, n in enumerate(ns)])


def test_shared_out_splits_read_invalid_pages_as_zeros():
    """A page id outside the pool, in the first tiles, the last ones and the
    tile of the new token, reads as zeros in the shared-out kernel as in the
    split kernel."""
    shape = W.LLAMA8B
    ps = [W.make_prompt(shape, 1800, 74, i, q_window=1) for i in range(40)]
    call = W.place(shape, ps, [W.Req(i, 1800, 1) for i in range(40)], W.rng_for(74, 4))
    attn = U.handle(shape)
    b = S.to_device(attn, call, append=True, poison=False).batch
    for page, bad in ((3, -1), (40, call.num_pages), (75, -7), (112, 2**31 - 1)):
        b.page_table[:, page] = bad
    want = attn.forward(b)
    one = S.to_device(attn, call, append=True, poison=False).batch
    one = S.Batch(q=b.q[:1].contiguous(), cu_q_lens=b.cu_q_lens[:2].contiguous(),
                  context_lens=b.context_lens[:1].contiguous(),
                  page_table=b.page_table[:1].contiguous(), k_pool=one.k_pool, v_pool=one.v_pool,
                  num_pages=call.num_pages, max_q_len=1, max_context_len=1800,
                  k_new=b.k_new[:1].contiguous(), v_new=b.v_new[:1].contiguous())
    got = attn.forward(one)
    assert np.array_equal(S.bits_of(got), S.bits_of(want)[:1])
    assert np.isfinite(W.bf16_to_f32(S.bits_of(got))).all()
