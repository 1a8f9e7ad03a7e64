"""How the attention kernels place tiles on workgroups: head counts, block counts and block sizes at
the edges of the dispatch, against the float64 oracle.

The list walk (one workgroup per tile, and the persistent grid on a work queue), the masked walk and
the dense walk run on the same small problems. Skip decisions and computed counts must equal the
oracle's except within 1e-4 of the threshold, outputs lie within the path's bound (tests/parity.py),
and the two launches of the list walk agree bit for bit.
"""
import math
import sys

import numpy as np
import pytest

from oracle import cosa_oracle as O
from paper_2607_25291_amd import binding as B
from paper_2607_25291_amd.inputs import random_inputs
from tests import parity as PR
from tests.gpu_util import (Run, bf16_to_f64, dev, host_bits, queue_counters, queue_left, tau_of,
                            torch)
from tests.test_gpu_paged import make_paged

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# batch, query heads, KV heads, block, blocks
CASES = [
    # an odd group size: one head per workgroup, one page buffer (both block sizes, one block up)
    (1, 1, 1, 128, 1), (1, 3, 1, 128, 2), (2, 3, 3, 128, 5), (1, 5, 1, 64, 3), (1, 7, 1, 64, 9),
    # even groups of 64-token blocks: single heads in the list walk, head pairs in the others
    (1, 2, 1, 64, 1), (2, 8, 2, 64, 7),
    # groups of eight heads with a remainder, and heads that do not divide the XCDs
    (1, 9, 9, 64, 6), (3, 6, 3, 128, 4), (1, 17, 17, 128, 3),
    # the last block count at which even groups run as single heads (384 pairs), and the next one
    (1, 64, 8, 128, 12), (1, 64, 8, 128, 13),
]


def random_lists(rng, Bt, H, nb):
    """A random subset of the candidates of every row in random order, the block itself among them."""
    order = np.full((Bt, H, nb, nb), -1, np.int32)
    count = np.zeros((Bt, H, nb), np.int32)
    for n, g, i in np.ndindex(Bt, H, nb):
        k = int(rng.integers(1, i + 2))
        pick = np.concatenate([[i], rng.permutation(i)[:k - 1]]).astype(np.int32)
        order[n, g, i, :k] = rng.permutation(pick)
        count[n, g, i] = k
    return order, count


@pytest.mark.parametrize("case", CASES, ids=lambda c: "b%d_q%d_kv%d_blk%d_nb%d" % c)
def test_walks_match_oracle(case):
    Bt, Hq, Hkv, block, nb = case
    say(f"[tiles] B={Bt} Hq={Hq} Hkv={Hkv} block={block} nb={nb}")
    L = nb * block
    q, k, v = random_inputs(Bt, Hq, Hkv, L, 128, seed=nb, scale=1.5)
    p = B.Problem(Bt, Hq, Hkv, L, 128, block, block // 8)
    run = Run.upload(p, q, k, v)
    order, count = random_lists(np.random.default_rng(Hq * 100 + nb), Bt, Hkv, nb)
    delta = L * math.exp(-1.0)
    ref = O.osk_attention(q, k, v, order, count, block=block, skip_mode=O.SKIP_ROWMAX, delta=delta)
    do, dc = dev(order), dev(count)
    sk = B.skip(B.SKIP_ROWMAX, delta)
    o, vis, _, nco = run.osk(do, dc, sk)
    vis = vis.cpu().numpy()
    for n, h, i in np.ndindex(Bt, Hq, nb):
        PR.check_visits(vis[n, h, i], ref["visit"][n, h, i], ref["margin"][n, h, i],
                        tau_of(delta, L), int(count[n, h * Hkv // Hq, i]))
    PR.check_output(bf16_to_f64(host_bits(o)), ref["o"])

    t = torch()
    queue = t.full((B.cosa_osk_attention_queue_bytes(),), 0xFF, dtype=t.uint8, device="cuda")
    oq, nq = t.full_like(o, 0x7BCD), t.full_like(nco, -1)
    B.cosa_osk_attention_queued(p, run.q, run.k, run.v, do, dc, sk, oq, queue, queue.numel(),
                                n_computed=nq)
    assert t.equal(o, oq) and t.equal(nco, nq)

    mask = np.zeros((Bt, Hkv, nb, nb), np.uint8)
    for n, g, i in np.ndindex(Bt, Hkv, nb):
        mask[n, g, i, order[n, g, i, :count[n, g, i]]] = 1
    ref_m = O.osk_attention(q, k, v, order, count, block=block, skip_mode=O.SKIP_NONE)["o"]
    om = t.full_like(o, 0x7BCD)
    B.cosa_masked_attention(p, run.q, run.k, run.v, dev(mask), om)
    PR.check_output(bf16_to_f64(host_bits(om)), ref_m)
    PR.check_output(bf16_to_f64(host_bits(run.dense())), O.dense_attention(q, k, v, block=block))


@pytest.mark.parametrize("lens", [(1,), (1, 1, 1), (5, 1, 5, 2, 3, 5), (2, 7, 4, 4, 1, 9, 6)],
                         ids=lambda x: "-".join(map(str, x)))
@pytest.mark.parametrize("heads,block", [((4, 2), 128), ((3, 3), 64), ((20, 10), 64)])
def test_packed_tiles(lens, heads, block):
    """Packed sequences, equal lengths and one-block ones among them: every block of every sequence
    is visited (dense equals a call per sequence, and a prefill that keeps every block equals dense
    attention)."""
    Hq, Hkv = heads
    say(f"[packed tiles] lens={lens} heads={heads} block={block}")
    nb = sum(lens)
    L = nb * block
    q, k, v = random_inputs(1, Hq, Hkv, L, 128, seed=nb, scale=1.5)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    p = B.Problem(1, Hq, Hkv, L, 128, block, block // 8)
    run = Run.upload(p, q, k, v)
    t = torch()
    o = t.full_like(run.q, 0x7BCD)
    B.cosa_dense_attention_varlen(p, B.varlen(cu), run.q, run.k, run.v, o)
    for first, n in zip(cu, lens):
        at = slice(first * block, (first + n) * block)
        one = Run(B.Problem(1, Hq, Hkv, n * block, 128, block, block // 8),
                  *(x[:, :, at].contiguous() for x in (run.q, run.k, run.v)))
        assert t.equal(o[:, :, at], one.dense())
    nbytes = B.cosa_prefill_workspace_bytes(p)
    ws = t.zeros(nbytes, dtype=t.uint8, device="cuda")
    op = t.full_like(run.q, 0x7BCD)
    B.cosa_prefill_varlen(p, B.varlen(cu), run.q, run.k, run.v, B.select(B.SELECT_ALL), None, ws,
                          nbytes, op)
    ref = O.dense_attention_varlen(q, k, v, cu, block=block)
    PR.check_output(bf16_to_f64(host_bits(op)), ref)


# heads per workgroup of a list walk from work queues (0: no queue), sampled keys staged first
@pytest.mark.parametrize("heads,block,nb,mode,lens,page,queued,staged", [
    # keys in place; the grid resident as a whole (no queue), then fed by queues
    ((2, 2), 128, 5, B.SELECT_FRACTION, None, 0, 0, False),
    ((32, 8), 128, 40, B.SELECT_FRACTION, None, 0, 2, False),
    ((16, 4), 64, 130, B.SELECT_TOP_P, None, 0, 2, True),
    ((8, 2), 64, 60, B.SELECT_ALL, (20, 1, 39), 0, 0, False),
    # the block counts on either side of the staging threshold (8 heads: 70 and 71), 64-token blocks
    ((16, 8), 64, 70, B.SELECT_FRACTION, None, 0, 2, False),
    ((16, 8), 64, 71, B.SELECT_FRACTION, None, 0, 2, True),
    ((24, 8), 64, 90, B.SELECT_FRACTION, (40, 50), 0, 1, False),
    # packed and staged: an odd number of blocks, pairs of query blocks across two sequences, key chunks
    # in front of a sequence; single heads, head pairs and pages
    ((24, 8), 64, 99, B.SELECT_FRACTION, (65, 31, 1, 2), 0, 1, True),
    ((16, 8), 64, 99, B.SELECT_FRACTION, (2, 63, 1, 33), 0, 2, True),
    ((16, 8), 64, 99, B.SELECT_FRACTION, (2, 63, 1, 33), 32, 2, True),
    ((8, 8), 128, 99, B.SELECT_TOP_P, (2, 63, 34), 128, 1, True),
    # packed and staged, 64 rows a query block
    ((16, 2), 64, 172, B.SELECT_FRACTION, (140, 2, 30), 0, 2, True),
    # packed and in place, from pages
    ((8, 8), 128, 75, B.SELECT_FRACTION, (3, 60, 12), 16, 1, False),
])
def test_prefill_equals_stages(heads, block, nb, mode, lens, page, queued, staged):
    """cosa_prefill on a workspace full of stale bytes (the work-queue counters among them), twice in
    a row, against its stages called one by one on contiguous keys and values. The work-queue counters
    and the space of the staged keys show which kernels ran."""
    Hq, Hkv = heads
    say(f"[prefill stages] heads={heads} block={block} nb={nb} mode={mode} lens={lens} page={page}")
    L = nb * block
    q, k, v = random_inputs(1, Hq, Hkv, L, 128, seed=nb, scale=1.5)
    p = B.Problem(1, Hq, Hkv, L, 128, block, block // 8)
    run = Run.upload(p, q, k, v)
    t = torch()
    sel = B.select(mode, 0.4)
    sk = B.skip(B.SKIP_ROWMAX, (min(lens) if lens else nb) * block * 0.5)
    order = t.zeros((1, Hkv, nb, nb), dtype=t.int32, device="cuda")
    count = t.zeros((1, Hkv, nb), dtype=t.int32, device="cuda")
    score = t.zeros((1, Hkv, nb, nb), dtype=t.float32, device="cuda")
    hrm = t.zeros((1, Hkv, nb, nb), dtype=t.uint8, device="cuda")
    o, o2 = t.zeros_like(run.q), t.zeros_like(run.q)
    nbytes = B.cosa_prefill_workspace_bytes(p)
    ws = t.full((nbytes,), 0xFF, dtype=t.uint8, device="cuda")
    if lens:
        vl = B.varlen(np.concatenate([[0], np.cumsum(lens)]).tolist())
        B.cosa_kap_score_varlen(p, vl, run.q, run.k, score, hrm)
        B.cosa_kap_select_ordered_varlen(p, vl, score, hrm, sel, order, count)
        B.cosa_osk_attention_varlen(p, vl, run.q, run.k, run.v, order, count, sk, o)
    else:
        B.cosa_kap_score(p, run.q, run.k, score, hrm)
        B.cosa_kap_select_ordered(p, score, hrm, sel, order, count)
        B.cosa_osk_attention(p, run.q, run.k, run.v, order, count, sk, o)
    own = t.ones((nb, nb), dtype=t.bool, device="cuda").tril()  # the entries that are scored
    if lens:
        seq = t.repeat_interleave(t.arange(len(lens)), t.tensor(lens)).cuda()
        own &= seq[:, None] == seq[None, :]
    if page:
        kc, vc, table, n_pages = make_paged(k, v, page, 3, nb)
        cache = [dev(x) for x in (kc, vc, table)]
        kv = B.paged_kv(*cache, page, n_pages)
    lay = B.cosa_prefill_workspace_layout(p)
    for rep in range(2):
        if lens and page:
            B.cosa_prefill_paged_varlen(p, vl, run.q, kv, sel, sk, ws, nbytes, o2)
        elif lens:
            B.cosa_prefill_varlen(p, vl, run.q, run.k, run.v, sel, sk, ws, nbytes, o2)
        else:
            B.cosa_prefill(p, run.q, run.k, run.v, sel, sk, ws, nbytes, o2)
        got = ws[lay.order:lay.order + 4 * order.numel()].view(t.int32).view(order.shape)
        assert t.equal(got, order), rep
        got = ws[lay.count:lay.count + 4 * count.numel()].view(t.int32).view(count.shape)
        assert t.equal(got, count), rep
        got = ws[lay.score:lay.score + 4 * score.numel()].view(t.float32).view(score.shape)
        assert t.equal(got[..., own], score[..., own]), rep
        got = ws[lay.hrm:lay.hrm + hrm.numel()].view(hrm.shape)
        assert t.equal(got[..., own], hrm[..., own]), rep
        assert t.equal(o, o2), rep
        o2.fill_(0x7BCD)
    queue = ws[lay.queue:lay.queue + B.cosa_osk_attention_queue_bytes()]
    assert queue_counters(queue) == [queue_left(p, queued) if queued else 0] * 8
    assert bool((ws[lay.keys:lay.queue] != 0xFF).any()) == staged


@pytest.mark.parametrize("heads,block,lens", [
    # as many sequences as a call takes; two lengths, so that pieces of the order are empty
    ((8, 4), 64, (3,) * 60 + (8,) * 8 + (3,) * 60),
    # single heads and head pairs, the longest sequences in front, beside and behind short ones
    ((3, 1), 128, (9,) * 20 + (31, 1, 2, 30) + (8,) * 20),
    ((8, 2), 128, (40, 1, 7) + (5,) * 30 + (3,) * 20),
])
def test_packs_in_front_and_tail(heads, block, lens):
    """Packs of which the longest sequences are walked one after the other and the rest together: dense
    attention and a prefill with its work queue equal a call per sequence, bit for bit."""
    Hq, Hkv = heads
    say(f"[pack order] heads={heads} block={block} sequences={len(lens)} blocks={sum(lens)}")
    t = torch()
    nb, spb = sum(lens), 8
    cus = t.cuda.get_device_properties(0).multi_processor_count
    # two tiles per resident workgroup are ranked together, at most two heads a tile
    assert nb * Hq > (1 if Hq % 2 else 2) * 2 * {64: 2, 128: 2 if Hq % 2 else 1}[block] * cus
    q, k, v = random_inputs(1, Hq, Hkv, nb * block, 128, seed=nb, scale=1.5)
    cu = np.concatenate([[0], np.cumsum(lens)]).tolist()
    p = B.Problem(1, Hq, Hkv, nb * block, 128, block, block // spb)
    run = Run.upload(p, q, k, v)
    sel, sk = B.select(B.SELECT_FRACTION, 0.6), B.skip(B.SKIP_ROWMAX, 0.4 * min(lens) * block)
    o, op = t.full_like(run.q, 0x7BCD), t.full_like(run.q, 0x7BCD)
    B.cosa_dense_attention_varlen(p, B.varlen(cu), run.q, run.k, run.v, o)
    nbytes = B.cosa_prefill_workspace_bytes(p)
    ws = t.zeros(nbytes, dtype=t.uint8, device="cuda")
    B.cosa_prefill_varlen(p, B.varlen(cu), run.q, run.k, run.v, sel, sk, ws, nbytes, op)
    lay = B.cosa_prefill_workspace_layout(p)
    assert queue_counters(ws[lay.queue:lay.queue + B.cosa_osk_attention_queue_bytes()])[0] > 0
    for first, n in zip(cu, lens):
        at = slice(first * block, (first + n) * block)
        one = Run(B.Problem(1, Hq, Hkv, n * block, 128, block, block // spb),
                  *(x[:, :, at].contiguous() for x in (run.q, run.k, run.v)))
        assert t.equal(o[:, :, at], one.dense()), first
        assert t.equal(op[:, :, at], one.prefill(sel, sk)[0]), first


@pytest.mark.parametrize("batch,heads,block,nb", [
    # one group of eight heads in front of the last one, and several; single heads and head pairs, a last
    # group of five
    (5, (8, 8), 128, 66), (3, (16, 8), 64, 140), (9, (8, 4), 128, 64), (2, (13, 13), 64, 300),
])
def test_head_groups(batch, heads, block, nb):
    """Batches whose (batch, KV head) pairs are walked in several groups: dense attention and a prefill
    with its work queue equal a call per batch entry, bit for bit."""
    Hq, Hkv = heads
    say(f"[head groups] batch={batch} heads={heads} block={block} nb={nb}")
    t = torch()
    L = nb * block
    per_cu = {(128, 2): 1, (128, 1): 2, (64, 2): 2, (64, 1): 4}[block, 1 if Hq == Hkv else 2]
    cus = t.cuda.get_device_properties(0).multi_processor_count
    tiles = nb * (1 if Hq == Hkv else Hq // Hkv // 2)
    assert batch * Hkv - 8 >= 2 * cus * per_cu / tiles  # list walks: what the last group holds
    q, k, v = random_inputs(1, Hq, Hkv, L, 128, seed=nb, scale=1.5)
    one = Run.upload(B.Problem(1, Hq, Hkv, L, 128, block, block // 4), q, k, v)
    # the entries of the batch: the heads' rows rotated by whole blocks
    turned = [[x.roll(n * 3 * block, 2) for x in (one.q, one.k, one.v)] for n in range(batch)]
    run = Run(B.Problem(batch, Hq, Hkv, L, 128, block, block // 4),
              *(t.cat(x).contiguous() for x in zip(*turned)))
    sel, sk = B.select(B.SELECT_FRACTION, 0.1), B.skip(B.SKIP_ROWMAX, 0.4 * L)
    o, op = run.dense(), run.prefill(sel, sk)[0]
    for n, x in enumerate(turned):
        alone = Run(one.problem, *(y.contiguous() for y in x))
        assert t.equal(o[n], alone.dense()[0]), n
        assert t.equal(op[n], alone.prefill(sel, sk)[0][0]), n


@pytest.mark.parametrize("heads,block,nb", [
    # two workgroups a compute unit: head pairs of 64-token blocks, single heads of 128-token blocks; the last
    # round full, nearly empty, and of one workgroup an XCD
    ((4, 1), 64, 256), ((4, 1), 64, 150), ((8, 4), 64, 66), ((3, 1), 128, 100), ((4, 4), 128, 66),
    # up to four: single heads of 64-token blocks
    ((5, 1), 64, 150), ((3, 1), 64, 256), ((1, 1), 64, 256),
    # the first grid beyond one workgroup a unit, dense grids on either side of 5/3 rounds, short walks
    ((2, 2), 128, 129), ((8, 2), 64, 212), ((8, 2), 64, 214), ((16, 4), 64, 31),
])
def test_resident_grids(heads, block, nb):
    """Grids that are resident as a whole with several workgroups to a compute unit, and those a little
    larger: every walk equals a call per query head (at most one workgroup a unit), bit for bit."""
    Hq, Hkv = heads
    say(f"[resident] heads={heads} block={block} nb={nb}")
    t = torch()
    L, G = nb * block, Hq // Hkv
    q, k, v = random_inputs(1, Hq, Hkv, L, 128, seed=nb, scale=1.5)
    run = Run.upload(B.Problem(1, Hq, Hkv, L, 128, block, block // 8), q, k, v)
    rng = np.random.default_rng(nb)
    mask = (np.tril(rng.random((1, Hkv, nb, nb)) < 0.2) | np.eye(nb, dtype=bool)).astype(np.uint8)
    order = np.full((1, Hkv, nb, nb), -1, np.int32)
    for g, i in np.ndindex(Hkv, nb):
        at = rng.permutation(np.flatnonzero(mask[0, g, i]))
        order[0, g, i, :len(at)] = at
    dm, do, dc = dev(mask), dev(order), dev(mask.sum(-1).astype(np.int32))
    sk = B.skip(B.SKIP_ROWMAX, L * math.exp(-1.0))
    dense, masked = run.dense(), t.full_like(run.q, 0x7BCD)
    B.cosa_masked_attention(run.problem, run.q, run.k, run.v, dm, masked)
    lists = [run.osk(do, dc, s) for s in (None, sk)]
    for h in range(Hq):
        g = h // G
        one = Run(B.Problem(1, 1, 1, L, 128, block, block // 8), run.q[:, h].contiguous(),
                  run.k[:, g].contiguous(), run.v[:, g].contiguous())
        assert t.equal(dense[:, h], one.dense()[:, 0]), h
        o = t.full_like(dense[:, :1], 0x7BCD)
        B.cosa_masked_attention(one.problem, one.q, one.k, one.v, dm[:, g].contiguous(), o)
        assert t.equal(masked[:, h], o[:, 0]), h
        for s, got in zip((None, sk), lists):
            ref = one.osk(do[:, g].contiguous(), dc[:, g].contiguous(), s)
            assert all(t.equal(x[:, h], y[:, 0]) for x, y in zip(got, ref)), h
